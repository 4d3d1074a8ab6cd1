"""Recorded launches and eager calls that outgrow the workspace they were recorded with: a replay has to find its own memory,
with nothing in it that an eager call or another stream put there.  Whole numbers: exact."""
import numpy as np
import pytest
import torch

from paper_1811_09736_amd import workloads

pytestmark = pytest.mark.gpu

# the scan that is recorded; an array whose sums publish one per tile of 8192 elements; one whose moments publish two per range of
# four tiles of 6144, more than twice as many
N, LARGE, HUGE = (1 << 20) + 8192 * 5, 1 << 24, 72 << 20
SUMS, MOMENTS = LARGE // 8192, 2 * (HUGE // (4 * 6144))
assert 1024 < SUMS <= 2048 < MOMENTS


@pytest.fixture(scope="module")
def tcr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1811_09736_amd import binding
    binding.set_variant("reset")
    binding.tuning_import("")
    yield binding
    binding.check_device_flags()


@pytest.fixture(scope="module")
def large(oracle):
    x = workloads.make_input(LARGE, "int1", 5)
    off = workloads.make_offsets(LARGE, "few7", 2).view(np.int64)
    return (torch.from_numpy(x).cuda(), torch.from_numpy(off).cuda(), oracle.irregular_reduce(x, off))


@pytest.fixture(scope="module")
def huge():
    # a one in eight zeros: moments of any segment are whole numbers below 2^24
    x = torch.zeros(HUGE, dtype=torch.float16, device="cuda")
    x[::8] = 1.0
    return x, torch.tensor([0, 24, 1 << 25, HUGE], device="cuda"), np.array([3.0, (1 << 22) - 3, (HUGE - (1 << 25)) / 8])


def same(t, want):
    return np.array_equal(t.cpu().numpy().astype(np.float64), want)


@pytest.mark.parametrize("again", [False, True])
def test_eager_reductions_outgrow_the_table_of_a_recorded_scan(tcr, oracle, large, huge, again):
    xl, od, sums = large
    xh, oh, counts = huge
    inputs = [workloads.make_input(N, "int4", (31, k)) for k in range(3)]
    refs = [oracle.scan(h) for h in inputs]
    x = torch.from_numpy(inputs[0]).cuda()
    out, second = (torch.empty(N, dtype=torch.float32, device="cuda") for _ in range(2))
    side, other = torch.cuda.Stream(), torch.cuda.Stream()

    def record(dst):
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            tcr.scan(x, out=dst)
        return graph

    def replay(graph, dst, k):
        x.copy_(torch.from_numpy(inputs[k]).cuda())
        dst.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert same(dst, refs[k])

    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        tcr.scan(x, out=out)
    torch.cuda.synchronize()
    graph = record(out)
    for k in (1, 2):
        replay(graph, out, k)
    with torch.cuda.stream(side):                              # SUMS, then MOMENTS: two larger tables
        assert same(tcr.irregular_reduce(xl, od), sums)
        a, q = tcr.irregular_moments(xh, oh)
    torch.cuda.synchronize()
    assert same(a, counts) and same(q, counts)
    later = record(second) if again else None                  # the new table is recorded, too
    for k in (0, 1, 2, 0):
        replay(graph, out, k)
        with torch.cuda.stream(other):                         # a stream that could be handed the outgrown table
            assert same(tcr.scan(x), refs[k])
        with torch.cuda.stream(side):
            assert same(tcr.scan(x), refs[k])
            assert same(tcr.irregular_reduce(xl, od), sums)
        torch.cuda.synchronize()
        if again:
            replay(later, second, (k + 1) % 3)
    tcr.check_device_flags(side)
    torch.cuda.synchronize()
    tcr.release_stream(other)


def test_a_scan_and_moments_outgrow_tables_with_recorded_scans(tcr, oracle, huge):
    n = 1 << 18
    side = torch.cuda.Stream()
    x = torch.from_numpy(workloads.make_input(n, "int4", 3)).cuda()
    big = torch.ones((1 << 25) + 100003, dtype=torch.float16, device="cuda")
    xh, oh, counts = huge

    def nothing():
        return True

    def scan():                                                # 1028 tiles
        return float(tcr.scan(big)[(1 << 24) - 1]) == float(1 << 24)

    def moments():                                             # MOMENTS sums
        a, q = tcr.irregular_moments(xh, oh)
        return same(a, counts) and same(q, counts)

    outs, graphs = [], []
    torch.cuda.synchronize()
    for call in (nothing, scan, moments):
        with torch.cuda.stream(side):
            assert call()
            tcr.scan(x)
        torch.cuda.synchronize()
        outs.append(torch.empty(n, dtype=torch.float32, device="cuda"))
        graphs.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(graphs[-1], stream=side):
            tcr.scan(x, out=outs[-1])
    for k in range(4):
        h = workloads.make_input(n, "int4", (4, k))
        x.copy_(torch.from_numpy(h).cuda())
        for o in outs:
            o.fill_(float("nan"))
        torch.cuda.synchronize()
        for g in graphs:
            g.replay()
        torch.cuda.synchronize()
        want = oracle.scan(h)
        assert all(same(o, want) for o in outs)
        with torch.cuda.stream(side):
            assert moments() and scan()
        torch.cuda.synchronize()
    tcr.check_device_flags(side)


def test_eager_calls_outgrow_the_partials_of_recorded_reductions(tcr, oracle):
    # the replays' partials stay theirs: neither handed back to the allocator nor to the later call
    n, seg = 1 << 24, 1 << 18
    side = torch.cuda.Stream()
    x = torch.from_numpy(workloads.make_input(n, "int1", 8)).cuda()
    off = torch.from_numpy(workloads.make_offsets(n, "lognormal256", 8).view(np.int64)).cuda()
    total = torch.empty(1, dtype=torch.float32, device="cuda")
    segs = torch.empty(n // seg, dtype=torch.float32, device="cuda")
    irregular = torch.empty(off.numel() - 1, dtype=torch.float32, device="cuda")
    outs = (total, segs, irregular)

    def calls():
        tcr.reduce(x, out=total)                               # 4096 partials, added by a second kernel
        tcr.segmented_reduce(x, seg, out=segs)
        tcr.irregular_reduce(x, off, out=irregular)            # look-up tables and tile sums

    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        calls()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        calls()
    big = torch.zeros((1 << 26) + 1, dtype=torch.float16, device="cuda")
    for k in range(3):
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            assert float(tcr.reduce(big[1:])) == 0.0           # 8192 tiles of an unaligned array
            assert not torch.any(tcr.segmented_reduce(big[:1 << 26], seg))
        torch.cuda.synchronize()
        taken = torch.full((1 << 20,), 3.0, device="cuda")     # whoever gets memory that was freed
        h = workloads.make_input(n, "int1", (9, k))
        x.copy_(torch.from_numpy(h).cuda())
        for o in outs:
            o.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert float(total) == oracle.reduce(h)
        assert same(segs, oracle.segmented_reduce(h, seg))
        assert same(irregular, oracle.irregular_reduce(h, off.cpu().numpy()))
        assert torch.all(taken == 3.0)
