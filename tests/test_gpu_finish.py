"""Reductions that finish in one launch: the workgroup that is done last adds up the partials, and the count of finished
workgroups serves the next launch, recorded or not.  Whole numbers: exact."""
import numpy as np
import pytest
import torch

from paper_1811_09736_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tcr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1811_09736_amd import binding
    binding.set_variant("reset")
    binding.tuning_import("")
    yield binding
    binding.set_workspace(None)
    binding.set_variant("reset")
    binding.check_device_flags()


# one wavefront, one workgroup with its last steps empty or ragged, the first and last partials, shares of 16384, 32768 and
# 65536 elements, and the first size of two kernels
FULL = [4096, 4097, 8191, 16 * 512 + 1, 65535, 65536, 65537, 131071, 131072, 131073, 16384 * 9 + 7, (1 << 21) - 1, (1 << 21) + 1,
        (1 << 22) + 8, (1 << 22) + 13, (1 << 23) - 3, 1 << 23, (1 << 23) + 1]


@pytest.mark.parametrize("n", FULL)
@pytest.mark.parametrize("form", ["mfma", "dpp"])
def test_full_reductions(tcr, oracle, n, form):
    x = workloads.make_input(n, "int4", n % 887)
    xd = torch.from_numpy(x).cuda()
    want = oracle.reduce(x)
    tcr.set_variant("formulation", form)
    try:
        for _ in range(3):
            assert float(tcr.reduce(xd).cpu()[0]) == want
    finally:
        tcr.set_variant("reset")


@pytest.mark.parametrize("nseg,seg", [(2, 1 << 18), (32, 1 << 18), (33, 1 << 18), (16, 1 << 19), (8, 1 << 20), (2, 131073), (16, 131073), (17, 131073),
                                      (32, 200001), (63, 131073), (3, 1000001), (1, 300001), (2, 262145)])
def test_long_segments(tcr, oracle, nseg, seg):
    x = workloads.make_input(nseg * seg, "int4", seg % 883)
    xd = torch.from_numpy(x).cuda()
    want = oracle.segmented_reduce(x, seg)
    wa, wq = oracle.segmented_moments(x, seg)
    assert np.max(wq) < 2 ** 24
    for _ in range(2):
        assert np.array_equal(tcr.segmented_reduce(xd, seg).cpu().numpy().astype(np.float64), want)
        a, q = tcr.segmented_moments(xd, seg)
        assert np.array_equal(a.cpu().numpy().astype(np.float64), wa) and np.array_equal(q.cpu().numpy().astype(np.float64), wq)


def test_the_same_from_run_to_run(tcr):
    x = torch.from_numpy(workloads.make_input(1 << 20, "uniform_pm1", 1)).cuda()
    first = tcr.reduce(x).clone()
    for _ in range(50):
        assert torch.equal(tcr.reduce(x), first)


def test_two_streams_at_once(tcr, oracle):
    xs = [workloads.make_input(1 << 21, "int4", k) for k in range(2)]
    xd = [torch.from_numpy(x).cuda() for x in xs]
    streams = [torch.cuda.Stream() for _ in range(2)]
    outs = [[torch.empty(1, dtype=torch.float32, device="cuda") for _ in range(40)] for _ in range(2)]
    torch.cuda.synchronize()
    for k in range(40):
        for i in range(2):
            tcr.reduce(xd[i], out=outs[i][k], stream=streams[i])
    torch.cuda.synchronize()
    for i in range(2):
        assert all(float(o) == oracle.reduce(xs[i]) for o in outs[i])
        tcr.release_stream(streams[i])


def test_recorded_and_replayed(tcr, oracle):
    inputs = [workloads.make_input(1 << 20, "int4", (9, k)) for k in range(3)]
    x = torch.from_numpy(inputs[0]).cuda()
    total = torch.empty(1, dtype=torch.float32, device="cuda")
    few = torch.empty(4, dtype=torch.float32, device="cuda")
    scan = torch.empty(1 << 20, dtype=torch.float32, device="cuda")
    side = torch.cuda.Stream()

    def calls():
        tcr.reduce(x, out=total)
        tcr.scan(x, out=scan)                                    # (the same workspace)
        tcr.segmented_reduce(x, 1 << 18, out=few)

    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        calls()
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        calls()
    for k in (1, 2, 0, 1, 2):
        x.copy_(torch.from_numpy(inputs[k]).cuda())
        for t in (total, few, scan):
            t.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        h = inputs[k]
        assert float(total) == oracle.reduce(h)
        assert np.array_equal(few.cpu().numpy().astype(np.float64), oracle.segmented_reduce(h, 1 << 18))
        assert np.array_equal(scan.cpu().numpy().astype(np.float64), oracle.scan(h))
        with torch.cuda.stream(side):
            assert float(tcr.reduce(x)) == oracle.reduce(h)       # eager in between, the same counter
    tcr.check_device_flags(side)


def test_caller_workspace_before_and_after_it_is_cleared(tcr, oracle):
    # arbitrary contents: until a call that chains tiles has cleared the buffer the count in it means nothing, and the
    # reductions take two kernels; afterwards one
    n = 1 << 20
    x = workloads.make_input(n, "int4", 21)
    xd = torch.from_numpy(x).cuda()
    buf = torch.full((tcr.workspace_bytes(tcr.OP_SCAN, n, n),), 0xA5, dtype=torch.uint8, device="cuda")
    try:
        tcr.set_workspace(buf)
        assert float(tcr.reduce(xd)) == oracle.reduce(x)
        assert np.array_equal(tcr.segmented_reduce(xd, 1 << 18).cpu().numpy().astype(np.float64), oracle.segmented_reduce(x, 1 << 18))
        assert np.array_equal(tcr.scan(xd).cpu().numpy().astype(np.float64), oracle.scan(x))
        for _ in range(3):
            assert float(tcr.reduce(xd)) == oracle.reduce(x)
            assert np.array_equal(tcr.segmented_reduce(xd, 1 << 18).cpu().numpy().astype(np.float64), oracle.segmented_reduce(x, 1 << 18))
    finally:
        torch.cuda.synchronize()
        tcr.set_workspace(None)


def test_a_buffer_of_the_smallest_size(tcr, oracle):
    # 64 partials: one per 65536 elements of 2^22 fit, the finer shares of an ordinary call do not
    x = workloads.make_input(1 << 22, "int4", 2)
    xd = torch.from_numpy(x).cuda()
    buf = torch.full((768,), 0x11, dtype=torch.uint8, device="cuda")
    try:
        tcr.set_workspace(buf)
        tcr.scan(xd[: 1 << 19])                                   # clears it
        for _ in range(2):
            assert np.array_equal(tcr.segmented_reduce(xd, 1 << 20).cpu().numpy().astype(np.float64), oracle.segmented_reduce(x, 1 << 20))
    finally:
        torch.cuda.synchronize()
        tcr.set_workspace(None)
