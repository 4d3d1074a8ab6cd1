"""The sums that reach a tile of the irregular reduction from tiles in front of it: from the tile next to it, from further away
than one and than several steps of the finishing kernel; and the tiles that search the offsets themselves.  (Arrays of up to
4096 tiles, both moments 2048, run as one launch: the finishing kernel at the edges of its groups of tiles is in
test_gpu_finish_groups.py.)  Whole numbers: exact."""
import numpy as np
import pytest
import torch

from paper_1811_09736_amd import workloads

pytestmark = pytest.mark.gpu

TILE, GROUP, STEP = 8192, 256, 4096          # elements per tile; tiles per finishing workgroup and per further step


@pytest.fixture(scope="module")
def tcr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1811_09736_amd import binding
    binding.set_variant("reset")
    binding.tuning_import("")
    yield binding
    binding.check_device_flags()


def check(tcr, oracle, x, xd, off, moments=True):
    off = np.asarray(off, dtype=np.int64)
    od = torch.from_numpy(off).cuda()
    want = oracle.irregular_reduce(x, off)
    got = tcr.irregular_reduce(xd, od)
    assert np.array_equal(got.cpu().numpy().astype(np.float64), want)
    assert torch.equal(got, tcr.irregular_reduce(xd, od))        # the same from run to run
    if moments:
        a, q = tcr.irregular_moments(xd, od)
        wa, wq = oracle.irregular_moments(x, off)
        assert np.max(wq) < 2 ** 24
        assert np.array_equal(a.cpu().numpy().astype(np.float64), wa) and np.array_equal(q.cpu().numpy().astype(np.float64), wq)


@pytest.mark.parametrize("tiles", [1, 2, 3, GROUP - 1, GROUP, GROUP + 1, 2 * GROUP, 2 * GROUP + 3, 5 * GROUP + 7, 2048, 2049])
def test_one_long_segment_and_short_ones_around_it(tcr, oracle, tiles):
    n = tiles * TILE - 5
    x = workloads.make_input(n, "int1", tiles)                    # |x| <= 1: the sums of squares stay below 2^24
    xd = torch.from_numpy(x).cuda()
    for off in ([0, 5, n - 3, n], [0, n], [n // 2, n // 2 + 1, n], [0, 3, 3, n - TILE // 2, n - 9, n - 9]):
        check(tcr, oracle, x, xd, off)
    mid = (tiles // 2) * TILE
    check(tcr, oracle, x, xd, [0, mid, n])                       # an entry on the edge of a tile
    if mid:
        check(tcr, oracle, x, xd, [0, mid - 1, mid + 1, n])


def test_sums_from_more_than_one_step_away(tcr, oracle):
    tiles = GROUP + STEP + 300
    n = tiles * TILE
    x = workloads.make_input(n, "int1", 7)
    xd = torch.from_numpy(x).cuda()
    far = (tiles - 1) * TILE + 11
    for off in ([0, n], [3, far, far + 2, n], [0, TILE * 255, far, n], [0, TILE * (GROUP + 1) - 1, far, n - 1, n]):
        check(tcr, oracle, x, xd, off, moments=False)


@pytest.mark.parametrize("shift", [0, 1, 7])
@pytest.mark.parametrize("recipe", ["uniform1", "uniform16", "uniform3000", "lognormal256", "few4"])
def test_searched_and_looked_up_ranges_agree(tcr, oracle, recipe, shift):
    # tile shape 1 of the tuning table keeps the look-up kernel in front
    n = 37 * TILE + 1234
    base = workloads.make_input(n + 8, "int1", 3)
    x, xd = base[shift:shift + n].copy(), torch.from_numpy(base).cuda()[shift:shift + n]
    off = workloads.make_offsets(n - 100, recipe, 5).view(np.int64) + 50
    check(tcr, oracle, x, xd, off)
    try:
        tcr.tuning_import("irregular:0=1;")
        check(tcr, oracle, x, xd, off)
    finally:
        tcr.tuning_import("")


def test_recorded_and_on_a_caller_workspace(tcr, oracle):
    n = 40 * TILE + 77
    inputs = [workloads.make_input(n, "int1", (3, k)) for k in range(2)]
    off = workloads.make_offsets(n, "lognormal256", 2).view(np.int64)
    od = torch.from_numpy(off).cuda()
    x = torch.from_numpy(inputs[0]).cuda()
    out = torch.empty(off.size - 1, dtype=torch.float32, device="cuda")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        tcr.irregular_reduce(x, od, out=out)
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        tcr.irregular_reduce(x, od, out=out)
    for k in (1, 0, 1, 1):
        x.copy_(torch.from_numpy(inputs[k]).cuda())
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy().astype(np.float64), oracle.irregular_reduce(inputs[k], off))
        with torch.cuda.stream(side):
            again = tcr.irregular_reduce(x, od)
        side.synchronize()
        assert torch.equal(again, out)
    # arbitrary contents: until a call that chains tiles has cleared the buffer, the count in it means nothing
    want, moments = oracle.irregular_reduce(inputs[1], off), oracle.irregular_moments(inputs[1], off)
    need = max(tcr.workspace_bytes(tcr.OP_IRREGULAR_MOMENTS, n, 0), tcr.workspace_bytes(tcr.OP_IRREGULAR_SCAN, n, 0))
    buf = torch.full((need,), 0x77, dtype=torch.uint8, device="cuda")
    try:
        tcr.set_workspace(buf)
        for _ in range(3):
            assert np.array_equal(tcr.irregular_reduce(x, od).cpu().numpy().astype(np.float64), want)
            a, q = tcr.irregular_moments(x, od)
            assert np.array_equal(a.cpu().numpy().astype(np.float64), moments[0])
            assert np.array_equal(q.cpu().numpy().astype(np.float64), moments[1])
            assert np.array_equal(tcr.irregular_scan(x, od).cpu().numpy().astype(np.float64), oracle.irregular_scan(inputs[1], off))
    finally:
        torch.cuda.synchronize()
        tcr.set_workspace(None)
