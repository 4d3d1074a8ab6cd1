"""Irregular reductions over segments of thousands of tiles: eagerly, on a caller's workspace, and recorded, where the sums of 64 tiles
are combined first -- or not, on a workspace without room for the combined sums or with segments that are not as long.  Whole
numbers: exact."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

TILE = 8192


@pytest.fixture(scope="module")
def tcr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1811_09736_amd import binding
    binding.set_variant("reset")
    binding.tuning_import("")
    yield binding
    binding.set_workspace(None)
    binding.check_device_flags()


@pytest.fixture(scope="module")
def data():
    torch.manual_seed(6)
    x = torch.randint(0, 9, (12400 * TILE,), device="cuda", dtype=torch.int8) == 0       # a ninth ones: squares below 2^24, too
    x = x.to(torch.float16)
    x[::5] = -x[::5]
    return x, torch.cat([torch.zeros(1, device="cuda", dtype=torch.float64), torch.cumsum(x.double(), 0)]), torch.cat(
        [torch.zeros(1, device="cuda", dtype=torch.float64), torch.cumsum(x.double().abs(), 0)])


def check(tcr, data, shift, n, off):
    x, sums, squares = data
    off = torch.tensor(off, dtype=torch.int64, device="cuda")
    want, wq = (c[shift + off[1:]] - c[shift + off[:-1]] for c in (sums, squares))
    assert float(wq.max()) < 2 ** 24
    xd = x[shift:shift + n]
    for _ in range(2):
        a, q = tcr.irregular_moments(xd, off)
        assert torch.equal(tcr.irregular_reduce(xd, off).double(), want)
        assert torch.equal(a.double(), want) and torch.equal(q.double(), wq)


@pytest.mark.parametrize("tiles", [4096, 4097, 4097 + 63, 8192, 12288 + 64, 12400])      # ranges of tiles; unaligned regular ones: one launch, then far sums
def test_long_segments(tcr, data, tiles):
    n = tiles * TILE - 11
    mid = (tiles // 2) * TILE
    for off in ([0, n], [7, mid, n - 1], [0, mid - 1, mid + 1, n], [0, 64 * TILE, 64 * TILE + 3, n], [5, n - TILE + 3, n]):
        check(tcr, data, 0, n, off)
    check(tcr, data, 3, n, [0, n])
    x, sums, squares = data
    total, square = float(sums[5 + n] - sums[5]), float(squares[5 + n] - squares[5])
    a, q = tcr.segmented_moments(x[5:5 + n], n)                          # the whole of an unaligned array
    assert float(tcr.reduce(x[5:5 + n])) == float(a) == total and float(q) == square


def test_small_workspaces_and_graphs(tcr, data):
    tiles = 8200
    n = tiles * TILE
    words = 2 * (tiles + 1) + 3 * tiles                                  # both moments, without the combined sums
    need = tcr.workspace_bytes(tcr.OP_IRREGULAR_MOMENTS, n, 0)
    assert need >= 256 + 2 * 8 * (words + 2 * ((tiles + 63) // 64))
    try:
        for size in (need, 256 + 2 * ((8 * words + 255) // 256 * 256)):
            tcr.set_workspace(torch.full((size,), 0x55, dtype=torch.uint8, device="cuda"))
            check(tcr, data, 0, n, [0, n])
            torch.cuda.synchronize()
    finally:
        tcr.set_workspace(None)
    x, sums, _ = data
    xd, off = x[:n].clone(), torch.tensor([3, n], dtype=torch.int64, device="cuda")
    out = torch.empty(1, device="cuda")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        tcr.irregular_reduce(xd, off, out=out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        tcr.irregular_reduce(xd, off, out=out)
    for sign in (-1.0, 1.0, -1.0):
        xd.copy_(x[:n] * sign)
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert float(out) == sign * float(sums[n] - sums[3])


# recorded on a stream that nothing else has been recorded on, so with a look-up kernel in front and kernels behind: combined sums
# (one and two segments; a ragged last group), single ones (a hundred segments; no room for the combined sums)
@pytest.mark.parametrize("tiles,nseg,room", [(4097, 1, True), (8200, 2, True), (12400, 1, True), (8200, 100, True), (4100, 1, False), (8200, 2, False),
                                             (1600, 3, True)])
def test_recorded_sums_and_moments(tcr, data, tiles, nseg, room):
    x, sums, squares = data
    n = tiles * TILE - 11
    words = 2 * (tiles + 1) + 3 * tiles
    off = np.sort(np.random.default_rng(tiles).integers(0, n, nseg + 1, endpoint=True))
    off[0], off[-1] = 7, n - 3
    od = torch.from_numpy(off).cuda()
    want, wq = (c[od[1:]] - c[od[:-1]] for c in (sums, squares))
    xd = x[:n].clone()
    side = torch.cuda.Stream()
    out = torch.empty(nseg, device="cuda")
    torch.cuda.synchronize()
    if not room:
        tcr.set_workspace(torch.full((256 + 2 * ((8 * words + 255) // 256 * 256),), 0x55, dtype=torch.uint8, device="cuda"))
    try:
        with torch.cuda.stream(side):
            tcr.irregular_reduce(xd, od, out=out)
            tcr.irregular_moments(xd, od)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            tcr.irregular_reduce(xd, od, out=out)
            a, q = tcr.irregular_moments(xd, od)
        for sign in (-1.0, 1.0, -1.0):
            xd.copy_(x[:n] * sign)
            for t in (out, a, q):
                t.fill_(float("nan"))
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out.double(), sign * want) and torch.equal(a.double(), sign * want) and torch.equal(q.double(), wq)
            with torch.cuda.stream(side):
                eager = tcr.irregular_reduce(xd, od)
            side.synchronize()
            assert torch.equal(eager, out)
        del graph
    finally:
        torch.cuda.synchronize()
        tcr.set_workspace(None)
