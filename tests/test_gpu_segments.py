"""Irregular sums and moments by workgroups that walk ranges of tiles (most arrays of more than 2^23 elements): numbers of segments
per tile around the limits between the ways in which a tile is shared out, batches of entries that end with a tile or
just behind it, segments around the edges of groups, tiles and ranges, parts added from elements and from published sums
(waited for or not), entries far from where their number alone would put them.  Whole numbers: exact; fractional ones the
same from run to run and within the rounding of the additions."""
import numpy as np
import pytest
import torch

from paper_1811_09736_amd import workloads

pytestmark = pytest.mark.gpu

TILE = 6144
N = (21 << 19) + 3 * TILE + 5                   # two tiles per range; moments of any segments, sums of up to 383 elements each
BIG = (5 << 22) + 4099                          # four tiles per range; sums of any segments as well


@pytest.fixture(scope="module")
def tcr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1811_09736_amd import binding
    binding.set_variant("reset")
    binding.tuning_import("")
    yield binding
    binding.set_variant("reset")
    binding.check_device_flags()


def check(tcr, oracle, x, xd, off):
    off = np.asarray(off, dtype=np.int64)
    od = torch.from_numpy(off).cuda()
    a, q = tcr.irregular_moments(xd, od)
    wa, wq = oracle.irregular_moments(x, off)
    assert np.max(wq) < 2 ** 24
    assert np.array_equal(tcr.irregular_reduce(xd, od).cpu().numpy().astype(np.float64), wa)
    assert np.array_equal(a.cpu().numpy().astype(np.float64), wa) and np.array_equal(q.cpu().numpy().astype(np.float64), wq)


@pytest.mark.parametrize("shift", [0, 3])
@pytest.mark.parametrize("per_tile", [7, 8, 9, 63, 64, 65, 255, 256, 257, 511, 512, 513, 1024, 2000])
def test_segments_per_tile(tcr, oracle, per_tile, shift):
    base = workloads.make_input(N + 8, "int1", per_tile)
    x, xd = base[shift:shift + N].copy(), torch.from_numpy(base).cuda()[shift:shift + N]
    ends = np.arange(0, N, TILE)[:, None] + np.round(np.linspace(0, TILE, per_tile, endpoint=False)).astype(np.int64)[None, :]
    check(tcr, oracle, x, xd, np.concatenate([np.unique(np.minimum(ends.ravel(), N)), [N]]))       # one on every tile's start
    jitter = np.random.default_rng(per_tile).integers(0, max(TILE // per_tile, 2), ends.shape)
    check(tcr, oracle, x, xd, np.concatenate([[0], np.sort(np.minimum((ends + jitter).ravel(), N)), [N, N, N]]))


# one tile per range: segments of 14 to 27 elements, and moments of one or two, from 2^22 elements on
@pytest.mark.parametrize("length", [1, 2, 15, 27])
def test_one_tile_per_range(tcr, oracle, length):
    n = (1 << 22) + 3 * TILE + 5
    x = workloads.make_input(n, "int1", length)
    off = np.sort(np.random.default_rng(length).integers(0, n, n // length))
    check(tcr, oracle, x, torch.from_numpy(x).cuda(), np.concatenate([[0], off, [n]]))


@pytest.mark.parametrize("wait", ["bounded", "none"])
@pytest.mark.parametrize("n", [N, BIG])
def test_parts_in_front_of_a_range(tcr, oracle, n, wait):
    x = workloads.make_input(n, "int1", 7)
    xd = torch.from_numpy(x).cuda()
    tcr.set_variant("scan_wait", wait)
    try:
        for reach in (1, 7, 8, 511, TILE - 1, TILE, TILE + 1, 5 * TILE, 300 * TILE + 9):
            off = [0]
            for edge in range(302 * TILE, n - TILE, 311 * TILE):                # a segment from `reach` in front of a tile's start
                off += sorted({max(edge - reach, off[-1]), edge + 5})
            # (empty segments in front of, between and behind them bring the mean length down to what sums take this way)
            check(tcr, oracle, x, xd, off + [n] * (n // 64))
    finally:
        tcr.set_variant("reset")


def test_entries_far_from_their_share(tcr, oracle):
    x = workloads.make_input(N, "int1", 5)
    xd = torch.from_numpy(x).cuda()
    few = np.arange(0, 40000, dtype=np.int64)
    check(tcr, oracle, x, xd, np.concatenate([few, [N]]))                        # all in the first tiles
    check(tcr, oracle, x, xd, np.concatenate([[3], N - 40000 + few, [N]]))       # all in the last ones
    check(tcr, oracle, x, xd, np.concatenate([np.zeros(30000, np.int64), np.full(30000, N // 2 + 1), [N - 9]]))
    check(tcr, oracle, x, xd, np.concatenate([np.full(100000, 2 * TILE), [N]]))  # hundreds of batches on one edge


@pytest.mark.parametrize("recipe", ["uniform16", "lognormal256", "few7"])
def test_rounding_and_repetition(tcr, oracle, recipe):
    n = (5 << 22) + 77                           # (every mean length takes this way here)
    x = workloads.make_input(n, "normal", 3)
    xd = torch.from_numpy(x).cuda()
    off = workloads.make_offsets(n, recipe, 3).view(np.int64)
    od = torch.from_numpy(off).cuda()
    results = []
    for wait in ("bounded", "none", "bounded"):
        tcr.set_variant("scan_wait", wait)
        results.append((tcr.irregular_reduce(xd, od), *tcr.irregular_moments(xd, od)))
    tcr.set_variant("reset")
    for r in results[1:]:
        assert all(torch.equal(a, b) for a, b in zip(r, results[0]))
    # additions in a row: 8 in a group, 12 groups of a lane, 6 across lanes, 4 wavefronts, 4 tiles; then 16 published sums in a
    # lane, 6 across lanes, 4 wavefronts and the one that joins the parts
    bound = 64 * 2.0 ** -24 * oracle.irregular_reduce(np.abs(x), off) + 1e-30
    for got in results[0][:2]:
        assert np.all(np.abs(got.cpu().numpy().astype(np.float64) - oracle.irregular_reduce(x, off)) <= bound)
    want = oracle.irregular_moments(x, off)[1]
    assert np.all(np.abs(results[0][2].cpu().numpy().astype(np.float64) - want) <= 64 * 2.0 ** -24 * want + 1e-30)


def exact_moments(x, off):
    """Sums and sums of squares of non-empty segments in 64 bits, each from its own elements alone."""
    starts, ends = off[:-1], off[1:]
    with np.errstate(invalid="ignore"):
        v = np.append(x.astype(np.float64), 0.0)
        cut = np.stack([starts, ends], 1).ravel()
        return np.add.reduceat(v, cut)[::2], np.add.reduceat(v * v, cut)[::2]


def check_special(tcr, x, off):
    xd, od = torch.from_numpy(x).cuda(), torch.from_numpy(off).cuda()
    wa, wq = exact_moments(x, off)
    a, q = tcr.irregular_moments(xd, od)
    for got, want in ((tcr.irregular_reduce(xd, od), wa), (a, wa), (q, wq)):
        assert np.array_equal(got.cpu().numpy().astype(np.float64), want, equal_nan=True)


# lengths of a tile's segments in each of the ways in which it is shared out: a wavefront, eight lanes and one lane each (and longer
# ones among them by eight lanes and by the whole wavefront)
MIXES = {"few": (1500, 9001), "some": (100, 500), "many": (9, 40), "mixed": (2, 3, 5, 130, 700, 11)}


def cuts(mix, n, first):
    lengths = np.random.default_rng(len(mix)).choice(MIXES[mix], n // min(MIXES[mix]))
    off = first + np.concatenate([[0], np.cumsum(lengths)])
    return off[off <= n - 5].astype(np.int64)


@pytest.mark.parametrize("mix", list(MIXES))
def test_subnormal_elements(tcr, mix):
    # every other segment holds binary16 subnormals, k * 2^-24: the sums are whole multiples of 2^-24 (2^-48) below 2^24 of them
    off = cuts(mix, BIG, 3)
    x = np.ones(BIG, dtype=np.float16)
    rng = np.random.default_rng(2)
    small = (rng.integers(-6, 7, BIG) * 2.0 ** -24).astype(np.float16)
    which = np.repeat(np.arange(off.size - 1) % 2 == 0, np.diff(off))
    x[off[0]:off[-1]][which] = small[off[0]:off[-1]][which]
    assert np.count_nonzero((x != 0) & (np.abs(x) < 2.0 ** -14)) > BIG // 4
    check_special(tcr, x, off)


@pytest.mark.parametrize("mix", list(MIXES))
def test_infinities_and_nan_stay_in_their_segments(tcr, mix):
    off = cuts(mix, BIG, 3)
    x = np.random.default_rng(3).integers(-2, 3, BIG).astype(np.float16)
    x[:off[0]] = np.nan                                        # (outside the segments)
    x[off[-1]:] = np.inf
    special = np.array([np.inf, -np.inf, np.nan], dtype=np.float16)
    hit = np.arange(1, off.size - 1, 3)                        # the neighbours on both sides stay finite
    x[off[hit]] = special[hit % 3]                             # its first element; its last one
    x[off[hit + 1] - 1] = special[(hit // 3) % 3]
    check_special(tcr, x, off)


def test_recorded_on_a_stream_whose_epochs_the_device_keeps(tcr, oracle):
    # a recorded scan leaves the stream's epochs to the device; ranges of tiles then run recorded and eagerly, with sums that other
    # ranges look up
    inputs = [workloads.make_input(BIG, "int1", (12, k)) for k in range(2)]
    off = np.concatenate([[5], np.sort(np.random.default_rng(3).integers(5, BIG // 2, BIG // 64)), [BIG // 2, BIG - 70001, BIG - 2]]).astype(np.int64)
    od = torch.from_numpy(off).cuda()
    x = torch.from_numpy(inputs[0]).cuda()
    scanned = torch.empty(BIG, dtype=torch.float32, device="cuda")
    out = torch.empty(off.size - 1, dtype=torch.float32, device="cuda")
    side = torch.cuda.Stream()

    def calls():
        tcr.scan(x, out=scanned)
        tcr.irregular_reduce(x, od, out=out)
        return tcr.irregular_moments(x, od)

    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        calls()
    side.synchronize()
    for _ in range(2):                                            # the second recording finds them on the device
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            a, q = calls()
        for k in (1, 0, 1):
            x.copy_(torch.from_numpy(inputs[k]).cuda())
            for t in (scanned, out, a, q):
                t.fill_(float("nan"))
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            wa, wq = oracle.irregular_moments(inputs[k], off)
            for got, want in ((out, wa), (a, wa), (q, wq), (scanned, oracle.scan(inputs[k]))):
                assert np.array_equal(got.cpu().numpy().astype(np.float64), want)
            with torch.cuda.stream(side):
                eager = tcr.irregular_reduce(x, od)
            side.synchronize()
            assert torch.equal(eager, out)
    del graph
    tcr.check_device_flags(side)
    torch.cuda.synchronize()
    tcr.release_stream(side)
