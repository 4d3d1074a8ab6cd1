"""Irregular scans of arrays of more than 2^24 elements, whose tiles find their entries with a search that starts where
they are likely to be (and of smaller ones, which search the whole array): tiles whose entries the search's last round has read or not, entries far from their share, segments
that start many tiles in front; and the zeros outside the segments where the look-up kernel of the largest arrays writes
them.  Whole numbers: exact."""
import numpy as np
import pytest
import torch

from paper_1811_09736_amd import workloads

pytestmark = pytest.mark.gpu

TILE = 8192
HELD = (12 << 20) + 3 * TILE + 13               # all workgroups at once: the other search
BEYOND = (1 << 24) + 5 * TILE + 3               # workgroups that follow each other


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


@pytest.fixture(scope="module")
def arrays():
    base = workloads.make_input(BEYOND + 8, "int1", 11)
    return base, torch.from_numpy(base).cuda()


def check(tcr, oracle, x, xd, off, modes=(0,)):
    off = np.asarray(off, dtype=np.int64)
    od = torch.from_numpy(off).cuda()
    for flags in modes:
        want = oracle.irregular_scan_exclusive(x, off) if flags & tcr.SCAN_EXCLUSIVE else oracle.irregular_scan(x, off)
        assert np.max(np.abs(want)) <= (2048 if flags & tcr.OUT_F16 else 1 << 24)
        got = tcr.irregular_scan_ex(xd, od, flags) if flags else tcr.irregular_scan(xd, od)
        assert np.array_equal(got.cpu().numpy().astype(np.float64), want)         # (0 outside the segments)


# the search's last round reads 256 entries, of which the tile's own are marked at once
@pytest.mark.parametrize("n", [HELD, BEYOND])
@pytest.mark.parametrize("per_tile", [1, 3, 127, 200, 254, 255, 256, 257, 300, 512, 767, 768, 769, 1500])
def test_entries_per_tile(tcr, oracle, arrays, n, per_tile):
    shift = per_tile % 3
    x, xd = arrays[0][shift:shift + n].copy(), arrays[1][shift:shift + n]
    ends = np.arange(0, n, TILE)[:, None] + np.round(np.linspace(0, TILE, per_tile, endpoint=False)).astype(np.int64)[None, :]
    cuts = np.unique(np.minimum(ends.ravel(), n))
    check(tcr, oracle, x, xd, np.concatenate([cuts[(cuts > 700) & (cuts < n - 9)], [n - 9]]), (0, 1, 2, 3) if per_tile in (3, 257) else (0,))


@pytest.mark.parametrize("n", [HELD, BEYOND])
def test_entries_far_from_their_share(tcr, oracle, arrays, n):
    x, xd = arrays[0][:n].copy(), arrays[1][:n]
    few = np.arange(0, 60000, dtype=np.int64)
    check(tcr, oracle, x, xd, np.concatenate([few, [n]]))
    check(tcr, oracle, x, xd, np.concatenate([[3], n - 60000 + few, [n]]))
    check(tcr, oracle, x, xd, np.concatenate([np.zeros(30000, np.int64), np.full(30000, n // 2 + 1), [n - 9]]))
    check(tcr, oracle, x, xd, np.concatenate([np.full(100000, 2 * TILE), [n]]))


@pytest.mark.parametrize("recipe", ["uniform16", "lognormal256", "few7"])
def test_recipes(tcr, oracle, arrays, recipe):
    for n in (HELD, BEYOND):
        x, xd = arrays[0][:n].copy(), arrays[1][:n]
        check(tcr, oracle, x, xd, workloads.make_offsets(n - 4000, recipe, 3).view(np.int64) + 2000, (0, 1))


@pytest.mark.parametrize("flags", [0, 3])
def test_zeros_outside_the_segments_of_a_large_array(tcr, oracle, flags):
    n = (5 << 23) + 77                           # chained tiles: seven long segments
    x = workloads.make_input(n, "int1", 2)
    xd = torch.from_numpy(x).cuda()
    for lo, hi in ((0, n), (5, n), (100003, n - 70001), (n // 2, n // 2 + 9), (0, 7)):
        off = np.sort(np.random.default_rng(lo).integers(lo, hi, 8, endpoint=True))
        off[0], off[-1] = lo, hi
        od = torch.from_numpy(off).cuda()
        torch.full((n,), float("nan"), device="cuda")                              # (what the next allocation may hold)
        got = tcr.irregular_scan_ex(xd, od, flags) if flags else tcr.irregular_scan(xd, od)
        got = got.cpu().numpy().astype(np.float64)
        want = oracle.irregular_scan_exclusive(x, off) if flags else oracle.irregular_scan(x, off)
        assert not np.any(got[:lo]) and not np.any(got[hi:])
        if flags == 0 or np.max(np.abs(want)) <= 2048:
            assert np.array_equal(got[lo:hi], want[lo:hi])


# the same in arrays that are not 16-byte aligned, with something in front of the results and behind them
@pytest.mark.parametrize("flags", [0, 2])
@pytest.mark.parametrize("shift", [1, 6])
def test_zeros_outside_the_segments_of_an_unaligned_large_array(tcr, oracle, shift, flags):
    n = (5 << 23) + 77
    base = workloads.make_input(n + 8, "int1", 2)
    x = base[shift:shift + n].copy()
    xd = torch.from_numpy(base).cuda()
    dtype = torch.float16 if flags else torch.float32
    for lo, hi in ((0, n), (5, n), (100003, n - 70001), (n // 2, n // 2 + 9), (0, 7)):
        off = np.sort(np.random.default_rng(lo + 1).integers(lo, hi, 8, endpoint=True))
        off[0], off[-1] = lo, hi
        od = torch.from_numpy(off).cuda()
        out = torch.full((n + 8,), float("nan"), dtype=dtype, device="cuda")
        st = tcr.raw().tcr_irregular_scan_filled(xd[shift:].data_ptr(), od.data_ptr(), out[shift:].data_ptr(), n, 7, flags,
                                                 int(torch.cuda.current_stream().cuda_stream))
        assert st == tcr.OK
        got = out.cpu().numpy()
        want = np.zeros(n)
        want[lo:hi] = oracle.irregular_scan(x, off)[lo:hi]
        assert np.array_equal(got[shift:shift + n], want.astype(got.dtype))
        assert np.all(np.isnan(got[:shift])) and np.all(np.isnan(got[shift + n:]))


# A float32 rounding is off by at most half a unit of the last place, evenly spread: 2^-24 * sqrt(1/3) of the power of two below
# the value, rms; relative to values spread evenly over their octave 2^-24 * sqrt(1/3) * sqrt(1/2).  A result of a long segment
# takes no more than six of its own size (wavefront sum 2 to 3, with the sums of the wavefronts in front, with the element's
# place, and what the sums of the tiles bring along); eight more would come from a lane that walks its elements on top of it.
@pytest.mark.parametrize("n,nseg,seg_len", [((1 << 20) * 24, 7, 0), ((1 << 20) * 20 + 77, 40, 0), ((1 << 20) * 24, 0, 100003)])
def test_roundings_of_long_sums(tcr, n, nseg, seg_len):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    if seg_len:
        n -= n % seg_len
        off = torch.arange(0, n + 1, seg_len, device="cuda")
    else:
        off = torch.floor(torch.linspace(0, 1, nseg + 1, device="cuda", dtype=torch.float64) ** 1.2 * n).long()
    x = torch.rand(n, generator=gen, device="cuda").half()
    got = (tcr.segmented_scan(x, seg_len) if seg_len else tcr.irregular_scan(x, off)).double()
    sums = torch.cat([torch.zeros(1, device="cuda", dtype=torch.float64), torch.cumsum(x.double(), 0)])
    want = sums[1:] - torch.repeat_interleave(sums[off[:-1]], off[1:] - off[:-1])
    error = ((got - want).pow(2).sum() / want.pow(2).sum()).sqrt().item()
    assert error <= 2.0 ** -24 * (6 / 3 / 2) ** 0.5, error
