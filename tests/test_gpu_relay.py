"""Scans whose carries one workgroup hands to all others: every mode, either kind of tile, sizes at the edges of tiles, of groups of 64 tiles
and of the dispatch, tiles that help themselves, short buffers and recorded launches, against the oracle."""
import numpy as np
import pytest
import torch

from paper_1811_09736_amd import workloads

pytestmark = pytest.mark.gpu

TILE, GROUP = 8192, 64 * 8192
HELD = 1 << 24                                  # up to here other forms take most calls (256 compute units)


@pytest.fixture(scope="module")
def tcr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1811_09736_amd import binding
    binding.set_variant("reset")
    binding.tuning_import("")
    yield binding
    binding.set_variant("reset")
    binding.set_workspace(None)
    binding.check_device_flags()


def regular(tcr, oracle, n, seg, flags, seed=5):
    n -= n % seg
    x = workloads.make_input(n, "int1", seed)
    want = oracle.segmented_scan(x, seg)
    if flags & 1:
        want = want - x.astype(np.float64)
    xd = torch.from_numpy(x).cuda()
    got = tcr.segmented_scan_ex(xd, seg, flags)
    assert got.dtype == (torch.float16 if flags & 2 else torch.float32)
    if flags & 2:                               # (the sums are exact, so each is rounded once)
        want = want.astype(np.float16).astype(np.float64)
    assert np.array_equal(got.cpu().numpy().astype(np.float64), want), (n, seg, flags)
    return xd


# one segment: beyond the tile, the group and the held array by one element, by a group of 8 and by none
@pytest.mark.parametrize("n", [HELD + 1, HELD + TILE, 33 * GROUP - 8, 33 * GROUP, 33 * GROUP + 1, (1 << 23) + 8, 11 << 20, (11 << 20) + 8])
@pytest.mark.parametrize("flags", [0, 1])
def test_one_segment(tcr, oracle, n, flags):
    regular(tcr, oracle, n, n, flags)


# segments in tiles of their own (the last one full, of eight elements, nearly full) and in tiles of the array
@pytest.mark.parametrize("seg", [32768, 65536, 65544, 73728 - 8, 1 << 20, 50003, 1048577, 6151, 8191])
@pytest.mark.parametrize("flags", [0, 1])
def test_segments(tcr, oracle, seg, flags):
    regular(tcr, oracle, (15 << 22) + 3 * GROUP // 2, seg, flags)


@pytest.mark.parametrize("seg", [2049, 4099, 50003, 65536, 1048577])
def test_binary16_results(tcr, oracle, seg):
    regular(tcr, oracle, (15 << 22) + GROUP + TILE, seg, 3)


def irregular(tcr, oracle, n, off, flags, shift=0):
    x = workloads.make_input(n + shift, "int1", 7)[shift:]
    xd = torch.from_numpy(np.concatenate([np.zeros(shift, np.float16), x])).cuda()[shift:]
    want = oracle.irregular_scan_exclusive(x, off) if flags & 1 else oracle.irregular_scan(x, off)
    got = tcr.irregular_scan_ex(xd, torch.from_numpy(off).cuda(), flags).cpu().numpy().astype(np.float64)
    lo, hi = int(off[0]), int(off[-1])
    assert not got[:lo].any() and not got[hi:].any()
    assert np.array_equal(got[lo:hi], want[lo:hi])


# starts on, next to and far from the edges of tiles and groups; elements in no segment on either side; an array that starts off a boundary
@pytest.mark.parametrize("n", [HELD + 9, 33 * GROUP + 5])
@pytest.mark.parametrize("shift", [0, 3])
@pytest.mark.parametrize("flags", [0, 1])
def test_irregular_edges(tcr, oracle, n, shift, flags):
    at = [7, 7, TILE - 1, TILE, 5 * TILE, 5 * TILE + 1, 9 * TILE - 2048, 20 * TILE - 2049, GROUP - 1, 2 * GROUP, 2 * GROUP, 3 * GROUP + 1, 30 * GROUP, n - 70000, n - 5]
    irregular(tcr, oracle, n, np.array(at, dtype=np.int64), flags, shift)


@pytest.mark.parametrize("recipe", ["uniform16", "lognormal256", "few7"])
def test_irregular_mixes(tcr, oracle, recipe):
    n = 3 * HELD // 2 + 1
    irregular(tcr, oracle, n, workloads.make_offsets(n, recipe, 3).view(np.int64), 0)


# no tile waits: each finds out itself, from sums that are there and elements where they are not
def test_tiles_that_help_themselves(tcr, oracle):
    tcr.set_variant("scan_wait", "none")
    try:
        regular(tcr, oracle, HELD + TILE + 3, HELD + TILE + 3, 0)
        regular(tcr, oracle, HELD + GROUP, 65536, 1)
        regular(tcr, oracle, HELD + GROUP, 100003, 0)
        n = HELD + 4099
        irregular(tcr, oracle, n, workloads.make_offsets(n, "few7", 3).view(np.int64), 0, 5)
        irregular(tcr, oracle, n, workloads.make_offsets(n, "lognormal256", 3).view(np.int64), 1)
    finally:
        tcr.set_variant("reset")


# (a caller's buffer one step short of two words per tile, and of the size that is said to do)
@pytest.mark.parametrize("seg", [0, 65536, 100003])
def test_short_buffer(tcr, oracle, seg):
    n = HELD + GROUP
    for size in (256 + 16 * (2 * 33 * 64 - 32), tcr.workspace_bytes(tcr.OP_SEGMENTED_SCAN, n - n % (seg or n), seg or n)):
        tcr.set_workspace(torch.full((size,), 0x5A, dtype=torch.uint8, device="cuda"))
        try:
            regular(tcr, oracle, n, seg or n, 0)
        finally:
            tcr.set_workspace(None)


def test_recorded(tcr, oracle):
    n = HELD + 2 * TILE + 8
    x = torch.from_numpy(workloads.make_input(n, "int1", 5)).cuda()
    off = torch.from_numpy(workloads.make_offsets(n, "lognormal256", 3).view(np.int64)).cuda()
    out, rows = torch.empty(n, device="cuda"), torch.empty(n, device="cuda")
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        tcr.scan(x, out)
        tcr.irregular_scan(x, off, rows)
    stream.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        tcr.scan(x, out)
        tcr.irregular_scan(x, off, rows)
    for turn in range(3):
        x.copy_(torch.from_numpy(workloads.make_input(n, "int1", 10 + turn)))
        out.zero_()
        rows.zero_()
        graph.replay()
        torch.cuda.synchronize()
        want, want_rows = tcr.scan(x), tcr.irregular_scan(x, off)
        assert torch.equal(out, want) and torch.equal(rows, want_rows), turn
        with torch.cuda.stream(stream):
            again = tcr.scan(x)
        stream.synchronize()
        assert torch.equal(again, want)
    assert np.array_equal(out.cpu().numpy().astype(np.float64), oracle.scan(x.cpu().numpy()))


# Rounding against 64 bits: a result adds up its tile (at most 5 + 4 + 5 + 6 levels of additions of parts of one sum) and one carry, itself a
# binary32 tree of 6 levels over tiles added to a binary64 sum: no more than 30 roundings of 2^-24 whatever the size, of values that
# grow with the sum; non-negative elements.
@pytest.mark.parametrize("call", ["scan", "seven", "rows"])
def test_rounding(tcr, call):
    n = 3 << 24
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    x = torch.rand(n, generator=gen, device="cuda").half()
    sums = torch.cumsum(x.double(), 0)
    if call == "scan":
        got, want = tcr.scan(x), sums
    elif call == "rows":
        m = n - n % 1000003
        got, want = tcr.segmented_scan(x[:m], 1000003), torch.cumsum(x[:m].double().view(-1, 1000003), 1).view(-1)
    else:
        off = torch.from_numpy(workloads.make_offsets(n, "few7", 5).view(np.int64)).cuda()
        got = tcr.irregular_scan(x, off)
        want = sums - torch.repeat_interleave(torch.cat([sums.new_zeros(1), sums])[off[:-1]], off[1:] - off[:-1])
    assert ((got.double() - want).abs() <= 30 * 2.0 ** -24 * want).all()
