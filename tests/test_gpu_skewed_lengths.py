"""Irregular calls whose mean segment length says little about their segments: empty segments by the ten thousand on one
position, one segment that dominates the array.  Whole numbers: exact; and no form that is chosen by the mean length takes far
longer than the one that would have been chosen without it."""
import numpy as np
import pytest
import torch

from paper_1811_09736_amd import workloads

pytestmark = pytest.mark.gpu

TILE = 8192
HELD = (13 << 20) + 3 * TILE + 13               # all workgroups at once
BEYOND = (1 << 24) + 5 * TILE + 3               # workgroups of four wavefronts that follow each other


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


def milliseconds(call, calls=5):
    """The fastest of a few calls."""
    call()
    best = float("inf")
    for _ in range(calls):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        call()
        end.record()
        end.synchronize()
        best = min(best, start.elapsed_time(end))
    return best


# a run of empty segments is left behind by whole turns of 512 entries where the tile has seen more entries than it has elements
# and the run goes on for 64 turns: runs about that long, with entries in front of them and behind in the same tile that make the
# run start and end anywhere in a turn
@pytest.mark.parametrize("run", [8193, 40959, 42000, 90001])
@pytest.mark.parametrize("around", [0, 3, 300, 1777])
@pytest.mark.parametrize("n", [HELD, BEYOND])
def test_runs_of_empty_segments(tcr, oracle, n, around, run):
    x = workloads.make_input(n, "int1", 11)
    at = (n // 2) // TILE * TILE + 2 * around + 5
    off = np.concatenate([np.arange(0, at - around, 100), np.arange(at - around, at), np.full(run, at),
                          np.arange(at, at + around), np.arange(at + around, n, 100)])
    got = tcr.irregular_scan(torch.from_numpy(x).cuda(), torch.from_numpy(off).cuda())
    assert np.array_equal(got.cpu().numpy().astype(np.float64), oracle.irregular_scan(x, off))


@pytest.mark.parametrize("n", [HELD, BEYOND])
def test_time_with_a_million_empty_segments_on_one_position(tcr, n):
    x = torch.ones(n, dtype=torch.float16, device="cuda")
    ends = torch.arange(0, n, 16, device="cuda")
    off = torch.cat([ends[:ends.numel() // 2], ends[ends.numel() // 2].repeat(1 << 20), ends[ends.numel() // 2:]])
    took = milliseconds(lambda: tcr.irregular_scan(x, off))
    tcr.set_variant("irregular_scan", "single")
    chained = milliseconds(lambda: tcr.irregular_scan(x, off))
    tcr.set_variant("reset")
    assert took <= 1.2 * chained, (took, chained)


# The sums of the tiles in front are looked up 64 at a time, by four wavefronts in turn: long segments that start and end around the
# edges of tiles and of 64 tiles, waited for or added up again.
@pytest.mark.parametrize("wait", ["bounded", "none"])
@pytest.mark.parametrize("n", [HELD, BEYOND, 33 * 64 * TILE, 33 * 64 * TILE + 1])
def test_long_segments_around_64_tiles(tcr, oracle, n, wait):
    x = workloads.make_input(n, "int1", 13)
    xd = torch.from_numpy(x).cuda()
    group = 64 * TILE
    tcr.set_variant("scan_wait", wait)
    try:
        for start in (0, 1, group - TILE - 1, group - TILE, group - 9, group - 1, group, group + 1, group + TILE, 3 * group - 3 * TILE + 77):
            for end in ((start + group) // group * group + 5 * group + 7, n - 3):
                off = np.array([0, start, end, *range(end + 1, min(end + 100000, n), 999), n])
                od = torch.from_numpy(off).cuda()
                assert np.array_equal(tcr.irregular_scan(xd, od).cpu().numpy().astype(np.float64), oracle.irregular_scan(x, off))
        got = tcr.irregular_scan_ex(xd, od, tcr.SCAN_EXCLUSIVE).cpu().numpy().astype(np.float64)
        assert np.array_equal(got, oracle.irregular_scan_exclusive(x, off))
        every = np.concatenate([np.arange(0, n, group), np.arange(group - 5, n, group), np.arange(group - TILE + 3, n, 2 * group)])
        off = np.unique(np.concatenate([every, [0, n]]))
        od = torch.from_numpy(off).cuda()
        assert np.array_equal(tcr.irregular_scan(xd, od).cpu().numpy().astype(np.float64), oracle.irregular_scan(x, off))
    finally:
        tcr.set_variant("reset")


# One segment of most of the array next to many short or empty ones, whose mean length is that of many short ones
@pytest.mark.parametrize("flags", [0, 3])
@pytest.mark.parametrize("n", [3 << 23, 7 << 22, 1 << 25, 1 << 26, 1 << 27])
def test_time_with_one_dominating_segment(tcr, n, flags):
    x = torch.ones(n, dtype=torch.float16, device="cuda")
    for off in (torch.cat([16 * torch.arange(0, 1 << 20, device="cuda"), torch.tensor([n], device="cuda")]),
                torch.cat([torch.tensor([0], device="cuda"), torch.full((1024,), n, device="cuda")])):
        took = milliseconds(lambda: tcr.irregular_scan_ex(x, off, flags))
        tcr.set_variant("irregular_scan", "single")
        chained = milliseconds(lambda: tcr.irregular_scan_ex(x, off, flags))
        tcr.set_variant("reset")
        assert took <= 1.2 * chained, (took, chained)


# What an eager call has made room for, the same call with other offsets can be recorded with
@pytest.mark.parametrize("n", [BEYOND, (7 << 22) - 9, (5 << 23) + 77])
def test_recorded_with_other_offsets(tcr, oracle, n):
    x = workloads.make_input(n, "int1", 6)
    xd = torch.from_numpy(x).cuda()
    first = torch.from_numpy(workloads.make_offsets(n, "lognormal256", 2).view(np.int64)).cuda()
    off = workloads.make_offsets(n, "few7", 2).view(np.int64)
    od = torch.from_numpy(off).cuda()
    out = torch.empty(n, dtype=torch.float32, device="cuda")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    holders = [torch.cuda.Stream() for _ in range(8)]          # (tables that earlier calls left behind are in use elsewhere)
    for s in holders:
        with torch.cuda.stream(s):
            tcr.scan(xd[:1 << 24])
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        tcr.irregular_scan(xd, first, out=out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        tcr.irregular_scan(xd, od, out=out)
    want = oracle.irregular_scan(x, off)
    for _ in range(3):
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy().astype(np.float64), want)
        with torch.cuda.stream(side):
            again = tcr.irregular_scan(xd, od)
        side.synchronize()
        assert torch.equal(again, out)
    tcr.check_device_flags(side)
    torch.cuda.synchronize()
    del graph
    for s in holders + [side]:
        tcr.release_stream(s)


# Sums and moments at the upper end of the arrays that tiles of their own on workgroups of eight wavefronts are for (the tuner's third
# shape): segments of 64 on average, and half of the array in segments of one element.  No slower than that form.
@pytest.mark.parametrize("kind,mix", [("sum", "64"), ("sum", "halves"), ("moments", "64"), ("moments", "halves")])
def test_time_of_reductions_around_two_to_the_23(tcr, kind, mix):
    n = 1 << 23
    x = torch.ones(n, dtype=torch.float16, device="cuda")
    off = (torch.from_numpy(np.sort(np.random.default_rng(1).integers(0, n, n // 64))).cuda() if mix == "64"
           else torch.cat([torch.arange(0, n // 2 + 1, device="cuda"), torch.tensor([n], device="cuda")]))

    def calls():
        for _ in range(30):
            tcr.irregular_reduce(x, off) if kind == "sum" else tcr.irregular_moments(x, off)

    took = milliseconds(calls)
    tcr.tuning_import("irregular:0=2;")
    other = milliseconds(calls)
    tcr.tuning_import("")
    assert took <= 1.07 * other, (took, other)
