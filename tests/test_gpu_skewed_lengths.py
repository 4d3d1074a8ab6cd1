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
