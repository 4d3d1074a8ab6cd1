"""Long segments shared among several wavefronts: the counts of wavefronts, of steps and of pieces change with the size of
the array and with the segment length, and so do the ends that are masked.  Whole numbers: every result is exact."""
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
    binding.check_device_flags()


# (segments, length): 1, 4 and 16 wavefronts per segment, a last step that is nearly empty or nearly full, odd lengths (no
# segment but the first starts on a tile or a group of 8), the last lengths of one workgroup and the first in pieces
SHAPES = [(5, 3001), (3, 4095), (3, 4097), (2100, 4099), (2, 8161), (2048, 8193), (9, 8192 + 512), (513, 16383), (2, 16385), (40, 16385),
          (7, 20481), (511, 32771), (3, 65537), (2, 131071), (2, 131072), (2, 131073), (5, 262144), (3, 300001), (2, 1 << 20),
          (700, 16384), (130, 65536), (300, 32768), (33, 131072), (1, 4194304 + 11), (1, 33554432 - 4097)]


@pytest.mark.parametrize("nseg,seg", SHAPES)
def test_split_segments(tcr, oracle, nseg, seg):
    n = nseg * seg
    x = workloads.make_input(n, "int4", seg % 977)
    xd = torch.from_numpy(x).cuda()
    want = oracle.segmented_reduce(x, seg)
    assert np.max(np.abs(want)) < 2 ** 24
    assert np.array_equal(tcr.segmented_reduce(xd, seg).cpu().numpy().astype(np.float64), want)
    if seg <= 1 << 21:                               # (squares of up to 16: their sums stay below 2^24)
        a, q = tcr.segmented_moments(xd, seg)
        wa, wq = oracle.segmented_moments(x, seg)
        assert np.max(wq) < 2 ** 24
        assert np.array_equal(a.cpu().numpy().astype(np.float64), wa)
        assert np.array_equal(q.cpu().numpy().astype(np.float64), wq)


def test_neighbours_of_a_segment_do_not_reach_it(tcr):
    # infinities on both sides of a segment whose ends are cut out of shared groups of 8
    seg = 5003
    x = torch.ones(3 * seg, dtype=torch.float16, device="cuda")
    x[:seg] = float("inf")
    x[2 * seg:] = float("inf")
    for length in (seg,):
        assert float(tcr.segmented_moments(x, length)[0][1]) == seg
        assert float(tcr.segmented_moments(x, length)[1][1]) == seg
    y = torch.ones(3 * 9001, dtype=torch.float16, device="cuda")
    y[:9001] = float("inf")
    y[2 * 9001:] = float("-inf")
    assert float(tcr.segmented_reduce(y, 9001)[1]) == 9001


@pytest.mark.parametrize("nseg,seg", [(8, 1 << 19), (9, 300001)])
def test_a_small_caller_workspace_still_serves_long_segments(tcr, oracle, nseg, seg):
    # one partial per 65536 elements is all that a call with these arguments has ever needed: 64 and 45 of them fit the
    # smallest workspace (two areas of 256 bytes), the finer pieces of an ordinary call do not
    x = workloads.make_input(nseg * seg, "int4", 3)
    xd = torch.from_numpy(x).cuda()
    want = oracle.segmented_reduce(x, seg)
    buf = torch.full((768,), 0x5A, dtype=torch.uint8, device="cuda")
    try:
        tcr.set_workspace(buf)
        got = tcr.segmented_reduce(xd, seg).cpu().numpy().astype(np.float64)
        torch.cuda.synchronize()
    finally:
        tcr.set_workspace(None)
    assert np.array_equal(got, want)
    assert np.array_equal(tcr.segmented_reduce(xd, seg).cpu().numpy().astype(np.float64), want)


def test_recorded_with_the_workspace_that_there_is(tcr, oracle):
    # a stream whose workspace holds fewer partials than the finest plan wants: the recorded call takes the coarse one
    nseg, seg = 8, 1 << 19
    x = workloads.make_input(nseg * seg, "int4", 5)
    xd = torch.from_numpy(x).cuda()
    out = torch.empty(nseg, dtype=torch.float32, device="cuda")
    small = torch.from_numpy(workloads.make_input(1 << 20, "int4", 6)).cuda()
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        tcr.reduce(small)                                # this stream's workspace: one partial per 4096 elements of 2^20
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        tcr.segmented_reduce(xd, seg, out=out)
    want = oracle.segmented_reduce(x, seg)
    for _ in range(3):
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy().astype(np.float64), want)
    tcr.release_stream(side)
