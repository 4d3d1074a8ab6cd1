"""Long sums of 2^23 to 2^24 elements in one launch: the last workgroup of a segment collects what the wavefronts publish, or adds
up again what is not there.  Whole numbers: exact."""
import numpy as np
import pytest
import torch

from paper_1811_09736_amd import workloads

pytestmark = pytest.mark.gpu

SPAN = 4096


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


@pytest.fixture(scope="module")
def array():
    x = workloads.make_input((1 << 24) + SPAN, "int1", 5)
    return x, torch.from_numpy(x).cuda()


# the first and last sizes, a last span of one element, of less than a tile, of whole and cut-off steps, a last workgroup with
# one to four wavefronts; and one beyond
SIZES = [(1 << 23) + 1, (1 << 23) + SPAN + 513, 2500 * SPAN + 8, 2501 * SPAN - 3, 2502 * SPAN - 4095, 2503 * SPAN + 2048, (1 << 24) - 1, 1 << 24,
         (1 << 24) + 1]


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("form", ["mfma", "dpp"])
@pytest.mark.parametrize("wait", ["bounded", "none"])     # none: every sum that is not there at the first look is added up again
def test_full(tcr, array, n, form, wait):
    tcr.set_variant("formulation", form)
    tcr.set_variant("scan_wait", wait)
    try:
        for _ in range(4):
            assert float(tcr.reduce(array[1][:n])) == float(array[0][:n].astype(np.float64).sum())
    finally:
        tcr.set_variant("reset")


@pytest.mark.parametrize("log2_seg", [18, 20, 22, 23])
@pytest.mark.parametrize("n", [1 << 24, 3 << 22])
@pytest.mark.parametrize("wait", ["bounded", "none"])
def test_segments(tcr, array, log2_seg, n, wait):
    n -= n % (1 << log2_seg)
    want = array[0][:n].astype(np.float64).reshape(-1, 1 << log2_seg).sum(1)
    tcr.set_variant("scan_wait", wait)
    try:
        for _ in range(3):
            assert np.array_equal(tcr.segmented_reduce(array[1][:n], 1 << log2_seg).cpu().numpy().astype(np.float64), want)
    finally:
        tcr.set_variant("reset")


def test_the_same_bits_whoever_adds(tcr):
    x = (torch.rand((1 << 23) + 77777, device="cuda") - 0.5).half()
    first = tcr.reduce(x).clone()
    tcr.set_variant("scan_wait", "none")
    try:
        for _ in range(5):
            assert torch.equal(tcr.reduce(x), first)
    finally:
        tcr.set_variant("reset")


def test_room_for_some_and_streams_and_graphs(tcr, array):
    n = (1 << 23) + 12345
    xd, want = array[1][:n], float(array[0][:n].astype(np.float64).sum())
    for size in (1 << 15, 1 << 18):                     # without and with room for the descriptors
        buf = torch.full((size,), 0x5A, dtype=torch.uint8, device="cuda")
        try:
            tcr.set_workspace(buf)
            assert all(float(tcr.reduce(xd)) == want for _ in range(3))
        finally:
            torch.cuda.synchronize()
            tcr.set_workspace(None)
    streams, outs = [torch.cuda.Stream() for _ in range(3)], []
    torch.cuda.synchronize()
    for _ in range(4):
        for s in streams:
            with torch.cuda.stream(s):
                outs.append(tcr.reduce(xd))
    torch.cuda.synchronize()
    assert all(float(o) == want for o in outs)
    out, s = torch.zeros(1, device="cuda"), torch.cuda.Stream()
    with torch.cuda.stream(s):
        tcr.reduce(xd, out=out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        tcr.reduce(xd, out=out)
    for _ in range(4):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert float(out) == want
        with torch.cuda.stream(s):
            assert float(tcr.reduce(xd)) == want
        torch.cuda.synchronize()
