"""tcr_irregular_scan_filled where it is refused: nothing is enqueued or recorded, the zeros outside the segments neither."""
import pytest
import torch

pytestmark = pytest.mark.gpu

N = (1 << 24) + 4096                     # larger than what one launch without look-up tables takes


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
def arrays():
    return (torch.ones(N, dtype=torch.float16, device="cuda"), torch.tensor([1000, 3000, N - 9000], dtype=torch.int64, device="cuda"),
            torch.empty(N, dtype=torch.float32, device="cuda"))


def filled(tcr, arrays, stream):
    x, off, out = arrays
    return tcr.raw().tcr_irregular_scan_filled(x.data_ptr(), off.data_ptr(), out.data_ptr(), N, 2, 0, stream.cuda_stream)


def test_recorded_without_a_workspace(tcr, arrays):
    x, off, out = arrays
    side, one = torch.cuda.Stream(), torch.zeros(1, device="cuda")
    tcr.release_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        assert filled(tcr, arrays, side) == tcr.ERR_UNSUPPORTED
        one.fill_(1.0)                   # something to record
    for _ in range(2):
        out.fill_(-5.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.all(out == -5.0) and float(one) == 1.0


def test_on_a_workspace_that_is_too_small(tcr, arrays):
    x, off, out = arrays
    stream = torch.cuda.current_stream()
    out.fill_(-5.0)
    try:
        tcr.set_workspace(torch.zeros(768, dtype=torch.uint8, device="cuda"))
        assert filled(tcr, arrays, stream) == tcr.ERR_WORKSPACE
        torch.cuda.synchronize()
        assert torch.all(out == -5.0)
    finally:
        tcr.set_workspace(None)
    assert filled(tcr, arrays, stream) == tcr.OK
    torch.cuda.synchronize()
    want = torch.zeros(N, device="cuda")
    want[1000:3000] = torch.arange(1, 2001, device="cuda")
    want[3000:N - 9000] = torch.arange(1, N - 12000 + 1, device="cuda")          # (below 2^24: exact)
    assert torch.equal(out, want)
