"""Scans of untuned lengths up to 8192 in arrays on both sides of the sizes from which the tiles are chained instead, with the
workspace at hand and without one.  Whole numbers, exact: against the cumulative sum of the segments' rows in binary32."""
import pytest
import torch

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


@pytest.fixture(scope="module")
def data():
    torch.manual_seed(4)
    return torch.randint(-1, 2, ((3 << 26) + 16384,), device="cuda", dtype=torch.int8).to(torch.float16)


def check(got, x, seg, exclusive):
    ref = torch.cumsum(x.view(-1, seg), 1, dtype=torch.float32)           # (rounded alike where binary16 does not hold them)
    if exclusive:
        ref = ref - x.view(-1, seg)
    assert torch.equal(got.view(-1, seg), ref.to(got.dtype))


@pytest.mark.parametrize("limit", [9 << 22, 5 << 23, 3 << 24, 11 << 22, 13 << 22, 7 << 23, 5 << 24, 1 << 27, 3 << 26])
@pytest.mark.parametrize("seg", [2047, 3071, 3073, 4095, 4097, 6143, 6145, 8191])
def test_both_sides_of_every_limit(tcr, data, limit, seg):
    for n in (limit // seg * seg, (limit // seg + 1) * seg):
        for shift, flags in ((0, 0), (0, 3), (1, 2)):
            x = data[shift:shift + n]
            check(tcr.segmented_scan_ex(x, seg, flags), x, seg, flags & 1)


@pytest.mark.parametrize("flags", [0, 2])
def test_without_a_workspace(tcr, data, flags):
    seg, n = 8191, ((1 << 27) // 8191 + 1) * 8191
    x = data[:n]
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    tcr.release_stream(side)
    out = torch.empty(n, dtype=torch.float16 if flags else torch.float32, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):                           # recorded on a stream that has none
        tcr.segmented_scan_ex(x, seg, flags, out=out)
    for _ in range(2):
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        check(out, x, seg, 0)
    try:
        tcr.set_workspace(torch.zeros(768, dtype=torch.uint8, device="cuda"))
        check(tcr.segmented_scan_ex(x, seg, flags), x, seg, 0)           # a caller's buffer with room for 32 tiles
        torch.cuda.synchronize()
    finally:
        tcr.set_workspace(None)
