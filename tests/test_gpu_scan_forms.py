"""Regular scans of untuned lengths beyond 2^24 elements around the limits between the forms that take them -- tiles that add up or look up what is in
front of them, carries handed out by one workgroup, chained tiles -- which go by length, type, size and alignment: against sums that are exact."""
import pytest
import torch

pytestmark = pytest.mark.gpu

M = 1 << 20


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


def check(tcr, n, seg, flags, shift=0, off=0):
    """shift, off: elements between a 256-byte boundary and the input, the results."""
    n -= n % seg
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seg)
    x = torch.randint(-1, 2, (n + shift,), generator=gen, device="cuda", dtype=torch.int8).half()[shift:]
    dtype = torch.float16 if flags & 2 else torch.float32
    out = torch.full((n + off + 8,), 77.0, dtype=dtype, device="cuda")
    tcr.segmented_scan_ex(x, seg, flags, out=out[off:off + n])
    want = torch.cumsum(x.view(-1, seg), 1, dtype=torch.float64).view(-1)
    if flags & 1:
        want -= x
    # (the sums are exact, so each is rounded once)
    assert torch.equal(out[off:off + n], want.to(dtype)), (n, seg, flags, shift, off)
    assert (out[:off] == 77).all() and (out[off + n:] == 77).all()


# 16-byte boundaries on both sides: sizes in front of and behind each limit
@pytest.mark.parametrize("seg,flags,n", [(6151, 0, 26 * M), (6151, 0, 27 * M), (8191, 1, 25 * M), (9001, 3, 41 * M), (32767, 2, 41 * M), (131072 + 3, 3, 41 * M), (262144 + 3, 3, 41 * M)])
def test_aligned(tcr, seg, flags, n):
    check(tcr, n, seg, flags)


# an input, or results, off a boundary: results are stored by element
@pytest.mark.parametrize("seg,flags,n", [(4099, 0, 60 * M), (6151, 0, 17 * M), (8191, 1, 28 * M), (32771, 0, 39 * M), (32771, 1, 41 * M), (300007, 0, 41 * M),
                                         (2051, 3, 61 * M), (4099, 2, 39 * M), (4099, 3, 41 * M), (8191, 2, 97 * M), (4099, 2, 97 * M), (50021, 3, 42 * M), (300007, 2, 41 * M)])
@pytest.mark.parametrize("shift,off", [(3, 0), (0, 1), (8, 8)])
def test_off_a_boundary(tcr, seg, flags, n, shift, off):
    check(tcr, n, seg, flags, shift, off)


# the chained form where a caller's buffer has no room for its tiles: each tile adds up what is in front of it
def test_chained_without_room(tcr):
    tcr.set_workspace(torch.full((4096,), 0x5A, dtype=torch.uint8, device="cuda"))
    try:
        check(tcr, 97 * M, 4099, 2, 3, 0)
    finally:
        tcr.set_workspace(None)


# a caller's buffer of the size that is said to do: adding and looking up where the library's own memory has carries handed out, chained tiles beyond 2^27
@pytest.mark.parametrize("seg,flags,n,shift", [(4099, 0, 60 * M, 0), (40001, 1, 39 * M, 0), (40001, 0, 41 * M, 0), (2051, 3, 61 * M, 0), (300007, 2, 63 * M, 0), (300007, 3, 65 * M, 0),
                                               (65536, 2, 63 * M, 0), (65536, 3, 65 * M, 0), (4099, 2, 129 * M, 0), (8191, 1, 129 * M, 0), (300007, 0, 129 * M, 0),
                                               (129 * M - 3, 2, 129 * M, 1), (129 * M - 3, 0, 129 * M, 0), (50021, 0, 129 * M, 3)])
def test_callers_buffer(tcr, seg, flags, n, shift):
    tcr.set_workspace(torch.full((tcr.workspace_bytes(tcr.OP_SEGMENTED_SCAN, n - n % seg, seg),), 0x5A, dtype=torch.uint8, device="cuda"))
    try:
        check(tcr, n, seg, flags, shift)
    finally:
        tcr.set_workspace(None)
