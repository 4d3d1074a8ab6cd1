"""Scans whose sums are looked up, of more than 2^24 elements, on a caller's buffer without room for a descriptor per tile: whatever
form is left is right, and no further from the exact sums than chained tiles on the same buffer."""
import numpy as np
import pytest
import torch

from paper_1811_09736_amd import workloads

pytestmark = pytest.mark.gpu

N = 3 << 23                                     # 3072 tiles of 8192 elements (irregular), 1536 of 16384 (regular), 768 chained ones


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


def on_buffer(tcr, descriptors, call):
    """call() with a workspace of 256 bytes and two areas of that many 8-byte words."""
    torch.cuda.synchronize()
    tcr.set_workspace(torch.full((256 + 16 * descriptors,), 0x5A, dtype=torch.uint8, device="cuda"))
    try:
        got = call()
        torch.cuda.synchronize()
        return got
    finally:
        tcr.set_workspace(None)


# one area step (32 descriptors) below the tiles, at them, and as few as two tables or one of chained tiles take
@pytest.mark.parametrize("descriptors", [3072, 3040, 1568, 800])
@pytest.mark.parametrize("flags", [0, 1])
def test_irregular(tcr, oracle, descriptors, flags):
    x = workloads.make_input(N, "int1", 4)
    xd = torch.from_numpy(x).cuda()
    for recipe in ("few7", "uniform16"):
        off = workloads.make_offsets(N, recipe, 5).view(np.int64)
        od = torch.from_numpy(off).cuda()
        got = on_buffer(tcr, descriptors, lambda: tcr.irregular_scan_ex(xd, od, flags))
        want = oracle.irregular_scan_exclusive(x, off) if flags else oracle.irregular_scan(x, off)
        assert np.array_equal(got.cpu().numpy().astype(np.float64), want)


@pytest.mark.parametrize("descriptors", [1536, 1504, 800])
@pytest.mark.parametrize("seg", [100003, 3000003])
def test_regular(tcr, oracle, descriptors, seg):
    n = N // seg * seg
    x = workloads.make_input(n, "int1", 4)
    got = on_buffer(tcr, descriptors, lambda: tcr.segmented_scan(torch.from_numpy(x).cuda(), seg))
    assert np.array_equal(got.cpu().numpy().astype(np.float64), oracle.segmented_scan(x, seg))


# (the chained tiles' own figure moves by a few per cent with the order in which their sums become known)
def test_rounding(tcr):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    x = torch.rand(N, generator=gen, device="cuda").half()
    off = torch.from_numpy(workloads.make_offsets(N, "few7", 5).view(np.int64)).cuda()
    sums = torch.cumsum(x.double(), 0)
    want = sums - torch.repeat_interleave(torch.cat([sums.new_zeros(1), sums])[off[:-1]], off[1:] - off[:-1])

    def error():
        got = on_buffer(tcr, 3040, lambda: tcr.irregular_scan(x, off)).double()
        return ((got - want).pow(2).sum() / want.pow(2).sum()).sqrt().item()

    here = error()
    tcr.set_variant("irregular_scan", "chain")
    chained = error()
    tcr.set_variant("reset")
    assert here <= 1.1 * chained, (here, chained)
