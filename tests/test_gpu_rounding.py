"""Rounding of the forms for arrays that do not fill the chip, against sums in 64 bits.  Non-negative inputs, so the bound is
relative: k additions in a row of binary32 numbers are off by at most k * 2^-24 of the sum (and the square of that, which is
nothing here).  Per form, the additions on the longest way from an element to its result; a matrix product adds 32 elements
to its accumulator."""
import numpy as np
import pytest
import torch

from paper_1811_09736_amd import workloads

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


@pytest.fixture(scope="module")
def tcr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1811_09736_amd import binding
    binding.set_variant("reset")
    binding.tuning_import("")
    yield binding
    binding.check_device_flags()


def off_by(got, want):
    got = got.cpu().numpy().astype(np.float64)
    return float(np.max(np.abs(got - want) / np.maximum(want, 1e-30)))


# one workgroup: 16 products in a row; one launch: 8 products, then 128 partials in two rounds of 64 lanes, or 160 in three;
# two kernels: 8 products, 4096 partials as four rounds.  16 row sums and 16 wavefronts are 4 additions each, 64 lanes 6.
@pytest.mark.parametrize("n,seg,adds", [(131072, 131072, 16 * 32 + 8), (131073, 131073, 8 * 32 + 8 + 8), (1 << 20, 1 << 20, 8 * 32 + 16),
                                        (1 << 23, 1 << 23, 8 * 32 + 16), (1 << 24, 1 << 24, 8 * 32 + 4 + 4 + 6 + 4 + 4), (1 << 22, 1 << 18, 8 * 32 + 16),
                                        (1 << 22, 1 << 16, 16 * 32 + 8), (1 << 20, 1 << 16, 16 * 32 + 8), (50001 * 40, 50001, 13 * 32 + 8),
                                        (131073 * 31, 131073, 8 * 32 + 17), (300001 * 3, 300001, 8 * 32 + 17)])
def test_reductions(tcr, oracle, n, seg, adds):
    x = workloads.make_input(n, "uniform_01", seg)
    xd = torch.from_numpy(x).cuda()
    off = np.arange(0, n + 1, seg, dtype=np.int64)
    wa, wq = oracle.irregular_moments(x, off)
    assert off_by(tcr.segmented_reduce(xd, seg), wa) <= adds * U
    a, q = tcr.segmented_moments(xd, seg)
    assert off_by(a, wa) <= adds * U and off_by(q, wq) <= adds * U


# a tile's own part: up to 16 sub-tiles of a wavefront, 16 wavefronts, 64 lanes of 8 elements; in front of it up to 256 sums
# in four rounds of 64 lanes, or up to 1024 tiles in sixteen steps of 64
@pytest.mark.parametrize("n,seg", [(1 << 16, 0), ((1 << 20) + 3, 0), (1 << 22, 0), (1 << 24, 0), ((1 << 24) + 3, 0), (1 << 22, 1 << 17), (1 << 24, 1 << 20),
                                   (100003 * 100, 100003), (1001 * 5000, 1001), (8191 * 300, 8191), (33 * 9000, 33)])
def test_scans(tcr, oracle, n, seg):
    x = workloads.make_input(n, "uniform_01", n % 1013)
    xd = torch.from_numpy(x).cuda()
    adds = (32 + 16 + 4) + (8 + 6 + 16 + 16) + (4 + 6 + 16 + 6)
    want = oracle.segmented_scan(x, seg) if seg else oracle.scan(x)
    got = tcr.segmented_scan(xd, seg) if seg else tcr.scan(xd)
    assert off_by(got, want) <= adds * U


@pytest.mark.parametrize("recipe", ["few7", "lognormal256", "uniform16"])
@pytest.mark.parametrize("n", [(1 << 20) + 5, 5200000, 1 << 24])
def test_irregular_scans(tcr, oracle, recipe, n):
    x = workloads.make_input(n, "uniform_01", 3)
    off = workloads.make_offsets(n, recipe, 3).view(np.int64)
    got = tcr.irregular_scan(torch.from_numpy(x).cuda(), torch.from_numpy(off).cuda())
    assert off_by(got, oracle.irregular_scan(x, off)) <= ((8 + 6 + 4 + 16) + (16 + 6 + 16)) * U
