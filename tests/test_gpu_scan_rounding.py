"""Rounding of scans of fractions against 64 bits, counted in roundings of a result's size: the error's 2-norm over the one that a single rounding of
every result leaves, squared.  Whole numbers, which most tests use, are exact in any order of additions; these limits lie between two orders."""
import pytest
import torch

pytestmark = pytest.mark.gpu

HELD = 1 << 24                                  # beyond it workgroups follow each other (256 compute units)


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


def fractions(n):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    return torch.rand(n, generator=gen, device="cuda").half()


def roundings(got, want):
    """A rounding of a value between 2^e and 2^(e+1) is off by at most 2^(e-24) either way, evenly: one twelfth of its square spacing."""
    spacing = torch.ldexp(torch.ones_like(want), torch.frexp(want)[1] - 24)
    return float(((got.double() - want) ** 2).sum() / (spacing ** 2).sum() * 12)


# Regular segments whose sum in front is looked up.  Added once, behind the sums of the tile, it leaves 3.3 to 5.4 roundings: that addition, and the ones
# that made it of wavefronts' and tiles' sums.  In front of a lane's eight additions, of which each then rounds a value of its size, 5.9 to 11.2.
@pytest.mark.parametrize("seg,limit", [(9001, 4.5), (16001, 6.0), (30003, 6.5), (32767, 6.5)])
@pytest.mark.parametrize("flags", [0, 1])
def test_the_sum_in_front_is_added_once(tcr, seg, limit, flags):
    n = HELD + (1 << 22)
    n -= n % seg
    x = fractions(n)
    want = torch.cumsum(x.double().view(-1, seg), 1)
    if flags & tcr.SCAN_EXCLUSIVE:
        want -= x.double().view(-1, seg)
    got = tcr.segmented_scan_ex(x, seg, flags).view(-1, seg)
    assert roundings(got, want) < limit
