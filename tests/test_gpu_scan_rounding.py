"""Rounding of scans of fractions against 64 bits, counted in roundings of a result's size: the error's 2-norm over the one that a single rounding of
every result leaves, squared.  Whole numbers, which most tests use, are exact in any order of additions; these limits lie between two orders."""
import numpy as np
import pytest
import torch

from paper_1811_09736_amd import workloads

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


# The same where the sum in front goes through binary64: long open parts that each tile adds up (2.2 roundings; 4.8 to 7.0 in binary32, in front of a lane's
# additions), and what is looked up where results are stored by element (2.5 to 3.4; 3.3 to 4.8).
@pytest.mark.parametrize("n,seg,shift,limit", [(HELD + (1 << 22), 6145, 0, 2.6), (HELD + (1 << 22), 8191, 0, 2.6), (HELD + (1 << 22), 4097, 3, 2.6), (3 << 24, 5001, 1, 2.6),
                                               (3 << 24, 8191, 5, 2.6), (3 << 24, 9001, 3, 2.9), (3 << 24, 50003, 2, 3.6), (3 << 24, 65536, 3, 4.0), (3 << 24, 100003, 7, 3.6)])
@pytest.mark.parametrize("flags", [0, 1])
def test_the_sum_in_front_in_binary64(tcr, n, seg, shift, limit, flags):
    n -= n % seg
    x = fractions(n + shift)[shift:]
    want = torch.cumsum(x.double().view(-1, seg), 1)
    if flags & tcr.SCAN_EXCLUSIVE:
        want -= x.double().view(-1, seg)
    got = tcr.segmented_scan_ex(x, seg, flags).view(-1, seg)
    assert roundings(got, want) < limit


# Irregular segments whose sum in front all four wavefronts of a tile look up, from a table or near by, or get from the relay: 2.6 to 3.1 roundings
# whichever it is; with looked-up sums added in binary32 3.9 to 6.1.
@pytest.mark.parametrize("recipe,n", [("lognormal100", 17 << 20), ("lognormal20", 17 << 20), ("half", 17 << 20), ("lognormal100", 21 << 20), ("lognormal100", 24 << 20)])
@pytest.mark.parametrize("flags", [0, 1])
def test_looked_up_sums(tcr, recipe, n, flags):
    x = fractions(n)
    sums = torch.cumsum(x.double(), 0)
    off = torch.cat([torch.arange(n // 2 + 1), torch.tensor([n])]) if recipe == "half" else torch.from_numpy(workloads.make_offsets(n, recipe, 5).view(np.int64))
    off = off.cuda()
    want = sums - torch.repeat_interleave(torch.cat([sums.new_zeros(1), sums])[off[:-1]], off[1:] - off[:-1])
    if flags & tcr.SCAN_EXCLUSIVE:
        want -= x.double()
    assert roundings(tcr.irregular_scan_ex(x, off, flags), want) < 3.5


# A tile that has waited in vain adds up what is in front of it by itself (the look-up of arrays that the chip holds at once, the relay of larger
# ones), and which tiles do is a matter of time: no more roundings than where all wait.  Waiting / adding up here: 9.5 / 8.5, 9.4 / 8.5, 5.3 / 6.2, 2.8 /
# 3.7, 2.8 / 2.9; with the sums of the tiles added one after the other in binary32 156, 56, 6.2, 3.9, 3.8.
@pytest.mark.parametrize("call,n,limit", [("one", 7 << 20, 11.0), ("one", 11 << 20, 11.0), ("scan", 3 << 24, 7.5), ("seven", 3 << 24, 4.5), ("rows", 3 << 24, 4.0)])
@pytest.mark.parametrize("wait", ["bounded", "none"])
def test_tiles_that_help_themselves(tcr, call, n, limit, wait):
    x = fractions(n)
    sums = torch.cumsum(x.double(), 0)
    tcr.set_variant("scan_wait", wait)
    try:
        if call == "scan":
            got, want = tcr.scan(x), sums
        elif call == "rows":
            m = n - n % 1000003
            got, want = tcr.segmented_scan(x[:m], 1000003), torch.cumsum(x[:m].double().view(-1, 1000003), 1).view(-1)
        else:
            off = torch.tensor([0, n]) if call == "one" else torch.from_numpy(workloads.make_offsets(n, "few7", 5).view(np.int64))
            off = off.cuda()
            got = tcr.irregular_scan(x, off)
            want = sums - torch.repeat_interleave(torch.cat([sums.new_zeros(1), sums])[off[:-1]], off[1:] - off[:-1])
    finally:
        tcr.set_variant("reset")
    assert roundings(got, want) < limit
