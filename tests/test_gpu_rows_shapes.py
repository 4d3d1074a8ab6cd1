"""The three shares of a workgroup of rows_reduce_kernel (16320, 8128 and 4032 elements in whole segments): counts of segments that fill a share
exactly, by one more and one less, with arrays off a 16-byte boundary, on either side of the sizes where the share changes.  Whole numbers, so
that sums and sums of squares are exact, against sums in 64 bits."""
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
    binding.check_device_flags()


def check(tcr, seg, nseg, moments, lead):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seg + nseg)
    x = torch.randint(-4, 5, (seg * nseg + lead,), generator=gen, device="cuda", dtype=torch.int8).half()[lead:]
    rows = x.double().view(nseg, seg)
    if moments:
        s, q = tcr.segmented_moments(x, seg)
        assert torch.equal(q.double(), (rows * rows).sum(1)), (seg, nseg, lead)
    else:
        s = tcr.segmented_reduce(x, seg)
    assert torch.equal(s.double(), rows.sum(1)), (seg, nseg, lead)


# (two segments at the least: one is another call)
@pytest.mark.parametrize("seg", [17, 25, 31, 33, 100, 784, 2015, 2032, 2033, 2709, 2711, 2999])
@pytest.mark.parametrize("share", [4032, 8128, 16320])
@pytest.mark.parametrize("moments", [False, True])
def test_shares_filled_and_not(tcr, seg, share, moments):
    full = share // seg
    for nseg in {full, full + 1, 3 * full - 1, 3 * full, 7 * full + 2} - {0, 1}:
        for lead in (0, 3):
            check(tcr, seg, nseg, moments, lead)


# (sums of 4032 elements a share begin at 3 * 2^20, and all changes are repeated below and above)
@pytest.mark.parametrize("seg,edge,moments", [(25, 7 << 21, False), (100, 3 << 20, False), (2015, 13 << 20, False), (2017, 13 << 20, False),
                                              (31, 1 << 26, True), (33, 5 << 22, True), (2033, 1 << 24, True), (2709, 1 << 24, True)])
def test_where_the_share_changes(tcr, seg, edge, moments):
    for n in (edge - seg, edge, edge + 2 * seg):
        check(tcr, seg, n // seg, moments, 0)
        check(tcr, seg, n // seg, moments, 7)


# and where it changes with how much of it whole segments fill
@pytest.mark.parametrize("seg,edge,moments", [(1200, 1 << 23, True), (1355, 1 << 23, True), (2035, 5 << 20, True), (2500, 13 << 20, True), (1999, 1 << 24, True),
                                              (784, 9 << 20, False), (784, 23 << 19, False), (1355, 9 << 20, False), (1700, 13 << 20, False)])
def test_where_the_filled_share_changes(tcr, seg, edge, moments):
    test_where_the_share_changes(tcr, seg, edge, moments)
