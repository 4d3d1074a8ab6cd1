"""Sums and both moments of segments of 3 to 30 elements: one, two, four and eight tiles per wavefront of the packed rows, and whole segments inside a
lane's eight elements (4 and 8), at counts around what a wavefront and a workgroup take, on either side of the sizes where that changes, for
arrays on 16, 4 and 2-byte boundaries.  Whole numbers against sums in 64 bits; fractions within the roundings of that few additions."""
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


def check(tcr, seg, nseg, lead):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seg + nseg)
    x = torch.randint(-4, 5, (seg * nseg + lead,), generator=gen, device="cuda", dtype=torch.int8).half()[lead:]
    rows = x.double().view(nseg, seg)
    s, q = tcr.segmented_moments(x, seg)
    assert torch.equal(s.double(), rows.sum(1)) and torch.equal(q.double(), (rows * rows).sum(1)), (seg, nseg, lead)
    assert torch.equal(tcr.segmented_reduce(x, seg), s), (seg, nseg, lead)


@pytest.mark.parametrize("seg", [3, 4, 5, 6, 7, 8, 9, 11, 12, 15, 18, 22, 24, 30])
def test_counts_around_a_wavefront_and_a_workgroup(tcr, seg):
    per_row = 32 // seg - (1 if seg % 2 and (32 // seg) % 2 else 0)
    for tiles in (1, 2, 4, 8):
        wave = 16 * tiles * per_row
        for nseg in {2, per_row + 1, wave - 1, wave, wave + 1, 4 * wave - 1, 4 * wave + per_row + 1}:
            for lead in (0, 1, 2):
                check(tcr, seg, max(nseg, 2), lead)


@pytest.mark.parametrize("seg", [3, 5, 7, 22, 4, 8])
@pytest.mark.parametrize("edge", [5 << 18, 9 << 19, 11 << 20, 3 << 22, 1 << 25])
def test_where_the_number_of_tiles_changes(tcr, seg, edge):
    for n in (edge - seg, edge, edge + seg):
        check(tcr, seg, n // seg, 0)


# exact products, added in binary64 and rounded once: half a spacing of binary32, 2^-24 of the result
@pytest.mark.parametrize("seg", [4, 8])
def test_fractions_subnormals_and_results_off_a_boundary(tcr, seg):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seg)
    x = torch.rand(seg * 4099, generator=gen, device="cuda").half()
    x[::3] *= 2.0 ** -14                         # (many of them subnormal)
    rows = x.double().view(-1, seg)
    s, q = tcr.segmented_moments(x, seg)
    for got, want in ((s, rows.sum(1)), (q, (rows * rows).sum(1))):
        assert ((got.double() - want).abs() <= 1.001 * 2.0 ** -24 * want).all()
    out = torch.full((2 * 4099 + 3,), -1.0, device="cuda")
    st = tcr.raw().tcr_segmented_moments(x.data_ptr(), out.data_ptr() + 4, out.data_ptr() + 4 * (4099 + 2), x.numel(), seg, torch.cuda.current_stream().cuda_stream)
    assert st == tcr.OK
    assert torch.equal(out[1:4100], s) and torch.equal(out[4101:8200], q) and out[0] == -1 and out[4100] == -1 and out[8200] == -1


# and with the width of a row: 9, 20 and 22 elements make rows of 18, 20 and 22
@pytest.mark.parametrize("seg,edge", [(9, 9 << 20), (20, 10 << 20), (22, 11 << 20), (7, 11 << 20), (7, 3 << 22)])
def test_where_the_width_of_a_row_counts(tcr, seg, edge):
    for n in (edge - seg, edge, edge + seg):
        check(tcr, seg, n // seg, 0)
