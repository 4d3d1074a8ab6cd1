"""The finishing kernel of irregular reductions at the edges of its groups of 256 tiles.  Arrays of these sizes run as one
launch by default, so the tuning table's tiles of 16384 elements, which have no such form, are asked for -- with the one
launch beside them.  Whole numbers: exact; fractional ones the same from run to run."""
import numpy as np
import pytest
import torch

from paper_1811_09736_amd import workloads

pytestmark = pytest.mark.gpu

TILE, GROUP = 16384, 256


@pytest.fixture(scope="module")
def tcr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1811_09736_amd import binding
    binding.set_variant("reset")
    binding.tuning_import("")
    yield binding
    binding.tuning_import("")
    binding.check_device_flags()


@pytest.mark.parametrize("tiles", [1, 2, 3, GROUP - 1, GROUP, GROUP + 1, 2 * GROUP, 2 * GROUP + 3, 4 * GROUP - 1])
def test_groups_of_tiles(tcr, oracle, tiles):
    n = tiles * TILE - 5
    x = workloads.make_input(n, "int1", tiles)                    # |x| <= 1: the sums of squares stay below 2^24
    f = workloads.make_input(n, "normal", tiles)
    xd, fd = torch.from_numpy(x).cuda(), torch.from_numpy(f).cuda()
    mid = (tiles // 2) * TILE
    cuts = [[0, 5, n - 3, n], [0, n], [n // 2, n // 2 + 1, n], [0, 3, 3, n - TILE // 2, n - 9, n - 9], [0, mid, n], [0, max(mid - 1, 0), mid + 1, n],
            [0] + [t * TILE + 7 for t in range(0, tiles, 97) if t * TILE + 7 < n] + [n]]
    for off in cuts:
        off = np.asarray(off, dtype=np.int64)
        od = torch.from_numpy(off).cuda()
        wa, wq = oracle.irregular_moments(x, off)
        for tuning in ("irregular:0=1;", ""):
            tcr.tuning_import(tuning)
            try:
                a, q = tcr.irregular_moments(xd, od)
                assert np.array_equal(tcr.irregular_reduce(xd, od).cpu().numpy().astype(np.float64), wa)
                assert np.array_equal(a.cpu().numpy().astype(np.float64), wa) and np.array_equal(q.cpu().numpy().astype(np.float64), wq)
                first, again = ((tcr.irregular_reduce(fd, od), *tcr.irregular_moments(fd, od)) for _ in range(2))
                assert all(torch.equal(u, v) for u, v in zip(first, again))
            finally:
                tcr.tuning_import("")
