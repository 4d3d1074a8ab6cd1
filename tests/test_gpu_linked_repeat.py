"""Irregular reductions give the same bits from run to run, in each of their two forms: one launch whose tiles take the sums
that other tiles publish, or add them up again where they are not there yet, and tiles with a finishing kernel behind.
Fractional inputs, whose sums depend on the order of the additions, and segments over many tiles."""
import numpy as np
import pytest
import torch

from paper_1811_09736_amd import workloads

pytestmark = pytest.mark.gpu

TILE = 8192


@pytest.fixture(scope="module")
def tcr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1811_09736_amd import binding
    binding.set_variant("reset")
    binding.tuning_import("")
    yield binding
    binding.tuning_import("")
    binding.set_variant("reset")
    binding.check_device_flags()


def cuts(n):
    """Segments that begin and end around edges of tiles, sub-tiles and lanes, many tiles apart."""
    edges = [0, 5, TILE - 1, 3 * TILE + 4099, 70 * TILE + 8, 70 * TILE + 519, 600 * TILE, 600 * TILE + 1, n - 2 * TILE - 77, n - 3]
    return np.array(sorted(e for e in set(edges) if 0 <= e <= n) + [n], dtype=np.int64)


@pytest.mark.parametrize("tiles", [40, 200, 1024, 1025, 2048, 4096])      # wide tiles, then narrow ones; sums only at last
@pytest.mark.parametrize("tuning", ["", "irregular:0=0;", "irregular:0=1;"])
def test_waiting_or_not_gives_the_same_bits(tcr, oracle, tiles, tuning):
    n = tiles * TILE - 3
    x = workloads.make_input(n + 1, "normal", tiles)
    bd = torch.from_numpy(x).cuda()
    tcr.tuning_import(tuning)
    try:
        for shift in (0, 1):
            xd = bd[shift:shift + n]
            for off in (cuts(n), workloads.make_offsets(n, "few7", 3).view(np.int64), workloads.make_offsets(n, "lognormal256", 3).view(np.int64)):
                od = torch.from_numpy(off).cuda()
                results = []
                for wait in ("bounded", "none", "none", "bounded"):
                    tcr.set_variant("scan_wait", wait)
                    results.append((tcr.irregular_reduce(xd, od), *tcr.irregular_moments(xd, od), tcr.reduce(xd) if shift else od))
                for r in results[1:]:
                    assert all(torch.equal(a, b) for a, b in zip(r, results[0]))
        # at most 64 additions in a row, each within 2^-24 of the sum of magnitudes: 8 in a lane, 6 across lanes, 4 sub-tiles and
        # 8 wavefronts; then 8 published sums in a lane, 6 across lanes and 8 steps, or 16 tiles in a thread, 6 across lanes, 4
        # wavefronts, 2 steps and the 3 that join them
        want = oracle.irregular_reduce(x[1:], off)
        bound = 64 * 2.0 ** -24 * oracle.irregular_reduce(np.abs(x[1:]), off) + 1e-30
        assert np.all(np.abs(results[0][0].cpu().numpy().astype(np.float64) - want) <= bound)
    finally:
        tcr.set_variant("reset")
        tcr.tuning_import("")
