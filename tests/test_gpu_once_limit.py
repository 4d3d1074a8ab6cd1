"""Full scans around the largest array that runs as one tile per workgroup: a ragged one just above it is scanned by the
pipelined chain over its whole groups of 8, whose multiple of 8 is itself still an array of that size.  Whole numbers: exact."""
import numpy as np
import pytest
import torch

from paper_1811_09736_amd import workloads

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


@pytest.fixture(scope="module")
def data(oracle):
    largest = torch.cuda.get_device_properties(0).multi_processor_count * 65536     # elements
    x = workloads.make_input(largest + 32, "int1", 3)
    return largest, x, torch.from_numpy(x).cuda(), oracle.scan(x)


@pytest.mark.parametrize("past", [-9, -8, -1, 0, 1, 2, 3, 5, 7, 8, 9, 15])
def test_ragged_ends(tcr, data, past):
    largest, x, xd, ref = data
    n = largest + past
    assert np.max(np.abs(ref)) < 2 ** 24
    assert np.array_equal(tcr.scan(xd[:n]).cpu().numpy().astype(np.float64), ref[:n])
    excl = tcr.scan_ex(xd[:n], tcr.SCAN_EXCLUSIVE | tcr.OUT_F16).cpu().numpy()
    assert np.array_equal(excl, np.concatenate([[0.0], ref[:n - 1]]).astype(np.float16))
