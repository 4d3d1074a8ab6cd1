"""The kernels that the auto-tuner's candidates stand for include the one that runs without tuning."""
import pytest


@pytest.fixture()
def lib():
    from paper_1811_09736_amd import binding
    binding.set_variant("reset")
    binding.tuning_import("")
    yield binding
    binding.tuning_import("")


@pytest.mark.parametrize("n,seg", [(1 << 17, 0), (100003, 0), ((1 << 17) + 1, 0), (1 << 20, 0), (1 << 23, 0), ((1 << 23) + 1, 0), (1 << 28, 0),
                                   (1 << 20, 1 << 18), (1 << 23, 1 << 18), (1 << 22, 1 << 20), (1 << 24, 1 << 20)])
def test_one_launch_is_among_the_candidates_of_long_reductions(lib, n, seg):
    op, cls = (lib.OP_SEGMENTED_REDUCE, seg.bit_length() - 1) if seg else (lib.OP_REDUCE, 41)
    default = lib.kernel_name(op, n, seg)
    assert ("reduce_final_kernel" not in default) == (n <= 1 << 23)
    names = set()
    for value in range(4):
        lib.tuning_import(f"reduce:{cls}={value};")
        names.add(lib.kernel_name(op, n, seg))
    assert default in names
