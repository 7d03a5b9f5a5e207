"""bench.py's names of the step kernels (no GPU)."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402


def test_step_kernel_and_its_block_whatever_the_block_size_setting():
    """Kernels whose wavefronts share a list have blocks of their own; the
    setting is that of the others."""
    for wg in (64, 128, 256):
        assert bench.kernel_name("fp64", 0, wg) == "k_force_fp64<false,true,4>"
        assert bench.kernel_threads("fp64", 0, wg) == 256
        assert bench.kernel_name("mixed_fixed", 0, wg) == "k_force_split<true,false,true,2>"
        assert bench.kernel_threads("mixed_fixed", 0, wg) == 128
        assert bench.kernel_threads("mixed_fixed", 1, wg) == wg
        assert bench.kernel_threads("mixed", 0, wg) == wg
