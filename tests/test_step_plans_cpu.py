"""Plans and workspace sizes of the draft step, which are pure host functions (no device here: 256 CUs are assumed)."""
import ctypes

import pytest

from test_boundary_cpu import _plan, lib  # noqa: F401  (lib: a fixture)


# h is re-laid by the kernels for more than 192 hidden rows alone: around 4 MiB of h
@pytest.mark.parametrize("n,d,packs", [
    (127, 16384, False), (128, 16384, False), (129, 16384, False), (171, 12288, False), (192, 16384, False), (192, 32768, False),
    (193, 10752, False), (193, 10880, True), (256, 8192, True), (255, 8192, False), (256, 16384, True), (65, 65536, False)])
def test_only_a_kernel_that_reads_a_re_laid_h_is_given_one(lib, n, d, packs):
    rc, text = _plan(lib, n, 5000, d, 8)
    assert rc == 0 and text.startswith("pack_h_kernel + head_mfma_wide_kernel<2>" if packs else "head_mfma_wide_kernel<"), text
