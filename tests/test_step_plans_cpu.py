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


# A workspace made for n rows serves any step of fewer, from 8 on: across the kernels' ranges (8 | 9, 32 | 33, 64 | 65, 256 | 257),
# and between rows whose lists keep within the library's own 4 MiB on small tiles and rows whose lists do not
@pytest.mark.parametrize("k,d,m", [
    (48500, 4096, 8), (41000, 4096, 4), (48170, 3968, 4), (41858, 7168, 5), (43545, 2816, 5), (38023, 7808, 7), (40759, 6016, 8),
    (21171, 7040, 16), (23606, 4992, 10), (27841, 6144, 33), (32768, 4096, 8), (128256, 3072, 8), (5000, 16384, 8), (64, 13824, 1),
    (261039, 8064, 11), (5205, 18816, 64), (3000, 1000, 16), (18000, 516, 9)])
def test_a_workspace_for_many_rows_serves_fewer(lib, k, d, m):
    sizes = [lib.vt_draft_head_step_ws_bytes(n, k, d, m) for n in [*range(8, 301), 400, 512, 513, 600]]
    assert sizes[0] > 0 and sizes == sorted(sizes)


def test_lists_that_keep_within_the_librarys_own_workspace_still_do(lib):
    own = 4 << 20
    for n, k, d, m in ((112, 48500, 4096, 8), (127, 48500, 4096, 8), (241, 41000, 4096, 4), (64, 65536, 4096, 8)):
        assert 0 < lib.vt_draft_head_step_ws_bytes(n, k, d, m) <= own
