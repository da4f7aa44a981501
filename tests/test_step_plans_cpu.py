"""Plans and workspace sizes of the draft step, which are pure host functions (no device here: 256 CUs are assumed)."""
import ctypes
import time

import pytest
import torch

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


# Rows of 16 MiB and more are refused before anything is launched: offsets inside a tile are 32-bit (24-bit factors up to 8 rows)
@pytest.mark.parametrize("n", [9, 64, 65, 200, 256])
def test_rows_too_long_for_the_offsets_inside_a_tile_are_refused(lib, n):
    A = ctypes.c_void_p(0x10000)
    lib.vt_last_device_error.restype = ctypes.c_char_p
    d = 1 << 23
    step = lambda dd: lib.vt_draft_head_step(A, 1, n, A, 1, 300, dd, A, 4, A, A, None, None, A, ctypes.c_size_t(1 << 60), None)
    assert step(d) == 6 and b"invalid argument" in lib.vt_last_device_error()
    if not torch.cuda.is_available():      # (never launched on the fake addresses where there is a device)
        assert step(d - 128) == 6 and b"invalid argument" not in lib.vt_last_device_error()


# A step without a workspace of its own asks for the size in every call: a shape's second answer takes no plans (20 us of them for 256 rows)
def test_the_size_of_a_workspace_is_kept(lib):
    def microseconds(*shape):
        best = 1e9
        for _ in range(20):
            start = time.perf_counter()
            for _ in range(100):
                lib.vt_draft_head_step_ws_bytes(*shape)
            best = min(best, time.perf_counter() - start)
        return best * 1e4
    smallest = microseconds(1, 1000, 128, 1)
    for shape in ((256, 4300, 4096, 8), (256, 32768, 8192, 16), (64, 32768, 4096, 8)):
        assert microseconds(*shape) < 4 * smallest


# 65 and more rows with few tokens: lists, or logits by parts; logits that are read in whole rows lose to both
@pytest.mark.parametrize("n,k,d,m", [(70, 809, 2048, 4), (91, 450, 4096, 3), (79, 733, 1024, 6), (100, 4100, 1024, 4), (105, 306, 1024, 3), (128, 12001, 128, 8),
                                     (72, 2846, 1024, 5), (69, 467, 5120, 6)])
def test_small_heads_do_not_store_logits_to_read_whole_rows(lib, n, k, d, m):
    rc, text = _plan(lib, n, k, d, m)
    assert rc == 0 and (text.endswith("step_finalize_kernel") or "row_select_parts_kernel" in text), text


# More than 8 rows: heads so short that a thread has eight of a row's logits at most are read whole, longer ones by parts (n = 9, k = 1293, d = 1024, m = 64
# took 1.28 times as long by parts, n = 24, k = 700 1.6)
@pytest.mark.parametrize("n,k,m,whole", [(9, 1293, 64, True), (24, 700, 33, True), (64, 7168, 16, True), (64, 7169, 16, False), (64, 8192, 64, False), (65, 4608, 10, True),
                                         (65, 4609, 64, False), (128, 4501, 16, False), (128, 4501, 33, False), (128, 4501, 48, True), (256, 3000, 16, True)])
def test_short_rows_of_stored_logits_are_read_whole(lib, n, k, m, whole):
    rc, text = _plan(lib, n, k, 512, m)
    assert rc == 0 and text.endswith(" + row_select_kernel" if whole else f" parts={text.rpartition('=')[2]}") and "slices" not in text, text
