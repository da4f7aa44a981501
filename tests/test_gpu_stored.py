"""Steps on stored logits: tiles whose columns are cut into slices, whole rows of 8, 16 and 32 values per thread, rows of which only the
parts with the largest logits are read, against fp64 on the device."""
import ctypes
import re

import pytest
import torch

import paper_2506_22694_amd as vt
from paper_2506_22694_amd import binding

pytestmark = pytest.mark.gpu


def _inputs(n, k, d, seed=0, dtype=torch.bfloat16):
    g = torch.Generator(device="cuda").manual_seed(seed)
    W = torch.randn(k, d, generator=g, device="cuda", dtype=dtype).mul_(0.02)
    h = torch.randn(n, d, generator=g, device="cuda", dtype=dtype)
    # equal rows, in the first and last tile and slot: their logits are equal bit for bit
    same = sorted({0, 63, 64, k // 2, k - 2, k - 1})
    W[same] = W[3].clone()
    return h, W, torch.randperm(2 * k, generator=g, device="cuda")[:k].sort().values.to(torch.int32), same


def _check(h, W, map_, same, m, got, by_id=True):
    ids, logp, lse, full = got
    z = h.double() @ W.double().t()
    ref = z - z.logsumexp(1, keepdim=True)
    # fp32 sums of d products of size 0.02, |logit| <= 20, in up to eight slices and ranges: a few ulp of 20 (2e-6) each
    assert (full - ref).abs().max().item() < 5e-5
    assert (logp - ref.topk(m, 1).values).abs().max().item() < 5e-5
    assert (lse - z.logsumexp(1)).abs().max().item() < 5e-5
    dup = full[:, torch.tensor(same, device="cuda")]
    assert torch.equal(dup, dup[:, :1].expand_as(dup))
    # the tokens are those of the step's own logits, equal ones in ascending order of their ids
    order = torch.sort(full, dim=1, descending=True, stable=True).indices[:, :m]
    assert torch.equal(logp, torch.gather(full, 1, order))
    if by_id:
        assert torch.equal(ids, map_[order])
    else:      # (large logits, or many, differ by less than the rounding of their log-probs: which of those comes first is in the logits alone)
        at = torch.searchsorted(map_, ids)
        assert torch.equal(map_[at], ids) and torch.equal(torch.gather(full, 1, at), logp)
        assert all(len(set(row)) == m for row in ids.tolist())


# Slices: the kernels' ranges of hidden rows and their edges, tiles of 64, 128 and 160 rows, two to eight slices of equal and of
# unequal length, slices whole multiples of 4 KiB apart (which have ranges of their own), ragged last tiles, k on and off multiples
# of four, h re-laid, rows of one, two and four stretches of 4096 logits
@pytest.mark.parametrize("n,k,d,m,slices,tile", [
    (9, 4300, 8192, 8, 7, 128), (32, 4097, 8192, 4, 7, 128), (33, 6001, 8192, 10, 5, 128), (64, 5002, 8192, 16, 6, 128),
    (65, 4303, 4096, 8, 7, 128), (128, 8193, 3072, 1, 3, 128), (129, 4096, 2048, 8, 4, 64), (160, 10001, 4096, 4, 3, 128),
    (192, 6500, 4096, 10, 5, 128), (193, 5000, 8192, 4, 6, 128), (224, 14000, 8192, 8, 2, 128), (256, 14001, 8192, 16, 2, 128),
    (256, 4100, 8064, 8, 7, 128), (256, 9999, 5248, 33, 3, 128), (100, 4096, 8192, 64, 4, 64), (250, 2050, 2048, 8, 7, 64),
    (128, 11900, 8192, 9, 3, 160), (300, 4300, 4096, 8, 3, 64)])
def test_step_by_slices_of_the_columns(n, k, d, m, slices, tile):
    plan = vt.draft_head_step_plan(n, k, d, m)
    assert f"tile_rows={tile} " in plan and f"column_slices={slices} + row_select" in plan, plan
    h, W, map_, same = _inputs(n, k, d, seed=n + k)
    _check(h, W, map_, same, m, vt.draft_head_step(h, W, map_, m, return_lse=True, return_full=True))


# Slices add up no longer chains than the tiles in one piece that a smaller workspace has: no larger error (of 500 and more log-probs, whose
# errors' 2-norm is known to a few percent; a chain twice as long has 1.4 to 2 times the error)
@pytest.mark.parametrize("n,k,d,m", [(126, 5389, 8192, 4), (200, 14066, 8192, 4), (224, 4300, 4096, 4), (136, 12835, 8192, 4), (250, 7000, 8192, 4),
                                     (256, 9000, 6144, 8)])
def test_slices_are_as_close_to_fp64_as_one_piece(n, k, d, m):
    assert "column_slices" in vt.draft_head_step_plan(n, k, d, m)
    h, W, map_, _ = _inputs(n, k, d, seed=k)
    z = h.double() @ W.double().t()
    top = (z - z.logsumexp(1, keepdim=True)).topk(m, 1).values
    ws, L = vt.StepWorkspace(n, k, d, m, h.device), vt.load_library()
    a, b = torch.empty((n, m), dtype=torch.int32, device="cuda"), torch.empty((n, m), device="cuda")
    step = lambda size: L.vt_draft_head_step(h.data_ptr(), 1, n, W.data_ptr(), 1, k, d, map_.data_ptr(), m, a.data_ptr(), b.data_ptr(), None, None,
                                             ws.buf.data_ptr(), size, torch.cuda.current_stream().cuda_stream)
    lo, hi = 0, ws.nbytes // 256
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if step(256 * mid) == 0 else (mid, hi)
    error = []
    for size in (256 * hi, ws.nbytes):
        assert step(size) == 0
        error.append((b - top).norm().item())
    assert error[1] < 1.2 * error[0]


# Stored logits that are read in whole rows: of 8, 16 and 32 values per thread and their edges, of two stretches and more, k on and off
# multiples of four, fewer groups of four than threads, more logits than candidates (hidden row of zeros).  Up to 8 hidden rows of heads that
# are not read by parts; more of them with the smallest workspace that is accepted, which has no room for the parts (up to 8 tokens
# it keeps lists)
@pytest.mark.parametrize("n,k,d,m", [
    (3, 8191, 128, 20), (8, 8192, 256, 16), (4, 8193, 128, 24), (2, 16384, 128, 16), (8, 16381, 128, 64), (5, 16385, 256, 17), (6, 32768, 128, 40),
    (8, 32767, 128, 20),
    (4, 3000, 1024, 16), (3, 4092, 128, 33), (7, 4096, 128, 17), (3, 2060, 256, -16), (8, 3840, 512, -64),
    (24, 8192, 128, 16), (24, 8193, 256, 9), (20, 16384, 128, 10), (17, 16385, 128, 12), (40, 16381, 128, 64), (33, 32768, 128, 16),
    (40, 3000, 128, 33), (9, 131073, 128, 64), (9, 65, 128, 64), (40, 66, 128, 9), (64, 651, 128, 33), (9, 1023, 256, 64), (24, 1025, 128, 10), (150, 961, 128, 33),
    (64, 7168, 128, 16), (65, 4608, 128, 9),
    (24, 65537, 128, 16), (100, 50000, 128, 9), (200, 4099, 256, 8), (70, 4100, 1024, 8), (256, 9000, 1024, 8)])
def test_stored_logits_in_whole_rows(n, k, d, m):
    dtype, m = (torch.float32, -m) if m < 0 else (torch.bfloat16, m)
    plan = vt.draft_head_step_plan(n, k, d, m, dtype)
    h, W, map_, same = _inputs(n, k, d, seed=k, dtype=dtype)
    h[n // 2] = 0
    if n <= 8:
        assert plan.endswith("row_select_kernel") and "slices" not in plan, plan
    ws, L = vt.StepWorkspace(n, k, d, m, h.device), vt.load_library()
    ids, logp = torch.empty((n, m), dtype=torch.int32, device="cuda"), torch.empty((n, m), device="cuda")
    lse, full = torch.empty(n, device="cuda"), torch.empty((n, k), device="cuda")
    code = int(dtype == torch.bfloat16)
    step = lambda size: L.vt_draft_head_step(h.data_ptr(), code, n, W.data_ptr(), code, k, d, map_.data_ptr(), m,
                                             ids.data_ptr(), logp.data_ptr(), lse.data_ptr(), full.data_ptr(), ws.buf.data_ptr(), size,
                                             torch.cuda.current_stream().cuda_stream)
    lo, hi = 0, ws.nbytes // 256
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if step(256 * mid) == 0 else (mid, hi)
    if n > 8 and m > 8:
        parts = re.search(r"row_select_parts_kernel parts=(\d+)$", plan)
        assert 256 * hi < 4 * n * k + 8 * n * (int(parts[1]) if parts else 8192), (plan, hi)
    for size in (256 * hi, ws.nbytes):
        full.fill_(7.0)
        assert step(size) == 0
        _check(h, W, map_, same, m, (ids, logp, lse, full), by_id=k < 50000)      # (see there)


# Heads for tiles of 129 to 139 rows: the logits of such a tile, and of the last one, end inside a group of four.  With all of the
# workspace, and with the smallest that is accepted (tiles of just that many rows)
@pytest.mark.parametrize("n,k,d,m,tile", [(17, 33008, 256, 16, 129), (40, 33280, 128, 10, 130), (12, 35328, 128, 9, 138), (64, 35364, 128, 16, 139)])
def test_stored_logits_of_tiles_that_are_no_multiple_of_four(n, k, d, m, tile):
    plan = vt.draft_head_step_plan(n, k, d, m)
    assert f"tile_rows={(tile + 3) // 4 * 4} " in plan and "row_select" in plan, plan
    h, W, map_, same = _inputs(n, k, d, seed=k)
    # the logits' buffer is the caller's: what lies behind it stays
    full = torch.full((n * k + 64,), 7.0, device="cuda")
    ids, logp, lse = torch.empty((n, m), dtype=torch.int32, device="cuda"), torch.empty((n, m), device="cuda"), torch.empty(n, device="cuda")
    ws, L = vt.StepWorkspace(n, k, d, m, h.device), vt.load_library()
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    step = lambda size: L.vt_draft_head_step(p(h), 1, n, p(W), 1, k, d, p(map_), m, p(ids), p(logp), p(lse), p(full), p(ws.buf),
                                             ctypes.c_size_t(size), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    lo, hi = 0, ws.nbytes // 256
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if step(256 * mid) == 0 else (mid, hi)
    for size in (256 * hi, ws.nbytes):
        full.fill_(7.0)
        assert step(size) == 0
        assert bool((full[n * k:] == 7.0).all())
        _check(h, W, map_, same, m, (ids, logp, lse, full[:n * k].view(n, k)))


# Stored logits of which only the parts with the largest are read: both kernels and every tile height, tiles of 132 to 144 rows, last
# tiles of one row and of one part, one, two and eight parts per thread, fewer parts than waves, rows off multiples of four, rounds,
# two workgroups to a CU, h re-laid; up to 8 rows both kernels, their parts of 64 and shorter ones.  And the same inputs by slices, and with
# more parts than the kernel takes.  Hidden row 0 has 1500 large logits side by side (more than the candidates' room where the parts
# beside them set the threshold), hidden row 1 is zero (all logits tie)
@pytest.mark.parametrize("n,k,d,m,each", [
    (9, 130, 128, 9, 0), (10, 4097, 256, 16, 0), (33, 8200, 128, 64, 1), (64, 12289, 128, 10, 1), (20, 20001, 128, 33, 2), (40, 26001, 256, 16, 2),
    (12, 33008, 256, 10, 8), (64, 36865, 128, 64, 8), (17, 44003, 128, 12, 8), (24, 65537, 128, 16, 8), (64, 100001, 128, 9, 8),
    (9, 131072, 128, 64, 8), (65, 7000, 128, 8, 1), (76, 4100, 1024, 7, 1), (128, 12001, 128, 1, 1), (129, 16383, 256, 8, 1),
    (150, 20002, 128, 64, 1), (192, 32768, 256, 8, 1), (193, 30001, 128, 5, 1), (256, 32767, 128, 64, 1), (200, 40001, 128, 16, 1),
    (256, 70001, 128, 9, 1), (256, 24000, 8192, 16, 1), (2, 16385, 512, 16, 1), (8, 33008, 1024, 16, 1), (3, 33013, 4096, 12, 1),
    (5, 50204, 1024, 16, 1), (2, 131075, 256, 64, 8), (2, 40000, 2304, 33, 1), (4, 100000, 128, 33, 2), (3, 20003, 256, -16, 1),
    (12, 8192, 128, 16, 1), (12, 8193, 256, 9, 1), (9, 16381, 128, 64, 1),
    (256, 5000, 8192, 33, 0), (9, 131073, 128, 64, 0)])
def test_stored_logits_by_parts(n, k, d, m, each):
    dtype, m = (torch.float32, -m) if m < 0 else (torch.bfloat16, m)      # (up to 8 rows: both element types)
    plan = vt.draft_head_step_plan(n, k, d, m, dtype)
    parts = re.search(r" \+ row_select_parts_kernel parts=(\d+)$", plan)
    assert "row_select" in plan and (parts is None if each == 0 else {1: 0, 2: 1024, 8: 2048}[each] < int(parts[1]) <= 1024 * each), plan
    h, W, map_, same = _inputs(n, k, d, seed=n + m, dtype=dtype)
    h[1] = 0
    lo = k // 3 // 4 * 4
    W[lo:lo + 1500] += (0.1 * h[0].float() / h[0].float().norm()).to(W.dtype)
    W[same] = W[3].clone()
    ids, logp, lse, full = vt.draft_head_step(h, W, map_, m, return_lse=True, return_full=True)
    _check(h, W, map_, same, m, (ids, logp, lse, full), by_id=False)
    assert torch.equal(ids[1], map_[:m])
    plain = vt.draft_head_step(h, W, map_, m)
    assert torch.equal(plain[0], ids) and torch.equal(plain[1], logp)


# All logits of a row equal, and as many above: the lowest ids, wherever they lie -- first, last, at random, and away from one wave of
# the workgroup that looks for them (which then has none of the best)
@pytest.mark.parametrize("n,k,d,m,tail", [
    (70, 9000, 128, 8, "parts"), (256, 32768, 128, 16, "parts"), (12, 40004, 128, 64, "parts"), (128, 20001, 128, 8, "parts"), (128, 12001, 128, 1, "parts"),
    (8, 8192, 128, 16, "whole"), (3, 16381, 128, 64, "whole"), (4, 30001, 128, 17, "whole"), (9, 131073, 128, 33, "whole"), (224, 5000, 4096, 4, "slices")])
@pytest.mark.parametrize("order", ["ascending", "descending", "random", "apart"])
def test_equal_logits(n, k, d, m, tail, order):
    plan = vt.draft_head_step_plan(n, k, d, m)
    assert plan.endswith("row_select_kernel") and ("column_slices" in plan) == (tail == "slices") if tail != "parts" else "row_select_parts_kernel" in plan, plan
    h, W, _, same = _inputs(n, k, d)
    h[2:] = 0
    W[:4096] = W[0].clone()      # row 1: 4096 equal logits, and those of `same`
    h[1] = W[0] * 50
    ids = torch.arange(k, device="cuda", dtype=torch.int32)
    if order == "descending":
        ids = ids.flip(0)
    elif order == "random":
        ids = ids[torch.randperm(k, device="cuda")]
    elif order == "apart":
        first = (torch.arange(k, device="cuda") % 1024 < 64).int()
        ids = torch.argsort(torch.argsort(first, stable=True), stable=True).int()
    got, logp = vt.draft_head_step(h, W, ids, m)
    z = h[:2].double() @ W.double().t()
    assert (logp[:2] - (z - z.logsumexp(1, keepdim=True)).topk(m, 1).values).abs().max().item() < 5e-5
    assert torch.equal(got[1], torch.cat([ids[:4096], ids[[j for j in same if j >= 4096]]]).sort().values[:m])
    assert torch.equal(got[2:], torch.arange(m, device="cuda", dtype=torch.int32).expand(n - 2, m))
    assert (logp[2:] + torch.log(torch.tensor(float(k)))).abs().max().item() < 5e-6


# Head rows whose logits are -inf: a whole tile's, the last one's (alone in its part on some of the shapes), and all but three.  Log-sum-exp
# and log-probs are those of the other logits
@pytest.mark.parametrize("n,k,d,m", [
    (9, 16385, 128, 12), (17, 33008, 256, 16), (128, 12001, 128, 1), (256, 32767, 128, 9), (224, 4301, 4096, 4), (2, 33025, 512, 16), (5, 50204, 1024, 16),
    (4, 3000, 1024, 16)])
def test_logits_of_minus_infinity(n, k, d, m):
    assert "row_select" in vt.draft_head_step_plan(n, k, d, m)
    h, W, map_, _ = _inputs(n, k, d, seed=k)
    h[:, 0] = 1
    every = torch.arange(k, device="cuda")
    for gone in ((every >= k // 2) & (every < k // 2 + 512) | (every == k - 1), (every != 5) & (every != k // 3) & (every != k - 1)):
        Wx = W.clone()
        Wx[gone, 0] = -float("inf")
        ids, logp, lse, full = vt.draft_head_step(h, Wx, map_, m, return_lse=True, return_full=True)
        z = h.double() @ Wx.double().t()
        assert (lse - z.logsumexp(1)).abs().max().item() < 5e-5
        ref = z - z.logsumexp(1, keepdim=True)
        for got, want in ((full, ref), (logp, ref.topk(m, 1).values)):
            there = want > -float("inf")
            assert torch.equal(got > -float("inf"), there) and not bool(got.isnan().any())
            assert (got - want)[there].abs().max().item() < 5e-5
        # (what is left of m tokens is -inf, in ascending order of their ids)
        order = torch.sort(full, dim=1, descending=True, stable=True).indices[:, :m]
        assert torch.equal(ids, map_[order])


# Rows of NaN have tokens of the head for tokens, the lowest ids, as lists give them; so has a row with fewer other logits than tokens.
# One NaN among a row's logits comes where it does with the smallest workspace that is accepted, which may keep lists
@pytest.mark.parametrize("n,k,d,m", [
    (224, 4300, 4096, 4), (20, 4806, 8192, 8), (128, 12001, 128, 8), (217, 26262, 128, 4), (9, 16385, 128, 12), (256, 32767, 128, 64), (24, 65537, 128, 16),
    (2, 33025, 512, 16), (3, 8191, 128, 20), (4, 100000, 128, 33)])
def test_logits_that_are_nan(n, k, d, m):
    assert "row_select" in vt.draft_head_step_plan(n, k, d, m)
    h, W, map_, _ = _inputs(n, k, d, seed=k)
    good = vt.draft_head_step(h, W, map_, m)
    hx = h.clone()
    hx[0] = float("nan")
    hx[n - 1, d // 2] = float("nan")
    out = {"out_ids": torch.full((n, m), -1, dtype=torch.int32, device="cuda"), "out_logp": torch.zeros((n, m), device="cuda")}
    ids, logp = vt.draft_head_step(hx, W, map_, m, **out)
    for i in (0, n - 1):
        assert torch.equal(ids[i], map_[:m]) and bool(logp[i].isnan().all())
    assert torch.equal(ids[1:n - 1], good[0][1:n - 1]) and torch.equal(logp[1:n - 1], good[1][1:n - 1])
    ws, L = vt.StepWorkspace(n, k, d, m, h.device), vt.load_library()
    a, b = torch.empty_like(ids), torch.empty_like(logp)
    for nan in (0x7FC0, 0x7FC0 - 0x8000):      # positive and negative ones
        Wx = W.clone()
        Wx.view(torch.int16)[k // 2] = nan
        out["out_ids"].fill_(-1)
        ids, logp = vt.draft_head_step(h, Wx, map_, m, **out)
        assert bool(logp.isnan().all()) and bool(torch.isin(ids, map_).all())
        assert all(len(set(row)) == m for row in ids.tolist())
        step = lambda size: L.vt_draft_head_step(h.data_ptr(), 1, n, Wx.data_ptr(), 1, k, d, map_.data_ptr(), m, a.data_ptr(), b.data_ptr(), None, None,
                                                 ws.buf.data_ptr(), size, torch.cuda.current_stream().cuda_stream)
        lo, hi = 0, ws.nbytes // 256
        while hi - lo > 1:
            mid = (lo + hi) // 2
            lo, hi = (lo, mid) if step(256 * mid) == 0 else (mid, hi)
        assert step(256 * hi) == 0
        # (logits that agree to rounding may change places)
        assert torch.equal(a == map_[k // 2], ids == map_[k // 2]) and (a != ids).sum().item() <= 2 + ids.numel() // 256
    if m > 1:
        Wx[:] = float("nan")
        Wx[k // 3] = 0
        out["out_ids"].fill_(-1)
        ids, logp = vt.draft_head_step(h, Wx, map_, m, **out)
        assert bool(torch.isin(ids, map_).all()) and all(len(set(row)) == m for row in ids.tolist())


# More than 256 rows run in groups: a whole one that keeps lists and the rest by slices whose logits the library's own 4 MiB do not hold
@pytest.mark.parametrize("n,k,d,m", [(464, 3045, 1280, 9), (588, 2885, 1280, 37), (716, 2696, 1280, 13), (300, 4300, 4096, 4)])
def test_groups_of_rows_on_the_librarys_own_memory(n, k, d, m):
    assert "slices" in vt.draft_head_step_plan(n % 256, k, d, m)
    h, W, map_, same = _inputs(n, k, d, seed=n)
    ids, logp, lse, full = vt.draft_head_step(h, W, map_, m, return_lse=True, return_full=True)
    _check(h, W, map_, same, m, (ids, logp, lse, full))
    a, b = torch.empty_like(ids), torch.empty_like(logp)
    vt.draft_head_step_static(h, W, map_, m, a, b)
    assert torch.equal(a, ids) and torch.equal(b, logp)


# The library's own memory, a tree level, several heads and a workspace of the size that earlier versions asked for
@pytest.mark.parametrize("n,k,d,m", [(224, 4300, 4096, 4), (40, 4300, 8192, 8), (70, 4100, 1024, 8)])
def test_the_other_ways_to_a_stored_step(n, k, d, m):
    assert "row_select" in vt.draft_head_step_plan(n, k, d, m)
    h, W, map_, same = _inputs(n, k, d)
    ids, logp, lse, full = vt.draft_head_step(h, W, map_, m, return_lse=True, return_full=True)
    _check(h, W, map_, same, m, (ids, logp, lse, full))
    plain = vt.draft_head_step(h, W, map_, m)
    assert torch.equal(plain[0], ids) and torch.equal(plain[1], logp)
    a, b = torch.empty_like(ids), torch.empty_like(logp)
    vt.draft_head_step_static(h, W, map_, m, a, b)
    assert torch.equal(a, ids) and torch.equal(b, logp)
    cum = torch.linspace(-3, 0, n, device="cuda")
    parent, token, score, a, b = vt.draft_tree_level(h, W, map_, m, cum, 5)
    assert torch.equal(a, ids) and torch.equal(b, logp)
    for x, y in zip(vt.tree_expand(cum, logp, ids, 5), (parent, token, score)):
        assert torch.equal(x, y)
    a, b = vt.draft_head_step_multi(h, [(W, map_)], [0] * n, m)
    assert torch.equal(a, ids) and torch.equal(b, logp)
    # the smallest workspace that is accepted: the tokens and log-probs are those of its logits, which may round differently
    L, ws = vt.load_library(), vt.StepWorkspace(n, k, d, m, h.device)
    a, b = torch.empty_like(ids), torch.empty_like(logp)
    step = lambda size: L.vt_draft_head_step(h.data_ptr(), 1, n, W.data_ptr(), 1, k, d, map_.data_ptr(), m, a.data_ptr(), b.data_ptr(), None, None,
                                             ws.buf.data_ptr(), ctypes.c_size_t(size), None)
    lo, hi = 0, ws.nbytes // 256
    while hi - lo > 1:
        mid = (lo + hi) // 2
        status = step(256 * mid)
        assert status in (0, 5)
        lo, hi = (lo, mid) if status == 0 else (mid, hi)
    assert step(256 * hi) == 0 and 256 * hi < ws.nbytes and 256 * hi <= binding.VT_STATIC_WS_BYTES
    torch.cuda.synchronize()
    assert (b - logp).abs().max().item() < 5e-5 and (a != ids).sum().item() <= 2 + ids.numel() // 256
