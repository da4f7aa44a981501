"""Draft steps of 9 .. 256 hidden rows at the edges of the kernels that serve them, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2506_22694_amd as vt
from paper_2506_22694_amd import synth
from test_gpu_parity import check_full, check_step, run_step

pytestmark = pytest.mark.gpu


# Tile heights follow from k (ceil(k / 256) rows, in 16-row groups, on 256 CUs); d: two stages only, an odd number of
# them, and 32 (d = 2048, 4096: the start of the march rotates over eight, four or two ranges of columns).
@pytest.mark.parametrize("n,k,d,m,variant", [
    # up to 64 hidden rows: 1 .. 12 row groups, fewer than eight of them with waves that share one, tiles with extra rows
    (9, 300, 128, 4, "<2,8>"), (33, 4096, 256, 8, "<4,8>"), (64, 8000, 128, 8, "<4,8>"), (17, 12000, 640, 5, "<2,8>"),
    (64, 16384, 2048, 8, "<4,8>"), (32, 20000, 256, 8, "<2,7>"), (64, 24576, 128, 8, "<4,7>"), (12, 28672, 128, 3, "<2,7>"),
    (64, 32768, 256, 16, "<4,8>"), (31, 32769, 128, 8, "<2,8>"), (64, 36864, 384, 8, "<4,8>"), (64, 40960, 128, 8, "<4,12>"),
    (33, 45056, 256, 2, "<4,12>"), (32, 49152, 128, 8, "<2,12>"), (64, 49153, 128, 8, "<4,"), (20, 70001, 256, 4, "<2,"),
    # 65 .. 256: two, three and four columns of hidden rows, 32 .. 160 tile rows, two epilogue passes, h re-laid
    (65, 31, 128, 8, "wide_kernel<1>"), (128, 5000, 256, 8, "wide_kernel<1>"), (100, 16384, 2048, 8, "wide_kernel<1>"),
    (129, 16000, 384, 4, "wide_kernel<2>"), (192, 24576, 128, 6, "wide_kernel<2>"), (193, 3000, 4096, 2, "wide_kernel<2>"),
    (160, 9000, 2048, 8, "wide_kernel<2>"), (80, 40960, 128, 8, "wide_kernel<1>"), (250, 40960, 128, 4, "wide_kernel<2>"),
    (256, 33000, 128, 16, "wide_kernel<2>"), (256, 600, 8192, 4, "pack_h_kernel + head_mfma_wide_kernel<2>"),
])
def test_step_many_rows_at_the_edges_of_the_tiles(n, k, d, m, variant):
    assert variant in vt.draft_head_step_plan(n, k, d, m)
    W, map_ = synth.trimmed_head_direct(k, d, seed=700 + n, dtype="bf16")
    h = synth.hidden_rows(n, d, seed=800 + k, dtype="bf16")
    # equal rows in other tiles, row groups and at the ragged end: equal logits, bit for bit, whatever the start of the march
    same = sorted({j for j in (3, 19, 128, 143, k // 2, k - 17, k - 1) if 0 <= j < k})
    W[same] = W[same[0]]
    ref = oracle.draft_head_step(h, W, map_, m)
    oi, ol, lse, full = run_step(h, W, map_, m, return_lse=True, return_full=True)
    assert check_step(oi, ol, ref, map_, m, lse) <= 2 + n // 32
    check_full(full, ref)
    dup = full[:, torch.tensor(same, device=full.device)]
    assert torch.equal(dup, dup[:, :1].expand_as(dup))
    oi2, ol2 = run_step(h, W, map_, m)
    assert torch.equal(oi, oi2) and torch.equal(ol, ol2)


def test_step_many_rows_captured_in_a_graph_replays_the_same():
    cases = []
    for n, k, d, m in ((40, 5000, 512, 8), (100, 3000, 2048, 4), (256, 700, 8192, 16)):
        W, map_ = synth.trimmed_head_direct(k, d, seed=31, dtype="bf16")
        h = torch.randn(n, d, device="cuda").bfloat16()
        W = torch.from_numpy(W.view(np.int16)).cuda().view(torch.bfloat16)
        out = (torch.empty(n, m, dtype=torch.int32, device="cuda"), torch.empty(n, m, device="cuda"))
        cases.append((h, W, torch.from_numpy(map_).cuda(), m, vt.StepWorkspace(n, k, d, m, h.device), out))
    step = lambda c: vt.draft_head_step(*c[:4], ws=c[4], out_ids=c[5][0], out_logp=c[5][1])
    for c in cases:
        step(c)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for c in cases:
            step(c)
    for rep in range(4):
        for c in cases:
            c[0].copy_(torch.randn_like(c[0]))
        g.replay()
        got = [[t.clone() for t in c[5]] for c in cases]
        for c, (ids, logp) in zip(cases, got):
            step(c)
            torch.cuda.synchronize()
            assert torch.equal(c[5][0], ids) and torch.equal(c[5][1], logp), rep


# Merges by eight waves: keys per thread 8 / 16 / 32 (512 lists of four; 513, 1002 lists; 2048, all that the merge holds), the edge
# of 256 lists that one wave could hold, one token, and a row whose logits are all equal (more candidates than the merge holds).
@pytest.mark.parametrize("n,k,m,lists", [
    (9, 65537, 8, 513), (64, 65536, 4, 512), (12, 128256, 8, 1002), (17, 262144, 8, 2048), (10, 49153, 1, 385), (33, 49280, 8, 385),
    (70, 40961, 8, 427), (64, 32768, 8, 256), (20, 32640, 8, 255)])
def test_merge_of_many_lists(n, k, m, lists):
    assert f"workgroups={lists} " in vt.draft_head_step_plan(n, k, 128, m)
    W, map_ = synth.trimmed_head_direct(k, 128, seed=900 + n, dtype="bf16")
    h = synth.hidden_rows(n, 128, seed=k, dtype="bf16")
    h[n // 2] = 0
    ref = oracle.draft_head_step(h, W, map_, m)
    oi, ol, lse = run_step(h, W, map_, m, return_lse=True)
    assert check_step(oi, ol, ref, map_, m, lse) <= 2 + n // 32
    assert oi[n // 2].tolist() == sorted(map_)[:m]
    if n * m <= 512:        # the same merge with a tree level behind it
        put = lambda a: torch.from_numpy(a.view(np.int16)).cuda().view(torch.bfloat16)
        cum = torch.linspace(0.0, -1.0, n, device="cuda")
        K = min(8, n * m)
        got = vt.draft_tree_level(put(h), put(W), torch.from_numpy(map_).cuda(), m, cum, K)
        want = vt.tree_expand(cum, ol, oi, K)
        for a, b in zip(got, want):
            assert torch.equal(a, b)


def test_merge_of_many_lists_with_more_tokens_than_waves():
    n, k, d, m = 8, 100352, 6400, 11
    assert "mfma" in vt.draft_head_step_plan(n, k, d, m)
    W = torch.randn(k, d, device="cuda", dtype=torch.bfloat16)
    h = torch.randn(n, d, device="cuda").mul_(0.02).bfloat16()
    map_ = torch.arange(k, dtype=torch.int32, device="cuda") * 2
    ids, logp = vt.draft_head_step(h, W, map_, m)
    z = torch.cat([h.double() @ W[a:a + 8192].double().t() for a in range(0, k, 8192)], 1)
    top = (z - z.logsumexp(1, keepdim=True)).topk(m, 1)
    # fp32 sums of 6400 products of size |h| |w| ~ 0.02: far below 1e-4; neighbours closer than that may swap
    assert (logp - top.values).abs().max().item() < 1e-4
    assert (ids.long() != 2 * top.indices).sum().item() <= 2


# Rows of stored logits longer than one stretch of 32768: a second stretch of one logit, whole stretches, a ragged fifth;
# more tokens than waves; `late`: the first stretch's logits say nothing about the rest, which overflows the collection
# (the row is read again); a row whose logits are all equal.
@pytest.mark.parametrize("n,k,m,late", [
    (9, 32769, 16, False), (10, 65536, 16, False), (9, 131076, 64, False), (12, 98304, 10, True), (9, 40001, 33, True),
    (16, 65536, 16, True)])
def test_stored_logits_longer_than_one_stretch(n, k, m, late):
    assert "row_select" in vt.draft_head_step_plan(n, k, 128, m)
    W, map_ = synth.trimmed_head_direct(k, 128, seed=1000 + n, dtype="bf16")
    if late:
        W[:32768] = 0
    h = synth.hidden_rows(n, 128, seed=k, dtype="bf16")
    h[n // 2] = 0
    ref = oracle.draft_head_step(h, W, map_, m)
    oi, ol, lse = run_step(h, W, map_, m, return_lse=True)
    assert check_step(oi, ol, ref, map_, m, lse) <= 2 + n * m // 256
    assert oi[n // 2].tolist() == sorted(map_)[:m]


# Two workgroups to a CU (heads of several rounds of tiles): just past one round, a ragged second round, rotated starts (d a
# multiple of 2048) with two groups of hidden rows and with four; equal rows in tiles of all eight starts
@pytest.mark.parametrize("n,k,d,m", [
    (9, 49153, 128, 8), (33, 60001, 128, 16), (32, 65536, 2048, 8), (64, 65536, 2048, 8), (20, 50000, 4096, 4), (64, 50000, 4096, 16)])
def test_step_of_several_rounds_of_tiles(n, k, d, m):
    plan = vt.draft_head_step_plan(n, k, d, m)
    assert "tile_rows=128 waves=8" in plan and "workgroups_per_cu=2" in plan
    W, map_ = synth.trimmed_head_direct(k, d, seed=1100 + n, dtype="bf16")
    h = synth.hidden_rows(n, d, seed=k, dtype="bf16")
    tiles = [0, 1, 8, 24, 40, 56, 255, 256, k // 128 - 1]
    assert {(b // 8 + b // 64) % 8 for b in tiles} >= {0, 1, 2, 3, 4, 5, 7}
    same = [128 * b + (37 * b) % 128 for b in tiles] + [k - 1]
    W[same] = W[same[0]]
    ref = oracle.draft_head_step(h, W, map_, m)
    oi, ol, lse, full = run_step(h, W, map_, m, return_lse=True, return_full=True)
    assert check_step(oi, ol, ref, map_, m, lse) <= 2 + n // 32
    check_full(full, ref)
    dup = full[:, torch.tensor(same, device=full.device)]
    assert torch.equal(dup, dup[:, :1].expand_as(dup))


# 4 MiB of h and more with 65 .. 192 hidden rows (h is read in place there), at the threshold, and a last group of that many
@pytest.mark.parametrize("n,k,d,m", [(127, 600, 16384, 4), (128, 600, 16384, 8), (192, 500, 12288, 4), (400, 300, 16384, 4)])
def test_step_of_many_long_rows(n, k, d, m):
    W, map_ = synth.trimmed_head_direct(k, d, seed=1200 + n, dtype="bf16")
    h = synth.hidden_rows(n, d, seed=k, dtype="bf16")
    same = [3, 140, k - 1]
    W[same] = W[same[0]]
    ref = oracle.draft_head_step(h, W, map_, m)
    oi, ol, lse, full = run_step(h, W, map_, m, return_lse=True, return_full=True)
    assert check_step(oi, ol, ref, map_, m, lse) <= 2 + n // 32
    check_full(full, ref)
    dup = full[:, torch.tensor(same, device=full.device)]
    assert torch.equal(dup, dup[:, :1].expand_as(dup))


# Ranges of columns that would start whole multiples of 4 KiB apart are cut unequally, in several rotations: four (d a multiple
# of 8192, tiles of 96, 128 and 160 rows), eight (d a multiple of 16384: stages of one block and of two, extra rows, twin tiles)
@pytest.mark.parametrize("n,k,d,m,rows,kernel", [
    (160, 24000, 8192, 8, 96, "wide_kernel<2>"), (190, 32000, 8192, 8, 128, "wide_kernel<2>"), (70, 39000, 8192, 8, 160, "wide_kernel<1>"),
    (9, 9000, 16384, 8, 48, "<2,8>"), (40, 20000, 16384, 8, 128, "<4,8>"), (20, 33000, 16384, 8, 129, "<2,8>"), (70, 8000, 16384, 4, 32, "wide_kernel<1>"),
    (16, 12000, 32768, 8, 48, "<2,8>"), (64, 24000, 16384, 8, 96, "<4,7>")])
def test_step_with_unequal_ranges_of_columns(n, k, d, m, rows, kernel):
    plan = vt.draft_head_step_plan(n, k, d, m)
    assert kernel in plan and f"tile_rows={rows} " in plan, plan
    g = torch.Generator(device="cuda").manual_seed(n)
    W = torch.randn(k, d, generator=g, device="cuda", dtype=torch.bfloat16).mul_(0.02)
    h = torch.randn(n, d, generator=g, device="cuda", dtype=torch.bfloat16)
    same = [b * rows + 5 for b in (0, 8, 16, 24, 32, 40, 48, 56, 72) if b * rows + 5 < k] + [k - 1]
    W[same] = W[same[0]].clone()
    map_ = torch.arange(k, dtype=torch.int32, device="cuda")
    ids, logp, lse, full = vt.draft_head_step(h, W, map_, m, return_lse=True, return_full=True)
    z = torch.cat([h.double() @ W[a:a + 4000].double().t() for a in range(0, k, 4000)], 1)
    ref = z - z.logsumexp(1, keepdim=True)
    # fp32 sums of d products of size 0.02, |logit| <= 20: a few ulp of 20 (2e-6) per range and of the log-sum-exp
    assert (full - ref).abs().max().item() < 5e-5
    assert (logp - ref.topk(m, 1).values).abs().max().item() < 5e-5
    dup = full[:, torch.tensor(same, device="cuda")]
    assert torch.equal(dup, dup[:, :1].expand_as(dup))


# The same with up to 8 hidden rows and more than 16 tokens (rows read twice): small kernels, whole and ragged stretches, equal logits
@pytest.mark.parametrize("n,k,m,late", [(1, 32769, 64, False), (8, 65536, 17, False), (3, 98309, 33, True), (2, 131072, 64, True), (5, 40000, 16, True)])
def test_stored_logits_of_few_rows_longer_than_one_stretch(n, k, m, late):
    assert "row_select" in vt.draft_head_step_plan(n, k, 128, m)
    W, map_ = synth.trimmed_head_direct(k, 128, seed=1300 + n, dtype="bf16")
    if late:
        W[:32768] = 0
    h = synth.hidden_rows(n, 128, seed=k, dtype="bf16")
    if n > 1:
        h[n // 2] = 0
    ref = oracle.draft_head_step(h, W, map_, m)
    oi, ol, lse = run_step(h, W, map_, m, return_lse=True)
    assert check_step(oi, ol, ref, map_, m, lse) <= 2 + n * m // 256
    if n > 1:
        assert oi[n // 2].tolist() == sorted(map_)[:m]
