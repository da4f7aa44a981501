"""The merge of up to 256 candidate lists per hidden row (one wave), where the best tokens lie unevenly among the lists."""
import numpy as np
import pytest
import torch

import oracle
import paper_2506_22694_amd as vt
from paper_2506_22694_amd import synth
from test_gpu_parity import check_step, run_step

pytestmark = pytest.mark.gpu


# `best` neighbouring tokens far above the field, from token `at` on: all of them in one list (ranks past the third or fourth of a list
# are read only then), across two lists, in the last one; lists of every length and parity; heads of one list, of 39 and of 256
@pytest.mark.parametrize("k,d", [(30, 128), (5000, 256), (32768, 128)])
@pytest.mark.parametrize("m", [1, 2, 3, 4, 5, 7, 8, 10, 11])
def test_best_tokens_in_few_lists(k, d, m):
    n = 2
    W, map_ = synth.trimmed_head_direct(k, d, seed=40 + m, dtype="bf16")
    h = synth.hidden_rows(n, d, seed=k, dtype="bf16")
    put = lambda a: torch.from_numpy(np.asarray(a).view(np.int16)).cuda().view(torch.bfloat16)
    hd = put(h).float().sum(0)
    for at, best in ((0, 11), (k // 2 - 5, 11), (k - 9, 9), (3, 2)):
        Wd = put(W)
        # logits 6, 6.5, .. for both hidden rows (up to rounding and their scalar product); the other tokens' are below 2
        Wd[at:at + best] = (hd * torch.arange(6, 6 + best / 2, 0.5, device="cuda").unsqueeze(1) / d).bfloat16()
        V = Wd.view(torch.int16).cpu().numpy().view(W.dtype)
        ref = oracle.draft_head_step(h, V, map_, m)
        ids, logp, lse = run_step(h, V, map_, m, return_lse=True)
        assert check_step(ids, logp, ref, map_, m, lse) == 0


# A small head beside a large one: the rows of either find their lists next to each other among empty ones
@pytest.mark.parametrize("ks", [(30000, 300), (300, 30000), (8, 20000), (16384, 16000)])
def test_lists_of_two_heads_merge_like_one_heads(ks):
    n, d, m = 8, 256, 8
    g = torch.Generator(device="cuda").manual_seed(ks[0])
    heads = [(torch.randn(k, d, generator=g, device="cuda").mul_(0.1).bfloat16(), torch.arange(k, dtype=torch.int32, device="cuda")) for k in ks]
    h = torch.randn(n, d, generator=g, device="cuda").bfloat16()
    which = [0, 1] * 4
    assert "heads=2" in vt.draft_head_step_multi_plan(n, d, ks, which, m)
    ids, logp, lse = vt.draft_head_step_multi(h, heads, which, m, return_lse=True)
    for i, q in enumerate(which):
        one_ids, one_logp = vt.draft_head_step(h[i:i + 1].expand(2, d).contiguous(), heads[q][0], heads[q][1], m)
        assert torch.equal(ids[i], one_ids[0])
        assert (logp[i] - one_logp[0]).abs().max().item() <= 4e-6      # sums over other tiles: a few ulp of a log-sum-exp near 10


# Logits of two values and many ties: whole tiles reach the threshold of a tile's selection (64, 128 or 144 candidates at once), and the
# better value lies in runs that end at the edges of tiles; up to four hidden rows share a row's work between two waves
@pytest.mark.parametrize("dtype,k,d", [("bf16", 130, 128), ("bf16", 5000, 256), ("bf16", 32767, 128), ("bf16", 128256, 3072), ("f32", 1024, 128), ("f32", 7001, 128)])
@pytest.mark.parametrize("n", [1, 3, 4, 5, 8])
@pytest.mark.parametrize("m", [4, 7, 11])
def test_ties_in_whole_tiles(dtype, k, d, n, m):
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(k + n)
    h = torch.ones(n, d, dtype=t, device="cuda")
    high = torch.rand(k, generator=g, device="cuda") < 0.5
    high[k // 2:] = False
    high[:min(k, 200)] = True
    level = torch.where(high, 2.0, -1.0)                        # (exact in bf16, and so are the sums over powers of two of columns)
    W = (level / 128).unsqueeze(1).expand(k, d).to(t).contiguous()
    z = (level.double() * d / 128)
    map_ = torch.arange(k, dtype=torch.int32, device="cuda") * 2 + 1
    ids, logp, lse = vt.draft_head_step(h, W, map_, m, return_lse=True)
    order = torch.sort(z, descending=True, stable=True).indices[:m]
    want = torch.logsumexp(z, 0)
    assert torch.equal(ids, map_[order].expand(n, m))           # equal logits: the smaller id first
    # sums of up to 128256 exponentials in fp32: a few ulp of a log-sum-exp below 64
    assert (lse.double() - want).abs().max().item() <= 2e-5
    assert (logp.double() - (z[order] - want)).abs().max().item() <= 2e-5


# 17 to 32 equal best logits in a tile of 9 and more hidden rows (a row's candidates fill two slots per lane), one more, and rows next to
# them where all the other tokens of the tile tie
@pytest.mark.parametrize("n,k,d,best", [(9, 2000, 256, 17), (12, 32768, 256, 24), (12, 32959, 128, 32), (33, 33000, 128, 33), (64, 70000, 128, 20), (130, 40000, 128, 31)])
@pytest.mark.parametrize("m", [1, 5, 8])
def test_ties_of_some_tokens_in_tiles_of_many_rows(n, k, d, best, m):
    W = torch.full((k, d), -0.25, dtype=torch.bfloat16, device="cuda")
    W[torch.arange(k, device="cuda") % 128 < best] = 0.5
    h = torch.where(torch.arange(n, device="cuda") % 3 == 1, -0.125, 0.125).bfloat16().unsqueeze(1).expand(n, d).contiguous()
    map_ = torch.arange(k, dtype=torch.int32, device="cuda") * 2 + 1
    ids, logp, lse = vt.draft_head_step(h, W, map_, m, return_lse=True)
    z = h.double() @ W.double().T
    order = torch.sort(z, dim=1, descending=True, stable=True).indices[:, :m]
    want = torch.logsumexp(z, 1)
    assert torch.equal(ids, map_[order])
    assert (lse.double() - want).abs().max().item() <= 2e-5       # (fp32 sums of up to 70000 exponentials)
    assert (logp.double() - (z.gather(1, order) - want.unsqueeze(1))).abs().max().item() <= 2e-5


# Stored logits: a row's candidates are ranked by their logits alone unless one is there twice.  Pairs, triples and a run of equal logits
# at the places around the m-th, target ids in no order; rows of one stretch and of several, aligned and not
@pytest.mark.parametrize("n,k", [(16, 1500), (20, 5000), (33, 32767), (64, 32768), (17, 40001)])
@pytest.mark.parametrize("m,run", [(9, 2), (16, 3), (16, 40), (33, 2)])
def test_equal_logits_among_stored_ones(n, k, m, run):
    d = 128
    g = torch.Generator(device="cuda").manual_seed(k + m)
    W = torch.zeros(k, d, dtype=torch.bfloat16, device="cuda")
    W[:, 0] = torch.randint(-8, 1, (k,), generator=g, device="cuda").bfloat16()       # the field: ties below zero
    places = torch.randperm(k, generator=g, device="cuda")
    W[places[:m - 1], 0] = torch.arange(2, m + 1, device="cuda").bfloat16()           # m - 1 different logits
    W[places[m - 1:m - 1 + run], 0] = 1.0                                             # the m-th: `run` times
    if run > 2:
        W[places[m + 60:m + 62], 0] = float(m)                                        # and the best one three times
    h = torch.zeros(n, d, dtype=torch.bfloat16, device="cuda")
    h[:, 0] = 2.0 ** -(torch.arange(n, device="cuda") % 3).float()
    map_ = torch.randperm(4 * k, generator=g, device="cuda")[:k].int()
    assert "row_select" in vt.draft_head_step_plan(n, k, d, m)
    ids, logp, lse = vt.draft_head_step(h, W, map_, m, return_lse=True)
    z = (h[:, :1].double() * W[:, 0].double())
    by_id = torch.argsort(map_.long())
    order = by_id[torch.sort(z[:, by_id], dim=1, descending=True, stable=True).indices[:, :m]]
    want = torch.logsumexp(z, 1)
    assert torch.equal(ids, map_[order])
    assert (lse.double() - want).abs().max().item() <= 2e-5       # (fp32 sums of up to 40001 exponentials)
    assert (logp.double() - (z.gather(1, order) - want.unsqueeze(1))).abs().max().item() <= 2e-5


# Fewer lists than lanes: keys dealt to the lanes up to 256 of them (four loads) and above (pairs), by lists again from 64 lists on and
# for an odd number of keys above 256; more tokens than lists, and as many as a list holds; every token of the head, and ties of all of them
@pytest.mark.parametrize("lists", [1, 5, 17, 32, 33, 36, 37, 63, 64, 65])
@pytest.mark.parametrize("n,m", [(1, 7), (2, 8), (3, 24), (1, 33), (8, 16)])
@pytest.mark.parametrize("ties", [False, True])
def test_merge_of_fewer_lists_than_lanes(lists, n, m, ties):
    k, d = 8 * lists - 3, 128
    m = min(m, k)
    g = torch.Generator(device="cuda").manual_seed(lists + m)
    plan = vt.draft_head_step_plan(n, k, d, m)
    assert f"workgroups={lists} rows_per_workgroup=8" in plan and "step_finalize" in plan
    W = torch.zeros(k, d, dtype=torch.bfloat16, device="cuda")
    W[:, 0] = (torch.randint(0, 3, (k,), generator=g, device="cuda") if ties else torch.randperm(k, generator=g, device="cuda") / 64).bfloat16()
    h = torch.zeros(n, d, dtype=torch.bfloat16, device="cuda")
    h[:, 0] = 2.0 ** -(torch.arange(n, device="cuda") % 3).float()
    map_ = torch.randperm(4 * k, generator=g, device="cuda")[:k].int()
    ids, logp, lse = vt.draft_head_step(h, W, map_, m, return_lse=True)
    z = h[:, :1].double() * W[:, 0].double()
    by_id = torch.argsort(map_.long())
    order = by_id[torch.sort(z[:, by_id], dim=1, descending=True, stable=True).indices[:, :m]]
    want = torch.logsumexp(z, 1)
    assert torch.equal(ids, map_[order])
    assert (lse.double() - want).abs().max().item() <= 1e-5       # (fp32 sums of up to 517 exponentials, a log-sum-exp below 16)
    assert (logp.double() - (z.gather(1, order) - want.unsqueeze(1))).abs().max().item() <= 1e-5


# The best tokens in one list, in two and in as many as there are, of the longest lists and of lists shorter than the tokens asked for
# (eight keys of a list at a time behind its first three or four)
@pytest.mark.parametrize("dtype,n,k,m", [("f32", 2, 2000, 12), ("f32", 3, 2040, 9), ("bf16", 2, 2000, 24), ("bf16", 4, 1999, 11), ("f32", 8, 2000, 64)])
@pytest.mark.parametrize("spread", [1, 2, 5, 8, 250])
def test_best_tokens_of_tiles_of_eight(dtype, n, k, m, spread):
    d, t = 128, torch.bfloat16 if dtype == "bf16" else torch.float32
    plan = vt.draft_head_step_plan(n, k, d, m, dtype=t)
    assert "workgroups=25" in plan and "step_finalize" in plan
    g = torch.Generator(device="cuda").manual_seed(m + spread)
    value = torch.rand(k, generator=g, device="cuda") - 4
    best = torch.randperm(k // 8, generator=g, device="cuda")[:spread]      # tiles
    at = (best.unsqueeze(1) * 8 + torch.arange(8, device="cuda")).flatten()[:max(m, 8)]
    value[at] = torch.randperm(at.numel(), generator=g, device="cuda") / 8.0
    W = torch.zeros(k, d, dtype=t, device="cuda")
    W[:, 0] = value.to(t)
    h = torch.zeros(n, d, dtype=t, device="cuda")
    h[:, 0] = 2.0 ** -(torch.arange(n, device="cuda") % 3).float()
    map_ = torch.arange(k, dtype=torch.int32, device="cuda") * 2 + 1
    ids, logp, lse = vt.draft_head_step(h, W, map_, m, return_lse=True)
    z = h[:, :1].double() * W[:, 0].double()
    order = torch.sort(z, dim=1, descending=True, stable=True).indices[:, :m]
    want = torch.logsumexp(z, 1)
    assert torch.equal(ids, map_[order])
    assert (lse.double() - want).abs().max().item() <= 1e-5       # (fp32 sums of 2000 exponentials, a log-sum-exp below 16)
    assert (logp.double() - (z.gather(1, order) - want.unsqueeze(1))).abs().max().item() <= 1e-5


# Several heads and more than eight tokens: a row's keys are all read and dealt to the lanes, or by lists where their number is odd; rows
# of one list, of a few and of most of them
@pytest.mark.parametrize("ks", [(1378, 236, 560, 93), (29045, 946, 72), (30000, 65), (16385, 16384)])
@pytest.mark.parametrize("n,m", [(4, 9), (4, 10), (8, 10), (3, 11)])
def test_lists_of_several_heads_with_more_than_eight_tokens(ks, n, m):
    d = 256
    g = torch.Generator(device="cuda").manual_seed(sum(ks) + m)
    heads = [(torch.randn(k, d, generator=g, device="cuda").mul_(0.1).bfloat16(), torch.arange(k, dtype=torch.int32, device="cuda")) for k in ks]
    h = torch.randn(n, d, generator=g, device="cuda").bfloat16()
    which = [i % len(ks) for i in range(n)]
    ids, logp, lse = vt.draft_head_step_multi(h, heads, which, m, return_lse=True)
    for i, q in enumerate(which):
        one_ids, one_logp = vt.draft_head_step(h[i:i + 1].expand(2, d).contiguous(), heads[q][0], heads[q][1], m)
        assert torch.equal(ids[i], one_ids[0])
        assert (logp[i] - one_logp[0]).abs().max().item() <= 4e-6      # sums over other tiles: a few ulp of a log-sum-exp near 10
