"""Inputs that once took several times as long as others of the same size: one against the other, with a wide margin."""
import statistics

import pytest
import torch

import paper_2506_22694_amd as vt

pytestmark = pytest.mark.gpu


def _times(*calls, passes=30, rounds=7):
    """The calls' median time, measured in turn."""
    t = [[] for _ in calls]
    for r in range(rounds + 1):
        for call, out in zip(calls, t):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(passes):
                call()
            end.record()
            torch.cuda.synchronize()
            if r > 0:
                out.append(start.elapsed_time(end))
    return [statistics.median(x) for x in t]


# 17 lists of 8 keys: 24 tokens went through 24 rounds over the lists (19.3 us a step, now 7.7)
def test_more_tokens_than_lists():
    k, d = 136, 512
    W = torch.randn(k, d, device="cuda").mul_(0.02).bfloat16()
    h = torch.randn(1, d, device="cuda").bfloat16()
    map_ = torch.arange(k, dtype=torch.int32, device="cuda")
    captured = []
    for m in (24, 8):
        ws = vt.StepWorkspace(1, k, d, m, W.device)
        out = {"out_ids": torch.empty((1, m), dtype=torch.int32, device="cuda"), "out_logp": torch.empty((1, m), device="cuda")}
        step = lambda m=m, ws=ws, out=out: vt.draft_head_step(h, W, map_, m, ws=ws, **out)
        step()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(10):
                step()
        captured.append(graph.replay)
    many, few = _times(*captured)
    assert many < 1.5 * few, (many, few)


# Large counts that avoid the ids which the splitters are sampled from: one workgroup ordered all 38 000 of them (322 us; no such counts 37)
def test_large_counts_outside_the_sample():
    V = 128256
    i = torch.arange(1024, dtype=torch.int64, device="cuda")
    sample = ((i << 16 | i * 40503 & 0xFFFF) * V) >> 26
    g = torch.Generator(device="cuda").manual_seed(1)
    spread = torch.where(torch.rand(V, generator=g, device="cuda") < 0.3, torch.randint(10**5, 10**7, (V,), generator=g, device="cuda"), 5)
    hidden = spread.clone()
    hidden[sample] = 5
    ws = torch.empty(vt.load_library().vt_build_trimmed_head_ws_bytes(V, 8, V), dtype=torch.uint8, device="cuda")
    out = torch.empty(V, dtype=torch.int32, device="cuda")
    t = _times(*[lambda c=c: vt.build_trimmed_head(c, None, V, ws=ws, out_map=out, order="rank") for c in (hidden, spread)])
    assert t[0] < 4 * t[1], t


# Rows of fewer groups of four logits than the workgroup's last wave begins with, in slices: they had no threshold, and their tokens were
# found one after the other (n = 128, k = 3000, d = 4096, m = 16 56 us, k = 4300 23)
def test_short_rows_in_slices():
    n, d, m = 128, 4096, 16
    h, calls = torch.randn(n, d, device="cuda").bfloat16(), []
    for k in (3000, 4300):
        assert "column_slices" in vt.draft_head_step_plan(n, k, d, m)
        W = torch.randn(k, d, device="cuda").mul_(0.02).bfloat16()
        args = (h, W, torch.arange(k, dtype=torch.int32, device="cuda"), m)
        kept = {"ws": vt.StepWorkspace(n, k, d, m, W.device), "out_ids": torch.empty((n, m), dtype=torch.int32, device="cuda"),
                "out_logp": torch.empty((n, m), device="cuda")}
        calls.append(lambda args=args, kept=kept: vt.draft_head_step(*args, **kept))
    short, long = _times(*calls)
    assert short < 1.4 * long, (short, long)


# A row of zeros (a batch's padding), all of whose logits are equal: by parts, in whole rows and in slices.  A thousand candidates took 25 us to
# rank (n = 128, k = 12001, d = 1024, m = 1 40.5 us, random rows 18), a reading per token more (n = 2, k = 16384, m = 16 96 / 14)
@pytest.mark.parametrize("n,k,d,m,most", [(128, 12001, 1024, 1, 1.7), (128, 12001, 1024, 8, 1.7), (2, 16384, 1024, 16, 3), (20, 4806, 8192, 8, 1.6)])
def test_rows_of_zeros(n, k, d, m, most):
    assert "row_select" in vt.draft_head_step_plan(n, k, d, m)
    W = torch.randn(k, d, device="cuda").mul_(0.02).bfloat16()
    h = torch.randn(n, d, device="cuda").bfloat16()
    zero = h.clone()
    zero[n // 2] = 0
    map_ = torch.arange(k, dtype=torch.int32, device="cuda")
    kept = {"ws": vt.StepWorkspace(n, k, d, m, W.device), "out_ids": torch.empty((n, m), dtype=torch.int32, device="cuda"),
            "out_logp": torch.empty((n, m), device="cuda")}
    padded, full = _times(*[lambda h=h: vt.draft_head_step(h, W, map_, m, **kept) for h in (zero, h)])
    assert padded < most * full, (padded, full)
