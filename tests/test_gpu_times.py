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
