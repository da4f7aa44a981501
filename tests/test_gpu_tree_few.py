"""A tree level of one or two hidden rows, merged and ranked in one workgroup: bit for bit the step and the expansion behind it."""
import pytest
import torch

import paper_2506_22694_amd as vt

pytestmark = pytest.mark.gpu


# up to 256 keys, fewer lists than lanes, one to 64 keys to a list, rounds over the lists (all logits equal), one candidate and 128,
# all kept and one; small-n and matrix-core kernels, fp32
@pytest.mark.parametrize("n,k,d,m,dtype", [
    (1, 1, 64, 1, "bf16"), (1, 64, 128, 64, "bf16"), (2, 64, 128, 64, "f32"), (2, 300, 512, 10, "bf16"), (1, 700, 256, 2, "f32"), (2, 5000, 3072, 8, "bf16"),
    (1, 5000, 1024, 4, "bf16"), (2, 8192, 512, 9, "bf16"), (1, 32768, 256, 11, "bf16"), (2, 65536, 128, 8, "bf16"), (1, 30000, 128, 33, "f32")])
@pytest.mark.parametrize("ties", [False, True])
def test_level_of_one_or_two_rows(n, k, d, m, dtype, ties):
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(k + m)
    W = torch.randn(k, d, generator=g, device="cuda").mul_(0.02).to(t)
    h = torch.randn(n, d, generator=g, device="cuda").to(t)
    if ties:
        h[0] = 0
    map_ = torch.randperm(3 * k, generator=g, device="cuda")[:k].sort().values.to(torch.int32)
    cum = torch.tensor([-1.5, -0.25][:n], device="cuda")
    ids, logp = vt.draft_head_step(h, W, map_, m)
    for K in sorted({1, min(8, n * m), n * m}):
        want = vt.tree_expand(cum, logp, ids, K)
        parent, token, score, a, b = vt.draft_tree_level(h, W, map_, m, cum, K)
        assert torch.equal(a, ids) and torch.equal(b, logp)
        for x, y in zip(want, (parent, token, score)):
            assert torch.equal(x, y), K
        # the scores may replace the ones they are made from
        own = cum.clone() if K <= n else torch.cat([cum, cum.new_zeros(K - n)])
        out = (torch.empty(K, dtype=torch.int32, device="cuda"), torch.empty(K, dtype=torch.int32, device="cuda"), own[:max(K, n)])
        vt.draft_tree_level(h, W, map_, m, own[:n], K, out=out)
        assert torch.equal(own[:K], want[2])
