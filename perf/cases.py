"""The work a speculative-decoding program has this library do, as cases that can be timed.

Offline, once per calibration corpus: count the token ids, choose k, select and gather the trimmed head.
Online, every draft step: project the hidden rows on the trimmed head, normalise, keep the best m tokens, remap
them; one draft round is a few such steps, each with the tree expansion on its result, and a rerank.

Shapes are Llama-3's (V = 128256, hidden sizes 2048 / 3072 / 4096 / 8192, 1024 for an independent drafter), the
paper's trimmed sizes, and what lies between them.  Values are the workloads': head entries N(0, 0.02^2), hidden
rows N(0, 1), token ids bounded Zipf over randomly permuted ids.

`prepare` holds what such a program holds between calls: the trimmed head and its map, a workspace, result
buffers (a serving loop allocates nothing per step).
"""
import torch

import paper_2506_22694_amd as vt

V_LLAMA3 = 128256
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
DEPTH, NODES = 3, 32          # of a draft tree: levels, and the tokens kept for the target to verify

# Drawn cases stay within the listed ones: the full-vocabulary head's bytes, the batch's multiplications.
MAX_HEAD_BYTES = V_LLAMA3 * 3072 * 2
MAX_FLOPS = 2 * 256 * 32768 * 8192


def listed():
    return [
        # the smallest call: a toy head in fp32 (what a program's own tests run), four rows, nothing but latency
        {"name": "tiny fp32 step", "op": "step", "dtype": "f32", "d": 256, "k": 1024, "n": 4, "m": 4},
        # greedy chain drafting, one token after another, on the library's own scratch
        {"name": "chain 1B", "op": "chain", "dtype": "bf16", "d": 2048, "k": 32768, "n": 1, "m": 1},
        # a whole draft round (three tree levels of 1, 8 and 8 nodes, then the rerank) on a task-specific head
        {"name": "task head round", "op": "round", "dtype": "bf16", "d": 3072, "k": 5000, "m": 8},
        # one level of an EAGLE-2 style tree, eight nodes, on a 3B model's trimmed head: the most frequent call
        {"name": "tree 3B", "op": "step", "dtype": "bf16", "d": 3072, "k": 32768, "n": 8, "m": 8},
        # the same level on the untrimmed head, which a program compares against
        {"name": "full head 3B", "op": "step", "dtype": "bf16", "d": 3072, "k": V_LLAMA3, "n": 8, "m": 8},
        # four requests' levels in one call, on the 8B model's head at the size the paper trims it to
        {"name": "tree 8B ragged", "op": "step", "dtype": "bf16", "d": 4096, "k": 32959, "n": 32, "m": 8},
        # a 64-node tree, or eight requests' levels
        {"name": "tree 8B", "op": "step", "dtype": "bf16", "d": 4096, "k": 32768, "n": 64, "m": 8},
        # a large serving batch: 256 rows on a 70B-sized hidden state, more candidates per node
        {"name": "batch", "op": "step", "dtype": "bf16", "d": 8192, "k": 32768, "n": 256, "m": 16},
        # requests of two tasks in one call: the general head and a function-calling one
        {"name": "two heads", "op": "multi", "dtype": "bf16", "d": 3072, "k": 32768, "k2": 5000, "n": 8, "m": 8},
        # calibration: the corpus' ids counted
        {"name": "count", "op": "count", "n_ids": 10_000_000, "zipf": 1.1, "wide": False},
        # calibration: the trimmed head of a 3B model selected and gathered
        {"name": "build", "op": "build", "n_ids": 10_000_000, "zipf": 1.1, "d": 3072, "k": 32768},
        # the study of k: k from the covered mass, then the rows in frequency order so that a prefix is any smaller k
        {"name": "choose and rank", "op": "rank", "n_ids": 10_000_000, "zipf": 1.1, "d": 2048, "k": 65536},
    ]


def _log_uniform(rng, lo, hi):
    return max(lo, min(hi, round(lo * (hi / lo) ** rng.random())))


def draw(rng):
    op = rng.choices(["step", "chain", "round", "multi", "count", "build", "rank"], [8, 1, 2, 2, 2, 2, 1])[0]
    if op == "count":
        return {"op": op, "n_ids": _log_uniform(rng, 200_000, 100_000_000), "zipf": rng.choice([1.05, 1.1]),
                "wide": rng.random() < 0.3}
    if op in ("build", "rank"):
        d = rng.choice([1024, 2048, 3072, 4096])
        return {"op": op, "n_ids": _log_uniform(rng, 200_000, 20_000_000), "zipf": rng.choice([1.05, 1.1]), "d": d,
                "k": _log_uniform(rng, 5000, 65536 * 2048 // max(d, 2048))}
    if op == "step" and rng.random() < 0.15:
        return {"op": op, "dtype": "f32", "d": rng.choice([256, 512, 1024, 2048]), "k": _log_uniform(rng, 1024, 32768),
                "n": rng.randint(1, 8), "m": rng.choice([1, 4, 8])}
    while True:
        d = rng.choice([1024, 2048, 3072, 4096, 8192] if op == "step" else [1024, 2048, 3072, 4096])
        k = rng.choice([22786, 32959, 32975, 33008, 35010]) if rng.random() < 0.3 else _log_uniform(rng, 4096, V_LLAMA3)
        n = 1 if op == "chain" else 8 if op == "round" else rng.randint(2, 8) if op == "multi" else _log_uniform(rng, 1, 256)
        k2 = rng.randint(4096, 8192) if op == "multi" else 0
        if (k + k2) * d * 2 * (DEPTH if op == "round" else 1) <= MAX_HEAD_BYTES and 2 * n * k * d <= MAX_FLOPS:
            break
    case = {"op": op, "dtype": "bf16", "d": d, "k": k}
    if op == "round":
        return {**case, "m": 8}
    case.update(n=n, m=1 if op == "chain" else rng.choice([1, 4, 8, 8, 10, 16] if op == "step" else [1, 4, 8]))
    return {**case, "k2": k2} if op == "multi" else case


# ---------------------------------------------------------------------------------------------- inputs
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _head(g, k, d, dtype):
    """(W_trim [k, d], ascending map [k]): rows as a gather from a full head would give them."""
    W = torch.randn((k, d), generator=g, device="cuda", dtype=dtype).mul_(0.02)
    ids = torch.randperm(max(k, V_LLAMA3), generator=g, device="cuda")[:k].sort().values.to(torch.int32)
    return W, ids


def _zipf_ids(g, n_ids, s, dtype=torch.int32):
    cdf = torch.arange(1, V_LLAMA3 + 1, device="cuda", dtype=torch.float64).pow_(-s).cumsum(0)
    cdf /= cdf[-1].clone()
    perm = torch.randperm(V_LLAMA3, generator=g, device="cuda").to(dtype)
    out = torch.empty(n_ids, dtype=dtype, device="cuda")
    for lo in range(0, n_ids, 1 << 24):
        hi = min(n_ids, lo + (1 << 24))
        u = torch.rand(hi - lo, generator=g, device="cuda", dtype=torch.float64)
        out[lo:hi] = perm[torch.searchsorted(cdf, u).clamp_(max=V_LLAMA3 - 1)]
    return out


def _results(n, m):
    return {"out_ids": torch.empty((n, m), dtype=torch.int32, device="cuda"),
            "out_logp": torch.empty((n, m), dtype=torch.float32, device="cuda")}


def prepare(case, seed):
    g, op = _generator(seed), case["op"]
    if op == "count":
        return {"op": op, "ids": _zipf_ids(g, case["n_ids"], case["zipf"], torch.int64 if case["wide"] else torch.int32)}
    if op in ("build", "rank"):
        counts = torch.bincount(_zipf_ids(g, case["n_ids"], case["zipf"]), minlength=V_LLAMA3)
        W = torch.randn((V_LLAMA3, case["d"]), generator=g, device="cuda", dtype=torch.bfloat16).mul_(0.02)
        return {"op": op, "counts": counts, "W": W, "k": case["k"]}
    dtype, d, k, m = DTYPES[case["dtype"]], case["d"], case["k"], case["m"]
    W, map_ = _head(g, k, d, dtype)
    state = {"op": op, "W": W, "map": map_, "m": m}
    if op == "round":
        rows = [1] + [m] * (DEPTH - 1)
        state["h"] = [torch.randn((n, d), generator=g, device="cuda", dtype=dtype) for n in rows]
        state["ws"] = vt.StepWorkspace(m, k, d, m, W.device)
        state["root"] = torch.zeros(1, device="cuda")
        state["results"] = [_results(n, m) for n in rows]
        # every level: the K = m survivors; beside them all n * m candidates' scores, from which the tree is kept
        state["out"] = [tuple(torch.empty(m, dtype=t, device="cuda") for t in (torch.int32, torch.int32, torch.float32))
                        for _ in rows]
        state["cum"] = torch.empty(sum(rows) * m, device="cuda")
        state["kept"] = torch.empty(NODES, dtype=torch.int32, device="cuda")
        return state
    n = case["n"]
    state["h"] = torch.randn((n, d), generator=g, device="cuda", dtype=dtype)
    state["results"] = _results(n, m)
    if op == "step":
        state["ws"] = vt.StepWorkspace(n, k, d, m, W.device)
    if op == "multi":
        state["heads"] = [(W, map_), _head(g, case["k2"], d, dtype)]
        state["head_of_row"] = [int(i % 2) for i in range(n)]
        state["ws"] = vt.MultiStepWorkspace(n, d, [k, case["k2"]], m, W.device)
    return state


# ---------------------------------------------------------------------------------------------- one pass
def run(state):
    op = state["op"]
    if op == "step":
        return vt.draft_head_step(state["h"], state["W"], state["map"], state["m"], ws=state["ws"], **state["results"])
    if op == "chain":
        return vt.draft_head_step_static(state["h"], state["W"], state["map"], state["m"], **state["results"])
    if op == "multi":
        return vt.draft_head_step_multi(state["h"], state["heads"], state["head_of_row"], state["m"], ws=state["ws"],
                                        **state["results"])
    if op == "round":
        return _draft_round(state)
    if op == "count":
        return vt.count_tokens(state["ids"], V_LLAMA3)
    if op == "build":
        return vt.build_trimmed_head(state["counts"], state["W"], state["k"])
    chosen = vt.choose_k(state["counts"], top_p=0.9)
    return chosen, vt.build_trimmed_head(state["counts"], state["W"], state["k"], order="rank")


def _draft_round(state):
    cum, scores, at, levels = state["root"], state["cum"], 0, []
    for h, out, results in zip(state["h"], state["out"], state["results"]):
        parent, token, nxt, ids, logp = vt.draft_tree_level(h, state["W"], state["map"], state["m"], cum, state["m"],
                                                            ws=state["ws"], out=out, **results)
        torch.add(logp, cum.unsqueeze(1), out=scores[at:at + logp.numel()].view_as(logp))
        at += logp.numel()
        levels.append((parent, token, nxt, ids, logp))
        cum = nxt
    return levels, scores, vt.tree_rerank(scores, NODES, out=state["kept"])


# ---------------------------------------------------------------------------------------------- work and exactness
def work(case):
    op = case["op"]
    if op == "count":
        return {"bytes": case["n_ids"] * (8 if case["wide"] else 4) + 8 * V_LLAMA3, "flops": 0}
    if op == "build":
        return {"bytes": 8 * V_LLAMA3 + case["k"] * (4 + 2 * case["d"] * 2), "flops": 0}
    if op == "rank":
        return {"bytes": 2 * 8 * V_LLAMA3 + case["k"] * (4 + 2 * case["d"] * 2), "flops": 0}
    size, d, m = (2 if case["dtype"] == "bf16" else 4), case["d"], case["m"]
    k = case["k"] + case.get("k2", 0)
    if op == "round":
        rows = 1 + m * (DEPTH - 1)
        flops = 2 * rows * k * d
    else:
        rows = case["n"]
        flops = 2 * rows * k * d if op != "multi" else 2 * d * sum(
            (case["k"], case["k2"])[i % 2] for i in range(rows))
    return {"bytes": k * (d * size + 4) + rows * (d * size + 8 * m), "flops": flops}


def tolerance(case):
    # Counts, selections and copies are whole numbers and bytes.  A step's log-probs are fp32 sums over d products and
    # a log-sum-exp over k terms, in another order in another correct implementation; a token or a node changes places
    # with its neighbour where their logits agree to that rounding.
    if case["op"] in ("count", "build", "rank"):
        return "exact"
    return {"rel": 2e-6, "max": 1e-5, "differ": 0.005}


def _exact_logp(h, W, m):
    lp = torch.empty((h.shape[0], m), dtype=torch.float64, device=h.device)
    z = torch.empty((h.shape[0], W.shape[0]), dtype=torch.float64, device=h.device)
    for lo in range(0, W.shape[0], 8192):
        z[:, lo:lo + 8192] = h.double() @ W[lo:lo + 8192].double().t()
    torch.sub(z.topk(m, dim=1).values, z.logsumexp(dim=1, keepdim=True), out=lp)
    return lp


def exact(case, seed):
    op, s = case["op"], prepare(case, seed)
    if op == "count":
        return torch.bincount(s["ids"], minlength=V_LLAMA3)
    if op in ("build", "rank"):
        order = torch.sort(s["counts"], descending=True, stable=True)      # equal counts: ascending ids
        map_ = order.indices[:case["k"]]
        if op == "build":
            map_ = map_.sort().values
        built = (map_.to(torch.int32), s["W"][map_])
        if op == "build":
            return built
        covered = order.values.cumsum(0)
        need = torch.ceil(covered[-1].double() * 0.9)
        k = int((covered.double() < need).sum()) + 1
        return (k, int(covered[k - 1]), int(covered[-1])), built
    if op == "multi":
        lp = torch.empty((case["n"], case["m"]), dtype=torch.float64, device="cuda")
        for j, (W, _) in enumerate(s["heads"]):
            lp[j::2] = _exact_logp(s["h"][j::2], W, case["m"])
        return None, lp
    if op == "round":
        m, cum, levels, scores = case["m"], torch.zeros(1, dtype=torch.float64, device="cuda"), [], []
        for h in s["h"]:
            lp = _exact_logp(h, s["W"], m)
            all_ = cum.unsqueeze(1) + lp
            cum = all_.flatten().topk(m).values
            levels.append((None, None, cum, None, lp))
            scores.append(all_.flatten())
        return levels, torch.cat(scores), None
    return None, _exact_logp(s["h"], s["W"], case["m"])
