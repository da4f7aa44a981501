"""Selection, rank order and choice of k where counts leave the exact range of their codes, against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2506_22694_amd as vt

pytestmark = pytest.mark.gpu


def _counts(kind, V, rng):
    if kind == "around 2048":              # the last exact histogram bin and the first wide ones
        return rng.integers(2040, 2120, size=V)
    if kind == "around 2^19":              # the last count the rank codes hold exactly
        return rng.integers(2**19 - 40, 2**19 + 40, size=V)
    if kind == "large and equal":
        return np.full(V, 3 * 2**30 + 5)
    if kind == "large, few values":        # equal codes, counts apart in their last bits, in no order
        return (1 << 40) + rng.integers(0, 3, size=V)
    if kind == "powers of two":
        # (the total stays below 2^53: the oracle's ceil(P * total) is exact there)
        return np.left_shift(1, rng.integers(0, 37, size=V).astype(np.int64))
    if kind == "heavy tail":
        return np.floor(1e6 * rng.random(V) ** 12).astype(np.int64) + (rng.random(V) < 0.01) * 10**7
    raise ValueError(kind)


# V: one workgroup, its edge, the largest V that one workgroup chooses k for and one more, many workgroups
@pytest.mark.parametrize("V", [1, 1024, 1025, 4096, 4097, 30011])
@pytest.mark.parametrize("kind", ["around 2048", "around 2^19", "large and equal", "large, few values", "powers of two", "heavy tail"])
def test_selection_at_the_edges_of_the_codes(kind, V):
    if kind == "large, few values" and V > 4097:
        V = 4097          # (one bin of all ids, one more of them than one workgroup takes)
    rng = np.random.default_rng(V + len(kind))
    c = np.asarray(_counts(kind, V, rng), dtype=np.int64)
    dc = torch.from_numpy(c).cuda()
    order = oracle.rank_order(c)
    for k in sorted({1, V // 7 + 1, V // 2 + 1, V}):
        a, _ = vt.build_trimmed_head(dc, None, k)
        assert np.array_equal(a.cpu().numpy(), oracle.select(c, k)), k
        b, _ = vt.build_trimmed_head(dc, None, k, order="rank")
        assert np.array_equal(b.cpu().numpy(), order[:k]), k
    for P in (0.0, 1e-9, 0.25, 0.9, 1.0):
        assert vt.choose_k(dc, top_p=P) == oracle.choose_k_top_p(c, P), P
    for f in (0, 1, 2047, 2048, 2049, 2**19, int(c[0]), int(c.max()) + 1):
        assert vt.choose_k(dc, min_count=f) == oracle.choose_k_min_count(c, f), f


@pytest.mark.parametrize("V,heads", [(700, 16), (5000, 5), (20000, 16)])
def test_several_heads_selected_in_as_many_batches_as_the_workspace_holds(V, heads):
    rng = np.random.default_rng(heads)
    c = np.stack([np.asarray(_counts(k, V, rng), dtype=np.int64) for k in
                  (["heavy tail", "around 2048", "powers of two", "large and equal"] * 4)[:heads]])
    ks = [int(rng.integers(1, V + 1)) for _ in range(heads)]
    for (m, _), row, k in zip(vt.build_trimmed_heads(torch.from_numpy(c).cuda(), None, ks), c, ks):
        assert np.array_equal(m.cpu().numpy(), oracle.select(row, k))


# rows of eight bits per id between the two kernels: V on and off the 16-byte stores, one range of bins and its edge;
# bins of 255, 256 and far more in one chunk, in neighbouring ids; a last batch of every length
@pytest.mark.parametrize("V", [1, 3, 16, 4098, 65536, 65537, 65552, 131075])
@pytest.mark.parametrize("dtype", [torch.int32, torch.int64])
def test_count_bins_beyond_eight_bits(V, dtype):
    rng = np.random.default_rng(V)
    hot = [t for t in (0, 1, 2, 3, V // 2, V - 2, V - 1) if 0 <= t < V]
    parts = [np.full(reps, t) for t, reps in zip(hot, (255, 256, 257, 511, 512, 70000, 40001))]
    ids = np.concatenate(parts + [rng.integers(0, V, size=150_000 + 1024 * (V % 7) + V % 5)])
    rng.shuffle(ids)
    for n in (ids.size, ids.size - 1, ids.size - 4097, 5):
        c = vt.count_tokens(torch.from_numpy(ids[:n]).to(dtype).cuda(), V)
        assert np.array_equal(c.cpu().numpy(), np.bincount(ids[:n], minlength=V)), n


# Counts outside what choose_k is for (values >= 0, their sum below 2^63): it answers, and ends
@pytest.mark.parametrize("V", [3, 4096, 5000])
@pytest.mark.parametrize("low,high", [(-5, 6), (-2**62, 2**62), (2**61, 2**62), (-9, 0)])
def test_choose_k_ends_on_counts_outside_its_range(V, low, high):
    c = np.random.default_rng(V).integers(low, high, size=V, dtype=np.int64)
    for P in (0.0, 0.5, 1.0):
        k, _, total = vt.choose_k(torch.from_numpy(c).cuda(), top_p=P)
        assert 0 <= k <= V and total == int(c.view(np.uint64).sum().astype(np.int64))


def _large_counts(kind, V, rng):
    if kind == "close together":           # one bin, one next digit, twenty open bits
        return (1 << 40) + rng.integers(0, 1 << 20, size=V)
    if kind == "few values":               # ... and two, in no order
        return (1 << 40) + rng.integers(0, 3, size=V)
    if kind == "mixed":                    # exact bins, wide bins and one crowded one
        return np.where(rng.random(V) < 0.5, rng.integers(0, 5000, size=V), (1 << 35) + rng.integers(0, 1 << 13, size=V))
    if kind == "around 2^17":              # the last values that a bin and its next digit tell apart
        return rng.integers(2**17 - 300, 2**17 + 300, size=V)
    if kind == "all bits":
        return rng.integers(0, 2**63 - 1, size=V, dtype=np.int64) >> rng.integers(0, 63, size=V)
    if kind == "equal":
        return np.full(V, (1 << 45) + 12345)
    if kind == "mixed, one bit more":      # large counts that agree above 24 low bits, not above 23
        return np.where(rng.random(V) < 0.5, rng.integers(0, 5000, size=V), (1 << 35) + rng.integers(0, 2, size=V) * (1 << 23) + rng.integers(0, 50, size=V))
    raise ValueError(kind)


# A k-th largest count of 2048 and more: found by all workgroups and the last of them; one workgroup, its edge, many
@pytest.mark.parametrize("V", [5, 1024, 1025, 30011, 128256])
@pytest.mark.parametrize("kind", ["close together", "few values", "mixed", "around 2^17", "all bits", "equal"])
def test_selection_of_large_counts(kind, V):
    rng = np.random.default_rng(V)
    c = np.asarray(_large_counts(kind, V, rng), dtype=np.int64)
    dc = torch.from_numpy(c).cuda()
    order = np.lexsort((np.arange(V), -c))          # (count descending, id ascending; the oracle's sort takes seconds here)
    for k in sorted({1, 2, V // 50 + 1, V // 3 + 1, V // 2 + 1, V - 1, V}):
        a, _ = vt.build_trimmed_head(dc, None, k)
        assert np.array_equal(a.cpu().numpy(), np.sort(order[:k])), k
    both = np.stack([c, np.arange(V) % 7])          # beside a head whose bins are exact
    for row, (a, _) in zip(both, vt.build_trimmed_heads(torch.from_numpy(both).cuda(), None, [V // 3 + 1, V // 2 + 1])):
        k = a.numel()
        assert np.array_equal(a.cpu().numpy(), np.sort(np.lexsort((np.arange(V), -row))[:k]))


# The same counts' choice of k: the bin in which the mass reaches the target is divided further
@pytest.mark.parametrize("V", [5, 1024, 4096, 4097, 30011, 128256])
@pytest.mark.parametrize("kind", ["close together", "few values", "mixed", "around 2^17", "equal", "all bits"])
def test_choice_of_k_among_large_counts(kind, V):
    c = np.asarray(_large_counts(kind, V, np.random.default_rng(V)), dtype=np.int64)
    # keep the total below 2^53, where the oracle's ceil(P * total) is exact
    c >>= max(0, int(c.astype(np.float64).sum()).bit_length() - 53)
    dc = torch.from_numpy(c).cuda()
    for P in (0.0, 1e-9, 1e-4, 0.25, 0.6, 0.9, 0.999, 1.0):
        assert vt.choose_k(dc, top_p=P) == oracle.choose_k_top_p(c, P), P


# Rank order: large counts in clusters of 1 to 9000 ids, far apart from each other and near inside
def _counts_in_runs(lengths, V, rng):
    c = rng.integers(0, 1000, size=V)
    at = 0
    for q, n in enumerate(lengths):                  # run q: one code (19 highest bits), 14 open bits
        n = min(n, V - at)
        c[at:at + n] = (1 << 33) + (q << 24) + rng.integers(0, 1 << 14, size=n)
        at += n
    return rng.permutation(c)


@pytest.mark.parametrize("V", [5, 1024, 1025, 30011, 128256])
@pytest.mark.parametrize("kind", ["close together", "few values", "mixed", "around 2^17", "all bits", "equal", "mixed, one bit more", "short runs", "medium runs", "long runs"])
def test_rank_order_of_large_counts(kind, V):
    rng = np.random.default_rng(V)
    runs = {"short runs": [1, 2, 15, 16, 17, 18, 33, 64, 65] * 30, "medium runs": [255, 256, 257, 258, 1023, 1024, 1025, 500, 40] * 3, "long runs": [1025, 4095, 4096, 4097, 9000, 1]}
    c = np.asarray(_counts_in_runs(runs[kind], V, rng) if kind in runs else _large_counts(kind, V, rng), dtype=np.int64)
    dc = torch.from_numpy(c).cuda()
    order = np.lexsort((np.arange(V), -c))
    for k in sorted({1, V // 100 + 1, V // 3 + 1, V}):
        a, _ = vt.build_trimmed_head(dc, None, k, order="rank")
        assert np.array_equal(a.cpu().numpy(), order[:k]), k


# The upper eight bits of the bins are there for the groups of 256 ids that have any: hot ids in one group, at the edges of
# groups and ranges, in none and in all; more and fewer chunks than a wave of the sum takes
@pytest.mark.parametrize("V,n_ids,hot", [
    (65536 + 512, 2_000_000, [0, 255, 256, 65535, 65536, 66047]), (128256, 9_000_000, list(range(40))), (700, 3_000_000, []),
    (4097, 20_000_000, [4096]), (300, 16_000_000, [1, 299]), (257, 100_000, [256])])
@pytest.mark.parametrize("dtype", [torch.int32, torch.int64])
def test_count_hot_ids_side_by_side(V, n_ids, hot, dtype):
    rng = np.random.default_rng(V)
    ids = rng.integers(0, V, size=n_ids)
    if hot:
        some = rng.random(n_ids) < 0.4
        ids[some] = rng.choice(hot, size=int(some.sum()))
    c = vt.count_tokens(torch.from_numpy(ids).to(dtype).cuda(), V)
    assert np.array_equal(c.cpu().numpy(), np.bincount(ids, minlength=V))
    ws = torch.full((vt.load_library().vt_count_tokens_ws_bytes(V, n_ids),), 255, dtype=torch.uint8, device="cuda")
    c = vt.count_tokens(torch.from_numpy(ids).to(dtype).cuda(), V, c, ws=ws)      # on top, with a workspace that held other things
    assert np.array_equal(c.cpu().numpy(), 2 * np.bincount(ids, minlength=V))


# Rank order by bins: one workgroup, several, a ragged last one, the sum over workgroups by eight rows of a wave (up to 128 workgroups) and
# by thirty-two (two rounds of that: test_rank_order_of_large_vocabularies);
# `crowded`: no id of the sample is large, so one bin holds all large counts; `far`: counts of a bin too far apart for keys in LDS
@pytest.mark.parametrize("V", [1, 64, 8191, 8192, 8193, 131072, 131073])
@pytest.mark.parametrize("kind", ["uniform", "crowded", "far", "shared"])
def test_rank_order_by_bins_of_sampled_counts(kind, V):
    rng = np.random.default_rng(V)
    if kind == "shared":                   # large values that a dozen ids share, around the last one with a bin of its own
        c = rng.integers(2040, 2040 + V // 12 + 20, size=V)
    else:
        c = rng.integers(0, 1 << (61 if kind == "far" else 24), size=V)
    if kind == "crowded":
        i = np.arange(1024, dtype=np.uint64)
        c[((i << np.uint64(16) | i * np.uint64(40503) & np.uint64(0xFFFF)) * np.uint64(V)) // np.uint64(1 << 26)] = 5
    dc = torch.from_numpy(c).cuda()
    order = np.lexsort((np.arange(V), -c))
    for k in sorted({1, V // 3 + 1, V}):
        a, _ = vt.build_trimmed_head(dc, None, k, order="rank")
        assert np.array_equal(a.cpu().numpy(), order[:k]), k


# Streams of few chunks: a workspace for chunks of 65536 ids (what callers of earlier versions may have stored) counts the same;
# ids at the edges of chunks, of the hottest bin's own words, one id alone, ids outside [0, V) with bits in the upper half
@pytest.mark.parametrize("V,n_ids", [(128256, 200_000), (700, 65537), (65537, 16385), (40000, 1_000_003)])
@pytest.mark.parametrize("dtype", [torch.int32, torch.int64])
def test_count_few_chunks(V, n_ids, dtype):
    rng = np.random.default_rng(n_ids)
    hot = np.where(rng.random(n_ids) < 0.3, V - 1, rng.integers(0, V, size=n_ids))
    bad = rng.integers(-5, V + 5, size=n_ids)
    if dtype == torch.int64:
        bad[::97] += 1 << 32
    L = vt.load_library()
    chunk = 2 * ((V + 3) // 4 * 4) + (V + 255) // 256
    small = ((n_ids + 65535) // 65536 * chunk + 255) // 256 * 256
    assert small <= L.vt_count_tokens_ws_bytes(V, n_ids)
    for ids in (hot, bad, np.full(n_ids, V // 2), rng.integers(0, 2, size=n_ids) * (V - 1)):
        d = torch.from_numpy(ids).to(dtype).cuda()
        want = np.bincount(ids[(ids >= 0) & (ids < V)], minlength=V)
        for size in (small, L.vt_count_tokens_ws_bytes(V, n_ids)):
            inv = torch.zeros(1, dtype=torch.int64, device="cuda")
            c = vt.count_tokens(d, V, n_invalid=inv, ws=torch.full((size,), 255, dtype=torch.uint8, device="cuda"))
            assert np.array_equal(c.cpu().numpy(), want) and inv.item() == n_ids - want.sum()


# Waves of one workgroup whose hottest bins are neighbours, two to a word of LDS: every block of 256 ids belongs to one wave
@pytest.mark.parametrize("dtype", [torch.int32, torch.int64])
def test_count_hottest_bins_that_share_a_word(dtype):
    V, n_ids = 3000, 4_000_000
    rng = np.random.default_rng(5)
    wave = np.arange(n_ids) // (256 if dtype == torch.int32 else 128)
    ids = np.where(rng.random(n_ids) < 0.9, 1234 + wave % 2 + 2 * (wave % 6 == 5), rng.integers(0, V, size=n_ids))
    c = vt.count_tokens(torch.from_numpy(ids).to(dtype).cuda(), V)
    assert np.array_equal(c.cpu().numpy(), np.bincount(ids, minlength=V))


# One chunk (a vocabulary of more ranges than there are workgroups): a thread's own word of its wave's hottest bin and the words
# where ids of other ranges go reach 32768, with 80 million ids twice
@pytest.mark.parametrize("dtype,n_ids", [(torch.int32, 80_000_000), (torch.int64, 40_000_000)])
def test_count_one_id_in_one_chunk(dtype, n_ids):
    V = 129 * 65536 + 77
    for at in (V - 1, 65536 * 3 + 1):
        ids = torch.full((n_ids,), at, dtype=dtype, device="cuda")
        ids[::1001] = torch.arange(ids[::1001].numel(), device="cuda").to(dtype) % V
        c = vt.count_tokens(ids, V)
        assert torch.equal(c, torch.bincount(ids, minlength=V))


# Streams whose chunks hold no whole batch of vectors (4096 of 16 bytes), just one, and one vector more; from an aligned id and not
@pytest.mark.parametrize("dtype", [torch.int32, torch.int64])
@pytest.mark.parametrize("off", [0, 1])
def test_count_around_one_batch(dtype, off):
    V = 128256
    rng = np.random.default_rng(off)
    per = 4 if dtype == torch.int32 else 2
    for n_ids in (1, per - 1, per, 4096 * per - 1, 4096 * per, 4096 * per + 1, 4097 * per, 2 * 4096 * per, 2 * 4096 * per + per, 40000, 3 * 4096 * per + 5):
        for ids in (rng.integers(0, V, size=n_ids), np.full(n_ids, 70000), rng.integers(-3, 40, size=n_ids)):
            d = torch.from_numpy(np.concatenate([np.full(off, 9), ids])).to(dtype).cuda()[off:]
            inv = torch.zeros(1, dtype=torch.int64, device="cuda")
            c = vt.count_tokens(d, V, n_invalid=inv)
            assert np.array_equal(c.cpu().numpy(), np.bincount(ids[ids >= 0], minlength=V)), n_ids
            assert inv.item() == (ids < 0).sum()


# A bin's ids are sorted by comparisons up to 1024 of them and by digits of eight bits above: at the edges of both, by no digit, by one
# and a bit, by all that the keys hold (51 bits), with few values and many
@pytest.mark.parametrize("V", [1023, 1024, 1025, 2048, 2049, 4096, 4097, 8192])
@pytest.mark.parametrize("bits", [0, 1, 8, 9, 16, 38, 51])
def test_rank_order_of_one_bin(V, bits):
    rng = np.random.default_rng(V + bits)
    few = rng.integers(0, 1 << bits, size=5)
    for c in (rng.integers(0, 1 << bits, size=V), rng.choice(few, size=V), np.sort(rng.integers(0, 1 << bits, size=V))):
        order = np.lexsort((np.arange(V), -c))
        for k in (1, V // 2, V):
            a, _ = vt.build_trimmed_head(torch.from_numpy(c).cuda(), None, k, order="rank")
            assert np.array_equal(a.cpu().numpy(), order[:k]), k


# Up to 400 workgroups (each finds the splitters for itself) and more, up to 512 of them and more (their tallies are summed up in two
# rounds), bins between splitters of a thousand ids and more: a few values
# to a bin and many, values below 2048, large ones alone
@pytest.mark.parametrize("V", [409600, 409601, 524288, 524289, 1_000_003])
@pytest.mark.parametrize("kind", ["below 4000", "2048 to 4096", "below 2^24", "heavy tail", "equal"])
def test_rank_order_of_large_vocabularies(V, kind):
    g = torch.Generator(device="cuda").manual_seed(V)
    if kind == "heavy tail":
        c = (1e9 / (1 + torch.randperm(V, generator=g, device="cuda").double()) ** 1.1).long()
    else:
        lo, hi = {"below 4000": (0, 4000), "2048 to 4096": (2048, 4096), "below 2^24": (0, 1 << 24), "equal": (5000, 5001)}[kind]
        c = torch.randint(lo, hi, (V,), generator=g, device="cuda")
    order = torch.sort(c, descending=True, stable=True).indices.int()
    for k in (1, V // 3, V):
        a, _ = vt.build_trimmed_head(c, None, k, order="rank")
        assert torch.equal(a, order[:k]), k


# Counts 2^51 and more apart in one bin: ordered by their highest 51 bits where that settles them, by all where it does not (neighbours
# that differ in their lowest bits alone, in no order, beside equal ones); within the 1024 that are compared, and above
@pytest.mark.parametrize("V", [2, 700, 1024, 1025, 8192, 30011])
@pytest.mark.parametrize("kind", ["all magnitudes", "settled", "mixed", "equal and far"])
def test_rank_order_of_counts_far_apart(V, kind):
    rng = np.random.default_rng(V)
    c = rng.integers(0, 2**63 - 1, size=V)
    if kind == "all magnitudes":
        c >>= rng.integers(0, 63, size=V)
    elif kind == "settled":
        c &= ~np.int64(0xFFFF)
    elif kind == "mixed":
        c[::3] = (1 << 62) + rng.integers(0, 2000, size=c[::3].size)
    else:
        c = rng.choice([0, 1, 1 << 62, (1 << 62) + 1, 1 << 40], size=V)
    order = np.lexsort((np.arange(V), -c))
    for k in sorted({1, V // 3 + 1, V}):
        a, _ = vt.build_trimmed_head(torch.from_numpy(c).cuda(), None, k, order="rank")
        assert np.array_equal(a.cpu().numpy(), order[:k]), k


def _sample(V):
    """The ids that the splitters are taken from."""
    i = np.arange(1024, dtype=np.uint64)
    return ((i << np.uint64(16) | i * np.uint64(40503) & np.uint64(0xFFFF)) * np.uint64(V)) // np.uint64(1 << 26)


# One bin of more ids than LDS holds, shared by all workgroups: large counts that avoid the sample, with as many values as ids, with one
# and with two, and with values that also avoid the sample of the bin itself (a slice is then too long as well); two such bins
@pytest.mark.parametrize("V", [20011, 65536, 131072, 1_000_003])
@pytest.mark.parametrize("kind", ["all", "one value", "two values", "slices", "two bins", "far"])
def test_rank_order_of_long_bins(V, kind):
    rng = np.random.default_rng(V)
    c = rng.integers(3000, 10**7, size=V)
    if kind == "one value":
        c[:] = 77777
    elif kind == "two values":
        c = rng.integers(0, 2, size=V) * 5000 + 5000
    elif kind == "far":
        c = rng.integers(3000, 2**62, size=V) >> rng.integers(0, 40, size=V)
    c[_sample(V)] = rng.integers(0, 200, size=1024)
    if kind == "slices":
        inside = np.flatnonzero(c >= 2048)
        c[inside[np.arange(1024) * inside.size // 1024]] = 4_000_000
    if kind == "two bins":
        c[_sample(V)[:512]] = 5_000_000
    order = torch.sort(torch.from_numpy(c).cuda(), descending=True, stable=True).indices.int()
    for k in sorted({1, V // 3 + 1, V}):
        a, _ = vt.build_trimmed_head(torch.from_numpy(c).cuda(), None, k, order="rank")
        assert torch.equal(a, order[:k]), k


# So many long bins that every one is left to its workgroup, most of them within LDS beside some that are shared
@pytest.mark.parametrize("V", [2_000_000, 6_000_001])
def test_rank_order_of_millions_of_large_counts(V):
    g = torch.Generator(device="cuda").manual_seed(V)
    c = torch.randint(2048, 1 << 30, (V,), generator=g, device="cuda")
    order = torch.sort(c, descending=True, stable=True).indices.int()
    for k in (1, V // 2, V):
        a, _ = vt.build_trimmed_head(c, None, k, order="rank")
        assert torch.equal(a, order[:k]), k
