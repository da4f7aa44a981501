// Per-row tail of the draft step for many hidden rows (Algorithm 2's drafting lines after the
// projection): given the raw trimmed logits z[i, 0..k) of a hidden row, its log-sum-exp, its m best
// logits (equal logits -> lower target id) and their target ids.
//
// With tens or hundreds of hidden rows the per-tile candidate lists of the fused path grow to
// megabytes and their selection rounds dominate; it is cheaper to let the matrix-core kernel store
// the logits (n * k * 4 bytes, written once, read back from the L2) and give every hidden row a
// workgroup of its own:
//   pass 1  every thread (1024 per row) folds its share of the row into (max, sum-exp) and keeps its largest logit;
//   T       a threshold that at least m logits reach, from the lanes' maxima (bit-serial selection inside each wave),
//           so the m best logits are all >= T;
//   pass 2  logits >= T become candidate keys in LDS (typically a few dozen), ranked by counting (rows of up to 32768
//           logits stay in registers in between, longer ones are sifted as they go by: row_select_kernel);
//   (up to 32768 logits a row is bound by a chain: the loads, a reduction, two barriers, a trip to the map, the ranking.  The
//   ranking of the logits alone runs beside that trip, and the sum of exponentials waits for no barrier of its own: a percent of
//   a step, n = 128 on 32768 x 2048, m = 16 43.1 -> 42.7 us, and more with many candidates, n = 4 on 3880 x 4096, m = 24 23.2 -> 20.3)
//   if more than 1024 logits reach T (massive ties, e.g. h = 0) a second threshold is found among their keys (rank_by_keys).
// Where the matrix-core kernel leaves the (max, sum-exp) of a row's parts beside the logits, all of this reads a few dozen parts
// instead of the row (row_select_parts_kernel).
#include "vt_device.h"
#include "vt_step.h"

namespace vt {

namespace {

constexpr int kRowThreads = 1024;
constexpr int kRowWaves = kRowThreads / kWave;
constexpr int kRowMaxCand = 1024;
constexpr int kRowMaxTokens = 64;     // tokens per row (m)
constexpr int kRowMaxRaw = 4096;      // rows of several stretches: logits above the first stretch's threshold

__device__ __forceinline__ unsigned long long block_max_u64(unsigned long long v, unsigned long long *red, int lane,
                                                            int w) {
    v = wave_max_u64(v);
    __syncthreads();
    if (lane == 0) red[w] = v;
    __syncthreads();
    unsigned long long r = red[0];
#pragma unroll
    for (int q = 1; q < kRowWaves; ++q) r = red[q] > r ? red[q] : r;
    return r;
}

}  // namespace

// Values of one thread for one stretch of kRowThreads * kRowVals logits: v[u] = z[base + u * kRowThreads + tid]
// (-inf past the end).  All loads are issued before the first use.
constexpr int kRowVals = 32;
constexpr int kRowSpan = kRowThreads * kRowVals;     // 32768 logits per stretch
static_assert(kRowSpan == kRowSelectWhole);

// VEC: four consecutive logits per load (k a multiple of 4, row 16-byte aligned): thread t's value u is logit
// base + 4 * ((u / 4) * kRowThreads + t) + u % 4; otherwise logit base + u * kRowThreads + t.
template <bool VEC>
__device__ __forceinline__ int stretch_index(int base, int u, int tid) {
    return VEC ? base + 4 * ((u >> 2) * kRowThreads + tid) + (u & 3) : base + u * kRowThreads + tid;
}
template <bool VEC, int VALS>
__device__ __forceinline__ void load_stretch(const float *__restrict__ zr, int base, int k, int tid,
                                             float (&v)[VALS]) {
    if constexpr (VEC) {
#pragma unroll
        for (int q = 0; q < VALS / 4; ++q) {
            const int j = base + 4 * (q * kRowThreads + tid);
            float4 t = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
            if (j < k) t = *reinterpret_cast<const float4 *>(zr + j);
            v[4 * q] = t.x;
            v[4 * q + 1] = t.y;
            v[4 * q + 2] = t.z;
            v[4 * q + 3] = t.w;
        }
    } else {
#pragma unroll
        for (int u = 0; u < VALS; ++u) {
            const int j = base + u * kRowThreads + tid;
            v[u] = j < k ? zr[j] : -INFINITY;
        }
    }
}

// A thread's place in a stretch.  Groups of four (or logits) of a row that has fewer than threads go to the waves in equal shares: with them
// in order the last waves have none, their maxima leave the row without a threshold (row_threshold), and all its logits are candidates
// -- beyond 1024 of them the tokens are found one after the other (five slices, n = 128, k = 3000, d = 4096, m = 16 56.4 -> 20.3 us,
// n = 250, k = 2050 56.1 / 21.8, n = 20, k = 1500, d = 8192, m = 64 151.6 / 19.7; in one piece, n = 4, k = 3000, d = 1024, m = 16 46.8 / 9.6).
// Threads without a group have the last place, which lies behind the row.
template <bool VEC, int VALS>
__device__ __forceinline__ int stretch_place(int k, int tid, int lane, int w) {
    if constexpr (VALS == 8) {
        const int groups = VEC ? (k + 3) / 4 : k;
        if (groups < kRowThreads) {
            const int first = w * groups / kRowWaves, behind = (w + 1) * groups / kRowWaves;
            return first + lane < behind ? first + lane : kRowThreads - 1;
        }
    }
    return tid;
}

// The row's logits from `splits` partial ones, `stride` floats apart, added up in the order of the slices (rows 16-byte aligned,
// whole groups of four; what lies behind k in the last one is not a logit).  64 values of a thread are requested at a time.
template <int VALS>
__device__ __forceinline__ void load_slices(const float *__restrict__ zr, int splits, size_t stride, int k, int tid, float (&v)[VALS]) {
    constexpr int PER = 64 / VALS;
#pragma unroll
    for (int u = 0; u < VALS; ++u) v[u] = 0.f;
    for (int s0 = 0; s0 < splits; s0 += PER) {
        float4 t[PER][VALS / 4];
#pragma unroll
        for (int s = 0; s < PER; ++s) {
            const float *zs = zr + (size_t)min(s0 + s, splits - 1) * stride;
#pragma unroll
            for (int q = 0; q < VALS / 4; ++q) t[s][q] = *reinterpret_cast<const float4 *>(zs + min(4 * (q * kRowThreads + tid), (k - 1) & ~3));
        }
#pragma unroll
        for (int s = 0; s < PER; ++s) {
            const bool there = s0 + s < splits;
#pragma unroll
            for (int q = 0; q < VALS / 4; ++q) {
                v[4 * q] += there ? t[s][q].x : 0.f;
                v[4 * q + 1] += there ? t[s][q].y : 0.f;
                v[4 * q + 2] += there ? t[s][q].z : 0.f;
                v[4 * q + 3] += there ? t[s][q].w : 0.f;
            }
        }
    }
#pragma unroll
    for (int u = 0; u < VALS; ++u) v[u] = stretch_index<true>(0, u, tid) < k ? v[u] : -INFINITY;
}

// One exchange through LDS gives the row maximum M and a value T that at least m of the logits seen so far reach: every
// wave finds the ceil(m / 16)-th largest of its lanes' maxima (the wave maximum itself for m <= 16, otherwise bit by bit
// with ballots); each wave's share then holds that many logits >= its value, so the smallest of the sixteen values is
// reached by at least 16 * ceil(m / 16) >= m logits.  (Lanes without an element hold the lowest code.)  lm: the lane's
// maximum.  Contains one barrier; tmax must not be in use.
__device__ __forceinline__ void row_threshold(float lm, int m, unsigned *tmax, int lane, int w, unsigned &T, unsigned &Mo) {
    const unsigned mine = lm == -INFINITY ? 0u : orderable_f32(lm);
    const unsigned wtop = wave_max_u32(mine);
    unsigned Tw = wtop;
    int need = (m + kRowWaves - 1) / kRowWaves;
    if (need > 1) {
        Tw = 0u;
        unsigned long long alive = ~0ull;
        for (int b = 31; b >= 0; --b) {
            const unsigned long long ones = __ballot((mine >> b) & 1u) & alive;
            const int c = __popcll(ones);
            if (c >= need) {
                alive = ones;
                Tw |= 1u << b;
            } else {
                need -= c;
                alive &= ~ones;
            }
        }
    }
    if (lane == 0) {
        tmax[w] = Tw;
        tmax[kRowWaves + w] = wtop;
    }
    __syncthreads();
    T = tmax[0], Mo = tmax[kRowWaves];
#pragma unroll
    for (int q = 1; q < kRowWaves; ++q) {
        T = tmax[q] < T ? tmax[q] : T;
        Mo = tmax[kRowWaves + q] > Mo ? tmax[kRowWaves + q] : Mo;
    }
}
// (the order code is monotone; code 0 = no element maps to "everything passes")
__device__ __forceinline__ float threshold_f32(unsigned T) { return T == 0u ? -INFINITY : from_orderable_f32(T); }

// Folds one stretch into the lane's (max, sum-exp).
template <int VALS>
__device__ __forceinline__ void fold_stretch(const float (&v)[VALS], float &lm, float &ls) {
    float cm = v[0];
#pragma unroll
    for (int u = 1; u < VALS; ++u) cm = fmaxf(cm, v[u]);
    const float mn = fmaxf(lm, cm);
    if (mn != -INFINITY) {
        float cs = 0.f;
#pragma unroll
        for (int u = 0; u < VALS; ++u) cs += __expf(v[u] - mn);     // exp(-inf) = 0 past the end
        ls = ls * __expf(lm - mn) + cs;
        lm = mn;
    }
}

// Every logit of a stretch that reaches Tf, with its position, into `val` / `pos` (cap entries; n counts on, until a lane finds no room).
template <bool VEC, int VALS>
__device__ __forceinline__ void collect_stretch(const float (&v)[VALS], int base, int k, int tid, float Tf, float *val,
                                                int *pos, unsigned *n, unsigned cap) {
#pragma unroll
    for (int g = 0; g < VALS; g += 4) {
        // (four logits to a branch: a dozen of a thousand threads' groups holds one)
        if (fmaxf(fmaxf(v[g], v[g + 1]), fmaxf(v[g + 2], v[g + 3])) >= Tf) {
#pragma unroll
            for (int u = g; u < g + 4; ++u) {
                const int j = stretch_index<VEC>(base, u, tid);
                if (j < k && v[u] >= Tf) {
                    // logit and position now, the target id later: a load from the map here would put a trip to
                    // memory behind every candidate a wave finds, one after the other
                    const unsigned slot = atomicAdd(n, 1u);
                    if (slot < cap) {
                        val[slot] = v[u];
                        pos[slot] = j;
                    } else {
                        Tf = INFINITY;
                    }
                }
            }
        }
    }
}

// The m best of ncand <= kRowMaxCand candidates by counting: the logits alone are ranked while the trip to the map for the target
// ids is under way; one that is there twice is ranked by its keys (distinct target ids: distinct keys).  Equal logits meet at the
// place of the first of them: a second comparison per logit, for equality, took 5 us where a short row has no threshold
// and all of its 651 logits are candidates.  All threads call it; rawv is -inf behind the candidates, cand kNoKey, s_at zero.
__device__ __forceinline__ int keys_above(const unsigned long long *cand, int ncand, unsigned long long key) {
    unsigned above = 0;
    for (int x = 0; x < ncand; x += 8) {
        unsigned long long t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) t[u] = cand[x + u];
#pragma unroll
        for (int u = 0; u < 8; ++u) above += t[u] > key ? 1u : 0u;
    }
    return (int)above;
}
__device__ __forceinline__ void rank_candidates(const float *rawv, const int *rawj, unsigned long long *cand, unsigned *s_at,
                                                const int *__restrict__ map, int ncand, int m, float lse, int *__restrict__ ids, float *__restrict__ logp) {
    const int tid = threadIdx.x;
    unsigned long long key = 0ull;
    int above = m;
    if (tid < ncand) {
        const float mine = rawv[tid];
        const int id = map[rawj[tid]];
        above = 0;
        for (int x = 0; x < ncand; x += 8) {
            float t[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) t[u] = rawv[x + u];
#pragma unroll
            for (int u = 0; u < 8; ++u) above += t[u] > mine ? 1 : 0;
        }
        if (above < m) atomicAdd(&s_at[above], 1u);
        key = make_key(mine, id);
        cand[tid] = key;
    }
    __syncthreads();
    if (above < m) {
        if (s_at[above] > 1u) above = keys_above(cand, ncand, key);
        if (above < m) {
            ids[above] = key_id(key);
            logp[above] = key_logit(key) - lse;
        }
    }
}

// More logits than candidates: many equal ones (a row of zeros: a batch's padding), many large ones side by side, NaN.  for_keys(f) calls f
// with the key of every logit that may be among the m best.  Every thread's best key, and of those the largest threshold that m of
// them reach for sure, of three: m of one wave's, a quarter of m in each of four waves, a sixteenth in all.  What reaches it is ranked: two
// readings of the row.  With the last of the three alone, which nearly all threads' keys reach where logits are equal and ids ascending,
// ranking took 25 us (n = 128, k = 12001, d = 1024, m = 1, a single reading now, 40.5 -> 19.9 us, n = 100, k = 20000, m = 8 45.5 / 30.5), one reading per
// token more (n = 2, k = 16384, m = 16 95.8 / 21.2, n = 4, k = 30000, m = 64 535 / 32).  Too many all the same: one token per reading.
constexpr int kKeyThresholds = 3;
// The kth largest v of the wave's lanes, bit by bit: of each half those from the highest in which lanes still in question differ (equal
// logits differ in a few bits of their ids; all 64 bits took 14 us).  All 64 lanes take part, kth <= 64.
struct OpOrU32 {
    __device__ __forceinline__ unsigned operator()(unsigned a, unsigned b) const { return a | b; }
};
__device__ __forceinline__ unsigned kth_largest_of(unsigned v, unsigned long long &alive, int &kth) {
    const unsigned first = (unsigned)__builtin_amdgcn_readlane((int)v, __ffsll((long long)alive) - 1);
    const unsigned differ = wave_allreduce_u32((alive >> lane_id() & 1ull) != 0ull ? v ^ first : 0u, OpOrU32{});
    const int bits = 32 - __clz((int)__builtin_amdgcn_readfirstlane((int)differ));
    unsigned T = bits < 32 ? first >> bits << bits : 0u;
    for (int b = bits - 1; b >= 0; --b) {
        const unsigned long long ones = __ballot((v >> b) & 1u) & alive;
        const int c = __popcll(ones);
        if (c >= kth) {
            alive = ones;
            T |= 1u << b;
        } else {
            kth -= c;
            alive &= ~ones;
        }
    }
    return T;
}
__device__ __forceinline__ unsigned long long wave_kth_largest_u64(unsigned long long v, int kth) {
    unsigned long long alive = ~0ull;
    const unsigned long long high = kth_largest_of((unsigned)(v >> 32), alive, kth);
    return high << 32 | kth_largest_of((unsigned)v, alive, kth);
}
// The keys of a row's logits that reach Tf (all: of all its logits), from memory.
template <typename F>
__device__ __forceinline__ void for_row_keys(const float *__restrict__ zr, const int *__restrict__ map, int k, float Tf, bool all, F f) {
    for (int j0 = 0; j0 < k; j0 += 8 * kRowThreads) {
        float v[8];
        int id[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int j = min(j0 + u * kRowThreads + (int)threadIdx.x, k - 1);
            v[u] = zr[j];
            id[u] = map[j];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (j0 + u * kRowThreads + (int)threadIdx.x < k && (v[u] >= Tf || all)) f(make_key(v[u], id[u]));
        }
    }
}
template <typename ForKeys>
__device__ __forceinline__ void rank_by_keys(ForKeys for_keys, int m, float lse, unsigned long long *cand, unsigned *s_count,
                                             unsigned long long (&of_waves)[kKeyThresholds][kRowWaves], unsigned long long (&thresholds)[kKeyThresholds],
                                             int *__restrict__ ids, float *__restrict__ logp) {
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    unsigned long long best = kNoKey;
    for_keys([&](unsigned long long key) { best = key > best ? key : best; });
    if (m == 1) {
        best = block_max_u64(best, of_waves[0], lane, w);
        if (tid == 0) {
            ids[0] = key_id(best);
            logp[0] = key_logit(best) - lse;
        }
        return;
    }
    // (1, 4 and 16 waves)
    int kth = 0;
    unsigned long long of_wave = kNoKey;
    for (int x = 0; x < kKeyThresholds; ++x) {
        const int share = (m + (1 << 2 * x) - 1) >> 2 * x;
        if (share != kth) of_wave = wave_kth_largest_u64(best, share);
        kth = share;
        if (lane == 0) of_waves[x][w] = of_wave;
    }
    __syncthreads();      // (and the count of before has been read)
    if (tid == 0) *s_count = 0u;
    if (tid < kKeyThresholds) thresholds[tid] = ~0ull;
    cand[tid] = kNoKey;
    __syncthreads();
    if (tid < kKeyThresholds * kRowWaves) {
        const int x = tid / kRowWaves;
        const unsigned long long mine = of_waves[x][tid % kRowWaves];
        int above = 0;
#pragma unroll
        for (int q = 0; q < kRowWaves; ++q) above += of_waves[x][q] > mine ? 1 : 0;
        if (above < 1 << 2 * x) atomicMin(&thresholds[x], mine);
    }
    __syncthreads();
    unsigned long long T = thresholds[0];
#pragma unroll
    for (int x = 1; x < kKeyThresholds; ++x) T = thresholds[x] > T ? thresholds[x] : T;
    for_keys([&](unsigned long long key) {
        if (key >= T) {
            const unsigned slot = atomicAdd(s_count, 1u);
            if (slot < (unsigned)kRowMaxCand) cand[slot] = key;
            else T = ~0ull;      // (no room: nothing more to find)
        }
    });
    __syncthreads();
    const int nkeys = (int)*s_count;
    if (nkeys <= kRowMaxCand) {
        if (tid < nkeys) {
            const unsigned long long key = cand[tid];
            const int above = keys_above(cand, nkeys, key);
            if (above < m) {
                ids[above] = key_id(key);
                logp[above] = key_logit(key) - lse;
            }
        }
        return;
    }
    unsigned long long prev = ~0ull;
    for (int r = 0; r < m; ++r) {
        best = kNoKey;
        for_keys([&](unsigned long long key) { best = key < prev && key > best ? key : best; });
        best = block_max_u64(best, of_waves[0], lane, w);
        if (tid == 0) {
            ids[r] = key_id(best);
            logp[r] = key_logit(best) - lse;
        }
        prev = best;
    }
}

// kRowWhole: the row fits one stretch (k <= 32768), which stays in registers for the second pass.  kRowSift: longer rows are
// read once, too: the first stretch's threshold is one that m logits of the row reach, so what later stretches have to offer above it
// is collected as they go by (with the next stretch requested before the one at hand is folded), and the row's own
// threshold thins that out at the end.  A row whose first stretch says little (more than kRowMaxRaw logits above its
// threshold) is read again.  Reading longer rows twice cost k = 65536, n = 256 24.3 us (now 21.0),
// k = 128256, n = 256 40.6 (27.9), n = 16 20.5 (17.3): up to 64 rows what is left is the rate at which one CU reads a row.
// (Reading twice was the faster one up to 8 hidden rows of more than 16 tokens, n = 4, k = 128256, m = 64 47.7 us once, 43.3 twice; those
// are read by parts now, for which any workspace that a step of theirs accepts has room.)
enum RowMode { kRowWhole, kRowSift };
// VALS: values per thread and stretch; fewer than 32 for rows that fit them (what a thread holds past the row's end costs it an
// exponential and a comparison like any other: n = 40, k = 4149, d = 2048, m = 10 17.4 -> 15.9 us, n = 12, k = 10860, d = 3072, m = 16
// 19.8 -> 19.2).  SLICED: z is [splits][gridDim.x][pitch], see load_slices; z_out, or null: where the
// sums go.
// NaN reaches no threshold.  A row with fewer than m other logits is ranked by the codes of all its logits, so that its tokens are
// tokens of the head -- and so is, with nan_by_code, any row with a NaN: a step that keeps lists where its workspace has no room
// for logits has the same tokens either way.
template <RowMode MODE, bool VEC, int VALS, bool SLICED>
__global__ void __launch_bounds__(kRowThreads) row_select_kernel(const float *__restrict__ z, const int *__restrict__ map,
                                                                 int k, int m, int splits, int pitch, int nan_by_code,
                                                                 float *__restrict__ z_out,
                                                                 int *__restrict__ out_ids,
                                                                 float *__restrict__ out_logp,
                                                                 float *__restrict__ out_lse,
                                                                 float *__restrict__ lse_buf) {
    static_assert(!SLICED || (MODE == kRowWhole && VEC), "slices of rows that one stretch holds");
    static_assert(VALS == kRowVals || MODE == kRowWhole, "rows of several stretches");
    constexpr bool SIFT = MODE == kRowSift;
    constexpr unsigned kRaw = SIFT ? kRowMaxRaw : kRowMaxCand;
    __shared__ float redf[kRowWaves];
    __shared__ unsigned long long of_waves[kKeyThresholds][kRowWaves], thresholds[kKeyThresholds];
    __shared__ unsigned tmax[2 * kRowWaves], tmax_first[2 * kRowWaves];
    __shared__ unsigned long long cand[kRowMaxCand];
    __shared__ float rawv[kRaw];
    __shared__ int rawj[kRaw];
    __shared__ unsigned s_nraw, s_ncand;
    __shared__ unsigned s_at[kRowMaxTokens];      // candidates with that many larger logits
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int i = blockIdx.x;
    const float *zr = z + (size_t)i * (SLICED ? pitch : k);
    const int at = stretch_place<VEC, VALS>(k, tid, lane, w);
    float v[VALS];
    // (all of this is first used behind the barrier of row_threshold.  Candidates are ranked in whole groups of eight: what is
    // behind the last one loses against all of them)
    if (tid == 0) {
        s_nraw = 0u;
        s_ncand = 0u;
    }
    cand[tid] = kNoKey;
    if constexpr (!SIFT) {
        rawv[tid] = -INFINITY;
        if (tid < kRowMaxTokens) s_at[tid] = 0u;
    }

    // ---- pass 1: (max, sum-exp) and the thread's largest logit
    float lm = -INFINITY, ls = 0.f;
    if constexpr (SLICED) {
        load_slices(zr, splits, (size_t)gridDim.x * pitch, k, at, v);
        if (z_out != nullptr) {
#pragma unroll
            for (int u = 0; u < VALS; ++u) {
                const int j = stretch_index<VEC>(0, u, at);
                if (j < k) z_out[(size_t)i * k + j] = v[u];
            }
        }
    } else {
        load_stretch<VEC, VALS>(zr, 0, k, at, v);
    }
    unsigned T, Mo;
    if constexpr (MODE == kRowWhole) {
        fold_stretch(v, lm, ls);
    } else {
        float v2[VALS];
        load_stretch<VEC, VALS>(zr, kRowSpan, k, at, v2);
        fold_stretch(v, lm, ls);
        row_threshold(lm, m, tmax_first, lane, w, T, Mo);
        const float Tf1 = threshold_f32(T);
        collect_stretch<VEC, VALS>(v, 0, k, at, Tf1, rawv, rawj, &s_nraw, kRaw);
        for (int base = kRowSpan; base < k; base += 2 * kRowSpan) {
            load_stretch<VEC, VALS>(zr, base + kRowSpan, k, at, v);
            fold_stretch(v2, lm, ls);
            collect_stretch<VEC, VALS>(v2, base, k, at, Tf1, rawv, rawj, &s_nraw, kRaw);
            if (base + kRowSpan < k) {
                load_stretch<VEC, VALS>(zr, base + 2 * kRowSpan, k, at, v2);
                fold_stretch(v, lm, ls);
                collect_stretch<VEC, VALS>(v, base + kRowSpan, k, at, Tf1, rawv, rawj, &s_nraw, kRaw);
            }
        }
    }
    row_threshold(lm, m, tmax, lane, w, T, Mo);
    const float M = from_orderable_f32(Mo);      // k >= 1: some lane holds an element
    const float Tf = threshold_f32(T);
    {
        const float Sw = wave_sum(lm == -INFINITY ? 0.f : ls * __expf(lm - M));
        if (lane == 0) redf[w] = Sw;             // (summed up behind the barrier that the candidates need anyway)
    }

    // ---- pass 2: every logit >= T is a candidate
    if constexpr (MODE == kRowWhole) {
        collect_stretch<VEC, VALS>(v, 0, k, at, Tf, rawv, rawj, &s_nraw, kRaw);
        __syncthreads();
    } else if (s_nraw > kRaw) {
        __syncthreads();
        if (tid == 0) s_nraw = 0u;
        __syncthreads();
        for (int base = 0; base < k; base += kRowSpan) {
            load_stretch<VEC, VALS>(zr, base, k, at, v);
            collect_stretch<VEC, VALS>(v, base, k, at, Tf, rawv, rawj, &s_nraw, kRaw);
        }
        __syncthreads();
    }
    const int nraw = (int)s_nraw;
    int ncand = nraw;
    if (SIFT && nraw <= (int)kRaw) {
        // the candidates' target ids, all requested at once
        for (int c = tid; c < nraw; c += kRowThreads) {
            if (rawv[c] >= Tf) {
                const unsigned slot = atomicAdd(&s_ncand, 1u);
                if (slot < (unsigned)kRowMaxCand) cand[slot] = make_key(rawv[c], map[rawj[c]]);
            }
        }
        __syncthreads();
        ncand = (int)s_ncand;
    }
    float S = 0.f;
#pragma unroll
    for (int q = 0; q < kRowWaves; ++q) S += redf[q];     // fixed order: reproducible
    const float lse = M + __logf(S);
    const bool by_code = ncand < m || (nan_by_code != 0 && lse != lse);
    if (ncand <= kRowMaxCand && !by_code) {
        static_assert(kRowMaxCand == kRowThreads && kRowMaxCand % 8 == 0 && kRaw % 8 == 0);
        if constexpr (SIFT) {
            // (thinned out: the keys are there)
            if (tid < ncand) {
                const unsigned long long key = cand[tid];
                const int above = keys_above(cand, ncand, key);
                if (above < m) {
                    out_ids[(size_t)i * m + above] = key_id(key);
                    out_logp[(size_t)i * m + above] = key_logit(key) - lse;
                }
            }
        } else {
            rank_candidates(rawv, rawj, cand, s_at, map, ncand, m, lse, out_ids + (size_t)i * m, out_logp + (size_t)i * m);
        }
    } else {
        auto for_keys = [&](auto f) {
            if constexpr (SLICED) {
                // (the sums are nowhere but here)
#pragma unroll
                for (int g = 0; g < VALS; g += 8) {
                    int id[8];      // (requested together)
#pragma unroll
                    for (int u = 0; u < 8; ++u) id[u] = map[min(stretch_index<VEC>(0, g + u, at), k - 1)];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        if (stretch_index<VEC>(0, g + u, at) < k && (v[g + u] >= Tf || by_code)) f(make_key(v[g + u], id[u]));
                    }
                }
            } else {
                for_row_keys(zr, map, k, Tf, by_code, f);
            }
        };
        rank_by_keys(for_keys, m, lse, cand, &s_nraw, of_waves, thresholds, out_ids + (size_t)i * m, out_logp + (size_t)i * m);
    }
    if (tid == 0) {
        lse_buf[i] = lse;
        if (out_lse != nullptr) out_lse[i] = lse;
    }
}

// The same on rows whose parts' (max, sum-exp) are there, 16 to 80 logits each: a threshold that at least m parts' maxima reach is one
// that m logits reach, and only the parts that reach it are read.  A CU reads a row of 32768 logits in 4 us and takes as many
// exponentials of them; the parts' sums cost the kernel before a wave's few registers (n = 179, k = 35010, d = 1024, m = 16: this kernel 13.5 -> 6.6 us,
// the step 42.0 -> 31.1; n = 256, k = 32768, d = 8192 11.4 -> 7.1; n = 10, k = 113259, d = 3072, m = 10 130.8 -> 123.1).  What is left is a chain of
// trips: the parts, their logits, the map.  E: parts per thread.
// Parts that are read, about 54 (m <= 16) or 130 (m = 64) of them where logits are random: a wave whose best parts are none of the 256 best
// (512 with several parts to a wave) is one row in a million.  More: many equal logits.
constexpr int kMaxPicked = 512;
__device__ __forceinline__ int picked_limit(int m) { return m <= kRowWaves ? kMaxPicked / 2 : kMaxPicked; }
template <int E>
__global__ void __launch_bounds__(kRowThreads) row_select_parts_kernel(const float *__restrict__ z, const int *__restrict__ map, int k, int m, int pitch,
                                                                       int nan_by_code, RowParts rp, int *__restrict__ out_ids, float *__restrict__ out_logp,
                                                                       float *__restrict__ out_lse, float *__restrict__ lse_buf) {
    __shared__ float redf[kRowWaves];
    __shared__ unsigned long long of_waves[kKeyThresholds][kRowWaves], thresholds[kKeyThresholds];
    __shared__ unsigned tmax[2 * kRowWaves];
    __shared__ unsigned long long cand[kRowMaxCand];
    __shared__ float rawv[kRowMaxCand];
    __shared__ int rawj[kRowMaxCand];
    __shared__ int2 picked[kMaxPicked];           // the parts: first logit, behind the last
    __shared__ unsigned s_npicked, s_nraw;
    __shared__ unsigned s_at[kRowMaxTokens];      // candidates with that many larger logits
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int i = blockIdx.x;
    const float *zr = z + (size_t)i * pitch;
    const unsigned long long *pr = rp.pms + (size_t)i * rp.parts;
    // every wave has its share of every stretch of the row, and of the parts of each length (in a tile's order the last, shorter ones
    // would all be one wave's, whose best logit then sets the threshold: n = 5, k = 50204, m = 16, tiles of 200 30.0 -> 35.1 us)
    const int at = lane * kRowWaves + ((w + lane) & (kRowWaves - 1));
    unsigned long long part[E];
#pragma unroll
    for (int e = 0; e < E; ++e) part[e] = pr[min(e * kRowThreads + at, rp.parts - 1)];
    if (tid == 0) {
        s_npicked = 0u;
        s_nraw = 0u;
    }
    cand[tid] = kNoKey;
    rawv[tid] = -INFINITY;
    if (tid < kRowMaxTokens) s_at[tid] = 0u;
    float lm = -INFINITY;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        if (e * kRowThreads + at >= rp.parts) part[e] = 0xFF800000ull;      // (-inf, 0)
        lm = fmaxf(lm, __uint_as_float((unsigned)part[e]));
    }
    unsigned T, Mo;
    row_threshold(lm, m, tmax, lane, w, T, Mo);
    const float M = from_orderable_f32(Mo);
    const float Tf = threshold_f32(T);
    float ls = 0.f;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const float top = __uint_as_float((unsigned)part[e]);
        // (-inf - -inf is NaN, in the part's sum: logits that are all -inf add nothing.  Here and not where the sum is made: 20 bytes ahead of
        // the other epilogue moved it in its lines of instructions, n = 8, k = 1200, d = 2048, m = 1 9.01 -> 9.11 us)
        ls += top == -INFINITY ? 0.f : __uint_as_float((unsigned)(part[e] >> 32)) * __expf(top - M);
        if (top >= Tf) {
            const int x = e * kRowThreads + at;
            if (x < rp.parts) {
                const unsigned slot = atomicAdd(&s_npicked, 1u);
                const int tile = x / rp.per_tile * rp.tile_rows, first = tile + x % rp.per_tile * rp.part_rows;
                if (slot < (unsigned)kMaxPicked) picked[slot] = make_int2(first, min(k, min(tile + rp.tile_rows, first + rp.part_rows)));
            }
        }
    }
    const float Sw = wave_sum(ls);
    if (lane == 0) redf[w] = Sw;
    __syncthreads();
    const int npicked = (int)s_npicked;
    float S = 0.f;
#pragma unroll
    for (int q = 0; q < kRowWaves; ++q) S += redf[q];     // fixed order: reproducible
    const float lse = M + __logf(S);

    // Logits of the picked parts, four to a load
    const int vecs = rp.part_rows / 4, total = npicked * vecs;
    auto collect = [&]() {
        float Tt = Tf;      // (a thread that finds no room goes on no further)
        for (int x0 = 0; x0 < total; x0 += 2 * kRowThreads) {
            float4 v[2];
            int j[2], end[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int x = x0 + u * kRowThreads + tid, from = min(x, total - 1);
                const int2 p = picked[from / vecs];
                j[u] = p.x + from % vecs * 4;
                end[u] = x < total ? p.y : 0;
                v[u] = *reinterpret_cast<const float4 *>(zr + min(j[u], pitch - 4));
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if (j[u] < end[u] && fmaxf(fmaxf(v[u].x, v[u].y), fmaxf(v[u].z, v[u].w)) >= Tt) {
                    const float q[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        if (q[c] >= Tt && j[u] + c < k) {
                            const unsigned slot = atomicAdd(&s_nraw, 1u);
                            if (slot < (unsigned)kRowMaxCand) {
                                rawv[slot] = q[c];
                                rawj[slot] = j[u] + c;
                            } else {
                                Tt = INFINITY;
                            }
                        }
                    }
                }
            }
        }
        __syncthreads();
    };
    int ncand = kRowMaxCand + 1;
    if (npicked <= picked_limit(m)) {
        collect();
        ncand = (int)s_nraw;
    }
    const bool by_code = ncand < m || (nan_by_code != 0 && lse != lse);
    if (ncand <= kRowMaxCand && !by_code) {
        rank_candidates(rawv, rawj, cand, s_at, map, ncand, m, lse, out_ids + (size_t)i * m, out_logp + (size_t)i * m);
    } else {
        rank_by_keys([&](auto f) { for_row_keys(zr, map, k, Tf, by_code, f); }, m, lse, cand, &s_nraw, of_waves, thresholds, out_ids + (size_t)i * m,
                     out_logp + (size_t)i * m);
    }
    if (tid == 0) {
        lse_buf[i] = lse;
        if (out_lse != nullptr) out_lse[i] = lse;
    }
}

// splits > 1: z is [splits][n][pitch], pitch a multiple of four, k <= kRowSelectSlices; z_out [n, k] or null takes the sums.
hipError_t launch_row_select(const float *z, const int *map, int n, int k, int m, int splits, int pitch, bool nan_by_code, float *z_out,
                             int *out_ids, float *out_logp, float *out_lse, float *lse_buf, const RowParts *by_parts, hipStream_t st) {
    if (by_parts != nullptr) {
        const RowParts &rp = *by_parts;
        if (splits != 1 || pitch % 4 != 0 || pitch < k || (reinterpret_cast<uintptr_t>(z) & 15) != 0 || rp.parts < 1 || rp.parts > kRowPartsMax ||
            rp.part_rows % 4 != 0 || rp.tile_rows % 4 != 0 || rp.per_tile * rp.part_rows < rp.tile_rows ||
            (int64_t)((rp.parts + rp.per_tile - 1) / rp.per_tile) * rp.tile_rows < k)
            return hipErrorInvalidValue;
        auto launch = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3(n), dim3(kRowThreads), 0, st, z, map, k, m, pitch, nan_by_code ? 1 : 0, rp, out_ids, out_logp, out_lse, lse_buf);
            return hipGetLastError();
        };
        if (rp.parts <= kRowThreads) return launch(&row_select_parts_kernel<1>);
        if (rp.parts <= 2 * kRowThreads) return launch(&row_select_parts_kernel<2>);
        return launch(&row_select_parts_kernel<8>);
    }
    auto launch = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(n), dim3(kRowThreads), 0, st, z, map, k, m, splits, pitch, nan_by_code ? 1 : 0, z_out, out_ids, out_logp, out_lse, lse_buf);
        return hipGetLastError();
    };
    if (splits > 1) {
        static_assert(kRowSelectSlices == 16 * kRowThreads);
        if (k > kRowSelectSlices || pitch % 4 != 0 || pitch < k || (reinterpret_cast<uintptr_t>(z) & 15) != 0) return hipErrorInvalidValue;
        if (k <= 8 * kRowThreads) return launch(&row_select_kernel<kRowWhole, true, 8, true>);
        return launch(&row_select_kernel<kRowWhole, true, 16, true>);
    }
    const bool vec = (k & 3) == 0 && (reinterpret_cast<uintptr_t>(z) & 15) == 0;
    if (k <= 8 * kRowThreads) return vec ? launch(&row_select_kernel<kRowWhole, true, 8, false>) : launch(&row_select_kernel<kRowWhole, false, 8, false>);
    if (k <= 16 * kRowThreads) return vec ? launch(&row_select_kernel<kRowWhole, true, 16, false>) : launch(&row_select_kernel<kRowWhole, false, 16, false>);
    if (k <= kRowSpan) return vec ? launch(&row_select_kernel<kRowWhole, true, kRowVals, false>) : launch(&row_select_kernel<kRowWhole, false, kRowVals, false>);
    return vec ? launch(&row_select_kernel<kRowSift, true, kRowVals, false>) : launch(&row_select_kernel<kRowSift, false, kRowVals, false>);
}

}  // namespace vt
