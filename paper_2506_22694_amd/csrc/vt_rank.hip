// Frequency-rank order and the alternative choices of k (Sec. 3.2: besides a fixed k, Top-P over
// the counts or a minimum-frequency threshold select the trimmed vocabulary).
//
// Rank order = all V ids sorted by (count descending, id ascending), the order in which
// Top-K(c, k) takes ids; every prefix is the selection for a smaller k.
//
// rsort_*: stable LSD radix sort over the whole device of (code, id) pairs, 8 bits per pass.  The code (vt_code.h) is
//   the count itself below 2^19 and its 19 highest bits with their exponent above -- 24 bits, three passes for any
//   int64.  The ids start ascending and every pass is stable, so equal codes stay in ascending-id order; where counts
//   of 2^19 and more share a code (a handful of ids, if any) the last kernel orders the run: up to 16 ids by counting in
//   each id's thread, up to 256 in a wave, up to 1024 in a workgroup, longer ones by radix passes of one workgroup (time
//   grows with the run and not with its square).
//   Where all counts of 2^19 and more agree above their 23 low bits (and have bits there) their code is those bits
//   instead, which leaves out nothing: every kernel derives that from what the first one found.
//   One workgroup per 1024 consecutive elements; a wave takes 64 consecutive elements, lanes with
//   equal digits find each other with nine ballots and rank themselves by population count, so
//   "earlier in the input" is (workgroup, wave, lane) order and no per-thread histogram is needed.
//     rsort_init     pairs from the counts, the digit totals of the three passes, per-workgroup digits of the first
//     rsort_hist     per-workgroup digit histogram of a later pass
//     rsort_scatter  every workgroup derives its own output offsets from the histogram table
//                    (sum over earlier digits and over earlier workgroups), then scatters
//     rsort_out      the ids in order
//   Eight launches in a fixed sequence; nothing is read back.  A pass whose digit is the same for every key moves
//   nothing and is skipped: each kernel derives that, and which buffer holds the data, from the digit totals alone.
//   (Eight passes over the bytes of the counts, nineteen launches, took 72 us at V = 128256 after 10^7 tokens; now 43.)
//   V = 128256: after 10^11 tokens 47 us (86 with two global atomics per large count, 95 over the bytes); all counts in
//   2^40 .. 2^40 + 2^20 48 (74; V = 32000 40, 6475 with every thread walking its run, 56); half of them in
//   2^35 .. 2^35 + 2^13 52 (75).  Slower than over the bytes: runs of 200 to 400 ids, V = 32000 around 2^19, 95 (441, 55).
// choose_*: no sort: a histogram over bins of counts (exact below 2048) with the mass of every bin, walked from the
//   largest counts down to the bin in which the mass reaches ceil(P * total).  With the read-back of k 107 us behind a full
//   sort, now 31.  Where that bin holds several values all workgroups histogram the next eleven bits of its ids, and the
//   one that is done last divides further; it reads all counts once per eleven bits that are still open, only where the
//   target falls between ids that share the 17 highest bits.
//   V = 128256, P = 0.25 after 10^7 tokens 18 us (48 with one workgroup for the whole division, 80 behind the sort), P = 0.9
//   after 10^9 22 (31, 92), equal counts 21 (870, 61), all counts in 2^40 .. 2^40 + 2^20 91 (412, 79).
#include "vt_build.h"
#include "vt_code.h"
#include "vt_device.h"

namespace vt {

namespace {

inline size_t round256(size_t x) { return (x + 255) / 256 * 256; }

constexpr int kSortWaves = kRankSortThreads / kWave;   // 16
constexpr int kDigits = 256;
constexpr int kPasses = 3;
constexpr unsigned kRankExact = 1u << 19;      // codes below are counts

struct SortBufs {
    unsigned long long *pairs[2];      // code << 32 | id
    unsigned *gtot;      // [2][kPasses][kDigits] digit totals over all elements, and what is added for the codes of low bits
    // of the counts >= kRankExact: the bits that their codes leave out, set in any of them and clear in any, and the same of
    // the bits above the low ones
    unsigned long long *rest;      // [4]
    unsigned *hist;      // [nblk][kDigits] per-workgroup digit counts of the current pass, descending digit first
    unsigned *hist_low;  // ... and of the first pass with codes of low bits
};
constexpr int kTotals = 2 * kPasses * kDigits;
constexpr int kLowBits = 23;
// the code of low bits of a count >= kRankExact, above all smaller counts' codes
__device__ __forceinline__ unsigned low_code(unsigned long long c) { return (1u << kLowBits) | ((unsigned)c & ((1u << kLowBits) - 1u)); }

// lanes of the wave whose `dgt` (0..256, 256 = not an element) equals this lane's
__device__ __forceinline__ unsigned long long match_digit9(int dgt) {
    unsigned long long m = ~0ull;
#pragma unroll
    for (int b = 0; b < 9; ++b) {
        const bool bit = (dgt >> b) & 1;
        const unsigned long long B = __ballot(bit);
        m &= bit ? B : ~B;
    }
    return m;
}
__device__ __forceinline__ int lanes_below(unsigned long long m) {
    return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

// A pass is idle iff one digit bin holds all n elements.  Every wave of every kernel evaluates this
// the same way from the digit totals (call with all 64 lanes active).
__device__ __forceinline__ bool pass_active(const unsigned *__restrict__ gtot, int p, int n) {
    bool idle = false;
    for (int d = (int)threadIdx.x & 63; d < kDigits; d += kWave) idle |= gtot[p * kDigits + d] == (unsigned)n;
    return __ballot(idle) == 0ull;
}
// Buffer (0 or 1) that holds the data before pass p: the parity of the active passes before it.
__device__ __forceinline__ int source_buffer(const unsigned *__restrict__ gtot, int p, int n) {
    int moved = 0;
    for (int q = 0; q < p; ++q) moved += pass_active(gtot, q, n) ? 1 : 0;
    return moved & 1;
}

// Every later kernel copies the digit totals (3 KiB) into LDS first: pass_active / source_buffer read them
// many times over.  Returns whether the codes of counts >= kRankExact are their low bits: the usual ones leave out bits that
// differ, and all those counts agree above the low bits, in bits that are not all zero (smaller counts share their codes too
// seldom for the counts to be read again in every pass).
// differ: the usual codes leave out bits that differ.
__device__ __forceinline__ bool stage_totals(const SortBufs &b, unsigned *gs, bool &differ) {
    // (one request for the four words, and no branch on one before the others)
    const unsigned long long left_out = b.rest[0] & b.rest[1], above = b.rest[2], above_differ = b.rest[2] & b.rest[3];
    differ = left_out != 0ull;
    const bool low = (above != 0ull) & (above_differ == 0ull) & differ;      // (uniform)
    if (threadIdx.x < kPasses * kDigits) {
        unsigned t = b.gtot[threadIdx.x];      // (requested with the flags)
        if (low) t += b.gtot[kPasses * kDigits + threadIdx.x];
        gs[threadIdx.x] = t;
    }
    __syncthreads();
    return low;
}
static_assert(kPasses * kDigits <= kRankSortThreads, "one total per thread");
// What a pass sorts the element of this pair by.
__device__ __forceinline__ unsigned sort_key(unsigned long long pair, bool low, const long long *__restrict__ counts) {
    const unsigned code = (unsigned)(pair >> 32);
    return low && code >= kRankExact ? low_code((unsigned long long)counts[(unsigned)pair]) : code;
}

__global__ void __launch_bounds__(kRankSortThreads) rsort_zero_kernel(unsigned *gtot) {
    for (int i = threadIdx.x; i < kTotals + 8; i += kRankSortThreads) gtot[i] = 0u;      // (and `rest` behind them)
}

__global__ void __launch_bounds__(kRankSortThreads) rsort_init_kernel(const long long *__restrict__ counts, int n,
                                                                      SortBufs b) {
    __shared__ unsigned h[kTotals];
    __shared__ unsigned long long s_rest[4];
    const int j = blockIdx.x * kRankSortThreads + threadIdx.x;
    const bool in = j < n;
    const unsigned long long c = in ? (unsigned long long)counts[j] : 0ull;
    const unsigned code = count_code<19, 18>(c);
    for (int i = threadIdx.x; i < kTotals; i += kRankSortThreads) h[i] = 0u;
    if (threadIdx.x < 4) s_rest[threadIdx.x] = 0ull;
    __syncthreads();
    if (in) b.pairs[0][j] = ((unsigned long long)code << 32) | (unsigned)j;
    // the upper digits are the same in nearly every code (zero): when a whole wave agrees on a digit one lane
    // adds for all, instead of 64 LDS atomics queueing on one address
    const unsigned long long live = __ballot(in);
#pragma unroll
    for (int p = 0; p < kPasses; ++p) {
        const int dg = (int)((code >> (8 * p)) & 255u);
        const int first = __builtin_amdgcn_readfirstlane(dg);
        const unsigned long long same = __ballot(in && dg == first);
        if (same == live && live != 0ull) {
            if ((threadIdx.x & 63) == (unsigned)(__ffsll((long long)live) - 1))
                atomicAdd(&h[p * kDigits + dg], (unsigned)__popcll(live));
        } else if (in) {
            atomicAdd(&h[p * kDigits + dg], 1u);
        }
    }
    const bool large = code >= kRankExact;
    const unsigned long long any_large = __ballot(large);
    if (any_large != 0ull) {
        const unsigned long long left_out = large ? c & low_bits(63 - __clzll((long long)c) - 18) : 0ull;
        const unsigned long long r[4] = {left_out, large ? ~left_out : 0ull, large ? c >> kLowBits : 0ull, large ? ~(c >> kLowBits) : 0ull};
        if (any_large != live) {      // (a few lanes, as a rule)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (large) atomicOr(&s_rest[q], r[q]);
            }
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const unsigned long long v = wave_or_u64(r[q]);
                if ((threadIdx.x & 63) == 0) atomicOr(&s_rest[q], v);
            }
        }
        const unsigned other = low_code(c);
#pragma unroll
        for (int p = 0; p < kPasses; ++p) {
            const unsigned from = (code >> (8 * p)) & 255u, to = (other >> (8 * p)) & 255u;
            if (large && from != to) {
                atomicAdd(&h[(kPasses + p) * kDigits + from], ~0u);      // (one less; sums wrap around)
                atomicAdd(&h[(kPasses + p) * kDigits + to], 1u);
            }
        }
    }
    __syncthreads();
    const int tid = threadIdx.x;
    if (tid < kPasses * kDigits && h[tid] != 0u) atomicAdd(&b.gtot[tid], h[tid]);
    if (tid < kDigits) {
        b.hist[blockIdx.x * kDigits + tid] = h[255 - tid];
        b.hist_low[blockIdx.x * kDigits + tid] = h[255 - tid] + h[kPasses * kDigits + 255 - tid];
    }
    if (s_rest[3] != 0ull) {      // (uniform) there are counts of 2^19 and more
        if (tid < 4) atomicOr(&b.rest[tid], s_rest[tid]);
        if (tid < kPasses * kDigits && h[kPasses * kDigits + tid] != 0u) atomicAdd(&b.gtot[kPasses * kDigits + tid], h[kPasses * kDigits + tid]);
    }
}

__global__ void __launch_bounds__(kRankSortThreads) rsort_hist_kernel(const long long *__restrict__ counts, int n, int p,
                                                                      SortBufs b) {
    __shared__ unsigned h[kDigits];
    __shared__ unsigned gs[kPasses * kDigits];
    bool differ;
    const bool low = stage_totals(b, gs, differ);
    if (!pass_active(gs, p, n)) return;
    const int src = source_buffer(gs, p, n);
    const int j = blockIdx.x * kRankSortThreads + threadIdx.x;
    const unsigned code = j < n ? sort_key(b.pairs[src][j], low, counts) : 0u;
    if (threadIdx.x < kDigits) h[threadIdx.x] = 0u;
    __syncthreads();
    if (j < n) atomicAdd(&h[255 - (int)((code >> (8 * p)) & 255u)], 1u);
    __syncthreads();
    if (threadIdx.x < kDigits) b.hist[blockIdx.x * kDigits + threadIdx.x] = h[threadIdx.x];
}

__global__ void __launch_bounds__(kRankSortThreads) rsort_scatter_kernel(const long long *__restrict__ counts, int n, int p,
                                                                         SortBufs b) {
    __shared__ unsigned wcnt[kSortWaves * kDigits];   // [wave][digit]: elements of that digit in earlier waves
    __shared__ unsigned part[4 * kDigits];            // sums over a quarter of the earlier workgroups
    __shared__ unsigned offs[kDigits];                // first output slot of this workgroup's run of each digit
    __shared__ unsigned gs[kPasses * kDigits];
    bool differ;
    const bool low = stage_totals(b, gs, differ);
    if (!pass_active(gs, p, n)) return;
    const int src = source_buffer(gs, p, n);
    const unsigned *hist = low && p == 0 ? b.hist_low : b.hist;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int blk = blockIdx.x;

    // (requested ahead of the offsets: it depends on nothing)
    const int j = blk * kRankSortThreads + tid;
    const bool in = j < n;
    const unsigned long long pair = in ? b.pairs[src][j] : 0ull;
    const unsigned key = in ? sort_key(pair, low, counts) : 0u;
    for (int i = tid; i < kSortWaves * kDigits; i += kRankSortThreads) wcnt[i] = 0u;
    // this workgroup's offsets: (elements with an earlier digit anywhere) + (same digit, earlier workgroups)
    {
        // (a wave reads 64 digits of one workgroup's row at a time, a quarter of the earlier workgroups per thread)
        const int d = tid & 255, q = tid >> 8;
        unsigned before = 0;
        const int b1 = blk * (q + 1) / 4;
        const unsigned *col = hist + d;
        int x = blk * q / 4;
        for (; x + 16 <= b1; x += 16) {         // sixteen independent loads at a time
            unsigned t[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) t[u] = col[(size_t)(x + u) * kDigits];
#pragma unroll
            for (int u = 0; u < 16; ++u) before += t[u];
        }
        for (; x < b1; ++x) before += col[(size_t)x * kDigits];
        part[q * kDigits + d] = before;
    }
    unsigned tot = 0, inc = 0;
    if (tid < kDigits) {
        tot = gs[p * kDigits + (255 - tid)];          // digit totals in descending-digit order
        inc = tot;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {         // inclusive scan inside each of the four waves
            const unsigned t = __shfl_up(inc, o);
            if (lane >= o) inc += t;
        }
        offs[tid] = inc;
    }
    __syncthreads();
    unsigned my_off = 0;
    if (tid < kDigits) {
        unsigned carry = 0;
        for (int ww = 0; ww < w; ++ww) carry += offs[ww * kWave + kWave - 1];
        my_off = carry + inc - tot + part[tid] + part[kDigits + tid] + part[2 * kDigits + tid] + part[3 * kDigits + tid];
    }
    __syncthreads();
    if (tid < kDigits) offs[tid] = my_off;

    // ---- ranks inside the workgroup
    const int dgt = in ? 255 - (int)((key >> (8 * p)) & 255u) : 256;
    const unsigned long long m = match_digit9(dgt);
    const int below = lanes_below(m);
    if (in && below == 0) wcnt[w * kDigits + dgt] = (unsigned)__popcll(m);
    __syncthreads();
    if (tid < kDigits) {
        unsigned run = 0;
        for (int ww = 0; ww < kSortWaves; ++ww) {
            const unsigned c = wcnt[ww * kDigits + tid];
            wcnt[ww * kDigits + tid] = run;
            run += c;
        }
    }
    __syncthreads();
    if (in) {
        const unsigned pos = offs[dgt] + wcnt[w * kDigits + dgt] + (unsigned)below;
        b.pairs[src ^ 1][pos] = pair;
    }
}

// ---- runs of equal codes whose counts differ (rsort_out)
constexpr int kShortRun = 16;                        // ordered by counting in every id's thread
constexpr int kWaveRun = 4 * kWave;                  // ... in a wave of the workgroup that the run starts in
constexpr int kGroupRun = kRankSortThreads;          // ... in that workgroup; longer: radix passes
constexpr int kRunPer = 4;                           // elements per thread and step of those
constexpr int kRunStep = kRunPer * kRankSortThreads, kRunGroups = kRunStep / kWave;

struct RunLds {
    int starts[kRankSortThreads / kShortRun + 1], long_starts[kRankSortThreads / kShortRun + 1];
    int n_starts, n_long, n_same;
    unsigned long long ones, zeros;
    unsigned base[kDigits];                          // next slot of each digit, descending
    unsigned part[kRunPer * kDigits];
    union {
        unsigned long long wave_count[kSortWaves][kWaveRun];      // run_key
        unsigned long long count[kGroupRun];
        unsigned short before[kRunGroups * kDigits]; // elements of a digit in the step's groups of 64 before
    };
};

// (count descending, place in the run ascending) as one number: the bits that a run's counts share may go
__device__ __forceinline__ unsigned long long run_key(long long c, int place) {
    return ((unsigned long long)c << 10) | (unsigned)(kGroupRun - 1 - place);
}
static_assert(kGroupRun == 1 << 10, "ten bits for the place; codes tell 19 bits apart");
// f(v[x]) for all x < n, eight of them read at a time (every lane the same one: a broadcast).
template <typename F>
__device__ __forceinline__ void for_each_key(const unsigned long long *v, int n, F &&f) {
    int x = 0;
    for (; x + 8 <= n; x += 8) {
        unsigned long long t[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) t[q] = v[x + q];
#pragma unroll
        for (int q = 0; q < 8; ++q) f(t[q]);
    }
    for (; x < n; ++x) f(v[x]);
}

// One run [lo, lo + length), longer than kGroupRun, by its counts: LSD passes of this workgroup over the digits in which the
// counts differ, between the two buffers.  Nobody else touches the run's ids (its codes stay what they are).
__device__ __forceinline__ void sort_long_run(const long long *__restrict__ counts, const SortBufs &b, int src, unsigned lo,
                                              unsigned length, int n_ids, int *__restrict__ out_ids, RunLds &s) {
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    if (tid == 0) s.ones = s.zeros = 0ull;
    __syncthreads();
    unsigned long long ones = 0, zeros = 0;
    for (unsigned x = tid; x < length; x += kRankSortThreads) {
        const unsigned long long c = (unsigned long long)counts[(unsigned)b.pairs[src][lo + x]];
        ones |= c;
        zeros |= ~c;
    }
    ones = wave_or_u64(ones);
    zeros = wave_or_u64(zeros);
    if (lane == 0) {
        atomicOr(&s.ones, ones);
        atomicOr(&s.zeros, zeros);
    }
    __syncthreads();
    const unsigned long long differ = s.ones & s.zeros;
    for (int shift = 0; shift < 64; shift += 8) {
        if (((differ >> shift) & 255ull) == 0ull) continue;      // (uniform)
        const unsigned long long *from = b.pairs[src] + lo;
        unsigned long long *to = b.pairs[src ^ 1] + lo;
        // element x0 + (u 16 + w) 64 + lane of the run, and 255 - its digit (256: past the end)
        unsigned long long pair[kRunPer];
        int dgt[kRunPer];
        auto load_step = [&](unsigned x0) {
#pragma unroll
            for (int u = 0; u < kRunPer; ++u) {
                const unsigned x = x0 + u * kRankSortThreads + tid;
                pair[u] = x < length ? from[x] : 0ull;
            }
#pragma unroll
            for (int u = 0; u < kRunPer; ++u) {
                const unsigned x = x0 + u * kRankSortThreads + tid;
                dgt[u] = x < length ? 255 - (int)(((unsigned long long)counts[(unsigned)pair[u]] >> shift) & 255ull) : 256;
            }
        };
        if (tid < kDigits) s.base[tid] = 0u;
        __syncthreads();
        for (unsigned x0 = 0; x0 < length; x0 += kRunStep) {
            load_step(x0);
#pragma unroll
            for (int u = 0; u < kRunPer; ++u) wave_tally(s.base, dgt[u], dgt[u] < kDigits);
        }
        __syncthreads();
        // counts of the digits -> first slots: four waves scan, then add what lies in the waves before
        unsigned mine = 0, inc = 0;
        if (tid < kDigits) {
            mine = inc = s.base[tid];
#pragma unroll
            for (int o = 1; o < kWave; o <<= 1) {
                const unsigned t = __shfl_up(inc, o);
                if (lane >= o) inc += t;
            }
            if (lane == kWave - 1) s.part[w] = inc;
        }
        __syncthreads();
        if (tid < kDigits) {
            for (int ww = 0; ww < w; ++ww) inc += s.part[ww];
            s.base[tid] = inc - mine;
        }
        for (unsigned x0 = 0; x0 < length; x0 += kRunStep) {
            load_step(x0);
            unsigned long long same[kRunPer];
#pragma unroll
            for (int u = 0; u < kRunPer; ++u) same[u] = match_digit9(dgt[u]);
            __syncthreads();            // the step before is done with `before`, `part` and `base`
            for (int i = tid; i < kRunGroups * kDigits / 2; i += kRankSortThreads) reinterpret_cast<unsigned *>(s.before)[i] = 0u;
            __syncthreads();
#pragma unroll
            for (int u = 0; u < kRunPer; ++u) {
                if (dgt[u] < kDigits && lanes_below(same[u]) == 0)
                    s.before[(u * kSortWaves + w) * kDigits + dgt[u]] = (unsigned short)__popcll(same[u]);
            }
            __syncthreads();
            {
                // thread (digit, quarter u of the groups)
                const int d = tid & 255, q = tid >> 8;
                unsigned run = 0;
#pragma unroll
                for (int i = 0; i < kSortWaves; ++i) {
                    unsigned short &x = s.before[(q * kSortWaves + i) * kDigits + d];
                    const unsigned c = x;
                    x = (unsigned short)run;
                    run += c;
                }
                s.part[q * kDigits + d] = run;
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < kRunPer; ++u) {
                if (dgt[u] < kDigits) {
                    unsigned pos = s.base[dgt[u]] + s.before[(u * kSortWaves + w) * kDigits + dgt[u]] + (unsigned)lanes_below(same[u]);
#pragma unroll
                    for (int q = 0; q < u; ++q) pos += s.part[q * kDigits + dgt[u]];
                    to[pos] = pair[u];
                }
            }
            __syncthreads();
            if (tid < kDigits) {
#pragma unroll
                for (int q = 0; q < kRunPer; ++q) s.base[tid] += s.part[q * kDigits + tid];
            }
        }
        __syncthreads();                // what was written is read by other waves
        src ^= 1;
    }
    static_assert(kRunPer * kDigits == kRankSortThreads, "a thread per digit and quarter");
    for (unsigned x = tid; x < length && lo + x < (unsigned)n_ids; x += kRankSortThreads)
        out_ids[lo + x] = (int)(unsigned)b.pairs[src][lo + x];
    __syncthreads();
}

__global__ void __launch_bounds__(kRankSortThreads) rsort_out_kernel(const long long *__restrict__ counts, int n, int n_ids, SortBufs b,
                                                                     int *__restrict__ out_ids) {
    __shared__ unsigned gs[kPasses * kDigits];
    __shared__ RunLds s;
    bool differ;
    const bool low = stage_totals(b, gs, differ);
    const int src = source_buffer(gs, kPasses, n);
    const unsigned long long *pairs = b.pairs[src];      // (sort_long_run writes there)
    const int tid = threadIdx.x;
    const unsigned j = blockIdx.x * kRankSortThreads + tid;
    const bool in = j < (unsigned)n;
    const unsigned long long pair = in ? pairs[j] : 0ull;
    const int id = (int)(unsigned)pair;
    if (low || !differ) {      // (uniform) the codes leave out nothing that differs
        if (in && j < (unsigned)n_ids) out_ids[j] = id;
        return;
    }
    const unsigned code = (unsigned)(pair >> 32);
    auto code_of = [&](unsigned x) { return (unsigned)(pairs[x] >> 32); };
    if (tid == 0) s.n_starts = s.n_long = 0;
    __syncthreads();
    if (in) {
        int before = 0, after = 0;
        if (code >= kRankExact) {
            while (before < kShortRun && before < (int)j && code_of(j - 1 - before) == code) ++before;
            while (after < kShortRun && (unsigned)after + 1 < (unsigned)n - j && code_of(j + 1 + after) == code) ++after;
        }
        if (before + after + 1 <= kShortRun) {
            // the order among themselves (the run is in ascending-id order)
            unsigned pos = j;
            if (before + after > 0) {
                const long long c = counts[id];
                for (int x = 1; x <= before; ++x) pos -= counts[(unsigned)pairs[j - x]] < c ? 1u : 0u;      // goes behind
                for (int x = 1; x <= after; ++x) pos += counts[(unsigned)pairs[j + x]] > c ? 1u : 0u;       // goes ahead
            }
            if (pos < (unsigned)n_ids) out_ids[pos] = id;
        } else if (before == 0) {
            s.starts[atomicAdd(&s.n_starts, 1)] = (int)j;      // (more than kShortRun apart)
        }
    }
    __syncthreads();
    const int n_starts = s.n_starts;
    if (n_starts == 0) return;      // (as a rule; the code below is far from being fetched)
    const int lane = tid & 63, w = tid >> 6;
    for (int q = w; q < n_starts; q += kSortWaves) {
        const unsigned lo = (unsigned)s.starts[q];
        if (lo >= (unsigned)n_ids) continue;      // nobody asks for them
        const unsigned run_code = code_of(lo);
        unsigned long long p[kWaveRun / kWave];
        int length = 0;
#pragma unroll
        for (int u = 0; u < kWaveRun / kWave; ++u) p[u] = lo + u * kWave + lane < (unsigned)n ? pairs[lo + u * kWave + lane] : 0ull;
#pragma unroll
        for (int u = 0; u < kWaveRun / kWave; ++u) length += __popcll(__ballot((unsigned)(p[u] >> 32) == run_code));
        if (length == kWaveRun && lo + kWaveRun < (unsigned)n && code_of(lo + kWaveRun) == run_code) {
            if (lane == 0) s.long_starts[atomicAdd(&s.n_long, 1)] = (int)lo;
            continue;
        }
        unsigned long long c[kWaveRun / kWave];
#pragma unroll
        for (int u = 0; u < kWaveRun / kWave; ++u) {
            const bool mine = u * kWave + lane < length;
            c[u] = mine ? run_key(counts[(unsigned)p[u]], u * kWave + lane) : 0ull;
            if (mine) s.wave_count[w][u * kWave + lane] = c[u];
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        unsigned pos[kWaveRun / kWave] = {};
        for_each_key(s.wave_count[w], length, [&](unsigned long long other) {
#pragma unroll
            for (int u = 0; u < kWaveRun / kWave; ++u) pos[u] += other > c[u] ? 1u : 0u;
        });
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int u = 0; u < kWaveRun / kWave; ++u) {
            if (u * kWave + lane < length && lo + pos[u] < (unsigned)n_ids) out_ids[lo + pos[u]] = (int)(unsigned)p[u];
        }
    }
    __syncthreads();
    const int n_long = s.n_long;
    for (int q = 0; q < n_long; ++q) {
        const unsigned lo = (unsigned)s.long_starts[q];
        const unsigned run_code = code_of(lo);
        // the run's end: element a has the code, element e (if there is one) has not
        unsigned a = lo, e = (unsigned)n;
        while (e - a > 1) {
            const unsigned step = (e - a + kRankSortThreads - 1) / kRankSortThreads;
            const unsigned off = (unsigned)tid * step;
            const bool same = off < e - a && code_of(a + off) == run_code;
            const int c = __popcll(__ballot(same));
            __syncthreads();
            if (tid == 0) s.n_same = 0;
            __syncthreads();
            if (lane == 0 && c != 0) atomicAdd(&s.n_same, c);
            __syncthreads();
            const unsigned n_same = (unsigned)s.n_same;      // (the first ones: a itself, and on)
            if (n_same * step < e - a) e = a + n_same * step;
            a += (n_same - 1) * step;
        }
        const unsigned length = e - lo;
        if (length > kGroupRun) {
            sort_long_run(counts, b, src, lo, length, n_ids, out_ids, s);
            continue;
        }
        const bool mine = (unsigned)tid < length;
        const int my_id = mine ? (int)(unsigned)pairs[lo + tid] : 0;
        const unsigned long long c = mine ? run_key(counts[my_id], tid) : 0ull;
        __syncthreads();
        s.count[tid] = c;
        __syncthreads();
        if (mine) {
            unsigned pos = lo;
            for_each_key(s.count, (int)length, [&](unsigned long long other) { pos += other > c ? 1u : 0u; });
            if (pos < (unsigned)n_ids) out_ids[pos] = my_id;
        }
    }
}

}  // namespace

// ---------------------------------------------------------------- choice of k
// out[0] = k, out[1] = mass of the k largest counts, out[2] = total mass.
//   mode 0: smallest k >= 1 with S_k >= ceil(P * total);  mode 1: k = #{c >= f_min}.
namespace {

constexpr int kWideBins = kBins - kBinExact;      // bins of more than one value: their mass is summed
// of the bin that is divided: digits of its ids, their mass, and the bits below its prefix that are set in any / clear in any
struct ChooseBufs {
    unsigned long long *mass;          // [kWideBins]
    unsigned long long *digit_mass;    // [kDigitBins]
    unsigned long long *bits;          // [2]
    unsigned *hist;                    // [kBins]
    unsigned *digits;                  // [kDigitBins]
    unsigned *done;                    // [2] workgroups that have added theirs
};
constexpr int kChooseZeroWords = kWideBins + kDigitBins + 2 + (kBins + kDigitBins + 2) / 2;      // 64-bit words, mass .. done
static_assert((kBins + kDigitBins) % 2 == 0, "whole 64-bit words");

__global__ void __launch_bounds__(kRankSortThreads) choose_zero_kernel(ChooseBufs b) {
    const int i = blockIdx.x * kRankSortThreads + threadIdx.x;
    if (i < kChooseZeroWords) b.mass[i] = 0ull;
}
__global__ void __launch_bounds__(64) choose_clear_kernel(long long *__restrict__ out) {
    if (threadIdx.x < 3) out[threadIdx.x] = 0;
}

__device__ __forceinline__ long long wave_sum_i64(long long v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// mode 1: everything there is to do, by atomics on `out`
__global__ void __launch_bounds__(kRankSortThreads) choose_min_kernel(const long long *__restrict__ counts, int V, long long f_min,
                                                                      long long *__restrict__ out) {
    const int j = blockIdx.x * kRankSortThreads + threadIdx.x;
    const long long c = j < V ? counts[j] : 0;
    const long long kept = j < V && c >= f_min ? 1 : 0;
    const long long n = wave_sum_i64(kept), mass = wave_sum_i64(kept ? c : 0), total = wave_sum_i64(c);
    __shared__ long long red[3][kSortWaves];
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        red[0][w] = n;
        red[1][w] = mass;
        red[2][w] = total;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        long long t = 0;
        for (int q = 0; q < kSortWaves; ++q) t += red[threadIdx.x][q];
        if (t != 0) atomicAdd(reinterpret_cast<unsigned long long *>(&out[threadIdx.x]), (unsigned long long)t);
    }
}

// As wave_tally, with the mass c of the ids; digits below `exact` have none (it follows from their number).
__device__ __forceinline__ void wave_tally_mass(unsigned *h, unsigned long long *m, int exact, int d, bool in, unsigned long long c) {
    const unsigned long long live = __ballot(in);
    if (live == 0ull) return;
    const int leader = __ffsll((long long)live) - 1;
    const int first = __builtin_amdgcn_readlane(d, leader);
    const bool same = in && d == first;
    const unsigned long long group = __ballot(same);
    if (in && !same) {
        atomicAdd(&h[d], 1u);
        if (d >= exact) atomicAdd(&m[d - exact], c);
    }
    if (lane_id() == leader) atomicAdd(&h[first], (unsigned)__popcll(group));
    if (first >= exact) {
        if (__popcll(group) <= 8) {      // (few lanes queue faster than a sum over the wave is made)
            if (same) atomicAdd(&m[first - exact], c);
        } else {
            const long long sum = wave_sum_i64(same ? (long long)c : 0ll);
            if (lane_id() == leader) atomicAdd(&m[first - exact], (unsigned long long)sum);
        }
    }
}

// The counts of this workgroup (all of them when gridDim.x = 1) into bins of LDS, ids and -- above 2048 -- mass.
__device__ __forceinline__ void bin_counts(const long long *__restrict__ counts, int V, unsigned *h, unsigned long long *m) {
    for (int i = threadIdx.x; i < kBins; i += kRankSortThreads) h[i] = 0u;
    for (int i = threadIdx.x; i < kWideBins; i += kRankSortThreads) m[i] = 0ull;
    __syncthreads();
    for (unsigned base = blockIdx.x * kRankSortThreads; base < (unsigned)V; base += gridDim.x * kRankSortThreads) {
        const bool in = base + threadIdx.x < (unsigned)V;
        const unsigned long long c = in ? (unsigned long long)counts[base + threadIdx.x] : 0ull;
        wave_tally_mass(h, m, kBinExact, count_bin(c), in, c);
    }
    __syncthreads();
}

__global__ void __launch_bounds__(kRankSortThreads) choose_hist_kernel(const long long *__restrict__ counts, int V, ChooseBufs b) {
    __shared__ unsigned h[kBins];
    __shared__ unsigned long long m[kWideBins];
    bin_counts(counts, V, h, m);
    for (int i = threadIdx.x; i < kBins; i += kRankSortThreads) {
        if (h[i] != 0u) atomicAdd(&b.hist[i], h[i]);
    }
    for (int i = threadIdx.x; i < kWideBins; i += kRankSortThreads) {
        if (m[i] != 0ull) atomicAdd(&b.mass[i], m[i]);
    }
}

// Inclusive prefix sums of (ids, mass) over the workgroup's threads.  Two barriers.
__device__ __forceinline__ void block_scan2(unsigned &n, unsigned long long &mass, unsigned *pn, unsigned long long *pm) {
    const int lane = lane_id(), w = (int)threadIdx.x >> 6;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const unsigned tn = __shfl_up(n, o);
        const unsigned long long tm = __shfl_up(mass, o);
        if (lane >= o) {
            n += tn;
            mass += tm;
        }
    }
    if (lane == kWave - 1) {
        pn[w] = n;
        pm[w] = mass;
    }
    __syncthreads();
    unsigned bn = 0;
    unsigned long long bm = 0;
    for (int q = 0; q < w; ++q) {
        bn += pn[q];
        bm += pm[q];
    }
    __syncthreads();
    n += bn;
    mass += bm;
}

// DIRECT: one workgroup, which bins all counts itself (small V).
constexpr int kChooseMaxBlocks = 128;
template <bool DIRECT>
__global__ void __launch_bounds__(kRankSortThreads) choose_mass_kernel(const long long *__restrict__ counts, int V, double P,
                                                                       ChooseBufs b, long long *__restrict__ out) {
    __shared__ unsigned h[DIRECT ? kBins : kDigitBins];
    __shared__ unsigned long long m[kDigitBins > kWideBins ? kDigitBins : kWideBins];
    __shared__ unsigned pn[kSortWaves];
    __shared__ unsigned long long pm[kSortWaves];
    __shared__ int s_bin, s_last;
    __shared__ unsigned s_n, s_ids;
    __shared__ unsigned long long s_m, s_mass, s_total, s_ones, s_zeros;
    constexpr int kPer = (kBins + kRankSortThreads - 1) / kRankSortThreads;
    const int tid = threadIdx.x, lane = tid & 63;
    if constexpr (DIRECT) bin_counts(counts, V, h, m);
    // bins from the highest down
    unsigned vn[kPer], n = 0;
    unsigned long long vm[kPer], mass = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int bin = kBins - 1 - (kPer * tid + i);
        vn[i] = bin < 0 ? 0u : DIRECT ? h[bin] : b.hist[bin];
        vm[i] = bin < 0 ? 0ull
                : bin < kBinExact ? (unsigned long long)vn[i] * (unsigned)bin
                                  : (DIRECT ? m[bin - kBinExact] : b.mass[bin - kBinExact]);
        n += vn[i];
        mass += vm[i];
    }
    unsigned upto_n = n;
    unsigned long long upto_m = mass;
    block_scan2(upto_n, upto_m, pn, pm);
    if (tid == kRankSortThreads - 1) s_total = upto_m;
    if (tid == 0) {
        s_bin = -1;
        s_ones = s_zeros = 0ull;
    }
    __syncthreads();
    const unsigned long long total = s_total;
    // one fp64 product, then its ceiling; never above the total (beyond 2^53 tokens the product of P = 1
    // can round up past it, and no prefix would reach it)
    const unsigned long long want = (unsigned long long)ceil(P * (double)(long long)total);
    const unsigned long long target = want > total ? total : want;
    // the first bin, from above, that holds ids and with which the mass reaches the target (k >= 1: a target of 0 too)
    auto reaches = [&](unsigned ids, unsigned long long ids_mass, unsigned above_n, unsigned long long above_m) {
        return ids != 0u && above_m + ids_mass >= target && (above_m < target || above_n == 0u);
    };
    auto found = [&](int bin, unsigned ids, unsigned long long ids_mass, unsigned above_n, unsigned long long above_m) {
        s_bin = bin;
        s_ids = ids;
        s_mass = ids_mass;
        s_n = above_n;
        s_m = above_m;
    };
    {
        unsigned above_n = upto_n - n;
        unsigned long long above_m = upto_m - mass;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            if (reaches(vn[i], vm[i], above_n, above_m)) found(kBins - 1 - (kPer * tid + i), vn[i], vm[i], above_n, above_m);
            above_n += vn[i];
            above_m += vm[i];
        }
    }
    __syncthreads();
    const int bin = s_bin;
    if (bin < 0) {      // no bin reaches it: counts below zero, or a mass of 2^63 and more
        if (blockIdx.x == 0 && tid < 3) out[tid] = tid == 2 ? (long long)total : 0;
        return;
    }
    // ids of count T, one after the other, until the target is reached; at least one
    auto finish = [&](unsigned long long T, unsigned before_n, unsigned long long before_m) {
        unsigned long long take = 1;
        if (target > before_m && T > 0) {
            take = (target - before_m + T - 1) / T;
            if (take > (unsigned)V - before_n) take = (unsigned)V - before_n;      // (only where the mass has wrapped around)
        }
        out[0] = (long long)(before_n + take);
        out[1] = (long long)(before_m + take * T);
        out[2] = (long long)total;
    };
    if (bin < kBinExact) {      // (not at the end of the kernel: its code would have to be fetched from there)
        if (blockIdx.x == 0 && tid == 0) finish((unsigned)bin, s_n, s_m);
        return;
    }
    // several values share the bin: the value at which the target is reached, digit by digit
    unsigned before_n = s_n, ids = s_ids;
    unsigned long long before_m = s_m, ids_mass = s_mass, T = bin_prefix(bin);
    int left = bin_shift(bin), nbits = left < kDigitBits ? left : kDigitBits;
    __syncthreads();                // (h and m are read, s_* too)
    auto clear = [&]() {
        for (int i = tid; i < kDigitBins; i += kRankSortThreads) {
            h[i] = 0u;
            m[i] = 0ull;
        }
        __syncthreads();
    };
    clear();
    {
        unsigned long long ones = 0, zeros = 0;
        for (unsigned base = blockIdx.x * kRankSortThreads; base < (unsigned)V; base += gridDim.x * kRankSortThreads) {
            const unsigned x = base + tid;
            const unsigned long long c = x < (unsigned)V ? (unsigned long long)counts[x] : 0ull;
            const bool in = (c >> left) == T;      // (zero past the end: T > 0)
            wave_tally_mass(h, m, 0, (int)((c >> (left - nbits)) & low_bits(nbits)), in, c);
            ones |= in ? c & low_bits(left) : 0ull;
            zeros |= in ? ~c & low_bits(left) : 0ull;
        }
        if (__ballot((ones | zeros) != 0ull) != 0ull) {
            ones = wave_or_u64(ones);
            zeros = wave_or_u64(zeros);
            if (lane == 0) {
                atomicOr(&s_ones, ones);
                atomicOr(&s_zeros, zeros);
            }
        }
        __syncthreads();
    }
    if constexpr (!DIRECT) {
        for (int i = tid; i < kDigitBins; i += kRankSortThreads) {
            if (h[i] != 0u) {
                atomicAdd(&b.digits[i], h[i]);
                atomicAdd(&b.digit_mass[i], m[i]);
            }
        }
        if (tid == 0 && (s_ones | s_zeros) != 0ull) {
            atomicOr(&b.bits[0], s_ones);
            atomicOr(&b.bits[1], s_zeros);
        }
        wait_stores_done();      // this wave's atomics have been performed
        __syncthreads();
        if (tid == 0) s_last = __hip_atomic_fetch_add(b.done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
        __syncthreads();
        if (!s_last) return;
        // the last workgroup goes on with everybody's digits
        for (int i = tid; i < kDigitBins; i += kRankSortThreads) {
            h[i] = __hip_atomic_load(&b.digits[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            m[i] = acquire_u64(&b.digit_mass[i]);
        }
        if (tid == 0) {
            s_ones = acquire_u64(&b.bits[0]);
            s_zeros = acquire_u64(&b.bits[1]);
        }
        __syncthreads();
    }
    const unsigned long long ones = s_ones, zeros = s_zeros;
    // Appends the digit at which the target is reached, of the ids in h and m.
    static_assert(kDigitBins == 2 * kRankSortThreads, "two digits per thread");
    auto find_digit = [&]() {
        const int d = kDigitBins - 1 - 2 * tid;      // and the one below
        const unsigned n0 = h[d], n1 = h[d - 1];
        const unsigned long long m0 = m[d], m1 = m[d - 1];
        unsigned un = n0 + n1;
        unsigned long long um = m0 + m1;
        if (tid == 0) found(0, 0u, 0ull, before_n, before_m);      // (found by some thread unless the mass wraps around)
        block_scan2(un, um, pn, pm);
        const unsigned above_n = before_n + un - n0 - n1;
        const unsigned long long above_m = before_m + um - m0 - m1;
        if (reaches(n0, m0, above_n, above_m)) found(d, n0, m0, above_n, above_m);
        if (reaches(n1, m1, above_n + n0, above_m + m0)) found(d - 1, n1, m1, above_n + n0, above_m + m0);
        __syncthreads();
        T = (T << nbits) | (unsigned)s_bin;
        left -= nbits;
        before_n = s_n;
        before_m = s_m;
        ids = s_ids;
        ids_mass = s_mass;
        __syncthreads();
    };
    find_digit();
    while (left > 0) {
        if (ids == 1u) {      // its mass is its count
            T = ids_mass;
            break;
        }
        left = skip_common_bits(T, left, ones, zeros);
        if (left == 0) break;
        nbits = left < kDigitBits ? left : kDigitBits;
        clear();
        constexpr int kInFlight = 8;
        for (unsigned x0 = 0; x0 < (unsigned)V; x0 += kInFlight * kRankSortThreads) {
            unsigned long long cx[kInFlight];
#pragma unroll
            for (int u = 0; u < kInFlight; ++u) {
                const unsigned x = x0 + u * kRankSortThreads + tid;
                cx[u] = x < (unsigned)V ? (unsigned long long)counts[x] : 0ull;
            }
#pragma unroll
            for (int u = 0; u < kInFlight; ++u)
                wave_tally_mass(h, m, 0, (int)((cx[u] >> (left - nbits)) & low_bits(nbits)), (cx[u] >> left) == T, cx[u]);
        }
        __syncthreads();
        find_digit();
    }
    if (tid == 0) finish(T, before_n, before_m);
}

}  // namespace

// (an earlier layout's size, which callers may have stored: two buffers of keys and ids, digit tables of eight passes)
size_t rank_sort_scratch_bytes(int n) {
    const size_t kb = round256((size_t)n * 8), ib = round256((size_t)n * 4);
    const size_t nblk = ((size_t)n + kRankSortThreads - 1) / kRankSortThreads;
    return 2 * kb + 2 * ib + round256(8 * kDigits * 4) + round256(kDigits * nblk * 4);
}

// Sorts all n ids by (count desc, id asc); writes the first n_ids of them.
void launch_rank_sort(const long long *counts, int n, void *scratch, int *out_ids, int n_ids, hipStream_t st) {
    char *p = static_cast<char *>(scratch);
    const size_t kb = round256((size_t)n * 8);
    const int nblk = (n + kRankSortThreads - 1) / kRankSortThreads;
    SortBufs b;
    b.pairs[0] = reinterpret_cast<unsigned long long *>(p);
    b.pairs[1] = reinterpret_cast<unsigned long long *>(p + kb);
    b.gtot = reinterpret_cast<unsigned *>(p + 2 * kb);
    b.rest = reinterpret_cast<unsigned long long *>(b.gtot + kTotals);
    b.hist = reinterpret_cast<unsigned *>(p + 2 * kb + round256((kTotals + 8) * 4));
    b.hist_low = b.hist + (size_t)nblk * kDigits;
    hipLaunchKernelGGL(rsort_zero_kernel, dim3(1), dim3(kRankSortThreads), 0, st, b.gtot);
    hipLaunchKernelGGL(rsort_init_kernel, dim3(nblk), dim3(kRankSortThreads), 0, st, counts, n, b);
    for (int pass = 0; pass < kPasses; ++pass) {
        if (pass > 0) hipLaunchKernelGGL(rsort_hist_kernel, dim3(nblk), dim3(kRankSortThreads), 0, st, counts, n, pass, b);
        hipLaunchKernelGGL(rsort_scatter_kernel, dim3(nblk), dim3(kRankSortThreads), 0, st, counts, n, pass, b);
    }
    hipLaunchKernelGGL(rsort_out_kernel, dim3(nblk), dim3(kRankSortThreads), 0, st, counts, n, n_ids, b, out_ids);
}

// (likewise: ids and counts in order, sums per workgroup, and the sort's buffers)
size_t choose_k_ws_bytes(int V) {
    return round256((size_t)V * 4) + round256((size_t)V * 8) +
           round256((((size_t)V + kRankSortThreads - 1) / kRankSortThreads) * sizeof(long long)) + rank_sort_scratch_bytes(V);
}

void launch_choose_k(const long long *counts, int V, int mode, double P, long long f_min, void *scratch, long long *out,
                     hipStream_t st) {
    const int nblk = (V + kRankSortThreads - 1) / kRankSortThreads;
    ChooseBufs b;
    b.mass = static_cast<unsigned long long *>(scratch);
    b.hist = reinterpret_cast<unsigned *>(b.mass + kWideBins);      // (every array on whole cache lines)
    b.digit_mass = reinterpret_cast<unsigned long long *>(b.hist + kBins);
    b.digits = reinterpret_cast<unsigned *>(b.digit_mass + kDigitBins);
    b.bits = reinterpret_cast<unsigned long long *>(b.digits + kDigitBins);
    b.done = reinterpret_cast<unsigned *>(b.bits + 2);
    if (mode == 0 && V <= kChooseDirectMaxV) {
        hipLaunchKernelGGL(choose_mass_kernel<true>, dim3(1), dim3(kRankSortThreads), 0, st, counts, V, P, b, out);
        return;
    }
    if (mode != 0) {
        hipLaunchKernelGGL(choose_clear_kernel, dim3(1), dim3(64), 0, st, out);
        hipLaunchKernelGGL(choose_min_kernel, dim3(nblk), dim3(kRankSortThreads), 0, st, counts, V, f_min, out);
        return;
    }
    hipLaunchKernelGGL(choose_zero_kernel, dim3((kChooseZeroWords + kRankSortThreads - 1) / kRankSortThreads),
                       dim3(kRankSortThreads), 0, st, b);
    hipLaunchKernelGGL(choose_hist_kernel, dim3(nblk), dim3(kRankSortThreads), 0, st, counts, V, b);
    // (every workgroup walks the bins, so no more of them than a division needs)
    hipLaunchKernelGGL(choose_mass_kernel<false>, dim3(nblk < kChooseMaxBlocks ? nblk : kChooseMaxBlocks), dim3(kRankSortThreads), 0, st, counts, V, P, b, out);
}

}  // namespace vt
