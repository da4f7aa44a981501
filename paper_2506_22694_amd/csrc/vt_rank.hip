// Frequency-rank order and the alternative choices of k (Sec. 3.2: besides a fixed k, Top-P over
// the counts or a minimum-frequency threshold select the trimmed vocabulary).
//
// Rank order = all V ids sorted by (count descending, id ascending), the order in which
// Top-K(c, k) takes ids; every prefix is the selection for a smaller k.
//
// rsort_*: stable LSD radix sort over the whole device of (code, id) pairs, 8 bits per pass.  The code (vt_code.h) is
//   the count itself below 2^19 and its 19 highest bits with their exponent above -- 24 bits, three passes for any
//   int64.  The ids start ascending and every pass is stable, so equal codes stay in ascending-id order; where counts
//   of 2^19 and more share a code (a handful of ids, if any) the last kernel orders them by counting.
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
//   (Eight passes over the bytes of the counts, nineteen launches, took 72 us at V = 128256 after 10^7 tokens; now 42.)
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
    unsigned *gtot;      // [kPasses][kDigits] digit totals over all elements
    // what the codes of counts >= kRankExact leave out: the bits set in any of them, and those clear in any
    unsigned long long *rest;
    unsigned *hist;      // [nblk][kDigits] per-workgroup digit counts of the current pass, descending digit first
};

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

// Every later kernel copies the digit totals (8 KiB) into LDS first: pass_active / source_buffer read them
// many times over.
template <int T>
__device__ __forceinline__ void stage_totals(const unsigned *__restrict__ gtot, unsigned *gs) {
    for (int i = threadIdx.x; i < kPasses * kDigits; i += T) gs[i] = gtot[i];
    __syncthreads();
}

__global__ void __launch_bounds__(256) rsort_zero_kernel(unsigned *gtot) {
    for (int i = threadIdx.x; i < kPasses * kDigits + 4; i += 256) gtot[i] = 0u;      // (and `rest` behind them)
}

__global__ void __launch_bounds__(kRankSortThreads) rsort_init_kernel(const long long *__restrict__ counts, int n,
                                                                      SortBufs b) {
    __shared__ unsigned h[kPasses * kDigits];
    const int j = blockIdx.x * kRankSortThreads + threadIdx.x;
    const bool in = j < n;
    const unsigned long long c = in ? (unsigned long long)counts[j] : 0ull;
    const unsigned code = count_code<19, 18>(c);
    for (int i = threadIdx.x; i < kPasses * kDigits; i += kRankSortThreads) h[i] = 0u;
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
    if (code >= kRankExact) {
        const unsigned long long left_out = c & ((1ull << (63 - __clzll((long long)c) - 18)) - 1ull);
        atomicOr(&b.rest[0], left_out);
        atomicOr(&b.rest[1], ~left_out);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kPasses * kDigits; i += kRankSortThreads) {
        if (h[i] != 0u) atomicAdd(&b.gtot[i], h[i]);
    }
    if (threadIdx.x < kDigits) b.hist[blockIdx.x * kDigits + threadIdx.x] = h[255 - threadIdx.x];
}

__global__ void __launch_bounds__(kRankSortThreads) rsort_hist_kernel(int n, int p, SortBufs b) {
    __shared__ unsigned h[kDigits];
    __shared__ unsigned gs[kPasses * kDigits];
    stage_totals<kRankSortThreads>(b.gtot, gs);
    if (!pass_active(gs, p, n)) return;
    const int src = source_buffer(gs, p, n);
    const int j = blockIdx.x * kRankSortThreads + threadIdx.x;
    const unsigned code = j < n ? (unsigned)(b.pairs[src][j] >> 32) : 0u;
    if (threadIdx.x < kDigits) h[threadIdx.x] = 0u;
    __syncthreads();
    if (j < n) atomicAdd(&h[255 - (int)((code >> (8 * p)) & 255u)], 1u);
    __syncthreads();
    if (threadIdx.x < kDigits) b.hist[blockIdx.x * kDigits + threadIdx.x] = h[threadIdx.x];
}

__global__ void __launch_bounds__(kRankSortThreads) rsort_scatter_kernel(int n, int p, SortBufs b) {
    __shared__ unsigned wcnt[kSortWaves * kDigits];   // [wave][digit]: elements of that digit in earlier waves
    __shared__ unsigned part[4 * kDigits];            // sums over a quarter of the earlier workgroups
    __shared__ unsigned offs[kDigits];                // first output slot of this workgroup's run of each digit
    __shared__ unsigned gs[kPasses * kDigits];
    stage_totals<kRankSortThreads>(b.gtot, gs);
    if (!pass_active(gs, p, n)) return;
    const int src = source_buffer(gs, p, n);
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int blk = blockIdx.x;

    // (requested ahead of the offsets: it depends on nothing)
    const int j = blk * kRankSortThreads + tid;
    const bool in = j < n;
    const unsigned long long pair = in ? b.pairs[src][j] : 0ull;
    for (int i = tid; i < kSortWaves * kDigits; i += kRankSortThreads) wcnt[i] = 0u;
    // this workgroup's offsets: (elements with an earlier digit anywhere) + (same digit, earlier workgroups)
    {
        // (a wave reads 64 digits of one workgroup's row at a time, a quarter of the earlier workgroups per thread)
        const int d = tid & 255, q = tid >> 8;
        unsigned before = 0;
        const int b1 = blk * (q + 1) / 4;
        const unsigned *col = b.hist + d;
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
    const int dgt = in ? 255 - (int)((pair >> (32 + 8 * p)) & 255ull) : 256;
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

__global__ void __launch_bounds__(256) rsort_out_kernel(const long long *__restrict__ counts, int n, int n_ids, SortBufs b,
                                                        int *__restrict__ out_ids) {
    __shared__ unsigned gs[kPasses * kDigits];
    stage_totals<256>(b.gtot, gs);
    const unsigned long long *__restrict__ pairs = b.pairs[source_buffer(gs, kPasses, n)];
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= n) return;
    const unsigned long long pair = pairs[j];
    const unsigned code = (unsigned)(pair >> 32);
    const int id = (int)(unsigned)pair;
    int pos = j;
    if (code >= kRankExact && (b.rest[0] & b.rest[1]) != 0ull) {      // (none when all of them leave out the same)
        // counts that share a code: their order among themselves (the run is in ascending-id order)
        const long long c = counts[id];
        for (int x = j - 1; x >= 0; --x) {
            const unsigned long long q = pairs[x];
            if ((unsigned)(q >> 32) != code) break;
            if (counts[(int)(unsigned)q] < c) --pos;           // smaller and before: goes behind
        }
        for (int x = j + 1; x < n; ++x) {
            const unsigned long long q = pairs[x];
            if ((unsigned)(q >> 32) != code) break;
            if (counts[(int)(unsigned)q] > c) ++pos;           // larger and after: goes ahead
        }
    }
    if (pos < n_ids) out_ids[pos] = id;
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
    unsigned long long sum = same ? c : 0ull;
    if (first >= exact && __popcll(group) > 1) sum = (unsigned long long)wave_sum_i64((long long)sum);
    if (lane_id() == leader) {
        atomicAdd(&h[first], (unsigned)__popcll(group));
        if (first >= exact) atomicAdd(&m[first - exact], sum);
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
    if (!DIRECT && bin < kBinExact && blockIdx.x != 0) return;
    unsigned before_n = s_n, ids = s_ids;
    unsigned long long before_m = s_m, ids_mass = s_mass, T = (unsigned)bin;
    if (bin >= kBinExact) {
        // several values share the bin: the value at which the target is reached, digit by digit
        T = bin_prefix(bin);
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
    }
    if (tid == 0) {
        // ids of count T, one after the other, until the target is reached; at least one
        unsigned long long take = 1;
        if (target > before_m && T > 0) {
            take = (target - before_m + T - 1) / T;
            if (take > (unsigned)V - before_n) take = (unsigned)V - before_n;      // (only where the mass has wrapped around)
        }
        out[0] = (long long)(before_n + take);
        out[1] = (long long)(before_m + take * T);
        out[2] = (long long)total;
    }
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
    b.rest = reinterpret_cast<unsigned long long *>(b.gtot + kPasses * kDigits);
    b.hist = reinterpret_cast<unsigned *>(p + 2 * kb + round256((kPasses * kDigits + 4) * 4));
    hipLaunchKernelGGL(rsort_zero_kernel, dim3(1), dim3(256), 0, st, b.gtot);
    hipLaunchKernelGGL(rsort_init_kernel, dim3(nblk), dim3(kRankSortThreads), 0, st, counts, n, b);
    for (int pass = 0; pass < kPasses; ++pass) {
        if (pass > 0) hipLaunchKernelGGL(rsort_hist_kernel, dim3(nblk), dim3(kRankSortThreads), 0, st, n, pass, b);
        hipLaunchKernelGGL(rsort_scatter_kernel, dim3(nblk), dim3(kRankSortThreads), 0, st, n, pass, b);
    }
    hipLaunchKernelGGL(rsort_out_kernel, dim3((n + 255) / 256), dim3(256), 0, st, counts, n, n_ids, b, out_ids);
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
    b.digit_mass = b.mass + kWideBins;
    b.bits = b.digit_mass + kDigitBins;
    b.hist = reinterpret_cast<unsigned *>(b.bits + 2);
    b.digits = b.hist + kBins;
    b.done = b.digits + kDigitBins;
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
