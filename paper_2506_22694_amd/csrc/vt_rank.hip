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
// choose_*: no sort: a histogram over bins of counts (exact below 2048) with the mass of every bin; one workgroup walks
//   it from the largest counts down and divides inside the bin in which the mass reaches ceil(P * total).
//   (With the read-back of k 107 us behind a full sort, now 31.)
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
struct ChooseBufs {
    unsigned long long *mass;      // [kWideBins]
    unsigned *hist;                // [kBins]
};

__global__ void __launch_bounds__(kRankSortThreads) choose_zero_kernel(ChooseBufs b) {
    for (int i = threadIdx.x; i < kBins; i += kRankSortThreads) b.hist[i] = 0u;
    for (int i = threadIdx.x; i < kWideBins; i += kRankSortThreads) b.mass[i] = 0ull;
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

// The counts of this workgroup (all of them when gridDim.x = 1) into bins of LDS, ids and -- above 2048 -- mass.
__device__ __forceinline__ void bin_counts(const long long *__restrict__ counts, int V, unsigned *h, unsigned long long *m) {
    for (int i = threadIdx.x; i < kBins; i += kRankSortThreads) h[i] = 0u;
    for (int i = threadIdx.x; i < kWideBins; i += kRankSortThreads) m[i] = 0ull;
    __syncthreads();
    for (int j = blockIdx.x * kRankSortThreads + threadIdx.x; j < V; j += gridDim.x * kRankSortThreads) {
        const unsigned long long c = (unsigned long long)counts[j];
        const int bin = count_bin(c);
        atomicAdd(&h[bin], 1u);
        if (bin >= kBinExact) atomicAdd(&m[bin - kBinExact], c);
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

// One workgroup.  DIRECT: it bins all counts itself (small V).
template <bool DIRECT>
__global__ void __launch_bounds__(kRankSortThreads) choose_mass_kernel(const long long *__restrict__ counts, int V, double P,
                                                                       ChooseBufs b, long long *__restrict__ out) {
    __shared__ unsigned h[DIRECT ? kBins : 256];
    __shared__ unsigned long long m[DIRECT ? kWideBins : 256];
    __shared__ unsigned pn[kSortWaves];
    __shared__ unsigned long long pm[kSortWaves];
    __shared__ int s_bin;
    __shared__ unsigned s_n;
    __shared__ unsigned long long s_m, s_total;
    constexpr int kPer = (kBins + kRankSortThreads - 1) / kRankSortThreads;
    const int tid = threadIdx.x;
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
    if (tid == 0) s_bin = -1;
    __syncthreads();
    const unsigned long long total = s_total;
    // one fp64 product, then its ceiling; never above the total (beyond 2^53 tokens the product of P = 1
    // can round up past it, and no prefix would reach it)
    const unsigned long long want = (unsigned long long)ceil(P * (double)(long long)total);
    const unsigned long long target = want > total ? total : want;
    // the first bin, from above, that holds ids and with which the mass reaches the target (k >= 1: a target of 0 too)
    unsigned above_n = upto_n - n;
    unsigned long long above_m = upto_m - mass;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        if (vn[i] != 0u && above_m + vm[i] >= target && (above_m < target || above_n == 0u)) {
            s_bin = kBins - 1 - (kPer * tid + i);
            s_n = above_n;
            s_m = above_m;
        }
        above_n += vn[i];
        above_m += vm[i];
    }
    __syncthreads();
    const int bin = s_bin;
    if (bin < 0) {      // no bin reaches it: counts below zero, or a mass of 2^63 and more
        if (tid < 3) out[tid] = tid == 2 ? (long long)total : 0;
        return;
    }
    unsigned before_n = s_n;
    unsigned long long before_m = s_m, T = (unsigned)bin;
    if (bin >= kBinExact) {
        // several values share the bin: the value at which the target is reached, up to eight bits at a time, from the
        // counts that agree with it so far
        T = bin_prefix(bin);
        for (int left = bin_shift(bin); left > 0;) {
            const int bits = left < 8 ? left : 8;
            left -= bits;
            __syncthreads();
            if (tid < 256) {
                h[tid] = 0u;
                m[tid] = 0ull;
            }
            __syncthreads();
            for (int x = tid; x < V; x += kRankSortThreads) {
                const unsigned long long c = (unsigned long long)counts[x];
                if ((c >> (left + bits)) == T) {
                    const unsigned d = (unsigned)(c >> left) & ((1u << bits) - 1u);
                    atomicAdd(&h[d], 1u);
                    atomicAdd(&m[d], c);
                }
            }
            __syncthreads();
            const unsigned dn = tid < 256 ? h[255 - tid] : 0u;
            const unsigned long long dm = tid < 256 ? m[255 - tid] : 0ull;
            unsigned un = dn;
            unsigned long long um = dm;
            block_scan2(un, um, pn, pm);
            const unsigned an = before_n + un - dn;
            const unsigned long long am = before_m + um - dm;
            if (dn != 0u && am + dm >= target && (am < target || an == 0u)) {
                s_bin = 255 - tid;
                s_n = an;
                s_m = am;
            }
            __syncthreads();
            T = (T << bits) | (unsigned)s_bin;
            before_n = s_n;
            before_m = s_m;
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
    b.hist = reinterpret_cast<unsigned *>(b.mass + kWideBins);
    if (mode == 0 && V <= kChooseDirectMaxV) {
        hipLaunchKernelGGL(choose_mass_kernel<true>, dim3(1), dim3(kRankSortThreads), 0, st, counts, V, P, b, out);
        return;
    }
    if (mode != 0) {
        hipLaunchKernelGGL(choose_clear_kernel, dim3(1), dim3(64), 0, st, out);
        hipLaunchKernelGGL(choose_min_kernel, dim3(nblk), dim3(kRankSortThreads), 0, st, counts, V, f_min, out);
        return;
    }
    hipLaunchKernelGGL(choose_zero_kernel, dim3(1), dim3(kRankSortThreads), 0, st, b);
    hipLaunchKernelGGL(choose_hist_kernel, dim3(nblk), dim3(kRankSortThreads), 0, st, counts, V, b);
    hipLaunchKernelGGL(choose_mass_kernel<false>, dim3(1), dim3(kRankSortThreads), 0, st, counts, V, P, b, out);
}

}  // namespace vt
