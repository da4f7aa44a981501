// Frequency-rank order and the alternative choices of k (Sec. 3.2: besides a fixed k, Top-P over
// the counts or a minimum-frequency threshold select the trimmed vocabulary).
//
// Rank order = all V ids sorted by (count descending, id ascending), the order in which
// Top-K(c, k) takes ids; every prefix is the selection for a smaller k.
//
// rank_*: a counting sort over bins that follow the counts, then a sort inside the bins that hold several values.
//   Counts below 2048 have a bin each (all but a few hundred of a vocabulary's counts, after 10^7 tokens).  Larger counts are
//   told apart by up to 512 splitters, counts of a fixed sample of 1024 ids (every second one where more of them are large): a
//   bin for every splitter's own value and one for what lies between two of them, so that a bin of several values holds a few
//   hundred ids wherever the counts lie, and values that many ids share have bins of their own.
//   One workgroup per 1024 consecutive ids; "earlier in the input" is (workgroup, wave, lane) order, so that equal counts
//   stay in ascending-id order:
//     rank_split    sorts the sample, where there are more than 400 workgroups
//     rank_hist     every workgroup tallies its ids per bin (and sorts the sample, the same one, for itself otherwise)
//     rank_scan     sums the tallies up over the workgroups, bin by bin
//     rank_scatter  places every id: its bin, the workgroups before, the waves before (a byte per bin and wave in LDS), the
//                   lanes before (lanes of one bin find each other with twelve ballots).  Ids of one-value bins go to the
//                   result at once
//     rank_runs     a workgroup per bin of several values orders its ids by (count, id) in LDS: up to 1024 by comparisons, up to
//                   8192 by digits of eight bits.  Longer bins are shared by all workgroups where they are few, and go through
//                   radix passes of their own workgroup where they are many
//   Four or five launches in a fixed sequence, nothing read back; launches are most of what it costs (a kernel of the chain 3 to
//   4 us, whatever it does).  Up to 4096 ids the last kernel alone, on one bin of all ids.
//   Against eight launches of LSD passes over 24-bit codes (us): V = 128256 after 10^7 tokens 44 -> 19, 10^9 44 -> 25, 10^11
//   47 -> 31 to 34; uniform below 2^20 53 -> 31, 2048 to 4096 34 -> 30, in 2^40 .. 2^40 + 2^20 49 -> 31; V = 32000 after 10^7 35 -> 16;
//   V = 8192 31 -> 15; V = 10^6 after 10^7 137 -> 44, 10^11 140 -> 84 to 111, uniform below 4000 103 -> 66, below 2^20 162 -> 75, equal
//   52 -> 46; V = 4 * 10^6 after 10^7 947 -> 94, uniform below 2^20 1119 -> 507.  Slower only where 20 000 and more large counts all avoid
//   the sample (V = 128256, 38 000 of them: 51 -> 61; V = 10^6, 100 000 of them: 150 -> 122).
//   512 samples instead of 1024 take 2 us less to sort and leave bins twice as long.
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
constexpr int kSplitters = 512;
constexpr int kWideBins = 2 * kSplitters + 4;                // 2 i: counts between splitters i - 1 and i, 2 i + 1: splitter i (2 kSplitters + 1 of them)
constexpr int kRankBins = kWideBins + kBinExact;             // from the largest counts down
constexpr int kBinWords = kRankBins / 4;                     // by fours
static_assert(kRankBins % 4 == 0 && kWideBins % 4 == 0 && kBinWords <= kRankSortThreads && kRankBins <= 1 << 12, "four bins to a thread");
constexpr int kScanBlocks = (kRankBins + kWave - 1) / kWave;
constexpr int kRunMax = 8192;         // ids that are ordered in LDS: keys of 51 bits of count and 13 of place
constexpr int kPlaceBits = 13;
static_assert(kRunMax == 1 << kPlaceBits);

// Ids that one workgroup orders in one launch: V = 4096 12 us in place of 17 after 10^7 tokens, 24 in place of 23 after 10^11; V = 8192
// 25 in place of 15, 38 in place of 23.  (Below 3800 ids the scratch would not hold the tables of the others.)
constexpr int kRankWholeMax = 4096;

// Workgroups that find the splitters each for itself; more of them, of which two share a CU at a time, read what one has found in a
// launch before (equal counts of 2048 and more, each for itself / one for all: V = 300 000 30.4 / 27.6 us, 524 288 34.2 / 31.3,
// 10^6 57.0 / 46.0, 16 * 10^6 633 / 369; after 10^7 tokens, few of them large, V = 128256 18.6 / 20.1, 300 000 24.8 / 25.7, 524 288
// 29.8 / 30.2, 4 * 10^6 103 / 94).
constexpr int kOwnSplitters = 400;

struct RankBufs {
    unsigned *rows;                // [nblk][kRankBins] ids of every workgroup per bin; after rank_scan those of the workgroups before
    unsigned *totals;              // [kRankBins]
    unsigned *start;               // [kWideBins] place of the first id of each bin of large counts
    unsigned long long *splitters; // [kSplitters] descending, zeros behind
    unsigned *ids[3];              // of the bins of several values, by place; what slices and radix passes move them to (where `rows` are)
    unsigned *n_long;              // bins of more than kRunMax ids
};

__device__ __forceinline__ int lanes_below(unsigned long long m) {
    return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}
// lanes of the wave whose value agrees with this one's in the lowest BITS bits
template <int BITS>
__device__ __forceinline__ unsigned long long match_lanes(int v) {
    unsigned long long m = ~0ull;
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
        const bool bit = (v >> b) & 1;
        const unsigned long long B = __ballot(bit);
        m &= bit ? B : ~B;
    }
    return m;
}

// The value of lane `lane ^ X`.
template <int X>
__device__ __forceinline__ unsigned lane_xor(unsigned v, int lane) {
    if constexpr (X == 1) return dpp_mov<0xB1>(v);                      // quad_perm [1,0,3,2]
    else if constexpr (X == 2) return dpp_mov<0x4E>(v);                 // quad_perm [2,3,0,1]
    else if constexpr (X == 4) return dpp_mov<0x1B>(dpp_mov<0x141>(v)); // row_half_mirror, quad_perm [3,2,1,0]
    else if constexpr (X == 8) return dpp_mov<0x128>(v);                // row_ror:8
    else if constexpr (X == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        return (lane & 16) != 0 ? r[0] : r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        return (lane & 32) != 0 ? r[0] : r[1];
    }
}
template <int SIZE, int STRIDE>
__device__ __forceinline__ void wave_sort_steps(unsigned long long &v, int lane) {
    if constexpr (STRIDE > 0) {
        const unsigned long long other =
            ((unsigned long long)lane_xor<STRIDE>((unsigned)(v >> 32), lane) << 32) | lane_xor<STRIDE>((unsigned)v, lane);
        const bool keep_larger = ((lane & SIZE) == 0 || SIZE == kWave) == ((lane & STRIDE) == 0);
        v = (other > v) == keep_larger ? other : v;
        wave_sort_steps<SIZE, STRIDE / 2>(v, lane);
    } else if constexpr (SIZE < kWave) {
        wave_sort_steps<2 * SIZE, SIZE>(v, lane);
    }
}

// Merges R <= 8 neighbouring runs of len = 2^lg values each, all over v[0 .. N), N <= 1024: every value looks up how many go
// ahead of it in the other runs, searches that do not wait for each other.
__device__ __forceinline__ void merge_runs(unsigned long long *v, int N, int lg, int R) {
    const int i = threadIdx.x, len = 1 << lg;
    unsigned long long x = 0ull;
    int place = 0;
    if (i < N) {
        x = v[i];
        const int run = (i >> lg) & (R - 1);
        const unsigned long long *first = v + (i & ~(R * len - 1));
        place = (i & ~(R * len - 1)) + (i & (len - 1));
        int ahead[8] = {};
        // (steps len / 2, .., 2, 1 and 1 once more: as many as len values go ahead)
        for (int l = lg - 1; l >= -1; --l) {
            const int step = 1 << max(l, 0);
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                if (q < R) {      // (uniform)
                    const unsigned long long t = first[(q << lg) + ahead[q] + step - 1];
                    ahead[q] += t > x || (t == x && q < run) ? step : 0;      // of equal values the earlier run's go ahead
                }
            }
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) place += q < R && q != run ? ahead[q] : 0;
    }
    __syncthreads();
    if (i < N) v[place] = x;
    __syncthreads();
}

// Sorts v[0 .. N) in LDS, largest first; N a power of two, 64 .. 1024.  All threads of the workgroup call it behind a
// barrier and find the result behind another.  64 values at a time are sorted in a wave's registers, then runs are merged,
// eight at a time.  512 values by bitonic steps in LDS took 10 us, this way 1.5.
__device__ __forceinline__ void sort_descending(unsigned long long *v, int N) {
    // (so that the second merge is known to be of two runs: 0.8 us of 5)
    __builtin_assume(N >= kWave && N <= kRankSortThreads);
    if ((int)threadIdx.x < N) {
        unsigned long long x = v[threadIdx.x];
        wave_sort_steps<2, 1>(x, lane_id());
        v[threadIdx.x] = x;
    }
    __syncthreads();
    if (N > kWave) merge_runs(v, N, 6, min(N >> 6, 8));
    if (N > 8 * kWave) merge_runs(v, N, 9, N >> 9);
}

// Sorts v[0 .. N) in LDS, N a multiple of 1024 up to kRunMax, by the bits from kPlaceBits on, largest first; equal ones keep their
// order.  differ: which of those bits are set in some and clear in others.  All threads call it behind a barrier and find the result
// behind another.  LSD passes of eight bits with the values in registers: a wave has N / 16 neighbours, and its lanes of one digit
// find each other with ballots.  A pass takes 2 to 4 us; merging the runs of 8192 values took searches of 55.
struct DigitLds {
    unsigned short at[kSortWaves * kDigits];      // [wave][digit]
    unsigned part[kSortWaves];
};
__device__ __forceinline__ void sort_by_digits(unsigned long long *v, int N, unsigned long long differ, DigitLds &s) {
    constexpr int kPer = kRunMax / kRankSortThreads;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, R = N / kRankSortThreads;
    for (int shift = kPlaceBits; shift < 64; shift += 8) {
        if (((differ >> (shift - kPlaceBits)) & 255ull) == 0ull) continue;      // (uniform)
        unsigned long long x[kPer];
        int d[kPer];
        unsigned local[kPer];
        reinterpret_cast<unsigned *>(s.at)[tid] = 0u;
        reinterpret_cast<unsigned *>(s.at)[tid + kRankSortThreads] = 0u;
#pragma unroll
        for (int r = 0; r < kPer; ++r) x[r] = r < R ? v[(w * R + r) * kWave + lane] : 0ull;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kPer; ++r) {
            if (r < R) {      // (uniform)
                d[r] = 255 - (int)((x[r] >> shift) & 255ull);
                const unsigned long long same = match_lanes<8>(d[r]);
                const unsigned short before = s.at[w * kDigits + d[r]];
                local[r] = before + (unsigned)lanes_below(same);
                if (lanes_below(same) == 0) s.at[w * kDigits + d[r]] = (unsigned short)(before + __popcll(same));
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            }
        }
        __syncthreads();
        // sums of a digit per wave -> places: thread (digit, four of the waves)
        unsigned short *const own = s.at + (tid & 3) * 4 * kDigits + (tid >> 2);
        unsigned n[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) n[q] = own[q * kDigits];
        const unsigned sum = n[0] + n[1] + n[2] + n[3];
        unsigned upto = sum;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const unsigned t = __shfl_up(upto, o);
            if (lane >= o) upto += t;
        }
        if (lane == kWave - 1) s.part[w] = upto;
        __syncthreads();
        unsigned run = upto - sum;
#pragma unroll
        for (int q = 0; q < kSortWaves; ++q) run += q < w ? s.part[q] : 0u;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            own[q * kDigits] = (unsigned short)run;
            run += n[q];
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kPer; ++r) {
            if (r < R) v[s.at[w * kDigits + d[r]] + local[r]] = x[r];
        }
        __syncthreads();
    }
}
static_assert(kSortWaves * kDigits == 4 * kRankSortThreads && kRunMax <= 65535, "four sums to a thread, places of 16 bits");
__device__ __forceinline__ int sort_size(int n) { return n <= kWave ? kWave : 1 << (32 - __clz(n - 1)); }

// The id whose count is sample i of 1024: one of every n / 1024 neighbours, not the same of all.
__device__ __forceinline__ int sample_id(int i, int n) {
    const unsigned long long at = ((unsigned long long)i << 16) | ((unsigned)(i * 40503) & 0xFFFFu);
    return (int)(at * (unsigned)n / ((unsigned long long)kRankSortThreads << 16));
}
// The bin of a count; sp: the splitters in LDS.
__device__ __forceinline__ int rank_bin(unsigned long long c, const unsigned long long *sp) {
    if (c < kBinExact) return kRankBins - 1 - (int)c;
    int i = 0;                            // splitters above c
#pragma unroll
    for (int step = kSplitters / 2; step > 0; step >>= 1) i += sp[i + step - 1] > c ? step : 0;
    i += sp[i] > c ? 1 : 0;
    return 2 * i + (i < kSplitters && sp[min(i, kSplitters - 1)] == c ? 1 : 0);
}
__device__ __forceinline__ bool one_value(int bin) { return bin >= kWideBins || (bin & 1) != 0; }

// The splitters, from the thread's sample v: sp[0 .. kSplitters) of 1024 values in LDS.  Behind a barrier; ends with one.
__device__ __forceinline__ void find_splitters(unsigned long long v, unsigned long long *sp, int &s_n) {
    const int tid = threadIdx.x;
    sp[tid] = 0ull;
    if (tid == 0) s_n = 0;
    __syncthreads();
    const unsigned long long large = __ballot(v >= kBinExact);
    if (large != 0ull) {
        int at = 0;
        if ((tid & 63) == 0) at = atomicAdd(&s_n, __popcll(large));
        at = __builtin_amdgcn_readfirstlane(at);
        if (v >= kBinExact) sp[at + lanes_below(large)] = v;
    }
    __syncthreads();
    const int n_sp = s_n;
    if (n_sp > 1) sort_descending(sp, sort_size(n_sp));
    if (n_sp > kSplitters) {      // (uniform) every second one
        const unsigned long long x = sp[(2 * tid + 1) & (kRankSortThreads - 1)];
        __syncthreads();
        if (tid < kSplitters) sp[tid] = x;
        __syncthreads();
    }
}
__global__ void __launch_bounds__(kRankSortThreads) rank_split_kernel(const long long *__restrict__ counts, int n, RankBufs b) {
    __shared__ unsigned long long sp[kRankSortThreads];
    __shared__ int s_n;
    find_splitters((unsigned long long)counts[sample_id(threadIdx.x, n)], sp, s_n);
    if (threadIdx.x < kSplitters) b.splitters[threadIdx.x] = sp[threadIdx.x];
}

// OWN: every workgroup finds the splitters for itself; else rank_split has.
template <bool OWN>
__global__ void __launch_bounds__(kRankSortThreads) rank_hist_kernel(const long long *__restrict__ counts, int n, RankBufs b) {
    __shared__ __align__(16) unsigned h[kRankBins];      // (read by fours)
    __shared__ unsigned long long sp[OWN ? kRankSortThreads : kSplitters];
    const int tid = threadIdx.x;
    const int j = blockIdx.x * kRankSortThreads + tid;
    const bool in = j < n;
    const unsigned long long c = in ? (unsigned long long)counts[j] : 0ull;
    unsigned long long v = 0ull;
    if constexpr (OWN)
        v = (unsigned long long)counts[sample_id(tid, n)];
    else if (tid < kSplitters)
        v = b.splitters[tid];
    for (int i = tid; i < kRankBins; i += kRankSortThreads) h[i] = 0u;
    if constexpr (OWN) {
        __shared__ int s_n;
        find_splitters(v, sp, s_n);
        if (blockIdx.x == 0 && tid < kSplitters) b.splitters[tid] = sp[tid];
    } else {
        if (tid < kSplitters) sp[tid] = v;
        __syncthreads();
    }
    wave_tally(h, rank_bin(c, sp), in);
    __syncthreads();
    uint4 *row = reinterpret_cast<uint4 *>(b.rows + (size_t)blockIdx.x * kRankBins);
    if (tid < kBinWords) row[tid] = *reinterpret_cast<const uint4 *>(h + 4 * tid);
}

// A workgroup takes 64 bins, a wave ROWS workgroups' rows of them at a time: 8, one round of which covers 131072 ids, or 32 for
// more (the rounds wait for memory one after the other: V = 10^6 39.8 -> 34.6 us).
template <int ROWS>
__global__ void __launch_bounds__(kRankSortThreads) rank_scan_kernel(int nblk, RankBufs b) {
    __shared__ unsigned part[kSortWaves][kWave];
    const int lane = (int)threadIdx.x & 63, w = (int)threadIdx.x >> 6;
    const int at = min((int)blockIdx.x * kWave + lane, kRankBins - 1);      // (past the end: the last one again)
    unsigned carry = 0u;
    for (int r0 = 0; r0 < nblk; r0 += kSortWaves * ROWS) {
        unsigned x[ROWS], own = 0u;
#pragma unroll
        for (int u = 0; u < ROWS; ++u) x[u] = b.rows[(size_t)min(r0 + w * ROWS + u, nblk - 1) * kRankBins + at];
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
            x[u] = r0 + w * ROWS + u < nblk ? x[u] : 0u;
            own += x[u];
        }
        part[w][lane] = own;
        __syncthreads();
        unsigned run = carry;
#pragma unroll
        for (int q = 0; q < kSortWaves; ++q) {
            const unsigned p = part[q][lane];
            run += q < w ? p : 0u;
            carry += p;
        }
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
            const int r = r0 + w * ROWS + u;
            if (r < nblk) b.rows[(size_t)r * kRankBins + at] = run;
            run += x[u];
        }
        __syncthreads();
    }
    if (w == 0) b.totals[at] = carry;
}

__global__ void __launch_bounds__(kRankSortThreads) rank_scatter_kernel(const long long *__restrict__ counts, int n, int n_ids,
                                                                        RankBufs b, int *__restrict__ out_ids) {
    __shared__ __align__(16) unsigned char wcnt[kRankBins * kSortWaves];      // [bin][wave] ids
    __shared__ __align__(16) unsigned base[kRankBins];      // place of this workgroup's first id of the bin
    __shared__ unsigned long long sp[kSplitters];
    __shared__ unsigned part[kSortWaves], s_long;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int j = blockIdx.x * kRankSortThreads + tid;
    const bool in = j < n;
    // everything is requested at once: the count, the splitters, and of four bins the totals and what lies before
    const unsigned long long c = in ? (unsigned long long)counts[j] : 0ull;
    const unsigned long long splitter = tid < kSplitters ? b.splitters[tid] : 0ull;
    uint4 tot = make_uint4(0u, 0u, 0u, 0u), bef = tot;
    if (tid < kBinWords) {
        tot = reinterpret_cast<const uint4 *>(b.totals)[tid];
        bef = reinterpret_cast<const uint4 *>(b.rows + (size_t)blockIdx.x * kRankBins)[tid];
    }
    for (int i = tid; i < kRankBins * kSortWaves / 16; i += kRankSortThreads) reinterpret_cast<uint4 *>(wcnt)[i] = make_uint4(0u, 0u, 0u, 0u);
    if (tid < kSplitters) sp[tid] = splitter;
    const unsigned sum = tot.x + tot.y + tot.z + tot.w;
    unsigned upto = sum;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const unsigned t = __shfl_up(upto, o);
        if (lane >= o) upto += t;
    }
    if (lane == kWave - 1) part[w] = upto;
    if (tid == 0) s_long = 0u;
    __syncthreads();
    unsigned above = upto - sum;
#pragma unroll
    for (int q = 0; q < kSortWaves; ++q) above += q < w ? part[q] : 0u;
    if (tid < kBinWords) {
        const uint4 first = make_uint4(above, above + tot.x, above + tot.x + tot.y, above + tot.x + tot.y + tot.z);
        *reinterpret_cast<uint4 *>(base + 4 * tid) = make_uint4(first.x + bef.x, first.y + bef.y, first.z + bef.z, first.w + bef.w);
        if (blockIdx.x == 0 && tid < kWideBins / 4) {
            reinterpret_cast<uint4 *>(b.start)[tid] = first;
            const unsigned n_long = (tot.x > (unsigned)kRunMax ? 1u : 0u) + (tot.z > (unsigned)kRunMax ? 1u : 0u);
            if (n_long != 0u) atomicAdd(&s_long, n_long);
        }
    }
    const int bin = rank_bin(c, sp);
    const unsigned long long same = match_lanes<12>(bin) & __ballot(in);
    const int below = lanes_below(same);
    if (in && below == 0) wcnt[bin * kSortWaves + w] = (unsigned char)__popcll(same);
    __syncthreads();
    if (blockIdx.x == 0 && tid == 0) *b.n_long = s_long;
    // ids of the bin in the waves before: bytes 0 .. w - 1 of sixteen
    const uint4 x = *reinterpret_cast<const uint4 *>(wcnt + bin * kSortWaves);
    auto bytes_before = [&](unsigned v, int first) {
        const int take = min(max(w - first, 0), 4);
        return take == 4 ? v : v & ((1u << (8 * take)) - 1u);
    };
    unsigned place = base[bin] + (unsigned)below;
    place = __builtin_amdgcn_sad_u8(bytes_before(x.x, 0), 0u, place);
    place = __builtin_amdgcn_sad_u8(bytes_before(x.y, 4), 0u, place);
    place = __builtin_amdgcn_sad_u8(bytes_before(x.z, 8), 0u, place);
    place = __builtin_amdgcn_sad_u8(bytes_before(x.w, 12), 0u, place);
    if (in) {
        if (!one_value(bin))
            b.ids[0][place] = (unsigned)j;
        else if (place < (unsigned)n_ids)
            out_ids[place] = j;
    }
}

// ---- the ids of a bin of several values
constexpr int kRunPer = 4;                           // elements per thread and step of the radix passes
constexpr int kRunStep = kRunPer * kRankSortThreads, kRunGroups = kRunStep / kWave;
struct RadixLds {
    unsigned long long ones, zeros;
    unsigned base[kDigits];                          // next slot of each digit, descending
    unsigned part[kRunPer * kDigits];
    unsigned short before[kRunGroups * kDigits];     // elements of a digit in the step's groups of 64 before
};

// Places [lo, lo + length) of ids by their counts: LSD passes of this workgroup over the digits in which the
// counts differ, between that buffer and another.  Nobody else touches those places.
__device__ __forceinline__ void sort_by_radix(const long long *__restrict__ counts, unsigned *ids, unsigned *other, unsigned lo,
                                              unsigned length, int n_ids, int *__restrict__ out_ids, RadixLds &s) {
    unsigned *from = ids + lo, *to = other + lo;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    if (tid == 0) s.ones = s.zeros = 0ull;
    __syncthreads();
    unsigned long long ones = 0, zeros = 0;
    for (unsigned x = tid; x < length; x += kRankSortThreads) {
        const unsigned long long c = (unsigned long long)counts[from[x]];
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
        // element x0 + (u 16 + w) 64 + lane of the run, and 255 - its digit (256: past the end)
        unsigned id[kRunPer];
        int dgt[kRunPer];
        auto load_step = [&](unsigned x0) {
#pragma unroll
            for (int u = 0; u < kRunPer; ++u) {
                const unsigned x = x0 + u * kRankSortThreads + tid;
                id[u] = x < length ? from[x] : 0u;
            }
#pragma unroll
            for (int u = 0; u < kRunPer; ++u) {
                const unsigned x = x0 + u * kRankSortThreads + tid;
                dgt[u] = x < length ? 255 - (int)(((unsigned long long)counts[id[u]] >> shift) & 255ull) : 256;
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
            for (int u = 0; u < kRunPer; ++u) same[u] = match_lanes<9>(dgt[u]);
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
                    to[pos] = id[u];
                }
            }
            __syncthreads();
            if (tid < kDigits) {
#pragma unroll
                for (int q = 0; q < kRunPer; ++q) s.base[tid] += s.part[q * kDigits + tid];
            }
        }
        __syncthreads();                // what was written is read by other waves
        unsigned *const written = to;
        to = from;
        from = written;
    }
    static_assert(kRunPer * kDigits == kRankSortThreads, "a thread per digit and quarter");
    for (unsigned x = tid; x < length && lo + x < (unsigned)n_ids; x += kRankSortThreads)
        out_ids[lo + x] = (int)from[x];
    __syncthreads();
}

struct RunLds {
    union {
        struct {
            unsigned long long key[kRunMax];
            DigitLds digits;
        };
        RadixLds radix;
    };
    unsigned long long ones, zeros;
    int far, mixed;
};

// Order-preserving code of 51 bits: counts below 2^45, of larger ones the 46 highest bits with their exponent.
__device__ __forceinline__ unsigned long long far_code(unsigned long long c) {
    if (c < (1ull << 45)) return c;
    const int e = 63 - __clzll((long long)c);
    return ((unsigned long long)(e - 44) << 45) + ((c >> (e - 45)) & ((1ull << 45) - 1ull));
}

// Orders places [lo, lo + length) by (count, place), none of the counts below `lower`.  WHOLE: all ids, the places are the ids.
template <bool WHOLE>
__device__ __forceinline__ void sort_run(const long long *__restrict__ counts, unsigned *ids, unsigned *other, unsigned lo, unsigned length,
                                         unsigned long long lower, int n_ids, int *__restrict__ out_ids, RunLds &s) {
    const int tid = threadIdx.x;
    auto id_at = [&](unsigned x) { return WHOLE ? x : ids[lo + x]; };
    auto by_radix = [&]() {
        __syncthreads();
        if constexpr (WHOLE) {
            for (unsigned x = tid; x < length; x += kRankSortThreads) ids[x] = x;
            __syncthreads();
        }
        sort_by_radix(counts, ids, other, lo, length, n_ids, out_ids, s.radix);
    };
    if (length > (unsigned)kRunMax) {
        by_radix();
        return;
    }
    const bool few = length <= kRankSortThreads;
    const int N = few ? sort_size((int)length) : (int)((length + kRankSortThreads - 1) / kRankSortThreads * kRankSortThreads);
    if (tid == 0) {
        s.far = s.mixed = 0;
        s.ones = s.zeros = 0ull;
    }
    __syncthreads();
    unsigned long long ones, zeros;
    auto make_keys = [&](auto code) {
        ones = zeros = 0ull;
        for (int x = tid; x < N; x += kRankSortThreads) {
            unsigned long long key = 0ull;
            if (x < (int)length) {
                const unsigned long long above = code((unsigned long long)counts[id_at((unsigned)x)] - lower);
                ones |= above;
                zeros |= ~above;
                key = (above << kPlaceBits) | (unsigned)(kRunMax - 1 - x);
            }
            s.key[x] = key;
        }
    };
    auto find_bits = [&]() {
        ones = wave_or_u64(ones);
        zeros = wave_or_u64(zeros);
        if ((tid & 63) == 0) {
            atomicOr(&s.ones, ones);
            atomicOr(&s.zeros, zeros);
        }
    };
    make_keys([](unsigned long long above) { return above; });
    if (__ballot((ones >> (64 - kPlaceBits)) != 0ull) != 0ull && (tid & 63) == 0) s.far = 1;
    if (!few) find_bits();
    __syncthreads();
    const bool far = s.far != 0;          // (uniform)
    if (far) {
        // counts 2^51 and more apart: by a code, which settles all of them but neighbours that share their 46 highest bits, if any
        // (by radix passes the bins of V = 128256 counts of all magnitudes took 77 us, not 32)
        if (tid == 0) s.ones = s.zeros = 0ull;
        __syncthreads();
        make_keys(far_code);
        if (!few) find_bits();
        __syncthreads();
    }
    if (!few)
        sort_by_digits(s.key, N, s.ones & s.zeros, s.digits);
    else if (length > 1u)
        sort_descending(s.key, N);
    auto place_at = [&](unsigned x) { return (unsigned)(kRunMax - 1) - ((unsigned)s.key[x] & (unsigned)(kRunMax - 1)); };
    if (far) {
        bool mixed = false;
        for (unsigned x = tid; x + 1 < length; x += kRankSortThreads)
            mixed |= (unsigned long long)counts[id_at(place_at(x))] < (unsigned long long)counts[id_at(place_at(x + 1))];
        if (mixed) s.mixed = 1;
        __syncthreads();
        if (s.mixed != 0) {               // (uniform)
            by_radix();
            return;
        }
    }
    for (unsigned x = tid; x < length; x += kRankSortThreads) {
        if (lo + x < (unsigned)n_ids) out_ids[lo + x] = (int)id_at(place_at(x));
    }
}

// Slice t of S of a bin: what lies between two of the values that divide a sample of the bin's own ids into S parts, or is the lower
// one.  Found, moved to the place that it has in the result, in order, and sorted there.
__device__ __forceinline__ void sort_slice(const long long *__restrict__ counts, const RankBufs &b, unsigned lo, unsigned length, unsigned t, unsigned S,
                                           unsigned long long lower, int n_ids, int *__restrict__ out_ids, RunLds &s, unsigned (&part)[2][kSortWaves]) {
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    __syncthreads();                      // (what was sorted before is written out)
    s.key[tid] = (unsigned long long)counts[b.ids[0][lo + (unsigned)((unsigned long long)length * (unsigned)tid / kRankSortThreads)]];
    __syncthreads();
    sort_descending(s.key, kRankSortThreads);
    const bool first = t == 0u;
    const unsigned long long high = first ? 0ull : s.key[t * kRankSortThreads / S];
    const unsigned long long low = t == S - 1u ? lower : s.key[(t + 1u) * kRankSortThreads / S];
    // a wave has a sixteenth of the bin, in order
    const unsigned begin = (unsigned)((unsigned long long)length * (unsigned)w / kSortWaves);
    const unsigned end = (unsigned)((unsigned long long)length * (unsigned)(w + 1) / kSortWaves);
    auto for_each = [&](auto &&f) {
        constexpr int kLoads = 16;
        for (unsigned x0 = begin; x0 < end; x0 += kLoads * kWave) {
            unsigned id[kLoads];
            unsigned long long c[kLoads];
#pragma unroll
            for (int u = 0; u < kLoads; ++u) id[u] = b.ids[0][lo + min(x0 + u * kWave + lane, end - 1u)];
#pragma unroll
            for (int u = 0; u < kLoads; ++u) c[u] = (unsigned long long)counts[id[u]];
#pragma unroll
            for (int u = 0; u < kLoads; ++u) {
                const bool there = x0 + u * kWave + lane < end, above = !first && c[u] >= high;
                f(id[u], there && !above && c[u] >= low, there && above);
            }
        }
    };
    // a wave keeps what it finds, as long as there is room
    constexpr unsigned kKept = 2 * kRunMax / kSortWaves;
    unsigned *const kept = reinterpret_cast<unsigned *>(s.key) + (unsigned)w * kKept;
    __syncthreads();                      // (everyone has the two values)
    unsigned n_in = 0u, n_above = 0u;
    for_each([&](unsigned id, bool in, bool above) {
        const unsigned long long mask = __ballot(in);
        const unsigned at = n_in + (unsigned)lanes_below(mask);
        if (in && at < kKept) kept[at] = id;
        n_in += (unsigned)__popcll(mask);
        n_above += (unsigned)__popcll(__ballot(above));
    });
    if (lane == 0) {
        part[0][w] = n_in;
        part[1][w] = n_above;
    }
    __syncthreads();
    unsigned total = 0u, before = 0u, at = lo;
#pragma unroll
    for (int q = 0; q < kSortWaves; ++q) {
        total += part[0][q];
        before += q < w ? part[0][q] : 0u;
        at += part[1][q];
    }
    if (total == 0u || at >= (unsigned)n_ids) return;      // (uniform)
    unsigned to = at + before;
    if (n_in <= kKept) {                  // (uniform over the wave)
        for (unsigned x = (unsigned)lane; x < n_in; x += kWave) b.ids[1][to + x] = kept[x];
    } else {
        for_each([&](unsigned id, bool in, bool) {
            const unsigned long long mask = __ballot(in);
            if (in) b.ids[1][to + (unsigned)lanes_below(mask)] = id;
            to += (unsigned)__popcll(mask);
        });
    }
    __syncthreads();
    sort_run<false>(counts, b.ids[1], b.ids[2], at, total, low, n_ids, out_ids, s);
}

// WHOLE: one bin of all n ids.
// Bins too long for LDS go to radix passes of their workgroups where there are many, as between 512 splitters of millions of ids, all
// large.  Where they are few (neighbours far apart in the sample, or large counts that all avoid it) all workgroups share them: a slice
// costs a reading of the whole bin, but by 500 workgroups and not by one (V = 128256, 38 000 large counts, none of them in the sample:
// 61 us, by one workgroup 312; V = 10^6, 100 000 122 / 1200; V = 10^6, all large, of all magnitudes 119 / 211).
constexpr unsigned kSharedBins = 64, kSliceIds = 2048, kMaxSlices = 512;
template <bool WHOLE>
__global__ void __launch_bounds__(kRankSortThreads) rank_runs_kernel(const long long *__restrict__ counts, int n, int n_ids, RankBufs b,
                                                                     int *__restrict__ out_ids) {
    __shared__ RunLds s;
    if constexpr (WHOLE) {
        sort_run<true>(counts, b.ids[0], b.ids[1], 0u, (unsigned)n, 0ull, n_ids, out_ids, s);
    } else {
        auto lower_of = [&](unsigned bin) { return bin < (unsigned)kSplitters ? b.splitters[bin] : 0ull; };      // below all counts of the bin
        const unsigned lo = b.start[2 * blockIdx.x], length = b.start[2 * blockIdx.x + 1] - lo, n_long = *b.n_long;
        const unsigned long long lower = lower_of(blockIdx.x);
        const bool shared = n_long != 0u && n_long <= kSharedBins;      // (uniform)
        // (unless nothing is there, or nobody asks for it)
        if (length != 0u && lo < (unsigned)n_ids && !(shared && length > (unsigned)kRunMax))
            sort_run<false>(counts, b.ids[0], b.ids[1], lo, length, lower, n_ids, out_ids, s);
        if (!shared) return;
        __shared__ unsigned part[2][kSortWaves];
        unsigned slices = 0u;             // of the bins before: a workgroup takes every gridDim-th
        for (int i0 = 0; i0 <= kSplitters; i0 += kWave) {
            const int i = min(i0 + (int)(threadIdx.x & 63), kSplitters);
            const unsigned bin_lo = b.start[2 * i], bin_length = b.start[2 * i + 1] - bin_lo;
            const bool is_long = i == i0 + (int)(threadIdx.x & 63) && bin_length > (unsigned)kRunMax && bin_lo < (unsigned)n_ids;
            for (unsigned long long m = __ballot(is_long); m != 0ull; m &= m - 1ull) {
                const int l = __ffsll((long long)m) - 1;
                const unsigned q_lo = (unsigned)__builtin_amdgcn_readlane((int)bin_lo, l), q_length = (unsigned)__builtin_amdgcn_readlane((int)bin_length, l);
                const unsigned S = min((q_length + kSliceIds - 1u) / kSliceIds, kMaxSlices);
                for (unsigned t = (blockIdx.x + gridDim.x - slices % gridDim.x) % gridDim.x; t < S; t += gridDim.x)
                    sort_slice(counts, b, q_lo, q_length, t, S, lower_of((unsigned)(i0 + l)), n_ids, out_ids, s, part);
                slices += S;
            }
        }
    }
}

}  // namespace

// ---------------------------------------------------------------- choice of k
// out[0] = k, out[1] = mass of the k largest counts, out[2] = total mass.
//   mode 0: smallest k >= 1 with S_k >= ceil(P * total);  mode 1: k = #{c >= f_min}.
namespace {

constexpr int kMassBins = kBins - kBinExact;      // bins of more than one value: their mass is summed
// of the bin that is divided: digits of its ids, their mass, and the bits below its prefix that are set in any / clear in any
struct ChooseBufs {
    unsigned long long *mass;          // [kMassBins]
    unsigned long long *digit_mass;    // [kDigitBins]
    unsigned long long *bits;          // [2]
    unsigned *hist;                    // [kBins]
    unsigned *digits;                  // [kDigitBins]
    unsigned *done;                    // [2] workgroups that have added theirs
};
constexpr int kChooseZeroWords = kMassBins + kDigitBins + 2 + (kBins + kDigitBins + 2) / 2;      // 64-bit words, mass .. done
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
    for (int i = threadIdx.x; i < kMassBins; i += kRankSortThreads) m[i] = 0ull;
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
    __shared__ unsigned long long m[kMassBins];
    bin_counts(counts, V, h, m);
    for (int i = threadIdx.x; i < kBins; i += kRankSortThreads) {
        if (h[i] != 0u) atomicAdd(&b.hist[i], h[i]);
    }
    for (int i = threadIdx.x; i < kMassBins; i += kRankSortThreads) {
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
    __shared__ unsigned long long m[kDigitBins > kMassBins ? kDigitBins : kMassBins];
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
    const int nblk = (n + kRankSortThreads - 1) / kRankSortThreads;
    RankBufs b{};
    b.ids[0] = reinterpret_cast<unsigned *>(p);
    p += round256((size_t)n * 4);
    b.ids[1] = reinterpret_cast<unsigned *>(p);
    b.ids[2] = reinterpret_cast<unsigned *>(p + round256((size_t)n * 4));
    if (n <= kRankWholeMax) {
        hipLaunchKernelGGL(rank_runs_kernel<true>, dim3(1), dim3(kRankSortThreads), 0, st, counts, n, n_ids, b, out_ids);
        return;
    }
    // (12 KiB per 1024 ids, more than the two times 4 KiB that slices and radix passes write there)
    b.rows = reinterpret_cast<unsigned *>(p);
    p += round256((size_t)nblk * kRankBins * 4);
    b.totals = reinterpret_cast<unsigned *>(p);
    p += round256(kRankBins * 4);
    b.start = reinterpret_cast<unsigned *>(p);
    p += round256(kWideBins * 4);
    b.splitters = reinterpret_cast<unsigned long long *>(p);
    b.n_long = reinterpret_cast<unsigned *>(p + kSplitters * 8);
    if (nblk <= kOwnSplitters) {
        hipLaunchKernelGGL(rank_hist_kernel<true>, dim3(nblk), dim3(kRankSortThreads), 0, st, counts, n, b);
    } else {
        hipLaunchKernelGGL(rank_split_kernel, dim3(1), dim3(kRankSortThreads), 0, st, counts, n, b);
        hipLaunchKernelGGL(rank_hist_kernel<false>, dim3(nblk), dim3(kRankSortThreads), 0, st, counts, n, b);
    }
    auto scan = nblk <= 8 * kSortWaves ? rank_scan_kernel<8> : rank_scan_kernel<32>;
    hipLaunchKernelGGL(scan, dim3(kScanBlocks), dim3(kRankSortThreads), 0, st, nblk, b);
    hipLaunchKernelGGL(rank_scatter_kernel, dim3(nblk), dim3(kRankSortThreads), 0, st, counts, n, n_ids, b, out_ids);
    hipLaunchKernelGGL(rank_runs_kernel<false>, dim3(kSplitters + 1), dim3(kRankSortThreads), 0, st, counts, n, n_ids, b, out_ids);
}
static_assert(kRankBins * 4 >= 8 * kRankSortThreads, "two buffers of ids lie where the rows are");

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
    b.hist = reinterpret_cast<unsigned *>(b.mass + kMassBins);      // (every array on whole cache lines)
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
