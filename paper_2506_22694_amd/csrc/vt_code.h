// Order-preserving codes of token counts: bins for histograms of counts.
//
// Counts are heavy-tailed: all but a few hundred of a vocabulary's counts are small (10^7 calibration tokens: 128000 of
// 128256 below 2048), and those few spread over many powers of two.  A code keeps small counts as they are and of larger
// ones the highest bits, like a floating-point number, so that one histogram covers every int64.
#pragma once
#include "vt_device.h"

namespace vt {

// ---- histogram bins: exact below 2048 (a bin is one value), then 32 bins per power of two: five bits after the leading one
constexpr int kBinExact = 2048;
constexpr int kBins = kBinExact + (64 - 11) * 32;      // 3744
__device__ __forceinline__ int count_bin(unsigned long long c) {
    if (c < (unsigned long long)kBinExact) return (int)c;
    const int e = 63 - __clzll((long long)c);
    return kBinExact + ((e - 11) << 5) + (int)((c >> (e - 5)) & 31ull);
}
// bin >= kBinExact: its counts c have c >> shift == prefix
__device__ __forceinline__ int bin_shift(int bin) { return 11 + ((bin - kBinExact) >> 5) - 5; }
__device__ __forceinline__ unsigned long long bin_prefix(int bin) { return 32ull + (unsigned)((bin - kBinExact) & 31); }

// ---- what a bin of several values leaves open, below its prefix
// The next level of the histogram: kDigitBits of the bits below the prefix.  6 + 11 highest bits of a count are then known,
// all of them below 2^17.
constexpr int kDigitBits = 11;
constexpr int kDigitBins = 1 << kDigitBits;

__device__ __forceinline__ unsigned long long low_bits(int n) { return (1ull << n) - 1ull; }      // n < 64

// OR over the wave
__device__ __forceinline__ unsigned long long wave_or_u64(unsigned long long v) {
    struct Or {
        __device__ __forceinline__ unsigned operator()(unsigned a, unsigned b) const { return a | b; }
    };
    const unsigned lo = wave_allreduce_u32((unsigned)v, Or{}), hi = wave_allreduce_u32((unsigned)(v >> 32), Or{});
    return ((unsigned long long)hi << 32) | lo;
}

// h[d] += 1 for every lane with `in` (all lanes call): the lanes that share the first one's digit are added at once --
// counts are often all the same, and 64 LDS atomics on one address queue.
__device__ __forceinline__ void wave_tally(unsigned *h, int d, bool in) {
    const unsigned long long live = __ballot(in);
    if (live == 0ull) return;
    const int leader = __ffsll((long long)live) - 1;
    const int first = __builtin_amdgcn_readlane(d, leader);
    const unsigned long long same = __ballot(in && d == first);
    if (in && d != first) atomicAdd(&h[d], 1u);
    if ((int)(threadIdx.x & 63) == leader) atomicAdd(&h[first], (unsigned)__popcll(same));
}

// The bits below the prefix that some ids of a bin have set and some have not (`ones`: set in any, `zeros`: clear in any).
// The others are common to all of them: what is left to find of a value of `left` open bits then starts at the highest bit
// that varies.  T: the bits above; takes the common bits over and returns how many stay open.
__device__ __forceinline__ int skip_common_bits(unsigned long long &T, int left, unsigned long long ones, unsigned long long zeros) {
    const unsigned long long vary = ones & zeros & low_bits(left);
    const int open = vary == 0ull ? 0 : 64 - __clzll((long long)vary);
    T = (T << (left - open)) | ((ones & low_bits(left)) >> open);
    return open;
}

}  // namespace vt
