// Order-preserving codes of token counts: bins for histograms of counts and digits for sorts of them.
//
// Counts are heavy-tailed: all but a few hundred of a vocabulary's counts are small (10^7 calibration tokens: 128000 of
// 128256 below 2048), and those few spread over many powers of two.  A code keeps small counts as they are and of larger
// ones the highest bits, like a floating-point number, so that one histogram or a few digits cover every int64.
#pragma once
#include <hip/hip_runtime.h>

namespace vt {

// exact below 2^EXACT_LOG; above, MANT_LOG bits after the leading one
template <int EXACT_LOG, int MANT_LOG>
__device__ __forceinline__ unsigned count_code(unsigned long long c) {
    if (c < (1ull << EXACT_LOG)) return (unsigned)c;
    const int e = 63 - __clzll((long long)c);
    return (1u << EXACT_LOG) + ((unsigned)(e - EXACT_LOG) << MANT_LOG) +
           (unsigned)((c >> (e - MANT_LOG)) & ((1ull << MANT_LOG) - 1));
}

// ---- histogram bins: exact below 2048 (a bin is one value), then 32 bins per power of two
constexpr int kBinExact = 2048;
constexpr int kBins = kBinExact + (64 - 11) * 32;      // 3744
__device__ __forceinline__ int count_bin(unsigned long long c) { return (int)count_code<11, 5>(c); }
// bin >= kBinExact: its counts c have c >> shift == prefix
__device__ __forceinline__ int bin_shift(int bin) { return 11 + ((bin - kBinExact) >> 5) - 5; }
__device__ __forceinline__ unsigned long long bin_prefix(int bin) { return 32ull + (unsigned)((bin - kBinExact) & 31); }

}  // namespace vt
