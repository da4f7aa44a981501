// Column ranges of the matrix-core kernels: where a workgroup's march over the columns starts, and the sums that make a
// logit independent of it.
#pragma once
#include "vt_device.h"

namespace vt {

typedef __attribute__((ext_vector_type(4))) float f32x4;

// All workgroups march over the columns of their rows in step, and rows of W are d * 2 bytes apart: when that is a
// multiple of 4 KiB the requests in flight crowd a subset of the HBM channels (n = 64, k = 32768, d = 4096: 63 us; d = 2048:
// 36 us).  So the contraction is cut into NR ranges of columns and workgroup b starts with range (b / 8 + b / 64) % NR --
// b % 8 is the XCD -- and wraps around (NR = 4: 44.5 and 32.9 us, NR = 8: 43.0 and 24.8; without the b / 64 tiles of 96 or
// 160 rows, whole multiples of many pages apart, meet again: d = 4096, n = 32, k = 22786 35.0 against 31.6 us, k = 40000
// 56.7 / 51.7).  To keep a logit's rounding independent
// of where its workgroup started (equal rows of W give equal logits in whichever tile they lie) every range is
// accumulated from zero in ascending order and the sums are added up as a balanced tree,
// ((R0 + R1) + (R2 + R3)) + ((R4 + R5) + (R6 + R7)): float addition commutes, so the ranges can finish in any rotation.
// The partial sums a rotation needs to hold: the open half of a pair, one sum per quad, and for an odd start the
// second half of its pair, whose first half comes last.  NR = 4 and 2 are the same tree, cut off.  (NR = 2 takes any number
// of ranges that finish in the same order in every tile.)
template <int NR, int N>
struct RangeSums {
    static constexpr int kSets = NR == 8 ? 4 : NR == 4 ? 2 : NR == 2 ? 1 : 0;
    f32x4 set[kSets > 0 ? kSets : 1][kSets > 0 ? N : 1];
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int s = 0; s < kSets; ++s) {
#pragma unroll
            for (int i = 0; i < N; ++i) set[s][i] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    // The j-th range to finish (range (rot + j) % NR) is complete in acc, which starts from zero again.
    __device__ __forceinline__ void close(f32x4 (&acc)[N], int rot, int j) {
        const f32x4 zero = f32x4{0.f, 0.f, 0.f, 0.f};
        if constexpr (NR == 2) {
#pragma unroll
            for (int i = 0; i < N; ++i) set[0][i] += acc[i];
        } else if constexpr (NR == 4) {
            // set[x] = R(2x) + R(2x + 1)
            const bool to1 = (((rot + j) >> 1) & 1) != 0;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                set[0][i] += to1 ? zero : acc[i];      // (adding zero changes nothing)
                set[1][i] += to1 ? acc[i] : zero;
            }
        } else if constexpr (NR == 8) {
            // set[0], set[1]: the quads; set[2]: the open pair's first half; set[3]: an odd start's first range
            const bool odd = (rot & 1) != 0;
            if (odd && j == 0) {
#pragma unroll
                for (int i = 0; i < N; ++i) set[3][i] = acc[i];
            } else if (((rot + j) & 1) == 0 && !(odd && j == 7)) {
#pragma unroll
                for (int i = 0; i < N; ++i) set[2][i] = acc[i];
            } else {
                const bool to1 = (((rot + j) >> 2) & 1) != 0;
                const bool last = odd && j == 7;
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    const f32x4 pair = (last ? set[3][i] : set[2][i]) + acc[i];
                    set[0][i] += to1 ? zero : pair;
                    set[1][i] += to1 ? pair : zero;
                }
            }
        }
#pragma unroll
        for (int i = 0; i < N; ++i) acc[i] = zero;
    }
    // the logits, from the closed ranges (and the last one of NR = 2, closed like the others)
    __device__ __forceinline__ void total(f32x4 (&acc)[N]) const {
        if constexpr (NR == 2) {
#pragma unroll
            for (int i = 0; i < N; ++i) acc[i] = set[0][i];
        } else if constexpr (NR >= 4) {
#pragma unroll
            for (int i = 0; i < N; ++i) acc[i] = set[0][i] + set[1][i];
        }
    }
    // ... with the last range still in acc
    template <bool IN_ORDER>
    __device__ __forceinline__ void finish(f32x4 (&acc)[N], int rot, int j) {
        if constexpr (IN_ORDER) {
#pragma unroll
            for (int i = 0; i < N; ++i) acc[i] += set[0][i];
        } else {
            close(acc, rot, j);
            total(acc);
        }
    }
};

// Columns from one range's start to the next, in units of which a row of d holds `units`: NR equal ranges -- where those
// would start whole multiples of 4 KiB apart, on the same channels again, each is longer by 4 KiB / NR and the last one
// shorter.  Four ranges, d = 8192: n = 100, k = 40000 146.6 -> 122.9 us, n = 160, k = 32768 134.0 -> 124.5, n = 100,
// k = 32768 100.8 / 101.8.  Eight, d = 16384: n = 20, k = 24445 145.6 -> 128.9, n = 64 156.4 -> 144.5, k = 40000 228 -> 205,
// but k = 33000 174 / 179.  (The kernel for up to 8 hidden rows keeps equal ranges, see there.)
template <int NR>
__device__ __forceinline__ int range_step(int units, int d) {
    const int step = units / NR;
    return NR > 1 && d % (NR * 2048) == 0 ? step + units * (2048 / NR) / d : step;
}

// The range workgroup b starts with.
template <int NR>
__device__ __forceinline__ int first_range(int b) {
    return ((b >> 3) + (b >> 6)) & (NR - 1);
}

}  // namespace vt
