// Draft step for more than 8 hidden rows (tree and batch drafting): z[n, k] = h[n, d] W_trim[k, d]^T on the matrix
// cores (v_mfma_f32_16x16x32_bf16), bound by the single pass over W_trim up to about 128 hidden rows.
//
// Both operands go from memory straight into LDS (global_load_lds_dwordx4: no registers hold data in flight, so the
// depth of the prefetch is a matter of LDS alone).  A stage is 64 columns (128 bytes) of the tile's rows of W_trim and of
// all hidden rows; a ring of stages fills LDS and one barrier per stage hands a slot on.  16-byte pieces of a row are
// stored in the order c ^ ((row / 2) & 7), which the loading lanes do by picking their piece of memory: operand reads
// (ds_read_b128, 16 rows x 4 pieces) then run at the full LDS rate (535 bytes/ns per CU; 301 at a row pitch of 272 bytes,
// 151 at 128 bytes unswizzled) and every 8 lanes still load one 128-byte line.
//
// The tile's logits meet in LDS (over the ring) and the workgroup epilogue produces (max, sum-exp) and the best
// candidates per hidden row; a merge kernel finishes the step.  Or the logits go straight from the accumulators to memory for
// row_select_kernel (16 bytes per lane; by way of LDS they took a tile of 128 x 224 4.7 us, now 1.5: n = 256, k = 32768, d = 8192
// 157.7 -> 155.5 us, n = 33, k = 21900, d = 4096, m = 16 42.9 / 41.1) -- those of all columns, or of a slice of them: heads of few
// rows are cut into larger tiles and slices (plan_stored in vt_api.hip).  Beside all columns' logits goes the (max, sum-exp) of what each
// wave holds of a row, 1 to 2 us for n = 256 where the lists of m tokens take 10.
#include "vt_device.h"
#include "vt_launch.h"
#include "vt_ranges.h"
#include "vt_step.h"
#include "vt_step_tail.h"
#include <type_traits>

namespace vt {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;

constexpr int kStageCols = 64;                 // columns per stage: 128 bytes per row
constexpr int kGroupBytes = 16 * 128;          // 16 rows of a stage
constexpr int kPieceBytes = 1024;              // one load instruction: 8 rows of a stage

// 64 lanes x 16 bytes from base + voff into LDS at lds + 16 * lane.  STREAM: read once (W_trim); otherwise kept in
// the L2 for the other workgroups (h).  M0 holds the LDS address, and a load that reads it needs a wait state behind the
// scalar write (the compiler puts one there by itself, but not inside a string of ours: the build looks for it).
template <bool STREAM>
__device__ __forceinline__ void lds_load16(unsigned lds, unsigned voff, const void *base) {
    if constexpr (STREAM)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(lds), "v"(voff), "s"(base) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(voff), "s"(base) : "memory", "m0");
}
__device__ __forceinline__ void lds_load4(unsigned lds, unsigned voff, const void *base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(lds), "v"(voff), "s"(base) : "memory", "m0");
}
// All but the N youngest loads of this wave have landed, its LDS reads are done; then the workgroup's barrier.
template <int N>
__device__ __forceinline__ void wait_and_sync() {
    static_assert(N <= 63, "vmcnt holds six bits");
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// The same with `younger` <= MOST stages of LPW loads each behind the one that is needed (fewer only near the end).
template <int LPW, int MOST>
__device__ __forceinline__ void wait_stage_and_sync(int younger) {
    if constexpr (MOST == 0) {
        wait_and_sync<0>();
    } else {
        if (younger >= MOST)
            wait_and_sync<LPW * MOST>();
        else
            wait_stage_and_sync<LPW, MOST - 1>(younger);
    }
}

// What becomes of a tile's logits: lists of candidates (or logits by way of LDS, where zbuf is not aligned), logits straight from the
// accumulators, or those of a slice of the columns, blockIdx.y, with ranges of its own that its tiles rotate, or in order.  Kernels of
// their own: as a branch in one kernel they took every step 0.2 to 0.5 us (n = 16, k = 9735, d = 3072 17.5 / 17.8, n = 80, k = 35010,
// d = 1024 23.6 / 24.1).
enum TileOut { kTileLists, kTileStored, kTileSlices, kTileSlicesInOrder };
constexpr bool in_slices(TileOut out) { return out == kTileSlices || out == kTileSlicesInOrder; }

// Where a workgroup's march over ns stages starts and where its ranges end.
template <int NR, TileOut OUT>
struct March {
    int ns, rot, start, step, last, last_length;
    bool ranges;
    // Slices of the columns (of ns stages each) start in different places anyway; where those are whole multiples of 4 KiB
    // apart a slice has ranges to itself (n = 32, k = 14000, d = 8192, two slices 57.3 -> 50.6 us; elsewhere 2 to 10 % slower).
    // In order: all tiles of a slice start at its first column, and the sums of any number of ranges take one set of registers.
    // A chain of additions is no longer in slices than an eighth of the row, what the tiles in one piece have where they have ranges: a
    // slice in one chain had up to twice the error of those (n = 126, k = 5389, d = 8192, three slices: log-probs of the best tokens
    // 3.0e-7 off, 1.5e-7 in one piece and in short chains).
    __device__ __forceinline__ March(int ns_, int d) : ns(ns_) {
        if constexpr (OUT == kTileSlicesInOrder) {
            ranges = d % 2048 == 0;
            rot = 0;
            // (an even number of stages: one of the kernel may be two blocks of 64 columns)
            step = d / (8 * kStageCols) & ~1;
            start = 0;
            last = -1;
            last_length = 0;
        } else {
            ranges = OUT == kTileSlices || (NR > 1 && d % 2048 == 0 && (NR > 2 || d >= 4096));
            rot = ranges ? first_range<NR>((int)blockIdx.x) : 0;
            // stages from one start to the next
            if constexpr (OUT == kTileSlices) {
                step = ns / NR & ~1;
                if (step % 32 == 0) step += 32 / NR;
            } else {
                step = NR == 2 ? 16 : range_step<NR>(ns, d);
            }
            start = bound(rot);
            last = NR - 1 - rot;
            last_length = ns - bound(NR - 1);
        }
    }
    __device__ __forceinline__ int bound(int r) const { return r * step; }
    // stage of the row that is multiplied at step s < ns
    __device__ __forceinline__ int stage_of(int s) const {
        const int u = start + s;
        return u >= ns ? u - ns : u;
    }
    // the number of stages in range (rot + j) % NR, the j-th to be marched through
    __device__ __forceinline__ int length_of(int j) const { return j == last ? last_length : step; }
};

// The columns of a workgroup: the first stage of 64, and how many.
template <TileOut OUT>
struct Columns {
    int slice, first, stages;
    __device__ __forceinline__ explicit Columns(const MfmaArgs &a) {
        if constexpr (in_slices(OUT)) {
            slice = (int)blockIdx.y;
            first = 2 * (slice * a.slice_units + min(slice, a.slice_more));
            stages = 2 * (a.slice_units + (slice < a.slice_more ? 1 : 0));
        } else {
            slice = 0;
            first = 0;
            stages = a.d / kStageCols;
        }
    }
};

// Tile logits in LDS: hidden row i at i * pitch floats.
__device__ __forceinline__ void store_logits4(float *dst, const f32x4 &v) {
    dst[0] = v.x;
    dst[1] = v.y;
    dst[2] = v.z;
    dst[3] = v.w;
}

// Four logits of a hidden row straight from the accumulators to zbuf, if the tile has them (16-byte aligned; where k is no
// multiple of four the last group reaches into the row's padding).
__device__ __forceinline__ void store_z4(float *z, int i, int n, int pitch, int row, int rows_b, const f32x4 &v) {
    if (i < n && row < rows_b) *reinterpret_cast<f32x4 *>(z + (size_t)i * pitch + row) = v;
}

// (max, sum-exp) of a hidden row's logits in this wave, four in every accumulator v[x * STEP], 16 rows of the head each: a lane
// has its four, three more lanes (16, 32 and 48 further) the others.  (Of logits that are all -inf NaN, see row_select_parts_kernel.)
template <int N, int STEP>
__device__ __forceinline__ void publish_part(const f32x4 *v, unsigned long long *pms, bool there, int lgrp) {
    auto across = [](float x, auto op) {
        auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
        unsigned y = op(r[0], r[1]);
        r = __builtin_amdgcn_permlane32_swap(y, y, false, false);
        return __uint_as_float(op(r[0], r[1]));
    };
    float top = fmaxf(fmaxf(v[0].x, v[0].y), fmaxf(v[0].z, v[0].w));
#pragma unroll
    for (int x = 1; x < N; ++x) top = fmaxf(top, fmaxf(fmaxf(v[x * STEP].x, v[x * STEP].y), fmaxf(v[x * STEP].z, v[x * STEP].w)));
    top = across(top, OpMaxF32{});
    float sum = 0.f;
#pragma unroll
    for (int x = 0; x < N; ++x)
        sum += (__expf(v[x * STEP].x - top) + __expf(v[x * STEP].y - top)) + (__expf(v[x * STEP].z - top) + __expf(v[x * STEP].w - top));
    sum = across(sum, OpAddF32{});
    if (there && lgrp == 0) *pms = ((unsigned long long)__float_as_uint(sum) << 32) | __float_as_uint(top);
}
// Logits behind the tile's end (its last row again) become -inf: nothing of the row.
__device__ __forceinline__ void end_rows(f32x4 &v, int row, int rows_b) {
    v.x = row < rows_b ? v.x : -INFINITY;
    v.y = row + 1 < rows_b ? v.y : -INFINITY;
    v.z = row + 2 < rows_b ? v.z : -INFINITY;
    v.w = row + 3 < rows_b ? v.w : -INFINITY;
}

// Workgroup epilogue on the logit tile of hidden rows i_lo .. i_hi - 1 (row i at zt + (i - i_lo) * tp), Q * 16 >= rows_b.
template <int Q>
__device__ __forceinline__ void tile_epilogue(const MfmaArgs &a, const float *zt, int tp, int i_lo, int i_hi, int row0, int rows_b,
                                              const int *lds_ids, unsigned long long *cand, int nwaves, int w, int lane) {
    if (a.zbuf != nullptr) {
        // one wave copies a hidden row's logits of this tile (contiguous in z) at a time
        for (int i = i_lo + w; i < i_hi; i += nwaves) {
            const float *src = zt + (size_t)(i - i_lo) * tp;
            float *dst = a.zbuf + (size_t)i * a.zpitch + row0;
            for (int t = lane; t < rows_b; t += kWave) dst[t] = src[t];
        }
        return;
    }
    int idq[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) idq[q] = lds_ids[min((lane & 15) + 16 * q, rows_b - 1)];
    // (zt is addressed by hidden row: shifted back by the rows that are not in it)
    const float *z0 = zt - (ptrdiff_t)i_lo * tp;
    for (int i0 = i_lo + 4 * w; i0 < i_hi; i0 += 4 * nwaves)
        block_epilogue_rows4<Q>(z0, tp, i0, i_hi, rows_b, a.L, idq, a.out_logp_full, (size_t)a.k, row0, a.pms, a.pkeys, a.nlists,
                                (int)blockIdx.x, lane, cand + (size_t)w * 64);
}

// ---------------------------------------------------------------- 9 .. 64 hidden rows
// A tile is RG groups of 16 rows of W_trim (1 .. 12).  From five groups on a workgroup has a wave per group, which
// multiplies its 16 rows by all 16 * NT hidden rows (2 + 2 NT operand reads for 2 NT products per stage: well below the LDS
// rate up to four groups of hidden rows); smaller tiles -- heads of up to 64 rows per CU -- have eight waves that share a
// row group, TPW groups of hidden rows each (TPW = NT otherwise).
// X: tiles of 128 + 1 .. 16 rows (the paper's trimmed sizes, so that all 256 CUs stream equal shares): the rows past
// the 128th are a ninth group in LDS that wave t < NT multiplies by hidden-row group t beside its own rows, the same
// operand layout, instructions and ranges, so equal rows give equal logits in whichever group they lie.
// A stage is KB blocks of 64 columns: one for the tiles whose block is several kilobytes per wave, two for smaller ones,
// which would spend their time at the barriers (k = 16384, n = 9, d = 2048: 23.4 us with one, 20.2 with two).
// NST stages in LDS; LPW load instructions per wave and stage.
// WGS = 2: heads of several rounds have two workgroups on a CU, with three stages and half of the registers each (two rings
// of two stages in flight hold what one of five does): a round's first loads and its epilogue, about 7 us in which the CU
// reads nothing, are hidden behind the other one's march.  k = 65536, n = 64, d = 2048 57.3 -> 51.4 us, n = 9 50.8 -> 46.6.
// k = 32768, d = 4096: n = 64 43.0 us with the logits stored, n = 32 42.1 (a plain read of the 268 MB: 40.8; the
// register-staged kernel before this one: 52.0 and 46.5).
template <int NT, int MAXW, int TPW, int KB, int NST, int LPW, bool X, int WGS, TileOut OUT>
__global__ void __launch_bounds__(MAXW *kWave) __attribute__((amdgpu_waves_per_eu(WGS == 1 ? 1 : WGS * ((MAXW + 3) / 4), WGS * ((MAXW + 3) / 4))))
head_mfma_kernel(const MfmaArgs a) {
    static_assert(!X || (MAXW == kStepWaves && TPW == NT), "the ninth group belongs to tiles of eight waves");
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int NR = OUT == kTileSlicesInOrder ? 2 : 8;
    constexpr int NA = TPW + (X ? 1 : 0);      // accumulators: own row group, and the ninth
    const int lane = lane_id();
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int RG = X ? kStepWaves : a.row_groups;
    const int GR = RG + (X ? 1 : 0);           // row groups in LDS
    const int NW = MAXW == kStepWaves ? kStepWaves : a.nwaves;
    if (a.ticket_clear != nullptr && blockIdx.x == 0 && threadIdx.x == 0)
        __hip_atomic_store(a.ticket_clear, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int tile_rows = 16 * RG + (X ? a.extra_rows : 0);
    const Columns<OUT> columns(a);
    const int row0 = blockIdx.x * tile_rows;
    const int rows_b = min(tile_rows, a.k - row0);
    const unsigned rs = (unsigned)a.d * 2u;
    const char *Wt = static_cast<const char *>(a.W) + (size_t)row0 * rs + (size_t)columns.first * 128;
    const char *hb = static_cast<const char *>(a.h) + (size_t)columns.first * 128;
    const March<NR, OUT> march(columns.stages, a.d);
    const unsigned block_bytes = (unsigned)(GR + NT) * kGroupBytes, stage_bytes = KB * block_bytes;
    const int nstages = march.ns / KB;             // (d is a multiple of 128: an even number of blocks)

    // Loads of a stage: pieces of 8 rows, first W's (two per group), then h's; the waves take LPW consecutive ones each,
    // and what is left over repeats pieces of h (the same bytes to the same place).  Rows past the end repeat the last.
    unsigned voff[LPW], lds_at[LPW];
#pragma unroll
    for (int j = 0; j < LPW; ++j) {
        const int x = w * LPW + j;
        const bool is_w = x < KB * 2 * GR;
        const int y = is_w ? x : (x - KB * 2 * GR) % (KB * 2 * NT);
        const int blk = KB == 1 ? 0 : y >= (is_w ? 2 * GR : 2 * NT) ? 1 : 0;
        const int p = y - blk * (is_w ? 2 * GR : 2 * NT);
        const int r = 8 * p + (lane >> 3);
        const int c = (lane & 7) ^ ((r >> 1) & 7);
        const int row = is_w ? min(r, rows_b - 1) : min(r, a.n - 1);
        voff[j] = (unsigned)row * rs + (unsigned)(blk * 128 + c * 16);
        lds_at[j] = (unsigned)blk * block_bytes + (unsigned)(is_w ? p : 2 * GR + p) * kPieceBytes;
    }
    auto load_stage = [&](int s, int slot) {
        const size_t col = (size_t)march.stage_of(s * KB) * 128;      // (ranges are whole stages)
#pragma unroll
        for (int j = 0; j < LPW; ++j) {
            const unsigned at = (unsigned)slot * stage_bytes + lds_at[j];
            if (w * LPW + j < KB * 2 * GR)
                lds_load16<true>(at, voff[j], Wt + col);
            else
                lds_load16<false>(at, voff[j], hb + col);
        }
    };
    // the tile's target ids, ahead of everything else
    if (OUT == kTileLists && w == 0) {
#pragma unroll
        for (int q = 0; q < 3; ++q)
            lds_load4((unsigned)a.ids_off + q * kWave * 4, (unsigned)min(q * kWave + lane, rows_b - 1) * 4u, a.map + row0);
    }
#pragma unroll
    for (int s = 0; s < NST - 1; ++s) {
        if (s < nstages) load_stage(s, s);
    }

    f32x4 acc[NA];
    RangeSums<NR, NA> sums;
    sums.clear();
#pragma unroll
    for (int t = 0; t < NA; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    // the wave's row group and hidden-row groups (eight waves on a small tile: some may have none)
    const int rg = TPW == NT ? w : w % RG, t0 = TPW == NT ? 0 : (w / RG) * TPW;
    const bool active = t0 < NT;
    const bool ninth = X && w < NT;
    // operand reads: lane (row lane % 16, 8 columns lane / 16) of k-step ks
    const int lrow = lane & 15, lgrp = lane >> 4;
    const unsigned rd = (unsigned)lrow * 128 + (unsigned)((lgrp ^ ((lrow >> 1) & 7)) * 16);
    const unsigned rd_w = rd + (unsigned)rg * kGroupBytes, rd_h = rd + (unsigned)(GR + t0) * kGroupBytes;
    const unsigned rd_xw = rd + (unsigned)kStepWaves * kGroupBytes, rd_xh = rd + (unsigned)(GR + w) * kGroupBytes;
    auto product = [&](const u32x4 &av, const u32x4 &bv, f32x4 &c) {
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av), __builtin_bit_cast(bf16x8, bv), c, 0, 0, 0);
    };
    int slot = 0, closed = 0;
    int left = march.length_of(0);      // blocks until the open range ends
    for (int s = 0; s < nstages; ++s) {
        wait_stage_and_sync<LPW, NST - 2>(nstages - 1 - s);      // stage s is in LDS, the slot of stage s - 1 is free
        if (s + NST - 1 < nstages) load_stage(s + NST - 1, slot == 0 ? NST - 1 : slot - 1);
        if (march.ranges) {
            if (left == 0) {
                sums.close(acc, march.rot, closed);
                ++closed;
                left = march.length_of(closed);
            }
            left -= KB;
        }
        const unsigned char *sb = smem + (unsigned)slot * stage_bytes;
        slot = slot == NST - 1 ? 0 : slot + 1;
        if (active) {
            u32x4 av[2 * KB], bv[2 * KB][TPW];
#pragma unroll
            for (int ks = 0; ks < 2 * KB; ++ks) {       // (piece 4 ks + lgrp: bit 2 of the piece number is 64 bytes)
                const unsigned char *kb = sb + (ks >> 1) * block_bytes;
                const unsigned half = (ks & 1) * 64u;
                av[ks] = *reinterpret_cast<const u32x4 *>(kb + (rd_w ^ half));
#pragma unroll
                for (int t = 0; t < TPW; ++t)
                    bv[ks][t] = *reinterpret_cast<const u32x4 *>(kb + (rd_h ^ half) + t * kGroupBytes);
            }
#pragma unroll
            for (int ks = 0; ks < 2 * KB; ++ks) {
#pragma unroll
                for (int t = 0; t < TPW; ++t) product(av[ks], bv[ks][t], acc[t]);
            }
        }
        if constexpr (X) {
            static_assert(!X || KB == 1, "tiles with extra rows have stages of one block");
            if (ninth) {
                u32x4 av[2], bv[2];
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) {
                    av[ks] = *reinterpret_cast<const u32x4 *>(sb + (rd_xw ^ (ks * 64u)));
                    bv[ks] = *reinterpret_cast<const u32x4 *>(sb + (rd_xh ^ (ks * 64u)));
                }
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) product(av[ks], bv[ks], acc[NA - 1]);
            }
        }
    }
    if (march.ranges) sums.template finish<OUT == kTileSlicesInOrder>(acc, march.rot, closed);
    if constexpr (OUT != kTileLists) {
        float *z = a.zbuf + (size_t)columns.slice * a.n * a.zpitch + row0;
        const bool by_parts = OUT == kTileStored && a.parts != 0;
        if (by_parts && (rows_b < 16 * GR)) {
#pragma unroll
            for (int t = 0; t < TPW; ++t) end_rows(acc[t], 16 * rg + 4 * lgrp, rows_b);
            if (X) end_rows(acc[NA - 1], kMfmaTileRows + 4 * lgrp, rows_b);
        }
        if (active) {
#pragma unroll
            for (int t = 0; t < TPW; ++t) store_z4(z, 16 * (t0 + t) + lrow, a.n, a.zpitch, 16 * rg + 4 * lgrp, min(rows_b, 16 * RG), acc[t]);
        }
        if (ninth) store_z4(z, 16 * w + lrow, a.n, a.zpitch, kMfmaTileRows + 4 * lgrp, rows_b, acc[NA - 1]);
        if (by_parts) {
            unsigned long long *pms = a.pms + (size_t)blockIdx.x * GR;
            if (active) {
#pragma unroll
                for (int t = 0; t < TPW; ++t) {
                    const int i = 16 * (t0 + t) + lrow;
                    publish_part<1, 1>(acc + t, pms + (size_t)i * a.parts + rg, i < a.n && 16 * rg < rows_b, lgrp);
                }
            }
            if (ninth) {
                const int i = 16 * w + lrow;
                publish_part<1, 1>(acc + NA - 1, pms + (size_t)i * a.parts + kStepWaves, i < a.n && kMfmaTileRows < rows_b, lgrp);
            }
        }
    } else {
        wait_and_sync<0>();      // every wave is done with the ring: it becomes the logit tile

        float *zt = reinterpret_cast<float *>(smem);
        const int tp = 16 * GR + 1;
        if (active) {
#pragma unroll
            for (int t = 0; t < TPW; ++t) {
                const int i = 16 * (t0 + t) + lrow;
                if (i < a.n) store_logits4(zt + (size_t)i * tp + 16 * rg + 4 * lgrp, acc[t]);
            }
        }
        if (ninth) {
            const int i = 16 * w + lrow;
            if (i < a.n) store_logits4(zt + (size_t)i * tp + kMfmaTileRows + 4 * lgrp, acc[NA - 1]);
        }
        __syncthreads();
        const int *lds_ids = reinterpret_cast<const int *>(smem + a.ids_off);
        unsigned long long *cand =
            reinterpret_cast<unsigned long long *>(smem + (((size_t)a.n * tp * sizeof(float) + 15) & ~(size_t)15));
        constexpr int Q = X ? 9 : MAXW > kStepWaves ? kMfmaMaxWaves : 8;
        tile_epilogue<Q>(a, zt, tp, 0, a.n, row0, rows_b, lds_ids, cand, NW, w, lane);
    }
}

// ---------------------------------------------------------------- 65 .. 256 hidden rows
// Tiles of 32 * MT rows by 64 * NTT hidden rows, eight waves as a 2 x 4 grid of (16 * MT) x (16 * NTT) each: with more hidden
// rows than 64 the operand reads of a wave per row group would exceed the LDS rate.  Per stage and wave there are two
// k-steps of MT * NTT products; the operands of one are read while the other is multiplied, the barrier that hands the
// slot on sits between them, and the loads of the freed slot are spread over the products that follow it -- issued
// in one go they kept the wave from its products (n = 256, k = 32768, d = 8192: 149 against 140 us).
// From 129 hidden rows on, and with 129 to 192 of them on tiles of 64 and more head rows, a stage's pieces of h are asked for
// before W's: h comes from the L2 soon and keeps the queue short for W behind it (W first / h first, us: n = 256, k = 32768,
// d = 5120 111.1 / 100.0, d = 3072 71.1 / 66.0, d = 8192 158.0 / 155.9; n = 181, k = 32768, d = 5120 90.5 / 85.9).
// 129 to 192 rows on tiles of 32 tie on average, but h first is up to 5 % slower where d is a multiple of 1024 and not of 2048
// (n = 181, d = 5120, k = 2950 48.0 / 50.3, k = 1500 46.6 / 49.0; d = 8192, k = 1500, n = 129 63.5 / 62.0); with up to 128 rows
// W's pieces are the larger part (n = 128, k = 8192, d = 5120 39.8 / 42.3; n = 100, k = 24000 59.1 / 61.5).
// The march of n = 256, d = 8192 is bound by power: the clock falls from 2.4 to 1.6 .. 1.9 GHz while loads and products run
// together, and stays at 2.4 with either alone.
// PACKED: h was re-laid by pack_h_kernel, a stage's pieces one after the other as they lie in LDS.
template <int MT, int NTT, int NST, int NR, bool PACKED, TileOut OUT>
__global__ void __launch_bounds__(kStepWaves *kWave) head_mfma_wide_kernel(const MfmaArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int TM = 32 * MT, TN = 64 * NTT;
    constexpr int kPieces = (TM + TN) / 8, LPW = (kPieces + kStepWaves - 1) / kStepWaves;
    constexpr unsigned kStage = (TM + TN) * 128u;
    constexpr int NP = MT * NTT;               // products per k-step
    constexpr bool kHiddenFirst = NTT == 4 || (NTT == 3 && MT >= 2);
    const int lane = lane_id();
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wn = w & 3, wm = w >> 2;
    if (a.ticket_clear != nullptr && blockIdx.x == 0 && threadIdx.x == 0)
        __hip_atomic_store(a.ticket_clear, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const Columns<OUT> columns(a);
    const int row0 = blockIdx.x * TM;
    const int rows_b = min(TM, a.k - row0);
    const unsigned rs = (unsigned)a.d * 2u;
    const char *Wt = static_cast<const char *>(a.W) + (size_t)row0 * rs + (size_t)columns.first * 128;
    // (re-laid: a stage's pieces lie one after the other)
    const char *hb = PACKED ? static_cast<const char *>(a.hpack) + (size_t)columns.first * (TN * 128) : static_cast<const char *>(a.h) + (size_t)columns.first * 128;
    const March<NR, OUT> march(columns.stages, a.d);

    unsigned voff[LPW], lds_at[LPW];
#pragma unroll
    for (int j = 0; j < LPW; ++j) {
        // every wave takes its share of W's pieces and of h's (left-over slots repeat pieces of h)
        const int x = j * kStepWaves + w;
        const bool is_w = x < TM / 8;
        const int p = is_w ? x : (x - TM / 8) % (TN / 8);
        const int r = 8 * p + (lane >> 3);
        const int c = (lane & 7) ^ ((r >> 1) & 7);
        const int row = is_w ? min(r, rows_b - 1) : min(r, a.n - 1);
        voff[j] = !is_w && PACKED ? (unsigned)(p * kPieceBytes + lane * 16) : (unsigned)row * rs + (unsigned)c * 16u;
        lds_at[j] = (unsigned)(is_w ? p : TM / 8 + p) * kPieceBytes;
    }
    const char *pw = Wt, *ph = hb;
    unsigned at = 0;
    auto aim = [&](int s, int slot) {
        const size_t u = (size_t)march.stage_of(s);
        pw = Wt + u * 128;
        ph = hb + u * (PACKED ? TN * 128 : 128);
        at = (unsigned)slot * kStage;
    };
    auto load_piece = [&](int j) {
        // (the last of W's rounds may be shared with h: the two differ by wave)
        if ((j + 1) * kStepWaves <= TM / 8 || (j * kStepWaves < TM / 8 && j * kStepWaves + w < TM / 8))
            lds_load16<true>(at + lds_at[j], voff[j], pw);
        else
            lds_load16<false>(at + lds_at[j], voff[j], ph);
    };
    if (OUT == kTileLists && w == 0) {
#pragma unroll
        for (int q = 0; q < (TM + kWave - 1) / kWave; ++q)
            lds_load4((unsigned)a.ids_off + q * kWave * 4, (unsigned)min(q * kWave + lane, rows_b - 1) * 4u, a.map + row0);
    }
#pragma unroll
    for (int s = 0; s < NST; ++s) {
        if (s >= march.ns) break;
        aim(s, s);
#pragma unroll
        for (int j = 0; j < LPW; ++j) load_piece(j);
    }
    f32x4 acc[NP];
    RangeSums<NR, NP> sums;
    sums.clear();
#pragma unroll
    for (int x = 0; x < NP; ++x) acc[x] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int lrow = lane & 15, lgrp = lane >> 4;
    const unsigned rd = (unsigned)lrow * 128 + (unsigned)((lgrp ^ ((lrow >> 1) & 7)) * 16);
    const unsigned rd_w = rd + (unsigned)(wm * MT) * kGroupBytes, rd_h = rd + (unsigned)(TM / 16 + wn * NTT) * kGroupBytes;
    u32x4 a0[MT], b0[NTT], a1[MT], b1[NTT];
    auto read_operands = [&](u32x4(&av)[MT], u32x4(&bv)[NTT], unsigned ks, int slot) {
        const unsigned char *sb = smem + (unsigned)slot * kStage;
#pragma unroll
        for (int m = 0; m < MT; ++m) av[m] = *reinterpret_cast<const u32x4 *>(sb + (rd_w ^ (ks * 64u)) + m * kGroupBytes);
#pragma unroll
        for (int t = 0; t < NTT; ++t) bv[t] = *reinterpret_cast<const u32x4 *>(sb + (rd_h ^ (ks * 64u)) + t * kGroupBytes);
    };
    auto product = [&](int x, const u32x4(&av)[MT], const u32x4(&bv)[NTT]) {
        acc[x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av[x / NTT]),
                                                         __builtin_bit_cast(bf16x8, bv[x % NTT]), acc[x], 0, 0, 0);
    };
    wait_stage_and_sync<LPW, NST - 1>(march.ns - 1);
    int slot = 0, closed = 0;
    int left = march.length_of(0);
    read_operands(a0, b0, 0, 0);
    for (int s = 0; s < march.ns; ++s) {
        read_operands(a1, b1, 1, slot);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int x = 0; x < NP; ++x) product(x, a0, b0);
        __builtin_amdgcn_sched_barrier(0);
        wait_stage_and_sync<LPW, NST - 2>(march.ns - 2 - s);      // stage s + 1 is in LDS; everyone has read stage s
        const bool more = s + NST < march.ns;
        if (more) aim(s + NST, slot);
        slot = slot == NST - 1 ? 0 : slot + 1;
        read_operands(a0, b0, 0, slot);            // (past the last stage: an old slot, never used)
        __builtin_amdgcn_sched_barrier(0);
        constexpr int kEvery = NP / LPW > 0 ? NP / LPW : 1;
#pragma unroll
        for (int x = 0; x < NP; ++x) {
            if (x % kEvery == 0 && x / kEvery < LPW) {
                if (more) load_piece(kHiddenFirst ? LPW - 1 - x / kEvery : x / kEvery);
                __builtin_amdgcn_sched_barrier(0);
            }
            product(x, a1, b1);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int j = 0; j < LPW; ++j) {
            if (j * kEvery >= NP && more) load_piece(kHiddenFirst ? LPW - 1 - j : j);
        }
        if (NR > 1 && march.ranges && --left == 0 && s + 1 < march.ns) {
            sums.close(acc, march.rot, closed);
            ++closed;
            left = march.length_of(closed);
        }
    }
    if (NR > 1 && march.ranges) sums.template finish<OUT == kTileSlicesInOrder>(acc, march.rot, closed);
    if constexpr (OUT != kTileLists) {
        float *z = a.zbuf + (size_t)columns.slice * a.n * a.zpitch + row0;
        const bool by_parts = OUT == kTileStored && a.parts != 0;
        if (by_parts && rows_b < TM) {
#pragma unroll
            for (int x = 0; x < NP; ++x) end_rows(acc[x], 16 * (wm * MT + x / NTT) + 4 * lgrp, rows_b);
        }
#pragma unroll
        for (int t = 0; t < NTT; ++t) {
#pragma unroll
            for (int m = 0; m < MT; ++m)
                store_z4(z, 16 * (wn * NTT + t) + lrow, a.n, a.zpitch, 16 * (wm * MT + m) + 4 * lgrp, rows_b, acc[m * NTT + t]);
        }
        if (by_parts) {
            unsigned long long *pms = a.pms + 2 * blockIdx.x + wm;
#pragma unroll
            for (int t = 0; t < NTT; ++t) {
                const int i = 16 * (wn * NTT + t) + lrow;
                publish_part<MT, NTT>(acc + t, pms + (size_t)i * a.parts, i < a.n && 16 * wm * MT < rows_b, lgrp);
            }
        }
    } else {
        wait_and_sync<0>();      // every wave is done with the ring: it becomes the logit tile

        // logit tile: all hidden rows at once, or (a.passes = 2) the lower and upper half of the wave columns in turn
        float *zt = reinterpret_cast<float *>(smem);
        constexpr int tp = TM + 1;
        const int *lds_ids = reinterpret_cast<const int *>(smem + a.ids_off);
        const int per_pass = TN / a.passes;            // hidden rows per pass
        unsigned long long *cand = reinterpret_cast<unsigned long long *>(
            smem + (((size_t)min(per_pass, a.n) * tp * sizeof(float) + 15) & ~(size_t)15));
        for (int pass = 0; pass < a.passes; ++pass) {
            const int i_lo = pass * per_pass, i_hi = min(a.n, i_lo + per_pass);
            if (i_lo >= i_hi) break;                   // (uniform)
            if (pass > 0) __syncthreads();             // the tile of the pass before is done with
#pragma unroll
            for (int t = 0; t < NTT; ++t) {
                const int i = 16 * (wn * NTT + t) + lrow;
                if (i >= i_lo && i < i_hi) {
#pragma unroll
                    for (int m = 0; m < MT; ++m)
                        store_logits4(zt + (size_t)(i - i_lo) * tp + 16 * (wm * MT + m) + 4 * lgrp, acc[m * NTT + t]);
                }
            }
            __syncthreads();
            tile_epilogue<2 * MT>(a, zt, tp, i_lo, i_hi, row0, rows_b, lds_ids, cand, kStepWaves, w, lane);
        }
    }
}

// Re-lays h for the kernel above: piece (stage u, 8 rows p) is 1 KiB, lane l's 16 bytes at 16 l (rows past n repeat
// row n - 1; their products are never read).  A wave per piece: four stages of a workgroup, p = blockIdx.y.  Bound by its
// launch and one trip to memory: 5.3 us for 4 MiB, with or without a 64-bit division for the address.
__global__ void __launch_bounds__(256) pack_h_kernel(const u32x4 *__restrict__ h, u32x4 *__restrict__ hp, int n, int d) {
    const int lane = (int)(threadIdx.x & 63), p = (int)blockIdx.y;
    const int u = (int)(blockIdx.x * 4 + (threadIdx.x >> 6));
    if (u >= d / kStageCols) return;
    const int r = 8 * p + (lane >> 3);
    const int c = (lane & 7) ^ ((r >> 1) & 7);
    hp[((size_t)u * gridDim.y + p) * kWave + lane] = h[(size_t)min(r, n - 1) * (unsigned)(d / 8) + (unsigned)(u * 8 + c)];
}

template <auto kern>
hipError_t launch_tile(const MfmaArgs &a, int threads, size_t lds, hipStream_t st) {
    static LdsLimitOnce lds_limit;
    const hipError_t e = allow_dynamic_lds(lds_limit, {reinterpret_cast<const void *>(kern)}, kMaxDynamicLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(a.nlists / a.splits, a.splits), dim3(threads), lds, st, a);
    return hipGetLastError();
}

// A lane's offset inside a tile or h is 32 bits: 255 rows of less than 16 MiB.
bool offsets_fit(const MfmaArgs &a) { return (size_t)a.d * 2 < ((size_t)1 << 24); }

constexpr int kTwinRingBytes = 79 * 1024;     // ... of two workgroups on a CU, each
constexpr int kRingBytes = 156 * 1024;         // LDS for the ring; the ids and what the epilogue needs fit behind it

// Variants of head_mfma_kernel: most waves, hidden-row groups per wave, blocks per stage, stages, loads per wave and stage.
struct RowsVariant {
    int max_waves, tpw, blocks, stages, loads;
};
constexpr RowsVariant rows_variant(int NT, int row_groups, bool extra, bool twin = false) {
    if (twin) return NT == 2 ? RowsVariant{8, 2, 1, 3, 3} : RowsVariant{8, 4, 1, 3, 3};
    if (extra) return NT == 2 ? RowsVariant{8, 2, 1, 7, 3} : RowsVariant{8, 4, 1, 6, 4};
    if (row_groups <= 2) return NT == 2 ? RowsVariant{8, 1, 2, 9, 2} : RowsVariant{8, 1, 2, 6, 3};
    if (row_groups <= 4) return NT == 2 ? RowsVariant{8, 1, 2, 6, 3} : RowsVariant{8, 2, 2, 4, 4};
    if (row_groups <= kMfmaFewWaves) return NT == 2 ? RowsVariant{7, 2, 2, 4, 6} : RowsVariant{7, 4, 1, 7, 4};
    if (row_groups == kStepWaves) return NT == 2 ? RowsVariant{8, 2, 1, 7, 3} : RowsVariant{8, 4, 1, 6, 3};
    return NT == 2 ? RowsVariant{12, 2, 1, 5, 3} : row_groups == 12 ? RowsVariant{12, 4, 1, 4, 3} : RowsVariant{12, 4, 1, 5, 3};
}
// (every piece of a stage has a load; the ring fits)
constexpr bool rows_variant_ok(int NT, int row_groups, bool extra, bool twin = false) {
    const RowsVariant v = rows_variant(NT, row_groups, extra, twin);
    const int groups = row_groups + (extra ? 1 : 0) + NT, waves = row_groups <= 4 ? kStepWaves : row_groups;
    return waves <= v.max_waves && v.loads * waves >= 2 * v.blocks * groups &&
           v.stages * v.blocks * groups * kGroupBytes <= (twin ? kTwinRingBytes : kRingBytes) && v.loads * (v.stages - 2) <= 63 &&
           v.tpw * (row_groups <= 4 ? kStepWaves / row_groups : 1) >= NT;
}
static_assert(rows_variant_ok(2, 8, false, true) && rows_variant_ok(4, 8, false, true));
static_assert(rows_variant_ok(2, 8, true) && rows_variant_ok(4, 8, true));
static_assert(rows_variant_ok(2, 1, false) && rows_variant_ok(2, 2, false) && rows_variant_ok(2, 3, false) && rows_variant_ok(2, 4, false));
static_assert(rows_variant_ok(2, 5, false) && rows_variant_ok(2, 6, false) && rows_variant_ok(2, 7, false) && rows_variant_ok(2, 8, false));
static_assert(rows_variant_ok(2, 9, false) && rows_variant_ok(2, 10, false) && rows_variant_ok(2, 11, false) && rows_variant_ok(2, 12, false));
static_assert(rows_variant_ok(4, 1, false) && rows_variant_ok(4, 2, false) && rows_variant_ok(4, 3, false) && rows_variant_ok(4, 4, false));
static_assert(rows_variant_ok(4, 5, false) && rows_variant_ok(4, 6, false) && rows_variant_ok(4, 7, false) && rows_variant_ok(4, 8, false));
static_assert(rows_variant_ok(4, 9, false) && rows_variant_ok(4, 10, false) && rows_variant_ok(4, 11, false) && rows_variant_ok(4, 12, false));
TileOut tile_out(const MfmaArgs &a) {
    if (a.zbuf == nullptr || a.zvec == 0) return kTileLists;
    return a.splits == 1 ? kTileStored : a.slice_ranges != 0 ? kTileSlices : kTileSlicesInOrder;
}
// (slices: tiles of 64 and of 128 rows, one workgroup to a CU; unaligned logits go through LDS and have no slices)
template <int NT, int RG, bool X, bool TWIN = false>
hipError_t launch_rows(const MfmaArgs &a, size_t lds, hipStream_t st) {
    constexpr RowsVariant v = rows_variant(NT, RG, X, TWIN);
    auto launch = [&](auto out) {
        return launch_tile<head_mfma_kernel<NT, v.max_waves, v.tpw, v.blocks, v.stages, v.loads, X, TWIN ? 2 : 1, decltype(out)::value>>(
            a, a.nwaves * kWave, lds, st);
    };
    if (tile_out(a) == kTileStored) return launch(std::integral_constant<TileOut, kTileStored>{});
    if constexpr ((RG == 4 || RG == 8) && !X && !TWIN) {
        if (tile_out(a) == kTileSlices) return launch(std::integral_constant<TileOut, kTileSlices>{});
        if (tile_out(a) == kTileSlicesInOrder) return launch(std::integral_constant<TileOut, kTileSlicesInOrder>{});
    }
    return a.splits == 1 ? launch(std::integral_constant<TileOut, kTileLists>{}) : hipErrorInvalidValue;
}
template <int NT>
hipError_t launch_rows_nt(const MfmaArgs &a, size_t lds, hipStream_t st) {
    if (a.extra_rows != 0) return launch_rows<NT, 8, true>(a, lds, st);
    if (a.twin != 0) return a.row_groups == kStepWaves ? launch_rows<NT, 8, false, true>(a, lds, st) : hipErrorInvalidValue;
    // (one representative row count per variant)
    if (a.row_groups <= 2) return launch_rows<NT, 2, false>(a, lds, st);
    if (a.row_groups <= 4) return launch_rows<NT, 4, false>(a, lds, st);
    if (a.row_groups <= kMfmaFewWaves) return launch_rows<NT, 7, false>(a, lds, st);
    if (a.row_groups == kStepWaves) return launch_rows<NT, 8, false>(a, lds, st);
    if (a.row_groups < kMfmaMaxWaves) return launch_rows<NT, 11, false>(a, lds, st);
    return launch_rows<NT, 12, false>(a, lds, st);
}

constexpr size_t wide_stage_bytes(int MT, int NTT) { return (size_t)(32 * MT + 64 * NTT) * 128; }
constexpr int wide_stages(int MT, int NTT) {
    const int s = (int)(kRingBytes / wide_stage_bytes(MT, NTT));
    return s < 6 ? s : 6;
}
// ranges: as many as the registers (256 per lane) hold sums of beside two sets of operands
constexpr int wide_ranges(int MT, int NTT) {
    const int acc = 4 * MT * NTT, ops = 8 * (MT + NTT);
    return 5 * acc + ops <= 208 ? 8 : 3 * acc + ops <= 208 ? 4 : 2;
}
// (slices: tiles of 64, 128 and 160 rows.  Two ranges that tiles rotate are chains of an eighth of the row from four slices on -- n = 250,
// k = 7000, d = 8192 46.8 us, in order 50.1 -- and longer ones with two and three: in order, n = 224, k = 14000, d = 8192 74.6 / 75.9,
// n = 256 83.4 / 87.0, n = 256, k = 9000, d = 6144 47.3 / 50.0)
template <int MT, int NTT, bool PACKED>
hipError_t launch_wide_as(const MfmaArgs &a, size_t lds, hipStream_t st) {
    constexpr int NST = wide_stages(MT, NTT), NR = wide_ranges(MT, NTT);
    auto launch = [&](auto out) {
        constexpr TileOut OUT = decltype(out)::value;
        return launch_tile<head_mfma_wide_kernel<MT, NTT, NST, (OUT == kTileSlicesInOrder ? 2 : NR), PACKED, OUT>>(a, kStepWaves * kWave, lds, st);
    };
    const TileOut out = tile_out(a);
    if (out == kTileStored) return launch(std::integral_constant<TileOut, kTileStored>{});
    if constexpr (MT == 2 || MT == 4 || MT == 5) {
        if (out == kTileSlices && (NR > 2 || a.splits >= 4)) return launch(std::integral_constant<TileOut, kTileSlices>{});
        if (out == kTileSlices || out == kTileSlicesInOrder) return launch(std::integral_constant<TileOut, kTileSlicesInOrder>{});
    }
    return a.splits == 1 ? launch(std::integral_constant<TileOut, kTileLists>{}) : hipErrorInvalidValue;
}
template <int MT, int NTT>
hipError_t launch_wide(const MfmaArgs &a, size_t lds, hipStream_t st) {
    if (a.hpack == nullptr) return launch_wide_as<MT, NTT, false>(a, lds, st);
    if constexpr (NTT == 4) {
        hipLaunchKernelGGL(pack_h_kernel, dim3((unsigned)((a.d / kStageCols + 3) / 4), 8 * NTT), dim3(256), 0, st, static_cast<const u32x4 *>(a.h),
                           static_cast<u32x4 *>(a.hpack), a.n, a.d);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        return launch_wide_as<MT, NTT, true>(a, lds, st);
    }
    return hipErrorInvalidValue;
}
template <int NTT>
hipError_t launch_wide_ntt(const MfmaArgs &a, size_t lds, hipStream_t st) {
    switch (a.row_groups) {
        case 2: return launch_wide<1, NTT>(a, lds, st);
        case 4: return launch_wide<2, NTT>(a, lds, st);
        case 6: return launch_wide<3, NTT>(a, lds, st);
        case 8: return launch_wide<4, NTT>(a, lds, st);
        case 10: return launch_wide<5, NTT>(a, lds, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

// ---------------------------------------------------------------- host side
size_t rows_ring_bytes(int NT, int row_groups, bool extra, bool twin) {
    const RowsVariant v = rows_variant(NT, row_groups, extra, twin);
    return (size_t)v.stages * v.blocks * (row_groups + (extra ? 1 : 0) + NT) * kGroupBytes;
}
size_t wide_ring_bytes(int MT, int NTT) { return wide_stages(MT, NTT) * wide_stage_bytes(MT, NTT); }

hipError_t launch_head_mfma_rows(int NT, const MfmaArgs &a, size_t lds, hipStream_t st) {
    if (!offsets_fit(a)) return hipErrorInvalidValue;
    switch (NT) {
        case 2: return launch_rows_nt<2>(a, lds, st);
        case 4: return launch_rows_nt<4>(a, lds, st);
        default: return hipErrorInvalidValue;
    }
}
hipError_t launch_head_mfma_wide(int NTT, const MfmaArgs &a, size_t lds, hipStream_t st) {
    if (!offsets_fit(a)) return hipErrorInvalidValue;
    switch (NTT) {
        case 2: return launch_wide_ntt<2>(a, lds, st);
        case 3: return launch_wide_ntt<3>(a, lds, st);
        case 4: return launch_wide_ntt<4>(a, lds, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace vt
