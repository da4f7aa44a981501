// Draft step for up to 8 hidden rows on the matrix cores, z[n, k] = h[n, d] W_trim[k, d]^T
// (v_mfma_f32_16x16x32_bf16), bound by the single pass over W_trim; several heads' rows in one launch; and the merge
// kernels behind this and the other streaming kernels.
//
// One workgroup (8 waves) owns a tile of 128 rows of W_trim, 16 per wave:
//   * W is read from HBM exactly once, with row-contiguous 256-byte segments per
//     load instruction (4 rows x 256 B), several units in flight per wave; a unit
//     (16 rows x 128 columns) passes through a small wave-private LDS buffer that
//     re-lays it out as MFMA A-operands (row pitch 272 B: conflict-free reads);
//   * h is the B-operand: all of it sits in LDS, shared by the waves (chunk by chunk where it is too long);
//   * accumulators stay in registers over the whole contraction; the logits are never written to memory;
//   * the tile's logits go to an LDS tile (aliasing the staging buffers) and the
//     same workgroup epilogue as the small-n kernel produces (max, sum-exp) and
//     the tile's best candidates per hidden row;
//   * a second small kernel merges the tiles: one wave per hidden row.
#include "vt_device.h"
#include "vt_launch.h"
#include "vt_ranges.h"
#include "vt_step.h"
#include "vt_step_tail.h"
#include "vt_tree_dev.h"
#include <mutex>
#include <type_traits>

namespace vt {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;

constexpr int kUnitCols = 128;                       // columns per staged unit (256 B per row)
constexpr int kStagePitch = 272;                     // bytes per staged row: 256 + 16 (bank spread)
constexpr int kStageUnitBytes = 16 * kStagePitch;    // one unit of one wave
constexpr int kStageBytes = kStepWaves * 2 * kStageUnitBytes;   // double-buffered, all waves of an 8-wave workgroup
constexpr int kPrefetchUnits = kMfmaPrefetchUnits;   // units of W in flight per wave (12 KiB)

__device__ __forceinline__ void stream_load16(u32x4 &dst, unsigned voff, const void *sbase) {
    asm volatile("global_load_dwordx4 %0, %1, %2 nt" : "=v"(dst) : "v"(voff), "s"(sbase) : "memory");
}
// h pieces stay cacheable: every workgroup re-reads them from L2
__device__ __forceinline__ void cached_load16(u32x4 &dst, unsigned voff, const void *sbase) {
    asm volatile("global_load_dwordx4 %0, %1, %2" : "=v"(dst) : "v"(voff), "s"(sbase) : "memory");
}
__device__ __forceinline__ void request_dword(int &dst, const int *p) {
    asm volatile("global_load_dword %0, %1, off" : "=v"(dst) : "v"(p) : "memory");
}
template <int N>
__device__ __forceinline__ void wait_ids(int (&b)[3]) {
    asm volatile("s_waitcnt vmcnt(%3)" : "+v"(b[0]), "+v"(b[1]), "+v"(b[2]) : "n"(N));
}
constexpr int kMaxPieces = kMfmaChunkPieces;   // 16-byte pieces of an h chunk per thread
template <int N>
__device__ __forceinline__ void wait_pieces(u32x4 (&b)[kMaxPieces]) {
    asm volatile("s_waitcnt vmcnt(%9)"
                 : "+v"(b[0]), "+v"(b[1]), "+v"(b[2]), "+v"(b[3]), "+v"(b[4]), "+v"(b[5]), "+v"(b[6]), "+v"(b[7]),
                   "+v"(b[8])
                 : "n"(N));
}
template <int N>
__device__ __forceinline__ void wait_unit(u32x4 (&b)[4]) {
    asm volatile("s_waitcnt vmcnt(%4)" : "+v"(b[0]), "+v"(b[1]), "+v"(b[2]), "+v"(b[3]) : "n"(N));
}

// MAXW: most waves a workgroup of this instantiation is launched with.  Eight is the rule: a wave per 16 rows of a
// 128-row tile.  With all of h in LDS the workgroup may have any number of waves up to
// MAXW = 12: the tile is then 16 * (waves / KS) rows, so that a head of any size up to 256 * 192 rows is cut into
// at most 256 tiles -- one round on 256 CUs -- instead of a second, nearly empty round of 128-row tiles.
// XG (eight waves, up to 8 hidden rows, d a multiple of 1024): the tile has 128 + extra_rows rows.  The rows past
// the 128th form one more 16-row group; wave w multiplies the w-th eighth of its columns after its own 16 rows, so
// all waves stream equal shares whatever the tile height is -- a head of k = 32975 rows is 256 tiles of 129 rows,
// one per CU, instead of 258 tiles of 128.  To keep a row's logit independent of the group it lies in, every logit is
// then formed from the partial sums P0 .. P7 of the eight column parts, each accumulated from zero in ascending
// order, as ((P0 + P1) + (P2 + P3)) + ((P4 + P5) + (P6 + P7)) -- in registers for a wave's own rows (the parts are
// the ranges described below), from LDS for the shared group.  All waves march over the columns of their
// own rows in step, as without the shared group.  (Measured alternatives at k = 32975, n = 8, d = 3072 / 4096:
// this kernel 40.1 / 54.0 us; every wave starting at another part, the eight partial sums kept in registers:
// 40.8 / 57.4; all rows cut into near-equal groups whose (group, part) tasks are dealt to the waves: 40.8 / 50.5;
// nine waves of 16 rows on 229 CUs: 41.4 / 51.4; the small-n kernel: 41.8 / 51.7.  The planner uses it where rows
// are not a multiple of 2 KiB.)
// MH: the tiles of several heads in one launch (see MultiHeadTable); one group of hidden rows, all of h in LDS.  H_FIRST: see h_first().
template <int MAXW, bool XG = false, bool MH = false, bool H_FIRST = false>
__global__ void __launch_bounds__(MAXW *kWave) __attribute__((amdgpu_waves_per_eu(1, (MAXW + 3) / 4)))
head_mfma_kernel(const MfmaArgs a, const std::conditional_t<MH, MultiHeadTable, SingleHead> mh) {
    static_assert(!MH || !XG, "several heads per launch: plain tiles");
    static_assert(!XG || MAXW == kStepWaves, "the shared row group is built for eight waves");
    extern __shared__ __align__(16) unsigned char smem[];
    const int NW = MAXW == kStepWaves ? kStepWaves : a.nwaves;     // waves of this workgroup
    unsigned char *stage = smem;                       // [waves][2][16][272]
    unsigned char *hbuf = smem + (size_t)NW * 2 * kStageUnitBytes;   // [8][hpitch]
    float *zt = reinterpret_cast<float *>(smem);       // logit tile, aliases both after the contraction

    const int lane = lane_id();
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (a.ticket_clear != nullptr && blockIdx.x == 0 && threadIdx.x == 0)
        __hip_atomic_store(a.ticket_clear, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // Small heads (up to 8 hidden rows only): with fewer than ~160 tiles of 128 rows the tiles shrink to
    // 16 * NW / KS rows and KS waves share a group of 16 rows, each taking 1 / KS of the columns; their partial
    // logits meet in the LDS tile of the epilogue, summed in wave order.
    const int KS = a.ksplit;
    const int tile_rows = 16 * (NW / KS) + (XG ? a.extra_rows : 0);
    const int rg = w / KS, ksi = w % KS;               // row group of the wave, its share of the columns
    // the head this tile belongs to, its first tile, size, rows and ids
    int hd = 0, tile_lo = 0, head_k = a.k;
    const void *head_W = a.W;
    const int *head_map = a.map;
    if constexpr (MH) {
        for (int q = 1; q < mh.n_heads; ++q) hd = (int)blockIdx.x >= mh.tile_first[q] ? q : hd;
        tile_lo = mh.tile_first[hd];
        head_k = mh.k[hd];
        head_W = mh.W[hd];
        head_map = mh.map[hd];
    }
    const int row0 = ((int)blockIdx.x - tile_lo) * tile_rows;
    const int rows_b = min(tile_rows, head_k - row0);
    const size_t rs = (size_t)a.d * 2;
    const int lrow = lane & 15, lgrp = lane >> 4;

    // per-lane byte offsets of the 4 load instructions of a unit: instruction j covers rows 4j..4j+3
    // of this wave's 16 rows, 16 lanes x 16 B per row; rows past the end of W repeat the last row
    unsigned voff[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int r = min(16 * rg + 4 * j + lgrp, rows_b - 1);
        // (24-bit factors: a 64-bit multiply-add here may name a register with a load in flight as its unused half)
        voff[j] = __umul24((unsigned)r, (unsigned)(a.d * 2)) + (unsigned)lrow * 16u;
    }
    // the shared group: rows 128 .. of the tile (rows past its end repeat the last row)
    // (kept as the distance from the wave's own rows: choosing between two arrays by a run-time flag would put
    // both into scratch memory)
    unsigned vdelta[XG ? 4 : 1];
    if constexpr (XG) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int r = min(kMfmaTileRows + 4 * j + lgrp, rows_b - 1);
            vdelta[j] = __umul24((unsigned)r, (unsigned)(a.d * 2)) + (unsigned)lrow * 16u - voff[j];
        }
    }
    const char *Wt = static_cast<const char *>(head_W) + (size_t)row0 * rs;
    const int nunits = a.d / kUnitCols;
    const int nun = nunits / KS;                       // units of this wave's own rows
    const int PL = nunits / 8;                         // XG: units per column part
    const int ntot = XG ? nun + PL : nun;              // units this wave streams
    // The start of the march rotates over column ranges (vt_ranges.h) where rows are a multiple of 4 KiB apart, the ones
    // that crowd (at d = 3072 the plain march is 0.6 us faster).  Eight ranges for tiles of eight waves (k = 32768, d = 2048:
    // 25.9 us for one hidden row and 28.8 for eight; 27.6 and 30.4 with four), four for any number of waves, whose tiles lie
    // a different number of pages apart at every height (k = 40000, d = 4096, n = 8: 59.0 against 60.7).
    // The ranges are equal at d = 16384 too, where they lie whole multiples of 4 KiB apart: starts 512 bytes off gained at
    // some sizes what they lost at others (n = 8: k = 20000 116.7 / 113.8 us, k = 32768 167.4 / 168.2; n = 6, k = 30000
    // 153.5 / 157.0).
    constexpr int NR = MAXW > kStepWaves ? 4 : 8;
    const bool rotate = KS == 1 && nunits >= 8 && a.d % 2048 == 0;
    const int rot = !rotate ? 0 : NR == 4 ? ((int)blockIdx.x >> 3) & 3 : first_range<NR>((int)blockIdx.x);
    const int upr = nunits / NR;                       // units per range (XG: per column part)
    const int ustart = KS > 1 ? ksi * nun : rot * upr;
    const int hstart = KS > 1 ? 0 : ustart;            // first unit of h's layout in LDS (the same for all waves)
    // unit processed at step s (0 <= s < nun)
    auto unit_of = [&](int s) {
        const int u = ustart + s;
        return u >= nunits ? u - nunits : u;
    };
    auto load_unit = [&](int u, u32x4(&dst)[4]) {
        if constexpr (XG) {
            u = min(u, ntot - 1);
            const bool own = u < nun;
            const char *p = Wt + (size_t)(own ? unit_of(u) : w * PL + (u - nun)) * (kUnitCols * 2);
            const unsigned shared = own ? 0u : 0xFFFFFFFFu;
#pragma unroll
            for (int j = 0; j < 4; ++j) stream_load16(dst[j], voff[j] + (vdelta[j] & shared), p);
        } else {
            const char *p = Wt + (size_t)unit_of(min(u, nun - 1)) * (kUnitCols * 2);
#pragma unroll
            for (int j = 0; j < 4; ++j) stream_load16(dst[j], voff[j], p);
        }
    };
    u32x4 areg[kPrefetchUnits][4];

    f32x4 acc[1];
    RangeSums<NR, 1> sums;
    sums.clear();
    acc[0] = f32x4{0.f, 0.f, 0.f, 0.f};
    int closed = 0;        // ranges finished so far
    int in_range = 0;      // units of the open range done so far
    f32x4 own = f32x4{0.f, 0.f, 0.f, 0.f};      // XG: the logits of the wave's own rows

    unsigned char *my_stage = stage + (size_t)w * 2 * kStageUnitBytes;
    // staging writes: instruction j, lane (row 4j + lgrp, 16-byte chunk lrow)
    // operand reads : lane (row lrow, k-group lgrp) of k-step ks -> bytes ks*64 + lgrp*16
    const int wr_off = lgrp * kStagePitch + lrow * 16;
    const int rd_off = lrow * kStagePitch + lgrp * 16;
    // up to 8 hidden rows: LDS holds 8 rows of h and lanes 8..15 of the operand repeat them (their products
    // are never read)
    constexpr int hrows = 8;
    const int hrow_off = (lrow & (hrows - 1)) * a.hpitch + lgrp * 16;

    // ---- h chunks: the columns of KC / 128 consecutive steps, of every hidden row (zero rows up to 8), live in LDS.  The next
    // chunk is fetched into registers while the current one is consumed, so its L2 latency is hidden;
    // two barriers per chunk swap it in.
    const int units_per_chunk = a.KC / kUnitCols;
    const int nchunks = (a.d + a.KC - 1) / a.KC;
    u32x4 hp[kMaxPieces];
    // piece e = q * 512 + tid of a chunk is (hidden row e / ppr, 16-byte piece e % ppr); one division per
    // chunk, then a carry per step
    auto fetch_chunk = [&](int c) {
        const int c0 = c * a.KC;
        const int ppr = min(a.KC, a.d - c0) >> 3;        // pieces per row
        const int step_r = (NW * kWave) / ppr, step_p = (NW * kWave) % ppr;
        int r = (int)threadIdx.x / ppr, pc = (int)threadIdx.x % ppr;
        const int s0 = c * (a.KC / kUnitCols);           // first step of the chunk
        const char *hbase = static_cast<const char *>(a.h);
#pragma unroll
        for (int q = 0; q < kMaxPieces; ++q) {
            hp[q] = u32x4{0u, 0u, 0u, 0u};
            // 16 pieces per unit: piece pc belongs to step s0 + pc / 16
            int ua = hstart + s0 + (pc >> 4);
            ua = ua >= nunits ? ua - nunits : ua;
            // few hidden rows may be picked out of a larger batch (their indices are packed in row_pack)
            const int hr = a.indexed ? (int)((a.row_pack >> (8 * (r & 7))) & 0xFFull) : r;
            const unsigned off = __umul24((unsigned)hr, (unsigned)(a.d * 2)) + (unsigned)ua * (kUnitCols * 2) + (unsigned)(pc & 15) * 16u;
            if (r < a.n) cached_load16(hp[q], off, hbase);
            r += step_r;
            pc += step_p;
            if (pc >= ppr) {
                pc -= ppr;
                ++r;
            }
        }
    };
    auto store_chunk = [&](int c) {
        const int ppr = min(a.KC, a.d - c * a.KC) >> 3;
        const int step_r = (NW * kWave) / ppr, step_p = (NW * kWave) % ppr;
        int r = (int)threadIdx.x / ppr, pc = (int)threadIdx.x % ppr;
#pragma unroll
        for (int q = 0; q < kMaxPieces; ++q) {
            if (r < hrows) *reinterpret_cast<u32x4 *>(hbuf + (size_t)r * a.hpitch + pc * 16) = hp[q];
            r += step_r;
            pc += step_p;
            if (pc >= ppr) {
                pc -= ppr;
                ++r;
            }
        }
    };
    // Target ids of the tile rows this lane ranks in the epilogue (two layouts, see below).  They are requested
    // by hand like everything else here and first of all: a load the compiler knows of would get a wait from
    // it wherever it sees fit, and since loads return in order any such wait also waits for the W prefetch.
    // (ids[2], up to 12 waves or a shared row group: the row lane + 128 of a tile of up to 192 rows)
    int ids[3];
    request_dword(ids[0], head_map + row0 + min(lane, rows_b - 1));
    request_dword(ids[1], head_map + row0 + min(lane + kWave, rows_b - 1));
    request_dword(ids[2], head_map + row0 + min(lane + 2 * kWave, rows_b - 1));
    // The first unit of W is asked for ahead of h, whose addresses take longer to form than its way takes from the L2 (k = 32768,
    // d = 2048, n = 1 25.3 -> 24.7 us, k = 5000, d = 3072, n = 1 12.9 -> 12.4, k = 8192, d = 2048, n = 8 13.5 -> 13.2; two units first
    // 25.1, 13.1 and 13.8, all three 25.3, 13.3 and 14.2) -- or behind it, see h_first().
    constexpr int kAhead = H_FIRST ? 0 : 1, kBehind = kPrefetchUnits - kAhead;
#pragma unroll
    for (int x = 0; x < kAhead; ++x) load_unit(x, areg[x]);
    fetch_chunk(0);                       // everything waits for it
#pragma unroll
    for (int x = kAhead; x < kPrefetchUnits; ++x) load_unit(x, areg[x]);
    wait_pieces<4 * kBehind>(hp);         // the other units stay in flight
    wait_ids<4 * kBehind>(ids);           // older than the chunk: they have landed too
    store_chunk(0);
    __syncthreads();
    const int id0 = ids[0], id1 = ids[1], id2 = ids[2];

    // Units are consumed in order; unit u sits in register slot u % kPrefetchUnits.  Between a hand-issued
    // load and its wait the compiler believes the registers already hold their data, so the order of loads
    // and waits must be the same on every path through the code, not only on those that the values of
    // u and c allow: the loop is written so that its shape alone guarantees it (a build step follows every
    // path of the compiled kernel and checks this).
    int u = 0;
    auto run_unit = [&](u32x4(&ar)[4], int uc) {
        // unit u's four loads are the oldest outstanding of the W stream
        wait_unit<4 * (kPrefetchUnits - 1)>(ar);
        unsigned char *sb = my_stage + (u & 1) * kStageUnitBytes;
#pragma unroll
        for (int j = 0; j < 4; ++j) *reinterpret_cast<u32x4 *>(sb + 4 * j * kStagePitch + wr_off) = ar[j];
        load_unit(u + kPrefetchUnits, ar);
        const unsigned char *hb = hbuf + hrow_off + (size_t)uc * (kUnitCols * 2);
        if (XG || rotate) {
            if (in_range == upr) {      // (XG: at u == nun this closes the last part of the wave's own rows)
                sums.close(acc, rot, closed);
                ++closed;
                in_range = 0;
            }
            ++in_range;
        }
        if constexpr (XG) {
            // own rows complete: their logits wait; the shared group's part starts from zero
            if (u == nun) own = sums.set[0][0] + sums.set[1][0];
            if (u >= nun) {
                // the shared group's unit w PL + (u - nun): where it lies in h's (rotated) layout in LDS
                int pos = w * PL + (u - nun) - hstart;
                pos = pos < 0 ? pos + nunits : pos;
                hb = hbuf + hrow_off + (size_t)pos * (kUnitCols * 2);
            }
        }
        // operands of two k-steps are read before their MFMAs are issued, so that the LDS latency is paid
        // once per pair and not once per MFMA
#pragma unroll
        for (int kp = 0; kp < 4; kp += 2) {
            u32x4 av[2], bv[2];
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                av[ks] = *reinterpret_cast<const u32x4 *>(sb + rd_off + (kp + ks) * 64);
                bv[ks] = *reinterpret_cast<const u32x4 *>(hb + (kp + ks) * 64);
            }
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
                acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av[ks]),
                                                                 __builtin_bit_cast(bf16x8, bv[ks]), acc[0], 0, 0, 0);
        }
        ++u;
    };
    // Chunks that have a successor hold a multiple of kPrefetchUnits units (the host plans them so): the
    // next chunk is requested, whole rounds of units run without any test in between, and by then every
    // piece of the next chunk has 4 * kPrefetchUnits younger loads behind it.
    for (int c = 0; c + 1 < nchunks; ++c) {
        fetch_chunk(c + 1);
        int uc = 0;
        do {
#pragma unroll
            for (int x = 0; x < kPrefetchUnits; ++x) run_unit(areg[x], uc++);
        } while (uc < units_per_chunk);
        wait_pieces<4 * kPrefetchUnits>(hp);
        __syncthreads();       // every wave is done with the current chunk
        store_chunk(c + 1);
        __syncthreads();
    }
    // the last chunk: any number of units -- whole rounds, then the one or two that remain
    {
        int uc = KS > 1 ? ustart : 0;      // position of the wave's first unit in h's LDS layout
        for (int rounds = (ntot - u) / kPrefetchUnits; rounds > 0; --rounds) {
#pragma unroll
            for (int x = 0; x < kPrefetchUnits; ++x) run_unit(areg[x], uc++);
        }
        static_assert(kPrefetchUnits == 3, "the remainder below is written for rounds of three");
        if (u < ntot) {
            run_unit(areg[0], uc++);
            if (u < ntot) run_unit(areg[1], uc++);
        }
    }
    // prefetches past the last unit are still in flight: let them land before their registers die
#pragma unroll
    for (int x = 0; x < kPrefetchUnits; ++x) wait_unit<0>(areg[x]);

    if constexpr (XG) {
        // acc[0]: the shared group's partial logits over this wave's column part; own: the own rows' logits
    } else if (rotate) {
        sums.close(acc, rot, closed);
        sums.total(acc);
    }

    // ---- logits of this tile -> LDS tile zt[i][t] (aliases staging and h)
    __syncthreads();
    const int tp = (XG ? kMfmaTileRows + 16 : MAXW == kStepWaves ? kMfmaTileRows : tile_rows) + 1;
    if (lrow < a.n) {                      // hidden row of this lane
        float *dst = zt + ((size_t)ksi * a.n + lrow) * tp + 16 * rg + 4 * lgrp;      // partial ksi of the row
        const f32x4 v = XG ? own : acc[0];
        dst[0] = v.x;
        dst[1] = v.y;
        dst[2] = v.z;
        dst[3] = v.w;
    }
    if constexpr (XG) {
        // the shared group: the eight waves' partials xq[part][hidden row][16] behind the tile and its candidate
        // keys, then the same tree as in the registers above
        float *xq = reinterpret_cast<float *>(smem + 8192 + kStepWaves * 3 * kWave * sizeof(unsigned long long));
        if (lrow < a.n) {
            float *dst = xq + ((size_t)w * a.n + lrow) * 16 + 4 * lgrp;
            dst[0] = acc[0].x;
            dst[1] = acc[0].y;
            dst[2] = acc[0].z;
            dst[3] = acc[0].w;
        }
        __syncthreads();
        const int e = (int)threadIdx.x;
        if (e < 16 * a.n) {
            const int i = e >> 4, r = e & 15;
            const float *x = xq + (size_t)i * 16 + r;
            const size_t ps = (size_t)a.n * 16;      // from one part to the next
            const float s01 = x[0] + x[ps], s23 = x[2 * ps] + x[3 * ps];
            const float s45 = x[4 * ps] + x[5 * ps], s67 = x[6 * ps] + x[7 * ps];
            zt[(size_t)i * tp + kMfmaTileRows + r] = (s01 + s23) + (s45 + s67);
        }
    }
    __syncthreads();

    if (a.zbuf != nullptr) {
        // store-only tail: the tile's logits go to z [n, k]; a workgroup per hidden row finishes the step
        // (row_select_kernel).  One wave copies a hidden row's 128 logits (512 contiguous bytes) at a time.
        const int per_tile = (tile_rows + kFewRowsPart - 1) / kFewRowsPart;
        for (int i = w; i < a.n; i += NW) {
            const float *src = zt + (size_t)i * tp;
            store_logits(a.zbuf + (size_t)i * a.zpitch + row0, a.parts != 0 ? a.pms + (size_t)i * a.parts + blockIdx.x * per_tile : nullptr, rows_b, lane,
                         [&](int t) { return src[t]; });
        }
        return;
    }

    {
        // a wave per hidden row (all of them at once for n <= 8); candidate keys of the threshold selection
        // sit behind the logit tile, 1 KiB per wave
        const size_t ztile = ((size_t)KS * a.n * tp * sizeof(float) + 15) & ~(size_t)15;
        constexpr int kCandPerWave = (MAXW > kStepWaves || XG) ? 3 * kWave : 2 * kWave;      // one key per tile row
        unsigned long long *cand =
            reinterpret_cast<unsigned long long *>(smem + (ztile > 8192 ? ztile : 8192)) + (size_t)w * kCandPerWave;
        const EpilogueShare share = epilogue_share(a.n, NW, w);
        for (int i = share.row; i < a.n; i += NW) {
            const float *zrow = zt + (size_t)i * tp;
            float *full = a.out_logp_full ? a.out_logp_full + (size_t)i * a.k + row0 : nullptr;
            unsigned long long *pms_slot = a.pms + (size_t)i * a.nlists + blockIdx.x;
            unsigned long long *pk_slot = a.pkeys + ((size_t)i * a.nlists + blockIdx.x) * a.L;
            if constexpr (MH) {
                // a hidden row of another head: nothing of this tile is its business -- an empty list, and a
                // (max, sum-exp) pair that adds nothing to any log-sum-exp
                if ((int)((mh.head_of_row >> (8 * i)) & 0xFFull) != hd) {
                    if (share.lse && lane == 0) publish_u64(pms_slot, (unsigned long long)__float_as_uint(-3.0e38f));
                    if (share.keys && lane < a.L) publish_u64(pk_slot + lane, kNoKey);
                    continue;
                }
            }
            // the logit is the sum of the KS partial tiles, in wave order
            if constexpr (MAXW > kStepWaves || XG) {
                const int idq3[3] = {id0, id1, id2};
                block_epilogue_core<3>(zrow, KS, a.n * tp, rows_b, a.L, idq3, full, pms_slot, pk_slot, lane, share, cand);
            } else {
                block_epilogue_small(zrow, KS, a.n * tp, rows_b, a.L, id0, id1, full, pms_slot, pk_slot, lane, share, cand);
            }
        }
    }
}

// The merge of one hidden row per workgroup with a tree level behind it: wave 0 merges the row (its results are
// written through to memory) and takes a ticket; the workgroup that draws the last ticket ranks all n * m
// candidates, reading the other rows' results with loads that bypass its caches.
// T threads: 128 when n * m <= 64, else 512 (the waves beyond the second only help with the ranking; with more
// threads the merging wave would not have the registers it needs).  BLOCK: all eight waves merge.
template <int T, bool BLOCK>
__global__ void __launch_bounds__(BLOCK ? kBlockMergeLaunch : T) step_finalize_tree_kernel(const FinalizeArgs f) {
    static_assert(!BLOCK || T == kBlockMergeThreads, "one workgroup size for the merge by eight waves");
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int s_last;
    __shared__ float s_lse;
    const int lane = lane_id();
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int i = blockIdx.x;
    bool merged = false;
    unsigned long long *stage = reinterpret_cast<unsigned long long *>(smem);
    if constexpr (BLOCK) {
        merged = merge_row_block(f, i, i, *reinterpret_cast<BlockMergeLds *>(smem), lane, w);
        wait_stores_done();
        __syncthreads();
    } else {
        finalize_row_pair(f, i, i, stage, &s_lse, lane, w);
    }
    if (w == 0) {
        if (BLOCK && !merged) finalize_row_alone(f, i, i, stage, lane);
        wait_stores_done();       // the row's results are written through: visible to whoever draws the last ticket
        if (lane == 0) {
            const unsigned v = __hip_atomic_fetch_add(f.ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const int last = v == (unsigned)(f.n - 1);
            if (last) __hip_atomic_store(f.ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_last = last;
        }
    }
    __syncthreads();
    if (!s_last || w >= T / kWave) return;      // (the ranking's barriers are met by the waves that are left)
    TreeArgs t;
    t.parent_cum = f.tree_cum;
    t.vals = f.out_logp;
    t.ids = f.out_ids;
    t.N = f.n * f.m;
    t.m = f.m;
    t.K = f.tree_K;
    t.index_order = 0;
    t.out_a = f.tree_parent;
    t.out_token = f.tree_token;
    t.out_score = f.tree_score;
    int N2 = kWave;
    while (N2 < t.N) N2 <<= 1;
    unsigned long long *keys = reinterpret_cast<unsigned long long *>(smem);
    unsigned *cnt = reinterpret_cast<unsigned *>(smem + (size_t)N2 * 8);
    int *wave_tot = reinterpret_cast<int *>(smem + (size_t)N2 * 12);
    tree_select_by_count<T, true>(t, N2, keys, cnt, wave_tot);
}

// The same for one or two hidden rows in one workgroup, two waves per row as in the merge without a level: the results meet in LDS,
// and nobody takes a ticket, waits for stores or reads other workgroups' results back (a level of n = 1, k = 5000, d = 3072, m = 8
// 14.0 -> 13.7 us, n = 2, m = 4 14.1 -> 13.4).  More rows' waves are in each other's way on one CU (n = 4, k = 5000, d = 1024 11.4 /
// 11.6, n = 8, k = 5000, d = 3072 15.9 / 16.3).
template <int T>
__global__ void __launch_bounds__(T) step_finalize_tree_few_kernel(const FinalizeArgs f, int stage_keys) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ float s_lse[T / (2 * kWave)], s_logp[T];
    __shared__ int s_ids[T];
    static_assert(T / (2 * kWave) * 64 <= T, "a thread per candidate: up to 64 tokens per row");
    __shared__ unsigned long long s_keys[T];
    __shared__ unsigned s_above[T];
    const int lane = lane_id(), tid = (int)threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int N = f.n * f.m;
    int N2 = kWave;
    while (N2 < N) N2 <<= 1;
    // (on its way while the rows are merged)
    const float parent = tid < N ? f.tree_cum[tid / f.m] : 0.f;
    s_above[tid] = 0u;
    constexpr int kRows = T / (2 * kWave);
    if (w < f.n) {
        auto lse_fn = [&]() {
            __syncthreads();
            return s_lse[w];
        };
        finalize_row(f.pkeys + (size_t)w * f.nlists * f.L, f.nlists, f.L, f.m, false, lse_fn, reinterpret_cast<unsigned long long *>(smem) + (size_t)w * stage_keys,
                     s_ids + w * f.m, s_logp + w * f.m, lane);
    } else {
        const int i = w - kRows;
        if (i >= 0 && i < f.n) {
            const float lse = row_lse(f.pms + (size_t)i * f.nlists, f.nlists, lane);
            if (lane == 0) {
                s_lse[i] = lse;
                f.lse_buf[i] = lse;
                if (f.out_lse) f.out_lse[i] = lse;
            }
        }
        __syncthreads();
    }
    __syncthreads();
    int id = 0;
    if (tid < N2) {
        unsigned long long key = kNoKey;
        if (tid < N) {
            id = s_ids[tid];
            const float logp = s_logp[tid];
            f.out_ids[tid] = id;
            f.out_logp[tid] = logp;
            key = make_key(__fadd_rn(parent, logp), tid);      // one fp32 addition
        }
        s_keys[tid] = key;
    }
    __syncthreads();
    // T / N2 threads share a candidate's scan
    const int c = tid & (N2 - 1), part = tid / N2, each = N2 * N2 / T;
    const unsigned long long mine = s_keys[c];
    unsigned above = 0;
    for (int j = part * each; j < (part + 1) * each; j += 4) {
        unsigned long long t[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) t[u] = s_keys[j + u];
#pragma unroll
        for (int u = 0; u < 4; ++u) above += t[u] > mine ? 1u : 0u;
    }
    if (N2 < T) {
        if (above != 0u) atomicAdd(&s_above[c], above);
        __syncthreads();
        above = s_above[c];
    }
    if (tid < N && (int)above < f.tree_K) {
        f.tree_parent[above] = tid / f.m;
        f.tree_token[above] = id;
        f.tree_score[above] = key_logit(mine);
    }
}

// Merges the per-tile partials, many lists of them: eight waves per hidden row.
__global__ void __launch_bounds__(kBlockMergeLaunch) step_finalize_block_kernel(const FinalizeArgs f) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = lane_id();
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int i = blockIdx.x;
    const int o = f.indexed ? (int)((f.row_pack >> (8 * (i & 7))) & 0xFFull) : i;      // output row
    if (merge_row_block(f, i, o, *reinterpret_cast<BlockMergeLds *>(smem), lane, w) || w != 0) return;
    finalize_row_alone(f, i, o, reinterpret_cast<unsigned long long *>(smem), lane);
}

// Merges the per-tile partials: one wave per hidden row, beside one for its log-sum-exp.
__global__ void __launch_bounds__(2 * kWave) step_finalize_kernel(const FinalizeArgs f) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ float s_lse;
    const int i = blockIdx.x;
    const int o = f.indexed ? (int)((f.row_pack >> (8 * (i & 7))) & 0xFFull) : i;      // output row
    finalize_row_pair(f, i, o, reinterpret_cast<unsigned long long *>(smem), &s_lse, lane_id(),
                      __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)));
}

constexpr int kTreeFewLds = kMaxDynamicLds - 8 * 1024;      // (the kernel's own arrays beside it)

template <int MAXW, bool XG = false, bool H_FIRST = false>
hipError_t launch_mfma_inst(const MfmaArgs &a, size_t lds, hipStream_t st) {
    auto kern = head_mfma_kernel<MAXW, XG, false, H_FIRST>;
    static LdsLimitOnce lds_limit;
    hipError_t e = allow_dynamic_lds(lds_limit, {reinterpret_cast<const void *>(kern)}, kMaxDynamicLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(a.nlists), dim3((MAXW == kStepWaves ? kStepWaves : a.nwaves) * kWave), lds, st, a,
                       SingleHead{});
    return hipGetLastError();
}
// Four waves to a group of 16 rows have so little of W each that they wait for h, and for the more of it the longer: h first (W's first unit
// first / h first: n = 8, d = 4096, k = 3329 14.57 / 14.27 us, k = 5000 15.14 / 14.89, k = 6500 16.11 / 15.95, k = 8192 a tie, n = 8, d = 3072, k = 5000
// 13.95 / 13.74, n = 6 13.54 / 13.40, k = 6500 -0.5 %; n = 8, d = 2048 and n = 5, d = 4096 -0.3 and -0.6 %).
bool h_first(const MfmaArgs &a) {
    return a.ksplit == 4 && a.nwaves == kStepWaves && a.n >= 6 && a.n * a.d > 16384 && a.nlists <= (a.n == 8 ? 208 : 160);
}
template <int MAXW>
hipError_t launch_mfma_multi_inst(const MfmaArgs &a, const MultiHeadTable &t, size_t lds, hipStream_t st) {
    auto kern = head_mfma_kernel<MAXW, false, true>;
    static LdsLimitOnce lds_limit;
    hipError_t e = allow_dynamic_lds(lds_limit, {reinterpret_cast<const void *>(kern)}, kMaxDynamicLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(a.nlists), dim3((MAXW == kStepWaves ? kStepWaves : a.nwaves) * kWave), lds, st, a, t);
    return hipGetLastError();
}

}  // namespace

size_t mfma_stage_bytes(int nwaves) { return (size_t)nwaves * 2 * kStageUnitBytes; }

hipError_t launch_head_mfma(const MfmaArgs &a, size_t lds, hipStream_t st) {
    // a chunk of h that has a successor is run in whole rounds of units
    if (a.n < 1 || a.n > 8 || a.KC <= 0 || a.KC % kUnitCols != 0 || (a.KC < a.d && (a.KC / kUnitCols) % kPrefetchUnits != 0))
        return hipErrorInvalidValue;
    // the column split needs one chunk, whole units per wave and the fused epilogue
    if (a.ksplit != 1 &&
        ((a.ksplit != 2 && a.ksplit != 4) || a.KC < a.d || (a.d / kUnitCols) % a.ksplit != 0 || a.zbuf != nullptr))
        return hipErrorInvalidValue;
    // waves per workgroup: eight, or (all of h in LDS) a multiple of the column split up to kMfmaMaxWaves
    if (a.nwaves != kStepWaves &&
        (a.KC < a.d || a.nwaves < a.ksplit || a.nwaves > kMfmaMaxWaves || a.nwaves % a.ksplit != 0 ||
         (size_t)a.d * 16 > (size_t)kMaxPieces * a.nwaves * kWave * 16))
        return hipErrorInvalidValue;
    // rows past the 128th as one more group shared by the eight waves: eight column parts of whole units, all of h in LDS
    if (a.extra_rows != 0 && (a.extra_rows < 1 || a.extra_rows > 16 || a.KC < a.d || a.ksplit != 1 || a.nwaves != kStepWaves ||
                              (a.d / kUnitCols) % 8 != 0))
        return hipErrorInvalidValue;
    {
        const int tile_rows = 16 * (a.nwaves / a.ksplit) + a.extra_rows;
        if (a.nlists != (a.k + tile_rows - 1) / tile_rows) return hipErrorInvalidValue;
    }
    if ((size_t)a.d * 2 >= ((size_t)1 << 24)) return hipErrorInvalidValue;      // row offsets inside a tile: 24-bit factors
    if (a.extra_rows != 0) return launch_mfma_inst<kStepWaves, true>(a, lds, st);
    if (h_first(a)) return launch_mfma_inst<kStepWaves, false, true>(a, lds, st);
    return a.nwaves == kStepWaves ? launch_mfma_inst<kStepWaves>(a, lds, st) : launch_mfma_inst<kMfmaMaxWaves>(a, lds, st);
}

hipError_t launch_head_mfma_multi(const MfmaArgs &a, const MultiHeadTable &t, size_t lds, hipStream_t st) {
    // up to 8 hidden rows in place, all of h in LDS, plain tiles (a column split only with eight waves), the kernel's
    // own epilogue; every head cut into tiles of the launch's height on its own
    if (a.n < 1 || a.n > 8 || a.KC != a.d || a.indexed != 0 || a.zbuf != nullptr || a.out_logp_full != nullptr ||
        a.extra_rows != 0 || a.ticket_clear != nullptr || a.d % kUnitCols != 0 || a.L < 1 || a.L > 16 ||
        a.nwaves < kStepWaves || a.nwaves > kMfmaMaxWaves || (a.ksplit != 1 && (a.nwaves != kStepWaves || (a.ksplit != 2 && a.ksplit != 4))) ||
        (a.d / kUnitCols) % a.ksplit != 0 || (size_t)a.d * 16 > (size_t)kMaxPieces * a.nwaves * kWave * 16 ||
        (size_t)a.d * 2 >= ((size_t)1 << 24) || t.n_heads < 1 || t.n_heads > 16 || t.tile_first[0] != 0)
        return hipErrorInvalidValue;
    const int tile_rows = 16 * (a.nwaves / a.ksplit);
    for (int q = 0; q < t.n_heads; ++q) {
        if (t.W[q] == nullptr || t.map[q] == nullptr || t.k[q] < 1 ||
            t.tile_first[q + 1] - t.tile_first[q] != (t.k[q] + tile_rows - 1) / tile_rows)
            return hipErrorInvalidValue;
    }
    for (int i = 0; i < a.n; ++i)
        if ((int)((t.head_of_row >> (8 * i)) & 0xFFull) >= t.n_heads) return hipErrorInvalidValue;
    if (a.nlists != t.tile_first[t.n_heads] || a.nlists > kStepMaxBlocks) return hipErrorInvalidValue;
    return a.nwaves == kStepWaves ? launch_mfma_multi_inst<kStepWaves>(a, t, lds, st)
                                  : launch_mfma_multi_inst<kMfmaMaxWaves>(a, t, lds, st);
}

hipError_t launch_step_finalize(const FinalizeArgs &f, size_t lds, hipStream_t st) {
    static LdsLimitOnce lds_limit;
    hipError_t e = allow_dynamic_lds(lds_limit,
                                     {reinterpret_cast<const void *>(step_finalize_kernel),
                                      reinterpret_cast<const void *>(step_finalize_block_kernel),
                                      reinterpret_cast<const void *>(step_finalize_tree_kernel<128, false>),
                                      reinterpret_cast<const void *>(step_finalize_tree_kernel<512, false>),
                                      reinterpret_cast<const void *>(step_finalize_tree_kernel<512, true>)},
                                     kMaxDynamicLds);
    if (e != hipSuccess) return e;
    static LdsLimitOnce few_limit;
    e = allow_dynamic_lds(few_limit,
                          {reinterpret_cast<const void *>(step_finalize_tree_few_kernel<128>),
                           reinterpret_cast<const void *>(step_finalize_tree_few_kernel<256>)}, kTreeFewLds);
    if (e != hipSuccess) return e;
    const bool block = block_merge_pays(f.n, f.nlists, f.L, f.m);
    lds += kDirectPad * sizeof(unsigned long long);
    if (block && lds < sizeof(BlockMergeLds)) lds = sizeof(BlockMergeLds);
    if (f.tree_cum != nullptr) {
        // one hidden row per workgroup; LDS: the merge's staging, then the ranking's keys and counters
        const int N = f.n * f.m;
        if (f.indexed || N > kFinalizeTreeMaxN || f.ticket == nullptr) return hipErrorInvalidValue;
        if (!block && f.n <= 2 && f.n * lds <= (size_t)kTreeFewLds) {
            const int stage_keys = (int)(lds / sizeof(unsigned long long));
            if (f.n == 1)
                hipLaunchKernelGGL(step_finalize_tree_few_kernel<128>, dim3(1), dim3(128), lds, st, f, stage_keys);
            else
                hipLaunchKernelGGL(step_finalize_tree_few_kernel<256>, dim3(1), dim3(256), 2 * lds, st, f, stage_keys);
            return hipGetLastError();
        }
        int N2 = kWave;
        while (N2 < N) N2 <<= 1;
        const size_t need = (size_t)N2 * 12 + 256;
        const size_t bytes = lds > need ? lds : need;
        if (block)
            hipLaunchKernelGGL((step_finalize_tree_kernel<512, true>), dim3(f.n), dim3(kBlockMergeLaunch), bytes, st, f);
        else if (N <= kWave)
            hipLaunchKernelGGL((step_finalize_tree_kernel<128, false>), dim3(f.n), dim3(128), bytes, st, f);
        else
            hipLaunchKernelGGL((step_finalize_tree_kernel<512, false>), dim3(f.n), dim3(512), bytes, st, f);
        return hipGetLastError();
    }
    if (block) {
        hipLaunchKernelGGL(step_finalize_block_kernel, dim3(f.n), dim3(kBlockMergeLaunch), lds, st, f);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(step_finalize_kernel, dim3(f.n), dim3(2 * kWave), lds, st, f);
    return hipGetLastError();
}

}  // namespace vt
