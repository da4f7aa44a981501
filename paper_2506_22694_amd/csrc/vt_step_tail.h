// Tail of the draft step, shared by its kernels: per-workgroup epilogue
// (log-sum-exp partial + best candidates of a tile of logits), publication,
// election of the last workgroup, and the final cross-workgroup merge
// (lse, top-m, remap to target ids).
#pragma once
#include <type_traits>
#include "vt_device.h"
#include "vt_step.h"

namespace vt {

// ------------------------------------------------------------------ top-L of a wave's candidates
// Every lane holds Q candidates: ord[q] = orderable logit (0 = none), id[q] =
// target id.  L rounds; round r finds the best remaining candidate of the whole
// wave under (logit desc, id asc) and parks it in lane r.  Returns lane r's key.
template <int Q>
__device__ __forceinline__ unsigned long long wave_select_top(unsigned (&ord)[Q], int (&id)[Q], int L, int lane) {
    unsigned res_ord = 0u;
    unsigned res_id = 0u;
    for (int r = 0; r < L; ++r) {
        unsigned bo = ord[0];
#pragma unroll
        for (int q = 1; q < Q; ++q) bo = ord[q] > bo ? ord[q] : bo;
        const unsigned wmax = wave_max_u32(bo);
        unsigned myid = 0xFFFFFFFFu;
        int cnt = 0;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if (ord[q] == wmax) {
                myid = (unsigned)id[q] < myid ? (unsigned)id[q] : myid;
                ++cnt;
            }
        }
        // exact ties are rare: one holder -> read its id; otherwise reduce for the lowest id
        const unsigned long long holders = __ballot(cnt > 0);
        const unsigned long long multi = __ballot(cnt > 1);
        unsigned wid;
        if (__popcll(holders) == 1 && multi == 0ull) {
            wid = __builtin_amdgcn_readlane(myid, __ffsll((long long)holders) - 1);
        } else {
            wid = wave_min_u32(myid);
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if (ord[q] == wmax && (unsigned)id[q] == wid) ord[q] = 0u;
        }
        if (lane == r) {
            res_ord = wmax;
            res_id = wid;
        }
    }
    return res_ord == 0u ? kNoKey : (((unsigned long long)res_ord << 32) | (unsigned)(~res_id));
}

template <bool NEIGHBOURS>
__device__ __forceinline__ unsigned wave_min_of_group_max_u32(unsigned v, int gsteps);

// The largest value P << 16 such that at least `kth` lanes hold v >= P << 16 (0 if fewer than kth lanes hold anything
// but 0): the upper half of the kth largest v, selected one bit at a time.  All 64 lanes take part.
__device__ __forceinline__ unsigned wave_kth_largest_prefix16(unsigned v, int kth) {
    unsigned T = 0u;
    unsigned long long alive = ~0ull;
    int need = kth;
#pragma unroll
    for (int b = 31; b >= 16; --b) {
        const unsigned long long ones = __ballot((v >> b) & 1u) & alive;
        const int c = __popcll(ones);
        if (c >= need) {
            alive = ones;
            T |= 1u << b;
        } else {
            need -= c;
            alive &= ~ones;
        }
    }
    return T;
}

// ------------------------------------------------------------------ top-L of a wave's candidates, by threshold
// Two candidates per lane (ord = 0: none).  With G = the power of two >= L the lanes form G groups; every
// group's best logit is a different candidate, so at least L candidates reach T = the smallest group maximum
// and the L best are among those that do (about 2 L of 128).  They are compacted into `cand` (wave-private
// LDS, 128 keys) and each finds its rank by counting: no L dependent selection rounds.  Rank r < L is
// published at slot r; slots past the number of candidates get the "no key" value.
__device__ __forceinline__ void wave_publish_top_by_threshold(const unsigned (&ord)[2], const int (&id)[2], int L,
                                                              unsigned long long *cand,
                                                              unsigned long long *__restrict__ pkeys_slot, int lane) {
    const unsigned top = ord[0] > ord[1] ? ord[0] : ord[1];
    unsigned T;
    if (L <= 8) {
        int gsteps = 6;
        while ((kWave >> gsteps) < L) --gsteps;
        T = wave_min_of_group_max_u32<false>(top, gsteps);
    } else {
        T = wave_kth_largest_prefix16(top, L);      // (16 or more groups would pass several times L candidates)
    }
    T = T == 0u ? 1u : T;               // a group without candidates: every real candidate passes
    const bool c0 = ord[0] >= T, c1 = ord[1] >= T;
    const unsigned long long m0 = __ballot(c0), m1 = __ballot(c1);
    const int n0 = __popcll(m0);
    const int ncand = n0 + __popcll(m1);
    const unsigned long long k0 = ((unsigned long long)ord[0] << 32) | (unsigned)(~(unsigned)id[0]);
    const unsigned long long k1 = ((unsigned long long)ord[1] << 32) | (unsigned)(~(unsigned)id[1]);
    if (c0) cand[__builtin_amdgcn_mbcnt_hi((unsigned)(m0 >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m0, 0u))] = k0;
    if (c1)
        cand[n0 + __builtin_amdgcn_mbcnt_hi((unsigned)(m1 >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m1, 0u))] = k1;
    // (the ranking reads eight keys at a time; with all 128 taken there is nothing to fill)
    if (lane < 8 && ncand + lane < 2 * kWave) cand[ncand + lane] = kNoKey;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (c0 || c1) {
        int a0 = 0, a1 = 0;
        for (int x = 0; x < ncand; x += 8) {
            unsigned long long t[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) t[q] = cand[x + q];       // every lane reads the same key: a broadcast
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                a0 += t[q] > k0 ? 1 : 0;
                a1 += t[q] > k1 ? 1 : 0;
            }
        }
        if (c0 && a0 < L) publish_u64(pkeys_slot + a0, k0);
        if (c1 && a1 < L) publish_u64(pkeys_slot + a1, k1);
    }
    if (lane < L && lane >= ncand) publish_u64(pkeys_slot + lane, kNoKey);
    __builtin_amdgcn_wave_barrier();     // the next row of this wave reuses cand
}

// The same for Q candidates per lane (tiles of more than 128 rows); `cap` keys (a multiple of eight) fit `cand`, Q * 64 where that is less.  Returns false,
// having published nothing, when more than `cap` candidates reach the threshold.
constexpr int kLargeTileCandCap = 256;
template <int Q>
__device__ __forceinline__ bool wave_publish_top_by_threshold_q(const unsigned (&ord)[Q], const int (&id)[Q], int L,
                                                                unsigned long long *cand, int cap,
                                                                unsigned long long *__restrict__ pkeys_slot,
                                                                int lane) {
    unsigned top = ord[0];
#pragma unroll
    for (int q = 1; q < Q; ++q) top = ord[q] > top ? ord[q] : top;
    unsigned T;
    if (L <= 8) {
        int gsteps = 6;
        while ((kWave >> gsteps) < L) --gsteps;
        T = wave_min_of_group_max_u32<false>(top, gsteps);
    } else {
        T = wave_kth_largest_prefix16(top, L);
    }
    T = T == 0u ? 1u : T;
    int ncand = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const bool c = ord[q] >= T;
        const unsigned long long mask = __ballot(c);
        if (mask != 0ull) {
            const int slot = ncand + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32),
                                                                    __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
            if (c && slot < cap) cand[slot] = ((unsigned long long)ord[q] << 32) | (unsigned)(~(unsigned)id[q]);
            ncand += __popcll(mask);
        }
    }
    if (ncand > cap) return false;
    // (the ranking reads eight keys at a time; a list of all Q * 64 keys needs no filling)
    if (lane < 8 && ncand + lane < min(cap, Q * kWave)) cand[ncand + lane] = kNoKey;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (int c = lane; c < ncand; c += kWave) {
        const unsigned long long key = cand[c];
        int above = 0;
        for (int x = 0; x < ncand; x += 8) {
            unsigned long long t[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) t[q] = cand[x + q];
#pragma unroll
            for (int q = 0; q < 8; ++q) above += t[q] > key ? 1 : 0;
        }
        if (above < L) publish_u64(pkeys_slot + above, key);
    }
    if (lane < L && lane >= ncand) publish_u64(pkeys_slot + lane, kNoKey);
    __builtin_amdgcn_wave_barrier();     // the next row of this wave reuses cand
    return true;
}

// ------------------------------------------------------------------ workgroup epilogue of one hidden row
// zrow: the row's logit tile in LDS (S partial sums per logit, `sstride` floats
// apart).  Publishes (max, sum-exp) and the L best keys of this workgroup.
// QMAX*64 >= rows_b.  idq: target ids of tile rows lane + 64*q.
// What bounds it: about 1.7 us of dependent LDS round trips and reductions after the stream's last load, not arithmetic
// (run twice, the second time takes as long).  Where a workgroup has two waves per hidden row, one does the keys and the
// other (max, sum-exp); the partial sums are read in one go; the keys are ranked in whole groups of eight.  Together:
// 4 x 1024 x 256 in fp32 10.2 -> 9.7 us, a round on 5000 x 3072 57.9 -> 55.7,
// n = 8 on 128256 x 3072 125.0 -> 123.8, two heads 43.2 -> 42.9, n = 1 on 32768 x 2048 a tie.
struct EpilogueShare {
    int row;           // the wave's first hidden row, >= n: none; the next ones follow a workgroup's waves apart
    bool keys, lse;
};
__device__ __forceinline__ EpilogueShare epilogue_share(int n, int waves, int w) {
    if (2 * n > waves) return EpilogueShare{w, true, true};
    return w < 2 * n ? EpilogueShare{w < n ? w : w - n, w < n, w >= n} : EpilogueShare{n, false, false};
}
template <int QMAX>
__device__ __forceinline__ void block_epilogue_core(const float *zrow, int S, int sstride, int rows_b, int L,
                                                    const int (&idq)[QMAX], float *__restrict__ logp_full_row,
                                                    unsigned long long *__restrict__ pms_slot,
                                                    unsigned long long *__restrict__ pkeys_slot, int lane, const EpilogueShare &share,
                                                    unsigned long long *cand = nullptr) {
    unsigned ord[QMAX];
    int id[QMAX];
    float zq[QMAX];
    float lmax = -INFINITY;
    // the sum over the partial logits in ascending order; every lane reads -- past the tile's end its last logit again -- and
    // all reads of a round are made before the first is used (one after the other they took 0.4 us with four partials)
    constexpr int kParts = QMAX <= 4 ? 4 : 1;
#pragma unroll
    for (int q = 0; q < QMAX; ++q) zq[q] = 0.f;
    for (int s0 = 0; s0 < S; s0 += kParts) {
        float part[kParts][QMAX];
#pragma unroll
        for (int s = 0; s < kParts; ++s) {
#pragma unroll
            for (int q = 0; q < QMAX; ++q) part[s][q] = zrow[(size_t)min(s0 + s, S - 1) * sstride + min(lane + q * kWave, rows_b - 1)];
        }
#pragma unroll
        for (int s = 0; s < kParts; ++s) {
#pragma unroll
            for (int q = 0; q < QMAX; ++q) zq[q] = s0 + s < S ? zq[q] + part[s][q] : zq[q];
        }
    }
#pragma unroll
    for (int q = 0; q < QMAX; ++q) {
        const bool ok = lane + q * kWave < rows_b;
        if (logp_full_row != nullptr && share.keys && ok) logp_full_row[lane + q * kWave] = zq[q];
        id[q] = idq[q];
        ord[q] = ok ? orderable_f32(zq[q]) : 0u;
        zq[q] = ok ? zq[q] : -INFINITY;
        lmax = fmaxf(lmax, zq[q]);
    }
    if (share.lse) {
        const float M = wave_max(lmax);
        float ls = 0.f;
#pragma unroll
        for (int q = 0; q < QMAX; ++q) ls += __expf(zq[q] - M);   // exp(-inf) = 0 for absent rows
        const float Ssum = wave_sum(ls);
        if (lane == 0)
            publish_u64(pms_slot, ((unsigned long long)__float_as_uint(Ssum) << 32) | __float_as_uint(M));
    }
    if (!share.keys) return;
    bool published = false;
    if constexpr (QMAX == 2) {
        if (cand != nullptr && L >= 5) {       // up to four rounds are no slower than the threshold (measured)
            wave_publish_top_by_threshold(ord, id, L, cand, pkeys_slot, lane);
            published = true;
        }
    } else {
        if (cand != nullptr && L >= 3 && L <= kWave)
            published = wave_publish_top_by_threshold_q<QMAX>(ord, id, L, cand, kLargeTileCandCap, pkeys_slot, lane);
    }
    if (!published) {
        const unsigned long long key = wave_select_top<QMAX>(ord, id, L, lane);
        if (lane < L) publish_u64(pkeys_slot + lane, key);
    }
}

// small tiles (<= 128 rows): ids were prefetched by the caller
__device__ __forceinline__ void block_epilogue_small(const float *zrow, int S, int sstride, int rows_b, int L, int id0,
                                                  int id1, float *__restrict__ logp_full_row,
                                                  unsigned long long *__restrict__ pms_slot,
                                                  unsigned long long *__restrict__ pkeys_slot, int lane, const EpilogueShare &share,
                                                  unsigned long long *cand = nullptr) {
    const int idq[2] = {id0, id1};
    block_epilogue_core<2>(zrow, S, sstride, rows_b, L, idq, logp_full_row, pms_slot, pkeys_slot, lane, share, cand);
}

// large tiles (<= 1024 rows): ids are read here; QMAX logits per lane, sized to the tile (4, 8 or 16)
template <int QMAX>
__device__ __forceinline__ void block_epilogue_large_q(const float *zrow, int S, int sstride, int rows_b, int L,
                                                       const int *__restrict__ map_tile,
                                                       float *__restrict__ logp_full_row,
                                                       unsigned long long *__restrict__ pms_slot,
                                                       unsigned long long *__restrict__ pkeys_slot, int lane, const EpilogueShare &share,
                                                       unsigned long long *cand) {
    int idq[QMAX];
#pragma unroll
    for (int q = 0; q < QMAX; ++q) idq[q] = map_tile[min(lane + q * kWave, rows_b - 1)];
    block_epilogue_core<QMAX>(zrow, S, sstride, rows_b, L, idq, logp_full_row, pms_slot, pkeys_slot, lane, share, cand);
}
__device__ __forceinline__ void block_epilogue_large(const float *zrow, int S, int sstride, int rows_b, int L,
                                                  const int *__restrict__ map_tile,
                                                  float *__restrict__ logp_full_row,
                                                  unsigned long long *__restrict__ pms_slot,
                                                  unsigned long long *__restrict__ pkeys_slot, int lane, const EpilogueShare &share,
                                                  unsigned long long *cand = nullptr) {
    if (rows_b <= 4 * kWave)
        block_epilogue_large_q<4>(zrow, S, sstride, rows_b, L, map_tile, logp_full_row, pms_slot, pkeys_slot, lane, share, cand);
    else if (rows_b <= 8 * kWave)
        block_epilogue_large_q<8>(zrow, S, sstride, rows_b, L, map_tile, logp_full_row, pms_slot, pkeys_slot, lane, share, cand);
    else
        block_epilogue_large_q<kStepMaxRowsPerBlock / kWave>(zrow, S, sstride, rows_b, L, map_tile, logp_full_row,
                                                             pms_slot, pkeys_slot, lane, share, cand);
}

// --------------------------------------------------------------------- logits of a tile to memory
// One wave stores a hidden row's logits of this tile (up to 8 hidden rows), and beside them, unless pms is null, the (max, sum-exp)
// of every 64 of them, by which row_select_kernel finds the parts it reads (of logits that are all -inf NaN, see there).
static_assert(kFewRowsPart == kWave);
template <typename Logit>
__device__ __forceinline__ void store_logits(float *__restrict__ z, unsigned long long *__restrict__ pms, int rows_b, int lane, Logit logit) {
    for (int t0 = 0; t0 < rows_b; t0 += kWave) {
        const int t = t0 + lane;
        float v = -INFINITY;
        if (t < rows_b) z[t] = v = logit(t);
        if (pms != nullptr) {
            const float top = wave_max(v), sum = wave_sum(__expf(v - top));
            if (lane == 0) pms[t0 / kWave] = ((unsigned long long)__float_as_uint(sum) << 32) | __float_as_uint(top);
        }
    }
}

// ------------------------------------------------------------------ four hidden rows per pass
// Tiles of at most 16 Q logits per hidden row (Q = 8: 128 rows, Q = 9: 144) and L <= 16: the 16 lanes of DPP row g
// rank hidden row i0 + g (Q logits per lane), so a wave finishes four hidden rows in
// the time of one.  zt: logit tile [hidden row][tp]; idq: ids of tile rows gl + 16 q.
template <int Q>
__device__ __forceinline__ void block_epilogue_rows4(const float *zt, int tp, int i0, int n, int rows_b, int L,
                                                     const int (&idq)[Q], float *__restrict__ logp_full, size_t k,
                                                     int row0, unsigned long long *__restrict__ pms,
                                                     unsigned long long *__restrict__ pkeys, int nlists, int blk,
                                                     int lane, unsigned long long *cand) {
    const int g = lane >> 4, gl = lane & 15;
    const int i = i0 + g;
    const bool active = i < n;
    const float *zrow = zt + (size_t)(active ? i : 0) * tp;
    unsigned ord[Q];
    int id[Q];
    float zq[Q];
    float lmax = -INFINITY;
    // every lane reads -- past the tile's end its last logit again -- and selects afterwards: no branch per logit
    // (a third of the instructions of a pass were those branches)
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int t = gl + 16 * q;
        const bool ok = active && t < rows_b;
        const float z = zrow[min(t, rows_b - 1)];
        id[q] = idq[q];
        zq[q] = ok ? z : -INFINITY;
        ord[q] = ok ? orderable_f32(z) : 0u;
        lmax = fmaxf(lmax, zq[q]);
    }
    if (logp_full != nullptr) {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int t = gl + 16 * q;
            if (active && t < rows_b) logp_full[(size_t)i * k + row0 + t] = zq[q];
        }
    }
    const float M = __uint_as_float(row16_allreduce_u32(__float_as_uint(lmax), OpMaxF32{}));
    float ls = 0.f;
#pragma unroll
    for (int q = 0; q < Q; ++q) ls += __expf(zq[q] - M);
    const float Ssum = __uint_as_float(row16_allreduce_u32(__float_as_uint(ls), OpAddF32{}));
    if (active && gl == 0)
        publish_u64(pms + (size_t)i * nlists + blk,
                    ((unsigned long long)__float_as_uint(Ssum) << 32) | __float_as_uint(M));
    if (L <= 8) {
        // Selection by threshold: T = the L-th largest of the 16 lanes' best logits, so at least L logits reach
        // it and the L best of the row are among those that do -- about L + 2 of the 128.  They are compacted
        // into 16 keys of LDS per row and each finds its rank by counting: no L dependent rounds.  More than 16
        // candidates in any row of the wave (3 in 1000 rows): the second form; more than 32 (many equal logits): the rounds.
        unsigned bo = ord[0];
#pragma unroll
        for (int q = 1; q < Q; ++q) bo = ord[q] > bo ? ord[q] : bo;
        const int above = row16_count_greater(bo);      // lanes of the row with a strictly better best logit
        // the smallest best logit that fewer than L others beat is the L-th largest
        unsigned T = row16_allreduce_u32(above < L ? bo : 0xFFFFFFFFu, OpMinU32{});
        T = T == 0u ? 1u : T;   // fewer than L lanes have logits at all: every logit is a candidate
        int cnt = 0;
#pragma unroll
        for (int q = 0; q < Q; ++q) cnt += ord[q] >= T ? 1 : 0;
        unsigned incl = (unsigned)cnt;
        incl += dpp_mov<0x111>(incl);       // row_shr:1 (lanes without a source read 0)
        incl += dpp_mov<0x112>(incl);       // row_shr:2
        incl += dpp_mov<0x114>(incl);       // row_shr:4
        incl += dpp_mov<0x118>(incl);       // row_shr:8
        const int total = (int)row16_allreduce_u32(incl, OpMaxU32{});
        if (__ballot(total > 16) == 0ull) {
            unsigned long long *crow = cand + 16 * g;
            crow[gl] = kNoKey;              // below every candidate: unused slots count for nothing
            int pos = (int)incl - cnt;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                if (ord[q] >= T) crow[pos++] = ((unsigned long long)ord[q] << 32) | (unsigned)(~(unsigned)id[q]);
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const unsigned long long mine = crow[gl];
            int rank = 0;
#pragma unroll
            for (int x = 0; x < 16; ++x) rank += crow[x] > mine ? 1 : 0;
            if (active) {
                unsigned long long *slot = pkeys + ((size_t)i * nlists + blk) * L;
                if (gl < total && rank < L) publish_u64(slot + rank, mine);
                if (gl < L && gl >= total) publish_u64(slot + gl, kNoKey);
            }
            __builtin_amdgcn_wave_barrier();     // the wave's next rows reuse cand
            return;
        }
        // 17 to 32 in a row: two rows after each other have 32 slots each, a lane ranks two keys.  (A tile of 64 hidden
        // rows meets one such row in five times, so some tile of every launch does, and the launch ends with the last tile.)
        if (__ballot(total > 32) == 0ull) {
            unsigned long long *crow = cand + 32 * (g & 1);
            const unsigned long long *cr = crow;
            for (int half = 0; half < 2; ++half) {
                const bool turn = (g >> 1) == half;
                if (turn) {
                    crow[gl] = kNoKey;
                    crow[gl + 16] = kNoKey;
                    int pos = (int)incl - cnt;
#pragma unroll
                    for (int q = 0; q < Q; ++q) {
                        if (ord[q] >= T) crow[pos++] = ((unsigned long long)ord[q] << 32) | (unsigned)(~(unsigned)id[q]);
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                const unsigned long long k0 = cr[gl], k1 = cr[gl + 16];
                int r0 = 0, r1 = 0;
#pragma unroll 8
                for (int x = 0; x < 32; ++x) {
                    const unsigned long long t = cr[x];
                    r0 += t > k0 ? 1 : 0;
                    r1 += t > k1 ? 1 : 0;
                }
                if (turn && active) {
                    unsigned long long *slot = pkeys + ((size_t)i * nlists + blk) * L;
                    if (gl < total && r0 < L) publish_u64(slot + r0, k0);
                    if (gl + 16 < total && r1 < L) publish_u64(slot + r1, k1);
                    if (gl < L && gl >= total) publish_u64(slot + gl, kNoKey);
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();     // the next two rows, or the wave's next four, reuse cand
            }
            return;
        }
    }
    unsigned res_ord = 0u, res_id = 0u;
    for (int r = 0; r < L; ++r) {
        unsigned bo = ord[0];
#pragma unroll
        for (int q = 1; q < Q; ++q) bo = ord[q] > bo ? ord[q] : bo;
        const unsigned wmax = row16_allreduce_u32(bo, OpMaxU32{});
        unsigned myid = 0xFFFFFFFFu;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if (ord[q] == wmax) myid = (unsigned)id[q] < myid ? (unsigned)id[q] : myid;
        }
        const unsigned wid = row16_allreduce_u32(myid, OpMinU32{});
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if (ord[q] == wmax && (unsigned)id[q] == wid) ord[q] = 0u;
        }
        if (gl == r) {
            res_ord = wmax;
            res_id = wid;
        }
    }
    if (active) {
        const unsigned long long key =
            res_ord == 0u ? kNoKey : (((unsigned long long)res_ord << 32) | (unsigned)(~res_id));
        if (gl < L) publish_u64(pkeys + ((size_t)i * nlists + blk) * L + gl, key);
    }
}

// A row's results are written through to memory (relaxed agent-scope stores, like the partials): a tree level
// fused behind the merge reads them from another workgroup, possibly on another XCD, whose L2 would not see a
// line that is still dirty in this one's.
__device__ __forceinline__ void store_result(int *__restrict__ ids_row, float *__restrict__ logp_row, int slot, int id,
                                             float logp) {
    __hip_atomic_store(ids_row + slot, id, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(reinterpret_cast<unsigned *>(logp_row) + slot, __float_as_uint(logp), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}

// ------------------------------------------------------------------ direct merge of at most kBlockMergeSpill keys (one wave)
// Butterfly over the wave whose first `gsteps` steps take the maximum inside groups of 2^gsteps lanes and whose remaining steps
// take the minimum over those groups: the smallest group maximum.  A group is NEIGHBOURS, or lanes that agree in their lowest bits.
template <bool NEIGHBOURS>
__device__ __forceinline__ unsigned wave_min_of_group_max_u32(unsigned v, int gsteps) {
    int step = 0;
    auto fold = [&](unsigned a, unsigned b) { v = gsteps > step++ ? (a > b ? a : b) : (a < b ? a : b); };
    auto halves = [&]() {
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        fold(r[0], r[1]);
    };
    auto rows = [&]() {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        fold(r[0], r[1]);
    };
    if constexpr (NEIGHBOURS) {
        fold(v, dpp_mov<0xB1>(v));      // quad_perm [1,0,3,2]
        fold(v, dpp_mov<0x4E>(v));      // quad_perm [2,3,0,1]
        fold(v, dpp_mov<0x141>(v));     // row_half_mirror
        fold(v, dpp_mov<0x140>(v));     // row_mirror
        rows();
        halves();
    } else {
        halves();
        rows();
        fold(v, dpp_mov<0x128>(v));     // row_ror:8
        fold(v, dpp_mov<0x141>(v));     // row_half_mirror
        fold(v, dpp_mov<0x4E>(v));      // quad_perm [2,3,0,1]
        fold(v, dpp_mov<0xB1>(v));      // quad_perm [1,0,3,2]
    }
    return v;
}

constexpr int kDirectMaxCand = 128;
constexpr int kDirectPad = 8;               // keys read at a time when the candidates are ranked
constexpr int kDirectLists = kStepMaxBlocks / kWave;      // lists per lane: up to 256 in all
constexpr int kBlockMergeSpill = 48 * kWave;              // keys of 256 lists of 12: more go to the merge by eight waves

// 16 bytes per lane with the coherence of acquire_u64 (agent scope: not served from this XCD's L2).
// Issue cost per wave is that of an 8-byte load, so two keys per load halve the request time.
__device__ __forceinline__ void acquire_load16(u32x4 &dst, const void *p) {
    asm volatile("global_load_dwordx4 %0, %1, off sc1" : "=v"(dst) : "v"(p) : "memory");
}
template <int N>
__device__ __forceinline__ void wait_loads16(u32x4 (&r)[N]) {
    static_assert(N % 4 == 0 && N <= 24);
    // (the first of them waits for all)
#pragma unroll
    for (int q = 0; q < N; q += 4) asm volatile("s_waitcnt vmcnt(0)" : "+v"(r[q]), "+v"(r[q + 1]), "+v"(r[q + 2]), "+v"(r[q + 3]));
}

// The first active lane's value in every lane.  The row's log-sum-exp goes through this before it is subtracted
// from the logits: the lanes' copies of a wave-wide float sum can differ in the last bits (the summand is a product,
// and the compiler contracts it with the first exchange step into a fused multiply-add -- a lane's own product
// unrounded, its partner's rounded), and tokens with bit-identical logits must get bit-identical log-probs
// whichever lane writes them.
__device__ __forceinline__ float lane_uniform(float x) {
    return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(x)));
}

// The log-sum-exp of up to 256 lists' (max, sum-exp) pairs, four per lane; one value in all lanes.
__device__ __forceinline__ float lse_of_lists(const unsigned long long *__restrict__ pms_row, int B, int lane) {
    unsigned long long ms[kDirectLists];
#pragma unroll
    for (int x = 0; x < kDirectLists; ++x) ms[x] = acquire_u64(pms_row + min(lane + kWave * x, B - 1));
    float lm = -INFINITY;
#pragma unroll
    for (int x = 0; x < kDirectLists; ++x) lm = fmaxf(lm, __uint_as_float((unsigned)ms[x]));      // (past the end: the last list's again)
    const float M = wave_max(lm);
    float ls = 0.f;
#pragma unroll
    for (int x = 0; x < kDirectLists; ++x) {
        const float e = __uint_as_float((unsigned)(ms[x] >> 32)) * __expf(__uint_as_float((unsigned)ms[x]) - M);
        ls += lane + kWave * x < B ? e : 0.f;
    }
    return lane_uniform(M + __logf(wave_sum(ls)));
}

// A value that m keys reach, of the lanes' best logits: with G = the power of two >= m the lanes form G groups; every group's
// best logit is a different key, so at least G >= m keys reach the smallest of the group maxima.
template <bool NEIGHBOURS>
__device__ __forceinline__ unsigned merge_threshold(unsigned top, int m) {
    unsigned T;
    if (m <= 8) {
        int gsteps = 6;                 // G = 64 >> gsteps groups, G >= m
        while ((kWave >> gsteps) < m) --gsteps;
        T = wave_min_of_group_max_u32<NEIGHBOURS>(top, gsteps);
    } else {
        // 9 or more tokens: the power of two above m would make 16 or more groups and several times m candidates.
        // Instead T = the upper 16 bits of the m-th largest of the lanes' best logits, found bit by bit with ballots
        // (at least m lanes, hence m keys, reach it; if fewer than m lanes hold a key at all, T comes out as 0).
        T = wave_kth_largest_prefix16(top, m);
    }
    return T == 0u ? 1u : T;            // an empty group: every real key is a candidate (real keys have a non-zero high word)
}

// Ranks the `ncand` keys in `stage` by counting and writes the m best.  false, with nothing written: there are more than
// kDirectMaxCand (massive ties).  lse_fn() is called once, when the results are about to be written.
template <typename LseFn>
__device__ __forceinline__ bool rank_candidates(unsigned long long *stage, int ncand, int m, LseFn &&lse_fn,
                                                int *__restrict__ out_ids_row, float *__restrict__ out_logp_row, int lane) {
    if (ncand > kDirectMaxCand) return false;
    if (lane < kDirectPad) stage[ncand + lane] = kNoKey;      // (the ranking reads whole groups of keys)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    unsigned long long mine[kDirectMaxCand / kWave];
    int above[kDirectMaxCand / kWave];
#pragma unroll
    for (int c = 0; c < kDirectMaxCand / kWave; ++c) {
        mine[c] = kNoKey;
        above[c] = 0;
        if (c * kWave >= ncand) break;      // (uniform)
        mine[c] = c * kWave + lane < ncand ? stage[c * kWave + lane] : kNoKey;
        for (int x = 0; x < ncand; x += kDirectPad) {
            unsigned long long t[kDirectPad];
#pragma unroll
            for (int q = 0; q < kDirectPad; ++q) t[q] = stage[x + q];      // every lane reads the same key: a broadcast
#pragma unroll
            for (int q = 0; q < kDirectPad; ++q) above[c] += t[q] > mine[c] ? 1 : 0;
        }
    }
    const float lse = lse_fn();
#pragma unroll
    for (int c = 0; c < kDirectMaxCand / kWave; ++c) {
        if (mine[c] != kNoKey && above[c] < m)
            store_result(out_ids_row, out_logp_row, above[c], key_id(mine[c]), key_logit(mine[c]) - lse);
    }
    __builtin_amdgcn_wave_barrier();
    return true;
}

// Up to 64 U keys in any order, U per lane: few lists, of which some lanes would have none, and groups of lanes no key at all
// (then every key is a candidate).  All of them are read in one go; U > 4: two to a load, `total` even.
template <int U, typename LseFn>
__device__ __forceinline__ bool finalize_row_flat(const unsigned long long *__restrict__ src, int total, int m, LseFn &&lse_fn,
                                                  unsigned long long *stage, int *__restrict__ out_ids_row,
                                                  float *__restrict__ out_logp_row, int lane) {
    unsigned long long key[U];
    if constexpr (U > 4) {
        u32x4 r[U / 2];
        const int npairs = total >> 1;
        // Straight-line code from the first request to the wait: the compiler does not know that these registers are still in
        // flight, and a branch in between makes it copy them at the join -- before their values have arrived.
#pragma unroll
        for (int u = 0; u < U / 2; ++u) acquire_load16(r[u], src + 2 * min(u * kWave + lane, npairs - 1));
        wait_loads16(r);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const u32x4 &v = r[u / 2];
            key[u] = (u / 2) * kWave + lane < npairs ? ((unsigned long long)v[2 * (u & 1) + 1] << 32) | v[2 * (u & 1)] : kNoKey;
        }
    } else {
#pragma unroll
        for (int u = 0; u < U; ++u) key[u] = acquire_u64(src + min(u * kWave + lane, total - 1));
#pragma unroll
        for (int u = 0; u < U; ++u) key[u] = u * kWave + lane < total ? key[u] : kNoKey;
    }
    unsigned top = 0u;
#pragma unroll
    for (int u = 0; u < U; ++u) top = (unsigned)(key[u] >> 32) > top ? (unsigned)(key[u] >> 32) : top;
    const unsigned T = merge_threshold<true>(top, m);
    int ncand = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const bool c = (unsigned)(key[u] >> 32) >= T;
        const unsigned long long mask = __ballot(c);
        if (mask != 0ull) {
            const int slot = ncand + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
            if (c && slot < kDirectMaxCand) stage[slot] = key[u];
            ncand += __popcll(mask);
        }
    }
    return rank_candidates(stage, ncand, m, lse_fn, out_ids_row, out_logp_row, lane);
}

// Up to 256 lists of L keys, each in descending order, four lists per lane.  The m best keys are among those whose logit reaches
// the threshold (a dozen or two; the groups are strided, since of neighbouring lanes all lists may be empty, as for a small head's
// rows beside a large one).  Only the first D keys of every list are read at first: a list's next key matters where the one before
// it reaches T, so the keys are looked at rank by rank until a rank has none (two or three of them, as a rule; all L keys of all
// lists, one test each, took 0.5 us longer).  Where the best tokens share a list (a head in order of frequency) what lies behind
// the first D is asked for in one or two trips; a trip per rank took longer than the short lists save (n = 8, m = 8, k = 5000,
// d = 3072, all in one list: 14.6 us with all keys read, 14.9, now 14.2; k = 32768 36.9 / 37.8 / 37.1, spread over the lists
// 37.0 / 35.8 / 35.8; n = 4, m = 11, in one list 37.0 / 38.6 / 37.6; n = 4, m = 10, d = 2048 28.0 / 29.3 / 28.7).
// The candidates are compacted into LDS and ranked by counting.  PAIRS: L is even, two keys to a load.  MORE: L may exceed
// D, and so many keys of a list are asked for at a time then (two forms, of four and eight, in one took the usual case 0.25 us longer).
// Returns false, having written nothing, when more than kDirectMaxCand keys reach T (massive ties): the caller then merges the
// lists round by round.  lse_fn() is called once, when the results are about to be written.
template <int D, bool PAIRS, int MORE, typename LseFn>
__device__ __forceinline__ bool finalize_row_direct(const unsigned long long *__restrict__ src, int B, int L, int m,
                                                    LseFn &&lse_fn, unsigned long long *stage, int *__restrict__ out_ids_row,
                                                    float *__restrict__ out_logp_row, int lane) {
    constexpr int X = kDirectLists;
    static_assert(!PAIRS || D % 2 == 0, "whole pairs");
    unsigned long long key[D][X];
    if constexpr (PAIRS) {
        u32x4 r[X * D / 2];
        // Straight-line code from the first request to the wait: the compiler does not know that these registers are still in
        // flight, and a branch in between makes it copy them at the join -- before their values have arrived.
#pragma unroll
        for (int x = 0; x < X; ++x) {
#pragma unroll
            for (int q = 0; q < D / 2; ++q) acquire_load16(r[x * (D / 2) + q], src + (size_t)min(lane + kWave * x, B - 1) * L + 2 * q);
        }
        wait_loads16(r);
#pragma unroll
        for (int x = 0; x < X; ++x) {
#pragma unroll
            for (int j = 0; j < D; ++j) {
                const u32x4 &v = r[x * (D / 2) + j / 2];
                key[j][x] = ((unsigned long long)v[2 * (j & 1) + 1] << 32) | v[2 * (j & 1)];
            }
        }
    } else {
#pragma unroll
        for (int j = 0; j < D; ++j) {
#pragma unroll
            for (int x = 0; x < X; ++x) key[j][x] = acquire_u64(src + (size_t)min(lane + kWave * x, B - 1) * L + j);
        }
    }
#pragma unroll
    for (int x = 0; x < X; ++x) {
#pragma unroll
        for (int j = 0; j < D; ++j) key[j][x] = lane + kWave * x < B ? key[j][x] : kNoKey;
    }
    unsigned top = 0u;
#pragma unroll
    for (int x = 0; x < X; ++x) {
        const unsigned o = (unsigned)(key[0][x] >> 32);
        top = o > top ? o : top;
    }
    const unsigned T = merge_threshold<false>(top, m);
    int ncand = 0;
    // the lists' keys of one rank; whether any is a candidate
    auto collect = [&](const unsigned long long (&k)[X]) -> bool {
        unsigned best = 0u;
#pragma unroll
        for (int x = 0; x < X; ++x) best = (unsigned)(k[x] >> 32) > best ? (unsigned)(k[x] >> 32) : best;
        if (__ballot(best >= T) == 0ull) return false;
#pragma unroll
        for (int x = 0; x < X; ++x) {
            const bool c = (unsigned)(k[x] >> 32) >= T;
            const unsigned long long mask = __ballot(c);
            if (mask != 0ull) {
                const int slot = ncand + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
                if (c && slot < kDirectMaxCand) stage[slot] = k[x];
                ncand += __popcll(mask);
            }
        }
        return true;
    };
    bool more = true;
#pragma unroll
    for (int j = 0; j < D; ++j) more = more && collect(key[j]);
    if constexpr (MORE == 0) return rank_candidates(stage, ncand, m, lse_fn, out_ids_row, out_logp_row, lane);
    // the next keys of the lists whose last one reaches T, R of each to a trip
    constexpr int R = MORE > 0 ? MORE : 1;
    for (int j = D; more && j < L; j += R) {
        unsigned long long next[R][X];
        bool open[X];
#pragma unroll
        for (int x = 0; x < X; ++x) {
            open[x] = (unsigned)(key[D - 1][x] >> 32) >= T;
            // (a list that is through asks for what the others of its kind ask for)
            const unsigned long long *list = src + (open[x] ? (size_t)(lane + kWave * x) * L : (size_t)0);
#pragma unroll
            for (int q = 0; q < R; ++q) next[q][x] = acquire_u64(list + (open[x] ? min(j + q, L - 1) : 0));
        }
#pragma unroll
        for (int x = 0; x < X; ++x) {
#pragma unroll
            for (int q = 0; q < R; ++q) next[q][x] = open[x] && j + q < L ? next[q][x] : kNoKey;
            key[D - 1][x] = next[R - 1][x];
        }
#pragma unroll
        for (int q = 0; q < R; ++q) more = more && ncand <= kDirectMaxCand && collect(next[q]);
    }
    return rank_candidates(stage, ncand, m, lse_fn, out_ids_row, out_logp_row, lane);
}

// ------------------------------------------------------------------ final merge of one hidden row (one wave)
// pkeys_row: [B][L] keys, each list sorted descending.  stage: wave-private LDS for (min(B, 256) + 1) * L + kDirectPad keys.
// Lists are merged 256 at a time (4 per lane); the best m of one
// group are carried into the next as one more list, so B is unbounded.
// lse_fn(): the row's log-sum-exp, one value in all lanes; called exactly once, when the results are about to be written.
template <typename LseFn>
__device__ __forceinline__ void finalize_row(const unsigned long long *__restrict__ pkeys_row, int B, int L, int m, bool several_heads, LseFn &&lse_fn,
                                             unsigned long long *stage, int *__restrict__ out_ids_row,
                                             float *__restrict__ out_logp_row, int lane) {
    constexpr int GROUP = kStepMaxBlocks;        // lists merged per pass
    constexpr int BQ = GROUP / kWave + 1;        // lists per lane
    constexpr int U = 32;                        // 64-lane loads in flight per batch (16 KiB)
    // (64 tokens: the threshold is the worst of the lanes' best keys, which more than kDirectMaxCand reach wherever there are so many)
    if (B <= GROUP && B * L <= (m < kWave ? kBlockMergeSpill : kDirectMaxCand)) {
        bool done;
        // Fewer lists than lanes: the keys are dealt to the lanes one by one (n = 1, 17 lists of 8, m = 24 7.7 us a step; by
        // lists 19.3, since lanes without one leave no threshold; n = 7, 11 lists of 8, m = 8 8.3 / 10.0).  (The usual case first.)
        if (B >= kWave && L == 8)
            done = finalize_row_direct<4, true, 4>(pkeys_row, B, L, m, lse_fn, stage, out_ids_row, out_logp_row, lane);
        else if (B * L <= 4 * kWave)
            done = finalize_row_flat<4>(pkeys_row, B * L, m, lse_fn, stage, out_ids_row, out_logp_row, lane);
        else if (several_heads && m > 8 && (B * L & 1) == 0)
            // (a small head's lists alone leave no threshold either: n = 4, m = 10, heads of 1378, 236, 560 and 93 rows 12.9 us, by
            // lists 16.2.  Up to eight tokens a few lists are a few groups, by lists 11.6 against 12.3)
            done = finalize_row_flat<48>(pkeys_row, B * L, m, lse_fn, stage, out_ids_row, out_logp_row, lane);
        else if (B < kWave && B * L <= 32 * kWave && (B * L & 1) == 0)
            done = finalize_row_flat<32>(pkeys_row, B * L, m, lse_fn, stage, out_ids_row, out_logp_row, lane);
        else if (L == 1)
            done = finalize_row_direct<1, false, 0>(pkeys_row, B, L, m, lse_fn, stage, out_ids_row, out_logp_row, lane);
        else if (L == 2)
            done = finalize_row_direct<2, true, 0>(pkeys_row, B, L, m, lse_fn, stage, out_ids_row, out_logp_row, lane);
        else if (L == 4)
            done = finalize_row_direct<4, true, 0>(pkeys_row, B, L, m, lse_fn, stage, out_ids_row, out_logp_row, lane);
        else if ((L & 1) == 0)
            done = finalize_row_direct<4, true, 8>(pkeys_row, B, L, m, lse_fn, stage, out_ids_row, out_logp_row, lane);
        else
            done = finalize_row_direct<3, false, 8>(pkeys_row, B, L, m, lse_fn, stage, out_ids_row, out_logp_row, lane);
        if (done) return;
    }

    unsigned res_ord = 0u;
    unsigned res_id = 0u;
    for (int b0 = 0; b0 < B; b0 += GROUP) {
        const int Bc = min(GROUP, B - b0);
        const int total = Bc * L;
        const unsigned long long *src = pkeys_row + (size_t)b0 * L;
        // everything this pass needs is requested before the first wait
        for (int base = 0; base < total; base += U * kWave) {
            unsigned long long kreg[U];
            if (base + U * kWave <= total) {
#pragma unroll
                for (int u = 0; u < U; ++u) kreg[u] = acquire_u64(src + base + u * kWave + lane);
#pragma unroll
                for (int u = 0; u < U; ++u) stage[base + u * kWave + lane] = kreg[u];
            } else {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (base + u * kWave < total) kreg[u] = acquire_u64(src + min(base + u * kWave + lane, total - 1));
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int e = base + u * kWave + lane;
                    if (e < total) stage[e] = kreg[u];
                }
            }
        }
        // the previous pass's result (lane r holds rank r) joins as list number Bc
        if (lane < L)
            stage[total + lane] = (b0 > 0 && lane < m && res_ord != 0u)
                                      ? (((unsigned long long)res_ord << 32) | (unsigned)(~res_id))
                                      : kNoKey;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // m rounds over the heads of the sorted lists
        const int nl = Bc + 1;
        unsigned ord[BQ];
        int id[BQ];
        int pos[BQ];
#pragma unroll
        for (int q = 0; q < BQ; ++q) {
            const int b = lane + kWave * q;
            const unsigned long long key = b < nl ? stage[(size_t)b * L] : kNoKey;
            ord[q] = (unsigned)(key >> 32);
            id[q] = key_id(key);
            pos[q] = 0;
        }
        res_ord = 0u;
        res_id = 0u;
        for (int r = 0; r < m; ++r) {
            // the successor of every head is read now, so that a pop below costs no LDS round trip
            unsigned long long succ[BQ];
#pragma unroll
            for (int q = 0; q < BQ; ++q)
                succ[q] = stage[(size_t)min(lane + kWave * q, nl - 1) * L + min(pos[q] + 1, L - 1)];
            unsigned bo = ord[0];
#pragma unroll
            for (int q = 1; q < BQ; ++q) bo = ord[q] > bo ? ord[q] : bo;
            const unsigned wmax = wave_max_u32(bo);
            unsigned myid = 0xFFFFFFFFu;
            int cnt = 0;
#pragma unroll
            for (int q = 0; q < BQ; ++q) {
                if (ord[q] == wmax) {
                    myid = (unsigned)id[q] < myid ? (unsigned)id[q] : myid;
                    ++cnt;
                }
            }
            const unsigned long long holders = __ballot(cnt > 0);
            const unsigned long long multi = __ballot(cnt > 1);
            unsigned wid;
            if (__popcll(holders) == 1 && multi == 0ull) {
                wid = __builtin_amdgcn_readlane(myid, __ffsll((long long)holders) - 1);
            } else {
                wid = wave_min_u32(myid);
            }
#pragma unroll
            for (int q = 0; q < BQ; ++q) {
                const bool win = ord[q] == wmax && (unsigned)id[q] == wid && wmax != 0u;
                const unsigned long long key = pos[q] + 1 < L ? succ[q] : kNoKey;
                ord[q] = win ? (unsigned)(key >> 32) : ord[q];
                id[q] = win ? key_id(key) : id[q];
                pos[q] += win ? 1 : 0;
            }
            if (lane == r) {
                res_ord = wmax;
                res_id = wid;
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    const float lse = lse_fn();
    if (lane < m) {
        store_result(out_ids_row, out_logp_row, lane, (int)res_id, from_orderable_f32(res_ord) - lse);
    }
}

// The row's log-sum-exp over any number of lists.
__device__ __forceinline__ float row_lse(const unsigned long long *__restrict__ pms_row, int B, int lane) {
    if (B <= kStepMaxBlocks) return lse_of_lists(pms_row, B, lane);
    float lm = -INFINITY, ls = 0.f;
    for (int b0 = 0; b0 < B; b0 += kWave) {
        const unsigned long long ms = acquire_u64(pms_row + min(b0 + lane, B - 1));
        if (b0 + lane < B) {
            const float Mb = __uint_as_float((unsigned)ms);
            const float Sb = __uint_as_float((unsigned)(ms >> 32));
            const float Mn = fmaxf(lm, Mb);
            ls = ls * __expf(lm - Mn) + Sb * __expf(Mb - Mn);   // exp(-inf) = 0 on the first term
            lm = Mn;
        }
    }
    const float M = wave_max(lm);
    return lane_uniform(M + __logf(wave_sum(ls * __expf(lm - M))));
}

// A hidden row's merge by the first two waves of its workgroup (all its threads call this): the log-sum-exp is reduced in the
// second wave while the first one selects (one after the other in one wave took 0.4 us longer).
__device__ __forceinline__ void finalize_row_pair(const FinalizeArgs &f, int i, int o, unsigned long long *stage, float *s_lse, int lane, int w) {
    const unsigned long long *pms_row = f.pms + (size_t)i * f.nlists, *pkeys_row = f.pkeys + (size_t)i * f.nlists * f.L;
    if (w == 0) {
        auto lse_fn = [&]() {
            __syncthreads();
            return *s_lse;
        };
        finalize_row(pkeys_row, f.nlists, f.L, f.m, f.several_heads != 0, lse_fn, stage, f.out_ids + (size_t)o * f.m, f.out_logp + (size_t)o * f.m, lane);
    } else {
        if (w == 1) {
            const float lse = row_lse(pms_row, f.nlists, lane);
            if (lane == 0) {
                *s_lse = lse;
                f.lse_buf[i] = lse;
                if (f.out_lse) f.out_lse[o] = lse;
            }
        }
        __syncthreads();
    }
}
// The same by one wave.
__device__ __forceinline__ void finalize_row_alone(const FinalizeArgs &f, int i, int o, unsigned long long *stage, int lane) {
    const float lse = row_lse(f.pms + (size_t)i * f.nlists, f.nlists, lane);
    if (lane == 0) {
        f.lse_buf[i] = lse;
        if (f.out_lse) f.out_lse[o] = lse;
    }
    finalize_row(f.pkeys + (size_t)i * f.nlists * f.L, f.nlists, f.L, f.m, f.several_heads != 0, [lse]() { return lse; }, stage,
                       f.out_ids + (size_t)o * f.m, f.out_logp + (size_t)o * f.m, lane);
}

// ------------------------------------------------------------------ merge of many lists (eight waves per hidden row)
// More keys than one wave holds in registers (more than 256 lists, or more than 3072 keys): the row's workgroup of
// eight waves holds them all (up to 2048 lists and 16384 keys, what the
// largest head has in tiles of 128 rows with 8 tokens), one key per load and thread, and selects by threshold like the direct merge above.  The
// waves form the groups: each finds the ceil(m / 8)-th largest of its lanes' best logits, so at least m keys reach T,
// the smallest of the eight values -- about three times m do.  They are compacted into `cand` and ranked by counting.
// What it replaces there, one wave that merges 256 sorted lists at a time in m dependent rounds, was bound by those
// rounds: m = 8, k = 65536 (512 lists) 10.0 -> 5.2 us, k = 128256 (668 lists of 64 hidden rows) 15.3 -> 5.4.  With more
// than 8 hidden rows it is also the faster one for lists that one wave could hold (256 lists of 8 keys: n = 64 6.1 -> 5.4,
// n = 128 6.7 -> 4.9); up to 8 rows the two tie (n = 8: 4.6 / 4.6), and so do they below about 1000 keys.
// What is left is a chain: loads, a reduction, a barrier, one LDS atomic per wave, a barrier, the ranking.  The log-sum-exp is
// reduced beside it in a ninth wave, and up to 2048 keys are loaded as four per thread, not eight with half of them twice
// (with the second form of the selection in the tiles, 64 rows of 32768 x 4096 51.3 -> 50.7 us, 12 of 5000 x 3072 16.8 -> 16.2;
// with a comparison of places beside every one of keys instead of the empty keys behind the last half of that was lost).
// Returns false, having written nothing, when more than kBlockMaxCand keys reach T (massive ties).
constexpr int kBlockMergeWaves = 8;
constexpr int kBlockMergeThreads = kBlockMergeWaves * kWave;
constexpr int kBlockMergeLaunch = kBlockMergeThreads + kWave;      // and a wave for the log-sum-exp
constexpr int kBlockMergeMaxKeys = 32 * kBlockMergeThreads;
constexpr int kBlockMergeMaxLists = 4 * kBlockMergeThreads;
constexpr int kBlockMaxCand = 1024;
static_assert(kStepMaxK / kMfmaTileRows <= kBlockMergeMaxLists && kStepMaxK / kMfmaTileRows * kRowSelectMinLManyRows <= kBlockMergeMaxKeys,
              "the lists of the largest head in tiles of 128 rows");

struct BlockMergeLds {
    unsigned long long cand[kBlockMaxCand];
    unsigned wave_kth[kBlockMergeWaves];
    float lse;
    int ncand;
};

__host__ __device__ __forceinline__ bool block_merge_pays(int n, int B, int L, int m) {
    const int total = B * L;
    return m <= kWave && B <= kBlockMergeMaxLists && total <= kBlockMergeMaxKeys &&
           (B > kStepMaxBlocks || total > kBlockMergeSpill || (n > kGemvMaxN && total > 1024));
}

template <int U>
__device__ __forceinline__ bool finalize_row_block(const unsigned long long *__restrict__ pms_row,
                                                   const unsigned long long *__restrict__ pkeys_row, int B, int total,
                                                   int m, BlockMergeLds &s, int *__restrict__ out_ids_row,
                                                   float *__restrict__ out_logp_row, float *__restrict__ out_lse_i,
                                                   float *__restrict__ lse_buf_i, int lane, int w) {
    if (w == kBlockMergeWaves) {
        // four of the lists' pairs per lane, or sixteen (more than 256 lists: four trips one after the other took longer than
        // everything beside them, and so did a maximum and a sum carried from pair to pair: 995 lists of 8 keys 7.0 us, 6.3 in one
        // trip, now 5.8; 1003 of 4 keys 5.9 / 5.4 / 5.0)
        float lm = -INFINITY, ls = 0.f;
        auto fold = [&](auto per_lane, int b0) {
            constexpr int Q = decltype(per_lane)::value;
            unsigned long long ms[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) ms[q] = acquire_u64(pms_row + min(b0 + q * kWave + lane, B - 1));
            float top = lm;
#pragma unroll
            for (int q = 0; q < Q; ++q) top = fmaxf(top, __uint_as_float((unsigned)ms[q]));      // (past the end: the last list's again)
            ls *= __expf(lm - top);                                       // exp(-inf) = 0 on the first term
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const float e = __uint_as_float((unsigned)(ms[q] >> 32)) * __expf(__uint_as_float((unsigned)ms[q]) - top);
                ls += b0 + q * kWave + lane < B ? e : 0.f;
            }
            lm = top;
        };
        if (B <= 4 * kWave)
            fold(std::integral_constant<int, 4>{}, 0);
        else
            for (int b0 = 0; b0 < B; b0 += 16 * kWave) fold(std::integral_constant<int, 16>{}, b0);
        __syncthreads();
        const float M = wave_max(lm);
        const float lse = lane_uniform(M + __logf(wave_sum(ls * __expf(lm - M))));
        if (lane == 0) s.lse = lse;
        __syncthreads();
        if (s.ncand > kBlockMaxCand) {
            __syncthreads();
            return false;
        }
        if (lane == 0) {
            *lse_buf_i = lse;
            if (out_lse_i) *out_lse_i = lse;
        }
        return true;
    }
    const int tid = w * kWave + lane;
    unsigned long long key[U];
#pragma unroll
    for (int u = 0; u < U; ++u) key[u] = acquire_u64(pkeys_row + min(u * kBlockMergeThreads + tid, total - 1));
    unsigned top = 0u;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (u * kBlockMergeThreads + tid >= total) key[u] = kNoKey;
        const unsigned o = (unsigned)(key[u] >> 32);
        top = o > top ? o : top;
    }
    const unsigned kth = m <= kBlockMergeWaves ? wave_max_u32(top)
                                               : wave_kth_largest_prefix16(top, (m + kBlockMergeWaves - 1) / kBlockMergeWaves);
    if (lane == 0) s.wave_kth[w] = kth;
    if (tid == 0) s.ncand = 0;
    // (the ranking reads eight keys at a time: what is behind the last candidate loses against all of them)
    for (int x = tid; x < kBlockMaxCand; x += kBlockMergeThreads) s.cand[x] = kNoKey;
    __syncthreads();
    unsigned T = s.wave_kth[0];
#pragma unroll
    for (int q = 1; q < kBlockMergeWaves; ++q) T = s.wave_kth[q] < T ? s.wave_kth[q] : T;
    T = T == 0u ? 1u : T;               // a wave without keys: every real key is a candidate
    int mine_n = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) mine_n += __popcll(__ballot((unsigned)(key[u] >> 32) >= T));
    if (mine_n != 0) {
        int at = 0;
        if (lane == 0) at = atomicAdd(&s.ncand, mine_n);      // (one per wave: one per load of keys took a round trip each)
        at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool c = (unsigned)(key[u] >> 32) >= T;
            const unsigned long long mask = __ballot(c);
            const int slot = at + __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
            if (c && slot < kBlockMaxCand) s.cand[slot] = key[u];
            at += __popcll(mask);
        }
    }
    __syncthreads();
    const int ncand = s.ncand;
    if (ncand > kBlockMaxCand) {
        __syncthreads();                // the caller reuses this LDS
        return false;
    }
    const float lse = s.lse;
    for (int c = tid; c < ncand; c += kBlockMergeThreads) {
        const unsigned long long mine = s.cand[c];
        int above = 0;
        for (int x = 0; x < ncand; x += 8) {
            unsigned long long t[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) t[q] = s.cand[x + q];      // every lane reads the same key: a broadcast
#pragma unroll
            for (int q = 0; q < 8; ++q) above += t[q] > mine ? 1 : 0;
        }
        if (above < m) store_result(out_ids_row, out_logp_row, above, key_id(mine), key_logit(mine) - lse);
    }
    return true;
}

__device__ __forceinline__ bool merge_row_block(const FinalizeArgs &f, int i, int o, BlockMergeLds &s, int lane, int w) {
    const unsigned long long *pms = f.pms + (size_t)i * f.nlists, *pkeys = f.pkeys + (size_t)i * f.nlists * f.L;
    int *ids = f.out_ids + (size_t)o * f.m;
    float *logp = f.out_logp + (size_t)o * f.m, *lse = f.out_lse ? f.out_lse + o : nullptr;
    const int total = f.nlists * f.L;
    if (total <= 4 * kBlockMergeThreads)
        return finalize_row_block<4>(pms, pkeys, f.nlists, total, f.m, s, ids, logp, lse, f.lse_buf + i, lane, w);
    if (total <= 8 * kBlockMergeThreads)
        return finalize_row_block<8>(pms, pkeys, f.nlists, total, f.m, s, ids, logp, lse, f.lse_buf + i, lane, w);
    if (total <= 16 * kBlockMergeThreads)
        return finalize_row_block<16>(pms, pkeys, f.nlists, total, f.m, s, ids, logp, lse, f.lse_buf + i, lane, w);
    return finalize_row_block<32>(pms, pkeys, f.nlists, total, f.m, s, ids, logp, lse, f.lse_buf + i, lane, w);
}

}  // namespace vt
