// C ABI of libvocabtrim.so: argument validation, workspace layout, kernel dispatch.
// Every entry point only enqueues work on the caller's stream.
#include "vocabtrim.h"

#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstring>
#include <mutex>

#include "vt_build.h"
#include "vt_step.h"
#include "vt_tree.h"

namespace {

inline bool aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }
inline size_t round_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
inline int elem_size(int dtype) { return dtype == VT_BF16 ? 2 : 4; }

// last HIP error seen by this thread's calls into the library (for vt_last_device_error)
thread_local hipError_t g_last_hip_error = hipSuccess;

inline int device_status(hipError_t e) {
    if (e == hipSuccess) return VT_OK;
    g_last_hip_error = e;
    return VT_ERR_DEVICE;
}
inline int launch_status() { return device_status(hipGetLastError()); }

// ---------------------------------------------------------------- library-owned step workspace
// Device memory of the draft step for callers that cannot allocate (vt_draft_head_step_static): one array per
// GPU, alive from the moment the code object is loaded on it until the process ends.  In host code the array's
// name is only a handle; the device address is asked for once per device and kept (both arrays' by the first call that uses either:
// a program makes that call outside stream capture).
static __device__ __align__(256) unsigned char scratch[VT_STATIC_WS_BYTES];
// ... and of the steps that plan_stored() has run on stored logits, which have the bits of vt_draft_head_step's only if they run the same
// way: 256 hidden rows by 256 tiles of 160 logits, 4 MiB of re-laid h and the small parts of a workspace at most.
constexpr size_t kStaticStoredBytes = (size_t)48 << 20;
static __device__ __align__(256) unsigned char stored_scratch[kStaticStoredBytes];
std::mutex g_scratch_mutex;
void *g_scratch_ptr[64][2] = {};      // per device ordinal; written under the mutex, never changed afterwards

int static_scratch_of_current_device(bool stored, void **out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return device_status(e);
    if (dev < 0 || dev >= 64) return device_status(hipErrorInvalidDevice);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    void **const known = g_scratch_ptr[dev];
    if (known[0] == nullptr || known[1] == nullptr) {
        void *p[2] = {nullptr, nullptr};
        e = hipGetSymbolAddress(&p[0], HIP_SYMBOL(scratch));
        if (e == hipSuccess) e = hipGetSymbolAddress(&p[1], HIP_SYMBOL(stored_scratch));
        if (e != hipSuccess) return device_status(e);
        if (p[0] == nullptr || p[1] == nullptr) return device_status(hipErrorInvalidSymbol);
        known[0] = p[0];
        known[1] = p[1];
    }
    *out = known[stored ? 1 : 0];
    return VT_OK;
}

// ---------------------------------------------------------------- draft-step plan
// Workgroups one round of the draft-step kernels may have: the compute units of the current device (one workgroup
// per CU: they take most of a CU's LDS), read once per process; 256 on MI355X, which is also the most the kernels'
// tables are sized for and the answer where no device is visible (the workspace-size functions are pure host code).
// The measured crossovers below (so many tiles of so many rows) are scaled to it.
int round_workgroups() {
    static const int cus = []() {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) {
            (void)hipGetLastError();
            return vt::kStepMaxBlocks;
        }
        return n < vt::kStepMaxBlocks ? n : vt::kStepMaxBlocks;
    }();
    return cus;
}

struct StepPlan {
    bool ok = false;
    bool gemv = false;     // small-n VALU path
    bool mfma = false;     // matrix-core path
    int NP = 0, CS = 0, S = 0;
    int NT = 0, nlists = 0, KC = 0, hpitch = 0, fin_stage_keys = 0, ksplit = 1, nwaves = vt::kStepWaves;
    size_t fin_lds = 0;
    int rpb = 0, nblocks = 0, tpitch = 0, L = 0;
    size_t lds = 0;
    // workspace layout (byte offsets)
    size_t off_lse = 0, off_pms = 0, off_pkeys = 0, off_hpack = 0, off_zbuf = 0, bytes = 0;
    bool row_select = false;   // matrix-core path: logits stored, one workgroup per hidden row finishes
    bool instead_of_lists = false;      // ... which a smaller workspace would have as lists
    int extra_rows = 0;        // matrix-core path: tile rows past the 128th
    // more than 8 hidden rows: 16-row groups of a tile, LDS offset of its target ids, epilogue passes
    int row_groups = 0, ids_off = 0, passes = 1;
    bool twin = false;
    bool wide = false;         // more than 64 hidden rows
    int splits = 1;            // more than 8 hidden rows: slices of the columns, a workgroup each per tile
    int parts = 0;             // ... stored logits: parts of a row with a (max, sum-exp) each, of part_rows rows, per_tile to a tile
    int part_rows = 0, per_tile = 0;
    size_t list_room = 0;      // ... bytes that the lists of fewer hidden rows may take on smaller tiles
};

using vt::kTicketBytes;
int slice_pitch(int k) { return (k + 3) / 4 * 4; }      // floats from one hidden row's partial logits to the next one's

// fixed: a tile shape the caller has chosen (several heads in one launch): waves, column split, number of tiles
struct FixedTiles {
    int nwaves = 0, ksplit = 1, nlists = 0;
};
// More than 8 hidden rows: whether the kernel stores its logits and a workgroup per hidden row finishes the step
// (the alternative: candidate lists per tile, merged by step_finalize_kernel).  The tile epilogue selects by threshold up
// to 8 tokens per row (four rows per wave, 16 candidate slots each) and takes a round per token beyond: there the stored
// logits win (k = 32768, d = 4096: n = 64, m = 9: 58.4 against 60.1 us, m = 11: 58.5 / 61.8; n = 32, m = 10: 53.8 /
// 55.1).  Up to 8 tokens the epilogue costs a tile the same few microseconds whatever its height, the logits as much as
// the tile holds: from about 224 rows of 8 tokens on they win where tiles are below 128 rows (n = 256, m = 8, lists
// against logits: k = 16384, d = 4096 68.5 / 61.6 us, k = 22786 76.4 / 73.7; but k = 32768, d = 8192 155.6 / 160.8, k = 65536,
// d = 2048 102.7 / 111.5; n = 200, k = 8000, d = 2048 32.7 / 34.2).
bool stores_logits(int n, int m, int tile_rows) {
    return m > vt::kRowSelectMinLManyRows || (n * m >= vt::kRowSelectMinWork && tile_rows < vt::kMfmaTileRows);
}
// What follows from a tile's row groups (and extra rows, kernel, slices): waves, LDS, number of workgroups.
void cut_many_rows(StepPlan &p, int n, int k, int m) {
    size_t ring, tile;                                // LDS: the stages; the logit tile and the candidate keys after them
    p.passes = 1;
    if (!p.wide) {
        p.nwaves = p.row_groups <= 4 ? vt::kStepWaves : p.row_groups;
        const int rows_in_lds = 16 * (p.row_groups + (p.extra_rows != 0 ? 1 : 0));
        ring = vt::rows_ring_bytes(p.NT, p.row_groups, p.extra_rows != 0, p.twin);
        tile = round_up((size_t)n * (rows_in_lds + 1) * sizeof(float), 16);
    } else {
        const int MT = p.row_groups / 2, NTT = p.NT / 4;
        p.nwaves = vt::kStepWaves;
        ring = vt::wide_ring_bytes(MT, NTT);
        tile = round_up((size_t)n * (32 * MT + 1) * sizeof(float), 16);
        if (tile + vt::kStepWaves * 512 > (size_t)vt::kMaxDynamicLds - 1024) {
            p.passes = 2;
            tile = round_up((size_t)32 * NTT * (32 * MT + 1) * sizeof(float), 16);
        }
    }
    const int tile_rows = 16 * p.row_groups + p.extra_rows;
    p.mfma = true;
    p.nlists = p.nblocks = (k + tile_rows - 1) / tile_rows * p.splits;
    p.L = m < tile_rows ? m : tile_rows;
    tile += (size_t)p.nwaves * 64 * sizeof(unsigned long long);      // 4 x 16 candidate keys per wave
    p.ids_off = (int)round_up(ring > tile ? ring : tile, 16);
    p.lds = (size_t)p.ids_off + vt::kMfmaMaxWaves * 16 * sizeof(int);
}
// More than 8 hidden rows, bf16: how the head is cut into tiles (kernel variant, LDS, number of tiles).
void plan_many_rows(StepPlan &p, int n, int k, int d, int m) {
    const int CUS = round_workgroups();
    const int R = (k + CUS - 1) / CUS;                // rows per tile for one tile per CU
    const int G = (R + 15) / 16;                      // ... in 16-row groups
    // Microseconds of `rounds` rounds of tiles of `rows` rows, roughly: W at a CU's share of the HBM rate, h from the L2,
    // and about 7 us for a round's first loads and its epilogue.
    const int n_padded = n <= 32 ? 32 : n <= vt::kRowsKernelMaxN ? vt::kRowsKernelMaxN : vt::kMfmaMaxN;
    auto cost = [&](int rows) {
        const int tiles = (k + rows - 1) / rows, rounds = (tiles + CUS - 1) / CUS;
        return rounds * ((double)rows * d * 2 / 25e3 + (double)n_padded * d * 2 / 75e3 + 7.0);
    };
    if (n <= vt::kRowsKernelMaxN) {
        const int NT = n <= 32 ? 2 : 4;
        p.NT = NT;
        if (R > vt::kMfmaTileRows && R <= vt::kMfmaTileRows + 16) {
            // 129 .. 144 rows per tile for one tile per CU (the paper's trimmed sizes): tiles of exactly that many rows
            p.row_groups = vt::kStepWaves;
            p.extra_rows = R - vt::kMfmaTileRows;
        } else if (G <= vt::kMfmaMaxWaves) {
            // one round: the tile height follows from the head
            p.row_groups = (G == 5 && NT == 4) ? vt::kStepWaves : G;
        } else {
            // several rounds: two 128-row tiles on a CU at a time, half of its LDS each, so that one streams while the other
            // starts or finishes -- or tiles of up to 192 rows where those come out even (one tile per CU against
            // two: k = 65536, n = 64, d = 2048 57.3 / 51.4 us, n = 9 50.8 / 46.6, k = 128256, n = 64 104.0 / 94.9,
            // k = 60000, n = 20, d = 1024 31.3 / 27.1; but k = 90000, n = 64, d = 3072, 704 tiles against 512 of 176
            // rows: 102.5 / 107.1).  A CU with two tiles pays half of a round's 7 us, one left over all of it.
            const int tiles = (k + vt::kMfmaTileRows - 1) / vt::kMfmaTileRows, rest = tiles % (2 * CUS);
            const double one = cost(vt::kMfmaTileRows) / ((tiles + CUS - 1) / CUS), pair = 2 * one - 10.5;
            const double paired = tiles / (2 * CUS) * pair + (rest == 0 ? 0.0 : rest <= CUS ? one : pair);
            p.row_groups = vt::kStepWaves + 1;
            for (int g = p.row_groups + 1; g <= vt::kMfmaMaxWaves; ++g)
                if (cost(16 * g) < cost(16 * p.row_groups)) p.row_groups = g;
            p.twin = paired <= cost(16 * p.row_groups);
            if (p.twin) p.row_groups = vt::kStepWaves;
        }
    } else {
        const int NTT = n <= 128 ? 2 : n <= 192 ? 3 : 4;
        p.wide = true;
        p.NT = 4 * NTT;
        // (smaller tiles mean more candidate lists: not where only theirs would outgrow the library's own workspace)
        auto list_bytes = [&](int rows) { return (size_t)n * ((k + rows - 1) / rows) * (1 + m) * sizeof(unsigned long long); };
        auto fits = [&](int rows) {
            return stores_logits(n, m, rows) || list_bytes(rows) + 65536 <= (size_t)VT_STATIC_WS_BYTES ||
                   list_bytes(rows) <= list_bytes(vt::kMfmaTileRows);
        };
        int MT = 4;
        for (int x : {1, 2, 3, 5})
            if (fits(32 * x) && cost(32 * x) < cost(32 * MT)) MT = x;
        // (fewer hidden rows take the cheaper tiles, as long as their lists stay within that bound)
        for (int x : {1, 2, 3, 5})
            if (!fits(32 * x) && cost(32 * x) <= cost(32 * MT)) p.list_room = (size_t)VT_STATIC_WS_BYTES - 65536;
        p.row_groups = 2 * MT;
    }
    cut_many_rows(p, n, k, m);
}
StepPlan plan_step_impl(int n, int k, int d, int m, int dtype, bool force_gemv, const FixedTiles &fixed = FixedTiles{});
// force_gemv: the caller needs what only the small-n kernel offers (row picking, the fused tree level)
StepPlan plan_step(int n, int k, int d, int m, int dtype, bool force_gemv = false) {
    StepPlan p = plan_step_impl(n, k, d, m, dtype, force_gemv);
    if (!p.ok && !force_gemv && n <= vt::kGemvMaxN) p = plan_step_impl(n, k, d, m, dtype, true);
    return p;
}
StepPlan plan_step_impl(int n, int k, int d, int m, int dtype, bool force_gemv, const FixedTiles &fixed) {
    StepPlan p;
    if (n <= 0 || k <= 0 || d <= 0 || m <= 0 || k > vt::kStepMaxK) return p;
    const int CUS = round_workgroups();
    int rpb = (k + CUS - 1) / CUS;
    rpb = (rpb + 7) / 8 * 8;
    p.rpb = rpb;
    p.nblocks = (k + rpb - 1) / rpb;
    p.tpitch = rpb + 1;
    p.L = m < rpb ? m : rpb;

    // Up to 8 rows on the matrix-core kernel: its tiles must fill most of the 256 CUs in exactly one round.  A
    // tile is 16 rows per group of KS waves (KS = 1, 2, 4 waves share a group's columns) and a workgroup has up to
    // kMfmaMaxWaves waves, so the tile height follows from the head: ceil(k / 256) rows rounded up to whole groups
    // (k = 32768: 8 waves x 16 rows; the paper's k ~ 33000: 9 waves, 144 rows, 229 - 244 tiles; k = 22786: 6 groups
    // of 2 waves, 96 rows, 238 tiles).  The split needs the kernel's own epilogue (few tokens per row), whole
    // 128-column units per wave and all of h in LDS at once.
    int ksplit = 0, nwaves = vt::kStepWaves, extra_rows = 0;
    if (!force_gemv && dtype == VT_BF16 && (d % 128) == 0 &&
        (d <= vt::kMfmaSmallMaxD || (n >= vt::kMfmaSmallManyRows && d <= vt::kMfmaSmallMaxDManyRows)) &&
        (n >= 2 || d <= vt::kMfmaSmallMaxDOneRow) && n <= vt::kGemvMaxN) {
        auto feasible = [&](int KS, int NW) {
            if (NW < KS || NW % KS != 0 || NW > vt::kMfmaMaxWaves) return false;
            const int tr = 16 * (NW / KS);
            const int tiles = (k + tr - 1) / tr;
            if (tiles < (KS == 4 ? vt::kMfmaSmallMinTiles32 : vt::kMfmaSmallMinTiles) * CUS / vt::kStepMaxBlocks || tiles > CUS)
                return false;
            // (the split also needs all of h in LDS at once: d <= 4096)
            if (KS > 1 && ((d / 128) % KS != 0 || m > vt::kRowSelectMinL || d > vt::kMfmaSmallMaxD)) return false;
            if (NW != vt::kStepWaves) {
                // another number of waves: all of h in LDS beside their staging buffers, fetched in one go
                if (vt::mfma_stage_bytes(NW) + 8 * ((size_t)d * 2 + 16) > (size_t)vt::kMaxDynamicLds) return false;
                if ((size_t)d > (size_t)vt::kMfmaChunkPieces * NW * 64) return false;
            }
            return true;
        };
        const int R = (k + CUS - 1) / CUS;                                    // rows per tile for one tile per CU
        const int G = (R + 15) / 16;                                          // ... in 16-row groups
        if (R > vt::kMfmaTileRows && R <= vt::kMfmaTileRows + 16 && (d % 1024) == 0 && (d % 2048) != 0 &&
            d <= vt::kMfmaSmallMaxD) {
            // 129 .. 144 rows per tile -- the paper's own trimmed sizes, k = 32959 .. 35010 -- : eight waves with 16
            // rows each and the rows past the 128th as one more group whose columns the eight waves share; the
            // tile is exactly R rows, so all 256 CUs stream equal shares (k = 32975, d = 3072: n = 8 40.1 us against
            // 41.4 with nine waves on 229 CUs and 41.8 on the small-n kernel, n = 1 37.0 / 37.4 / 38.9).  Rows a
            // multiple of 2 KiB long lose on it (d = 4096: 54.0 / 51.4 / 51.7 us, d = 2048: 30.1 / 27.5 / 29.1) and
            // take nine waves.
            ksplit = 1;
            nwaves = vt::kStepWaves;
            extra_rows = R - vt::kMfmaTileRows;
        }
        // more or fewer waves than eight where that measured faster than the choices below (n = 8, d = 3072:
        // k = 40000, ten waves: 46.4 against 47.5 us; 49152, twelve: 53.6 / 55.1; 20000, five groups of two: 29.1 / 29.7;
        // six groups of two measured slower; nine waves: see above)
        if (ksplit == 0 && G == 9 && feasible(1, G)) {
            ksplit = 1;
            nwaves = G;
        }
        if (ksplit == 0 && G >= 10 && feasible(1, G)) {
            ksplit = 1;
            nwaves = G;
        }
        // six waves of 16 rows (k = 20481 .. 24576: 214 - 256 tiles instead of 160 - 192 of 128 rows) pay for up to 4
        // hidden rows, seven for one (k = 22786, d = 3072: n = 1 27.4 against 28.2 us, n = 2 27.5 / 28.4, n = 4 30.8 /
        // 31.2, n = 8 32.2 / 31.7; d = 2048, n = 1: 20.6 / 21.9; k = 26000, n = 1: 29.9 / 30.1, n = 2: a tie)
        if (ksplit == 0 && ((G == 6 && n <= 4) || (G == 7 && n == 1)) && feasible(1, G)) {
            ksplit = 1;
            nwaves = G;
        }
        if (ksplit == 0 && G == 5 && feasible(2, 10)) {
            ksplit = 2;
            nwaves = 10;
        }
        // otherwise eight waves and the tile that fills the chip best
        for (int KS = 1; KS <= 4 && ksplit == 0; KS *= 2) {
            if (feasible(KS, vt::kStepWaves)) {
                ksplit = KS;
                nwaves = vt::kStepWaves;
            }
        }
    }
    if (fixed.nwaves != 0) {
        // (the same limits as above: whole units per wave, the kernel's own epilogue, all of h in LDS at once)
        ksplit = 0;
        nwaves = vt::kStepWaves;
        extra_rows = 0;
        if (dtype == VT_BF16 && (d % 128) == 0 && d <= vt::kMfmaSmallMaxD && n <= vt::kGemvMaxN && m <= vt::kRowSelectMinL &&
            (d / 128) % fixed.ksplit == 0 && (fixed.ksplit == 1 || fixed.nwaves == vt::kStepWaves) &&
            fixed.nwaves >= vt::kStepWaves && fixed.nwaves <= vt::kMfmaMaxWaves &&
            vt::mfma_stage_bytes(fixed.nwaves) + 8 * ((size_t)d * 2 + 16) <= (size_t)vt::kMaxDynamicLds &&
            (size_t)d <= (size_t)vt::kMfmaChunkPieces * fixed.nwaves * 64) {
            ksplit = fixed.ksplit;
            nwaves = fixed.nwaves;
        } else {
            return p;
        }
    }
    const bool prefer_mfma = ksplit != 0;
    if (n <= vt::kGemvMaxN && !prefer_mfma) {
        const int NP = n <= 1 ? 1 : (n <= 2 ? 2 : (n <= 4 ? 4 : 8));
        const int epc = dtype == VT_BF16 ? 8 : 4;
        const int CT = (d + 64 * epc - 1) / (64 * epc);
        static const int cs_bf16[] = {1, 2, 3, 4, 6};
        static const int cs_f32[] = {1, 2, 4};
        const int *cs_set = dtype == VT_BF16 ? cs_bf16 : cs_f32;
        const int ncs = dtype == VT_BF16 ? 5 : 3;
        for (int S = 1; S <= vt::kStepWaves && !p.gemv; S *= 2) {
            const int need = (CT + S - 1) / S;
            for (int q = 0; q < ncs; ++q) {
                const int CS = cs_set[q];
                if (CS >= need && CS * NP <= 24) {
                    const size_t tile = (size_t)S * NP * p.tpitch * sizeof(float);
                    if (tile <= 96 * 1024) {
                        p.gemv = true;
                        p.NP = NP;
                        p.CS = CS;
                        p.S = S;
                        // + 2 KiB per wave behind the tile: candidate keys of the epilogue's threshold selection
                        p.lds = ((tile + 15) & ~(size_t)15) + (size_t)vt::kStepWaves * 256 * sizeof(unsigned long long);
                    }
                    break;
                }
            }
        }
    }
    if (!p.gemv) {
        // larger n or d: the matrix-core path (bf16, d a multiple of 128, n <= 256)
        if (dtype != VT_BF16 || (d % 128) != 0 || n > vt::kMfmaMaxN) return p;
        if (n > vt::kGemvMaxN) {
            plan_many_rows(p, n, k, d, m);
        } else {
            const bool var_waves = prefer_mfma && nwaves != vt::kStepWaves;
            const size_t stage = vt::mfma_stage_bytes(var_waves ? nwaves : vt::kStepWaves);
            // the hidden rows occupy 8 rows of LDS (the other half of the 16-row operand repeats them)
            const size_t hrows = 8;
            const size_t hmax = ((size_t)vt::kMaxDynamicLds - stage) / hrows;
            if (hmax < 272) return p;
            int KC = (int)(((hmax - 16) / 2) / 128) * 128;
            const int kc_regs =
                (int)((vt::kMfmaChunkPieces * (var_waves ? nwaves : vt::kStepWaves) * 64 * 16) / (hrows * 2) / 128 * 128);
            if (KC > kc_regs) KC = kc_regs;   // the chunk must fit the register prefetch
            if (KC >= d) {
                KC = d;
            } else {
                // several chunks: near-equal sizes (d = 2560: 2304 + 256 -> 1536 + 1024), every chunk but the
                // last a multiple of the kernel's prefetch depth in 128-column units
                const int U = d / 128, P = vt::kMfmaPrefetchUnits;
                const int umax = KC / 128 / P * P;
                if (umax < P) return p;
                const int nch = (U + umax - 1) / umax;
                KC = (((U + nch - 1) / nch + P - 1) / P * P) * 128;
            }
            p.mfma = true;
            p.NT = 1;
            p.KC = KC;
            p.hpitch = KC * 2 + 16;
            p.ksplit = (prefer_mfma && KC == d) ? ksplit : 1;
            p.nwaves = (prefer_mfma && KC == d) ? nwaves : vt::kStepWaves;
            p.extra_rows = (prefer_mfma && KC == d) ? extra_rows : 0;
            p.row_groups = p.nwaves / p.ksplit;
            const int tile_rows = 16 * p.row_groups + p.extra_rows;
            p.nlists = fixed.nwaves != 0 ? fixed.nlists : (k + tile_rows - 1) / tile_rows;
            p.L = m < tile_rows ? m : tile_rows;
            p.nblocks = p.nlists;
            // a wave per row in the epilogue: a candidate key per tile row and wave, not below 8 KiB
            const int tp = (p.extra_rows != 0 ? vt::kMfmaTileRows + 16 : p.nwaves == vt::kStepWaves ? vt::kMfmaTileRows : tile_rows) + 1;
            const size_t zt = ((size_t)p.ksplit * n * tp * sizeof(float) + 15) & ~(size_t)15;
            const size_t tile =
                (zt > 8192 ? zt : 8192) +
                (size_t)p.nwaves * ((p.nwaves == vt::kStepWaves && p.extra_rows == 0) ? 2 : 3) * 64 * sizeof(unsigned long long) +
                (p.extra_rows != 0 ? (size_t)8 * n * 16 * sizeof(float) : 0);      // + the shared group's partials
            p.lds = stage + hrows * p.hpitch;
            if (tile > p.lds) p.lds = tile;
        }
        if (p.lds > (size_t)vt::kMaxDynamicLds) return p;
        const int group = p.nlists < vt::kStepMaxBlocks ? p.nlists : vt::kStepMaxBlocks;
        p.fin_stage_keys = (group + 1) * p.L;
        const int fc = (int)(vt::kFinalizeLdsBytes / ((size_t)p.fin_stage_keys * sizeof(unsigned long long)));
        // Many tokens per row: the candidate lists cost L selection rounds per tile; the kernel stores its logits instead
        // and a workgroup per hidden row finishes the step (measured: 12 or more tokens with up to 8 hidden rows; above,
        // see stores_logits()).  Always when the lists of a row no longer fit the merge's LDS staging.
        p.row_select = fc < 1 || (n > vt::kGemvMaxN ? stores_logits(n, p.L, 16 * p.row_groups + p.extra_rows)
                                                    : p.L > vt::kRowSelectMinL);
        // one hidden row per workgroup: n <= 256 rows spread over as many CUs, and a merging wave has its
        // SIMD to itself (the selection rounds are bound by instruction issue)
        p.fin_lds = (size_t)p.fin_stage_keys * sizeof(unsigned long long);
        // (Merging in the main kernel's last workgroup to arrive was measured for n <= 8: 41.1 against 39.9 us --
        // eight merge workgroups on eight CUs beat eight waves on one; and for n <= 3 once more: 39.6 against 35.3.)
    } else {
        // many tokens per row: the selection rounds of the fused tail grow with L in every workgroup and the merge
        // stages B * L keys per row; the per-row tail on stored logits takes over (measured crossover)
        p.row_select = p.L > vt::kGemvRowSelectBase - n / 2;
    }

    size_t off = kTicketBytes;
    p.off_lse = off;
    off = round_up(off + (size_t)n * sizeof(float), 256);
    const size_t pms_bytes = round_up((size_t)p.nblocks * n * sizeof(unsigned long long), 256);
    const size_t key_bytes = round_up((size_t)n * p.nblocks * p.L * sizeof(unsigned long long), 256);
    const size_t zbuf_bytes = round_up((size_t)n * k * sizeof(float), 256);
    p.off_pms = off;
    p.off_pkeys = off + pms_bytes;
    p.off_zbuf = off;
    if (p.mfma && n > vt::kGemvMaxN && p.row_select) {
        // the stored logits lie where the lists would (up to 8 tokens per row the larger of the two is reserved: with
        // fewer hidden rows the same workspace serves lists)
        size_t room = zbuf_bytes;
        if (m <= vt::kRowSelectMinLManyRows && pms_bytes + key_bytes > room) room = pms_bytes + key_bytes;
        off += p.list_room > room ? p.list_room : room;
    } else {
        off += p.list_room > pms_bytes + key_bytes ? p.list_room : pms_bytes + key_bytes;
        p.off_zbuf = off;
        if (p.row_select) off += zbuf_bytes;
    }
    if (p.wide && vt::packs_h(p.NT / 4, n, d)) {
        p.off_hpack = off;
        off = round_up(off + (size_t)d * p.NT * 32, 256);
    }
    p.bytes = off;
    p.ok = true;
    return p;
}

// Parts of a row of stored logits: what a wave of the matrix-core kernels for more than 8 hidden rows holds of it (16 logits, or half
// of a tile), 64 logits of a tile up to 8.  False: too many.
bool row_parts(StepPlan &p, int n, int k) {
    p.extra_rows = (p.extra_rows + 3) / 4 * 4;      // (groups of four logits do not reach into the next tile)
    const int tile_rows = p.gemv ? p.rpb : 16 * p.row_groups + p.extra_rows, tiles = (k + tile_rows - 1) / tile_rows;
    p.part_rows = n <= vt::kGemvMaxN ? vt::kFewRowsPart : p.wide ? 8 * p.row_groups : 16;
    p.per_tile = (tile_rows + p.part_rows - 1) / p.part_rows;
    p.parts = (tiles - 1) * p.per_tile + (k - (tiles - 1) * tile_rows + p.part_rows - 1) / p.part_rows;
    if (!p.gemv) p.nlists = p.nblocks = tiles;
    if (p.parts <= vt::kRowPartsMax) return true;
    p.parts = 0;
    return false;
}
// The layout of a workspace for logits in `splits` slices.
void lay_out_stored(StepPlan &p, int n, int k, int d) {
    size_t off = round_up(p.off_lse + (size_t)n * sizeof(float), 256);
    if (p.parts != 0) {
        p.off_pms = off;
        const size_t parts = n <= vt::kGemvMaxN ? (size_t)p.parts : (size_t)k / 14 + 32;      // (of the smallest tiles)
        off = round_up(off + n * parts * sizeof(unsigned long long), 256);
    }
    p.off_zbuf = off;
    off = round_up(off + (size_t)p.splits * n * slice_pitch(k) * sizeof(float), 256);
    p.off_hpack = 0;
    if (p.wide && vt::packs_h(p.NT / 4, n, d)) {
        p.off_hpack = off;
        off = round_up(off + (size_t)d * p.NT * 32, 256);
    }
    p.bytes = off;
}

// Up to 8 hidden rows parts pay where a row's whole reading takes longer than a second trip (whole / by parts: n = 2, d = 3072, m = 16,
// k = 16000 24.0 / 24.2 us, 18000 28.8 / 28.3, 32975 43.0 / 38.2; n = 4, d = 1024, m = 64, k = 30000 22.4 / 22.6, k = 3000, m = 16 9.6 / 10.9;
// n = 4, k = 79094, d = 2048, m = 16 66.7 / 57.4)
bool few_rows_by_parts(int k, int m) { return k > (m <= 16 ? vt::kRowSelectWhole / 2 : vt::kRowSelectWhole); }
// More of them, where a thread of row_select_kernel has eight logits at most: parts against whole rows of eight 1.60 for k = 700, d = 1024, m = 33 and
// 64 (m = 10 1.06), 1.28 for k = 1293, n = 9, m = 64, 1.0 to 1.17 for k = 2048 and 3000, 1.0 to 1.05 for k = 4608, n <= 64 and k = 7001 0.98 to 1.04, k = 7600
// 0.89 to 1.06, k = 8190, n = 64 0.97, n = 81 and k = 6138 0.92 to 1.0; n > 64 off multiples of four, logits one by one, m = 10 to 33 0.90 to
// 1.04 (n = 256, k = 4501), m = 64 0.96 to 2.1.
bool whole_rows_pay(int n, int k, int m) {
    if (n <= vt::kRowsKernelMaxN) return k <= 7168;
    return k <= 4608 && (m > 40 || k % 4 == 0);
}
// Slices of the columns beside tiles of 16 g rows: as many as fill the chip, of 256 columns and more; 1: none.  Up to d = 8192, the
// longest rows measured.
constexpr int kSliceGroups[] = {4, 8, 10};
int slices_of(int k, int d, int g) {
    const int tiles = (k + 16 * g - 1) / (16 * g), S = round_workgroups() / tiles;
    return S >= 2 && k <= vt::kRowSelectSlices && d <= 8192 && d / 128 >= 2 * S ? S : 1;
}

// The same step with its logits stored, and the columns cut into slices where that pays: larger tiles then (each hidden row is
// read once per tile, so small tiles of many hidden rows are bound by reading h), a workgroup per tile and slice, and
// row_select_kernel adds the partial logits up.  ok = false: the plan itself is the better one.
// The costs are microseconds, fitted to 945 shapes (n = 16 .. 256, k = 4300 .. 20000, d = 1024 .. 8192, m = 4, 8, 16; 5 %
// off on average): W at a CU's share of the HBM rate, h from the L2, and the tail.  Two slices gain least and are the first to
// lose on another card.  Up to 64 rows a tree level is fused behind the merge of lists, which stored logits give up: there
// the slices have to gain what its launch costs.  Measured (us, plan / slices): n = 224, k = 4300, d = 8192 81.9 / 36.5,
// k = 10000, d = 4096 54.7 / 39.3, n = 160, k = 6500, d = 4096 40.7 / 30.2, n = 100, k = 4300, d = 2048 21.9 / 18.2, n = 64, k = 4300,
// d = 4096 24.1 / 18.8; what the rule leaves: n = 100, k = 14000, d = 4096 37.1 / 39.3, n = 32, k = 10000, d = 4096 22.9 / 24.9.
StepPlan plan_stored(const StepPlan &whole, int n, int k, int d, int m) {
    StepPlan p = whole;
    p.ok = false;
    if (whole.ok && n <= vt::kGemvMaxN && whole.row_select && few_rows_by_parts(k, m) && row_parts(p, n, k)) {
        lay_out_stored(p, n, k, d);
        p.ok = true;
        return p;
    }
    if (!whole.ok || !whole.mfma || n <= vt::kGemvMaxN || (k > vt::kRowSelectWhole && !whole.row_select)) return p;
    const int CUS = round_workgroups();
    const bool few = n <= vt::kRowsKernelMaxN;
    const int hrows = whole.wide ? 16 * whole.NT : whole.NT * 16;      // hidden rows of the tiles
    const int rows = 16 * whole.row_groups + whole.extra_rows, rounds = (whole.nlists + CUS - 1) / CUS;
    // Lists of up to 8 tokens take a tile's epilogue 5 to 10 us from 129 hidden rows on, and the logits of rows of up to 32768 with their
    // parts less (lists / parts: n = 217, k = 26262, d = 3072, m = 4 61.4 / 57.5 us, n = 70, k = 26000, d = 1024, m = 8 22.5 / 20.4).  Of 5 to 7
    // tokens they do from 92, 83 and 74 rows on, on small tiles from the first (n = 92, k = 10000, d = 1024, m = 5 18.7 / 16.6), and of up to
    // 4 where the hidden rows fill their tiles (n = 119, k = 19000, m = 3 and 4 1 %, m = 1 and 2 a tie, on tiles of 48 3 %; n = 136 -2 to 1 %,
    // n = 150 2 to 5 %; n = 110, k = 30000, d = 1024, m = 3 -3 %, n = 124, k = 21867, d = 1536, m = 2 26.7 / 27.4).  Tiles on nearly all CUs
    // store later than fewer of them (n = 96, d = 1024, m = 6: 240 tiles 22.3 / 22.5, 241 22.2 / 23.1; n = 128, k = 32768, m = 4 23.6 / 25.1, m = 8
    // 26.5 / 25.1; n = 160, k = 28000, d = 8192, m = 2 112.2 / 114.9, n = 180, d = 1536 34.9 / 34.4)
    const bool all_cus = whole.nlists > CUS - 16;
    auto parts_pay = [&]() {
        if (m >= vt::kRowSelectMinLManyRows) return true;
        if (all_cus && rows > vt::kMfmaTileRows / 2) return n >= (m <= 4 ? 176 : 145);
        if (m <= 4) return n >= 145 || (!all_cus && n >= 119 && n <= 128 && (m >= 3 || rows <= vt::kMfmaTileRows / 2));
        return n >= 65 + 9 * (vt::kRowSelectMinLManyRows - m) || rows < vt::kMfmaTileRows;
    };
    const bool by_parts = whole.row_select || (!few && parts_pay());
    const double as_planned = 9.0 + rounds * ((double)rows * d / 18e3 + (double)hrows * d / 38e3) +
                              (!whole.row_select ? rounds * 0.03 * n - 0.6 : std::max(k * (2.2e-6 * n + 3.5e-5), few ? 1.5 : 0.0));
    double best = as_planned;
    for (int g : kSliceGroups) {
        // (d = 1024: parts / slices n = 194, k = 5070, m = 4 18.6 / 20.1 us, n = 135, k = 4461, m = 1 16.5 / 16.7)
        if ((few && g > 8) || (by_parts && d <= 1024)) continue;
        const int S = slices_of(k, d, g);
        if (S < (few ? 4 : g > 8 ? 3 : 2)) continue;
        const double t = 10.3 + (double)16 * g * d / S / 19e3 + (double)hrows * d / S / 34e3 + (double)S * k * (1.8e-6 * n + 6.5e-5);
        if (t < best && t < (S == 2 ? 0.90 : 0.93) * as_planned && (!few || t < as_planned - 4.0)) {
            best = t;
            p.row_groups = g;
            p.splits = S;
        }
    }
    if (p.splits > 1) {
        p.extra_rows = 0;
        p.twin = false;
    } else if (!by_parts || (whole.row_select && whole_rows_pay(n, k, m)) || !row_parts(p, n, k)) {
        return p;      // (in one piece only with the (max, sum-exp) of the rows' parts)
    }
    p.instead_of_lists = !whole.row_select;
    p.row_select = true;
    p.list_room = 0;
    cut_many_rows(p, n, k, m);
    lay_out_stored(p, n, k, d);
    p.ok = p.lds <= (size_t)vt::kMaxDynamicLds;
    return p;
}

// Hidden rows handled per launch group.  A step whose n no single plan covers (more than 256 rows; more
// than 8 rows in fp32 or with d not a multiple of 128; very long fp32 rows) runs as consecutive groups
// of `chunk` rows, each streaming W_trim again -- slower, but every shape has an answer.
// Tree level fused behind the step (n <= 8 path only): null members = none.
struct TreeFuse {
    const float *cum = nullptr;
    int K = 0;
    int32_t *parent = nullptr;
    int32_t *token = nullptr;
    float *score = nullptr;
    // rows picked out of a larger batch (small-n kernel without the per-row tail only): hidden row i of the
    // group is row (row_pack >> 8 i) & 255 of h and of the outputs
    unsigned long long row_pack = 0;
    int indexed = 0;
};
int run_step_group(const void *h, int n, const void *W_trim, int w_type, int k, int d, const int32_t *map, int m,
                   int32_t *out_ids, float *out_logp, float *out_lse, float *out_logp_full, void *ws, size_t ws_bytes,
                   hipStream_t st, const TreeFuse &tf);

int pick_chunk(int n, int k, int d, int m, int dtype);
int step_chunk(int n, int k, int d, int m, int dtype);      // the same, from what is kept of the last shapes

// several heads' tiles in one launch (defined with the launch code below)
constexpr int kNotFused = -1;
StepPlan plan_heads_fused(int n, int d, const int32_t *k, const int *used, int nused, int m, int w_type);
int run_step_heads_fused(const void *h, int n, int d, const void *const *W_trim, int w_type, const int32_t *k,
                         const int32_t *const *map, int n_heads, const int32_t *head_of_row, const vt::RowList *rows, int m,
                         int32_t *out_ids, float *out_logp, float *out_lse, void *ws, size_t ws_step_bytes, hipStream_t st);

// All n rows of a validated step: consecutive launch groups of `chunk` rows on one workspace.
int run_step_rows(const void *h, int n, const void *W_trim, int w_type, int k, int d, const int32_t *map, int m,
                  int32_t *out_ids, float *out_logp, float *out_lse, float *out_logp_full, void *ws, size_t ws_bytes, hipStream_t st) {
    const int chunk = step_chunk(n, k, d, m, w_type);
    if (chunk == 0) return VT_ERR_SHAPE;
    const size_t row_bytes = (size_t)d * elem_size(w_type);
    for (int i0 = 0; i0 < n; i0 += chunk) {
        const int nc = n - i0 < chunk ? n - i0 : chunk;
        const int rc = run_step_group(static_cast<const char *>(h) + (size_t)i0 * row_bytes, nc, W_trim, w_type, k, d, map,
                                      m, out_ids + (size_t)i0 * m, out_logp + (size_t)i0 * m,
                                      out_lse ? out_lse + i0 : nullptr,
                                      out_logp_full ? out_logp_full + (size_t)i0 * k : nullptr, ws, ws_bytes, st, TreeFuse{});
        if (rc != VT_OK) return rc;
    }
    return VT_OK;
}

// Workspace a step of up to n rows on a head of k rows may need, whatever the element type.  A workspace for n rows serves
// a step of fewer (from 8 on) too, whose kernel and tiles may be others: inside a kernel's range the size grows with the rows
// (list_room takes care of the one choice of tiles that the rows decide), so the ends of the ranges below n are looked at.
size_t step_ws_bytes(int n, int k, int d, int m) {
    size_t b = n > vt::kMfmaMaxN          ? step_ws_bytes(vt::kMfmaMaxN, k, d, m)
               : n > vt::kRowsKernelMaxN ? step_ws_bytes(vt::kRowsKernelMaxN, k, d, m)
               : n > 32                   ? step_ws_bytes(32, k, d, m)
               : n > vt::kGemvMaxN       ? step_ws_bytes(vt::kGemvMaxN, k, d, m)
                                          : 0;
    for (int dtype : {VT_BF16, VT_F32}) {
        const int c = pick_chunk(n, k, d, m, dtype);
        if (c == 0) continue;
        for (bool force_gemv : {false, true}) {      // either kernel may serve a group of up to 8 rows
            const StepPlan p = plan_step(c, k, d, m, dtype, force_gemv);
            if (p.ok && p.bytes > b) b = p.bytes;
            if (n % c != 0) {
                const StepPlan r = plan_step(n % c, k, d, m, dtype, force_gemv);
                if (r.ok && r.bytes > b) b = r.bytes;
            }
        }
    }
    return b;
}

// The same with room for plan_stored()'s plans, of n rows and of fewer (slices come and go with the rows).  What a program asks for; a
// step accepts step_ws_bytes(), the size that earlier versions returned.
// Not all of up to 256 row counts are planned, but from n rows down until what is left cannot be more, whatever its slices: n = 256,
// k = 32768, d = 8192, m = 16 27.8 -> 1.6 us, k = 4300, d = 4096, m = 8 25.5 / 19.6, n = 64, k = 32768, m = 8 3.0 / 0.9 (step_ws_bytes() alone
// 0.4 to 0.9).
size_t plan_full_step_ws_bytes(int n, int k, int d, int m) {
    size_t b = step_ws_bytes(n, k, d, m);
    if (b == 0) return 0;
    auto room_for = [&](int r, int dtype) {
        const StepPlan p = plan_stored(plan_step(r, k, d, m, dtype), r, k, d, m);
        if (p.ok && p.bytes > b) b = p.bytes;
    };
    for (int r = n < vt::kGemvMaxN ? n : vt::kGemvMaxN; r >= 1 && few_rows_by_parts(k, m); --r) {
        room_for(r, VT_BF16);
        room_for(r, VT_F32);
    }
    int most = 1;
    for (int g : kSliceGroups) {
        const int S = slices_of(k, d, g);
        if (S > most) most = S;
    }
    // (lay_out_stored()'s, with room for every rounding)
    auto at_most = [&](int r) {
        const size_t row = sizeof(float) + ((size_t)k / 14 + 32) * sizeof(unsigned long long) + (size_t)most * slice_pitch(k) * sizeof(float);
        return (size_t)vt::kTicketBytes + r * row + (size_t)d * 512 + 5 * 256;
    };
    // (up to 8 tokens: a smaller batch keeps lists, unless it has the four slices that up to 64 rows ask for)
    const int fewest = m > vt::kRowSelectMinLManyRows ? vt::kGemvMaxN
                       : k > vt::kRowSelectWhole      ? vt::kRowSelectMinWork / m - 1
                       : most < 4                     ? vt::kRowsKernelMaxN
                                                      : vt::kGemvMaxN;
    for (int r = n < vt::kMfmaMaxN ? n : vt::kMfmaMaxN; r > fewest && at_most(r) > b; --r) room_for(r, VT_BF16);
    return b;
}
size_t full_step_ws_bytes(int n, int k, int d, int m) {
    // programs repeat their few shapes (a step without a workspace of its own asks in every call): the last answers are kept per host thread
    struct Size {
        int n = 0, k = 0, d = 0, m = 0;
        size_t bytes = 0;
    };
    constexpr unsigned kKept = 64;
    static thread_local Size kept[kKept];
    Size &s = kept[((unsigned)n * 7u + (unsigned)m * 3u + (unsigned)k + (unsigned)d / 128u) % kKept];
    if (s.n != n || s.k != k || s.d != d || s.m != m) s = Size{n, k, d, m, plan_full_step_ws_bytes(n, k, d, m)};
    return s.bytes;
}

// Layout of a multi-head workspace: the step workspace first, then the staged hidden rows and the staged results
// of one head's rows.
struct MultiLayout {
    size_t off_h = 0, off_ids = 0, off_logp = 0, off_lse = 0, bytes = 0;
};
MultiLayout multi_layout(int n, int d, const int32_t *k, int n_heads, int m, bool full) {
    // consecutive steps repeat their shapes: the last answer is kept per host thread
    struct Key {
        int n = 0, d = 0, m = 0, n_heads = 0;
        int32_t k[VT_MAX_HEADS] = {};
        MultiLayout L;
    };
    static thread_local Key kept[2];
    Key &last = kept[full ? 1 : 0];
    if (last.n == n && last.d == d && last.m == m && last.n_heads == n_heads) {
        bool same = true;
        for (int hd = 0; hd < n_heads; ++hd) same = same && last.k[hd] == k[hd];
        if (same) return last.L;
    }
    MultiLayout L;
    size_t step = 0;
    for (int hd = 0; hd < n_heads; ++hd) {
        // a head may receive any number of the n rows, and the plan (hence its workspace) changes with it
        for (int nn = 1; nn <= n; ++nn) {
            const size_t b = step_ws_bytes(nn, k[hd], d, m);
            if (b > step) step = b;
        }
        const size_t b = full ? full_step_ws_bytes(n, k[hd], d, m) : 0;
        if (b > step) step = b;
    }
    // ... and several heads' tiles in one launch: at most one tile per CU, whatever their shape
    if (n <= vt::kGemvMaxN) {
        for (int nw = vt::kStepWaves; nw <= vt::kMfmaMaxWaves; ++nw) {
            for (int ks = 1; ks <= (nw == vt::kStepWaves ? 4 : 1); ks *= 2) {
                FixedTiles ft;
                ft.nwaves = nw;
                ft.ksplit = ks;
                ft.nlists = vt::kStepMaxBlocks;
                const StepPlan p = plan_step_impl(n, vt::kStepMaxBlocks * 16 * (nw / ks), d, m, VT_BF16, false, ft);
                if (p.ok && p.bytes > step) step = p.bytes;
            }
        }
    }
    size_t off = round_up(step, 256);
    L.off_h = off;
    off = round_up(off + (size_t)n * d * sizeof(float), 256);      // sized for the wider element type
    L.off_ids = off;
    off = round_up(off + (size_t)n * m * sizeof(int32_t), 256);
    L.off_logp = off;
    off = round_up(off + (size_t)n * m * sizeof(float), 256);
    L.off_lse = off;
    off = round_up(off + (size_t)n * sizeof(float), 256);
    L.bytes = off;
    last.n = n;
    last.d = d;
    last.m = m;
    last.n_heads = n_heads;
    for (int hd = 0; hd < n_heads; ++hd) last.k[hd] = k[hd];
    last.L = L;
    return L;
}

int pick_chunk(int n, int k, int d, int m, int dtype) {
    if (plan_step(n, k, d, m, dtype).ok) return n;
    for (int c : {256, 8, 4, 2, 1}) {
        if (c < n && plan_step(c, k, d, m, dtype).ok && (n % c == 0 || plan_step(n % c, k, d, m, dtype).ok)) return c;
    }
    return 0;
}

// What a step of one shape comes to: the groups its rows run in, the workspace it asks for, the plan of a whole group.  A step is
// asked three times and more -- size check, launch, and a program repeats its few shapes -- at 0.06 us a plan and eight plans a call,
// so the last answers are kept per host thread.
struct StepShape {
    int n = 0, k = 0, d = 0, m = 0, dtype = -1;
    int chunk = 0;
    size_t ws_bytes = 0;       // that a step asks for; with more it may run as plan_stored() has it
    StepPlan plan, stored;     // of `chunk` rows
    size_t stored_bytes = 0;   // the most that a plan_stored() of its groups takes: of `chunk` rows, of what is left of n
    bool is(int n_, int k_, int d_, int m_, int dtype_) const { return n == n_ && k == k_ && d == d_ && m == m_ && dtype == dtype_; }
    const StepPlan &with(size_t bytes) const { return stored.ok && stored.bytes <= bytes ? stored : plan; }
};
const StepShape &step_shape(int n, int k, int d, int m, int dtype) {
    constexpr unsigned kKept = 8;
    static thread_local StepShape kept[kKept];
    StepShape &s = kept[((unsigned)n * 7u + (unsigned)m * 3u + (unsigned)k + (unsigned)d / 128u + (unsigned)dtype) % kKept];
    if (!s.is(n, k, d, m, dtype)) {
        s.dtype = -1;
        s.chunk = pick_chunk(n, k, d, m, dtype);
        s.ws_bytes = step_ws_bytes(n, k, d, m);
        s.plan = s.chunk != 0 ? plan_step(s.chunk, k, d, m, dtype) : StepPlan{};
        s.stored = plan_stored(s.plan, s.chunk, k, d, m);
        s.stored_bytes = s.stored.ok ? s.stored.bytes : 0;
        if (s.chunk != 0 && n % s.chunk != 0) {
            const StepPlan rest = plan_stored(plan_step(n % s.chunk, k, d, m, dtype), n % s.chunk, k, d, m);
            if (rest.ok && rest.bytes > s.stored_bytes) s.stored_bytes = rest.bytes;
        }
        s.n = n;
        s.k = k;
        s.d = d;
        s.m = m;
        s.dtype = dtype;
    }
    return s;
}
int step_chunk(int n, int k, int d, int m, int dtype) { return step_shape(n, k, d, m, dtype).chunk; }

}  // namespace

extern "C" {

const char *vt_status_string(int status) {
    switch (status) {
        case VT_OK: return "VT_OK";
        case VT_ERR_NULL: return "VT_ERR_NULL: a required pointer is NULL";
        case VT_ERR_SHAPE: return "VT_ERR_SHAPE: a size is out of range";
        case VT_ERR_DTYPE: return "VT_ERR_DTYPE: unknown or unsupported element or index type";
        case VT_ERR_ALIGN: return "VT_ERR_ALIGN: pointer or row size not 16-byte aligned";
        case VT_ERR_WORKSPACE: return "VT_ERR_WORKSPACE: workspace missing, misaligned or too small";
        case VT_ERR_DEVICE: return "VT_ERR_DEVICE: a HIP call failed";
        default: return "unknown vt_status";
    }
}

const char *vt_last_device_error(void) { return hipGetErrorString(g_last_hip_error); }

// ------------------------------------------------------------------ Algorithm 1
size_t vt_count_tokens_ws_bytes(int32_t V, int64_t n_ids) {
    if (V <= 0 || n_ids < 0) return 0;
    return round_up(vt::hist_scratch_bytes(V, n_ids), 256);
}

int vt_count_tokens(const void *ids, int id_type, int64_t n_ids, int32_t V, int64_t *counts,
                    uint64_t *n_invalid, void *ws, size_t ws_bytes, void *stream) {
    if (id_type != VT_I32 && id_type != VT_I64) return VT_ERR_DTYPE;
    if (V <= 0 || n_ids < 0 || n_ids > ((int64_t)1 << 37)) return VT_ERR_SHAPE;
    if (counts == nullptr || (ids == nullptr && n_ids > 0)) return VT_ERR_NULL;
    if (n_ids == 0) return VT_OK;
    const size_t idb = id_type == VT_I64 ? 8 : 4;
    if (!aligned(ids, idb) || !aligned(counts, 8) || (n_invalid && !aligned(n_invalid, 8))) return VT_ERR_ALIGN;
    if (ws == nullptr || !aligned(ws, 256) || ws_bytes < round_up(vt::hist_min_scratch_bytes(V, n_ids), 256)) return VT_ERR_WORKSPACE;
    (void)hipGetLastError();
    return device_status(vt::launch_count_tokens(ids, id_type == VT_I64, n_ids, V,
                                                 reinterpret_cast<long long *>(counts),
                                                 reinterpret_cast<unsigned long long *>(n_invalid),
                                                 ws, ws_bytes, static_cast<hipStream_t>(stream)));
}

// ------------------------------------------------------------------ Eq. 1
size_t vt_build_trimmed_head_ws_bytes(int32_t V, int32_t d, int32_t k) {
    (void)d;
    (void)k;
    // the larger of: selection histograms (id order), buffers of a sort of all V (count, id) pairs (rank order)
    const size_t a = vt::select_scratch_bytes(V > 0 ? V : 1), b = vt::rank_sort_scratch_bytes(V > 0 ? V : 1);
    return 256 + round_up(a > b ? a : b, 256);
}

int vt_build_trimmed_head(const int64_t *counts, int32_t V, const void *W, int w_type, int32_t d, int32_t k,
                          int32_t *map, void *W_trim, void *ws, size_t ws_bytes, void *stream) {
    if (w_type != VT_F32 && w_type != VT_BF16) return VT_ERR_DTYPE;
    if (V <= 0 || d <= 0 || k < 1 || k > V) return VT_ERR_SHAPE;
    if (counts == nullptr || map == nullptr) return VT_ERR_NULL;
    if ((W == nullptr) != (W_trim == nullptr)) return VT_ERR_NULL;
    const size_t row_bytes = (size_t)d * elem_size(w_type);
    if (!aligned(counts, 8) || !aligned(map, 4)) return VT_ERR_ALIGN;
    if (W != nullptr && ((row_bytes & 15) != 0 || !aligned(W, 16) || !aligned(W_trim, 16))) return VT_ERR_ALIGN;
    if (ws == nullptr || !aligned(ws, 256) || ws_bytes < vt_build_trimmed_head_ws_bytes(V, d, k))
        return VT_ERR_WORKSPACE;
    (void)hipGetLastError();
    hipStream_t st = static_cast<hipStream_t>(stream);
    vt::launch_select_topk(reinterpret_cast<const long long *>(counts), V, k, static_cast<char *>(ws) + 256, map, st);
    if (W != nullptr) vt::launch_gather_rows(W, row_bytes, map, k, W_trim, st);
    return launch_status();
}

int vt_build_trimmed_head_by_rank(const int64_t *counts, int32_t V, const void *W, int w_type, int32_t d, int32_t k,
                                  int32_t *map, void *W_trim, void *ws, size_t ws_bytes, void *stream) {
    if (w_type != VT_F32 && w_type != VT_BF16) return VT_ERR_DTYPE;
    if (V <= 0 || d <= 0 || k < 1 || k > V) return VT_ERR_SHAPE;
    if (counts == nullptr || map == nullptr) return VT_ERR_NULL;
    if ((W == nullptr) != (W_trim == nullptr)) return VT_ERR_NULL;
    const size_t row_bytes = (size_t)d * elem_size(w_type);
    if (!aligned(counts, 8) || !aligned(map, 4)) return VT_ERR_ALIGN;
    if (W != nullptr && ((row_bytes & 15) != 0 || !aligned(W, 16) || !aligned(W_trim, 16))) return VT_ERR_ALIGN;
    if (ws == nullptr || !aligned(ws, 256) || ws_bytes < vt_build_trimmed_head_ws_bytes(V, d, k))
        return VT_ERR_WORKSPACE;
    (void)hipGetLastError();
    hipStream_t st = static_cast<hipStream_t>(stream);
    // the k best ids in rank order are the first k of the full rank order
    vt::launch_rank_sort(reinterpret_cast<const long long *>(counts), V, static_cast<char *>(ws) + 256, map, k, st);
    if (W != nullptr) vt::launch_gather_rows(W, row_bytes, map, k, W_trim, st);
    return launch_status();
}

size_t vt_choose_k_ws_bytes(int32_t V) {
    if (V < 1) return 256;
    return vt::choose_k_ws_bytes(V);
}

int vt_choose_k(const int64_t *counts, int32_t V, int mode, double p, int64_t min_count, int64_t *out, void *ws,
                size_t ws_bytes, void *stream) {
    if (mode != VT_K_TOP_P && mode != VT_K_MIN_COUNT) return VT_ERR_DTYPE;
    if (V <= 0) return VT_ERR_SHAPE;
    if (mode == VT_K_TOP_P && !(p >= 0.0 && p <= 1.0)) return VT_ERR_SHAPE;
    if (counts == nullptr || out == nullptr) return VT_ERR_NULL;
    if (!aligned(counts, 8) || !aligned(out, 8)) return VT_ERR_ALIGN;
    if (ws == nullptr || !aligned(ws, 256) || ws_bytes < vt_choose_k_ws_bytes(V)) return VT_ERR_WORKSPACE;
    (void)hipGetLastError();
    hipStream_t st = static_cast<hipStream_t>(stream);
    vt::launch_choose_k(reinterpret_cast<const long long *>(counts), V, mode, p, (long long)min_count, ws,
                        reinterpret_cast<long long *>(out), st);
    return launch_status();
}

// ------------------------------------------------------------------ Algorithm 2, drafting lines
size_t vt_draft_head_step_ws_bytes(int32_t n, int32_t k, int32_t d, int32_t m) {
    return full_step_ws_bytes(n, k, d, m);      // sized for either element type
}

int vt_draft_head_step_plan(int32_t n, int32_t k, int32_t d, int32_t m, int w_type, char *text, size_t text_bytes) {
    if (w_type != VT_F32 && w_type != VT_BF16) return VT_ERR_DTYPE;
    if (n <= 0 || k <= 0 || d <= 0 || m < 1 || m > k || m > VT_MAX_TOP_M || k > vt::kStepMaxK) return VT_ERR_SHAPE;
    if (text == nullptr || text_bytes == 0) return VT_ERR_NULL;
    const int chunk = pick_chunk(n, k, d, m, w_type);
    if (chunk == 0) return VT_ERR_SHAPE;
    StepPlan p = plan_step(chunk, k, d, m, w_type);
    if (!p.ok) return VT_ERR_SHAPE;
    // (with a workspace of vt_draft_head_step_ws_bytes)
    const StepPlan stored = plan_stored(p, chunk, k, d, m);
    if (stored.ok) p = stored;
    char head[160];
    if (p.gemv) {
        std::snprintf(head, sizeof head, "head_gemv_kernel<%s,%d,%d> workgroups=%d rows_per_workgroup=%d column_segments=%d",
                      w_type == VT_BF16 ? "bf16" : "f32", p.NP, p.CS, p.nblocks, p.rpb, p.S);
    } else if (p.wide) {
        char by_slices[32] = "";
        if (p.splits > 1) std::snprintf(by_slices, sizeof by_slices, " column_slices=%d", p.splits);
        std::snprintf(head, sizeof head, "%shead_mfma_wide_kernel<%d> workgroups=%d tile_rows=%d%s",
                      p.off_hpack != 0 ? "pack_h_kernel + " : "", p.NT <= 8 ? 1 : 2, p.nlists, 16 * p.row_groups, by_slices);
    } else {
        // (the second template argument: the most waves of the instantiation)
        std::snprintf(head, sizeof head, "head_mfma_kernel<%d,%d> workgroups=%d tile_rows=%d waves=%d column_split=%d%s", p.NT,
                      p.nwaves == vt::kStepWaves                         ? vt::kStepWaves
                      : p.NT > 1 && p.nwaves <= vt::kMfmaFewWaves ? vt::kMfmaFewWaves
                                                                         : vt::kMfmaMaxWaves,
                      p.nlists, 16 * p.row_groups + p.extra_rows, p.nwaves, p.ksplit, p.twin ? " workgroups_per_cu=2" : "");
        if (p.splits > 1) std::snprintf(head + std::strlen(head), sizeof head - std::strlen(head), " column_slices=%d", p.splits);
    }
    char tail[48];
    if (p.parts != 0)
        std::snprintf(tail, sizeof tail, " + row_select_parts_kernel parts=%d", p.parts);
    else
        std::snprintf(tail, sizeof tail, " + %s", p.row_select ? "row_select_kernel" : "step_finalize_kernel");
    char groups[48] = "";
    if (chunk < n) std::snprintf(groups, sizeof groups, " x %d row groups", (n + chunk - 1) / chunk);
    std::snprintf(text, text_bytes, "%s%s%s", head, tail, groups);
    return VT_OK;
}

int vt_draft_head_step_multi_plan(int32_t n, int32_t d, const int32_t *k, int32_t n_heads, const int32_t *head_of_row,
                                  int32_t m, int w_type, char *text, size_t text_bytes) {
    if (w_type != VT_F32 && w_type != VT_BF16) return VT_ERR_DTYPE;
    if (n < 1 || n > VT_MULTI_MAX_ROWS || d < 1 || n_heads < 1 || n_heads > VT_MAX_HEADS) return VT_ERR_SHAPE;
    if (k == nullptr || head_of_row == nullptr || text == nullptr || text_bytes == 0) return VT_ERR_NULL;
    int rows_of[VT_MAX_HEADS] = {};
    for (int i = 0; i < n; ++i) {
        if (head_of_row[i] < 0 || head_of_row[i] >= n_heads) return VT_ERR_SHAPE;
        ++rows_of[head_of_row[i]];
    }
    int used[VT_MAX_HEADS], nused = 0;
    for (int hd = 0; hd < n_heads; ++hd) {
        if (k[hd] < 1 || k[hd] > vt::kStepMaxK) return VT_ERR_SHAPE;
        if (rows_of[hd] == 0) continue;
        if (m < 1 || m > k[hd] || m > VT_MAX_TOP_M) return VT_ERR_SHAPE;
        used[nused++] = hd;
    }
    const StepPlan p = plan_heads_fused(n, d, k, used, nused, m, w_type);
    if (p.ok) {
        std::snprintf(text, text_bytes,
                      "head_mfma_kernel<1,%d> heads=%d workgroups=%d tile_rows=%d waves=%d column_split=%d + step_finalize_kernel",
                      p.nwaves == vt::kStepWaves ? vt::kStepWaves : vt::kMfmaMaxWaves, nused, p.nlists,
                      16 * (p.nwaves / p.ksplit), p.nwaves, p.ksplit);
    } else {
        std::snprintf(text, text_bytes, "head by head (%d)", nused);
    }
    return VT_OK;
}

int vt_draft_head_step_ws_init(void *ws, size_t ws_bytes, void *stream) {
    if (ws == nullptr || !aligned(ws, 256) || ws_bytes < kTicketBytes) return VT_ERR_WORKSPACE;
    (void)hipGetLastError();
    vt::launch_ws_clear(static_cast<unsigned *>(ws), (int)(kTicketBytes / sizeof(unsigned)),
                        static_cast<hipStream_t>(stream));
    return launch_status();
}

int vt_draft_head_step(const void *h, int h_type, int32_t n, const void *W_trim, int w_type, int32_t k, int32_t d,
                       const int32_t *map, int32_t m, int32_t *out_ids, float *out_logp, float *out_lse,
                       float *out_logp_full, void *ws, size_t ws_bytes, void *stream) {
    if ((h_type != VT_F32 && h_type != VT_BF16) || (w_type != VT_F32 && w_type != VT_BF16)) return VT_ERR_DTYPE;
    if (h_type != w_type) return VT_ERR_DTYPE;
    if (n <= 0 || k <= 0 || d <= 0 || k > vt::kStepMaxK) return VT_ERR_SHAPE;
    if (m < 1 || m > k || m > VT_MAX_TOP_M) return VT_ERR_SHAPE;
    if (h == nullptr || W_trim == nullptr || map == nullptr || out_ids == nullptr || out_logp == nullptr)
        return VT_ERR_NULL;
    const size_t row_bytes = (size_t)d * elem_size(w_type);
    if ((row_bytes & 15) != 0 || !aligned(h, 16) || !aligned(W_trim, 16) || !aligned(map, 4) ||
        !aligned(out_ids, 4) || !aligned(out_logp, 4) || (out_lse && !aligned(out_lse, 4)) ||
        (out_logp_full && !aligned(out_logp_full, 4)))
        return VT_ERR_ALIGN;
    const StepShape &shape = step_shape(n, k, d, m, w_type);
    if (shape.chunk == 0) return VT_ERR_SHAPE;
    if (ws == nullptr || !aligned(ws, 256) || ws_bytes < shape.ws_bytes) return VT_ERR_WORKSPACE;
    (void)hipGetLastError();
    const int rc = run_step_rows(h, n, W_trim, w_type, k, d, map, m, out_ids, out_logp, out_lse, out_logp_full, ws, ws_bytes,
                                 static_cast<hipStream_t>(stream));
    if (rc != VT_OK) return rc;
    return launch_status();
}

int vt_draft_head_step_static(const void *h, int h_type, int32_t n, const void *W_trim, int w_type, int32_t k,
                              int32_t d, const int32_t *map, int32_t m, int32_t *out_ids, float *out_logp,
                              float *out_lse, float *out_logp_full, void *stream) {
    // the size check comes first and touches no device: a shape is either out of range altogether (0) or needs
    // more than the library's own array holds
    if (n <= 0 || k <= 0 || d <= 0 || m < 1) return VT_ERR_SHAPE;
    const StepShape &shape = step_shape(n, k, d, m, w_type);
    if (shape.ws_bytes == 0) return VT_ERR_SHAPE;
    if (shape.ws_bytes > (size_t)VT_STATIC_WS_BYTES) return VT_ERR_WORKSPACE;
    const bool stored = shape.stored_bytes > (size_t)VT_STATIC_WS_BYTES && shape.stored_bytes <= kStaticStoredBytes;
    void *ws = nullptr;
    const int rc = static_scratch_of_current_device(stored, &ws);
    if (rc != VT_OK) return rc;
    // Nothing has to be cleared here: a step rewrites everything it reads in the array before it reads it (the
    // one counted word, the ticket of a fused tree level, is zeroed by the kernel that runs before its user).
    return vt_draft_head_step(h, h_type, n, W_trim, w_type, k, d, map, m, out_ids, out_logp, out_lse, out_logp_full,
                              ws, stored ? kStaticStoredBytes : (size_t)VT_STATIC_WS_BYTES, stream);
}

// ------------------------------------------------------------------ several heads in one step
size_t vt_draft_head_step_multi_ws_bytes(int32_t n, int32_t d, const int32_t *k, int32_t n_heads, int32_t m) {
    if (n < 1 || n > VT_MULTI_MAX_ROWS || d < 1 || k == nullptr || n_heads < 1 || n_heads > VT_MAX_HEADS || m < 1)
        return 0;
    for (int hd = 0; hd < n_heads; ++hd) {
        if (k[hd] < 1 || k[hd] > vt::kStepMaxK) return 0;
    }
    return multi_layout(n, d, k, n_heads, m, true).bytes;
}

int vt_draft_head_step_multi(const void *h, int h_type, int32_t n, int32_t d, const void *const *W_trim, int w_type,
                             const int32_t *k, const int32_t *const *map, int32_t n_heads,
                             const int32_t *head_of_row, int32_t m, int32_t *out_ids, float *out_logp,
                             float *out_lse, void *ws, size_t ws_bytes, void *stream) {
    if ((h_type != VT_F32 && h_type != VT_BF16) || (w_type != VT_F32 && w_type != VT_BF16)) return VT_ERR_DTYPE;
    if (h_type != w_type) return VT_ERR_DTYPE;
    if (n < 1 || n > VT_MULTI_MAX_ROWS || d < 1 || n_heads < 1 || n_heads > VT_MAX_HEADS) return VT_ERR_SHAPE;
    if (h == nullptr || W_trim == nullptr || k == nullptr || map == nullptr || head_of_row == nullptr ||
        out_ids == nullptr || out_logp == nullptr)
        return VT_ERR_NULL;
    const size_t row_bytes = (size_t)d * elem_size(w_type);
    if ((row_bytes & 15) != 0 || !aligned(h, 16) || !aligned(out_ids, 4) || !aligned(out_logp, 4) ||
        (out_lse && !aligned(out_lse, 4)))
        return VT_ERR_ALIGN;
    // rows of every head, in ascending row order
    vt::RowList rows[VT_MAX_HEADS];
    for (int hd = 0; hd < n_heads; ++hd) rows[hd].n = 0;
    for (int i = 0; i < n; ++i) {
        const int hd = head_of_row[i];
        if (hd < 0 || hd >= n_heads) return VT_ERR_SHAPE;
        rows[hd].idx[rows[hd].n++] = (short)i;
    }
    for (int hd = 0; hd < n_heads; ++hd) {
        if (k[hd] < 1 || k[hd] > vt::kStepMaxK) return VT_ERR_SHAPE;
        if (rows[hd].n == 0) continue;           // an unused head needs no valid pointers
        if (m < 1 || m > k[hd] || m > VT_MAX_TOP_M) return VT_ERR_SHAPE;
        if (W_trim[hd] == nullptr || map[hd] == nullptr) return VT_ERR_NULL;
        if (!aligned(W_trim[hd], 16) || !aligned(map[hd], 4)) return VT_ERR_ALIGN;
        if (pick_chunk(rows[hd].n, k[hd], d, m, w_type) == 0) return VT_ERR_SHAPE;
    }
    // (sizes that earlier versions returned have no room for plan_stored()'s plans)
    MultiLayout L = multi_layout(n, d, k, n_heads, m, true);
    if (ws_bytes < L.bytes) L = multi_layout(n, d, k, n_heads, m, false);
    if (ws == nullptr || !aligned(ws, 256) || ws_bytes < L.bytes) return VT_ERR_WORKSPACE;
    (void)hipGetLastError();
    hipStream_t st = static_cast<hipStream_t>(stream);
    char *wsb = static_cast<char *>(ws);
    {
        const int rc = run_step_heads_fused(h, n, d, W_trim, w_type, k, map, n_heads, head_of_row, rows, m, out_ids, out_logp,
                                            out_lse, ws, L.off_h, st);
        if (rc != kNotFused) return rc == VT_OK ? launch_status() : rc;
    }
    for (int hd = 0; hd < n_heads; ++hd) {
        const vt::RowList &R = rows[hd];
        if (R.n == 0) continue;
        const int first = R.idx[0];
        const bool consecutive = R.idx[R.n - 1] - first == R.n - 1;
        if (consecutive) {
            // the head's rows lie next to each other in h: the step reads and writes them in place
            const int rc = run_step_rows(static_cast<const char *>(h) + (size_t)first * row_bytes, R.n, W_trim[hd], w_type,
                                         k[hd], d, map[hd], m, out_ids + (size_t)first * m, out_logp + (size_t)first * m,
                                         out_lse ? out_lse + first : nullptr, nullptr, ws, L.off_h, st);
            if (rc != VT_OK) return rc;
            continue;
        }
        const StepPlan plan = plan_step(R.n, k[hd], d, m, w_type);
        if (R.n <= vt::kGemvMaxN && plan.ok && !plan.row_select) {
            // few rows: the kernel picks its hidden rows out of h and writes their output rows itself
            TreeFuse pick;
            pick.indexed = 1;
            for (int i = 0; i < R.n; ++i) pick.row_pack |= (unsigned long long)(R.idx[i] & 0xFF) << (8 * i);
            const int rc = run_step_group(h, R.n, W_trim[hd], w_type, k[hd], d, map[hd], m, out_ids, out_logp, out_lse,
                                          nullptr, ws, L.off_h, st, pick);
            if (rc != VT_OK) return rc;
            continue;
        }
        int32_t *ids_s = reinterpret_cast<int32_t *>(wsb + L.off_ids);
        float *logp_s = reinterpret_cast<float *>(wsb + L.off_logp);
        float *lse_s = reinterpret_cast<float *>(wsb + L.off_lse);
        vt::launch_gather_h_rows(h, wsb + L.off_h, row_bytes, R, st);
        const int rc = run_step_rows(wsb + L.off_h, R.n, W_trim[hd], w_type, k[hd], d, map[hd], m, ids_s, logp_s, lse_s,
                                     nullptr, ws, L.off_h, st);
        if (rc != VT_OK) return rc;
        vt::launch_scatter_rows(ids_s, logp_s, lse_s, m, out_ids, out_logp, out_lse, R, st);
    }
    return launch_status();
}

// ------------------------------------------------------------------ several heads built from one W
int vt_build_trimmed_heads(const int64_t *counts, int32_t V, int32_t n_heads, const void *W, int w_type, int32_t d,
                           const int32_t *k, int32_t *const *map, void *const *W_trim, void *ws, size_t ws_bytes,
                           void *stream) {
    if (n_heads < 1 || n_heads > VT_MAX_HEADS) return VT_ERR_SHAPE;
    if (counts == nullptr || k == nullptr || map == nullptr) return VT_ERR_NULL;
    if ((W == nullptr) != (W_trim == nullptr)) return VT_ERR_NULL;
    if (V <= 0) return VT_ERR_SHAPE;
    // every head is checked before the first one is built
    for (int hd = 0; hd < n_heads; ++hd) {
        if (k[hd] < 1 || k[hd] > V) return VT_ERR_SHAPE;
        if (map[hd] == nullptr || (W != nullptr && W_trim[hd] == nullptr)) return VT_ERR_NULL;
        if (ws_bytes < vt_build_trimmed_head_ws_bytes(V, d, k[hd])) return VT_ERR_WORKSPACE;
    }
    // the checks of the single-head build, for every head
    if (w_type != VT_F32 && w_type != VT_BF16) return VT_ERR_DTYPE;
    if (d <= 0) return VT_ERR_SHAPE;
    const size_t row_bytes = (size_t)d * elem_size(w_type);
    if (!aligned(counts, 8)) return VT_ERR_ALIGN;
    if (W != nullptr && ((row_bytes & 15) != 0 || !aligned(W, 16))) return VT_ERR_ALIGN;
    for (int hd = 0; hd < n_heads; ++hd) {
        if (!aligned(map[hd], 4) || (W != nullptr && !aligned(W_trim[hd], 16))) return VT_ERR_ALIGN;
    }
    if (ws == nullptr || !aligned(ws, 256)) return VT_ERR_WORKSPACE;
    static_assert(VT_MAX_HEADS == vt::kSelectMaxHeads, "heads per batched launch");
    (void)hipGetLastError();
    hipStream_t st = static_cast<hipStream_t>(stream);
    // as many heads together as the workspace holds tables for (all of them unless V is small): the selection's four
    // launches and the row copy once per batch, with the head as grid.y
    const size_t room = (ws_bytes - 256) / vt::select_scratch_stride(V);
    const int batch = room < 1 ? 1 : room < (size_t)n_heads ? (int)room : n_heads;
    for (int h0 = 0; h0 < n_heads; h0 += batch) {
        const int nh = n_heads - h0 < batch ? n_heads - h0 : batch;
        vt::launch_select_topk_heads(reinterpret_cast<const long long *>(counts) + (size_t)h0 * V, V, nh, k + h0,
                                     static_cast<char *>(ws) + 256, map + h0, st);
        if (W != nullptr)
            vt::launch_gather_rows_heads(W, row_bytes, nh, k + h0, const_cast<const int *const *>(map + h0), W_trim + h0, st);
    }
    return launch_status();
}

int vt_draft_tree_level(const void *h, int h_type, int32_t n, const void *W_trim, int w_type, int32_t k, int32_t d,
                        const int32_t *map, int32_t m, const float *parent_cum, int32_t K, int32_t *out_parent,
                        int32_t *out_token, float *out_cum, int32_t *out_ids, float *out_logp, void *ws,
                        size_t ws_bytes, void *stream) {
    if ((h_type != VT_F32 && h_type != VT_BF16) || (w_type != VT_F32 && w_type != VT_BF16)) return VT_ERR_DTYPE;
    if (h_type != w_type) return VT_ERR_DTYPE;
    if (n <= 0 || k <= 0 || d <= 0 || k > vt::kStepMaxK) return VT_ERR_SHAPE;
    if (m < 1 || m > k || m > VT_MAX_TOP_M) return VT_ERR_SHAPE;
    if ((int64_t)n * m > VT_TREE_MAX_CANDIDATES || K < 1 || (int64_t)K > (int64_t)n * m) return VT_ERR_SHAPE;
    if (h == nullptr || W_trim == nullptr || map == nullptr || out_ids == nullptr || out_logp == nullptr ||
        parent_cum == nullptr || out_parent == nullptr || out_token == nullptr || out_cum == nullptr)
        return VT_ERR_NULL;
    const size_t row_bytes = (size_t)d * elem_size(w_type);
    if ((row_bytes & 15) != 0 || !aligned(h, 16) || !aligned(W_trim, 16) || !aligned(map, 4) ||
        !aligned(out_ids, 4) || !aligned(out_logp, 4) || !aligned(parent_cum, 4) || !aligned(out_parent, 4) ||
        !aligned(out_token, 4) || !aligned(out_cum, 4))
        return VT_ERR_ALIGN;
    const StepShape &shape = step_shape(n, k, d, m, w_type);
    const int chunk = shape.chunk;
    if (chunk == 0) return VT_ERR_SHAPE;
    if (ws == nullptr || !aligned(ws, 256) || ws_bytes < shape.ws_bytes) return VT_ERR_WORKSPACE;
    (void)hipGetLastError();
    hipStream_t st = static_cast<hipStream_t>(stream);
    // one launch when the small-n kernel covers the whole step: its last workgroup also ranks the candidates
    // (the same kernel as vt_draft_head_step would use for this shape, so both calls return the same bits)
    // ... or, on the matrix-core path, when its merge kernel (one workgroup per hidden row) covers all rows: the
    // workgroup that finishes last ranks the candidates
    // (rows in several groups: no plan covers them all)
    const StepPlan small = chunk >= n ? shape.with(ws_bytes) : StepPlan{};
    const bool fuse_gemv = small.ok && small.gemv && n * m <= vt::kStepWaves * 64;
    const bool fuse_mfma = small.ok && small.mfma && !small.row_select && n * m <= vt::kFinalizeTreeMaxN;
    if (fuse_gemv || fuse_mfma) {
        TreeFuse tf;
        tf.cum = parent_cum;
        tf.K = K;
        tf.parent = out_parent;
        tf.token = out_token;
        tf.score = out_cum;
        const int rc = run_step_group(h, n, W_trim, w_type, k, d, map, m, out_ids, out_logp, nullptr, nullptr, ws, ws_bytes, st, tf);
        if (rc != VT_OK) return rc;
        return launch_status();
    }
    for (int i0 = 0; i0 < n; i0 += chunk) {
        const int nc = n - i0 < chunk ? n - i0 : chunk;
        const int rc = run_step_group(static_cast<const char *>(h) + (size_t)i0 * row_bytes, nc, W_trim, w_type, k, d, map,
                                      m, out_ids + (size_t)i0 * m, out_logp + (size_t)i0 * m, nullptr, nullptr, ws, ws_bytes, st,
                                      TreeFuse{});
        if (rc != VT_OK) return rc;
    }
    vt::TreeArgs a;
    a.parent_cum = parent_cum;
    a.vals = out_logp;
    a.ids = out_ids;
    a.N = n * m;
    a.m = m;
    a.K = K;
    a.index_order = 0;
    a.out_a = out_parent;
    a.out_token = out_token;
    a.out_score = out_cum;
    return device_status(vt::launch_tree_select(a, st));
}

}  // extern "C"

namespace {

// One launch group of the draft step: n rows that a single plan covers.  Arguments are validated.
// Up to 8 hidden rows on two or more heads: one launch of the matrix-core kernel over all those heads' tiles -- every
// head streams once and the fixed costs of a step (launches, epilogue, merge) are paid once, not per head -- then
// the merge kernel.  All tiles have one height, the smallest for which every head, cut on its own, fits one tile
// per CU in all: 32, 64 or 128 rows with eight waves (4, 2, 1 waves per 16-row group), 144 .. 192 rows with 9 .. 12
// waves.  Returns kNotFused where that does not apply (the caller then runs the heads one after another).
// The plan of that launch (ok = false where it does not apply): used = the heads that have rows.
StepPlan plan_heads_fused(int n, int d, const int32_t *k, const int *used, int nused, int m, int w_type) {
    StepPlan p;
    if (n > vt::kGemvMaxN || w_type != VT_BF16 || nused < 2) return p;
    const int CUS = round_workgroups();
    static const int shapes[][2] = {{8, 4}, {8, 2}, {8, 1}, {9, 1}, {10, 1}, {11, 1}, {12, 1}};
    for (const auto &sh : shapes) {
        const int T = 16 * (sh[0] / sh[1]);
        int tiles = 0;
        for (int q = 0; q < nused; ++q) tiles += (k[used[q]] + T - 1) / T;
        if (tiles > CUS) continue;
        FixedTiles ft;
        ft.nwaves = sh[0];
        ft.ksplit = sh[1];
        ft.nlists = tiles;
        p = plan_step_impl(n, tiles * T, d, m, w_type, false, ft);
        if (p.ok) break;
    }
    if (p.ok && (!p.mfma || p.row_select || p.KC != d || p.NT != 1)) p.ok = false;
    return p;
}
int run_step_heads_fused(const void *h, int n, int d, const void *const *W_trim, int w_type, const int32_t *k,
                         const int32_t *const *map, int n_heads, const int32_t *head_of_row, const vt::RowList *rows, int m,
                         int32_t *out_ids, float *out_logp, float *out_lse, void *ws, size_t ws_step_bytes, hipStream_t st) {
    int used[VT_MAX_HEADS], nused = 0;
    for (int hd = 0; hd < n_heads; ++hd)
        if (rows[hd].n != 0) used[nused++] = hd;
    const StepPlan p = plan_heads_fused(n, d, k, used, nused, m, w_type);
    if (!p.ok || p.bytes > ws_step_bytes) return kNotFused;
    const int T = 16 * (p.nwaves / p.ksplit);
    vt::MultiHeadTable t{};
    t.n_heads = nused;
    t.tile_first[0] = 0;
    int slot_of_head[VT_MAX_HEADS];
    for (int q = 0; q < nused; ++q) {
        const int hd = used[q];
        slot_of_head[hd] = q;
        t.W[q] = W_trim[hd];
        t.map[q] = map[hd];
        t.k[q] = k[hd];
        t.tile_first[q + 1] = t.tile_first[q] + (k[hd] + T - 1) / T;
    }
    for (int i = 0; i < n; ++i) t.head_of_row |= (unsigned long long)slot_of_head[head_of_row[i]] << (8 * i);
    char *wsb = static_cast<char *>(ws);
    vt::MfmaArgs a{};
    a.h = h;
    a.n = n;
    a.d = d;
    a.m = m;
    a.L = p.L;
    a.nlists = p.nlists;
    a.KC = p.KC;
    a.hpitch = p.hpitch;
    a.pms = reinterpret_cast<unsigned long long *>(wsb + p.off_pms);
    a.pkeys = reinterpret_cast<unsigned long long *>(wsb + p.off_pkeys);
    a.ksplit = p.ksplit;
    a.nwaves = p.nwaves;
    hipError_t e = vt::launch_head_mfma_multi(a, t, p.lds, st);
    if (e != hipSuccess) return device_status(e);
    vt::FinalizeArgs f{};
    f.pms = a.pms;
    f.pkeys = a.pkeys;
    f.nlists = p.nlists;
    f.several_heads = t.n_heads > 1 ? 1 : 0;
    f.L = p.L;
    f.n = n;
    f.m = m;
    f.out_ids = out_ids;
    f.out_logp = out_logp;
    f.out_lse = out_lse;
    f.lse_buf = reinterpret_cast<float *>(wsb + p.off_lse);
    f.ticket = reinterpret_cast<unsigned *>(wsb);
    e = vt::launch_step_finalize(f, p.fin_lds, st);
    return e == hipSuccess ? VT_OK : device_status(e);
}

int run_step_group(const void *h, int n, const void *W_trim, int w_type, int k, int d, const int32_t *map, int m,
                   int32_t *out_ids, float *out_logp, float *out_lse, float *out_logp_full, void *ws, size_t ws_bytes,
                   hipStream_t st, const TreeFuse &tf) {
    const StepShape &shape = step_shape(n, k, d, m, w_type);
    if (shape.chunk != n) return VT_ERR_SHAPE;
    const StepPlan p = shape.with(ws_bytes);
    char *wsb = static_cast<char *>(ws);
    unsigned long long *pms = reinterpret_cast<unsigned long long *>(wsb + p.off_pms);
    unsigned long long *pkeys = reinterpret_cast<unsigned long long *>(wsb + p.off_pkeys);
    float *lse_buf = reinterpret_cast<float *>(wsb + p.off_lse);
    if (p.gemv) {
        vt::StepArgs a;
        a.h = h;
        a.W = W_trim;
        a.map = map;
        a.n = n;
        a.k = k;
        a.d = d;
        a.m = m;
        a.S = p.S;
        a.rpb = p.rpb;
        a.tpitch = p.tpitch;
        a.L = p.L;
        a.nblocks = p.nblocks;
        a.pms = pms;
        a.pkeys = pkeys;
        a.out_logp_full = out_logp_full;
        a.zbuf = nullptr;
        a.zpitch = p.parts != 0 ? slice_pitch(k) : k;
        a.parts = p.parts;
        if (p.row_select) a.zbuf = out_logp_full != nullptr && p.parts == 0 ? out_logp_full : reinterpret_cast<float *>(wsb + p.off_zbuf);
        if (tf.indexed && (p.row_select || out_logp_full != nullptr)) return VT_ERR_SHAPE;
        a.row_pack = tf.indexed ? tf.row_pack : 0x0706050403020100ull;
        // a tree level fused behind the merge kernel: rows in order, at most kFinalizeTreeMaxN candidates
        const bool tree_behind_merge = tf.cum != nullptr && !p.row_select;
        if (tree_behind_merge && (tf.indexed || n * m > vt::kFinalizeTreeMaxN)) return VT_ERR_SHAPE;
        a.ticket_clear = tree_behind_merge ? reinterpret_cast<unsigned *>(wsb) : nullptr;
        const size_t lds = p.lds;
        const bool bf16 = w_type == VT_BF16;
        hipError_t e = hipErrorInvalidValue;
        switch (p.NP) {
            case 1: e = vt::launch_head_gemv_np1(bf16, p.CS, a, lds, st); break;
            case 2: e = vt::launch_head_gemv_np2(bf16, p.CS, a, lds, st); break;
            case 4: e = vt::launch_head_gemv_np4(bf16, p.CS, a, lds, st); break;
            case 8: e = vt::launch_head_gemv_np8(bf16, p.CS, a, lds, st); break;
            default: break;
        }
        if (e != hipSuccess) return device_status(e);
        if (!p.row_select) {
            vt::FinalizeArgs f{};
            f.pms = pms;
            f.pkeys = pkeys;
            f.nlists = p.nblocks;
            f.L = p.L;
            f.n = n;
            f.m = m;
            f.out_ids = out_ids;
            f.out_logp = out_logp;
            f.out_lse = out_lse;
            f.lse_buf = lse_buf;
            f.row_pack = tf.row_pack;
            f.indexed = tf.indexed;
            f.tree_cum = tf.cum;
            f.tree_K = tf.K;
            f.tree_parent = tf.parent;
            f.tree_token = tf.token;
            f.tree_score = tf.score;
            f.ticket = reinterpret_cast<unsigned *>(wsb);
            e = vt::launch_step_finalize(f, (size_t)(p.nblocks + 1) * p.L * sizeof(unsigned long long), st);
            if (e != hipSuccess) return device_status(e);
        }
        if (p.row_select) {
            const vt::RowParts parts{pms, p.parts, p.per_tile, p.part_rows, p.rpb};
            const hipError_t e = vt::launch_row_select(a.zbuf, map, n, k, m, 1, a.zpitch, false, nullptr, out_ids, out_logp, out_lse, lse_buf,
                                                       p.parts != 0 ? &parts : nullptr, st);
            if (e != hipSuccess) return device_status(e);
            if (out_logp_full != nullptr) vt::launch_sub_lse(a.zbuf, a.zpitch, out_logp_full, lse_buf, n, k, st);
            if (tf.cum != nullptr) {       // the fused tree level needs the merge kernel: run the expansion kernel
                vt::TreeArgs t;
                t.parent_cum = tf.cum;
                t.vals = out_logp;
                t.ids = out_ids;
                t.N = n * m;
                t.m = m;
                t.K = tf.K;
                t.index_order = 0;
                t.out_a = tf.parent;
                t.out_token = tf.token;
                t.out_score = tf.score;
                return device_status(vt::launch_tree_select(t, st));
            }
            return VT_OK;
        }
    } else {
        // a fused tree level needs the merge kernel (no per-row tail) and at most kFinalizeTreeMaxN candidates; row
        // picking needs up to 8 rows and the merge kernel too
        if ((tf.cum != nullptr && (p.row_select || tf.indexed || n * m > vt::kFinalizeTreeMaxN)) ||
            (tf.indexed && (n > vt::kGemvMaxN || p.row_select || out_logp_full != nullptr)))
            return VT_ERR_SHAPE;
        vt::MfmaArgs a;
        a.h = h;
        a.W = W_trim;
        a.map = map;
        a.n = n;
        a.k = k;
        a.d = d;
        a.m = m;
        a.L = p.L;
        a.nlists = p.nlists;
        a.KC = p.KC;
        a.hpitch = p.hpitch;
        a.pms = pms;
        a.pkeys = pkeys;
        a.out_logp_full = out_logp_full;
        a.hpack = p.off_hpack != 0 ? static_cast<void *>(wsb + p.off_hpack) : nullptr;
        a.zbuf = nullptr;
        a.splits = p.splits;
        a.slice_units = d / 128 / p.splits;
        a.slice_more = d / 128 % p.splits;
        a.slice_ranges = d % (2048 * p.splits) == 0 ? 1 : 0;
        a.zpitch = p.splits > 1 || p.parts != 0 ? slice_pitch(k) : k;
        a.parts = p.parts;
        if (p.row_select) a.zbuf = out_logp_full != nullptr && p.splits == 1 && p.parts == 0 ? out_logp_full : reinterpret_cast<float *>(wsb + p.off_zbuf);
        // (a group of four must not reach into the next tile, whose workgroup stores there, nor behind the row)
        a.zvec = a.zpitch % 4 == 0 && aligned(a.zbuf, 16) && (16 * p.row_groups + p.extra_rows) % 4 == 0 ? 1 : 0;
        a.row_pack = tf.row_pack;
        a.indexed = tf.indexed;
        a.ksplit = p.ksplit;
        a.nwaves = p.nwaves;
        a.extra_rows = p.extra_rows;
        a.row_groups = p.row_groups;
        a.ids_off = p.ids_off;
        a.passes = p.passes;
        a.twin = p.twin ? 1 : 0;
        a.ticket_clear = tf.cum != nullptr ? reinterpret_cast<unsigned *>(wsb) : nullptr;
        hipError_t e = n <= vt::kGemvMaxN ? vt::launch_head_mfma(a, p.lds, st)
                       : p.wide           ? vt::launch_head_mfma_wide(p.NT / 4, a, p.lds, st)
                                          : vt::launch_head_mfma_rows(p.NT, a, p.lds, st);
        if (e != hipSuccess) return device_status(e);
        if (p.row_select) {
            const vt::RowParts parts{pms, p.parts, p.per_tile, p.part_rows, 16 * p.row_groups + p.extra_rows};
            e = vt::launch_row_select(a.zbuf, map, n, k, m, a.splits, a.zpitch, p.instead_of_lists, out_logp_full, out_ids, out_logp, out_lse, lse_buf,
                                      p.parts != 0 ? &parts : nullptr, st);
            if (e != hipSuccess) return device_status(e);
            if (out_logp_full != nullptr) {
                const float *z = p.parts != 0 ? a.zbuf : out_logp_full;
                vt::launch_sub_lse(z, p.parts != 0 ? a.zpitch : k, out_logp_full, lse_buf, n, k, st);
            }
            return VT_OK;
        }
        vt::FinalizeArgs f{};
        f.row_pack = tf.row_pack;
        f.indexed = tf.indexed;
        f.pms = pms;
        f.pkeys = pkeys;
        f.nlists = p.nlists;
        f.L = p.L;
        f.n = n;
        f.m = m;
        f.out_ids = out_ids;
        f.out_logp = out_logp;
        f.out_lse = out_lse;
        f.lse_buf = lse_buf;
        f.tree_cum = tf.cum;
        f.tree_K = tf.K;
        f.tree_parent = tf.parent;
        f.tree_token = tf.token;
        f.tree_score = tf.score;
        f.ticket = reinterpret_cast<unsigned *>(wsb);
        if (tf.cum != nullptr && (n * m > vt::kFinalizeTreeMaxN || tf.indexed)) return VT_ERR_SHAPE;
        e = vt::launch_step_finalize(f, p.fin_lds, st);
        if (e != hipSuccess) return device_status(e);
    }
    if (out_logp_full != nullptr)
        vt::launch_sub_lse(out_logp_full, k, out_logp_full, lse_buf, n, k, st);
    return VT_OK;
}

}  // namespace

extern "C" {

int vt_tree_expand(const float *parent_cum, const float *step_logp, const int32_t *step_ids, int32_t n, int32_t m,
                   int32_t K, int32_t *out_parent, int32_t *out_token, float *out_cum, void *stream) {
    if (!parent_cum || !step_logp || !step_ids || !out_parent || !out_token || !out_cum) return VT_ERR_NULL;
    if (n < 1 || m < 1 || (int64_t)n * m > VT_TREE_MAX_CANDIDATES || K < 1 || K > n * m) return VT_ERR_SHAPE;
    vt::TreeArgs a;
    a.parent_cum = parent_cum;
    a.vals = step_logp;
    a.ids = step_ids;
    a.N = n * m;
    a.m = m;
    a.K = K;
    a.index_order = 0;
    a.out_a = out_parent;
    a.out_token = out_token;
    a.out_score = out_cum;
    return device_status(vt::launch_tree_select(a, static_cast<hipStream_t>(stream)));
}

int vt_tree_rerank(const float *cum, int32_t N, int32_t T, int32_t *out_idx, void *stream) {
    if (!cum || !out_idx) return VT_ERR_NULL;
    if (N < 1 || N > VT_TREE_MAX_CANDIDATES || T < 1 || T > N || T > VT_TREE_MAX_KEEP) return VT_ERR_SHAPE;
    static_assert(VT_TREE_MAX_CANDIDATES == vt::kTreeMaxN && VT_TREE_MAX_KEEP == vt::kTreeMaxKeepSorted, "limits");
    vt::TreeArgs a;
    a.parent_cum = nullptr;
    a.vals = cum;
    a.ids = nullptr;
    a.N = N;
    a.m = 1;
    a.K = T;
    a.index_order = 1;
    a.out_a = out_idx;
    a.out_token = nullptr;
    a.out_score = nullptr;
    return device_status(vt::launch_tree_select(a, static_cast<hipStream_t>(stream)));
}

}  // extern "C"
