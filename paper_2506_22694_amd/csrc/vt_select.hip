// Eq. 1 of the paper: V_trim = V[Top-K(c, k)], W_trim = W[Top-K(c, k), :].
//
// Selection = the k-th largest count (threshold T, and the number r of T-valued ids to keep; ties go to the lower id),
// then an id-ordered compaction that emits the selected ids already ascending -- no sort.  It runs over the whole device,
// one workgroup per 1024 ids, as four small launches, each a chain of latencies (launch, memory, scan) and not of work:
//   sel_zero    clears the histograms
//   sel_hist    histogram of all counts over 3744 bins, exact values below 2048 (vt_code.h)
//   sel_count   every workgroup finds the bin of the k-th largest count.  Below 2048 that bin is T itself, and the
//               workgroup tallies its ids above / at T.  A larger T is looked for inside its bin: all workgroups histogram
//               the next eleven bits of its ids, and the one that is done last settles T
//   sel_write   the compaction: ballots, and the tallies of the workgroups before this one (above 2048: a chained scan)
// (A radix select byte by byte took eleven launches, 47 us at V = 128256 after 10^7 tokens; this one 18.)
// The last workgroup reads all counts once for every eleven bits that are still open: only where more ids share the 17
// highest bits of T than are taken of them, and from the highest bit on in which they differ.
// V = 128256, k = 1000 after 10^9 tokens 22 us (65 with one workgroup for the whole search and a recount of all ids before
// it in every workgroup of sel_write, 51 byte by byte), k = 5000 after 10^11 23 (65, 58); V = 10^6, k = 1000 76 (917, 150).
// All counts in 2^40 .. 2^40 + 2^20, where all ids share those bits: V = 128256 70 us (254, 47), V = 10^6 437 (2713, 119).
// gather_rows_kernel: W_trim[j, :] = W[map[j], :], a pure copy at HBM speed.
#include "vt_build.h"
#include "vt_code.h"
#include "vt_device.h"

namespace vt {

namespace {
constexpr int kSelWaves = kSelectThreads / kWave;   // 16
constexpr int kBinsPerThread = (kBins + kSelectThreads - 1) / kSelectThreads;   // 4

struct SelBufs {
    unsigned *hist;               // [kBins] ids per bin
    unsigned *digits;             // [kDigitBins] of the bin of the k-th largest count
    unsigned long long *bits;     // [2] of its ids, below the bin's prefix: bits set in any, bits clear in any
    unsigned *done;               // [2] workgroups that have added theirs; that sel_write has numbered
    unsigned long long *thresh;   // T
    int *take;                    // r
    int *tallied;                 // 1: tab is there, 0: sel_write's workgroups sum up as they go
    unsigned *tab;                // [nblk][2] ids above / at the threshold per workgroup
};
constexpr int kSelZeroWords = kBins + kDigitBins + 4 + 2;      // hist .. done

// Several heads per launch (grid.y = head): head y selects k[y] of the counts at counts + y V into map[y], with
// the scratch of a single selection at scratch + y stride.
struct SelBatch {
    unsigned char *scratch;
    size_t stride;
    int nblk;
    int k[kSelectMaxHeads];
    int *map[kSelectMaxHeads];
};
constexpr size_t kSelTabOffset = (size_t)kSelZeroWords * sizeof(unsigned) + 16;
static_assert(kBins % 2 == 0 && kDigitBins % 2 == 0 && kSelZeroWords % 2 == 0, "the 64-bit words are aligned");
__device__ __forceinline__ SelBufs head_bufs(const SelBatch &sb) {
    unsigned char *p = sb.scratch + (size_t)blockIdx.y * sb.stride;
    SelBufs b;
    b.hist = reinterpret_cast<unsigned *>(p);
    b.digits = b.hist + kBins;
    b.bits = reinterpret_cast<unsigned long long *>(b.digits + kDigitBins);
    b.done = reinterpret_cast<unsigned *>(b.bits + 2);
    b.thresh = reinterpret_cast<unsigned long long *>(b.done + 2);
    b.take = reinterpret_cast<int *>(b.thresh + 1);
    b.tallied = b.take + 1;
    b.tab = reinterpret_cast<unsigned *>(p + kSelTabOffset);
    return b;
}

__global__ void __launch_bounds__(256) sel_zero_kernel(SelBatch sb) {
    unsigned *p = head_bufs(sb).hist;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < kSelZeroWords; i += gridDim.x * 256) p[i] = 0u;
}

__global__ void __launch_bounds__(kSelectThreads) sel_hist_kernel(const long long *__restrict__ counts_all, int V,
                                                                  SelBatch sb) {
    const SelBufs b = head_bufs(sb);
    const long long *__restrict__ counts = counts_all + (size_t)blockIdx.y * V;
    __shared__ unsigned h[kBins];
    const int j = blockIdx.x * kSelectThreads + threadIdx.x;
    const bool in = j < V;
    const unsigned long long c = in ? (unsigned long long)counts[j] : 0ull;
    for (int i = threadIdx.x; i < kBins; i += kSelectThreads) h[i] = 0u;
    __syncthreads();
    wave_tally(h, count_bin(c), in);
    __syncthreads();
    for (int i = threadIdx.x; i < kBins; i += kSelectThreads) {
        if (h[i] != 0u) atomicAdd(&b.hist[i], h[i]);
    }
}

// Inclusive prefix sum over the workgroup's threads; `part` [kSelWaves] of LDS.  Two barriers.
__device__ __forceinline__ unsigned block_scan(unsigned v, unsigned *part) {
    const int lane = lane_id(), w = (int)threadIdx.x >> 6;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const unsigned t = __shfl_up(v, o);
        if (lane >= o) v += t;
    }
    if (lane == kWave - 1) part[w] = v;
    __syncthreads();
    unsigned before = 0;
#pragma unroll
    for (int q = 0; q < kSelWaves; ++q) before += q < w ? part[q] : 0u;
    __syncthreads();
    return before + v;
}

__global__ void __launch_bounds__(kSelectThreads) sel_count_kernel(const long long *__restrict__ counts_all, int V,
                                                                   SelBatch sb) {
    const SelBufs b = head_bufs(sb);
    const long long *__restrict__ counts = counts_all + (size_t)blockIdx.y * V;
    const int k = sb.k[blockIdx.y];
    __shared__ unsigned part[kSelWaves], s_gt[kSelWaves], s_eq[kSelWaves];
    __shared__ unsigned h[kDigitBins];
    __shared__ unsigned long long s_ones, s_zeros;
    __shared__ int s_bin, s_rem, s_size, s_last;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int j = blockIdx.x * kSelectThreads + tid;
    const unsigned long long c = j < V ? (unsigned long long)counts[j] : 0ull;
    // bins from the highest down, four per thread
    unsigned v[kBinsPerThread], sum = 0;
#pragma unroll
    for (int i = 0; i < kBinsPerThread; ++i) {
        const int bin = kBins - 1 - (kBinsPerThread * tid + i);
        v[i] = bin >= 0 ? b.hist[bin] : 0u;
        sum += v[i];
    }
    unsigned above = block_scan(sum, part) - sum;      // ids in higher bins
#pragma unroll
    for (int i = 0; i < kBinsPerThread; ++i) {
        if (above < (unsigned)k && above + v[i] >= (unsigned)k) {      // one bin of one thread: 1 <= k <= V
            s_bin = kBins - 1 - (kBinsPerThread * tid + i);
            s_rem = k - (int)above;
        }
        above += v[i];
    }
    __syncthreads();
    const int bin = s_bin;
    int rem = s_rem;
    const int mine = j < V ? count_bin(c) : -1;
    if (bin < kBinExact) {
        const int ngt = __popcll(__ballot(mine > bin)), neq = __popcll(__ballot(mine == bin));
        if (lane == 0) {
            s_gt[w] = (unsigned)ngt;
            s_eq[w] = (unsigned)neq;
        }
        __syncthreads();
        if (tid == 0) {
            unsigned g = 0, e = 0;
#pragma unroll
            for (int q = 0; q < kSelWaves; ++q) {
                g += s_gt[q];
                e += s_eq[q];
            }
            b.tab[2 * blockIdx.x] = g;
            b.tab[2 * blockIdx.x + 1] = e;
            if (blockIdx.x == 0) {
                *b.thresh = (unsigned)bin;
                *b.take = rem;
                *b.tallied = 1;
            }
        }
        return;
    }
    // ---- several values share the bin: the next digit of its ids, and the bits in which they differ
    int left = bin_shift(bin);
    unsigned long long T = bin_prefix(bin);
    int nbits = left < kDigitBits ? left : kDigitBits;
    const bool in = mine == bin;
    for (int i = tid; i < kDigitBins; i += kSelectThreads) h[i] = 0u;
    if (tid == 0) s_ones = s_zeros = 0ull;
    __syncthreads();
    wave_tally(h, (int)((c >> (left - nbits)) & low_bits(nbits)), in);
    if (__ballot(in) != 0ull) {
        const unsigned long long set = wave_or_u64(in ? c & low_bits(left) : 0ull);
        const unsigned long long clear = wave_or_u64(in ? ~c & low_bits(left) : 0ull);
        if (lane == 0) {
            atomicOr(&s_ones, set);
            atomicOr(&s_zeros, clear);
        }
    }
    __syncthreads();
    for (int i = tid; i < kDigitBins; i += kSelectThreads) {
        if (h[i] != 0u) atomicAdd(&b.digits[i], h[i]);
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

    // ---- the last workgroup: all others' digits are there
    const unsigned long long ones = acquire_u64(&b.bits[0]), zeros = acquire_u64(&b.bits[1]);
    // d0, d1: ids with digit kDigitBins - 1 - 2 tid and the one below.  Appends the digit of the rem-th largest to T and
    // leaves rem of the ids that have it (s_size).
    static_assert(kDigitBins == 2 * kSelectThreads, "two digits per thread");
    auto find_digit = [&](unsigned d0, unsigned d1) {
        const unsigned upto = block_scan(d0 + d1, part);
        const unsigned above0 = upto - d0 - d1, above1 = upto - d1;
        if (above0 < (unsigned)rem && upto >= (unsigned)rem) {
            const bool upper = above1 >= (unsigned)rem;
            s_bin = kDigitBins - 1 - 2 * tid - (upper ? 0 : 1);
            s_rem = rem - (int)(upper ? above0 : above1);
            s_size = (int)(upper ? d0 : d1);
        }
        __syncthreads();
        T = (T << nbits) | (unsigned)s_bin;
        rem = s_rem;
        left -= nbits;
    };
    const unsigned *mine2 = b.digits + kDigitBins - 2 - 2 * tid;
    find_digit(__hip_atomic_load(mine2 + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
               __hip_atomic_load(mine2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    constexpr int kInFlight = 8;
    while (left > 0) {
        if (rem == s_size) {      // all of them: from the lowest value they can have on
            T = (T << left) - 1;
            rem = 0;
            break;
        }
        left = skip_common_bits(T, left, ones, zeros);
        if (left == 0) break;
        nbits = left < kDigitBits ? left : kDigitBits;
        for (int i = tid; i < kDigitBins; i += kSelectThreads) h[i] = 0u;
        __syncthreads();
        for (unsigned x0 = 0; x0 < (unsigned)V; x0 += kInFlight * kSelectThreads) {
            unsigned long long cx[kInFlight];
#pragma unroll
            for (int u = 0; u < kInFlight; ++u) {
                const unsigned x = x0 + u * kSelectThreads + tid;
                cx[u] = x < (unsigned)V ? (unsigned long long)counts[x] : 0ull;      // (zero has no bits above the open ones)
            }
#pragma unroll
            for (int u = 0; u < kInFlight; ++u)
                wave_tally(h, (int)((cx[u] >> (left - nbits)) & low_bits(nbits)), (cx[u] >> left) == T);
        }
        __syncthreads();
        find_digit(h[kDigitBins - 1 - 2 * tid], h[kDigitBins - 2 - 2 * tid]);
    }
    // nobody has tallied the ids above / at T: sel_write's workgroups do, and pass the sums on in `tab`
    for (int x = tid; x < 2 * (int)gridDim.x; x += kSelectThreads) b.tab[x] = 0u;
    if (tid == 0) {
        *b.thresh = T;
        *b.take = rem;
        *b.tallied = 0;
    }
}

// Ids above and at the threshold in all workgroups before number `me`, which holds g and e of them: a chained scan over
// `state` (zero at first), a word per workgroup that is published twice, with the workgroup's own sums and with the sums
// up to it.  One wave calls it.  The numbers are given out as workgroups start, so a workgroup only ever waits for such
// as already run and publish their own sums before they wait for anybody: every wait ends.
constexpr unsigned long long kScanOwn = 1ull << 62, kScanUpTo = 2ull << 62, kScanSums = (1ull << 62) - 1;
__device__ __forceinline__ unsigned long long scan_before(unsigned long long *state, int me, unsigned g, unsigned e) {
    const int lane = lane_id();
    const unsigned long long own = ((unsigned long long)g << 31) | e;      // (below 2^31 each)
    if (lane == 0) publish_u64(state + me, kScanOwn | own);
    unsigned long long before = 0;
    for (int at = me - 1;; at -= kWave) {      // lane l: workgroup at - l
        unsigned long long v;
        do {
            v = at - lane >= 0 ? acquire_u64(state + (at - lane)) : kScanUpTo;
        } while (__ballot(v == 0ull) != 0ull);
        const unsigned long long complete = __ballot((v & kScanUpTo) != 0ull);
        const int last = complete != 0ull ? __ffsll((long long)complete) - 1 : kWave - 1;
        unsigned long long sum = lane <= last ? v & kScanSums : 0ull;
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) sum += __shfl_xor(sum, o);
        before += sum;
        if (complete != 0ull) break;
    }
    if (lane == 0) publish_u64(state + me, kScanUpTo | (before + own));
    return before;
}

__global__ void __launch_bounds__(kSelectThreads) sel_write_kernel(const long long *__restrict__ counts_all, int V,
                                                                   SelBatch sb) {
    const SelBufs b = head_bufs(sb);
    const long long *__restrict__ counts = counts_all + (size_t)blockIdx.y * V;
    int *__restrict__ map = sb.map[blockIdx.y];
    __shared__ int s_gt[kSelWaves], s_eq[kSelWaves], s_gb[kSelWaves], s_eb[kSelWaves];
    __shared__ int s_me;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    // everything is requested at once: this thread's count, the threshold, the tallies of the workgroups before this one
    int j = blockIdx.x * kSelectThreads + tid;
    unsigned long long c = j < V ? (unsigned long long)counts[j] : 0ull;
    const unsigned long long T = *b.thresh;
    const int r = *b.take, tallied = *b.tallied;
    int gb = 0, eb = 0;
    for (int x = tid; x < (int)blockIdx.x; x += kSelectThreads) {
        gb += (int)b.tab[2 * x];
        eb += (int)b.tab[2 * x + 1];
    }
    if (tallied == 0) {      // (uniform) workgroups are numbered as they start; what was read of tab is not meant
        if (tid == 0) s_me = (int)__hip_atomic_fetch_add(b.done + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        j = s_me * kSelectThreads + tid;
        c = j < V ? (unsigned long long)counts[j] : 0ull;
    }
    const bool gt = j < V && c > T, eq = j < V && c == T;
    const unsigned long long bg = __ballot(gt), be = __ballot(eq);
    if (tallied != 0) {
        gb = wave_sum_i32(gb);
        eb = wave_sum_i32(eb);
    }
    if (lane == 0) {
        s_gb[w] = gb;
        s_eb[w] = eb;
        s_gt[w] = __popcll(bg);
        s_eq[w] = __popcll(be);
    }
    __syncthreads();
    if (tallied == 0) {
        if (w == 0) {
            const unsigned g = (unsigned)wave_sum_i32(lane < kSelWaves ? s_gt[lane & (kSelWaves - 1)] : 0);
            const unsigned e = (unsigned)wave_sum_i32(lane < kSelWaves ? s_eq[lane & (kSelWaves - 1)] : 0);
            const unsigned long long before = scan_before(reinterpret_cast<unsigned long long *>(b.tab), s_me, g, e);
            if (lane < kSelWaves) {
                s_gb[lane] = lane == 0 ? (int)(before >> 31) : 0;
                s_eb[lane] = lane == 0 ? (int)(before & 0x7FFFFFFFull) : 0;
            }
        }
        __syncthreads();
    }
    int gt_before = 0, eq_before = 0;
#pragma unroll
    for (int q = 0; q < kSelWaves; ++q) {
        gt_before += s_gb[q] + (q < w ? s_gt[q] : 0);
        eq_before += s_eb[q] + (q < w ? s_eq[q] : 0);
    }
    const unsigned long long below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    gt_before += __popcll(bg & below);
    eq_before += __popcll(be & below);
    if (gt || (eq && eq_before < r)) map[gt_before + min(eq_before, r)] = j;
}

}  // namespace

size_t select_scratch_bytes(int V) {
    const size_t nblk = ((size_t)V + kSelectThreads - 1) / kSelectThreads;
    return kSelTabOffset + 2 * nblk * sizeof(unsigned);
}

size_t select_scratch_stride(int V) { return (select_scratch_bytes(V) + 255) / 256 * 256; }

// counts: [n_heads, V]; scratch: n_heads * select_scratch_stride(V) bytes
void launch_select_topk_heads(const long long *counts, int V, int n_heads, const int *k, void *scratch, int *const *map,
                              hipStream_t st) {
    SelBatch sb;
    sb.scratch = static_cast<unsigned char *>(scratch);
    sb.stride = select_scratch_stride(V);
    sb.nblk = (V + kSelectThreads - 1) / kSelectThreads;
    for (int hd = 0; hd < kSelectMaxHeads; ++hd) {
        sb.k[hd] = hd < n_heads ? k[hd] : 1;
        sb.map[hd] = hd < n_heads ? map[hd] : nullptr;
    }
    const dim3 grid(sb.nblk, n_heads);
    hipLaunchKernelGGL(sel_zero_kernel, dim3(6, n_heads), dim3(256), 0, st, sb);
    hipLaunchKernelGGL(sel_hist_kernel, grid, dim3(kSelectThreads), 0, st, counts, V, sb);
    hipLaunchKernelGGL(sel_count_kernel, grid, dim3(kSelectThreads), 0, st, counts, V, sb);
    hipLaunchKernelGGL(sel_write_kernel, grid, dim3(kSelectThreads), 0, st, counts, V, sb);
}

void launch_select_topk(const long long *counts, int V, int k, void *scratch, int *map, hipStream_t st) {
    launch_select_topk_heads(counts, V, 1, &k, scratch, &map, st);
}

// One wave copies one row at a time with 16-byte lanes, four loads in flight; rows are independent.
__device__ __forceinline__ void copy_row(const u32x4 *__restrict__ src, u32x4 *__restrict__ dst, size_t nvec, int lane) {
    size_t c = lane;
    for (; c + 3 * kWave < nvec; c += 4 * kWave) {
        const u32x4 a0 = __builtin_nontemporal_load(src + c);
        const u32x4 a1 = __builtin_nontemporal_load(src + c + kWave);
        const u32x4 a2 = __builtin_nontemporal_load(src + c + 2 * kWave);
        const u32x4 a3 = __builtin_nontemporal_load(src + c + 3 * kWave);
        __builtin_nontemporal_store(a0, dst + c);
        __builtin_nontemporal_store(a1, dst + c + kWave);
        __builtin_nontemporal_store(a2, dst + c + 2 * kWave);
        __builtin_nontemporal_store(a3, dst + c + 3 * kWave);
    }
    for (; c < nvec; c += kWave) __builtin_nontemporal_store(__builtin_nontemporal_load(src + c), dst + c);
}

__global__ void __launch_bounds__(256) gather_rows_kernel(const char *__restrict__ W, size_t row_bytes,
                                                          const int *__restrict__ map, int k,
                                                          char *__restrict__ W_trim) {
    const int lane = lane_id();
    const int wave = (int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
    const int nwaves = (int)((gridDim.x * blockDim.x) >> 6);
    const size_t nvec = row_bytes >> 4;
    for (int j = wave; j < k; j += nwaves) {
        copy_row(reinterpret_cast<const u32x4 *>(W + (size_t)map[j] * row_bytes),
                 reinterpret_cast<u32x4 *>(W_trim + (size_t)j * row_bytes), nvec, lane);
    }
}

// The same for several heads in one launch (grid.y = head).
struct GatherBatch {
    int k[kSelectMaxHeads];
    const int *map[kSelectMaxHeads];
    char *W_trim[kSelectMaxHeads];
};
__global__ void __launch_bounds__(256) gather_rows_heads_kernel(const char *__restrict__ W, size_t row_bytes,
                                                                GatherBatch gb) {
    const int lane = lane_id();
    const int wave = (int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
    const int nwaves = (int)((gridDim.x * blockDim.x) >> 6);
    const size_t nvec = row_bytes >> 4;
    const int k = gb.k[blockIdx.y];
    const int *__restrict__ map = gb.map[blockIdx.y];
    char *__restrict__ W_trim = gb.W_trim[blockIdx.y];
    for (int j = wave; j < k; j += nwaves) {
        copy_row(reinterpret_cast<const u32x4 *>(W + (size_t)map[j] * row_bytes),
                 reinterpret_cast<u32x4 *>(W_trim + (size_t)j * row_bytes), nvec, lane);
    }
}

void launch_gather_rows_heads(const void *W, size_t row_bytes, int n_heads, const int *k, const int *const *map,
                              void *const *W_trim, hipStream_t st) {
    GatherBatch gb;
    int kmax = 1;
    for (int hd = 0; hd < kSelectMaxHeads; ++hd) {
        gb.k[hd] = hd < n_heads ? k[hd] : 0;
        gb.map[hd] = hd < n_heads ? map[hd] : nullptr;
        gb.W_trim[hd] = hd < n_heads ? static_cast<char *>(W_trim[hd]) : nullptr;
        if (hd < n_heads && k[hd] > kmax) kmax = k[hd];
    }
    int blocks = (kmax + 3) / 4;          // 4 waves per workgroup
    if (blocks > 2048) blocks = 2048;
    hipLaunchKernelGGL(gather_rows_heads_kernel, dim3(blocks, n_heads), dim3(256), 0, st, static_cast<const char *>(W),
                       row_bytes, gb);
}

void launch_gather_rows(const void *W, size_t row_bytes, const int *map, int k, void *W_trim, hipStream_t st) {
    int blocks = (k + 3) / 4;          // 4 waves per workgroup
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(gather_rows_kernel, dim3(blocks), dim3(256), 0, st, static_cast<const char *>(W), row_bytes,
                       map, k, static_cast<char *>(W_trim));
}

}  // namespace vt
