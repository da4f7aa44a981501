// Eq. 1 of the paper: V_trim = V[Top-K(c, k)], W_trim = W[Top-K(c, k), :].
//
// Selection = the k-th largest count (threshold T, and the number r of T-valued ids to keep; ties go to the lower id),
// then an id-ordered compaction that emits the selected ids already ascending -- no sort.  It runs over the whole device,
// one workgroup per 1024 ids, as four small launches, each a chain of latencies (launch, memory, scan) and not of work:
//   sel_zero    clears the histogram
//   sel_hist    histogram of all counts over 3744 bins, exact values below 2048 (vt_code.h)
//   sel_count   every workgroup finds the bin of the k-th largest count.  Below 2048 that bin is T itself, and the
//               workgroup tallies its ids above / at T.  A larger T is refined inside its bin by the first workgroup, which
//               reads all counts again (10 us per eight bits at V = 128256; only when the k-th largest count is that large)
//   sel_write   the compaction: ballots, and the tallies of the workgroups before this one
// (A radix select byte by byte took eleven launches, 47 us at V = 128256 after 10^7 tokens; this one 18.)
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
    unsigned long long *thresh;   // T
    int *take;                    // r; tallied: 1 = tab is valid
    int *tallied;
    unsigned *tab;                // [nblk][2] ids above / at the threshold per workgroup
};

// Several heads per launch (grid.y = head): head y selects k[y] of the counts at counts + y V into map[y], with
// the scratch of a single selection at scratch + y stride.
struct SelBatch {
    unsigned char *scratch;
    size_t stride;
    int nblk;
    int k[kSelectMaxHeads];
    int *map[kSelectMaxHeads];
};
constexpr size_t kSelTabOffset = (size_t)kBins * sizeof(unsigned) + 16;
static_assert((kBins * sizeof(unsigned)) % 8 == 0, "the threshold behind the histogram is aligned");
__device__ __forceinline__ SelBufs head_bufs(const SelBatch &sb) {
    unsigned char *p = sb.scratch + (size_t)blockIdx.y * sb.stride;
    SelBufs b;
    b.hist = reinterpret_cast<unsigned *>(p);
    b.thresh = reinterpret_cast<unsigned long long *>(p + kBins * sizeof(unsigned));
    b.take = reinterpret_cast<int *>(b.thresh + 1);
    b.tallied = b.take + 1;
    b.tab = reinterpret_cast<unsigned *>(p + kSelTabOffset);
    return b;
}

__global__ void __launch_bounds__(256) sel_zero_kernel(SelBatch sb) {
    unsigned *p = head_bufs(sb).hist;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < kBins; i += gridDim.x * 256) p[i] = 0u;
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
    const int bin = count_bin(c);
    // the ids of a wave that share the first one's bin are added at once: in the tail most counts are the same
    const unsigned long long live = __ballot(in);
    const int first = __builtin_amdgcn_readfirstlane(bin);
    const unsigned long long same = __ballot(in && bin == first);
    if (in && bin != first) atomicAdd(&h[bin], 1u);
    if (live != 0ull && lane_id() == 0) atomicAdd(&h[first], (unsigned)__popcll(same));      // (lane 0 is live if any is)
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
    __shared__ unsigned h[256];
    __shared__ int s_bin, s_rem;
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
    }
    if (blockIdx.x != 0) return;
    unsigned long long T = (unsigned)bin;
    if (bin >= kBinExact) {
        // several values share the bin: the rest of T, up to eight bits at a time, from the counts that agree with it so far
        T = bin_prefix(bin);
        for (int left = bin_shift(bin); left > 0;) {
            const int bits = left < 8 ? left : 8;
            left -= bits;
            if (tid < 256) h[tid] = 0u;
            __syncthreads();
            for (int x = tid; x < V; x += kSelectThreads) {
                const unsigned long long cx = (unsigned long long)counts[x];
                if ((cx >> (left + bits)) == T) atomicAdd(&h[(unsigned)(cx >> left) & ((1u << bits) - 1u)], 1u);
            }
            __syncthreads();
            const unsigned mine_d = tid < 256 ? h[255 - tid] : 0u;      // digits from the highest down
            const unsigned upto = block_scan(mine_d, part);
            if (upto >= (unsigned)rem && upto - mine_d < (unsigned)rem) {
                s_bin = 255 - tid;
                s_rem = rem - (int)(upto - mine_d);
            }
            __syncthreads();
            T = (T << bits) | (unsigned)s_bin;
            rem = s_rem;
            __syncthreads();
        }
    }
    if (tid == 0) {
        *b.thresh = T;
        *b.take = rem;
        *b.tallied = bin < kBinExact ? 1 : 0;
    }
}

__global__ void __launch_bounds__(kSelectThreads) sel_write_kernel(const long long *__restrict__ counts_all, int V,
                                                                   SelBatch sb) {
    const SelBufs b = head_bufs(sb);
    const long long *__restrict__ counts = counts_all + (size_t)blockIdx.y * V;
    int *__restrict__ map = sb.map[blockIdx.y];
    __shared__ int s_gt[kSelWaves], s_eq[kSelWaves], s_gb[kSelWaves], s_eb[kSelWaves];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    // everything is requested at once: this thread's count, the threshold, the tallies of the workgroups before this one
    const int j = blockIdx.x * kSelectThreads + tid;
    const unsigned long long c = j < V ? (unsigned long long)counts[j] : 0ull;
    const unsigned long long T = *b.thresh;
    const int r = *b.take, tallied = *b.tallied;
    int gb = 0, eb = 0;
    for (int x = tid; x < (int)blockIdx.x; x += kSelectThreads) {
        gb += (int)b.tab[2 * x];
        eb += (int)b.tab[2 * x + 1];
    }
    if (tallied == 0) {      // (uniform) the tallies are those of T's bin: count the ids before this workgroup again
        gb = eb = 0;
        for (int x = tid; x < (int)blockIdx.x * kSelectThreads; x += kSelectThreads) {
            const unsigned long long cx = (unsigned long long)counts[x];
            gb += cx > T ? 1 : 0;
            eb += cx == T ? 1 : 0;
        }
    }
    gb = wave_sum_i32(gb);
    eb = wave_sum_i32(eb);
    const bool gt = j < V && c > T, eq = j < V && c == T;
    const unsigned long long bg = __ballot(gt), be = __ballot(eq);
    if (lane == 0) {
        s_gb[w] = gb;
        s_eb[w] = eb;
        s_gt[w] = __popcll(bg);
        s_eq[w] = __popcll(be);
    }
    __syncthreads();
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
    hipLaunchKernelGGL(sel_zero_kernel, dim3(4, n_heads), dim3(256), 0, st, sb);
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
