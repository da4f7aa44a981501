// Internal interface of the calibration-side kernels (count, select, gather).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

namespace vt {

// ---- Algorithm 1 ----
constexpr int kHistBinsPerBlock = 65536;   // 16-bit bins privatised in LDS per workgroup (128 KiB, two per word)
constexpr int kHistBlocks = 256;           // workgroups per launch: id-stream chunks x bin ranges
constexpr int kHistThreads = 1024;
constexpr int kHistChunkIds = 16384;      // ids of a chunk at least, with up to seven ranges (this kernel at V = 128256 with chunks of
                                          // 4096 / 8192 / 16384 / 32768 / 65536: 10^6 ids 16.8 / 16.6 / 14.5 / 14.0 / 16.0 us, 64-bit
                                          // 17.2 / 16.6 / 15.0 / 15.2 / 18.3, 200 000 11.4 / 10.6 / 11.1 / 12.5 / 13.6)
constexpr int kHistUnroll = 4;            // 16-byte id vectors in flight per thread (2 / 4 / 6: 24.9 / 22.1 / 22.8 us at
                                          // 10^7 ids, 130 / 99 / 101 at 10^8, 64-bit 202 / 165 / 175)

int hist_num_ranges(int V);
int hist_num_chunks(int64_t n_ids, int V);
size_t hist_scratch_bytes(int V, int64_t n_ids);
size_t hist_min_scratch_bytes(int V, int64_t n_ids);
// partial: hist_scratch_bytes(V, n_ids), or from hist_min_scratch_bytes(V, n_ids) on with fewer chunks; no initialisation
hipError_t launch_count_tokens(const void *ids, bool ids64, int64_t n_ids, int V, long long *counts,
                         unsigned long long *n_invalid, void *partial, size_t partial_bytes, hipStream_t st);

// ---- Eq. 1 ----
constexpr int kSelectThreads = 1024;
constexpr int kSelectMaxHeads = 16;        // heads per batched launch (VT_MAX_HEADS)
// scratch: select_scratch_bytes(V) of device memory, no initialisation
size_t select_scratch_bytes(int V);
void launch_select_topk(const long long *counts, int V, int k, void *scratch, int *map, hipStream_t st);
void launch_gather_rows(const void *W, size_t row_bytes, const int *map, int k, void *W_trim, hipStream_t st);
// several heads per launch sequence (grid.y = head): counts [n_heads, V]; scratch n_heads * select_scratch_stride(V)
size_t select_scratch_stride(int V);
void launch_select_topk_heads(const long long *counts, int V, int n_heads, const int *k, void *scratch, int *const *map,
                              hipStream_t st);
void launch_gather_rows_heads(const void *W, size_t row_bytes, int n_heads, const int *k, const int *const *map,
                              void *const *W_trim, hipStream_t st);

// ---- Sec. 3.2: frequency-rank order, Top-P / minimum-count choice of k ----
constexpr int kRankSortThreads = 1024;
size_t rank_sort_scratch_bytes(int n);
// sorts all n ids by (count desc, id asc); out_ids [n_ids] receives the first n_ids of them
void launch_rank_sort(const long long *counts, int n, void *scratch, int *out_ids, int n_ids, hipStream_t st);
// out: [3] = k, mass of the k largest counts, total mass; scratch: choose_k_ws_bytes(V)
size_t choose_k_ws_bytes(int V);
// up to this V one workgroup does it all (and the workspace holds no tables)
constexpr int kChooseDirectMaxV = 4096;
void launch_choose_k(const long long *counts, int V, int mode, double P, long long f_min, void *scratch, long long *out,
                     hipStream_t st);

}  // namespace vt
