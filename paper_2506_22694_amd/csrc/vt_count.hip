// Algorithm 1 (Count Token Frequencies): c[t] += 1 for every token id of the stream.
//
// The V counters do not fit one CU's LDS as 32-bit words (V = 128256 -> 513 KB), so the bins
// are 16 bits wide, two per LDS word, the vocabulary is cut into ranges of 65536 bins (128 KiB of
// LDS; two ranges for V = 128256) and the id stream into chunks.  Workgroup (chunk, range) reads
// its chunk with 16-byte loads, counts the ids that fall into its range with LDS atomics (no
// global atomic sees the Zipf-hot ids more than once per 32768 occurrences), and writes its private histogram to scratch:
// the low eight bits of every bin, and the upper eight of those groups of 256 ids that have any, which a flag tells (a few
// dozen ids of a chunk exceed 255, next to each other where ids follow the frequency).
// A second kernel sums the chunk histograms into the caller's int64 counters.  Ids outside [0, V) are skipped and tallied.
// What bounds it is what a CU does per id and range: ten vector instructions (no branch, no mask) and an LDS atomic.  The waves
// share their hottest bin through words of their own, without which the workgroups that have it took a third longer (10^8 ids, Zipf
// 1.1: 135 -> 99 us; one id alone 670 -> 101); an LDS atomic under a mask per id cost four scalar instructions and a branch
// (10^7 ids 25.0 -> 22.1 us, 64-bit 29.8 -> 28.4, in equal shares 21.6 -> 20.2).  Beyond that it is the reading of the stream once
// per range: more in flight makes it slower (64-bit, 10^8: four vectors per thread 165 us, six 175, eight 205, six twice 200, two
// 201), since the two workgroups of a chunk drift apart and miss each other's lines in the L2.
//
// A 16-bit bin never holds much more than 15 bits: an increment that finds bit 15 set clears it, and whoever found it set when
// clearing adds 32768 to the result counter.  Until then the bin can only grow by the increments in flight in the workgroup
// (eight per thread, twice: 16384 at most), short of 65536, so a bin never carries into its neighbour in the same word,
// whatever the id distribution.
#include "vt_build.h"
#include "vt_device.h"
#include "vt_launch.h"
#include <type_traits>

namespace vt {

int hist_num_ranges(int V) { return (V + kHistBinsPerBlock - 1) / kHistBinsPerBlock; }

// Chunks of at least `ids` ids; chunks x ranges = one round of workgroups over the 256 CUs at most
static int chunks_of(int64_t n_ids, int V, int ids) {
    int cap = kHistBlocks / hist_num_ranges(V);
    if (cap < 1) cap = 1;
    const int64_t c = (n_ids + ids - 1) / ids;
    return c < 1 ? 1 : c > cap ? cap : (int)c;
}
// A chunk's rows are written and summed for all V ids: with eleven and more ranges of bins that is the larger part of a short
// stream (V = 10^6, 200 000 ids: chunks of 16384 26.2 us, of 65536 22.7; V = 700 000 21.4 / 20.2; V = 500 000 18.1 / 18.4, of
// 32768 18.0, and 10^6 ids 24.2 / 25.1 / 21.3; V = 300 000 14.5 / 16.4).
int hist_num_chunks(int64_t n_ids, int V) {
    const int ranges = hist_num_ranges(V);
    return chunks_of(n_ids, V, kHistChunkIds * (ranges < 8 ? 1 : ranges < 11 ? 2 : 4));
}

// What lies between the two kernels: rows of the low bytes and of the upper bytes of the chunks' bins, and a flag per group of
// 256 ids and chunk: whether the group's upper bytes are there.
constexpr int kGroupIds = 256;
struct HistScratch {
    size_t pitch, groups;                          // bytes per row: V rounded up to four; groups of 256 ids
    unsigned char *low, *high, *flags;             // [nchunks][pitch] twice, [nchunks][groups]
    __host__ __device__ HistScratch(unsigned char *p, int V, int nchunks) {
        pitch = ((size_t)V + 3) & ~(size_t)3;
        groups = ((size_t)V + kGroupIds - 1) / kGroupIds;
        low = p;
        high = low + pitch * nchunks;
        flags = high + pitch * nchunks;
    }
};
static size_t chunk_bytes(int V) {
    const HistScratch sc(nullptr, V, 1);
    return 2 * sc.pitch + sc.groups;
}
size_t hist_scratch_bytes(int V, int64_t n_ids) { return hist_num_chunks(n_ids, V) * chunk_bytes(V); }
// (a scratch of this size is enough, for fewer chunks)
size_t hist_min_scratch_bytes(int V, int64_t n_ids) { return chunks_of(n_ids, V, 1 << 16) * chunk_bytes(V); }

// `head` ids (fewer than one 16-byte vector) precede the first 16-byte aligned id.
constexpr int kHistWaves = kHistThreads / kWave;
constexpr unsigned kHistHot = 128;      // increments of one bin among a workgroup's first two vectors per thread (8192 ids, 4096 of 64 bits) that make it a hot one
// LDS: the bins, and behind them (see the kernel)
constexpr unsigned kHistHotAt = kHistBinsPerBlock * 2, kHistAsideAt = kHistHotAt + 4 * kHistThreads, kHistHotBinAt = kHistAsideAt + 4 * kWave;
constexpr unsigned kHistLaterAt = kHistHotBinAt + 4 * kHistWaves, kHistLds = kHistLaterAt + 4;
constexpr unsigned kNoHot = 0xFFFFFFFFu;
// SHORT: no chunk has a whole batch of vectors.  Nothing then has a hottest bin, and without its words and their sum a stream of
// 1000 ids takes 7.5 us and not 7.8 (V = 128256; 7.4 before there were any), one of 10^6 14.1 and not 14.5.
template <bool IDS64, bool SHORT>
__global__ void __launch_bounds__(kHistThreads) hist_partial_kernel(const void *__restrict__ ids_v, long long n_ids,
                                                                    int head, int V, int nchunks,
                                                                    unsigned char *partial,
                                                                    unsigned long long *__restrict__ counts,
                                                                    unsigned long long *__restrict__ n_invalid) {
    // two 16-bit bins per word; behind them (one block of LDS, so that a bin's offset is its address)
    //   hot     a word per thread: its ids of the wave's hottest bin
    //   aside   a word per lane: where ids of other ranges go
    //   hot_bin the waves' hottest bins, where their ids are many; and whether any are
    extern __shared__ __align__(16) unsigned words[];
    // (LDS addresses as numbers: what the compiler knows as a pointer it forms again for every access)
    typedef __attribute__((address_space(3))) unsigned lds_word;
    const unsigned base = (unsigned)(uintptr_t)(lds_word *)words;
    const int chunk = blockIdx.x, range = blockIdx.y;
    const int lo = range * kHistBinsPerBlock;
    const int nb = min(kHistBinsPerBlock, V - lo);
    const int nw = ((nb + 3) & ~3) >> 1;                  // whole groups of four bins: the rows are written by fours
    const unsigned hot_at = base + kHistHotAt + 4u * threadIdx.x, aside_at = base + kHistAsideAt + 4u * (threadIdx.x & 63u);
    unsigned &hot_word = words[kHistHotAt / 4 + threadIdx.x];
    for (int b = threadIdx.x; b < nw; b += kHistThreads) words[b] = 0u;
    if constexpr (!SHORT) hot_word = 0u;
    if (threadIdx.x < kWave) words[kHistAsideAt / 4 + threadIdx.x] = 0u;
    if constexpr (!SHORT) {
        if (threadIdx.x < kHistWaves) words[kHistHotBinAt / 4 + threadIdx.x] = kNoHot;
        if (threadIdx.x == 0) words[kHistLaterAt / 4] = 0u;
    }
    __syncthreads();

    // chunk boundaries in units of 16-byte vectors (4 int32 or 2 int64), tail handled by the last chunk
    constexpr int IPV = IDS64 ? 2 : 4;
    constexpr int IDB = IDS64 ? 8 : 4;
    const long long nvec = (n_ids - head) / IPV;
    const long long v0 = nvec * chunk / nchunks, v1 = nvec * (chunk + 1) / nchunks;
    unsigned invalid = 0;
    // One id.  (The scalar head and tail of the stream, a few ids at most.)
    auto tally = [&](long long t) {
        if ((unsigned long long)t >= (unsigned long long)V) {
            invalid += 1u;
        } else {
            const unsigned b = (unsigned)((int)t - lo);
            if (b < (unsigned)nb) atomicAdd(&words[b >> 1], 1u << ((b & 1u) << 4));
        }
    };
    // The wave's hottest bin, as far as it has seen: its ids are counted in words that the threads have to themselves.  (With
    // Zipf ids eight lanes of 64 hit the hottest bin, and LDS atomics on one address queue.)
    unsigned hot = kNoHot;
    bool looked = false;
    // The ids of NV 16-byte vectors: all their LDS atomics are issued before the first result is looked at -- a
    // wave that waited for every atomic's return before the next id spent most of its time in that wait -- and the
    // rare bin that has reached 32768 is handled behind one test for the whole batch.
    constexpr int IPV0 = IDS64 ? 2 : 4;
    auto tally_ids = [&](auto ncount, auto with_hot, unsigned *t, const unsigned *high) {
        constexpr int N = decltype(ncount)::value;
        constexpr bool HOT = decltype(with_hot)::value;      // the wave has a hottest bin
        // 64-bit ids with anything in the upper half are outside [0, V), V < 2^31: rare, so one test for the batch, which makes
        // them 32-bit ids outside
        if constexpr (IDS64) {
            unsigned some = 0u;
#pragma unroll
            for (int q = 0; q < N; ++q) some |= high[q];
            if (some != 0u) {
#pragma unroll
                for (int q = 0; q < N; ++q) t[q] = high[q] != 0u ? 0xFFFFFFFFu : t[q];
            }
        }
        // ids outside [0, V): one test for the batch as well (the largest id; a negative one is a large unsigned number) and the
        // count behind it; only the workgroups of range 0 report them
        if (range == 0) {
            unsigned mx = t[0];
#pragma unroll
            for (int q = 1; q < N; ++q) mx = t[q] > mx ? t[q] : mx;
            if (mx >= (unsigned)V) {
#pragma unroll
                for (int q = 0; q < N; ++q) invalid += t[q] >= (unsigned)V ? 1u : 0u;
            }
        }
        // Every lane adds somewhere -- its bin, its own word, or aside -- so that nothing is branched or masked per id.
        unsigned b[N], at[N], inc[N], old[N];
#pragma unroll
        for (int q = 0; q < N; ++q) {
            // bin inside this range; an id outside [lo, lo + nb) wraps far past nb
            b[q] = t[q] - (unsigned)lo;
            const unsigned even = b[q] & ~1u;
            asm("v_lshl_add_u32 %0, %1, 1, %2" : "=v"(at[q]) : "v"(even), "s"(base));      // (the compiler takes one instruction more)
            if constexpr (HOT) at[q] = b[q] == hot ? hot_at : at[q];
            at[q] = b[q] < (unsigned)nb ? at[q] : aside_at;
            inc[q] = 1u << (b[q] << 4 & 31u);        // 1 for the low half of the word, 0x10000 for the high one
        }
#pragma unroll
        for (int q = 0; q < N; ++q) old[q] = __hip_atomic_fetch_add((lds_word *)(uintptr_t)at[q], inc[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        unsigned any = 0u;
#pragma unroll
        for (int q = 0; q < N; ++q) any |= old[q];
        if ((any & 0x80008000u) != 0u) {
#pragma unroll
            for (int q = 0; q < N; ++q) {
                if ((old[q] & 0x80008000u) != 0u) {
                    unsigned *const word = words + (at[q] - base) / 4;
                    if (at[q] == aside_at) {
                        *word = 0u;
                    } else if (HOT && at[q] == hot_at) {
                        atomicAdd(&counts[lo + (int)hot], (unsigned long long)(atomicExch(word, 0u) >> ((hot & 1u) << 4)));
                    } else {
                        // whoever finds bit 15 set when it is cleared moves the bin's 32768 to the result counter
                        const unsigned was = atomicAnd(word, 0x7FFF7FFFu);
                        if ((was & 0x8000u) != 0u) atomicAdd(&counts[lo + (int)(b[q] & ~1u)], 32768ull);
                        if ((was & 0x80000000u) != 0u) atomicAdd(&counts[lo + (int)(b[q] | 1u)], 32768ull);
                    }
                }
            }
        }
        if constexpr (!HOT && !SHORT) {
            if (!looked) {
                // once, after the first ids: the bin that the wave found fullest, where it is one of the workgroup's hottest
                looked = true;
                unsigned most = 0u, bin = 0u;
#pragma unroll
                for (int q = 0; q < N; ++q) {
                    const unsigned o = at[q] == aside_at ? 0u : old[q] >> ((b[q] & 1u) << 4) & 0xFFFFu;
                    bin = o > most ? b[q] : bin;
                    most = o > most ? o : most;
                }
                const unsigned wave_most = wave_max_u32(most);
                if (__ballot(true) == ~0ull && wave_most >= kHistHot)
                    hot = (unsigned)__builtin_amdgcn_readlane((int)bin, __ffsll((long long)__ballot(most == wave_most)) - 1);
            }
        }
    };
    const u32x4 *vp = reinterpret_cast<const u32x4 *>(static_cast<const char *>(ids_v) + (size_t)head * IDB);
    auto unpack = [&](const u32x4 q, unsigned *t, unsigned *high) {
        t[0] = q.x;
        if constexpr (IDS64) {
            high[0] = q.y;
            t[1] = q.z;
            high[1] = q.w;
        } else {
            t[1] = q.y;
            t[2] = q.z;
            t[3] = q.w;
        }
    };
    auto tally_vec = [&](auto with_hot, const u32x4 q) {
        unsigned t[IPV0], high[2];
        unpack(q, t, high);
        tally_ids(std::integral_constant<int, IPV0>{}, with_hot, t, high);
    };
    auto tally_vec2 = [&](auto with_hot, const u32x4 q0, const u32x4 q1) {
        unsigned t[2 * IPV0], high[4];
        unpack(q0, t, high);
        unpack(q1, t + IPV0, high + 2);
        tally_ids(std::integral_constant<int, 2 * IPV0>{}, with_hot, t, high);
    };
    // kHistUnroll vectors per thread are requested at a time: one 16-byte load per
    // thread in flight (16 KiB per CU) is far below what the memory latency needs.  Plain (cached) loads:
    // the workgroups of one chunk (one per range) are dispatched to the same XCD and read the same ids at
    // about the same time, so three of the four reads can hit its L2; a streaming hint would drop the
    // lines after the first use (10^7 ids: 41.2 -> 35.1 us)
    // (Buffer loads: a uniform address and the thread's own offset.  With 64-bit addresses per thread the compiler kept one of
    // them where the next vector arrives, and waited for a batch's first vector before it requested the others.)
    constexpr int kBatch = kHistUnroll * kHistThreads;
    static_assert(kHistUnroll % 2 == 0, "vectors are counted in pairs");
    const u32x4 *at_vec = vp + v0;
    long long left = v1 - v0;
    u32x4 q[kHistUnroll];
    auto descriptor = [&](int vectors) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<u32x4 *>(at_vec), 0, vectors * 16, 0x00020000); };
    for (; !SHORT && left >= kBatch; left -= kBatch, at_vec += kBatch) {
        // (the scalar offsets stay below the size, which is a constant here.  They are no part of the check against it, or are
        // subtracted from it: beside a smaller size they would reach past the end)
        const auto rsrc = descriptor(kBatch);
#pragma unroll
        for (int u = 0; u < kHistUnroll; ++u) q[u] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, threadIdx.x * 16, u * kHistThreads * 16, 0);
#pragma unroll
        for (int u = 0; u < kHistUnroll; u += 2) {
            if (hot != kNoHot)
                tally_vec2(std::true_type{}, q[u], q[u + 1]);
            else
                tally_vec2(std::false_type{}, q[u], q[u + 1]);
        }
    }
    looked = true;      // (fewer lanes from here on)
    if (left > 0) {
        // (fewer than a batch; a thread past the end reads the last vector again, and does not count it)
        const auto rsrc = descriptor((int)left);
#pragma unroll
        for (int u = 0; u < kHistUnroll; ++u)
            q[u] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, min(u * kHistThreads + (int)threadIdx.x, (int)left - 1) * 16, 0, 0);
#pragma unroll
        for (int u = 0; u < kHistUnroll; ++u) {
            if (u * kHistThreads + (int)threadIdx.x < left) {
                if (!SHORT && hot != kNoHot)
                    tally_vec(std::true_type{}, q[u]);
                else
                    tally_vec(std::false_type{}, q[u]);
            }
        }
    }
    if (chunk == 0 && (int)threadIdx.x < head) {   // scalar head
        if constexpr (IDS64) tally(static_cast<const long long *>(ids_v)[threadIdx.x]);
        else tally((long long)static_cast<const int *>(ids_v)[threadIdx.x]);
    }
    if (chunk == nchunks - 1) {   // scalar tail (< IPV ids)
        const long long i = head + nvec * IPV + threadIdx.x;
        if (i < n_ids) {
            if constexpr (IDS64) tally(static_cast<const long long *>(ids_v)[i]);
            else tally((long long)static_cast<const int *>(ids_v)[i]);
        }
    }
    // The threads' own words: the wave's sum goes to its bin at once while it is small (sixteen waves' 1023 at most beside the
    // 49151 that a bin may hold: no carry), otherwise one wave adds the sums behind the barrier.
    if constexpr (!SHORT) {
        const unsigned sum = (unsigned)wave_sum_i32((int)(hot_word >> ((hot & 1u) << 4)));
        if (lane_id() == 0 && sum != 0u) {
            if (sum < 1024u) {
                atomicAdd(&words[hot >> 1], sum << ((hot & 1u) << 4));
            } else {
                words[kHistHotAt / 4 + threadIdx.x] = sum;
                words[kHistHotBinAt / 4 + (threadIdx.x >> 6)] = hot;
                words[kHistLaterAt / 4] = 1u;
            }
        }
    }
    __syncthreads();
    if (!SHORT && words[kHistLaterAt / 4] != 0u) {      // (uniform)
        if (threadIdx.x < kWave) {
            // most often all waves have the same hottest bin: one lane adds all that belong to a bin
            const int w = min((int)threadIdx.x, kHistWaves - 1);
            const unsigned bin = words[kHistHotBinAt / 4 + w];
            const unsigned n = bin != kNoHot && (int)threadIdx.x < kHistWaves ? words[kHistHotAt / 4 + kWave * w] : 0u;
            unsigned long long left = __ballot(n != 0u);
            while (left != 0ull) {
                const int leader = __ffsll((long long)left) - 1;
                const bool same = bin == (unsigned)__builtin_amdgcn_readlane((int)bin, leader);
                const unsigned sum = (unsigned)wave_sum_i32(same ? (int)n : 0);
                if ((int)threadIdx.x == leader) {
                    unsigned &word = words[bin >> 1];
                    const unsigned sh = (bin & 1u) << 4, total = (word >> sh & 0xFFFFu) + sum, keep = total & 0x7FFFu;
                    word = (word & ~(0xFFFFu << sh)) | keep << sh;
                    if (total != keep) atomicAdd(&counts[lo + (int)bin], (unsigned long long)(total - keep));
                }
                left &= ~__ballot(same);
                // (the next leader's bin may share the word)
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            }
        }
        __syncthreads();
    }
    // A row of the scratch holds eight bits per id, half the size of the bins; rows of the upper eight bits lie behind them
    // and are written, and read back, for the groups of 256 ids alone that have any.  (Those bits added to the result by
    // atomics instead: all chunks to the same few counters, one behind the other where hot ids share a cache line -- Zipf ids
    // in order of frequency, V = 128256, 10^7 45.9 us against 26.4, V = 32000, 10^8 131 / 94; in random order 24.7 / 25.0.)
    const HistScratch sc(partial, V, nchunks);
    unsigned char *dst = sc.low + (size_t)chunk * sc.pitch + lo, *dst_hi = sc.high + (size_t)chunk * sc.pitch + lo;
    unsigned char *flags = sc.flags + (size_t)chunk * sc.groups + lo / kGroupIds;
    auto low_bytes = [](unsigned w0, unsigned w1) { return __builtin_amdgcn_perm(w1, w0, 0x06040200u); };      // of two words, four bins
    auto high_bytes = [](unsigned w0, unsigned w1) { return __builtin_amdgcn_perm(w1, w0, 0x07050301u); };
    if ((V & 15) == 0) {
        for (int b = 16 * threadIdx.x; b < nb; b += 16 * kHistThreads) {      // sixteen lanes hold a group
            const u32x4 x0 = *reinterpret_cast<const u32x4 *>(words + b / 2), x1 = *reinterpret_cast<const u32x4 *>(words + b / 2 + 4);
            const unsigned any = (x0.x | x0.y | x0.z | x0.w | x1.x | x1.y | x1.z | x1.w) & 0xFF00FF00u;
            const bool flagged = (__ballot(any != 0u) >> (threadIdx.x & 48) & 0xFFFFull) != 0ull;
            u32x4 y;
            y.x = low_bytes(x0.x, x0.y);
            y.y = low_bytes(x0.z, x0.w);
            y.z = low_bytes(x1.x, x1.y);
            y.w = low_bytes(x1.z, x1.w);
            *reinterpret_cast<u32x4 *>(dst + b) = y;
            if (flagged) {
                y.x = high_bytes(x0.x, x0.y);
                y.y = high_bytes(x0.z, x0.w);
                y.z = high_bytes(x1.x, x1.y);
                y.w = high_bytes(x1.z, x1.w);
                *reinterpret_cast<u32x4 *>(dst_hi + b) = y;
            }
            if ((threadIdx.x & 15) == 0) flags[b / kGroupIds] = flagged ? 1 : 0;
        }
    } else {
        for (int b = 4 * threadIdx.x; b < nb; b += 4 * kHistThreads) {      // a wave holds a group
            const unsigned w0 = words[b / 2], w1 = words[b / 2 + 1];
            const bool flagged = __ballot(((w0 | w1) & 0xFF00FF00u) != 0u) != 0ull;
            *reinterpret_cast<unsigned *>(dst + b) = low_bytes(w0, w1);
            if (flagged) *reinterpret_cast<unsigned *>(dst_hi + b) = high_bytes(w0, w1);
            if ((threadIdx.x & 63) == 0) flags[b / kGroupIds] = flagged ? 1 : 0;
        }
    }
    // every range-workgroup of a chunk sees the same invalid ids: only range 0 reports them
    if (n_invalid != nullptr && range == 0) {
        const int tot = wave_sum_i32((int)invalid);
        if (lane_id() == 0 && tot != 0) atomicAdd(n_invalid, (unsigned long long)tot);
    }
}

// A workgroup sums a group of 256 neighbouring ids (a 4-byte word per lane) over the chunks: wave g takes the chunks g,
// g + 8, .., sixteen loads in flight; the words' bytes are added as pairs of 16 bits (at most 256 chunks of 255: 65280), and
// the eight partial sums meet in LDS.
constexpr int kReduceWaves = 8;
__global__ void __launch_bounds__(kReduceWaves *kWave) hist_reduce_kernel(unsigned char *partial, int nchunks, int V,
                                                                          long long *__restrict__ counts) {
    __shared__ unsigned part[kReduceWaves][4][kWave];
    const HistScratch sc(partial, V, nchunks);
    const int lane = (int)threadIdx.x & 63, g = (int)threadIdx.x >> 6;
    const int wi = blockIdx.x * kWave + lane;
    const int Vw = (int)(sc.pitch >> 2);           // words per scratch row
    const unsigned *low = reinterpret_cast<const unsigned *>(sc.low), *high = reinterpret_cast<const unsigned *>(sc.high);
    // the wave's chunks g + 8 l whose upper bits have to be read (requested with the first rows)
    const int mine = g + kReduceWaves * lane;
    const unsigned char flag = sc.flags[(size_t)min(mine, nchunks - 1) * sc.groups + blockIdx.x];
    // (every load is made, past the end that of the last word or chunk: a branch around one would wait for it)
    const int at = min(wi, Vw - 1);
    unsigned even = 0, odd = 0;                    // ids 4 wi, 4 wi + 2 and 4 wi + 1, 4 wi + 3
    unsigned even_hi = 0, odd_hi = 0;
    constexpr int kLoads = 16;
    unsigned upper = 0;                            // bit l: chunk g + 8 l
    for (int l0 = 0; g + kReduceWaves * l0 < nchunks; l0 += kLoads) {
        unsigned t[kLoads], t_hi[kLoads] = {};
#pragma unroll
        for (int u = 0; u < kLoads; ++u) {
            const int c = g + kReduceWaves * (l0 + u);
            t[u] = low[(size_t)min(c, nchunks - 1) * Vw + at];
        }
        if (l0 == 0) {
            // the flags are the oldest load: the rows stay in flight (the test is kept from moving up ahead of them)
            unsigned f = flag;
            asm volatile("" : "+v"(f));
            upper = (unsigned)__ballot(f != 0u && mine < nchunks);
        }
        const unsigned now = upper >> l0 & ((1u << kLoads) - 1u);
        if (now != 0u) {
#pragma unroll
            for (int u = 0; u < kLoads; ++u)
                t_hi[u] = high[(size_t)min(g + kReduceWaves * (l0 + u), nchunks - 1) * Vw + at];
        }
#pragma unroll
        for (int u = 0; u < kLoads; ++u) {
            const unsigned x = g + kReduceWaves * (l0 + u) < nchunks ? t[u] : 0u;
            even += x & 0x00FF00FFu;
            odd += (x >> 8) & 0x00FF00FFu;
        }
        if (now != 0u) {
#pragma unroll
            for (int u = 0; u < kLoads; ++u) {
                const unsigned x = (now >> u & 1u) != 0u ? t_hi[u] : 0u;      // (the others were never written)
                even_hi += x & 0x00FF00FFu;
                odd_hi += (x >> 8) & 0x00FF00FFu;
            }
        }
    }
    static_assert(kHistBlocks / kReduceWaves <= 32, "a bit per chunk of a wave");
    part[g][0][lane] = even;
    part[g][1][lane] = odd;
    part[g][2][lane] = even_hi;
    part[g][3][lane] = odd_hi;
    __syncthreads();
    // thread t < 256: id 256 * block + t
    const int t = (int)threadIdx.x, id = blockIdx.x * kGroupIds + t;
    if (t < kGroupIds && id < V) {
        unsigned sum = 0, sum_hi = 0;
#pragma unroll
        for (int q = 0; q < kReduceWaves; ++q) {
            sum += part[q][t & 1][t >> 2] >> (8 * (t & 2)) & 0xFFFFu;
            sum_hi += part[q][2 + (t & 1)][t >> 2] >> (8 * (t & 2)) & 0xFFFFu;
        }
        counts[id] += (long long)(sum + (sum_hi << 8));
    }
}
static_assert(kHistBlocks <= 257, "sums over the chunks of eight-bit parts fit 16 bits");

hipError_t launch_count_tokens(const void *ids, bool ids64, int64_t n_ids, int V, long long *counts,
                         unsigned long long *n_invalid, void *partial, size_t partial_bytes, hipStream_t st) {
    int nchunks = hist_num_chunks(n_ids, V);
    if (nchunks * chunk_bytes(V) > partial_bytes) nchunks = (int)(partial_bytes / chunk_bytes(V));
    if (nchunks < 1) return hipErrorInvalidValue;
    const size_t lds = kHistLds;
    static LdsLimitOnce lds_limit;
    hipError_t e = allow_dynamic_lds(lds_limit,
                                     {reinterpret_cast<const void *>(hist_partial_kernel<false, false>),
                                      reinterpret_cast<const void *>(hist_partial_kernel<true, false>),
                                      reinterpret_cast<const void *>(hist_partial_kernel<false, true>),
                                      reinterpret_cast<const void *>(hist_partial_kernel<true, true>)}, (int)lds);
    if (e != hipSuccess) return e;
    // ids before the first 16-byte boundary are counted one by one
    const int idb = ids64 ? 8 : 4;
    const uintptr_t mis = reinterpret_cast<uintptr_t>(ids) & 15u;
    long long head = mis ? (long long)((16 - mis) / idb) : 0;
    if (head > n_ids) head = n_ids;
    unsigned char *scratch = static_cast<unsigned char *>(partial);
    // chunks without a whole batch: the kernel that knows no hottest bin
    const bool brief = ((n_ids - head) * idb / 16 + nchunks - 1) / nchunks < kHistUnroll * kHistThreads;
    auto partial_kernel = ids64 ? (brief ? hist_partial_kernel<true, true> : hist_partial_kernel<true, false>)
                                : (brief ? hist_partial_kernel<false, true> : hist_partial_kernel<false, false>);
    hipLaunchKernelGGL(partial_kernel, dim3(nchunks, hist_num_ranges(V)), dim3(kHistThreads), lds, st, ids, (long long)n_ids,
                       (int)head, V, nchunks, scratch, reinterpret_cast<unsigned long long *>(counts), n_invalid);
    hipLaunchKernelGGL(hist_reduce_kernel, dim3((V + kGroupIds - 1) / kGroupIds), dim3(kReduceWaves * kWave), 0, st, scratch,
                       nchunks, V, counts);
    return hipGetLastError();
}

}  // namespace vt
