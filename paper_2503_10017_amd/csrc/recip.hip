// The end of the FastNN iteration (paper section 3.2.5, "FastNN Algorithm", step 4): the reduction
// of the matches to a sorted set (a distribution sort over the pixel range).  The reciprocity test
// and the removal of converged seeds (steps 2-3) ride in resolve_step_kernel (search.hip).
#include "fnn_device.hpp"
#include "fnn_kernels.hpp"
#include "trace.hpp"

namespace fnn {

constexpr int DEDUP_THREADS = 1024;
constexpr int DEDUP_AHEAD = 4;
static_assert(MAX_SLOTS + 2 * DEDUP_AHEAD * DEDUP_THREADS <= 0xFFFFFFFFLL, "seeds are counted in 32 bits");
constexpr size_t DEDUP_LDS_BYTES = 60 * 1024;  // dynamic LDS a launch may ask for without raising the kernel's limit (64 KB incl. static)

struct DedupArgs {
    const int32_t* seed_i;
    const int32_t* seed_j;
    const int32_t* seed_iter;
    int32_t n_seeds;
    int32_t n_words;      // ceil(n / 32): words of the per-pair pixel bitmap
    uint32_t* bitmap;     // [batch][n_words], zero on entry
    int32_t* word_rank;   // [batch][n_words] scratch
    int32_t* pairs;
    int32_t* n_pairs;
};

// The match set M, sorted by (i, j) without duplicates.  A match's j is the nearest
// neighbour of its i, so two converged seeds with equal i carry equal j and sorting the
// pairs is sorting their i.  That is done as a distribution sort over the pixel range: mark
// the i of every converged seed in a bitmap, rank the set bits with a prefix sum of word
// popcounts, and let every converged seed write its pair at the rank of its i (seeds that
// share a match write the same value to the same place).
//
// LOCAL: bitmap and ranks live in the workgroup's LDS (passed as dynamic shared memory: n_words
// 32-bit words of bitmap, then n_words ranks of type RANK) instead of the workspace, which takes
// the global-memory round trips out of this latency-bound kernel; the launcher uses it whenever
// the two tables fit, with 16-bit ranks (at most 65535 seeds) for the larger images.
//
// Every thread keeps the loads of DEDUP_AHEAD seeds in flight (1024x768, 12288 seeds: 30.5 -> 18.6 us, 16
// pairs of 3072 seeds 11.1 -> 7.1 us, one pair 6.8 -> 5.2 us): one workgroup per
// pair has nothing else to hide their latency behind, and whether a seed converged decides about its
// match but not about reading it.
template <bool LOCAL, typename RANK>
__global__ __launch_bounds__(DEDUP_THREADS) void recip_dedup_kernel(DedupArgs a) {
    __shared__ int wave_sums[17];
    extern __shared__ uint32_t dedup_tables[];
    const int b = blockIdx.x;
    const int64_t base = (int64_t)b * a.n_seeds;
    const uint32_t n_seeds = a.n_seeds;  // without a sign: the loops below count past the last seed, near 2^31 too
    uint32_t* bitmap = LOCAL ? dedup_tables : a.bitmap + (int64_t)b * a.n_words;
    RANK* word_rank = LOCAL ? reinterpret_cast<RANK*>(dedup_tables + a.n_words)
                            : reinterpret_cast<RANK*>(a.word_rank + (int64_t)b * a.n_words);
    if (LOCAL) {
        for (int w = threadIdx.x; w < a.n_words; w += DEDUP_THREADS) bitmap[w] = 0;
        __syncthreads();
    }

    for (uint32_t s0 = threadIdx.x; s0 < n_seeds; s0 += DEDUP_AHEAD * DEDUP_THREADS) {
        int32_t iter[DEDUP_AHEAD], match[DEDUP_AHEAD];
#pragma unroll
        for (int k = 0; k < DEDUP_AHEAD; ++k) {
            const uint32_t s = min(s0 + k * DEDUP_THREADS, n_seeds - 1);
            iter[k] = a.seed_iter[base + s];
            match[k] = a.seed_i[base + s];
        }
#pragma unroll
        for (int k = 0; k < DEDUP_AHEAD; ++k) {
            const uint32_t i = (uint32_t)match[k];
            if (s0 + k * DEDUP_THREADS < n_seeds && iter[k] >= 0) atomicOr(&bitmap[i >> 5], 1u << (i & 31));
        }
    }
    __syncthreads();

    // contiguous run of words per thread, so that ranks ascend with the thread index; an odd number of them, so that the threads' words lie in
    // different LDS banks (1024x768, 24 words: eight threads of a wave to a bank; the whole call 980.7 -> 976.8 us with 25)
    const int per_thread = ((a.n_words + DEDUP_THREADS - 1) / DEDUP_THREADS) | 1;
    const int w0 = min((int)threadIdx.x * per_thread, a.n_words);
    const int w1 = min(w0 + per_thread, a.n_words);
    int mine = 0;
    for (int w = w0; w < w1; ++w)
        mine += __popc(__hip_atomic_load(&bitmap[w], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    int count;
    int rank = block_scan_int(mine, wave_sums, count);
    for (int w = w0; w < w1; ++w) {
        word_rank[w] = (RANK)rank;
        rank += __popc(__hip_atomic_load(&bitmap[w], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    }
    __syncthreads();

    for (uint32_t s0 = threadIdx.x; s0 < n_seeds; s0 += DEDUP_AHEAD * DEDUP_THREADS) {
        int32_t iter[DEDUP_AHEAD], match_i[DEDUP_AHEAD], match_j[DEDUP_AHEAD];
#pragma unroll
        for (int k = 0; k < DEDUP_AHEAD; ++k) {
            const uint32_t s = min(s0 + k * DEDUP_THREADS, n_seeds - 1);
            iter[k] = a.seed_iter[base + s];
            match_i[k] = a.seed_i[base + s];
            match_j[k] = a.seed_j[base + s];
        }
#pragma unroll
        for (int k = 0; k < DEDUP_AHEAD; ++k) {
            if (s0 + k * DEDUP_THREADS < n_seeds && iter[k] >= 0) {
                const uint32_t i = (uint32_t)match_i[k];
                const uint32_t word = __hip_atomic_load(&bitmap[i >> 5], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const int pos = (int)__hip_atomic_load(&word_rank[i >> 5], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) +
                                __popc(word & ((1u << (i & 31)) - 1u));
                a.pairs[(base + pos) * 2 + 0] = (int32_t)i;
                a.pairs[(base + pos) * 2 + 1] = match_j[k];
            }
        }
    }
    for (uint32_t i = count + threadIdx.x; i < n_seeds; i += DEDUP_THREADS) {
        a.pairs[(base + i) * 2 + 0] = -1;
        a.pairs[(base + i) * 2 + 1] = -1;
    }
    if (threadIdx.x == 0) a.n_pairs[b] = count;
}

// Dynamic LDS the 16-bit-rank variant of the final sort may use on this device (0: none beyond
// the default): what the device grants one workgroup, less the kernel's static LDS and some
// slack, raised once through the kernel's attribute.
static size_t dedup_large_lds_limit() {
    static DeviceCache limit;
    const long long granted = limit.get([](int dev) -> long long {
        int per_block = 0;
        if (hipDeviceGetAttribute(&per_block, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess ||
            per_block <= 64 * 1024)
            return 0;
        const int grant = per_block - 1024;
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(recip_dedup_kernel<true, uint16_t>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, grant) == hipSuccess)
            return grant;
        (void)hipGetLastError();  // not granted: the workspace variant serves these sizes
        return 0;
    });
    return granted > 0 ? (size_t)granted : 0;
}

hipError_t launch_recip_dedup(const RecipState& st, int32_t n_seeds, int batch,
                              const int32_t* seed_i, const int32_t* seed_j, const int32_t* seed_iter,
                              int32_t* pairs, int32_t* n_pairs, hipStream_t s) {
    DedupArgs a;
    a.seed_i = seed_i;
    a.seed_j = seed_j;
    a.seed_iter = seed_iter;
    a.n_seeds = n_seeds;
    a.n_words = (int32_t)st.n_words;
    a.bitmap = st.bitmap;
    a.word_rank = st.word_rank;
    a.pairs = pairs;
    a.n_pairs = n_pairs;
    const size_t tables = (size_t)st.n_words * 2 * sizeof(uint32_t);
    if (tables <= DEDUP_LDS_BYTES)
        return launch(TK_RECIP_DEDUP, recip_dedup_kernel<true, int32_t>, dim3(batch), dim3(DEDUP_THREADS), tables, s, a);
    // larger images: 16-bit ranks, and a workgroup may be granted more than the default 64 KB
    const size_t narrow = (size_t)st.n_words * (sizeof(uint32_t) + sizeof(uint16_t));
    if (n_seeds <= 65535 && narrow <= dedup_large_lds_limit())
        return launch(TK_RECIP_DEDUP, recip_dedup_kernel<true, uint16_t>, dim3(batch), dim3(DEDUP_THREADS), narrow, s, a);
    return launch(TK_RECIP_DEDUP, recip_dedup_kernel<false, int32_t>, dim3(batch), dim3(DEDUP_THREADS), 0, s, a);
}

}  // namespace fnn
