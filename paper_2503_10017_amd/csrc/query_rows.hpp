// Which rows of the query map a search's slots stand for (device code).
#pragma once
#include "fnn_kernels.hpp"

namespace fnn {

__device__ __forceinline__ int64_t query_row(const SearchArgs& a, int64_t qbase, int slot) {
    int64_t row;
    if (a.q_keys) row = (int64_t)(0xFFFFFFFFu - (uint32_t)(a.q_keys[qbase + slot] & 0xFFFFFFFFull));
    else if (a.q_idx) row = a.q_idx[qbase + slot];
    else row = slot;
    return min(max(row, (int64_t)0), (int64_t)a.src_rows - 1);  // never read outside the map
}

// The rows of this lane's query in N consecutive 32-query blocks from slot0 on.  All N index loads
// are in flight together: taken one by one behind the tests above, each waited for the one
// before it and for that block's row, two memory latencies per block before a wave could start (one
// 512x384 pair: first search 37.6 -> 33.4 us, 16 pairs with 1450 queries each 241 -> 228 us, with the
// waits moved out of the candidate loop, see arrived()).  Slots past the live queries repeat the
// last one; their results are dropped.
// LIVE_LIST: q_idx was written by other workgroups of the same launch, so it is read past this compute unit's and this XCD's caches.
template <int N, bool LIVE_LIST = false>
__device__ __forceinline__ void query_rows(const SearchArgs& a, int64_t qbase, int slot0, int n_act, int c, int32_t (&row)[N]) {
    int slot[N];
#pragma unroll
    for (int i = 0; i < N; ++i) slot[i] = min(slot0 + i * 32 + c, n_act - 1);
    if constexpr (LIVE_LIST) {
#pragma unroll
        for (int i = 0; i < N; ++i) row[i] = __hip_atomic_load(a.q_idx + qbase + slot[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else if (a.q_keys) {
        uint32_t low[N];
#pragma unroll
        for (int i = 0; i < N; ++i) low[i] = reinterpret_cast<const uint32_t*>(a.q_keys + qbase + slot[i])[0];
#pragma unroll
        for (int i = 0; i < N; ++i) row[i] = (int32_t)min(0xFFFFFFFFu - low[i], (uint32_t)a.src_rows - 1u);
    } else if (a.q_idx) {
        int32_t idx[N];
#pragma unroll
        for (int i = 0; i < N; ++i) idx[i] = a.q_idx[qbase + slot[i]];
#pragma unroll
        for (int i = 0; i < N; ++i) row[i] = idx[i];
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) row[i] = slot[i];
    }
#pragma unroll
    for (int i = 0; i < N; ++i) row[i] = min(max(row[i], 0), a.src_rows - 1);  // never read outside the map
}

}  // namespace fnn
