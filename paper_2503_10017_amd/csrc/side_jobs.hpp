// Device code of the small initialisations that ride along with a launch over the maps (see PrepExtra).
#pragma once
#include "fnn_kernels.hpp"

namespace fnn {

// Spread over all threads of a two-dimensional grid of one-dimensional workgroups.
__device__ __forceinline__ void side_jobs(const PrepExtra& x, int batch) {
    const int64_t tid = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * blockDim.x + threadIdx.x;
    const int64_t n_threads = (int64_t)gridDim.x * gridDim.y * blockDim.x;
    if (x.zero_ptr)
        for (int64_t i = tid; i < x.zero_count; i += n_threads) x.zero_ptr[i] = 0;
    if (x.zero_more)
        for (int64_t i = tid; i < x.zero_more_count; i += n_threads) x.zero_more[i] = 0;
    if (x.seeds) {
        const int64_t total = (int64_t)batch * x.n_seeds;
        for (int64_t i = tid; i < total; i += n_threads) {
            x.cur_u[i] = x.seeds[i];
            x.seed_id[i] = (int32_t)(i % x.n_seeds);
            if (x.seed_iter) x.seed_iter[i] = -1;
        }
        for (int64_t b = tid; b < batch; b += n_threads) x.n_active[b] = x.n_seeds;
    }
}

}  // namespace fnn
