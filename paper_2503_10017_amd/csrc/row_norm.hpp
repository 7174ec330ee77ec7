// How rows are divided by their norm (device code).
#pragma once
#include <hip/hip_runtime.h>

namespace fnn {

// A row's first N channels divided by `norm` (FNN_FLAG_NORMALIZE); an all-zero row stays zero.
template <int N, int M>
__device__ __forceinline__ void divide_row(float (&x)[M], float norm) {
    if (norm > 0.0f) {
#pragma unroll
        for (int k = 0; k < N; ++k) x[k] = __fdiv_rn(x[k], norm);
    }
}
// FNN_FLAG_NORMALIZE on aligned fp32 rows (see the header's note on them): the fusing is the compiler's, the root the hardware's.  prep_rows_f32_kernel and
// quantise_kernel divide alike, whichever of them prepares a call's maps.
template <int N, int M>
__device__ __forceinline__ void normalize_aligned_row(float (&x)[M]) {
    float sum = 0.0f;
#pragma unroll
    for (int k = 0; k < N; ++k) sum = __fadd_rn(sum, __fmul_rn(x[k], x[k]));
    divide_row<N>(x, __fsqrt_rn(sum));
}

}  // namespace fnn
