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
// FNN_FLAG_NORMALIZE on aligned fp32 rows (see the header's note on them): one product and fused steps, written out, and the hardware's root.  prep_rows_f32_kernel and
// quantise_kernel, which may read a row twice, must divide alike to the last place: left to the compiler, `sum + x * x` may be fused in one kernel and not in another.
template <int N, int M>
__device__ __forceinline__ void normalize_aligned_row(float (&x)[M]) {
    float sum = __fmul_rn(x[0], x[0]);
#pragma unroll
    for (int k = 1; k < N; ++k) sum = __builtin_fmaf(x[k], x[k], sum);
    divide_row<N>(x, __fsqrt_rn(sum));
}

}  // namespace fnn
