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
// FNN_FLAG_NORMALIZE on aligned fp32 rows (see the header's note on them): the second square is rounded, the others are fused steps on top of it, and the root is the hardware's.
// prep_rows_f32_kernel and quantise_kernel, which may read a row twice, must divide alike to the last place: left to the compiler, `sum + x * x` may be fused in one kernel and not in
// another.  (That it is the second square is how the compiler fused the sum; results of existing calls are not changed for a last place.)
template <int N, int M>
__device__ __forceinline__ void normalize_aligned_row(float (&x)[M]) {
    float sum = __builtin_fmaf(x[0], x[0], __fmul_rn(x[1], x[1]));
#pragma unroll
    for (int k = 2; k < N; ++k) sum = __builtin_fmaf(x[k], x[k], sum);
    divide_row<N>(x, __fsqrt_rn(sum));
}

}  // namespace fnn
