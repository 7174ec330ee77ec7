// Device code shared by the 8-bit passes of the searches and of the dense mode.
#pragma once
#include "fnn_device.hpp"
#include "fnn_kernels.hpp"

namespace fnn {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));

constexpr int COARSE_WAVES = 4;  // waves per workgroup
constexpr int COARSE_TURN = 8;   // candidate tiles staged per turn, two per wave
constexpr int TILE_BYTES = 32 * COARSE_ROW_BYTES;
constexpr float UNBOUNDED = 1e18f;  // the "bound" of a row that has none; its square is still a number

#define FNN_LDS_PTR(p) ((void __attribute__((address_space(3)))*)(p))

__device__ __forceinline__ int max3i(int a, int b, int c) { return max(max(a, b), c); }
__device__ __forceinline__ int fold16i(int seed, const i32x16& x) {
    const int t0 = max3i(x[0], x[1], x[2]);
    const int t1 = max3i(x[3], x[4], x[5]);
    const int t2 = max3i(x[6], x[7], x[8]);
    const int t3 = max3i(x[9], x[10], x[11]);
    const int t4 = max3i(x[12], x[13], x[14]);
    return max3i(seed, max3i(t0, t1, t2), max3i(t3, t4, x[15]));
}

__device__ __forceinline__ i32x16 product8(const i32x4& a, const i32x4& b) {
    const i32x16 zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    return __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, zero, 0, 0, 0);
}

// Where groups of candidates share a bound, the bits that say which of DENSE_CELL_PIXELS candidates need a cell lie in words of 64: three for
// 64 groups, the first, second and third candidates of all, five times, and one for the 64 candidates that are alone in theirs (dense_coarse.hip).
__device__ __forceinline__ int mask_candidate(int bit) {
    const int word = bit >> 6, group = (word / 3 << 6) + (bit & 63);  // triples: ten of a tile
    const int tile = word < 15 ? group / 10 : (bit & 63) >> 1, of_tile = group % 10;
    const int h = word < 15 ? of_tile / 5 : bit & 1, v = word < 15 ? 3 * (of_tile % 5) + word % 3 : 15;
    return tile * 32 + tile_row(v, h);
}

}  // namespace fnn
