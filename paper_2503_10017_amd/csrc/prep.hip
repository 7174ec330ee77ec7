// Prepare step: copy the caller's descriptor maps into the workspace in the format the
// matrix instructions consume -- the compute format of Algorithm 3 ("HybridCast": inputs
// rounded to 16 bits, round-to-nearest-even) or plain fp32 -- with the channel count zero
// padded to the instruction's K and the pixel count zero padded to whole 32-pixel tiles.
#include "dense_perm.hpp"
#include "fnn_device.hpp"
#include "fnn_kernels.hpp"
#include "row_norm.hpp"
#include "side_jobs.hpp"
#include "trace.hpp"

namespace fnn {

__device__ __forceinline__ float load_as_float(const void* base, int64_t idx, int dtype) {
    if (dtype == FNN_F32) return reinterpret_cast<const float*>(base)[idx];
    const uint16_t raw = reinterpret_cast<const uint16_t*>(base)[idx];
    if (dtype == FNN_F16) {
        return (float)__builtin_bit_cast(_Float16, raw);
    }
    return __uint_as_float((uint32_t)raw << 16);
}

// The same for the raw bits of one 16-bit element.
__device__ __forceinline__ float bits_as_float(uint16_t raw, int dtype) {
    return dtype == FNN_F16 ? (float)__builtin_bit_cast(_Float16, raw) : __uint_as_float((uint32_t)raw << 16);
}

typedef uint32_t words4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint4 pack8(const uint16_t* x) {
    return make_uint4(x[0] | ((uint32_t)x[1] << 16), x[2] | ((uint32_t)x[3] << 16), x[4] | ((uint32_t)x[5] << 16), x[6] | ((uint32_t)x[7] << 16));
}

// x as the compute format holds it (round to nearest even), back in fp32.
__device__ __forceinline__ float round_to_compute(float x, int compute) {
    if (compute == FNN_F16) return (float)(_Float16)x;
    if (compute == FNN_BF16) return __uint_as_float((uint32_t)float_to_bf16_rne(x) << 16);
    return x;
}

// |x|^2 of a row's first N channels: k ascending, every step one fused multiply-add.  Written out, so that
// it does not rest on what the compiler chooses to fuse; a channel that is zero changes nothing.
template <int N, int M>
__device__ __forceinline__ float squared_length(const float (&x)[M]) {
    float sum = 0.0f;
#pragma unroll
    for (int k = 0; k < N; ++k) sum = __builtin_fmaf(x[k], x[k], sum);
    return sum;
}
// The norm term of the L2 score, -1/2 |x|^2, as the norm channels hold it: a rounded value and, in a
// 16-bit format, the rounded remainder.  fp16 ends at 65504: a longer row's term is held at the ends of
// the two halves' ranges instead of as -inf and the +inf that remains, whose sum is not a number.
constexpr float F16_LARGEST = 65504.0f;
__device__ __forceinline__ void split_norm_term(float term, int compute, float& hi, float& lo) {
    const float lowest = compute == FNN_F16 ? -F16_LARGEST : -__builtin_inff();
    hi = round_to_compute(__builtin_fmaxf(term, lowest), compute);
    lo = round_to_compute(__builtin_fmaxf(term - hi, lowest), compute);
}

// The norm of one source descriptor, and -1/2 |x|^2 of one as prepared (divided by `norm` if that is set, then
// rounded to the compute format), read element by element: squared_length() in a rolled loop.
__device__ __forceinline__ float descriptor_norm(const void* src, int64_t first, int d, int dtype) {
    float sum = 0.0f;
    for (int k = 0; k < d; ++k) {
        const float x = load_as_float(src, first + k, dtype);
        sum = __builtin_fmaf(x, x, sum);
    }
    return __builtin_sqrtf(sum);
}
__device__ __forceinline__ float prepared_norm_term(const void* src, int64_t first, int d, int dtype, int compute, float norm) {
    float sum = 0.0f;
    for (int k = 0; k < d; ++k) {
        float x = load_as_float(src, first + k, dtype);
        if (norm > 0.0f) x = __fdiv_rn(x, norm);
        x = round_to_compute(x, compute);
        sum = __builtin_fmaf(x, x, sum);
    }
    return -0.5f * sum;
}

// Any storage format, channel count, row stride and alignment: one thread produces 8 consecutive channels
// of one output row, element by element.  OPTIONS: with NORMALIZE, L2 or SPLIT, where every thread reads
// the whole row for a norm; launch_prep() says which maps take that and which the staged kernel below.
template <bool OPTIONS>
__global__ __launch_bounds__(256) void prep_kernel(PrepArgs a) {
    side_jobs(a.extra, a.batch);
    const int side_idx = blockIdx.y / a.batch;
    const int b = blockIdx.y % a.batch;
    const PrepSide& sd = a.side[side_idx];
    const int groups = a.dp / 8;
    const int64_t total = sd.n_pad * groups;
    const int esize = (a.compute == FNN_F32) ? 4 : 2;
    char* dst = reinterpret_cast<char*>(sd.dst) + (int64_t)b * sd.n_pad * a.dp * esize;
    const void* src = sd.src[b];
    const bool split = OPTIONS && a.split;
    const int data_channels = split ? 3 * a.d : a.d;  // channels that carry data: the descriptor, or three copies of it
    for (int64_t item = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; item < total;
         item += (int64_t)gridDim.x * blockDim.x) {
        const int64_t row = item / groups;                               // stored row
        const int64_t pix = sd.segment_major ? slot_pixel(row) : row;   // pixel it holds
        const int g = (int)(item % groups);
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int k = g * 8 + e;
            const int ch = split ? k % a.d : k;
            v[e] = (pix < sd.n && k < data_channels) ? load_as_float(src, pix * sd.row_stride + ch, sd.dtype) : 0.0f;
        }
        if constexpr (OPTIONS) {
            float norm = 0.0f;
            if (a.normalize && pix < sd.n) {
                norm = descriptor_norm(src, pix * sd.row_stride, a.d, sd.dtype);
                if (norm > 0.0f) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) v[e] = __fdiv_rn(v[e], norm);
                }
            }
            if (split) {  // the copies' layout: see prep_staged_kernel
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int k = g * 8 + e;
                    if (k < data_channels) {
                        const int copy = k / a.d;
                        const float hi = (float)(_Float16)v[e];
                        const float lo = __fsub_rn(v[e], hi);
                        v[e] = (copy == 0 || copy == (sd.second_image ? 2 : 1)) ? hi : lo;
                    }
                }
            }
            // L2 score: channels d.. hold the unit partners and -|x|^2/2 (see FNN_FLAG_L2)
            const int extra = a.compute == FNN_F32 ? 1 : 2;
            if (a.l2 && pix < sd.n && g * 8 + 8 > a.d && g * 8 < a.d + 2 * extra) {
                float hi, lo;
                split_norm_term(prepared_norm_term(src, pix * sd.row_stride, a.d, sd.dtype, a.compute, norm), a.compute, hi, lo);
                const int ones0 = a.d + (sd.second_image ? extra : 0);   // first unit channel
                const int term0 = a.d + (sd.second_image ? 0 : extra);   // first norm channel
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int k = g * 8 + e;
                    if (k >= ones0 && k < ones0 + extra) v[e] = 1.0f;
                    if (k == term0) v[e] = hi;
                    if (extra == 2 && k == term0 + 1) v[e] = lo;
                }
            }
        }
        if (a.compute == FNN_F32) {
            float4* out = reinterpret_cast<float4*>(dst + (row * a.dp + g * 8) * 4);
            out[0] = make_float4(v[0], v[1], v[2], v[3]);
            out[1] = make_float4(v[4], v[5], v[6], v[7]);
        } else {
            uint16_t hbits[8];
#pragma unroll
            for (int e = 0; e < 8; ++e)
                hbits[e] = (a.compute == FNN_F16) ? float_to_f16_rne(v[e]) : float_to_bf16_rne(v[e]);
            uint4 packed;
            packed.x = hbits[0] | ((uint32_t)hbits[1] << 16);
            packed.y = hbits[2] | ((uint32_t)hbits[3] << 16);
            packed.z = hbits[4] | ((uint32_t)hbits[5] << 16);
            packed.w = hbits[6] | ((uint32_t)hbits[7] << 16);
            *reinterpret_cast<uint4*>(dst + (row * a.dp + g * 8) * 2) = packed;
        }
    }
}

// The options that need a whole row at once (FNN_FLAG_NORMALIZE, FNN_FLAG_L2, FNN_FLAG_SPLIT), for any
// storage format, channel count, row stride and alignment.
// A workgroup takes STAGE_ROWS stored rows at a time: it copies the rows' bytes into LDS as they lie in
// memory (16 bytes per lane where the rows are aligned and close together, else one element per
// lane), every thread then makes one output row in registers, and the finished rows leave LDS as
// one contiguous run of 16-byte stores.  What bounds it is the memory traffic.  One 512x384 pair, 24
// channels, every thread reading its part of a row element by element, and the whole row again for a
// norm (with FNN_FLAG_SPLIT one thread per row, lanes 96 bytes in and 160 bytes out apart), against this, microseconds:
// fp16 maps with FNN_FLAG_L2 39.2 / 17.4, with FNN_FLAG_NORMALIZE 36.1 / 14.5, fp32 maps with FNN_FLAG_SPLIT
// 32.9 / 19.2; 17-channel fp32 maps with FNN_FLAG_NORMALIZE 35.3 / 18.4.  Fewer rows: see staging_pays().  Plain
// casts stay with the kernel above (23-channel bf16 14 against 16 us, small maps 4 against 8).
constexpr int STAGE_ROWS = 256;
constexpr int STAGE_MAX_ROW_BYTES = 192;  // widest row held in LDS (48 KB per workgroup)

// Pixel that staged row r of the run of stored rows [row0, row0 + STAGE_ROWS) holds, and the place of that
// pixel's output row in the run.  Segment major: the run is blocks t0..t0+7 of a super-block, staged as
// 32 runs of 8 consecutive pixels.
struct StageRun {
    int64_t first;   // natural order: the first pixel; segment major: the super-block's pixel t0 of lane 0
    bool segments;
    __device__ __forceinline__ StageRun(int64_t row0, bool segment_major) : segments(segment_major) {
        first = segment_major ? slot_pixel(row0) : row0;
    }
    __device__ __forceinline__ int64_t pixel(int r) const { return segments ? first + (int64_t)(r >> 3) * DENSE_S + (r & 7) : first + r; }
    __device__ __forceinline__ int out_row(int r) const { return segments ? (r & 7) * 32 + (r >> 3) : r; }
};
static_assert(STAGE_ROWS == 32 * 8 && DENSE_S % 8 == 0, "a run of stored rows is 8 whole blocks of one super-block");

// IN = ceil(d / 8).
template <int IN, int COMPUTE>
__global__ __launch_bounds__(STAGE_ROWS) void prep_staged_kernel(PrepArgs a) {
    extern __shared__ uint4 stage[];
    side_jobs(a.extra, a.batch);
    const int side_idx = blockIdx.y / a.batch;
    const int b = blockIdx.y % a.batch;
    const PrepSide& sd = a.side[side_idx];
    constexpr int ESIZE = (COMPUTE == FNN_F32) ? 4 : 2;
    constexpr int EXTRA = (COMPUTE == FNN_F32) ? 1 : 2;  // channels per L2 term
    const int tid = threadIdx.x, d = a.d;
    const int es = sd.dtype == FNN_F32 ? 4 : 2;
    const int pitch = sd.vector_rows ? (int)sd.row_stride * es : d * es;  // bytes between staged rows
    const int out_bytes = a.dp * ESIZE;
    const char* src = reinterpret_cast<const char*>(sd.src[b]);
    char* dst = reinterpret_cast<char*>(sd.dst) + (int64_t)b * sd.n_pad * out_bytes;
    char* lds = reinterpret_cast<char*>(stage);
    const int64_t valid = (sd.n - 1) * sd.row_stride * es + (int64_t)d * es;  // bytes of the map (n > 0 here or no row is read)

    for (int64_t row0 = (int64_t)blockIdx.x * STAGE_ROWS; row0 < sd.n_pad; row0 += (int64_t)gridDim.x * STAGE_ROWS) {
        const StageRun run(row0, sd.segment_major != 0);
        if (sd.vector_rows) {
            const int seg_units = (run.segments ? 8 : STAGE_ROWS) * pitch / 16;
            const int units = STAGE_ROWS * pitch / 16;
            auto offset = [&](int u) -> int64_t {
                const int seg = run.segments ? u / seg_units : 0;
                return run.pixel(seg * 8) * pitch + (int64_t)(u - seg * seg_units) * 16;
            };
            for (int u0 = tid; u0 < units; u0 += 4 * STAGE_ROWS) {  // four loads in flight per lane
                words4 x[4];
                bool whole[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int u = u0 + i * STAGE_ROWS;
                    const int64_t off = offset(u);
                    whole[i] = u < units && off + 16 <= valid;
                    x[i] = whole[i] ? *reinterpret_cast<const words4*>(src + off) : (words4)(0u);
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int u = u0 + i * STAGE_ROWS;
                    if (whole[i]) {
                        reinterpret_cast<words4*>(stage)[u] = x[i];
                    } else if (u < units) {  // the end of the map: only whole elements inside it
                        const int64_t off = offset(u);
                        for (int e = 0; e < 16 && off + e + es <= valid; e += es) {
                            if (es == 4) *reinterpret_cast<uint32_t*>(lds + u * 16 + e) = *reinterpret_cast<const uint32_t*>(src + off + e);
                            else *reinterpret_cast<uint16_t*>(lds + u * 16 + e) = *reinterpret_cast<const uint16_t*>(src + off + e);
                        }
                    }
                }
            }
        } else {
            for (int i0 = tid; i0 < STAGE_ROWS * d; i0 += 8 * STAGE_ROWS) {  // eight loads in flight per lane
                uint32_t x[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const int i = i0 + k * STAGE_ROWS, r = i / d, ch = i - r * d;
                    const int64_t pix = run.pixel(min(r, STAGE_ROWS - 1));
                    const int64_t at = min(pix, sd.n - 1) * sd.row_stride + ch;  // rows past the map repeat the last one, see `real`
                    x[k] = es == 4 ? reinterpret_cast<const uint32_t*>(src)[at] : reinterpret_cast<const uint16_t*>(src)[at];
                }
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const int i = i0 + k * STAGE_ROWS;
                    if (i < STAGE_ROWS * d) {
                        if (es == 4) *reinterpret_cast<uint32_t*>(lds + i * 4) = x[k];
                        else *reinterpret_cast<uint16_t*>(lds + i * 2) = (uint16_t)x[k];
                    }
                }
            }
        }
        __syncthreads();

        float v[IN * 8];
        const bool real = run.pixel(tid) < sd.n;  // rows past the map are zero
        const char* row = lds + tid * pitch;
        if (d == IN * 8 && pitch % 16 == 0) {  // uniform
            if (es == 4) {
#pragma unroll
                for (int q = 0; q < IN * 2; ++q) {
                    const float4 x = reinterpret_cast<const float4*>(row)[q];
                    v[4 * q + 0] = x.x;
                    v[4 * q + 1] = x.y;
                    v[4 * q + 2] = x.z;
                    v[4 * q + 3] = x.w;
                }
            } else {
#pragma unroll
                for (int q = 0; q < IN; ++q) {
                    const uint4 x = reinterpret_cast<const uint4*>(row)[q];
                    const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
                    for (int e = 0; e < 8; ++e) v[8 * q + e] = bits_as_float((uint16_t)(w[e / 2] >> (16 * (e & 1))), sd.dtype);
                }
            }
        } else {
#pragma unroll
            for (int k = 0; k < IN * 8; ++k) v[k] = k < d ? load_as_float(row, k, sd.dtype) : 0.0f;
        }
        if (!real) {
#pragma unroll
            for (int k = 0; k < IN * 8; ++k) v[k] = 0.0f;
        }
        __syncthreads();  // the staged rows are in registers: the finished ones may take their place

        // channels at and past d are zero; the builtin is the correctly rounded root
        if (a.normalize) divide_row<IN * 8>(v, __builtin_sqrtf(squared_length<IN * 8>(v)));
        char* out = lds + run.out_row(tid) * out_bytes;
        if (COMPUTE == FNN_F16 && a.split) {
            // copy 0 holds hi, and of copies 1 and 2 image 1 holds (hi, lo), image 2 (lo, hi), so that a row
            // of one times a row of the other sums hi*hi + hi*lo + lo*hi
            const int lo_copy = sd.second_image ? 1 : 2;
            uint16_t hi[IN * 8], lo[IN * 8];
#pragma unroll
            for (int k = 0; k < IN * 8; ++k) {
                const _Float16 x = (_Float16)v[k];
                hi[k] = __builtin_bit_cast(uint16_t, x);
                lo[k] = float_to_f16_rne(__fsub_rn(v[k], (float)x));
            }
            if (d == IN * 8) {  // uniform: a copy is IN whole 16-byte vectors
#pragma unroll
                for (int g = 0; g < IN; ++g) {
                    const uint4 h4 = pack8(hi + 8 * g), l4 = pack8(lo + 8 * g);
                    uint4* o = reinterpret_cast<uint4*>(out) + g;
                    o[0] = h4;
                    o[lo_copy * IN] = l4;
                    o[(3 - lo_copy) * IN] = h4;
                }
                for (int q = 3 * IN; q < a.dp / 8; ++q) reinterpret_cast<uint4*>(out)[q] = make_uint4(0, 0, 0, 0);
            } else {
                uint16_t* o = reinterpret_cast<uint16_t*>(out);
#pragma unroll
                for (int k = 0; k < IN * 8; ++k) {
                    if (k < d) {
                        o[k] = hi[k];
                        o[lo_copy * d + k] = lo[k];
                        o[(3 - lo_copy) * d + k] = hi[k];
                    }
                }
                for (int k = 3 * d; k < a.dp; ++k) o[k] = 0;
            }
        } else {
            // L2 score: channels d.. hold the unit partners and -|x|^2/2 (see FNN_FLAG_L2)
            float hi = 0.0f, lo = 0.0f;
            if (a.l2) {
#pragma unroll
                for (int k = 0; k < IN * 8; ++k) v[k] = round_to_compute(v[k], COMPUTE);
                split_norm_term(-0.5f * squared_length<IN * 8>(v), COMPUTE, hi, lo);
            }
            const bool extras = a.l2 && real;
            const int ones0 = d + (sd.second_image ? EXTRA : 0);   // first unit channel
            const int term0 = d + (sd.second_image ? 0 : EXTRA);   // first norm channel
            auto channel = [&](int k) -> float {  // k is known at compile time, d is uniform
                float x = k < IN * 8 ? v[k < IN * 8 ? k : 0] : 0.0f;
                if (extras) {
                    if (k >= ones0 && k < ones0 + EXTRA) x = 1.0f;
                    if (k == term0) x = hi;
                    if (EXTRA == 2 && k == term0 + 1) x = lo;
                }
                return x;
            };
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (q * 8 < a.dp) {  // uniform
                    if (COMPUTE == FNN_F32) {
                        float4* o = reinterpret_cast<float4*>(out) + 2 * q;
                        o[0] = make_float4(channel(8 * q), channel(8 * q + 1), channel(8 * q + 2), channel(8 * q + 3));
                        o[1] = make_float4(channel(8 * q + 4), channel(8 * q + 5), channel(8 * q + 6), channel(8 * q + 7));
                    } else {
                        uint16_t bits[8];
#pragma unroll
                        for (int e = 0; e < 8; ++e)
                            bits[e] = (COMPUTE == FNN_F16) ? float_to_f16_rne(channel(8 * q + e)) : float_to_bf16_rne(channel(8 * q + e));
                        reinterpret_cast<uint4*>(out)[q] = pack8(bits);
                    }
                }
            }
        }
        __syncthreads();
        const int n_out = (int)min((int64_t)STAGE_ROWS, sd.n_pad - row0);
        uint4* to = reinterpret_cast<uint4*>(dst + row0 * out_bytes);
        for (int u = tid; u < n_out * out_bytes / 16; u += STAGE_ROWS) to[u] = stage[u];
        __syncthreads();  // the next run is staged in the same place
    }
}

// Fast path for the options that need a whole row at once (FNN_FLAG_NORMALIZE, FNN_FLAG_L2) on
// fp32 sources with d a multiple of 8: one thread per row.  The row is read once with 16-byte
// loads; norm and squared length are formed in registers, channels ascending.  Despite their
// names the intrinsics leave both roundings to the compiler: it fuses most products with their additions
// (for 16 channels and more as x[0]^2 + rounded x[1]^2 first), and the root is the hardware's, off
// by one unit in the last place for some rows.  The header allows both for this path; written
// out like squared_length() they would change the last place of about 1 % of the norms.
// IN = d / 8, OUT = dp / 8.
template <int IN, int OUT, int COMPUTE>
__global__ __launch_bounds__(256) void prep_rows_f32_kernel(PrepArgs a) {
    side_jobs(a.extra, a.batch);
    const int side_idx = blockIdx.y / a.batch;
    const int b = blockIdx.y % a.batch;
    const PrepSide& sd = a.side[side_idx];
    constexpr int ESIZE = (COMPUTE == FNN_F32) ? 4 : 2;
    constexpr int D = IN * 8, DP = OUT * 8;
    constexpr int EXTRA = (COMPUTE == FNN_F32) ? 1 : 2;  // channels per L2 term
    char* dst = reinterpret_cast<char*>(sd.dst) + (int64_t)b * sd.n_pad * DP * ESIZE;
    const float* src = reinterpret_cast<const float*>(sd.src[b]);
    for (uint32_t row = blockIdx.x * blockDim.x + threadIdx.x; row < (uint32_t)sd.n_pad; row += gridDim.x * blockDim.x) {
        const int64_t pix = sd.segment_major ? slot_pixel(row) : (int64_t)row;
        float v[DP];
#pragma unroll
        for (int e = 0; e < DP; ++e) v[e] = 0.0f;
        if (pix < sd.n) {
            const float4* p = reinterpret_cast<const float4*>(src + pix * sd.row_stride);
#pragma unroll
            for (int q = 0; q < IN * 2; ++q) {
                const float4 x = p[q];
                v[4 * q + 0] = x.x;
                v[4 * q + 1] = x.y;
                v[4 * q + 2] = x.z;
                v[4 * q + 3] = x.w;
            }
            if (a.normalize) {
                normalize_aligned_row<D>(v);
            }
#pragma unroll
            for (int e = 0; e < D; ++e) v[e] = round_to_compute(v[e], COMPUTE);
            if (a.l2) {
                float sum = 0.0f;
#pragma unroll
                for (int e = 0; e < D; ++e) sum = __fadd_rn(sum, __fmul_rn(v[e], v[e]));
                float hi, lo;
                split_norm_term(-0.5f * sum, COMPUTE, hi, lo);
                const int ones0 = D + (sd.second_image ? EXTRA : 0);
                const int term0 = D + (sd.second_image ? 0 : EXTRA);
#pragma unroll
                for (int e = D; e < D + 2 * EXTRA; ++e) {
                    if (e >= ones0 && e < ones0 + EXTRA) v[e] = 1.0f;
                    if (e == term0) v[e] = hi;
                    if (EXTRA == 2 && e == term0 + 1) v[e] = lo;
                }
            }
        }
        if (COMPUTE == FNN_F32) {
            float4* out = reinterpret_cast<float4*>(dst + (int64_t)row * DP * 4);
#pragma unroll
            for (int q = 0; q < OUT * 2; ++q) out[q] = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
        } else {
            uint4* out = reinterpret_cast<uint4*>(dst + (int64_t)row * DP * 2);
#pragma unroll
            for (int q = 0; q < OUT; ++q) {
                uint32_t w[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    // the values are already representable: the conversion is exact
                    const float lo = v[8 * q + 2 * e], hi = v[8 * q + 2 * e + 1];
                    const uint32_t l16 = (COMPUTE == FNN_F16) ? float_to_f16_rne(lo) : float_to_bf16_rne(lo);
                    const uint32_t h16 = (COMPUTE == FNN_F16) ? float_to_f16_rne(hi) : float_to_bf16_rne(hi);
                    w[e] = l16 | (h16 << 16);
                }
                out[q] = make_uint4(w[0], w[1], w[2], w[3]);
            }
        }
    }
}

template <int IN, int OUT>
static hipError_t launch_prep_rows(const PrepArgs& a, dim3 grid, hipStream_t s) {
    if (a.compute == FNN_F32) return launch(TK_PREP, prep_rows_f32_kernel<IN, OUT, FNN_F32>, grid, dim3(256), 0, s, a);
    if (a.compute == FNN_F16) return launch(TK_PREP, prep_rows_f32_kernel<IN, OUT, FNN_F16>, grid, dim3(256), 0, s, a);
    return launch(TK_PREP, prep_rows_f32_kernel<IN, OUT, FNN_BF16>, grid, dim3(256), 0, s, a);
}

// FNN_FLAG_SPLIT on few aligned fp32 rows of D = 8 * IN channels: one thread per row, straight from memory to memory
// (the copies' layout: see prep_staged_kernel).
template <int IN>
__global__ __launch_bounds__(256) void prep_split_rows_kernel(PrepArgs a) {
    side_jobs(a.extra, a.batch);
    const int side_idx = blockIdx.y / a.batch;
    const int b = blockIdx.y % a.batch;
    const PrepSide& sd = a.side[side_idx];
    constexpr int D = IN * 8, OUT = padded_d(3 * D, FNN_F16) / 8;
    uint4* dst = reinterpret_cast<uint4*>(sd.dst) + (int64_t)b * sd.n_pad * OUT;
    const float* src = reinterpret_cast<const float*>(sd.src[b]);
    const int lo_copy = sd.second_image ? 1 : 2;
    for (uint32_t row = blockIdx.x * blockDim.x + threadIdx.x; row < (uint32_t)sd.n_pad; row += gridDim.x * blockDim.x) {
        const int64_t pix = sd.segment_major ? slot_pixel(row) : (int64_t)row;
        float v[D];
#pragma unroll
        for (int q = 0; q < IN * 2; ++q) {
            const float4 x = pix < sd.n ? reinterpret_cast<const float4*>(src + pix * sd.row_stride)[q] : make_float4(0.f, 0.f, 0.f, 0.f);
            v[4 * q + 0] = x.x;
            v[4 * q + 1] = x.y;
            v[4 * q + 2] = x.z;
            v[4 * q + 3] = x.w;
        }
        if (a.normalize) divide_row<D>(v, __builtin_sqrtf(squared_length<D>(v)));
        uint16_t hi[D], lo[D];
#pragma unroll
        for (int k = 0; k < D; ++k) {
            const _Float16 x = (_Float16)v[k];
            hi[k] = __builtin_bit_cast(uint16_t, x);
            lo[k] = float_to_f16_rne(__fsub_rn(v[k], (float)x));
        }
        uint4* out = dst + (int64_t)row * OUT;
#pragma unroll
        for (int g = 0; g < IN; ++g) {
            const uint4 h4 = pack8(hi + 8 * g);
            out[g] = h4;
            out[lo_copy * IN + g] = pack8(lo + 8 * g);
            out[(3 - lo_copy) * IN + g] = h4;
        }
#pragma unroll
        for (int q = 3 * IN; q < OUT; ++q) out[q] = make_uint4(0, 0, 0, 0);
    }
}

// Fast path: fp32 source whose rows are whole 16-byte vectors and need no channel padding
// (d == dp).  GROUPS = dp / 8 is a compile-time constant so that the row / group split of the
// item index costs a multiply, and every thread moves two 16-byte loads into one (16-bit
// formats) or two (fp32) 16-byte stores.
template <int GROUPS, int COMPUTE>
__global__ __launch_bounds__(256) void prep_f32_kernel(PrepArgs a) {
    side_jobs(a.extra, a.batch);
    const int side_idx = blockIdx.y / a.batch;
    const int b = blockIdx.y % a.batch;
    const PrepSide& sd = a.side[side_idx];
    const uint32_t total = (uint32_t)sd.n_pad * GROUPS;
    constexpr int ESIZE = (COMPUTE == FNN_F32) ? 4 : 2;
    char* dst = reinterpret_cast<char*>(sd.dst) + (int64_t)b * sd.n_pad * (GROUPS * 8) * ESIZE;
    const float* src = reinterpret_cast<const float*>(sd.src[b]);
    for (uint32_t item = blockIdx.x * blockDim.x + threadIdx.x; item < total; item += gridDim.x * blockDim.x) {
        const uint32_t row = item / GROUPS;
        const uint32_t g = item - row * GROUPS;
        const int64_t pix = sd.segment_major ? slot_pixel(row) : (int64_t)row;
        float4 lo = make_float4(0.f, 0.f, 0.f, 0.f), hi = lo;
        if (pix < sd.n) {
            const float4* p = reinterpret_cast<const float4*>(src + pix * sd.row_stride + g * 8);
            lo = p[0];
            hi = p[1];
        }
        if (COMPUTE == FNN_F32) {
            float4* out = reinterpret_cast<float4*>(dst + ((int64_t)item * 8) * 4);
            out[0] = lo;
            out[1] = hi;
        } else {
            const float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
            uint16_t hbits[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) hbits[e] = (COMPUTE == FNN_F16) ? float_to_f16_rne(v[e]) : float_to_bf16_rne(v[e]);
            uint4 packed;
            packed.x = hbits[0] | ((uint32_t)hbits[1] << 16);
            packed.y = hbits[2] | ((uint32_t)hbits[3] << 16);
            packed.z = hbits[4] | ((uint32_t)hbits[5] << 16);
            packed.w = hbits[6] | ((uint32_t)hbits[7] << 16);
            *reinterpret_cast<uint4*>(dst + ((int64_t)item * 8) * 2) = packed;
        }
    }
}

template <int GROUPS>
static hipError_t launch_prep_fast(const PrepArgs& a, dim3 grid, hipStream_t s) {
    if (a.compute == FNN_F32) return launch(TK_PREP, prep_f32_kernel<GROUPS, FNN_F32>, grid, dim3(256), 0, s, a);
    if (a.compute == FNN_F16) return launch(TK_PREP, prep_f32_kernel<GROUPS, FNN_F16>, grid, dim3(256), 0, s, a);
    return launch(TK_PREP, prep_f32_kernel<GROUPS, FNN_BF16>, grid, dim3(256), 0, s, a);
}

// Rows that the staged kernel copies whole, gaps included: 16-byte aligned maps whose rows lie close together.
static bool rows_copied_whole(const PrepArgs& a, const PrepSide& sd) {
    if (sd.row_stride > STAGE_MAX_ROW_BYTES || sd.row_stride * elem_size(sd.dtype) > STAGE_MAX_ROW_BYTES || sd.row_stride > 2 * (int64_t)a.d)
        return false;
    for (int b = 0; b < a.batch; ++b)
        if (((uintptr_t)sd.src[b] % 16) != 0) return false;
    return true;
}

template <int IN>
static hipError_t launch_prep_staged(PrepArgs a, hipStream_t s) {
    int64_t most = 0;
    int row_bytes = a.dp * elem_size(a.compute);
    for (int i = 0; i < a.n_sides; ++i) {
        PrepSide& sd = a.side[i];
        const int64_t stride_bytes = sd.row_stride * elem_size(sd.dtype);
        sd.vector_rows = rows_copied_whole(a, sd);
        const int staged = sd.vector_rows ? (int)stride_bytes : a.d * elem_size(sd.dtype);
        if (staged > row_bytes) row_bytes = staged;
        if (sd.n_pad > most) most = sd.n_pad;
    }
    int64_t blocks = (most + STAGE_ROWS - 1) / STAGE_ROWS;
    if (blocks > 4096) blocks = 4096;
    const dim3 grid((unsigned)blocks, (unsigned)(a.n_sides * a.batch));
    const size_t lds = (size_t)STAGE_ROWS * row_bytes;
    if (a.compute == FNN_F32) return launch(TK_PREP, prep_staged_kernel<IN, FNN_F32>, grid, dim3(STAGE_ROWS), lds, s, a);
    if (a.compute == FNN_F16) return launch(TK_PREP, prep_staged_kernel<IN, FNN_F16>, grid, dim3(STAGE_ROWS), lds, s, a);
    return launch(TK_PREP, prep_staged_kernel<IN, FNN_BF16>, grid, dim3(STAGE_ROWS), lds, s, a);
}

__global__ __launch_bounds__(256) void fill_none_kernel(int32_t* idx, float* score, int64_t count) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x) {
        idx[i] = -1;
        if (score) score[i] = -__builtin_inff();
    }
}

hipError_t launch_fill_i32f32(int32_t* idx, float* score, int64_t count, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    int64_t blocks = (count + 255) / 256;
    if (blocks > 2048) blocks = 2048;
    return launch(TK_FILL, fill_none_kernel, dim3((unsigned)blocks), dim3(256), 0, s, idx, score, count);
}

// The side jobs alone.
__global__ __launch_bounds__(256) void init_kernel(PrepArgs a) { side_jobs(a.extra, a.batch); }

// Whether maps with options go through LDS.  Few rows are all latency, and staging adds three barriers and,
// where rows are not copied whole or are not whole 8-channel groups, a longer chain per thread.  One pair, fp32 maps
// of 24 channels off their alignment, element by element against staged, microseconds: NORMALIZE 6.2 / 9.3 at
// 2 x 3072 rows, 7.7 / 9.6 at 2 x 12288, 16.1 / 11.2 at 2 x 49152; L2 8.9 / 9.6, 9.0 / 9.8, 13.8 / 12.0; SPLIT 5.1 / 9.3,
// 7.3 / 10.0, 20.1 / 14.4.  Up to 8 channels one thread holds a row anyway (fp16 maps of 5, fp32 products: 4.2 / 4.8 at
// 2 x 3072, 10.3 / 12.8 at 2 x 196608; 16-bit products cross near 2 x 65536).  Aligned fp32 maps of 17 channels copied
// whole: NORMALIZE 5.4 / 6.6 at 2 x 3072, 10.0 / 9.1 at 2 x 49152, L2 7.0 / 6.7 and 10.6 / 8.3.
// The copies of a SPLIT row that is not made of whole groups are written to LDS two bytes at a time, lanes a
// row apart: with 64 prepared channels all of them hit one bank (17 channels: 5.0 / 12.0 at 2 x 3072, 43 / 53 at
// 2 x 196608), with others it pays for many rows (12 channels: 5.1 / 6.6, 12.3 / 9.2 at 2 x 49152, 35.3 / 21.3; off their
// alignment 12.2 / 12.3 and 35.5 / 25.6; 31 channels 22.4 / 23.1 and 59.1 / 50.0; off their alignment 22.2 / 28.2 and
// 59.0 / 61.1).
static int64_t rows_prepared(const PrepArgs& a) {
    int64_t rows = 0;
    for (int i = 0; i < a.n_sides; ++i) rows += a.side[i].n_pad * a.batch;
    return rows;
}
static bool staging_pays(const PrepArgs& a) {
    const int64_t rows = rows_prepared(a);
    bool whole = true;
    for (int i = 0; i < a.n_sides; ++i) whole = whole && rows_copied_whole(a, a.side[i]);
    if (a.split && a.d % 8 != 0) {
        if (a.d == 1 || a.dp == 64) return false;
        return a.dp <= 80 ? rows > (whole ? 65536 : 131072) : whole && rows > 131072;
    }
    if (a.d <= 8 && !a.split) return a.compute != FNN_F32 && rows > 131072;
    return rows > 32768 || (whole && (a.d % 8 == 0 || a.l2));
}

hipError_t launch_prep(const PrepArgs& a, hipStream_t s) {
    int64_t most = 0;
    for (int i = 0; i < a.n_sides; ++i) {
        const int64_t items = a.side[i].n_pad * (a.dp / 8);
        if (items > most) most = items;
    }
    if (most == 0) {
        // no map to convert (empty, or all used in place): only the side jobs, if any
        int64_t work = a.extra.zero_ptr ? a.extra.zero_count : 0;
        if (a.extra.seeds && (int64_t)a.batch * a.extra.n_seeds > work) work = (int64_t)a.batch * a.extra.n_seeds;
        if (work <= 0) return hipSuccess;
        int64_t init_blocks = (work + 255) / 256;
        if (init_blocks > 1024) init_blocks = 1024;
        return launch(TK_PREP, init_kernel, dim3((unsigned)init_blocks, 1), dim3(256), 0, s, a);
    }
    int64_t blocks = (most + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    dim3 grid((unsigned)blocks, (unsigned)(a.n_sides * a.batch));
    bool vector_rows = most < (int64_t)1 << 31;  // fp32 sources whose rows are whole, aligned 16-byte vectors
    for (int i = 0; i < a.n_sides && vector_rows; ++i) {
        const PrepSide& sd = a.side[i];
        vector_rows = sd.dtype == FNN_F32 && sd.row_stride % 4 == 0;
        for (int b = 0; b < a.batch && vector_rows; ++b) vector_rows = ((uintptr_t)sd.src[b] % 16) == 0;
    }
    if (vector_rows && !a.split && (a.normalize || a.l2) && a.d % 8 == 0) {
        const int in = a.d / 8, out = a.dp / 8;
        if (in == 1 && out == 1) return launch_prep_rows<1, 1>(a, grid, s);
        if (in == 1 && out == 2) return launch_prep_rows<1, 2>(a, grid, s);
        if (in == 2 && out == 2) return launch_prep_rows<2, 2>(a, grid, s);
        if (in == 2 && out == 3) return launch_prep_rows<2, 3>(a, grid, s);
        if (in == 3 && out == 3) return launch_prep_rows<3, 3>(a, grid, s);
        if (in == 3 && out == 4) return launch_prep_rows<3, 4>(a, grid, s);
        if (in == 4 && out == 4) return launch_prep_rows<4, 4>(a, grid, s);
    }
    // one pair of fp32 maps of 24 channels, a thread per row against staged: 4.2 / 5.3 us at 2 x 3072 rows, 6.2 / 6.0 at
    // 2 x 12288 (four pairs of 3072: 5.1 / 6.0), 12.1 / 10.4 at 2 x 49152
    if (vector_rows && a.split && a.d % 8 == 0 && rows_prepared(a) <= 24576) {
        switch (a.d / 8) {
            case 1: return launch(TK_PREP, prep_split_rows_kernel<1>, grid, dim3(256), 0, s, a);
            case 2: return launch(TK_PREP, prep_split_rows_kernel<2>, grid, dim3(256), 0, s, a);
            case 3: return launch(TK_PREP, prep_split_rows_kernel<3>, grid, dim3(256), 0, s, a);
            case 4: return launch(TK_PREP, prep_split_rows_kernel<4>, grid, dim3(256), 0, s, a);
        }
    }
    const bool fast = vector_rows && a.d == a.dp && !a.l2 && !a.normalize && !a.split;
    if (fast) {
        switch (a.dp / 8) {
            case 1: return launch_prep_fast<1>(a, grid, s);
            case 2: return launch_prep_fast<2>(a, grid, s);
            case 3: return launch_prep_fast<3>(a, grid, s);
            case 4: return launch_prep_fast<4>(a, grid, s);
        }
    }
    if (!a.normalize && !a.l2 && !a.split) return launch(TK_PREP, prep_kernel<false>, grid, dim3(256), 0, s, a);
    if (!staging_pays(a)) return launch(TK_PREP, prep_kernel<true>, grid, dim3(256), 0, s, a);
    switch ((a.d + 7) / 8) {
        case 1: return launch_prep_staged<1>(a, s);
        case 2: return launch_prep_staged<2>(a, s);
        case 3: return launch_prep_staged<3>(a, s);
        case 4: return launch_prep_staged<4>(a, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace fnn
