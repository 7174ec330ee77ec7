// Pass 1 of a large search in two steps whose keys are, bit for bit, those of search_kernel.
//
// Step 1 (coarse_kernel) scores every query against every candidate in 8-bit integers: one K=32 instruction per
// 32x32 block, at the rate of a K=16 fp16 one, and eight 3-input maxima, with nothing tracked per
// tile (22.6 ns per block and SIMD in a bare loop; search_kernel's arithmetic for 24 channels 42-47 ns).  It keeps one
// number per query and CELL of 512 or 1024 candidates, an upper bound of the cell's scores, and one per query, a
// lower bound of its best score.  Step 2 (refine_kernel) multiplies each cell again, in the format the call asked
// for and with the same instructions as search_kernel, but only for the queries whose upper bound there reaches
// their lower bound; every other cell holds no candidate that could win or tie.  Of the 192 segments of a 512x384 map
// a query needs 1 on average where it has a clear partner, 4 of maps that have nothing in common, and the more the less the descriptors
// tell apart: 7 to 25 with features of 32 to 128 pixels, 50 with descriptors of rank 6 in 24 channels, 140 with rank 4 (24 channels, unit rows).
//
// The bounds.  With a row a = s q + r, q its 8-bit row, s its segment's scale, r the remainder, a product is
//     a.b = s_a s_b (q_a.q_b) + (s_a q_a).r_b + r_a.b,     |second| + |third| <= |a| |r_b| + |r_a| (|b| + |r_b|),
// the integer sum is exact, and |a|, |r_a| are taken from the row, |r_b| and |b| from the segment's worst row.
// What the matrix instructions round when they sum up to 96 products in fp32, and what is rounded here, is
// below 4e-5 |a| |b| (ROUNDING, counted on both sides).  Rows whose squares leave fp32's range, or that are not finite, take
// no part in the 8-bit scores: their bounds are so wide that they are always refined.
#include <type_traits>

#include "coarse_device.hpp"
#include "fnn_device.hpp"
#include "fnn_kernels.hpp"
#include "query_rows.hpp"
#include "row_norm.hpp"
#include "side_jobs.hpp"
#include "trace.hpp"

namespace fnn {

// ---- the 8-bit maps ------------------------------------------------------------------------------
constexpr float ROUNDING = 2e-5f;          // of a row's length, on top of its remainder
constexpr float LEAST_SQUARE = 1e-30f;     // |x|^2 of a row that the bounds hold for
constexpr float LARGEST_SQUARE = 1e30f;
// fp16 values below 2^-14 may count as 0 in the matrix instructions.  Where a step of the scale is wider than twice
// that they are 0 in the 8-bit row too; elsewhere their length (at most sqrt(96) * 2^-14) joins the remainder.
constexpr float F16_SMALL = 6.2e-5f;
constexpr float F16_SMALL_LENGTH = 6.1e-4f;

__device__ __forceinline__ uint32_t bf16_up(float x) { return (__float_as_uint(x) + 0xFFFFu) >> 16; }  // x >= 0

// The channels of a prepared row as fp32 numbers.  SPLIT: the high halves of a two-term row's descriptor, which stand in for
// it: what the low halves add, at most 2^-11 of it, joins the remainder (LOW_HALVES), and so does the product of two
// low halves that the score leaves out.
constexpr float LOW_HALVES = 5.2e-4f;
template <int CT, int DP, bool SPLIT>
struct PreparedRow {
    static constexpr int CHANNELS = SPLIT ? FNN_MAX_D : DP;
    static __device__ __forceinline__ void load(const char* row, int d, float (&x)[CHANNELS]) {
        if constexpr (SPLIT) {
#pragma unroll
            for (int g = 0; g < CHANNELS / 8; ++g) {
                f16x8 hi = {0, 0, 0, 0, 0, 0, 0, 0};
                if (8 * g < d) hi = *reinterpret_cast<const f16x8*>(row + 16 * g);  // uniform; rows hold 3 d channels
#pragma unroll
                for (int e = 0; e < 8; ++e) x[8 * g + e] = 8 * g + e < d ? (float)hi[e] : 0.0f;
            }
        } else if constexpr (CT == CT_F32) {
#pragma unroll
            for (int q = 0; q < DP / 4; ++q) {
                const float4 v = reinterpret_cast<const float4*>(row)[q];
                x[4 * q] = v.x;
                x[4 * q + 1] = v.y;
                x[4 * q + 2] = v.z;
                x[4 * q + 3] = v.w;
            }
        } else {
#pragma unroll
            for (int q = 0; q < DP / 8; ++q) {
                const uint4 v = reinterpret_cast<const uint4*>(row)[q];
                const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const uint32_t bits = (w[e / 2] >> (16 * (e & 1))) & 0xFFFFu;
                    x[8 * q + e] = CT == CT_F16 ? (float)__builtin_bit_cast(_Float16, (uint16_t)bits) : __uint_as_float(bits << 16);
                }
            }
        }
    }
};

// The largest of a value over a workgroup (every thread gets it); `word` is LDS that nothing else uses.
__device__ __forceinline__ float workgroup_max(float x, float* word) {  // x >= 0: its bits order like the value
    x = half_max(x);
    x = __builtin_fmaxf(x, __shfl_xor(x, 32));
    if ((threadIdx.x & 63) == 0) atomicMax(reinterpret_cast<uint32_t*>(word), __float_as_uint(x));
    __syncthreads();
    return *word;
}

// One workgroup turns one segment of prepared rows into 8-bit rows, a thread ROWS of them.  Between the segment's largest value
// and the rounding the rows stay in registers, or, where they are too many (RELOAD), are read a second time.
// RAW: the rows are the caller's fp32 rows of 24 channels; they are divided by their norm, if the call says so, and rounded to the compute format here, and the
// prepared map is written too (four raw pairs of 517x389 and 433x301 pixels, normalised: a prepare launch and this one 65.7 us, this one alone 50.1).  Two-term rows, 160 bytes each, go through LDS so that a wave writes 16 bytes of a row beside the next 16 (four pairs of
// 512x384, the whole call: a prepare launch and a second reading of the caller's rows 627 us, every thread writing its own row 618, so 585).  Bound by memory.
enum QuantiseRows { ROWS_PREPARED, ROWS_RAW, ROWS_RAW_NORMALIZED };
template <int CT, int DP, bool SPLIT, QuantiseRows FROM, int THREADS, int ROWS, bool RELOAD>
__global__ __launch_bounds__(THREADS) void quantise_kernel(QuantiseArgs a) {
    using Row = PreparedRow<CT, DP, SPLIT>;
    constexpr int K = Row::CHANNELS, SEGMENT = THREADS * ROWS, KEPT = RELOAD ? 1 : ROWS;
    constexpr bool RAW = FROM != ROWS_PREPARED;
    __shared__ float top[4];  // largest value, remainder, length, and whether a row has no bound
    constexpr int SPLIT_QUADS = DP / 8;  // a prepared two-term row, in 16-byte pieces
    __shared__ uint4 rows_out[RAW && SPLIT ? THREADS / 64 : 1][RAW && SPLIT ? 32 * SPLIT_QUADS : 1];  // 32 of them per wave, so that they are written side by side
    side_jobs(a.extra, a.batch);
    {
        const int64_t tid = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * THREADS + threadIdx.x;
        const int64_t n_threads = (int64_t)gridDim.x * gridDim.y * THREADS;
        for (int64_t i = tid; i < a.lower_count; i += n_threads) a.lower[i] = 0;
    }
    const QuantiseSide& sd = a.side[blockIdx.y / a.batch];
    const int b = blockIdx.y % a.batch, seg = blockIdx.x;
    if (seg >= sd.out.n_segs) return;  // uniform: the two maps may differ in size
    if (threadIdx.x < 4) top[threadIdx.x] = 0.0f;
    __syncthreads();

    const char* prepared = sd.prepared + (int64_t)b * sd.bstride;
    float x[KEPT][K], square[KEPT];
    bool bounded[KEPT];
    // row i of this thread into x[at]: its values, their squares' sum, and whether the bounds hold for it; returns its largest value
    auto read = [&](int i, int at, bool write) -> float {
        const int64_t pixel = (int64_t)seg * SEGMENT + i * THREADS + threadIdx.x;
        int64_t row = min(pixel, sd.n - 1);  // rows past the map repeat its last one, whose scores are real
        if (sd.gather) row = min(max((int64_t)sd.gather[(int64_t)b * sd.n + row], (int64_t)0), sd.gather_rows - 1);
        if constexpr (RAW) {
            using O = Ops<CT, 24>;
            const float4* p = reinterpret_cast<const float4*>(sd.raw[b] + row * sd.raw_stride);
            uint32_t w[12];
            if constexpr (FROM == ROWS_RAW_NORMALIZED) {
                float r[24];
#pragma unroll
                for (int q = 0; q < 6; ++q) {
                    const float4 v = p[q];
                    r[4 * q] = v.x;
                    r[4 * q + 1] = v.y;
                    r[4 * q + 2] = v.z;
                    r[4 * q + 3] = v.w;
                }
                normalize_aligned_row<24>(r);
#pragma unroll
                for (int q = 0; q < 12; ++q) w[q] = round_pair<CT>(r[2 * q], r[2 * q + 1]);
            } else {
#pragma unroll
                for (int q = 0; q < 6; ++q) {
                    const float4 v = p[q];
                    w[2 * q] = round_pair<CT>(v.x, v.y);
                    w[2 * q + 1] = round_pair<CT>(v.z, v.w);
                }
            }
            if (SPLIT && write) {  // [hi, hi, lo] in image 1, [hi, lo, hi] in image 2, as the prepare pass writes them
                uint32_t low[12];
#pragma unroll
                for (int q = 0; q < 6; ++q) {
                    const float4 v = p[q];
                    low[2 * q] = round_pair<CT>(__fsub_rn(v.x, (float)(_Float16)v.x), __fsub_rn(v.y, (float)(_Float16)v.y));
                    low[2 * q + 1] = round_pair<CT>(__fsub_rn(v.z, (float)(_Float16)v.z), __fsub_rn(v.w, (float)(_Float16)v.w));
                }
                const bool real = pixel < sd.n, second = blockIdx.y >= (unsigned)a.batch;
                const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
                const int64_t first = pixel - lane;  // the wave's 64 rows lie side by side
                uint4* out = reinterpret_cast<uint4*>(const_cast<char*>(prepared));
#pragma unroll
                for (int part = 0; part < 2; ++part) {  // 32 rows at a time
                    if (lane >> 5 == part) {
#pragma unroll
                        for (int q = 0; q < SPLIT_QUADS; ++q) {
                            uint32_t o[4];
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const int at = 4 * q + e, copy = at / 12, k = at % 12;
                                o[e] = copy == 0 ? w[k] : (copy == 1 ? (second ? low[k] : w[k]) : (copy == 2 ? (second ? w[k] : low[k]) : 0));
                                if (!real) o[e] = 0;
                            }
                            rows_out[wave][(lane & 31) * SPLIT_QUADS + q] = make_uint4(o[0], o[1], o[2], o[3]);
                        }
                    }
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // only the wave itself reads them, in the order of its instructions
                    __builtin_amdgcn_wave_barrier();
#pragma unroll
                    for (int k = 0; k < SPLIT_QUADS / 2; ++k) {
                        const int at = k * 64 + lane;
                        if (first + 32 * part + at / SPLIT_QUADS < sd.n_pad) out[(first + 32 * part) * SPLIT_QUADS + at] = rows_out[wave][at];
                    }
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                }
            }
            if (!SPLIT && write && pixel < sd.n_pad) {
                uint4* out = reinterpret_cast<uint4*>(const_cast<char*>(prepared) + pixel * O::ROW_BYTES);
                const bool real = pixel < sd.n;  // padding rows of the prepared map are zero
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    out[q] = real ? make_uint4(w[4 * q], w[4 * q + 1], w[4 * q + 2], w[4 * q + 3]) : make_uint4(0, 0, 0, 0);
            }
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const uint32_t bits = k < 24 ? (w[k < 24 ? k / 2 : 0] >> (16 * (k & 1))) & 0xFFFFu : 0;
                x[at][k] = CT == CT_F16 ? (float)__builtin_bit_cast(_Float16, (uint16_t)bits) : __uint_as_float(bits << 16);
            }
        } else {
            constexpr int ROW_BYTES = DP * (CT == CT_F32 ? 4 : 2);
            Row::load(prepared + row * ROW_BYTES, a.split_d, x[at]);
        }
        float most = 0.0f, sum = 0.0f;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            most = __builtin_fmaxf(most, __builtin_fabsf(x[at][k]));
            sum = __builtin_fmaf(x[at][k], x[at][k], sum);
        }
        square[at] = sum;
        // compared as integers, which puts a sum that is not a number past the largest
        const uint32_t bits = __float_as_uint(sum) & 0x7FFFFFFFu;
        bounded[at] = (bits == 0 && __float_as_uint(most) == 0) ||
                      (bits >= __float_as_uint(LEAST_SQUARE) && bits <= __float_as_uint(LARGEST_SQUARE));
        return bounded[at] ? most : 0.0f;
    };
    float largest = 0.0f;
    if constexpr (RELOAD) {
#pragma unroll 1
        for (int i = 0; i < ROWS; ++i) largest = __builtin_fmaxf(largest, read(i, 0, true));
    } else {
#pragma unroll
        for (int i = 0; i < ROWS; ++i) largest = __builtin_fmaxf(largest, read(i, i, true));
    }
    largest = workgroup_max(largest, &top[0]);
    const float scale = largest * (1.0f / 127.0f);
    const float inverse = largest > 0.0f ? 127.0f / largest : 0.0f;
    const float small = CT == CT_F16 && scale < 2.0f * F16_SMALL ? F16_SMALL_LENGTH : 0.0f;

    float residual = 0.0f, length = 0.0f, unbounded = 0.0f;
    const int64_t first = ((int64_t)b * sd.out.n_segs + seg) * SEGMENT;
    auto write = [&](int i, int at) {
        const int64_t out_row = first + i * THREADS + threadIdx.x;
        // x / scale is rounded to the nearest integer by adding 1.5 * 2^23, which leaves it in the low bits; an unbounded row's
        // integers mean nothing
        constexpr float INTEGER = 12582912.0f;
        uint32_t words[COARSE_ROW_BYTES / 4];
        float left = 0.0f;
#pragma unroll
        for (int w = 0; w < COARSE_ROW_BYTES / 4; ++w) {
            uint32_t q[4] = {0, 0, 0, 0};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int k = 4 * w + e;
                if (k < K) {
                    const float v = x[at][k < K ? k : 0];
                    const float t = __builtin_fmaf(v, inverse, INTEGER);
                    const float r = __builtin_fmaf(-scale, t - INTEGER, v);
                    left = __builtin_fmaf(r, r, left);
                    q[e] = __float_as_uint(t);
                }
            }
            const uint32_t low = __builtin_amdgcn_perm(q[1], q[0], 0x0C0C0400u);  // bytes (0 0 q1 q0)
            words[w] = __builtin_amdgcn_perm(q[3], __builtin_amdgcn_perm(q[2], low, 0x0C040100u), 0x04020100u);
        }
        constexpr float LOW = SPLIT ? LOW_HALVES : 0.0f;
        const float len = __builtin_sqrtf(square[at]) * (1.0f + 1e-5f + LOW);
        const float rest = __builtin_sqrtf(left) * (1.0f + 1e-5f) + (ROUNDING + LOW) * len + small;
        uint32_t bound = bf16_up(UNBOUNDED) | (bf16_up(UNBOUNDED) << 16);
        if (bounded[at]) {
            residual = __builtin_fmaxf(residual, rest);
            length = __builtin_fmaxf(length, len);
            const float per_scale = scale > 0.0f ? 1.0f / scale : 0.0f;  // a segment of zero rows: every score is 0
            bound = bf16_up(rest * per_scale * (1.0f + 1e-6f)) | (bf16_up(len * per_scale * (1.0f + 1e-6f)) << 16);
        } else {
            unbounded = 1.0f;
        }
        uint4* out = reinterpret_cast<uint4*>(sd.out.rows + out_row * COARSE_ROW_BYTES);
        out[0] = make_uint4(words[0], words[1], words[2], words[3]);
        out[1] = make_uint4(words[4], words[5], words[6], words[7]);
        sd.out.row_bound[out_row] = bound;
    };
    if constexpr (RELOAD) {
#pragma unroll 1
        for (int i = 0; i < ROWS; ++i) {
            (void)read(i, 0, false);
            write(i, 0);
        }
    } else {
#pragma unroll
        for (int i = 0; i < ROWS; ++i) write(i, i);
    }
    residual = workgroup_max(residual, &top[1]);
    length = workgroup_max(length, &top[2]);
    unbounded = workgroup_max(unbounded, &top[3]);
    if (threadIdx.x == 0) {
        SegInfo info = {scale, residual, length + residual, 0.0f};
        if (unbounded > 0.0f) info = {scale, UNBOUNDED, UNBOUNDED, 0.0f};
        sd.out.seg[(int64_t)b * sd.out.n_segs + seg] = info;
    }
}

// Queries that are not listed are the rows of their map in order: those from slot `first` on are the rows of the map from
// row `first` on.  Returns how far to move the map's start.
__device__ __forceinline__ int64_t take_slots_from(SearchArgs& a, int first) {
    if (a.q_idx || a.q_keys) return 0;
    a.src_rows -= first;
    return first;
}

// Whether a search's findings say that 8-bit scores do not pay.
__device__ __forceinline__ bool gives_up(const SearchVote& v, float even) { return v.given_up || (float)v.again * (1.0f + even) > (float)v.of * even; }

// ---- step 1 ------------------------------------------------------------------------------------
// A pair whose bounds rule too little out (see dense_coarse.hip) is given up.  Long searches (VOTE) find out on the way: behind the first cell of a chunk the
// waves share the lower bounds of 64 queries each, behind the second some of them count the queries that the cell leaves in doubt against what all
// workgroups know by then, and behind the third and fourth they look whether the votes were too many.  Short ones would lose 10 % to that;
// there step 2 counts the cells that it had to take.  Step 2 then takes every cell for every query, and the later searches of the call begin
// there.  Every result comes out of the same products either way.  Microseconds in one step /
// in two without this / with it, fp16, 24 channels, 512x384: 16 pairs of 3072 seeds, rank 4 1663 / 2651 / 2059, one descriptor throughout 1466 / 2641 /
// 1872, features of 4 pixels 1615 / 1474 / 1420; the seeds' one search, rank 4 461 / 802 / 723, features of 4 pixels 468 / 445 / 433; every
// pixel of one pair, rank 4 1654 / 2670 / 1973.
// (Those were taken before products and maxima came in turn.  In one step / with votes since, image 2 a permutation of image 1: 16 pairs of 3072 seeds, rank 4 1113 / 1411, one
// descriptor throughout 1433 / 1802, full rank 992 / 817; the seeds' one search 493 / 683, 382 / 564 and 494 / 407; every pixel of one pair 1671 / 1946, 1280 / 1528 and 1653 / 995.)
constexpr int VOTE_CELLS = 4;  // shortest chunk that is worth it
constexpr int VOTERS = 64;     // of a pair, about; a quarter of them may decide

// fn(std::integral_constant<int, n>) for the n in 0..MOST that is `count` (uniform).
template <int MOST, typename F>
__device__ __forceinline__ bool with_count(int count, const F& fn) {
    if constexpr (MOST > 0) {
        if (count < MOST) return with_count<MOST - 1>(count, fn);
    }
    return fn(std::integral_constant<int, MOST>{});
}

// The four waves of a workgroup hold PAIRS pairs of query blocks each and sweep the same tiles, which reach LDS by direct loads
// (a tile is 1 KB: one 16-byte load per lane), the next turn's while this turn's are multiplied.
// Bound by the vector maxima and the matrix instructions, which take about the same time each, at the clock that the power limit leaves.
// A product is followed by the maxima of the one before it: two products and then their sixteen maxima leave either unit
// waiting for the other (a bare loop of such pairs 25.7 ns per block and SIMD, of this order 22.6, with operands of zeros, at the full clock, 22.5 and
// 17.8; every pixel of one 512x384 pair 1130 -> 1035 us, 16 pairs of 3072 queries 372 -> 347).  Tests for the blocks that hold a query would
// keep the compiler from that order, so a wave takes the loop made for its number of them.
template <int PAIRS, int CELL_TILES, bool VOTE>
__global__ __launch_bounds__(COARSE_WAVES * 64) __attribute__((amdgpu_waves_per_eu(2)))
void coarse_kernel(SearchArgs a, CoarseArgs ca) {
    constexpr int TURNS = CELL_TILES / COARSE_TURN, CELLS = SEG_TILES / CELL_TILES;
    static_assert(TURNS % 2 == 0, "a cell is an even number of turns, so it starts on stage slot 0");
    __shared__ uint4 stage0[COARSE_TURN][64], stage1[COARSE_TURN][64];  // two variables, see dense_staged_kernel
    __shared__ uint32_t leave;
    const int lane = threadIdx.x & 63, c = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // one XCD owns a contiguous run of (pair, unit) work, see search_kernel
    const int n_wgs = gridDim.x * gridDim.y;
    int wg = blockIdx.y * gridDim.x + blockIdx.x;
    if ((n_wgs & 7) == 0) wg = (wg & 7) * (n_wgs >> 3) + (wg >> 3);
    const int b = wg / gridDim.x;
    const int wgi = wg % gridDim.x;
    int n_act = a.nq;
    if (a.nq_active) n_act = min(max(a.nq_active[b], 0), a.nq);
    if (n_act < ca.min_live) return;
    if (ca.earlier && gives_up(ca.earlier[b], ca.even)) {
        if (ca.vote && wgi == 0 && threadIdx.x == 0) ca.vote[b].given_up = 1;  // for the searches that follow
        return;
    }
    if (VOTE && ca.first_slot > 0 && ca.vote[b].given_up) return;  // an earlier launch of this search found out
    n_act = min(n_act - ca.first_slot, ca.slab);  // slots are counted from first_slot on
    if (n_act <= 0) return;

    // pairs of query blocks are dealt evenly to the waves of all quads; those with one more sit at
    // different places of their workgroups, that is on different SIMDs
    const int n_cells = ca.tgt.n_segs * CELLS;
    const int pairs = (n_act + 63) / 64;
    const int quads = (pairs + PAIRS * COARSE_WAVES - 1) / (PAIRS * COARSE_WAVES);
    const int chunks = min(max(1, (int)gridDim.x / quads), n_cells);
    const int per_wave = pairs / (quads * COARSE_WAVES), more = pairs % (quads * COARSE_WAVES);

    if (ca.src_listed) {
        a.q_idx = nullptr;
        a.src_rows = a.nq;
    }
    const int64_t shift = take_slots_from(a, ca.first_slot);
    const char* src = ca.src.rows + ((int64_t)b * ca.src.n_segs * SEG_PIXELS + shift) * COARSE_ROW_BYTES;
    const uint32_t* src_bound = ca.src.row_bound + (int64_t)b * ca.src.n_segs * SEG_PIXELS + shift;
    const char* tgt = ca.tgt.rows + (int64_t)b * ca.tgt.n_segs * SEG_PIXELS * COARSE_ROW_BYTES;
    const SegInfo* info = ca.tgt.seg + (int64_t)b * ca.tgt.n_segs;
    const int64_t qbase = (int64_t)b * a.nq + ca.first_slot;

    const int units = quads * chunks;
    for (int unit = wgi; unit < units; unit += gridDim.x) {  // uniform in the workgroup
        const int chunk = unit / quads, quad = unit % quads;
        const int rank = ((wave + quad) & (COARSE_WAVES - 1)) * quads + quad;
        const int slot0 = (rank * per_wave + min(rank, more)) * 64;
        const int slot_end = min(n_act, slot0 + (per_wave + (rank < more ? 1 : 0)) * 64);
        const int cell0 = (int)((int64_t)chunk * n_cells / chunks), cell1 = (int)((int64_t)(chunk + 1) * n_cells / chunks);
        const char* first = tgt + (int64_t)cell0 * CELL_TILES * TILE_BYTES;
        const int total = (cell1 - cell0) * TURNS;

        auto stage_turn = [&](uint4 (&slot)[COARSE_TURN][64], int k) {
            const char* from = first + (int64_t)min(k, total - 1) * (COARSE_TURN * TILE_BYTES) + c * COARSE_ROW_BYTES + h * 16;
#pragma unroll
            for (int i = 0; i < 2; ++i)
                __builtin_amdgcn_global_load_lds((const void*)(from + (2 * wave + i) * TILE_BYTES), FNN_LDS_PTR(&slot[2 * wave + i][0]), 16, 0, 0);
        };
        stage_turn(stage0, 0);

        i32x4 q[PAIRS][2];
        int best[PAIRS][2];
        float low[PAIRS];        // lane l of pair p: the slot slot0 + 64 p + l
        uint32_t bound[PAIRS];
        {
            int32_t row[2 * PAIRS];
            query_rows<2 * PAIRS>(a, qbase, slot0, n_act, c, row);
#pragma unroll
            for (int p = 0; p < PAIRS; ++p) {
                const int32_t even = row[2 * p], odd = row[2 * p + 1];
                q[p][0] = *reinterpret_cast<const i32x4*>(src + (int64_t)even * COARSE_ROW_BYTES + 16 * h);
                q[p][1] = *reinterpret_cast<const i32x4*>(src + (int64_t)odd * COARSE_ROW_BYTES + 16 * h);
                bound[p] = src_bound[h ? odd : even];
            }
        }
#pragma unroll
        for (int p = 0; p < PAIRS; ++p) {
            arrived(q[p][0]);
            arrived(q[p][1]);
            arrived(bound[p]);
            best[p][0] = best[p][1] = -0x7FFFFFFF;
            low[p] = -__builtin_inff();
        }

        // The cells of the chunk, for a wave whose first LIVE pairs hold a query; true if the pair of images is given up.
        auto sweep = [&](auto live_tag) -> bool {
            constexpr int LIVE = decltype(live_tag)::value, BLOCKS = 2 * LIVE;
            auto turn = [&](int k, auto slot_tag) {
                constexpr int SLOT = decltype(slot_tag)::value;
                __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wave's share of the turn is in LDS
                __syncthreads();                     // everyone's is, and everyone has left the other slot
                stage_turn(SLOT ? stage0 : stage1, k + 1);
                if constexpr (LIVE > 0) {
                    auto tile = [&](int j) { return __builtin_bit_cast(i32x4, SLOT ? stage1[j][lane] : stage0[j][lane]); };
                    i32x4 cur = tile(0);
                    i32x16 score[2];
                    score[0] = product8(cur, q[0][0]);
#pragma unroll
                    for (int j = 0; j < COARSE_TURN; ++j) {
                        const i32x4 next = tile(j + 1 < COARSE_TURN ? j + 1 : j);
#pragma unroll
                        for (int i = 0; i < BLOCKS; ++i) {
                            const int then = i + 1 < BLOCKS ? i + 1 : 0;
                            if (i + 1 < BLOCKS || j + 1 < COARSE_TURN) score[(i + 1) & 1] = product8(then ? cur : next, q[then / 2][then & 1]);
                            __builtin_amdgcn_sched_barrier(0);  // a product, then the maxima of the one before it
                            best[i / 2][i & 1] = fold16i(best[i / 2][i & 1], score[i & 1]);
                            asm volatile("" : "+v"(best[i / 2][i & 1]));  // ... which the optimiser would otherwise move to the end of the cell
                            __builtin_amdgcn_sched_barrier(0);
                        }
                        cur = next;
                    }
                }
            };
            for (int cell = cell0; cell < cell1; ++cell) {
                const int k = (cell - cell0) * TURNS;
#pragma unroll 1
                for (int tt = 0; tt < TURNS; tt += 2) {
                    turn(k + tt, std::integral_constant<int, 0>{});
                    turn(k + tt + 1, std::integral_constant<int, 1>{});
                }
                // lanes 0..31 finish the first block of a pair, lanes 32..63 the second
                const SegInfo si = info[cell / CELLS];
                uint16_t* upper = ca.upper + ((int64_t)b * n_cells + cell) * ca.slab + slot0 + lane;
                float first_up = 0.0f;
#pragma unroll
                for (int p = 0; p < LIVE; ++p) {
                    const auto sw = __builtin_amdgcn_permlane32_swap((uint32_t)best[p][0], (uint32_t)best[p][1], false, false);
                    const float score = (float)max((int)sw[0], (int)sw[1]) * si.scale;
                    const float error = __builtin_fmaf(__uint_as_float(bound[p] & 0xFFFF0000u), si.residual,
                                                       __uint_as_float(bound[p] << 16) * si.length);
                    low[p] = __builtin_fmaxf(low[p], score - error);
                    float up = score + error;
                    up = __builtin_fmaf(__builtin_fabsf(up), 1.0f / 126.0f, up);  // so that cutting it to bf16 leaves a bound
                    if (p == 0) first_up = up;
                    if (slot0 + p * 64 + lane < slot_end) upper[p * 64] = (uint16_t)(__float_as_uint(up) >> 16);
                    best[p][0] = best[p][1] = -0x7FFFFFFF;
                }
                const int done = cell - cell0;
                if (VOTE && done < VOTE_CELLS && cell0 + VOTE_CELLS <= cell1) {  // uniform in the workgroup
                    const bool here = slot0 + lane < slot_end;
                    uint32_t* lower = &ca.lower[(int64_t)b * ca.slot_pitch + ca.first_slot + slot0 + lane];
                    // a wave each of a few workgroups votes (see the end of refine_kernel)
                    const int apart = (units + VOTERS - 1) / VOTERS;
                    if (done == 0) {
                        if (here) atomicMax(lower, order_bits(low[0]));
                    } else if (done == 1) {
                        if (chunk % apart == 0 && (chunk / apart & (COARSE_WAVES - 1)) == wave) {
                            const uint32_t known = here ? atomicMax(lower, order_bits(low[0])) : 0;
                            const uint32_t doubt = __popcll(__ballot(here && first_up >= __builtin_fmaxf(low[0], unorder_bits(known))));
                            if (lane == 0 && here) {
                                u64 tally = 1ull << 48 | (u64)min(64, slot_end - slot0) << 24 | doubt;
                                tally += atomicAdd(&ca.vote[b].tally, tally);
                                // a query is in doubt about one more of s cells with the odds even : s - 1, where `even` cells of all leave it in doubt
                                const float even = ca.even * n_cells, others = 2.0f * chunks - 1.0f;
                                const float all = (float)((uint32_t)(tally >> 24) & 0xFFFFFFu), doubtful = (float)((uint32_t)tally & 0xFFFFFFu);
                                if (tally >> 48 >= VOTERS / 4 && doubtful * (even + others) > all * even)
                                    __hip_atomic_store(&ca.vote[b].given_up, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                            }
                        }
                    } else {
                        if (threadIdx.x == 0) leave = __hip_atomic_load(&ca.vote[b].given_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        __syncthreads();  // (the next write lies behind the barriers of the next turns)
                        if (leave) return true;
                    }
                }
            }
            return false;
        };
        // uniform in the wave; the waves of a workgroup meet at the same number of barriers whatever their LIVE
        const int n_live = max(0, min(PAIRS, (slot_end - slot0 + 63) / 64));
        const bool given_up = with_count<PAIRS>(n_live, sweep);
#pragma unroll
        for (int p = 0; p < PAIRS; ++p) {
            const int slot = slot0 + p * 64 + lane;
            if (slot < slot_end) atomicMax(&ca.lower[(int64_t)b * ca.slot_pitch + ca.first_slot + slot], order_bits(low[p]));
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);  // the turn past the last one has landed too
        __syncthreads();                     // before the next unit's first turn takes its place
        if (given_up) return;
    }
}

// ---- step 2 ------------------------------------------------------------------------------------
// A workgroup owns one cell (or a part of one) and a range of the queries: its tiles stay in registers, RT per wave, and the
// queries that need it are collected in LDS and streamed past them, 32 at a time.
template <int CT, int DP>
constexpr int refine_tiles() { return Ops<CT, DP>::ROW_BYTES / 8 <= 8 ? 8 : 4; }  // a tile is ROW_BYTES / 8 registers
template <int CT, int DP>
constexpr int refine_waves() { return Ops<CT, DP>::ROW_BYTES <= 48 ? 4 : (Ops<CT, DP>::ROW_BYTES < 160 ? 3 : 2); }  // per SIMD
constexpr int REFINE_SCAN = 4096;             // queries looked at between two looks at the list's length
constexpr int REFINE_LIST = REFINE_SCAN + 1024;
constexpr int REFINE_PART = 512;               // a multiple of 32
constexpr int REFINE_MOST = 4 * REFINE_SCAN;   // queries of a workgroup, at the most
constexpr int REFINE_LEAST = 1024;             // (ca.range: whole 1024s, whose bits may be in an order of their own)
constexpr int REFINE_SHORT = 128;              // of REFINE_SCAN queries; lists no longer than this are not worth a workgroup

// MASK: which queries need a cell is read from a table of bits; the keys name units of DENSE_J tiles instead of tiles.
template <int CT, int DP, int RT, int WAVES, bool MASK>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(refine_waves<CT, DP>())))
void refine_kernel(SearchArgs a, CoarseArgs ca) {
    using O = Ops<CT, DP>;
    using Frag = typename O::Frag;
    constexpr int THREADS = 64 * WAVES, PER = REFINE_SCAN / THREADS, UNIT = MASK ? DENSE_J : 1;
    static_assert(RT % UNIT == 0, "a wave holds whole units");
    __shared__ int list_row[REFINE_LIST];        // queries that need this segment: their rows,
    __shared__ uint16_t list_slot[REFINE_LIST];  // and their slots in the workgroup's range
    __shared__ u64 keys[REFINE_PART];            // what the waves found for REFINE_PART of them
    __shared__ int n_list;
    const int lane = threadIdx.x & 63, c = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int cell = blockIdx.x, b = blockIdx.z;
    const DenseWay way = MASK ? ca.judge.way(b) : DENSE_ONE_STEP;
    if (MASK && (way == DENSE_ONE_STEP || (ca.second_round && way != DENSE_GROUPS))) return;
    const bool grouped = MASK && ca.side == 1 && way == DENSE_GROUPS;
    const int cell_shift = ca.cell_shift - (grouped ? 1 : 0);
    int n_act = a.nq;
    if (a.nq_active) n_act = min(max(a.nq_active[b], 0), a.nq);
    bool every = n_act < ca.min_live;             // step 1 left these queries to this kernel
    constexpr bool VOTES = !MASK && CT != CT_F32 && DP <= 32;  // as coarse_votes() says (more arguments cost the widest rows a resident workgroup)
    if (VOTES) every = every || (ca.vote && ca.vote[b].given_up) || (ca.earlier && gives_up(ca.earlier[b], ca.even));
    uint32_t again = 0;
    n_act = min(n_act - ca.first_slot, ca.slab);  // slots are counted from first_slot on
    if (grouped) n_act = min((n_act + DENSE_CELL_PIXELS - 1) & ~(DENSE_CELL_PIXELS - 1), ca.slab);  // bits that stand for no candidate are 0
    int range = ca.range;
    if (MASK && !ca.second_round && range < REFINE_MOST && ca.judge.marked[DENSE_RECORD * b + ca.side] * (REFINE_SCAN / DENSE_SAMPLES) < REFINE_SHORT * ca.n_cells) range = REFINE_MOST;
    const int begin = blockIdx.y * range;
    n_act = min(n_act, begin + range);
    const int tile0 = (cell * WAVES + wave) * RT;
    if (n_act <= begin) return;

    const char* tgt = a.tgt + (int64_t)b * a.tgt_bstride;
    const char* src = a.src + (int64_t)b * a.src_bstride + take_slots_from(a, ca.first_slot) * O::ROW_BYTES;
    const int64_t qbase = (int64_t)b * a.nq + ca.first_slot;
    const float ninf = -__builtin_inff();
    const uint16_t* upper = ca.upper + ((int64_t)b * ca.n_cells + (cell >> ca.cell_shift)) * ca.slab;
    const int64_t bits = b * ca.slot_pitch * 64 + (int64_t)(cell >> cell_shift) * ca.slab;  // (MASK)
    const uint32_t* lower = ca.lower + (int64_t)b * ca.slot_pitch + ca.first_slot;
    Frag cand[RT];
#pragma unroll
    for (int j = 0; j < RT; ++j) cand[j] = O::load_tile(tgt + (int64_t)min(tile0 + j, a.m_tiles - 1) * (32 * O::ROW_BYTES), c, h);
    const bool tail = (tile0 + RT) * 32 > a.m;  // uniform: some of this wave's candidates lie past the map

    if (threadIdx.x == 0) n_list = 0;
    for (int i = threadIdx.x; i < REFINE_PART; i += THREADS) keys[i] = 0;
    __syncthreads();
    // Bits are looked at for the whole range at once where the list has room for what they mark (a look at a quarter of them cost a memory latency and four barriers each;
    // the three launches of 512x384 244 -> 233 us, the five of 1024x768 1577 -> 1350)
    bool whole = false;
    if constexpr (MASK) {
        constexpr int WIDE = REFINE_MOST / THREADS;  // bits of a thread, 64 or 32
        static_assert(WIDE == 64 || WIDE == 32, "a word of the table, or half of one");
        const int slot = begin + (int)threadIdx.x * WIDE;
        uint64_t need = 0;
        if (slot < n_act) {
            const int64_t at = (bits + slot) / WIDE;
            if constexpr (WIDE == 64) need = ca.mask[at];
            else need = reinterpret_cast<const uint32_t*>(ca.mask)[at];
            if (n_act - slot < WIDE) need &= ((uint64_t)1 << (n_act - slot)) - 1;
        }
        const int mine = __popcll(need);
        int upto = mine;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int y = __shfl_up(upto, d);
            if (lane >= d) upto += y;
        }
        const int count = __shfl(upto, 63);
        int at = 0;
        if (lane == 0 && count) at = atomicAdd(&n_list, count);
        at = __shfl(at, 0) + upto - mine;
        __syncthreads();
        const int total = n_list;
        if (total == 0) return;  // uniform
        whole = total <= REFINE_LIST;
        __syncthreads();  // read by every wave
        if (whole) {
            for (; need; need &= need - 1, ++at) {
                int found = slot + __builtin_ctzll(need);
                if (grouped) found = (found & ~(DENSE_CELL_PIXELS - 1)) + mask_candidate(found & (DENSE_CELL_PIXELS - 1));
                list_slot[at] = (uint16_t)(found - begin);
                list_row[at] = (int)query_row(a, qbase, found);
            }
        } else if (threadIdx.x == 0) {
            n_list = 0;
        }
        __syncthreads();
    }
    const int step = whole ? REFINE_MOST : REFINE_SCAN;
    for (int base = begin; base < n_act; base += step) {  // uniform
        if (whole) {
            // listed above
        } else if (!MASK && every) {
            // listed side by side: one after the other, PER to a thread, the loads of their rows were a memory latency each (16 512x384 pairs
            // of seeds, about a hundred of each still live in the second iteration: the call 1027 -> 1005 us)
            const int count = min(REFINE_SCAN, n_act - base);
            for (int i = threadIdx.x; i < count; i += THREADS) {
                list_slot[i] = (uint16_t)(base - begin + i);
                list_row[i] = (int)query_row(a, qbase, base + i);
            }
            if (threadIdx.x == 0) n_list = count;
        } else {
            const int slot = base + (int)threadIdx.x * PER;
            uint32_t need = 0;
            if (slot < n_act) {
                if constexpr (MASK) {
                    static_assert(PER <= 16, "a thread's bits lie in one 16-bit word");
                    const int64_t word = (bits + slot) / 16;
                    need = (uint32_t)reinterpret_cast<const uint16_t*>(ca.mask)[word] >> (slot & 15) & ((1u << PER) - 1);
                } else {
                    // the tables' rows hold whole 64s of slots: all PER are there
                    uint4 u[PER / 8], l[PER / 4];
#pragma unroll
                    for (int i = 0; i < PER / 8; ++i) u[i] = reinterpret_cast<const uint4*>(upper + slot)[i];
#pragma unroll
                    for (int i = 0; i < PER / 4; ++i) l[i] = reinterpret_cast<const uint4*>(lower + slot)[i];
#pragma unroll
                    for (int i = 0; i < PER; ++i) {
                        const uint4 u8 = u[i / 8], l4 = l[i / 4];
                        const uint32_t uw = (i & 7) < 2 ? u8.x : ((i & 7) < 4 ? u8.y : ((i & 7) < 6 ? u8.z : u8.w));
                        const uint32_t lw = (i & 3) == 0 ? l4.x : ((i & 3) == 1 ? l4.y : ((i & 3) == 2 ? l4.z : l4.w));
                        const float up = __uint_as_float(i & 1 ? uw & 0xFFFF0000u : uw << 16);
                        if (up >= unorder_bits(lw)) need |= 1u << i;
                    }
                }
                if (!grouped && n_act - slot < PER) need &= (1u << (n_act - slot)) - 1;
            }
            // a prefix sum over the wave, one LDS atomic for its total
            const int mine = __popc(need);
            int upto = mine;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int y = __shfl_up(upto, d);
                if (lane >= d) upto += y;
            }
            const int count = __shfl(upto, 63);
            int at = 0;
            if (lane == 0 && count) at = atomicAdd(&n_list, count);
            at = __shfl(at, 0) + upto - mine;
            for (; need; need &= need - 1, ++at) {
                int found = slot + __builtin_ctz(need);
                if (grouped) found = (found & ~(DENSE_CELL_PIXELS - 1)) + mask_candidate(found & (DENSE_CELL_PIXELS - 1));
                list_slot[at] = (uint16_t)(found - begin);
                list_row[at] = (int)query_row(a, qbase, found);
            }
        }
        __syncthreads();
        const int n = n_list;
        __syncthreads();  // read by every wave before the next round adds to it
        if (n > REFINE_LIST - REFINE_SCAN || base + step >= n_act) {  // uniform
            again += n;
            auto sweep = [&](int part, int part_end, auto tail_tag) {
                constexpr bool TAIL = decltype(tail_tag)::value;
                Frag next = O::load(src + (int64_t)list_row[min(part + c, n - 1)] * O::ROW_BYTES, h);
#pragma unroll 1
                for (int first = part; first < part_end; first += 32) {
                    const Frag q = next;
                    next = O::load(src + (int64_t)list_row[min(first + 32 + c, n - 1)] * O::ROW_BYTES, h);
                    float best = ninf;
                    int best_unit = 0x7FFFFFFF;
                    int bound = a.m - tile0 * 32 - 4 * h;
                    if (TAIL) asm volatile("" : "+v"(bound));  // else its comparisons are kept from block to block
#pragma unroll
                    for (int u = 0; u < RT; u += UNIT) {
                        float top = best;
#pragma unroll
                        for (int j = u; j < u + UNIT; ++j) {
                            f32x16 acc = O::mma(cand[j], q);
                            if (TAIL) {
#pragma unroll
                                for (int v = 0; v < 16; ++v)
                                    if (32 * j + tile_row(v, 0) >= bound) acc[v] = ninf;
                            }
                            top = fold16(top, acc);
                            // more than two products in flight cost registers, that is resident waves
                            if (UNIT > 1 && (j & 1)) {
                                asm volatile("" : "+v"(top));
                                __builtin_amdgcn_sched_barrier(0);
                            }
                        }
                        if (top > best) best_unit = (tile0 + u) / UNIT;
                        best = top;
                        if (UNIT == 1 && (u & 1)) {
                            asm volatile("" : "+v"(best));
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    }
                    // both halves of the wave file what they found
                    if (first + c < n) atomicMax(&keys[first - part + c], pack_key(best, best_unit));
                }
            };
            for (int part = 0; part < n; part += REFINE_PART) {  // uniform
                const int part_end = min(n, part + REFINE_PART);
                if (tail) sweep(part, part_end, std::true_type{});  // uniform in the wave, and there is no barrier inside
                else sweep(part, part_end, std::false_type{});
                __syncthreads();
                for (int i = threadIdx.x; i < part_end - part; i += THREADS) {
                    atomicMax(&a.out_keys[qbase + begin + list_slot[part + i]], keys[i]);
                    keys[i] = 0;
                }
                __syncthreads();
            }
            if (threadIdx.x == 0) n_list = 0;
            __syncthreads();
        }
    }
    // additions to one word are served one after the other: the workgroups of every 16th cell speak for the rest
    if (VOTES && ca.vote && !every && threadIdx.x == 0 && cell % 16 == 0) {
        atomicAdd(&ca.vote[b].again, (u64)again);
        atomicAdd(&ca.vote[b].of, (u64)(n_act - begin));
    }
}

// ---- launches --------------------------------------------------------------------------------------
template <int CT, int DP, bool SPLIT, QuantiseRows FROM = ROWS_PREPARED>
static hipError_t launch_quantise_t(const QuantiseArgs& a, hipStream_t s) {
    const int segs = a.side[0].out.n_segs > a.side[1].out.n_segs ? a.side[0].out.n_segs : a.side[1].out.n_segs;
    const dim3 grid(segs, 2 * a.batch);
    if (a.seg_pixels == 4096) return launch(TK_QUANTISE, quantise_kernel<CT, DP, SPLIT, FROM, 1024, 4, true>, grid, dim3(1024), 0, s, a);
    if (a.seg_pixels == 2048) return launch(TK_QUANTISE, quantise_kernel<CT, DP, SPLIT, FROM, 1024, 2, false>, grid, dim3(1024), 0, s, a);
    if (a.seg_pixels != SEG_PIXELS) return hipErrorInvalidValue;
    return launch(TK_QUANTISE, quantise_kernel<CT, DP, SPLIT, FROM, 512, SEG_PIXELS / 512, false>, grid, dim3(512), 0, s, a);
}
hipError_t launch_quantise(const QuantiseArgs& a, int compute, int dp, hipStream_t s) {
    if (a.raw_rows && a.split_d) return launch_quantise_t<CT_F16, 80, true, ROWS_RAW>(a, s);
    if (a.raw_rows) {
        if (a.normalize) return compute == FNN_F16 ? launch_quantise_t<CT_F16, 24, false, ROWS_RAW_NORMALIZED>(a, s) : launch_quantise_t<CT_BF16, 24, false, ROWS_RAW_NORMALIZED>(a, s);
        if (compute == FNN_F16) return launch_quantise_t<CT_F16, 24, false, ROWS_RAW>(a, s);
        return launch_quantise_t<CT_BF16, 24, false, ROWS_RAW>(a, s);
    }
    if (a.split_d) {
        if (dp == 24) return launch_quantise_t<CT_F16, 24, true>(a, s);
        if (dp == 32) return launch_quantise_t<CT_F16, 32, true>(a, s);
        if (dp == 48) return launch_quantise_t<CT_F16, 48, true>(a, s);
        if (dp == 64) return launch_quantise_t<CT_F16, 64, true>(a, s);
        if (dp == 80) return launch_quantise_t<CT_F16, 80, true>(a, s);
        if (dp == 96) return launch_quantise_t<CT_F16, 96, true>(a, s);
    } else if (compute == FNN_F16) {
        if (dp == 24) return launch_quantise_t<CT_F16, 24, false>(a, s);
        if (dp == 32) return launch_quantise_t<CT_F16, 32, false>(a, s);
    } else if (compute == FNN_BF16) {
        if (dp == 24) return launch_quantise_t<CT_BF16, 24, false>(a, s);
        if (dp == 32) return launch_quantise_t<CT_BF16, 32, false>(a, s);
    } else {
        if (dp == 8) return launch_quantise_t<CT_F32, 8, false>(a, s);
        if (dp == 16) return launch_quantise_t<CT_F32, 16, false>(a, s);
        if (dp == 24) return launch_quantise_t<CT_F32, 24, false>(a, s);
        if (dp == 32) return launch_quantise_t<CT_F32, 32, false>(a, s);
    }
    return hipErrorInvalidValue;
}

// The model behind the choice, in nanoseconds, fitted to calls between 16384 and a million pixels before search_unit and coarse_kernel put their products and maxima
// in turn and the late iterations became one launch.  Both ways of 126 calls near the line with the present kernels, inputs not in the caches: the 56 that it
// takes lose 2.6 % at worst (two 512x384 pairs of fp16 products whose seeds settle at once, 281 us in one step, 289 in two) and gain up to 63 %; the 70 that it leaves
// would gain up to 14 % (16 pairs with squared distance 1964 / 1718; 3072 queries of one 640x480 pair 63 / 57, of two 512x384 pairs 73 / 67, of 32 channels 79 / 71; fp32
// products, 200x150, 131 / 119), and one that it takes for two of its four searches another 27 % in all four (fp32 products, 256x192, 768 seeds, 172 / 136).  The model knows sizes
// only: it counts on half of the seeds in the second iteration, and on maps that tell pixels apart (three 512x384 pairs, features of 1 pixel 374 / 372, of 4 418 / 413).
constexpr double BYTES_PER_NS = 4500.0;  // what the passes over the maps reach
static int coarse_row_bytes(int compute, int dp) { return dp * elem_size(compute); }
// Cells that a slot is multiplied with again: 4 of 1024 pixels for unit rows of 16 channels and more, however large the map; with few
// channels, a share of the map (of 96 segments 5.3, 6.6, 10, 28 and 89 at 12, 10, 8, 6 and 4 channels).  FNN_FLAG_L2 has
// wider bounds, because its norm terms are multiplied by channels of ones (20 of 96, 29 of 192; 47 and 77 of 96 at 8 and 6).
double coarse_cells_again(double cells, int d, bool l2) {
    const double few = (l2 ? 8.0 : 6.0) / d;
    const double again = (l2 ? 32.0 : 5.0) + 0.26 * few * few * few * few * cells;
    return again < cells ? again : cells;
}
double coarse_gain(int64_t nq, int64_t m, int batch, int compute, int dp, int d, bool l2) {
    const bool cheap = compute != FNN_F32 && dp <= 32;
    // rows of 16 channels take one matrix instruction per block as it is
    if (m < 16 * SEG_PIXELS || nq > 0x7FFFFFFF / 2 || (cheap && dp <= 16)) return -1e30;
    if (batch * m > (int64_t)1 << 26) return -1e30;  // the tables of bounds would pass 1 GB
    // what a block of 32x32 scores takes one SIMD in search_kernel, and in coarse_kernel
    const double exact = compute == FNN_F32 ? 18.75 * dp : (cheap ? 46.0 : 1.64 * dp), coarse = 26.0;
    const double blocks = (double)batch * ((nq + 31) / 32) * ((m + 31) / 32) / 1024.0;
    // (the second step runs at two thirds of search_kernel's rate)
    const double segments = (double)m / SEG_PIXELS, again = 1.5 * coarse_cells_again(segments, d, l2) / segments;
    return blocks * (exact * (1.0 - again) - coarse) - 5000.0 - (double)batch * m * coarse_row_bytes(compute, dp) / BYTES_PER_NS;
}
// Wider rows and fp32 products cost so much more than an 8-bit score that two steps lose little at worst (one descriptor throughout, two
// 512x384 pairs in fp32: a quarter).
bool coarse_votes(int compute, int dp) { return compute != FNN_F32 && dp <= 32; }
double coarse_cost(int64_t rows, int compute, int dp) {
    return 4000.0 + (double)rows * (coarse_row_bytes(compute, dp) + COARSE_ROW_BYTES + 4) / BYTES_PER_NS;
}

// What coarse_kernel's split of a search leaves to the busiest wave, times the waves that share a SIMD with it: the time of a
// launch whose workgroups are all resident, in products of one pair of query blocks and one cell.
static int coarse_wgs_per_pair(int resident, int batch) {
    int wgs = resident / batch;
    if (wgs >= 8) wgs &= ~7;  // a multiple of 8 per pair keeps the XCD renumbering a bijection
    return wgs < 1 ? 1 : wgs;
}
static int64_t coarse_longest(int wide, int resident, int batch, int64_t pairs, int64_t n_cells) {
    const int64_t wgs = coarse_wgs_per_pair(resident, batch), quads = (pairs + wide * COARSE_WAVES - 1) / (wide * COARSE_WAVES);
    int64_t chunks = wgs / quads < n_cells ? wgs / quads : n_cells;
    if (chunks < 1) chunks = 1;
    const int64_t rounds = (quads * chunks + wgs - 1) / wgs;
    const int64_t per_wave = (pairs + quads * COARSE_WAVES - 1) / (quads * COARSE_WAVES), cells = (n_cells + chunks - 1) / chunks;
    return resident * rounds * per_wave * cells;
}

// Half segments split a small search more evenly and spread step 2 over more workgroups; whole ones read a tile a third as often and keep the pipeline
// of products and maxima filled for longer.  The split that leaves less to the busiest wave is taken, with the workgroups that 256 compute units hold of either
// kernel (a workspace is sized without a device), where a half segment's products count 18 % more and half segments have two
// products of each wave on a SIMD ahead of whole ones.  Where step 2 would have few workgroups, or dear ones, half segments win anyway.  (Over 210 calls from 256x192 to
// 1024x768, 1 to 16 pairs, 2048 to 12288 queries, the slower split is taken in 25, which costs 1.9 % on average there and 7.7 % at most.)  Whole / half segments, all
// of a call's time in us: 3072 queries: 256x192, 2 pairs 47.9 / 34.2, 4 51.3 / 47.5, 8 71.8 / 73.4; 320x240, 2 48.8 / 39.8, 4 59.5 / 57.3, 8 101.9 / 97.8, 16 171.1 / 177.4; 512x384, 1
// 45.9 / 42.0, 2 58.9 / 61.4, 3 86.0 / 82.9, 4 100.0 / 105.7, 8 190.6 / 206.5, 16 370.0 / 403.5; 640x480, 2 87.0 / 85.0, 3 118.0 / 120.2; 768x576, 1 66.9 / 66.5; 1024x768, 1 94.0 / 100.7; 12288
// queries: 256x192, 2 pairs 77.7 / 69.4, 8 205.0 / 209.8, 16 375.9 / 431.9; 512x384, 4 297.0 / 322.4; seeds that walk: 512x384, 4 pairs 414 / 426, 6 584 / 585, 16
// 1338 / 1437; 640x480, 1 313 / 284, 1024x768 1017 / 1086; every pixel of 256x192 126 / 116, of 320x240 220 / 234; fp32 products, 512x384, 3072 seeds of 1 pair 268 / 225,
// of 4 581 / 565, 768 of 8 582 / 562; two-term rows of 1 pair 263 / 238, of 2 383 / 355, of 4 585 / 609.
constexpr int COARSE_WGS_8 = 512, COARSE_WGS_6 = 768, COARSE_WGS_HALF = 1024;
int coarse_cells(int64_t nq, int64_t n_segs, int batch, int compute) {
    if (n_segs < 1 || nq < 1) return 1;
    const int64_t pairs = (nq + 63) / 64;
    const int64_t eight = coarse_longest(8, COARSE_WGS_8, batch, pairs, n_segs), six = coarse_longest(6, COARSE_WGS_6, batch, pairs, n_segs);
    const double half = 0.5 * coarse_longest(2, COARSE_WGS_HALF, batch, pairs, 2 * n_segs), whole = (double)(eight < six ? eight : six);
    return n_segs * batch < 160 || (compute == FNN_F32 && n_segs * batch <= 1024) || 1.18 * half < whole + 2 * COARSE_WGS_8 ? 2 : 1;
}

int64_t coarse_slab(int64_t nq, int64_t n_segs, int batch) {
    const int64_t most = ((int64_t)128 << 20) / ((n_segs > 0 ? n_segs : 1) * batch) / 1024 * 1024;  // 256 MB of bounds (whole segments)
    const int64_t all = round_up(nq, 64);
    if (most < 8192) return all < 8192 ? all : 8192;
    return all < most ? all : most;
}

// Workgroups that the current device holds at once (0: unknown).
template <int PAIRS, int CELL>
static int coarse_resident() {  // (voting costs registers, not resident workgroups)
    static DeviceCache resident_wgs;
    const long long resident = resident_wgs.get([](int dev) -> long long {
        int per_cu = 0;
        hipDeviceProp_t prop;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, coarse_kernel<PAIRS, CELL, false>, COARSE_WAVES * 64, 0) != hipSuccess ||
            hipGetDeviceProperties(&prop, dev) != hipSuccess)
            return -1;
        return (long long)(per_cu > 0 ? per_cu : 1) * prop.multiProcessorCount;
    });
    return resident > 0 ? (int)resident : 0;
}
template <int PAIRS, int CELL>
static hipError_t launch_coarse_t(const SearchArgs& a, const CoarseArgs& ca, int batch, hipStream_t s) {
    const int resident = coarse_resident<PAIRS, CELL>();
    if (resident == 0) return hipErrorUnknown;
    if (CELL == SEG_TILES && ca.vote)
        return launch_detail(TK_COARSE, PAIRS * 2, coarse_kernel<PAIRS, CELL, CELL == SEG_TILES>, dim3(coarse_wgs_per_pair(resident, batch), batch), dim3(COARSE_WAVES * 64), 0, s, a, ca);
    return launch_detail(TK_COARSE, PAIRS * 2, coarse_kernel<PAIRS, CELL, false>, dim3(coarse_wgs_per_pair(resident, batch), batch), dim3(COARSE_WAVES * 64), 0, s, a, ca);
}
// CELL: tiles of a workgroup.
template <int CT, int DP, int CELL, bool MASK = false>
static hipError_t launch_refine_t(const SearchArgs& a, CoarseArgs ca, int batch, hipStream_t s) {
    constexpr int RT = refine_tiles<CT, DP>() * CELL / SEG_TILES, WAVES = CELL / RT;
    const int64_t slots = a.nq - ca.first_slot < ca.slab ? a.nq - ca.first_slot : ca.slab;
    const unsigned cells = (unsigned)((a.m_tiles + CELL - 1) / CELL);
    // Where neighbouring pixels resemble each other, what a cell is marked by lies together: a workgroup with many queries may need the
    // cell for all of them and be what the launch waits for.  Short ranges even that out (dense mode, fp16, 24 channels, 512x384, features of 128
    // pixels, both launches with ranges of 16384 / 4096: 1104 / 548 us), shorter ones where workgroups are fewer (the whole call, features of 32 pixels, ranges of 4096 / 2048 / 1024: four pairs
    // of 192x144 400 / 358 / 330, of 224x168 641 / 540 / 540, one of 288x216 474 / 394 / 357; of one pixel 313 / 320 / 325, 463 / 452 / 453, 325 / 318 / 324); but each reads its tiles again and fills up its last block, so they are taken
    // while the workgroups are few and where the samples say that the lists are long (features of one pixel, four pairs: 324 / 365 us; 1024x768
    // 1085 / 1662).  Rows that cost more per product lose more to the last block of a list than they gain (fp32, 384x288, features of one pixel 356 / 794).
    // What the candidates' second round lists is little, but few workgroups would take it one after the other: their ranges are halved until there are four for every compute unit (one pair of 288x216
    // in ranges of 16384 / 2048, features of 1, 4, 64 and 128 pixels 323 / 314, 332 / 334, 432 / 380 and 579 / 423 us; twice as many workgroups 321, 340, 379 and 407; two-term rows, 400x300 859 / 881).
    ca.range = REFINE_MOST;
    if (MASK && CT != CT_F32 && DP <= 32 && ca.second_round)
        for (; ca.range > REFINE_LEAST && cells * ((slots + ca.range - 1) / ca.range) * batch < 1024;) ca.range /= 2;
    else if (MASK && CT != CT_F32 && DP <= 32)
        for (ca.range = REFINE_LEAST; ca.range < REFINE_MOST && cells * ((slots + ca.range - 1) / ca.range) * batch > (ca.range < REFINE_SCAN ? 4096 : 16384);) ca.range *= 2;
    const unsigned ranges = (unsigned)((slots + ca.range - 1) / ca.range);
    return launch(TK_REFINE, refine_kernel<CT, DP, RT, WAVES, MASK>, dim3(cells, ranges, batch), dim3(64 * WAVES), 0, s, a, ca);
}
template <int CT, int DP>
static hipError_t launch_both_t(const SearchArgs& a, CoarseArgs ca, int batch, hipStream_t s) {
    const bool half = coarse_cells(a.nq, ca.tgt.n_segs, batch, CT) == 2;
    ca.n_cells = ca.tgt.n_segs * (half ? 2 : 1);
    ca.cell_shift = 0;
    // Waves of up to 16 query blocks read a tile the fewest times; with up to 12 a third wave fits on every SIMD.  Whichever leaves less to the
    // busiest wave is the faster, and where both leave the same to the same quads, the third wave is (16 / 12 blocks, fp16, 24 channels, the
    // whole call: 16 512x384 pairs of 2300 queries 316 / 315 us, 3072 369 / 368, 3500 411 / 418, 4608 522 / 502, 7000 706 / 745; 12 pairs of 3072
    // 290 / 285; 30 320x240 pairs of 3072 312 / 316, 4608 426 / 425; six 640x480 pairs of 4800 329 / 317; every pixel of one 512x384 pair 1135 / 1085).
    bool six = false;
    if (!half) {
        const int wide = coarse_resident<8, SEG_TILES>(), narrow = coarse_resident<6, SEG_TILES>();
        if (wide == 0 || narrow == 0) return hipErrorUnknown;
        const int slab_pairs = (int)((a.nq < ca.slab ? a.nq : ca.slab) + 63) / 64;
        const int64_t of8 = coarse_longest(8, wide, batch, slab_pairs, ca.n_cells), of6 = coarse_longest(6, narrow, batch, slab_pairs, ca.n_cells);
        six = of6 < of8 || (of6 == of8 && (slab_pairs + 31) / 32 == (slab_pairs + 23) / 24);
    }
    for (int64_t first = 0; first < a.nq; first += ca.slab) {
        ca.first_slot = (int32_t)first;
        hipError_t e = half ? launch_coarse_t<2, SEG_TILES / 2>(a, ca, batch, s)
                            : (six ? launch_coarse_t<6, SEG_TILES>(a, ca, batch, s) : launch_coarse_t<8, SEG_TILES>(a, ca, batch, s));
        if (e == hipSuccess) e = half ? launch_refine_t<CT, DP, SEG_TILES / 2>(a, ca, batch, s) : launch_refine_t<CT, DP, SEG_TILES>(a, ca, batch, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_coarse_search(const SearchArgs& a, const CoarseArgs& ca, int batch, int compute, int dp, hipStream_t s) {
    if (a.nq <= 0 || batch <= 0) return hipSuccess;
    if (compute == FNN_F16) {
        if (dp == 24) return launch_both_t<CT_F16, 24>(a, ca, batch, s);
        if (dp == 32) return launch_both_t<CT_F16, 32>(a, ca, batch, s);
        if (dp == 48) return launch_both_t<CT_F16, 48>(a, ca, batch, s);
        if (dp == 64) return launch_both_t<CT_F16, 64>(a, ca, batch, s);
        if (dp == 80) return launch_both_t<CT_F16, 80>(a, ca, batch, s);
        if (dp == 96) return launch_both_t<CT_F16, 96>(a, ca, batch, s);
    } else if (compute == FNN_BF16) {
        if (dp == 24) return launch_both_t<CT_BF16, 24>(a, ca, batch, s);
        if (dp == 32) return launch_both_t<CT_BF16, 32>(a, ca, batch, s);
    } else {
        if (dp == 8) return launch_both_t<CT_F32, 8>(a, ca, batch, s);
        if (dp == 16) return launch_both_t<CT_F32, 16>(a, ca, batch, s);
        if (dp == 24) return launch_both_t<CT_F32, 24>(a, ca, batch, s);
        if (dp == 32) return launch_both_t<CT_F32, 32>(a, ca, batch, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_refine(const SearchArgs& a, const CoarseArgs& ca, int batch, int compute, int dp, hipStream_t s) {
    if (a.nq <= 0 || batch <= 0) return hipSuccess;
    if (compute == FNN_F16) {
        if (dp == 24) return launch_refine_t<CT_F16, 24, SEG_TILES, true>(a, ca, batch, s);
        if (dp == 32) return launch_refine_t<CT_F16, 32, SEG_TILES, true>(a, ca, batch, s);
        if (dp == 48) return launch_refine_t<CT_F16, 48, SEG_TILES, true>(a, ca, batch, s);
        if (dp == 64) return launch_refine_t<CT_F16, 64, SEG_TILES, true>(a, ca, batch, s);
        if (dp == 80) return launch_refine_t<CT_F16, 80, SEG_TILES, true>(a, ca, batch, s);
        if (dp == 96) return launch_refine_t<CT_F16, 96, SEG_TILES, true>(a, ca, batch, s);
    } else if (compute == FNN_BF16) {
        if (dp == 24) return launch_refine_t<CT_BF16, 24, SEG_TILES, true>(a, ca, batch, s);
        if (dp == 32) return launch_refine_t<CT_BF16, 32, SEG_TILES, true>(a, ca, batch, s);
    } else {
        if (dp == 8) return launch_refine_t<CT_F32, 8, SEG_TILES, true>(a, ca, batch, s);
        if (dp == 16) return launch_refine_t<CT_F32, 16, SEG_TILES, true>(a, ca, batch, s);
        if (dp == 24) return launch_refine_t<CT_F32, 24, SEG_TILES, true>(a, ca, batch, s);
        if (dp == 32) return launch_refine_t<CT_F32, 32, SEG_TILES, true>(a, ca, batch, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace fnn
