// Pass 1 of the dense mode in 8-bit integers: the same sweep as dense_kernel -- every 32x32 block of scores formed once and
// folded into the best candidate of its queries and the best query of its candidates -- with one matrix
// instruction per block, nothing located and nothing masked (rows past a map repeat its last one).  What is kept are the
// maxima per query and cell of candidates and per candidate and segment of queries; bounds on what the 8 bits left out say
// which cells the second step of the searches (coarse.hip) has to multiply again, in both directions.
#include <type_traits>

#include "coarse_device.hpp"
#include "dense_perm.hpp"
#include "fnn_kernels.hpp"
#include "trace.hpp"

namespace fnn {

constexpr int DC_J = 4;                                  // candidate tiles resident per wave
constexpr int DC_GROUP = COARSE_WAVES * DC_J;            // tiles of a workgroup: 512 candidates
constexpr int DC_TURNS = DENSE_SB_PIXELS / 32 / COARSE_TURN;  // turns of a sweep
constexpr int DC_STEPS = COARSE_TURN / 2;                // steps of a turn, two query blocks each
static_assert(DC_TURNS % 2 == 0, "a sweep is an even number of turns, so it starts on stage slot 0");
constexpr int LOWEST = -0x7FFFFFFF;
// Maxima are kept as multiples of 16, in 16 bits: at most 128 * 128 * 32 / 16 (a row without bounds may reach one more, whose bound does not care)
constexpr int KEPT_SHIFT = 4;

template <int CTRL>
__device__ __forceinline__ int dpp_max_int(int x) { return max(x, __builtin_amdgcn_update_dpp(0, x, CTRL, 0xF, 0xF, true)); }
// transpose_max16 for integers
__device__ __forceinline__ int transpose_max16_int(const int (&x)[16], int lane) {
    const int held = held_register(lane);
    const bool e0 = held & 1, e1 = held & 2, e2 = held & 4, e3 = held & 8;
    int y8[8], y4[4], y2[2];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int even = dpp_max_int<0xB1>(x[2 * k]), odd = dpp_max_int<0xB1>(x[2 * k + 1]);
        y8[k] = e0 ? odd : even;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int even = dpp_max_int<0x4E>(y8[2 * k]), odd = dpp_max_int<0x4E>(y8[2 * k + 1]);
        y4[k] = e1 ? odd : even;
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int even = dpp_max_int<0x141>(y4[2 * k]), odd = dpp_max_int<0x141>(y4[2 * k + 1]);
        y2[k] = e2 ? odd : even;
    }
    const int even = dpp_max_int<0x140>(y2[0]), odd = dpp_max_int<0x140>(y2[1]);
    const int y1 = e3 ? odd : even;
    const auto sw = __builtin_amdgcn_permlane16_swap((uint32_t)y1, (uint32_t)y1, false, false);
    return max((int)sw[0], (int)sw[1]);
}

// The prepared rows of image 1 of a pair, in the order that the dense kernels sweep: a thread of a two-dimensional grid copies 16 bytes at a time.
__device__ __forceinline__ void dense_permute(const DenseSwept& w, int b) {
    const uint4* from = reinterpret_cast<const uint4*>(w.from + (int64_t)b * w.from_bstride);
    uint4* to = reinterpret_cast<uint4*>(w.to + (int64_t)b * w.n_pad * w.row_bytes);
    const int words = w.row_bytes / 16;
    const int64_t n_threads = (int64_t)gridDim.x * gridDim.y * blockDim.x;
    for (int64_t i = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * blockDim.x + threadIdx.x; i < w.n_pad * words; i += n_threads)
        to[i] = from[slot_pixel(i / words) * words + i % words];
}

// A workgroup sweeps one run of queries past a few cells of candidates, a group of 16 tiles after the other.  At the end of every
// SEGMENT of queries the candidates' maxima are reduced over the lanes and kept.
// Bound by the vector unit: 16 three-input maxima per block, 16.8 instructions in all, that is 67 cycles beside 32 of the
// matrix instruction.  A bare loop of them takes 35.7 ns per block and SIMD, the kernel 38 to 40 (dense_staged_kernel 56).
template <int SEGMENT>
__global__ __launch_bounds__(COARSE_WAVES * 64) __attribute__((amdgpu_waves_per_eu(3)))
void dense_coarse_kernel(DenseCoarseArgs a) {
    __shared__ uint4 stage0[COARSE_TURN][64], stage1[COARSE_TURN][64];  // two variables, see dense_staged_kernel
    __shared__ int row_best[DENSE_SB_PIXELS];                           // best score of every query in the cell
    const int lane = threadIdx.x & 63, c = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int held = held_register(lane);
    const int cell0 = blockIdx.x * a.cells_per_wg, sb = blockIdx.y, b = blockIdx.z;
    if (a.judge.alike(b)) {
        if (a.swept.to) dense_permute(a.swept, b);
        return;
    }
    constexpr int SEGS = DENSE_SB_PIXELS / SEGMENT, SEG_TURNS = DC_TURNS / SEGS;
    const int64_t pixels1 = (int64_t)a.map[0].n_segs * SEGMENT, pixels2 = (int64_t)a.map[1].n_segs * SEGMENT;
    const char* blocks = a.map[0].rows + ((int64_t)b * pixels1 + (int64_t)(a.first_sb + sb) * DENSE_SB_PIXELS) * COARSE_ROW_BYTES;
    const char* tiles = a.map[1].rows + (int64_t)b * pixels2 * COARSE_ROW_BYTES;
    uint16_t* rows = a.best[0] + ((int64_t)b * a.n_cells + cell0) * ((int64_t)a.n_sb * DENSE_SB_PIXELS) + (int64_t)sb * DENSE_SB_PIXELS;
    uint16_t* cols = a.best[1] + ((int64_t)b * a.map[0].n_segs + (int64_t)(a.first_sb + sb) * SEGS) * pixels2;
    // groups of this workgroup's cells that hold a pixel of image 2 (uniform)
    const int group0 = cell0 * a.cell_groups;
    const int n_groups = min(a.cells_per_wg * a.cell_groups, (a.n_tiles[1] + DC_GROUP - 1) / DC_GROUP - group0);
    if (n_groups <= 0) return;
    const int total = n_groups * DC_TURNS;

    auto stage_turn = [&](uint4 (&slot)[COARSE_TURN][64], int k) {
        uint32_t l;  // read afresh: see dense_stage_turn
        asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
        const char* from = blocks + (int64_t)(min(k, total - 1) % DC_TURNS) * (COARSE_TURN * TILE_BYTES);
        const uint32_t off = (l & 31) * COARSE_ROW_BYTES + (l >> 5) * 16;
#pragma unroll
        for (int i = 0; i < 2; ++i)
            __builtin_amdgcn_global_load_lds((const void*)(from + (2 * wave + i) * TILE_BYTES + off), FNN_LDS_PTR(&slot[2 * wave + i][0]), 16, 0, 0);
    };
    stage_turn(stage0, 0);
    for (int i = threadIdx.x; i < DENSE_SB_PIXELS; i += COARSE_WAVES * 64) row_best[i] = LOWEST;

    int k = 0;
    for (int g = 0; g < n_groups; ++g) {
        const int tile0 = (group0 + g) * DC_GROUP + wave * DC_J;
        i32x4 cand[DC_J];
        int best[DC_J][16];
#pragma unroll
        for (int j = 0; j < DC_J; ++j) {
            cand[j] = *reinterpret_cast<const i32x4*>(tiles + (int64_t)(tile0 + j) * TILE_BYTES + c * COARSE_ROW_BYTES + 16 * h);
            arrived(cand[j]);
#pragma unroll
            for (int v = 0; v < 16; ++v) best[j][v] = LOWEST;
        }
        auto turn = [&](int tt, auto slot_tag) {
            constexpr int SLOT = decltype(slot_tag)::value;
            __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wave's share of the turn is in LDS
            __syncthreads();                     // everyone's is, and everyone has left the other slot
            stage_turn(SLOT ? stage0 : stage1, k + tt + 1);
            int found[DC_STEPS];  // best score of a step's queries (lanes 0..31 its first block, 32..63 its second)
#pragma unroll
            for (int s = 0; s < DC_STEPS; ++s) {
                const i32x4 qa = __builtin_bit_cast(i32x4, SLOT ? stage1[2 * s][lane] : stage0[2 * s][lane]);
                const i32x4 qb = __builtin_bit_cast(i32x4, SLOT ? stage1[2 * s + 1][lane] : stage0[2 * s + 1][lane]);
                int ra = LOWEST, rb = LOWEST;
#pragma unroll
                for (int j = 0; j < DC_J; ++j) {
                    const i32x16 pa = product8(cand[j], qa), pb = product8(cand[j], qb);
                    ra = fold16i(ra, pa);
                    rb = fold16i(rb, pb);
#pragma unroll
                    for (int v = 0; v < 16; ++v) best[j][v] = max3i(best[j][v], pa[v], pb[v]);
                }
                const auto sw = __builtin_amdgcn_permlane32_swap((uint32_t)ra, (uint32_t)rb, false, false);
                found[s] = max((int)sw[0], (int)sw[1]);
                __builtin_amdgcn_sched_barrier(0);  // steps are scheduled one by one: more products in flight would spill
            }
#pragma unroll
            for (int s = 0; s < DC_STEPS; ++s) atomicMax(&row_best[(tt * COARSE_TURN + 2 * s) * 32 + lane], found[s]);
        };
#pragma unroll 1
        for (int seg = 0; seg < SEGS; ++seg) {
#pragma unroll 1
            for (int tt = seg * SEG_TURNS; tt < (seg + 1) * SEG_TURNS; tt += 2) {
                turn(tt, std::integral_constant<int, 0>{});
                turn(tt + 1, std::integral_constant<int, 1>{});
            }
#pragma unroll
            for (int j = 0; j < DC_J; ++j) {
                const int top = transpose_max16_int(best[j], lane);
                if ((lane & 16) == 0)
                    cols[seg * pixels2 + (int64_t)(tile0 + j) * 32 + tile_row(held, h)] = (uint16_t)(top >> KEPT_SHIFT);
#pragma unroll
                for (int v = 0; v < 16; ++v) best[j][v] = LOWEST;
            }
        }
        k += DC_TURNS;
        if ((g + 1) % a.cell_groups == 0 || g + 1 == n_groups) {  // the end of a cell (uniform)
            __syncthreads();
            for (int i = threadIdx.x * 2; i < DENSE_SB_PIXELS; i += COARSE_WAVES * 128) {
                const int2 two = *reinterpret_cast<const int2*>(&row_best[i]);
                *reinterpret_cast<uint32_t*>(rows + i) = ((uint32_t)(two.x >> KEPT_SHIFT) & 0xFFFFu) | ((uint32_t)(two.y >> KEPT_SHIFT) << 16);
                *reinterpret_cast<int2*>(&row_best[i]) = make_int2(LOWEST, LOWEST);
            }
            rows += (int64_t)a.n_sb * DENSE_SB_PIXELS;
        }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);  // the turn past the last one has landed too
}

// Which cells may hold the best partner of a slot: the bounds that turn 8-bit scores into products (coarse.hip) give every slot a
// lower bound of its best score, and a cell whose upper bound reaches it is marked.  A lane takes SELECT_SLOTS slots,
// 64 apart; the waves of a workgroup share the cells.  Bound by memory; the table is read twice, the second time mostly
// from cache.
constexpr int SELECT_WAVES = 4;
constexpr int SELECT_SLOTS = 4;
constexpr int SELECT_DEEP = 6;  // cells in flight per wave
struct SelectSide {
    const uint16_t* best;       // [batch][n_cells][pitch]
    uint64_t* mask;             // [batch][n_cells][pitch / 64]
    int32_t n_cells;
    int64_t pitch;              // a multiple of 64
    int32_t cells_per_seg;      // of the other map
    const uint32_t* row_bound;  // of the slots, [batch][bound_pitch]
    int64_t bound_pitch;
    const SegInfo* seg;         // of the other map, [batch][n_segs]
    int32_t n_segs;
};
struct SelectArgs {
    SelectSide side[2];     // blockIdx.z
    DenseJudge judge;
};
__global__ __launch_bounds__(SELECT_WAVES * 64) void dense_select_kernel(SelectArgs args) {
    const SelectSide a = blockIdx.z ? args.side[1] : args.side[0];  // (an index would hide from the compiler that the pointers are global)
    if (args.judge.alike(blockIdx.y)) return;
    if ((int64_t)blockIdx.x * (64 * SELECT_SLOTS) >= a.pitch) return;  // uniform: the sides differ in size
    __shared__ float low[SELECT_WAVES][SELECT_SLOTS][64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int b = blockIdx.y;
    const int64_t slot0 = (int64_t)blockIdx.x * (64 * SELECT_SLOTS);  // whole 64s past the pitch do not exist
    const uint16_t* column = a.best + (int64_t)b * a.n_cells * a.pitch + slot0 + lane;
    uint64_t* mask = a.mask + ((int64_t)b * a.n_cells * a.pitch + slot0) / 64;
    const SegInfo* seg = a.seg + (int64_t)b * a.n_segs;
    bool here[SELECT_SLOTS];
    float length[SELECT_SLOTS], residual[SELECT_SLOTS], best[SELECT_SLOTS];
#pragma unroll
    for (int e = 0; e < SELECT_SLOTS; ++e) {
        here[e] = slot0 + 64 * e < a.pitch;  // uniform
        const uint32_t bound = here[e] ? a.row_bound[(int64_t)b * a.bound_pitch + slot0 + 64 * e + lane] : 0;
        length[e] = __uint_as_float(bound & 0xFFFF0000u);
        residual[e] = __uint_as_float(bound << 16);
        best[e] = -__builtin_inff();
    }
    // visit(cell, slot, 8-bit score, its segment) for this wave's cells
    auto sweep = [&](auto visit) {
        for (int cell0 = wave; cell0 < a.n_cells; cell0 += SELECT_WAVES * SELECT_DEEP) {
            int kept[SELECT_DEEP][SELECT_SLOTS];
#pragma unroll
            for (int i = 0; i < SELECT_DEEP; ++i)
#pragma unroll
                for (int e = 0; e < SELECT_SLOTS; ++e)
                    kept[i][e] = (int16_t)column[(int64_t)min(cell0 + i * SELECT_WAVES, a.n_cells - 1) * a.pitch + (here[e] ? 64 * e : 0)];
#pragma unroll
            for (int i = 0; i < SELECT_DEEP; ++i) {
                const int cell = cell0 + i * SELECT_WAVES;
                if (cell < a.n_cells) {  // uniform
                    const SegInfo si = seg[cell / a.cells_per_seg];
#pragma unroll
                    for (int e = 0; e < SELECT_SLOTS; ++e) visit(cell, e, kept[i][e], si);
                }
            }
        }
    };
    auto error = [&](int e, const SegInfo& si) { return __builtin_fmaf(length[e], si.residual, residual[e] * si.length); };
    sweep([&](int, int e, int v, const SegInfo& si) {
        best[e] = __builtin_fmaxf(best[e], (float)(v * (1 << KEPT_SHIFT)) * si.scale - error(e, si));
    });
#pragma unroll
    for (int e = 0; e < SELECT_SLOTS; ++e) low[wave][e][lane] = best[e];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < SELECT_SLOTS; ++e)
#pragma unroll
        for (int w = 0; w < SELECT_WAVES; ++w) best[e] = __builtin_fmaxf(best[e], low[w][e][lane]);
    sweep([&](int cell, int e, int v, const SegInfo& si) {
        const uint64_t need = __ballot((float)((v + 1) * (1 << KEPT_SHIFT)) * si.scale + error(e, si) >= best[e]);
        if (lane == 0 && here[e]) mask[(int64_t)cell * (a.pitch / 64) + e] = need;
    });
}

// Whether the 8-bit scores of a pair tell enough apart.  How many cells the bounds leave over is a matter of what the maps hold (a
// textureless wall, descriptors of few dimensions or of very different lengths leave most of them), so DENSE_SAMPLES pixels of
// either image, spread over it, are scored against every cell of the other first: what they need is counted, and the launches of
// the two steps, or else those of the one-step sweep, leave the pair alone.  One 512x384 pair, fp16, 24 channels, the whole call in one
// step / in two without this / with it (17 us for pairs that keep two steps): features of 1 pixel 2.16 / 1.69 / 1.71 ms, of 64 2.05 / 2.26 / 1.89
// (short ranges, see launch_refine_t), rank 6 2.13 / 2.82 / 2.17, rank 4 2.12 / 4.60 / 2.15, lengths spread by exp(N(0, 1)) 2.20 / 3.58 / 2.23,
// one descriptor throughout 1.93 / 4.32 / 1.95.
constexpr int SAMPLE_BLOCKS = DENSE_SAMPLES / 32;
constexpr int SAMPLE_WAVES = 8;
constexpr int SAMPLE_TILES = 8;  // in flight per wave
__device__ __forceinline__ int64_t sample_pixel(int k, int64_t n) { return (int64_t)(((uint64_t)((uint32_t)k * 0x9E3779B1u) * (uint64_t)n) >> 32); }
__device__ __forceinline__ int sample_cells(const DenseCoarseArgs& a, int side) { return side == 0 ? a.n_cells : a.map[0].n_segs; }
// A workgroup scores the samples of one image against one cell of the other.  Bound by the latency of its loads.
__global__ __launch_bounds__(SAMPLE_WAVES * 64) void dense_sample_kernel(DenseCoarseArgs a) {
    __shared__ int best[DENSE_SAMPLES];
    const int lane = threadIdx.x & 63, c = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int cell = blockIdx.x, side = blockIdx.y, b = blockIdx.z;
    if (cell >= sample_cells(a, side)) return;
    const CoarseMap& own = a.map[side];
    const CoarseMap& other = a.map[side ^ 1];
    const int64_t own_row0 = (int64_t)b * own.n_segs * a.seg_pixels;
    const int cell_pixels = side == 0 ? 512 * a.cell_groups : a.seg_pixels;  // 1024 to 4096
    const char* tiles = other.rows + ((int64_t)b * other.n_segs * a.seg_pixels + (int64_t)cell * cell_pixels) * COARSE_ROW_BYTES;
    const int64_t mine = sample_pixel(threadIdx.x & (DENSE_SAMPLES - 1), a.pixels[side]);
    const uint32_t bound = own.row_bound[own_row0 + mine];
    const SegInfo si = other.seg[(int64_t)b * other.n_segs + (int64_t)cell * cell_pixels / a.seg_pixels];
    if (threadIdx.x < DENSE_SAMPLES) best[threadIdx.x] = LOWEST;
    i32x4 q[SAMPLE_BLOCKS];
#pragma unroll
    for (int k = 0; k < SAMPLE_BLOCKS; ++k)
        q[k] = *reinterpret_cast<const i32x4*>(own.rows + (own_row0 + sample_pixel(k * 32 + c, a.pixels[side])) * COARSE_ROW_BYTES + 16 * h);
    int top[SAMPLE_BLOCKS];
#pragma unroll
    for (int k = 0; k < SAMPLE_BLOCKS; ++k) top[k] = LOWEST;
#pragma unroll 1
    for (int t = wave * SAMPLE_TILES; t < cell_pixels / 32; t += SAMPLE_WAVES * SAMPLE_TILES) {
        i32x4 tile[SAMPLE_TILES];
#pragma unroll
        for (int i = 0; i < SAMPLE_TILES; ++i) tile[i] = *reinterpret_cast<const i32x4*>(tiles + (int64_t)(t + i) * TILE_BYTES + c * COARSE_ROW_BYTES + 16 * h);
#pragma unroll
        for (int i = 0; i < SAMPLE_TILES; ++i)
#pragma unroll
            for (int k = 0; k < SAMPLE_BLOCKS; ++k) top[k] = fold16i(top[k], product8(tile[i], q[k]));
    }
    __syncthreads();
    if (wave * SAMPLE_TILES < cell_pixels / 32) {
#pragma unroll
        for (int k = 0; k < SAMPLE_BLOCKS; ++k) atomicMax(&best[k * 32 + c], top[k]);
    }
    __syncthreads();
    if (threadIdx.x < DENSE_SAMPLES) {
        const int k = threadIdx.x, kept = best[k] >> KEPT_SHIFT;
        const float error = __builtin_fmaf(__uint_as_float(bound & 0xFFFF0000u), si.residual, __uint_as_float(bound << 16) * si.length);
        a.sample_upper[side][((int64_t)b * sample_cells(a, side) + cell) * DENSE_SAMPLES + k] = (float)((kept + 1) * (1 << KEPT_SHIFT)) * si.scale + error;
        atomicMax(&a.sample_lower[(b * 2 + side) * DENSE_SAMPLES + k], order_bits((float)(kept * (1 << KEPT_SHIFT)) * si.scale - error));
    }
}
constexpr int JUDGE_CELLS = 16;  // of a workgroup
__global__ __launch_bounds__(DENSE_SAMPLES) void dense_judge_kernel(DenseCoarseArgs a) {
    const int k = threadIdx.x, side = blockIdx.y, b = blockIdx.z, cells = sample_cells(a, side), first = blockIdx.x * JUDGE_CELLS;
    const float* upper = a.sample_upper[side] + (int64_t)b * cells * DENSE_SAMPLES + k;
    const float lower = unorder_bits(a.sample_lower[(b * 2 + side) * DENSE_SAMPLES + k]);
    float up[JUDGE_CELLS];
#pragma unroll
    for (int i = 0; i < JUDGE_CELLS; ++i) up[i] = upper[(int64_t)min(first + i, cells - 1) * DENSE_SAMPLES];
    int marks = 0;
#pragma unroll
    for (int i = 0; i < JUDGE_CELLS; ++i)
        if (first + i < cells) marks += __popcll(__ballot(up[i] >= lower));  // uniform
    if ((threadIdx.x & 63) == 0 && marks) atomicAdd(&a.marked[b * 2 + side], marks);
}

// Wider cells keep the table of a large map small, narrower ones leave less to multiply again.  Segments of 2048 pixels and cells of 1024 against 4096 and
// 4096, one pair of such maps, the whole call in ms: 196608 pixels 1.75 / 1.91, 262144 2.86 / 2.91, 294912 3.71 / 3.76, 307200 4.16 / 4.06,
// 371712 6.10 / 5.88, 442368 8.43 / 8.16, 786432 26.4 / 24.9.
constexpr int64_t DENSE_WIDE_PIXELS = 300000;
int dense_seg_pixels(int64_t n) { return n > DENSE_WIDE_PIXELS ? 4096 : 2048; }
int dense_cell_groups(int64_t n, int64_t m) { return m > DENSE_WIDE_PIXELS ? dense_seg_pixels(n) / 512 : 2; }  // a cell lies in one segment
// What a block of 32x32 scores takes one SIMD in the dense kernels, in dense_coarse_kernel, and in the second step
static double dense_exact(int compute, int dp) { return compute == FNN_F32 ? 15.8 * dp : (dp <= 32 ? 2.33 * dp : 1.83 * dp); }
constexpr double DENSE_COARSE = 38.0;
static double dense_second(int compute, int dp) { return compute == FNN_F32 ? 18.75 * dp : (dp <= 32 ? 46.0 : 1.64 * dp); }
// ... there with its lists and what their uneven lengths leave idle: one 512x384 pair of 16-bit rows loses from a share of about 0.26 on
// (0.24 0.97 of the one step's time, 0.25 0.99), 384x288 in fp32 is at 0.87 with 0.61
double dense_coarse_limit(int compute, int dp) {
    return 0.85 * (dense_exact(compute, dp) - DENSE_COARSE) / (compute != FNN_F32 && dp <= 32 ? 58.0 : dense_second(compute, dp));
}
double dense_coarse_gain(int64_t n, int64_t m, int batch, int compute, int dp, int d, bool l2) {
    if (n < 16384 || m < 16384 || (compute != FNN_F32 && dp <= 16)) return -1e30;
    if ((double)m * (n / dense_seg_pixels(n)) * 2.0 > 4e9) return -1e30;  // the candidates' table of a pair would be too large
    const double cell = 512.0 * dense_cell_groups(n, m), row_bytes = dp * elem_size(compute);
    const double cells[2] = {m / cell, (double)n / dense_seg_pixels(n)};
    const double again = coarse_cells_again(cells[0], d, l2) / cells[0] + coarse_cells_again(cells[1], d, l2) / cells[1];
    const double blocks = (double)batch * ((n + 31) / 32) * ((m + 31) / 32) / 1024.0;
    const double bytes = batch * ((double)(n + m) * (2.0 * row_bytes + 40.0) + 8.0 * n * (m / cell) + 8.0 * m * ((double)n / dense_seg_pixels(n)));
    return blocks * (dense_exact(compute, dp) - DENSE_COARSE - dense_second(compute, dp) * again) - 45000.0 - bytes / 4500.0 - batch * (double)(n + m) * 0.1;
}

hipError_t launch_dense_sample(const DenseCoarseArgs& a, int batch, hipStream_t s) {
    const int cells = a.n_cells > a.map[0].n_segs ? a.n_cells : a.map[0].n_segs;
    const hipError_t e = launch(TK_DENSE_SAMPLE, dense_sample_kernel, dim3(cells, 2, batch), dim3(SAMPLE_WAVES * 64), 0, s, a);
    if (e != hipSuccess) return e;
    return launch(TK_DENSE_SAMPLE, dense_judge_kernel, dim3((cells + JUDGE_CELLS - 1) / JUDGE_CELLS, 2, batch), dim3(DENSE_SAMPLES), 0, s, a);
}
hipError_t launch_dense_coarse(DenseCoarseArgs a, int batch, hipStream_t s) {
    // six workgroups for every resident one (three per compute unit), so that the last ones leave little of the chip idle
    a.cells_per_wg = 1;
    const int64_t cells = (int64_t)a.n_cells * a.n_sb * batch;
    while (a.cells_per_wg < 4 && cells / (a.cells_per_wg * 2) >= 4608) a.cells_per_wg *= 2;
    const dim3 grid((a.n_cells + a.cells_per_wg - 1) / a.cells_per_wg, a.n_sb, batch);
    if (a.seg_pixels == 2048) return launch_detail(TK_DENSE, 2, dense_coarse_kernel<2048>, grid, dim3(COARSE_WAVES * 64), 0, s, a);
    return launch_detail(TK_DENSE, 2, dense_coarse_kernel<4096>, grid, dim3(COARSE_WAVES * 64), 0, s, a);
}

static SelectSide select_side(const DenseCoarseArgs& a, int side) {
    SelectSide sa;
    const CoarseMap& own = a.map[side];
    const CoarseMap& other = a.map[side ^ 1];
    sa.best = a.best[side];
    sa.mask = a.mask[side];
    sa.n_cells = side == 0 ? a.n_cells : a.map[0].n_segs;
    sa.pitch = side == 0 ? (int64_t)a.n_sb * DENSE_SB_PIXELS : (int64_t)own.n_segs * a.seg_pixels;
    sa.cells_per_seg = side == 0 ? a.seg_pixels / (512 * a.cell_groups) : 1;
    sa.row_bound = own.row_bound + (side == 0 ? (int64_t)a.first_sb * DENSE_SB_PIXELS : 0);
    sa.bound_pitch = (int64_t)own.n_segs * a.seg_pixels;
    sa.seg = other.seg;
    sa.n_segs = other.n_segs;
    return sa;
}
hipError_t launch_dense_select(const DenseCoarseArgs& a, int first_side, int sides, int batch, hipStream_t s) {
    SelectArgs args;
    args.judge = a.judge;
    int64_t pitch = 0;
    for (int i = 0; i < sides; ++i) {
        args.side[i] = select_side(a, first_side + i);
        if (args.side[i].pitch > pitch) pitch = args.side[i].pitch;
    }
    if (sides == 1) args.side[1] = args.side[0];
    const int64_t per_wg = 64 * SELECT_SLOTS;
    return launch(TK_DENSE_SELECT, dense_select_kernel, dim3((unsigned)((pitch + per_wg - 1) / per_wg), batch, sides), dim3(SELECT_WAVES * 64), 0, s, args);
}

}  // namespace fnn
