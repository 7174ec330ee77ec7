// Pass 1 of the dense mode in 8-bit integers: the same sweep as dense_kernel -- every 32x32 block of scores formed once and
// folded into the best candidate of its queries and the best query of its candidates -- with one matrix
// instruction per block, nothing located and nothing masked (rows past a map repeat its last one).  What is kept are the
// maxima per query and cell of candidates, and per candidate, or GROUP of three candidates, and cell of queries; bounds on what the 8 bits left out say
// which cells the second step of the searches (coarse.hip) has to multiply again, in both directions.
//
// Why groups.  The sweep is bound by its vector maxima.  A maximum of every candidate and one of every query take 16 three-input maxima per block; with
// the maxima of three candidates formed first (5, and one candidate is left over), six values go on into the queries' maximum (3) and six into the
// candidates' (3): 11.  A group's maximum bounds each of its candidates from above, but says of none of them how good its best is at
// least.  That comes from the products themselves: the GROUP_TOP cells with the group's largest bounds are multiplied first, and what a
// candidate scored there rules out cells in a second round (of 192 cells, 1 to 5 are left; with bounds of its own a candidate needs 2 to 3.3 in all).
#include <type_traits>

#include "coarse_device.hpp"
#include "dense_perm.hpp"
#include "fnn_kernels.hpp"
#include "trace.hpp"

namespace fnn {

constexpr int CELL_TILES = DENSE_CELL_PIXELS / 32;
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

// The 16 scores of a lane's candidates become six groups: registers 3k, 3k+1, 3k+2, and the last one alone.  Of the DENSE_CELL_PIXELS candidates
// that a workgroup holds, the 320 triples lie side by side in the table, and then the 64 single ones.
constexpr int GROUPS = 6;  // of a tile's half
constexpr int CELL_TRIPLES = CELL_TILES * 2 * (GROUPS - 1);
static_assert(CELL_TRIPLES + CELL_TILES * 2 == DENSE_CELL_GROUPS && CELL_TRIPLES % 64 == 0, "groups are taken 64 at a time");
__device__ __forceinline__ void group_maxima(const i32x16& x, int (&g)[GROUPS]) {
#pragma unroll
    for (int k = 0; k < GROUPS - 1; ++k) g[k] = max3i(x[3 * k], x[3 * k + 1], x[3 * k + 2]);
    g[GROUPS - 1] = x[15];
}
__device__ __forceinline__ int group_entry(int tile, int h, int k) { return k < GROUPS - 1 ? (tile * 2 + h) * (GROUPS - 1) + k : CELL_TRIPLES + tile * 2 + h; }

// The prepared rows of image 1 of a pair, in the order that the dense kernels sweep: a thread of a two-dimensional grid copies 16 bytes at a time.
__device__ __forceinline__ void dense_permute(const DenseSwept& w, int b) {
    const uint4* from = reinterpret_cast<const uint4*>(w.from + (int64_t)b * w.from_bstride);
    uint4* to = reinterpret_cast<uint4*>(w.to + (int64_t)b * w.n_pad * w.row_bytes);
    const int words = w.row_bytes / 16;
    const int64_t n_threads = (int64_t)gridDim.x * gridDim.y * blockDim.x;
    for (int64_t i = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * blockDim.x + threadIdx.x; i < w.n_pad * words; i += n_threads)
        to[i] = from[slot_pixel(i / words) * words + i % words];
}

// A workgroup sweeps one run of queries past a few cells of candidates.  At the end of every cell of queries the candidates' maxima, or those of
// their groups, are reduced over the lanes and kept.
// Bound by the vector unit: in groups 11 three-input maxima per block, 12.4 instructions in all, 50 cycles beside 32 of the matrix instruction, at the clock that the power
// limit leaves.  A product is followed by the maxima of the one before it, as in coarse_kernel.  One 512x384 pair / a third of 1024x768: a maximum for every candidate
// (16 per block; 35.7 ns per block and SIMD in a bare loop, here 43) 1601 / 7745 us, groups of three 1281 / 6340, with the order of products and maxima 1207 / 6240, with eight
// resident tiles instead of four 1154 / 5950 (31 ns).  Larger groups, in the compiler's order and with four tiles: of five 1212 / 6040, of a whole half tile 1125 / 5785; but of 192
// cells groups of five leave 25 to multiply again, half tiles 60.  Without groups the order of products and maxima and more tiles have no registers and gain nothing.
struct SweepLds {  // (two variables for the stage, see dense_staged_kernel)
    uint4 (&stage0)[COARSE_TURN][64];
    uint4 (&stage1)[COARSE_TURN][64];
    int (&row_best)[DENSE_SB_PIXELS];  // best score of every query in the cell
};
template <int SEGMENT, bool GROUPED>
__device__ __forceinline__ void dense_sweep(const DenseCoarseArgs& a, const SweepLds& lds) {
    constexpr int DC_J = GROUPED ? 8 : 4;          // candidate tiles resident per wave
    constexpr int DC_GROUP = COARSE_WAVES * DC_J;  // tiles of a workgroup
    constexpr int DC_KEPT = GROUPED ? GROUPS : 16; // maxima of a tile that a lane keeps
    constexpr int CELL_GROUPS = CELL_TILES / DC_GROUP;
    static_assert(CELL_GROUPS * DC_GROUP == CELL_TILES, "a cell is whole groups of tiles");
    auto& stage0 = lds.stage0;
    auto& stage1 = lds.stage1;
    auto& row_best = lds.row_best;
    const int lane = threadIdx.x & 63, c = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int cell0 = blockIdx.x * a.cells_per_wg, sb = blockIdx.y, b = blockIdx.z;
    constexpr int COL_CELL = GROUPED ? SEGMENT / 2 : SEGMENT, COL_CELLS = DENSE_SB_PIXELS / COL_CELL, COL_TURNS = DC_TURNS / COL_CELLS;
    static_assert(COL_TURNS % 2 == 0, "a cell starts on stage slot 0");
    const int64_t pixels1 = (int64_t)a.map[0].n_segs * SEGMENT, pixels2 = (int64_t)a.map[1].n_segs * SEGMENT;
    const char* blocks = a.map[0].rows + ((int64_t)b * pixels1 + (int64_t)(a.first_sb + sb) * DENSE_SB_PIXELS) * COARSE_ROW_BYTES;
    const char* tiles = a.map[1].rows + (int64_t)b * pixels2 * COARSE_ROW_BYTES;
    uint16_t* rows = a.best[0] + ((int64_t)b * a.n_cells + cell0) * ((int64_t)a.n_sb * DENSE_SB_PIXELS) + (int64_t)sb * DENSE_SB_PIXELS;
    const int64_t col_pitch = GROUPED ? pixels2 / DENSE_CELL_PIXELS * DENSE_CELL_GROUPS : pixels2;
    uint16_t* cols = a.best[1] + b * (a.map[0].n_segs * pixels2) + (int64_t)(a.first_sb + sb) * COL_CELLS * col_pitch;
    // groups of this workgroup's cells that hold a pixel of image 2 (uniform)
    const int cell_groups = CELL_GROUPS * a.cell_runs, group0 = cell0 * cell_groups;
    const int n_groups = min(a.cells_per_wg * cell_groups, (a.n_tiles[1] + DC_GROUP - 1) / DC_GROUP - group0);
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
        int best[DC_J][DC_KEPT];
#pragma unroll
        for (int j = 0; j < DC_J; ++j) {
            cand[j] = *reinterpret_cast<const i32x4*>(tiles + (int64_t)(tile0 + j) * TILE_BYTES + c * COARSE_ROW_BYTES + 16 * h);
            arrived(cand[j]);
#pragma unroll
            for (int v = 0; v < DC_KEPT; ++v) best[j][v] = LOWEST;
        }
        auto turn = [&](int tt, auto slot_tag) {
            constexpr int SLOT = decltype(slot_tag)::value;
            __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wave's share of the turn is in LDS
            __syncthreads();                     // everyone's is, and everyone has left the other slot
            stage_turn(SLOT ? stage0 : stage1, k + tt + 1);
            int found[DC_STEPS];  // best score of a step's queries (lanes 0..31 its first block, 32..63 its second)
            auto block = [&](int i) { return __builtin_bit_cast(i32x4, SLOT ? stage1[i][lane] : stage0[i][lane]); };
            if constexpr (GROUPED) {
                // product number i: step i / (2 DC_J), tile i / 2 % DC_J, the first or second of the step's blocks
                constexpr int STEP = 2 * DC_J, PRODUCTS = DC_STEPS * STEP;
                i32x4 q[2][2];
                q[0][0] = block(0);
                q[0][1] = block(1);
                i32x16 score[2];
                score[0] = product8(cand[0], q[0][0]);
                int row[2], first[GROUPS];
#pragma unroll
                for (int i = 0; i < PRODUCTS; ++i) {
                    const int s = i / STEP, j = i / 2 % DC_J, e = i & 1, then = i + 1;
                    if (i % STEP == 0) {
                        row[0] = row[1] = LOWEST;
                        if (s + 1 < DC_STEPS) {
                            q[(s + 1) & 1][0] = block(2 * s + 2);
                            q[(s + 1) & 1][1] = block(2 * s + 3);
                        }
                    }
                    if (then < PRODUCTS) score[then & 1] = product8(cand[then / 2 % DC_J], q[then / STEP & 1][then & 1]);
                    __builtin_amdgcn_sched_barrier(0);  // a product, then the maxima of the one before it
                    int group[GROUPS];
                    group_maxima(score[e], group);
                    row[e] = max3i(max3i(row[e], group[0], group[1]), max3i(group[2], group[3], group[4]), group[5]);
                    asm volatile("" : "+v"(row[e]));  // ... which the optimiser would otherwise move to the end of the turn
#pragma unroll
                    for (int v = 0; v < GROUPS; ++v) {
                        if (e == 0) {
                            first[v] = group[v];
                        } else {
                            best[j][v] = max3i(best[j][v], first[v], group[v]);
                            asm volatile("" : "+v"(best[j][v]));
                        }
                    }
                    if (i % STEP == STEP - 1) {
                        const auto sw = __builtin_amdgcn_permlane32_swap((uint32_t)row[0], (uint32_t)row[1], false, false);
                        found[s] = max((int)sw[0], (int)sw[1]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {
#pragma unroll
                for (int s = 0; s < DC_STEPS; ++s) {
                    const i32x4 qa = block(2 * s), qb = block(2 * s + 1);
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
            }
#pragma unroll
            for (int s = 0; s < DC_STEPS; ++s) atomicMax(&row_best[(tt * COARSE_TURN + 2 * s) * 32 + lane], found[s]);
        };
#pragma unroll 1
        for (int cc = 0; cc < COL_CELLS; ++cc) {
#pragma unroll 1
            for (int tt = cc * COL_TURNS; tt < (cc + 1) * COL_TURNS; tt += 2) {
                turn(tt, std::integral_constant<int, 0>{});
                turn(tt + 1, std::integral_constant<int, 1>{});
            }
            int fresh = lane;
            asm volatile("" : "+v"(fresh));  // else what hangs on it is kept over the sweep
            const int held = held_register(fresh), half = fresh >> 5;
#pragma unroll
            for (int r = 0; r < DC_J * DC_KEPT; r += 16) {  // sixteen registers at a time; of groups, across the tiles
                int x[16];
#pragma unroll
                for (int v = 0; v < 16; ++v) x[v] = best[(r + v) / DC_KEPT][(r + v) % DC_KEPT];
                const int top = transpose_max16_int(x, fresh);
                uint16_t* to = cols + cc * col_pitch + (GROUPED ? (int64_t)(group0 + g) * DENSE_CELL_GROUPS : (int64_t)(tile0 + r / 16) * 32);  // uniform
                const uint32_t at = GROUPED ? group_entry(wave * DC_J + (r + held) / GROUPS, half, (r + held) % GROUPS) : tile_row(held, half);
                if ((fresh & 16) == 0) to[at] = (uint16_t)(top >> KEPT_SHIFT);
            }
#pragma unroll
            for (int j = 0; j < DC_J; ++j)
#pragma unroll
                for (int v = 0; v < DC_KEPT; ++v) best[j][v] = LOWEST;
        }
        k += DC_TURNS;
        if ((g + 1) % cell_groups == 0 || g + 1 == n_groups) {  // the end of a cell (uniform)
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
#define FNN_SWEEP_LDS                                                   \
    __shared__ uint4 stage0[COARSE_TURN][64], stage1[COARSE_TURN][64]; \
    __shared__ int row_best[DENSE_SB_PIXELS];                          \
    const SweepLds lds = {stage0, stage1, row_best}
// a maximum for every candidate
template <int SEGMENT>
__global__ __launch_bounds__(COARSE_WAVES * 64) __attribute__((amdgpu_waves_per_eu(3)))
void dense_coarse_kernel(DenseCoarseArgs a) {
    FNN_SWEEP_LDS;
    if (a.judge.way(blockIdx.z) == DENSE_ONE_STEP) {
        if (a.swept.to) dense_permute(a.swept, blockIdx.z);
    } else {
        dense_sweep<SEGMENT, false>(a, lds);
    }
}
// one for every group, or for every candidate: a pair has the way that its samples say
template <int SEGMENT>
__global__ __launch_bounds__(COARSE_WAVES * 64) __attribute__((amdgpu_waves_per_eu(2)))
void dense_groups_kernel(DenseCoarseArgs a) {
    FNN_SWEEP_LDS;
    const DenseWay way = a.judge.way(blockIdx.z);
    if (way == DENSE_ONE_STEP) {
        if (a.swept.to) dense_permute(a.swept, blockIdx.z);
    } else if (way == DENSE_GROUPS) {
        dense_sweep<SEGMENT, true>(a, lds);
    } else {
        dense_sweep<SEGMENT, false>(a, lds);
    }
}
#undef FNN_SWEEP_LDS

// Which cells may hold the best partner of a slot: the bounds that turn 8-bit scores into products (coarse.hip) give every slot a
// lower bound of its best score, and a cell whose upper bound reaches it is marked.  A lane takes SELECT_SLOTS slots,
// 64 apart; the waves of a workgroup share the cells.  Bound by memory; the table is read twice, the second time mostly
// from cache.
constexpr int SELECT_WAVES = 4;
constexpr int SELECT_SLOTS = 4;
constexpr int SELECT_DEEP = 6;  // cells in flight per wave
struct SelectSide {
    const uint16_t* best;       // [n_cells][pitch, or the groups of so many slots] of every pair,
    int64_t best_pitch;         // ... so many entries apart
    uint64_t* mask;             // [n_cells][pitch / 64]
    int64_t mask_pitch;
    int32_t n_cells;            // that hold a pixel
    int64_t pitch;              // slots, a multiple of 1024
    int32_t cells_per_seg;      // of the other map
    const uint32_t* row_bound;  // of the slots, [batch][bound_pitch]
    int64_t bound_pitch;
    const SegInfo* seg;         // of the other map, [batch][n_segs]
    int32_t n_segs;
    // groups of slots
    int32_t grouped;            // of the pairs that are DENSE_GROUPS; their cells are half as large
    int32_t n_group_cells;
    float* least;               // [batch][entries of a cell] the smallest upper bound of the first round's cells
    const u64* keys;            // the second round: [batch][n_keys] what the first left
    int64_t n_keys;
    const SegInfo* own_seg;     // of the slots, [batch][own_n_segs]
    int32_t own_n_segs;
    int32_t own_seg_pixels;
};
struct SelectArgs {
    SelectSide side[2];     // blockIdx.z
    DenseJudge judge;
};
// visit(cell, 8-bit scores of N entries of a lane, 64 apart, their segment) for this wave's cells
template <int N, int DEEP, typename F>
__device__ __forceinline__ void for_cells(int n_cells, int cells_per_seg, const uint16_t* column, int64_t row_entries, const SegInfo* seg, int wave, const F& visit) {
    for (int cell0 = wave; cell0 < n_cells; cell0 += SELECT_WAVES * DEEP) {
        int kept[DEEP][N];
#pragma unroll
        for (int i = 0; i < DEEP; ++i)
#pragma unroll
            for (int e = 0; e < N; ++e) kept[i][e] = (int16_t)column[(int64_t)min(cell0 + i * SELECT_WAVES, n_cells - 1) * row_entries + 64 * e];
#pragma unroll
        for (int i = 0; i < DEEP; ++i) {
            const int cell = cell0 + i * SELECT_WAVES;
            if (cell < n_cells) visit(cell, kept[i], seg[cell / cells_per_seg]);  // uniform
        }
    }
}
__device__ __forceinline__ float bound_error(uint32_t bound, const SegInfo& si) {
    return __builtin_fmaf(__uint_as_float(bound & 0xFFFF0000u), si.residual, __uint_as_float(bound << 16) * si.length);
}
__device__ __forceinline__ uint32_t worst_bound(uint32_t a, uint32_t b) {  // lengths and remainders are not negative: they order like integers
    return max(a & 0xFFFF0000u, b & 0xFFFF0000u) | max(a & 0xFFFFu, b & 0xFFFFu);
}
__device__ __forceinline__ float upper_score(int kept, const SegInfo& si, float error) {
    return __builtin_fmaf((float)((kept + 1) * (1 << KEPT_SHIFT)), si.scale, error);  // the same wherever it is formed: two rounds share the cells by it
}

__device__ __forceinline__ void select_slots(const SelectSide& a, int b, float (&low)[SELECT_WAVES][SELECT_SLOTS][64]) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t slot0 = (int64_t)blockIdx.x * (64 * SELECT_SLOTS);
    const uint16_t* column = a.best + b * a.best_pitch + slot0 + lane;
    uint64_t* mask = a.mask + b * a.mask_pitch + slot0 / 64;
    const SegInfo* seg = a.seg + (int64_t)b * a.n_segs;
    uint32_t bound[SELECT_SLOTS];
    float best[SELECT_SLOTS];
#pragma unroll
    for (int e = 0; e < SELECT_SLOTS; ++e) {
        bound[e] = a.row_bound[(int64_t)b * a.bound_pitch + slot0 + 64 * e + lane];
        best[e] = -__builtin_inff();
    }
    for_cells<SELECT_SLOTS, SELECT_DEEP>(a.n_cells, a.cells_per_seg, column, a.pitch, seg, wave, [&](int, const int (&v)[SELECT_SLOTS], const SegInfo& si) {
#pragma unroll
        for (int e = 0; e < SELECT_SLOTS; ++e) best[e] = __builtin_fmaxf(best[e], (float)(v[e] * (1 << KEPT_SHIFT)) * si.scale - bound_error(bound[e], si));
    });
#pragma unroll
    for (int e = 0; e < SELECT_SLOTS; ++e) low[wave][e][lane] = best[e];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < SELECT_SLOTS; ++e)
#pragma unroll
        for (int w = 0; w < SELECT_WAVES; ++w) best[e] = __builtin_fmaxf(best[e], low[w][e][lane]);
    for_cells<SELECT_SLOTS, SELECT_DEEP>(a.n_cells, a.cells_per_seg, column, a.pitch, seg, wave, [&](int cell, const int (&v)[SELECT_SLOTS], const SegInfo& si) {
        uint64_t mine = 0;  // a cell's words are written side by side
#pragma unroll
        for (int e = 0; e < SELECT_SLOTS; ++e) {
            const uint64_t need = __ballot(upper_score(v[e], si, bound_error(bound[e], si)) >= best[e]);
            mine = lane == e ? need : mine;
        }
        if (lane < SELECT_SLOTS) mask[(int64_t)cell * (a.pitch / 64) + lane] = mine;
    });
}

// The same for groups of slots.  The first round marks the GROUP_TOP cells with a group's largest upper bounds; the second, when those have been multiplied, the
// others whose upper bound reaches a slot's best product.  A lane takes a group of each of SELECT_SETS runs of 64; the bits of a cell
// are in the order of mask_candidate: three words for 64 triples, one for 64 single slots.  (512x384 / 1024x768, the two rounds: a lane for every slot, three of which read the same
// entry, 83 + 76 / 282 + 516 us; so, but with the first round's cells looked up in its words instead of by their bounds, 75 + 86 / 218 + 421.)
constexpr int SELECT_SETS = 2, SELECT_SETS_DEEP = 8;
constexpr int TRIPLE_SETS = CELL_TRIPLES / 64;
constexpr int SELECT_PARTS = DENSE_CELL_GROUPS / (64 * SELECT_SETS);  // workgroups for a run of DENSE_CELL_PIXELS slots
static_assert(SELECT_PARTS * 64 * SELECT_SETS == DENSE_CELL_GROUPS, "whole runs of 64");
constexpr int GROUP_TOP = 6, GROUP_TOP_FEW = 3, FEW_CELLS = 32;       // (of a small map's few cells, fewer)
__device__ __forceinline__ void select_groups(const SelectSide& a, int b, float (&handed)[SELECT_WAVES][SELECT_SETS][GROUP_TOP][64]) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int run = blockIdx.x / SELECT_PARTS, set0 = blockIdx.x % SELECT_PARTS * SELECT_SETS;  // of the run's sets of 64 groups
    const int64_t slot0 = (int64_t)run * DENSE_CELL_PIXELS, row_entries = a.pitch / DENSE_CELL_PIXELS * DENSE_CELL_GROUPS;
    const uint16_t* column = a.best + b * a.best_pitch + (int64_t)run * DENSE_CELL_GROUPS + 64 * set0 + lane;
    uint64_t* mask = a.mask + b * a.mask_pitch + slot0 / 64 + 3 * set0;
    float* least_of = a.least + (int64_t)b * row_entries + (int64_t)run * DENSE_CELL_GROUPS + 64 * set0 + lane;
    const SegInfo* seg = a.seg + (int64_t)b * a.n_segs;
    int64_t slot[SELECT_SETS][3];
    uint32_t bound[SELECT_SETS];  // the group's worst length and remainder
#pragma unroll
    for (int e = 0; e < SELECT_SETS; ++e) {
        bound[e] = 0;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const bool single = set0 + e == TRIPLE_SETS;  // uniform
            slot[e][k] = slot0 + mask_candidate((3 * (set0 + e) + (single ? 0 : k)) * 64 + lane);
            const uint32_t own = a.row_bound[(int64_t)b * a.bound_pitch + slot[e][k]];
            bound[e] = worst_bound(bound[e], own);
        }
    }
    const bool last_single = set0 + SELECT_SETS == TRIPLE_SETS + 1;  // uniform: the last of the sets is the single slots
    // a cell's words, side by side; marked(e, k): whether slot k of this lane's group of set e is
    auto write = [&](int cell, auto marked) {
        uint64_t mine = 0;
#pragma unroll
        for (int e = 0; e < SELECT_SETS; ++e)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const uint64_t need = __ballot(marked(e, k));
                mine = lane == 3 * e + k ? need : mine;
            }
        if (lane < (last_single ? 3 * SELECT_SETS - 2 : 3 * SELECT_SETS)) mask[(int64_t)cell * (a.pitch / 64) + lane] = mine;
    };
    if (a.keys) {
        // Products are compared with bounds times the scale of the slots' segment; a group with a row that has no bounds, or of a segment of zeros, needs every cell, and so do
        // all slots a cell with such a row (a product of infinity is reached by no bound, but others may equal it).
        const float scale = a.own_seg[(int64_t)b * a.own_n_segs + slot0 / a.own_seg_pixels].scale;
        float product[SELECT_SETS][3], least[SELECT_SETS];
        bool every[SELECT_SETS];
#pragma unroll
        for (int e = 0; e < SELECT_SETS; ++e) {
            least[e] = least_of[64 * e];
            every[e] = !(scale > 0.0f) || __uint_as_float(bound[e] & 0xFFFF0000u) >= 0.5f * UNBOUNDED;
#pragma unroll
            for (int k = 0; k < 3; ++k) product[e][k] = slot[e][k] < a.n_keys ? key_score(a.keys[(int64_t)b * a.n_keys + slot[e][k]]) : 0.0f;
        }
        for_cells<SELECT_SETS, SELECT_SETS_DEEP>(a.n_group_cells, 2, column, row_entries, seg, wave, [&](int cell, const int (&v)[SELECT_SETS], const SegInfo& si) {
            float upper[SELECT_SETS];
            bool all[SELECT_SETS], left[SELECT_SETS];
#pragma unroll
            for (int e = 0; e < SELECT_SETS; ++e) {
                upper[e] = upper_score(v[e], si, bound_error(bound[e], si));
                left[e] = upper[e] < least[e];  // not one of the first round's
                all[e] = every[e] || si.residual >= 0.5f * UNBOUNDED;
            }
            write(cell, [&](int e, int k) { return slot[e][k] < a.n_keys && left[e] && (all[e] || upper[e] * scale >= product[e][k]); });
        });
        return;
    }
    float most[SELECT_SETS][GROUP_TOP];  // the largest upper bounds, in order
    auto put = [](float (&t)[GROUP_TOP], float x) {
#pragma unroll
        for (int i = GROUP_TOP - 1; i > 0; --i) t[i] = __builtin_amdgcn_fmed3f(x, t[i - 1], t[i]);
        t[0] = __builtin_fmaxf(t[0], x);
    };
#pragma unroll
    for (int e = 0; e < SELECT_SETS; ++e)
#pragma unroll
        for (int i = 0; i < GROUP_TOP; ++i) most[e][i] = -__builtin_inff();
    for_cells<SELECT_SETS, SELECT_SETS_DEEP>(a.n_group_cells, 2, column, row_entries, seg, wave, [&](int, const int (&v)[SELECT_SETS], const SegInfo& si) {
#pragma unroll
        for (int e = 0; e < SELECT_SETS; ++e) put(most[e], upper_score(v[e], si, bound_error(bound[e], si)));
    });
#pragma unroll
    for (int e = 0; e < SELECT_SETS; ++e)
#pragma unroll
        for (int i = 0; i < GROUP_TOP; ++i) handed[wave][e][i][lane] = most[e][i];
    __syncthreads();
    float least[SELECT_SETS];
#pragma unroll
    for (int e = 0; e < SELECT_SETS; ++e) {
#pragma unroll
        for (int w = 1; w < SELECT_WAVES; ++w)
#pragma unroll
            for (int i = 0; i < GROUP_TOP; ++i) put(most[e], handed[(wave + w) % SELECT_WAVES][e][i][lane]);
        least[e] = a.n_group_cells < FEW_CELLS ? most[e][GROUP_TOP_FEW - 1] : most[e][GROUP_TOP - 1];
        if (wave == 0) least_of[64 * e] = least[e];
    }
    for_cells<SELECT_SETS, SELECT_SETS_DEEP>(a.n_group_cells, 2, column, row_entries, seg, wave, [&](int cell, const int (&v)[SELECT_SETS], const SegInfo& si) {
        bool top[SELECT_SETS];
#pragma unroll
        for (int e = 0; e < SELECT_SETS; ++e) top[e] = upper_score(v[e], si, bound_error(bound[e], si)) >= least[e];
        write(cell, [&](int e, int k) { return top[e] && slot[e][k] < a.n_keys; });
    });
}
__global__ __launch_bounds__(SELECT_WAVES * 64) void dense_select_kernel(SelectArgs args) {
    const SelectSide a = blockIdx.z ? args.side[1] : args.side[0];  // (an index would hide from the compiler that the pointers are global)
    const DenseWay way = args.judge.way(blockIdx.y);
    if (way == DENSE_ONE_STEP) return;
    __shared__ union {
        float low[SELECT_WAVES][SELECT_SLOTS][64];
        float handed[SELECT_WAVES][SELECT_SETS][GROUP_TOP][64];
    } lds;
    // uniform: the sides differ in size
    if (a.grouped && way == DENSE_GROUPS) {
        if ((int64_t)(blockIdx.x / SELECT_PARTS) * DENSE_CELL_PIXELS < a.pitch) select_groups(a, blockIdx.y, lds.handed);
    } else if (!a.keys && (int64_t)blockIdx.x * (64 * SELECT_SLOTS) < a.pitch) {
        select_slots(a, blockIdx.y, lds.low);
    }
}

// Which way of a pair is the fastest.  How many cells the bounds leave over is a matter of what the maps hold (a textureless wall, descriptors of few
// dimensions or of very different lengths leave most of them), so DENSE_SAMPLES pixels of either image, spread over it, are scored against every
// cell of the other first, what they need is counted (dense_costs), and every launch takes the pairs that are its own.  A group's bound is that of its longest row,
// which reaches past the best of the others where lengths differ; what the samples' groups mark says so.  Whole calls in us, fp16, 24 channels, in one step / with a maximum for every
// candidate / for three; as the samples say is within 2 % of the fastest.  One 512x384 pair: features of 1 pixel 2192 / 1709 / 1543, of 64 2097 / 1888 / 1784, of 128 2080 / 2078 / 2046; rank 8
// 2195 / 2149 / 1824, rank 7 2189 / 2496 / 2064; lengths spread by exp(0.2 N(0, 1)) 2197 / 1736 / 2259, by exp(0.7 N(0, 1)) 2234 / 2665 / 2803.  Four of 192x144: features of 4 pixels 391 /
// 301 / 302, of 128 386 / 333 / 351, rank 7 392 / 366 / 353, lengths spread by exp(0.2 N(0, 1)) 394 / 292 / 342.
// A pair that is left to one step pays 25 to 40 us for its 8-bit maps, the samples and the launches that leave it alone: rank 6, four of 192x144 368 / 394 without / with them, one of 352x256 547 /
// 577, of 512x384 2148 / 2191.
constexpr int SAMPLE_BLOCKS = DENSE_SAMPLES / 32;
constexpr int SAMPLE_WAVES = 8;
constexpr int SAMPLE_TILES = 8;  // in flight per wave
__device__ __forceinline__ int64_t spread_pixel(int k, int64_t n) { return (int64_t)(((uint64_t)((uint32_t)k * 0x9E3779B1u) * (uint64_t)n) >> 32); }
// Where groups are possible, whole groups.
constexpr int SAMPLE_GROUP = 3;
__device__ __forceinline__ int64_t sample_pixel(int k, int64_t n, bool grouped) {
    if (!grouped) return spread_pixel(k, n);
    const int g = k / SAMPLE_GROUP;
    const int64_t at = (spread_pixel(g, n) & ~(int64_t)31) + tile_row(SAMPLE_GROUP * (g / 2 % (GROUPS - 1)) + k % SAMPLE_GROUP, g & 1);
    return at < n ? at : n - 1;
}
__device__ __forceinline__ int sample_cells(const DenseCoarseArgs& a, int side) { return side == 0 ? a.n_cells : a.n_col_cells; }
// A workgroup scores the samples of one image against one cell of the other.  Bound by the latency of its loads.
__global__ __launch_bounds__(SAMPLE_WAVES * 64) void dense_sample_kernel(DenseCoarseArgs a) {
    __shared__ int best[DENSE_SAMPLES];
    __shared__ uint32_t bounds[DENSE_SAMPLES];
    const int lane = threadIdx.x & 63, c = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int cell = blockIdx.x, side = blockIdx.y, b = blockIdx.z;
    if (cell >= sample_cells(a, side)) return;
    const CoarseMap& own = a.map[side];
    const CoarseMap& other = a.map[side ^ 1];
    const int64_t own_row0 = (int64_t)b * own.n_segs * a.seg_pixels;
    const bool grouped = side == 1 && a.grouped;
    const int cell_pixels = side == 0 ? DENSE_CELL_PIXELS * a.cell_runs : a.seg_pixels >> a.grouped;  // 1024 to 4096
    const char* tiles = other.rows + ((int64_t)b * other.n_segs * a.seg_pixels + (int64_t)cell * cell_pixels) * COARSE_ROW_BYTES;
    const int64_t mine = sample_pixel(threadIdx.x & (DENSE_SAMPLES - 1), a.pixels[side], grouped);
    const uint32_t bound = own.row_bound[own_row0 + mine];
    const SegInfo si = other.seg[(int64_t)b * other.n_segs + (int64_t)cell * cell_pixels / a.seg_pixels];
    if (threadIdx.x < DENSE_SAMPLES) {
        best[threadIdx.x] = LOWEST;
        bounds[threadIdx.x] = bound;
    }
    i32x4 q[SAMPLE_BLOCKS];
#pragma unroll
    for (int k = 0; k < SAMPLE_BLOCKS; ++k)
        q[k] = *reinterpret_cast<const i32x4*>(own.rows + (own_row0 + sample_pixel(k * 32 + c, a.pixels[side], grouped)) * COARSE_ROW_BYTES + 16 * h);
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
        const int64_t at = ((int64_t)b * sample_cells(a, side) + cell) * DENSE_SAMPLES + k;
        const float score = (float)(kept * (1 << KEPT_SHIFT)) * si.scale, error = bound_error(bound, si);
        a.sample_upper[side][at] = upper_score(kept, si, error);
        atomicMax(&a.sample_lower[(b * 2 + side) * DENSE_SAMPLES + k], order_bits(score - error));
        if (grouped) {  // a group's maximum stands for each of its candidates, with the group's worst length and remainder
            const int first = k / SAMPLE_GROUP * SAMPLE_GROUP;
            int top = kept;
            uint32_t worst = bound;
            for (int i = first; i < first + SAMPLE_GROUP && i < DENSE_SAMPLES; ++i) {
                top = max(top, best[i] >> KEPT_SHIFT);
                worst = worst_bound(worst, bounds[i]);
            }
            a.sample_group[at] = upper_score(top, si, bound_error(worst, si));
            atomicMax(&a.sample_best[b * DENSE_SAMPLES + k], order_bits(score));
        }
    }
}
constexpr int JUDGE_CELLS = 16;  // of a workgroup
static_assert(JUDGE_CELLS % 2 == 0, "both halves of a segment");
// The last workgroup to file its marks decides.
__global__ __launch_bounds__(DENSE_SAMPLES) void dense_judge_kernel(DenseCoarseArgs a, DenseCosts costs) {
    __shared__ int32_t all[DENSE_MARKS];
    __shared__ uint32_t filed;
    const int k = threadIdx.x, side = blockIdx.y, b = blockIdx.z, cells = sample_cells(a, side), first = blockIdx.x * JUDGE_CELLS;
    const bool grouped = side == 1 && a.grouped;
    auto take = [&](const float* table, float (&up)[JUDGE_CELLS]) {
#pragma unroll
        for (int i = 0; i < JUDGE_CELLS; ++i) up[i] = table[((int64_t)b * cells + min(first + i, cells - 1)) * DENSE_SAMPLES + k];
    };
    const float lower = unorder_bits(a.sample_lower[(b * 2 + side) * DENSE_SAMPLES + k]);
    float up[JUDGE_CELLS];
    take(a.sample_upper[side], up);
    const bool speaks = (k & 63) == 0;
    int marks = 0;
#pragma unroll
    for (int i = 0; i < JUDGE_CELLS; ++i) {
        // where cells are half segments, those of single candidates are two of them (cells past the last repeat it)
        if (grouped && i % 2) continue;
        const float most = grouped ? __builtin_fmaxf(up[i], up[i + 1 - i % 2]) : up[i];
        if (first + i < cells) marks += __popcll(__ballot(most >= lower));  // uniform
    }
    auto file = [&](int what, int count) {
        if (speaks && count) atomicAdd(&a.marked[DENSE_RECORD * b + what], count);
    };
    file(side == 0 ? MARKS_ROWS : MARKS_SINGLES, marks);
    if (grouped) {
        // What the second round of a group's cells is about: its bound against each candidate's best product, for which the 8-bit score stands here.
        const float best = unorder_bits(a.sample_best[b * DENSE_SAMPLES + k]);
        take(a.sample_group, up);
        marks = 0;
#pragma unroll
        for (int i = 0; i < JUDGE_CELLS; ++i)
            if (first + i < cells) marks += __popcll(__ballot(up[i] >= best));  // uniform
        file(MARKS_GROUPS, marks);
    }
    if (k < DENSE_MARKS) all[k] = 0;
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wave's marks have arrived
    __syncthreads();                     // everyone's have: the marks come before the count, and the counts of all before what the last one reads
    if (k == 0) filed = __hip_atomic_fetch_add(a.filed, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (filed + 1 != gridDim.x * gridDim.y * gridDim.z) return;  // uniform
    static_assert(FNN_MAX_BATCH <= DENSE_SAMPLES, "a thread for every pair");
    const bool here = k < (int)gridDim.z;
    int32_t own[DENSE_MARKS], sum[DENSE_MARKS];
#pragma unroll
    for (int w = 0; w < DENSE_MARKS; ++w) {
        own[w] = here ? __hip_atomic_load(&a.marked[DENSE_RECORD * k + w], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
        if (here) atomicAdd(&all[w], own[w]);
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < DENSE_MARKS; ++w) sum[w] = all[w];
    if (here) a.marked[DENSE_RECORD * k + PAIR_WAY] = costs.way(own, sum);
}

// Wider cells keep the table of a large map small, narrower ones leave less to multiply again.  Segments of 2048 pixels and cells of 1024 against 4096 and
// 4096, one pair of such maps, the whole call in ms: 196608 pixels 1.75 / 1.91, 262144 2.86 / 2.91, 294912 3.71 / 3.76, 307200 4.16 / 4.06,
// 371712 6.10 / 5.88, 442368 8.43 / 8.16, 786432 26.4 / 24.9.
constexpr int64_t DENSE_WIDE_PIXELS = 300000;
int dense_seg_pixels(int64_t n) { return n > DENSE_WIDE_PIXELS ? 4096 : 2048; }
int dense_cell_runs(int64_t n, int64_t m) { return m > DENSE_WIDE_PIXELS ? dense_seg_pixels(n) / DENSE_CELL_PIXELS : 1; }  // a cell lies in one segment
// What a block of 32x32 scores takes one SIMD in the dense kernels, in dense_coarse_kernel, and in the second step
static double dense_exact(int compute, int dp) { return compute == FNN_F32 ? 15.8 * dp : (dp <= 32 ? 2.33 * dp : 1.83 * dp); }
constexpr double DENSE_COARSE = 38.0, DENSE_COARSE_GROUPS = 29.0;
static double dense_second(int compute, int dp) { return compute == FNN_F32 ? 18.75 * dp : (dp <= 32 ? 46.0 : 1.64 * dp); }
// Groups of candidates leave some GROUP_TOP cells more of them to the second step, which is dear where products are (fp32, 24 channels, a maximum for every candidate / groups:
// 320x240 839 / 911 us, four pairs of 256x192 and 320x240 1613 / 1978; two-term rows, 384x288 894 / 865).
static double first_round(double cells) { return cells < FEW_CELLS ? GROUP_TOP_FEW : GROUP_TOP; }
bool dense_grouped(int64_t n, int compute, int dp) {
    const double cells = 2.0 * n / dense_seg_pixels(n);
    return dense_second(compute, dp) * (first_round(cells) + 2.0) < (DENSE_COARSE - DENSE_COARSE_GROUPS) * cells;
}
static double dense_coarse_block(int64_t n, int compute, int dp) { return dense_grouped(n, compute, dp) ? DENSE_COARSE_GROUPS : DENSE_COARSE; }
// The model behind the choice, in nanoseconds.  The one-step kernels leave their staged loop where a workgroup meets padding and have few workgroups to share what that leaves
// uneven: maps of image 1 that are not whole runs of 4096 queries take 1.4 to 1.8 times a whole one's time per block, of which 1.4 are counted on (fp16, 24 channels, ns per block beside 50 us: 28672 / 27648 queries on
// 196608 candidates, four pairs 68 / 97, 61440 / 62208 queries on 61440, four 66 / 85, 122880 / 120000 on 196608 59 / 86).  Candidates that are not whole runs of 512 cost little: 196608 queries on 28672 / 30000, four pairs
// 66 / 65, 61440 on 61440 / 90000 66 / 68, 122880 on 28672 / 45000 65 / 69.  Two steps cost 45 us of launches, more
// on large maps.  Measured in one step / two, 16-bit rows of 24 channels: 256x192 1 pair 236 / 252 us, 2 379 / 355, 4 674 / 564, 16 2341 / 1923; 352x256 564 / 455; not whole:
// 160x120, 16 pairs 738 / 764; 192x144 1 pair 192 / 206, 4 371 / 312, 16 1321 / 829; 224x168 241 / 223, 4 632 / 449, 16 2379 / 1469; 288x216 406 / 324, 4 1819 / 852; 32 channels, 192x144, 8 803 /
// 515; squared distance, 320x240, 2 1233 / 1253, 256x192, 4 770 / 790; fp32, 128x128, 4 494 / 749, 192x144, 4 1409 / 713; two-term rows, 128x128, 4 253 / 322, 192x144 253 / 275.
struct DenseModel {
    double blocks, exact, cell, cells[2], passes;  // cells of image 2, and of image 1 (half segments where groups are possible)
    bool grouped, whole;
};
static DenseModel dense_model(int64_t n, int64_t m, int batch, int compute, int dp, bool l2) {
    DenseModel M;
    M.grouped = dense_grouped(n, compute, dp);
    M.cell = (double)DENSE_CELL_PIXELS * dense_cell_runs(n, m);
    M.cells[0] = m / M.cell;
    M.cells[1] = (M.grouped ? 2.0 : 1.0) * n / dense_seg_pixels(n);
    M.blocks = (double)batch * ((n + 31) / 32) * ((m + 31) / 32) / 1024.0;
    M.whole = n % DENSE_SB_PIXELS == 0;
    const bool narrow = compute != FNN_F32 && dp <= 32 && !l2;  // (of the others the second step costs more than counted here, too)
    M.exact = dense_exact(compute, dp) * (narrow && !M.whole ? 1.4 : 1.0);
    const double row_bytes = dp * elem_size(compute);
    const double bytes = batch * ((double)(n + m) * (2.0 * row_bytes + 40.0) + 8.0 * n * (m / M.cell) + 8.0 * m * ((double)n / dense_seg_pixels(n)));
    M.passes = bytes / 4500.0 + batch * (double)(n + m) * 0.1;  // over maps and tables; most of it hides behind the sweep
    if (M.passes > 30000.0) M.passes = 30000.0;
    return M;
}
double dense_coarse_gain(int64_t n, int64_t m, int batch, int compute, int dp, int d, bool l2) {
    if (n < 16384 || m < 16384 || (compute != FNN_F32 && dp <= 16)) return -1e30;
    if ((double)m * (n / dense_seg_pixels(n)) * 2.0 > 4e9) return -1e30;  // the candidates' table of a pair would be too large
    const DenseModel M = dense_model(n, m, batch, compute, dp, l2);
    const double again = coarse_cells_again(M.cells[0], d, l2) / M.cells[0] + ((M.grouped ? first_round(M.cells[1]) : 0.0) + coarse_cells_again(M.cells[1], d, l2)) / M.cells[1];
    return M.blocks * (M.exact - dense_coarse_block(n, compute, dp) - dense_second(compute, dp) * again) - 45000.0 - M.passes;
}
// What the samples' marks say a pair would take, in 1/1024 ns over one step, from here on: the 8-bit maps and the samples are paid for either way, and so are launches that leave
// every pair alone.  For 16-bit rows of up to 32 channels the numbers are fitted to what 324 calls took each way (192x144 to 640x480, 1 to 16 pairs; features of 1 to 128 pixels, rank 7 to 10, lengths
// spread by exp(0.2 N(0, 1)) to exp(0.7 N(0, 1))): the way they name takes 0.2 % more than the fastest of the three on average, 8 % at the most; the numbers behind
// dense_coarse_gain, which count what is paid already and one step too low, 2.2 and 35 % (four 192x144 pairs, exp(0.2 N(0, 1)), one step / a maximum for every candidate 392 / 290 us).
// Most of what is left are features of 64 pixels and more, whose lists lie together.
// Wider rows and fp32 have those numbers (one 512x384 pair, modelled / measured, us over one step: lengths spread by exp(0.3 N(0, 1)) -57 / -59), a quarter more per group's mark and 3 ns a block for the second round.
// Pairs of one call go the same way unless one gains more than a seventh of its time by another: launches that take a part of the pairs leave the chip idle at their end (four 512x384
// pairs whose lengths are spread by exp(0.7 N(0, 1)) 8.39 ms in one step, 8.62 with a maximum for every candidate, 9.98 where each pair went its own way).  Small pairs, which hardly fill the chip
// one by one, always do (four of 192x144 with features of 64 pixels 368 us in one step, 369 for groups of three, 570 where two went either way).
DenseCosts dense_costs(const DenseCoarseArgs& a, int batch, int compute, int dp, bool l2) {
    const int64_t n = a.pixels[0], m = a.pixels[1];
    const DenseModel M = dense_model(n, m, batch, compute, dp, l2);
    double exact = M.exact, second = dense_second(compute, dp), singles = DENSE_COARSE, groups = DENSE_COARSE_GROUPS + 3.0, per_group = 1.25, first = 1.0;  // per block; over a single one's, per group's mark and of the first round's cells
    double fixed_singles = (45000.0 + M.passes) / batch, fixed_groups = fixed_singles;
    if (compute != FNN_F32 && dp <= 32) {
        exact = 1.085 * dense_exact(compute, dp) * (M.whole ? 1.0 : (n < 100000 ? 1.6 : 1.4));
        second = l2 ? 78.0 : (dp <= 24 ? 46.0 : 64.0);
        singles = 40.5;
        groups = 35.0;
        per_group = 1.2;
        first = 0.8;
        fixed_singles = 25000.0 / batch + 0.125 * (double)(n + m);
        fixed_groups = fixed_singles + 20000.0 / batch;
    }
    const double blocks = M.blocks / batch;
    auto fixed = [](double ns) { return (int64_t)(ns * 1024.0); };
    auto each = [&](int64_t cells) { return fixed(blocks * second / (DENSE_SAMPLES * (double)cells)); };
    DenseCosts j = {};
    j.pairs = batch;
    j.each[MARKS_ROWS] = each(a.n_cells);
    j.each[MARKS_SINGLES] = each(a.grouped ? (a.n_col_cells + 1) / 2 : a.n_col_cells);
    j.each[MARKS_GROUPS] = fixed(per_group * blocks * second / (DENSE_SAMPLES * (double)a.n_col_cells));
    j.singles = fixed(fixed_singles - blocks * (exact - singles));
    j.groups = a.grouped ? fixed(fixed_groups - blocks * (exact - groups)) : INT64_MAX / 256;  // (a call has 64 pairs at the most)
    j.least_groups = fixed(first * blocks * second * first_round(M.cells[1]) / M.cells[1]);
    j.margin = blocks * M.exact < 1e6 ? INT64_MAX / 2 : fixed(0.15 * blocks * M.exact);
    return j;
}

hipError_t launch_dense_sample(const DenseCoarseArgs& a, const DenseCosts& costs, int batch, hipStream_t s) {
    const int cells = a.n_cells > a.n_col_cells ? a.n_cells : a.n_col_cells;
    const hipError_t e = launch(TK_DENSE_SAMPLE, dense_sample_kernel, dim3(cells, 2, batch), dim3(SAMPLE_WAVES * 64), 0, s, a);
    if (e != hipSuccess) return e;
    return launch(TK_DENSE_SAMPLE, dense_judge_kernel, dim3((cells + JUDGE_CELLS - 1) / JUDGE_CELLS, 2, batch), dim3(DENSE_SAMPLES), 0, s, a, costs);
}
hipError_t launch_dense_coarse(DenseCoarseArgs a, int batch, hipStream_t s) {
    // six workgroups for every resident one (three per compute unit), so that the last ones leave little of the chip idle
    a.cells_per_wg = 1;
    const int64_t cells = (int64_t)a.n_cells * a.n_sb * batch;
    while (a.cells_per_wg < 4 && cells / (a.cells_per_wg * 2) >= 4608) a.cells_per_wg *= 2;
    const dim3 grid((a.n_cells + a.cells_per_wg - 1) / a.cells_per_wg, a.n_sb, batch);
    if (a.grouped) {
        if (a.seg_pixels == 2048) return launch_detail(TK_DENSE, 3, dense_groups_kernel<2048>, grid, dim3(COARSE_WAVES * 64), 0, s, a);
        return launch_detail(TK_DENSE, 3, dense_groups_kernel<4096>, grid, dim3(COARSE_WAVES * 64), 0, s, a);
    }
    if (a.seg_pixels == 2048) return launch_detail(TK_DENSE, 2, dense_coarse_kernel<2048>, grid, dim3(COARSE_WAVES * 64), 0, s, a);
    return launch_detail(TK_DENSE, 2, dense_coarse_kernel<4096>, grid, dim3(COARSE_WAVES * 64), 0, s, a);
}

static SelectSide select_side(const DenseCoarseArgs& a, int side, const u64* keys) {
    SelectSide sa = {};
    const CoarseMap& own = a.map[side];
    const CoarseMap& other = a.map[side ^ 1];
    sa.best = a.best[side];
    sa.mask = a.mask[side];
    sa.pitch = side == 0 ? (int64_t)a.n_sb * DENSE_SB_PIXELS : (int64_t)own.n_segs * a.seg_pixels;
    sa.n_cells = side == 0 ? a.n_cells : (int32_t)((a.pixels[0] + a.seg_pixels - 1) / a.seg_pixels);
    sa.n_group_cells = a.n_col_cells;
    sa.best_pitch = (side == 0 ? a.n_cells : other.n_segs) * sa.pitch;
    sa.mask_pitch = (side == 0 ? a.n_cells : (int64_t)other.n_segs << a.grouped) * (sa.pitch / 64);
    sa.cells_per_seg = side == 0 ? a.seg_pixels / (DENSE_CELL_PIXELS * a.cell_runs) : 1;
    sa.row_bound = own.row_bound + (side == 0 ? (int64_t)a.first_sb * DENSE_SB_PIXELS : 0);
    sa.bound_pitch = (int64_t)own.n_segs * a.seg_pixels;
    sa.seg = other.seg;
    sa.n_segs = other.n_segs;
    sa.grouped = side == 1 && a.grouped;
    sa.least = a.least;
    sa.keys = keys;
    sa.n_keys = a.pixels[side];
    sa.own_seg = own.seg;
    sa.own_n_segs = own.n_segs;
    sa.own_seg_pixels = a.seg_pixels;
    return sa;
}
hipError_t launch_dense_select(const DenseCoarseArgs& a, int first_side, int sides, const u64* col_keys, int batch, hipStream_t s) {
    SelectArgs args;
    args.judge = a.judge;
    int64_t wgs = 0;
    for (int i = 0; i < sides; ++i) {
        args.side[i] = select_side(a, first_side + i, col_keys);
        const int64_t need = args.side[i].pitch / (64 * SELECT_SLOTS);
        static_assert(SELECT_PARTS * 64 * SELECT_SLOTS <= DENSE_CELL_PIXELS, "enough workgroups for groups, too");
        if (need > wgs) wgs = need;
    }
    if (sides == 1) args.side[1] = args.side[0];
    return launch(TK_DENSE_SELECT, dense_select_kernel, dim3((unsigned)wgs, batch, sides), dim3(SELECT_WAVES * 64), 0, s, args);
}

}  // namespace fnn
