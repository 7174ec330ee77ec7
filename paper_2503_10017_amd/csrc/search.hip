// One-directional nearest-neighbour search: the single loop of Algorithm 2 ("FastNN-Lite",
// section 3.4.3) with its distance block fused away.  Each wave keeps a few 32-query blocks
// resident in registers, streams candidate tiles past them, forms every 32x32 block of
// scores with matrix instructions (fp32 accumulation, Algorithm 3) and folds it at once into
// a per-query running best, so no score ever leaves the register file and memory traffic is
// one pass over the candidate map per resident query group.
//
// The search runs in two passes: pass 1 finds, per query, the best score and the tile of 32
// candidates that holds it, at roughly 0.6 vector operations per score; pass 2 recomputes
// that one tile per query to name the lowest candidate index attaining the score.
//
// Work split (decided on the device from the live query count, so the host never needs to
// read it back): the queries form row groups of G*R*32, the candidate tiles are cut into
// chunks, one wave takes one (row group, chunk) unit -- every candidate tile it loads meets
// G groups of R query blocks, a group past the live queries is skipped -- and merges its
// result into the packed keys with a 64-bit atomic max (score first, lowest index on ties).
#include <type_traits>

#include "fnn_device.hpp"
#include "fnn_kernels.hpp"
#include "query_rows.hpp"
#include "search_unit.hpp"
#include "trace.hpp"

namespace fnn {

// Pass 1 kernel.  (waves_per_eu >= 2 caps the kernel at 256 registers, which lets the matrix
// instructions write their results straight into ordinary vector registers.)
template <int CT, int DP, int R, int P, int G>
__global__ __launch_bounds__(SEARCH_WAVES * 64) __attribute__((amdgpu_waves_per_eu(2)))
void search_kernel(SearchArgs a) {
    const int lane = threadIdx.x & 63, c = lane & 31, h = lane >> 5;
    // Workgroups are dealt to the 8 XCDs round-robin by their linear id, and each XCD has
    // its own L2.  Renumber them so that every XCD owns one contiguous run of (pair, unit)
    // work: the row groups that sweep the same candidate chunk then share one L2 instead
    // of fetching the chunk from HBM once per XCD.
    const int n_wgs = gridDim.x * gridDim.y;
    int wg = blockIdx.y * gridDim.x + blockIdx.x;
    if ((n_wgs & 7) == 0) wg = (wg & 7) * (n_wgs >> 3) + (wg >> 3);
    const int b = wg / gridDim.x;
    const int wave = (wg % gridDim.x) * SEARCH_WAVES + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n_waves = gridDim.x * SEARCH_WAVES;

    int n_act = a.nq;
    if (a.nq_active) n_act = min(max(a.nq_active[b], 0), a.nq);
    if (n_act <= 0 || a.m_tiles <= 0) return;

    const int row_groups = (n_act + 32 * R * G - 1) / (32 * R * G);
    int chunks = max(1, n_waves / row_groups);
    int tiles_per_chunk = max((a.m_tiles + chunks - 1) / chunks, SEARCH_MIN_TILES);
    chunks = (a.m_tiles + tiles_per_chunk - 1) / tiles_per_chunk;

    const char* src = a.src + (int64_t)b * a.src_bstride;
    const char* tgt = a.tgt + (int64_t)b * a.tgt_bstride;
    const int64_t qbase = (int64_t)b * a.nq;

    // With a single row group every unit of this pair serves the same queries, so the waves of
    // a workgroup first merge their results in LDS and the workgroup sends one atomic per query
    // instead of one per wave: atomics on one address are served serially, and with few live
    // queries that chain is what the search waits for.  (row_groups is the same for the whole
    // workgroup, so the barriers below are uniform.)
    __shared__ u64 wg_keys[32 * R * G];
    const bool combine = row_groups == 1;
    if (combine) {
        for (int i = threadIdx.x; i < 32 * R * G; i += SEARCH_WAVES * 64) wg_keys[i] = 0;
        __syncthreads();
    }

    const int64_t units = (int64_t)row_groups * chunks;
    for (int64_t unit = wave; unit < units; unit += n_waves) {
        // The few-query units below start at slot 0.  Where the query fragments of the ordinary unit leave no
        // registers to spare, the compiler must not see that as a constant: it prepared the lane addresses
        // of all three units ahead of the loop and spilled them, and a kernel that uses scratch
        // memory takes 2 us longer to start (fp16, 24 channels, G = 4, one 1024x768 map: 22.1 us for 48 live
        // queries with 21 registers spilled, 19.2 us without; 100 live 24.2 and 20.6; eight 512x384 maps in
        // bf16, 48 live, 18.9 and 16.4).  The narrower variants keep the constant (100 queries of four 512x384
        // pairs, G = 1: 13.1 us with it, 13.8 us without).
        int first_slot = 0;
        if (G * R * Ops<CT, DP>::ROW_BYTES / 8 >= 96) asm volatile("" : "+s"(first_slot));
        const int chunk = (int)(unit / row_groups);
        const int rg = (int)(unit % row_groups);
        const int slot0 = rg * 32 * R * G;
        const int t0 = chunk * tiles_per_chunk;
        const int t1 = min(t0 + tiles_per_chunk, a.m_tiles);
        if (n_act <= 32 * R) {
            // few live queries (one row group, so combine is set): only the blocks that hold a
            // live query are multiplied, and the ring is as long as the registers allow
            if (n_act <= 32)
                search_unit<CT, DP, 1, stream_ring<CT, DP, 1>(), 1, true>(a, src, tgt, qbase, n_act, first_slot, t0, t1, true, wg_keys, c, h);
            else if (n_act <= 64)
                search_unit<CT, DP, 2, stream_ring<CT, DP, 2>(), 1, true>(a, src, tgt, qbase, n_act, first_slot, t0, t1, true, wg_keys, c, h);
            else
                search_unit<CT, DP, R, stream_ring<CT, DP, R>(), 1, true>(a, src, tgt, qbase, n_act, first_slot, t0, t1, true, wg_keys, c, h);
        } else {
            search_unit<CT, DP, R, P, G, false>(a, src, tgt, qbase, n_act, slot0, t0, t1, combine, wg_keys, c, h);
        }
    }
    if (combine) {
        __syncthreads();
        for (int i = threadIdx.x; i < min(n_act, 32 * R * G); i += SEARCH_WAVES * 64) {
            const u64 key = wg_keys[i];
            if (key != 0) atomicMax(&a.out_keys[qbase + i], key);
        }
    }
}

// ---- the first searches of a call, on maps that are not prepared yet -----------------------
// Same arithmetic and same keys as search_kernel, for the case "every query live, candidates
// still in the caller's fp32 map" (the first forward and the first backward search of the
// FastNN iteration).  A workgroup's four waves take four row groups of ONE candidate chunk:
// each turn every wave fetches one 32-pixel tile of the caller's map, rounds it to the compute
// format in registers (the cast of Algorithm 3), puts the fragment into the workgroup's LDS
// ring and -- first row-group quad only -- stores it to the prepared map; after a barrier all
// four waves read the four staged tiles from LDS and multiply them with their resident query
// blocks.  The map is thus read once per quad instead of once per wave, the raw tiles of the
// next two turns are always in flight, and the separate prepare pass over the map disappears.
constexpr int FIRST_G = 3;        // groups of R query blocks per wave: 3072 queries = 8 row groups = 2 quads
constexpr int FIRST_TURN = SEARCH_WAVES;  // tiles staged per turn (one per wave)
constexpr int FIRST_AHEAD = 2;    // turns whose raw tiles are in flight
constexpr int FIRST_MIN_CHUNK = 32;  // tiles a chunk must hold for the staged kernel to be worth its start-up

// A candidate tile on its way to the LDS ring: the 12 fp32 values of the caller's row (RAWT), or
// the fragment of an already prepared map.
template <int CT, bool RAWT>
struct FirstTile {
    using O = Ops<CT, 24>;
    using Pending = std::conditional_t<RAWT, typename O::Raw, typename O::Frag>;
    static __device__ __forceinline__ Pending fetch(const FirstSearchArgs& fa, const char* tgt, int b, int t, int t1, int c, int h) {
        if constexpr (RAWT) {
            const int64_t pixel = (int64_t)t * 32 + c;
            if (t < t1 && pixel < fa.s.m) return O::load_raw(fa.raw_tgt.map[b] + pixel * fa.raw_tgt.row_stride, h);
            return O::zero_raw();  // padding rows of the prepared map are zero
        } else {
            return O::stream_tile(tgt + (int64_t)min(t, t1 - 1) * (32 * O::ROW_BYTES), c, h);
        }
    }
    static __device__ __forceinline__ typename O::Frag fragment(const Pending& p) {
        if constexpr (RAWT) return O::round_raw(p);
        else return p;
    }
};

template <int CT, int G, bool RAWT>
__global__ __launch_bounds__(SEARCH_WAVES * 64) __attribute__((amdgpu_waves_per_eu(2)))
void search_first_kernel(FirstSearchArgs fa) {
    using O = Ops<CT, 24>;
    using Frag = typename O::Frag;
    using Tile = FirstTile<CT, RAWT>;
    constexpr int R = SEARCH_R;
    // The loop reacts to where its code lies.  A hint always takes the code that masks the map's last tile out of
    // the straight path; hints on the other two branches cost the fp16 variant for the caller's maps 1-2 %
    // (every pixel of a 512x384 pair as a query 1678 us with them, 1646 us without, 16 pairs of 3072 queries
    // 447 and 443 us).
    constexpr bool HINTS = !(RAWT && CT == CT_F16);
    const SearchArgs& a = fa.s;
    __shared__ uint4 stage_lo[2][FIRST_TURN][64];
    __shared__ uint2 stage_hi[2][FIRST_TURN][64];
    const int lane = threadIdx.x & 63, c = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // one XCD owns a contiguous run of (pair, unit) work, see search_kernel
    const int n_wgs = gridDim.x * gridDim.y;
    int wg = blockIdx.y * gridDim.x + blockIdx.x;
    if ((n_wgs & 7) == 0) wg = (wg & 7) * (n_wgs >> 3) + (wg >> 3);
    const int b = wg / gridDim.x;
    const int wgi = wg % gridDim.x;
    const int n_act = a.nq;
    if (n_act <= 0 || a.m_tiles <= 0) return;

    // On prepared maps the groups of R query blocks are dealt evenly to the waves of all quads: 25 groups
    // (3185 queries) give the 12 waves of three quads two or three each, where filling one quad after the
    // other left the third with a single group and three idle waves (four pairs of 517x389 and 433x301
    // pixels: 105 + 154 us for the two first searches, 99 + 145 dealt evenly).  The waves with one
    // group more sit at different places of their workgroups, that is on different SIMDs.  The variant for the
    // caller's fp32 maps fills the quads in turn: its loop is sensitive to how it is laid out, and with
    // the even deal every pixel of a 512x384 pair as a query took 1750 instead of 1690 us.
    const int row_groups = (n_act + 32 * R * G - 1) / (32 * R * G);
    const int quads = (row_groups + SEARCH_WAVES - 1) / SEARCH_WAVES;
    int chunks = max(1, (int)gridDim.x / quads);
    int tiles_per_chunk = (a.m_tiles + chunks - 1) / chunks;
    tiles_per_chunk = (tiles_per_chunk + FIRST_TURN - 1) / FIRST_TURN * FIRST_TURN;
    chunks = (a.m_tiles + tiles_per_chunk - 1) / tiles_per_chunk;

    const char* src = a.src + (int64_t)b * a.src_bstride;
    char* tgt = const_cast<char*>(a.tgt) + (int64_t)b * a.tgt_bstride;
    const int64_t qbase = (int64_t)b * a.nq;
    const float ninf = -__builtin_inff();

    const int units = quads * chunks;
    for (int unit = wgi; unit < units; unit += gridDim.x) {  // uniform in the workgroup
        const int chunk = unit / quads, quad = unit % quads;
        int slot0 = (quad * SEARCH_WAVES + wave) * 32 * R * G, slot_end = n_act;  // this wave's slots
        if constexpr (!RAWT) {
            const int groups = (n_act + 32 * R - 1) / (32 * R);
            const int per_wave = groups / (quads * SEARCH_WAVES), more = groups % (quads * SEARCH_WAVES);
            const int rank = ((wave + quad) & (SEARCH_WAVES - 1)) * quads + quad;
            slot0 = (rank * per_wave + min(rank, more)) * 32 * R;
            slot_end = min(n_act, slot0 + (per_wave + (rank < more ? 1 : 0)) * 32 * R);
        }
        const int t0 = chunk * tiles_per_chunk;
        const int t1 = min(t0 + tiles_per_chunk, a.m_tiles);
        const int n_turns = (t1 - t0 + FIRST_TURN - 1) / FIRST_TURN;

        static_assert(FIRST_AHEAD == 2, "the turn loop below is unrolled by the two ring slots");
        typename Tile::Pending raw[FIRST_AHEAD];
#pragma unroll
        for (int p = 0; p < FIRST_AHEAD; ++p) raw[p] = Tile::fetch(fa, tgt, b, t0 + p * FIRST_TURN + wave, t1, c, h);

        // The running best of a query block lives in two registers that trade places from tile to
        // tile (the tiles of a turn are unrolled, so which one is current is known at compile time):
        // the fold writes the new best beside the old one, which the "did it rise" test still needs,
        // instead of into a scratch register that then has to be copied.
        static_assert(FIRST_TURN % 2 == 0, "after a turn the current best is in best[0] again");
        Frag q[G][R];
        float best[2][G][R];
        int best_tile[G][R];
        bool live[G];
#pragma unroll
        for (int g = 0; g < G; ++g) live[g] = slot0 + g * 32 * R < slot_end;  // uniform in the wave
        {
            int32_t row[G * R];
            query_rows<G * R>(a, qbase, slot0, n_act, c, row);
            if (fa.raw_queries) {
                // group by group: a group's raw rows take twice the registers of its fragments
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    typename O::Raw x[R];
#pragma unroll
                    for (int r = 0; r < R; ++r) x[r] = O::load_raw(fa.raw_src.map[b] + (int64_t)row[g * R + r] * fa.raw_src.row_stride, h);
#pragma unroll
                    for (int r = 0; r < R; ++r) q[g][r] = O::round_raw(x[r]);
                }
            } else {
#pragma unroll
                for (int i = 0; i < G * R; ++i) q[i / R][i % R] = O::load(src + (int64_t)row[i] * O::ROW_BYTES, h);
            }
        }
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int r = 0; r < R; ++r) {
                arrived(q[g][r]);
                best[0][g][r] = ninf;
                best[1][g][r] = ninf;
                best_tile[g][r] = 0x7FFFFFFF;
            }

        // The quads of a chunk that read the caller's map would all ask for the same fp32 tile at the same moment
        // and queue on one channel of L2: they start up to 2 us apart instead (fp16, every pixel of a 512x384
        // pair as a query, 128 quads per chunk: 1756 us so, 1786 us in step).  Prepared tiles are half the bytes and
        // do not queue, there the late start only costs (stored bf16 1593 us so, 1545 us in step; fp16 1685 and 1649).
        if constexpr (RAWT)
            for (int i = 0; i < (quad & 7); ++i) __builtin_amdgcn_s_sleep(8);

        // one turn: stage my tile of the turn, then multiply the four staged tiles
        auto turn = [&](int k, auto slot_tag) {
            constexpr int SLOT = decltype(slot_tag)::value;
            const int mine = t0 + k * FIRST_TURN + wave;
            const Frag f = Tile::fragment(raw[SLOT]);
            stage_lo[SLOT][wave][lane] = f.lo;
            stage_hi[SLOT][wave][lane] = f.hi;
            if (RAWT && quad == 0 && mine < t1) O::store_tile(tgt + (int64_t)mine * (32 * O::ROW_BYTES), c, h, f);
            raw[SLOT] = Tile::fetch(fa, tgt, b, mine + FIRST_AHEAD * FIRST_TURN, t1, c, h);
            __syncthreads();
#pragma unroll
            for (int j = 0; j < FIRST_TURN; ++j) {
                const int t = t0 + k * FIRST_TURN + j;
                const int now = j & 1, then = now ^ 1;
                if (HINTS ? __builtin_expect(t < t1, 1) : t < t1) {  // uniform
                    Frag cur;
                    cur.lo = stage_lo[SLOT][j][lane];
                    cur.hi = stage_hi[SLOT][j][lane];
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        if (HINTS ? __builtin_expect(live[g], 1) : live[g]) {
                            f32x16 acc[R];
#pragma unroll
                            for (int r = 0; r < R; ++r) acc[r] = O::mma(cur, q[g][r]);
                            if (__builtin_expect(t * 32 + 32 > a.m, 0)) {  // only the last tile of the map can be partial
                                const int bound = a.m - t * 32 - 4 * h;
#pragma unroll
                                for (int r = 0; r < R; ++r)
#pragma unroll
                                    for (int v = 0; v < 16; ++v)
                                        if (tile_row(v, 0) >= bound) acc[r][v] = ninf;
                            }
#pragma unroll
                            for (int r = 0; r < R; ++r) {
                                const float top = fold16(best[now][g][r], acc[r]);
                                if (top > best[now][g][r]) best_tile[g][r] = t;
                                best[then][g][r] = top;
                            }
                        }
                    }
                } else {  // past the chunk's last tile: the best just moves on
#pragma unroll
                    for (int g = 0; g < G; ++g)
#pragma unroll
                        for (int r = 0; r < R; ++r) best[then][g][r] = best[now][g][r];
                }
            }
        };
        for (int k = 0; k < n_turns; k += 2) {
            turn(k, std::integral_constant<int, 0>{});
            if (k + 1 < n_turns) turn(k + 1, std::integral_constant<int, 1>{});  // uniform
        }

#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int r = 0; r < R; ++r) {
                float mine = best[0][g][r];
                const float ob = __shfl_xor(mine, 32);
                const int ot = __shfl_xor(best_tile[g][r], 32);
                if (ob > mine || (ob == mine && ot < best_tile[g][r])) {
                    mine = ob;
                    best_tile[g][r] = ot;
                }
                const int slot = slot0 + (g * R + r) * 32 + c;
                if (h == 0 && slot < slot_end) atomicMax(&a.out_keys[qbase + slot], pack_key(mine, best_tile[g][r]));
            }
        __syncthreads();  // the next unit's first turn reuses ring slot 0
    }
}

// The key is rewritten with the candidate index; optionally index and score are stored as well.
// clear_count: one count per pair that is set to 0 on the way (NULL: none).
// load_query(b, row, h) supplies the query fragment.
template <int CT, int DP, typename LoadQuery>
__device__ __forceinline__ void resolve_body(const SearchArgs& a, int32_t* out_idx, float* out_score, int32_t* clear_count,
                                             LoadQuery load_query) {
    const int lane = threadIdx.x & 63, c = lane & 31, h = lane >> 5;
    const int wave = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n_waves = gridDim.x * 4;
    const int b = blockIdx.y;
    if (clear_count && blockIdx.x == 0 && threadIdx.x == 0) clear_count[b] = 0;
    int n_act = a.nq;
    if (a.nq_active) n_act = min(max(a.nq_active[b], 0), a.nq);
    const char* tgt = a.tgt + (int64_t)b * a.tgt_bstride;
    const int64_t qbase = (int64_t)b * a.nq;

    for (uint32_t slot = wave; slot < (uint32_t)n_act; slot += n_waves) {  // without a sign, see resolve_step_kernel
        const u64 key = a.out_keys[qbase + slot];
        const int64_t qrow = query_row(a, qbase, slot);  // fetched beside the key, not behind the test of it
        Resolved res = {-1, -__builtin_inff()};
        if (key != 0) {
            res = resolve_tile<CT, DP>(a, tgt, key, load_query(b, qrow, h), c, h);
            if (lane == 0) a.out_keys[qbase + slot] = pack_key(res.score, res.idx);
        }
        if (lane == 0 && out_idx) {
            out_idx[qbase + slot] = res.idx;
            if (out_score) out_score[qbase + slot] = res.score;
        }
    }
}

template <int CT, int DP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
void resolve_kernel(SearchArgs a, int32_t* out_idx, float* out_score, int32_t* clear_count) {
    using O = Ops<CT, DP>;
    resolve_body<CT, DP>(a, out_idx, out_score, clear_count, [&](int b, int64_t row, int h) {
        return O::load(a.src + (int64_t)b * a.src_bstride + row * O::ROW_BYTES, h);
    });
}

// The same with the queries still in the caller's fp32 map (rounded on the way, like the
// fused first search rounds them).
template <int CT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
void resolve_raw_kernel(FirstSearchArgs fa, int32_t* out_idx, float* out_score, int32_t* clear_count) {
    using O = Ops<CT, 24>;
    resolve_body<CT, 24>(fa.s, out_idx, out_score, clear_count, [&](int b, int64_t row, int h) {
        return O::round_raw(O::load_raw(fa.raw_src.map[b] + row * fa.raw_src.row_stride, h));
    });
}

// Pass 2 of the search back into image 1 and, in the same launch, the bookkeeping of the
// iteration (section 3.2.5, steps 2-3): U^{t+1} is named, compared with U^t, and the seeds still
// moving are compacted into the other half of the ping-pong state.  A wave takes one slot at a time;
// a workgroup collects its survivors in LDS and reserves room for them with one atomic add per
// round (an add and two barriers for every 16 slots took 41 instead of 22 us for the first step of 16
// pairs), so the survivors' order differs from run to run; every result is filed under its seed's number
// and the match set is sorted by a kernel of its own, so no output depends on it.  As a launch of its
// own the bookkeeping took one workgroup per pair 4-16 us of every iteration with live seeds (its
// share of a 1024x768 call was 30 us) and 1.6 us (2.5 us of host time) of every other.
constexpr int STEP_WAVES = 16;
constexpr int STEP_ROUND = 1024;  // slots a workgroup takes before it hands its survivors on (8 KB of LDS)
constexpr int STEP_MAX_WGS = 512;  // of all pairs: two workgroups of 16 waves per compute unit are resident
static_assert(MAX_SLOTS + (int64_t)STEP_MAX_WGS * STEP_ROUND <= 0xFFFFFFFFLL, "a round past the last slot must not wrap around");
template <int CT, int DP>
__global__ __launch_bounds__(STEP_WAVES * 64)
void resolve_step_kernel(SearchArgs a, StepArgs st) {
    using O = Ops<CT, DP>;
    __shared__ int2 moving[STEP_ROUND];  // survivors of a round: (U^{t+1}, seed number)
    __shared__ int n_moving, first_pos;
    const int lane = threadIdx.x & 63, c = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int b = blockIdx.y;
    const int n_act = min(max(a.nq_active[b], 0), a.nq);
    const char* src = a.src + (int64_t)b * a.src_bstride;
    const char* tgt = a.tgt + (int64_t)b * a.tgt_bstride;
    const int64_t base = (int64_t)b * a.nq;

    // slots are counted in 32 bits without a sign: the round after the last one may lie past 2^31
    const uint32_t step = gridDim.x * STEP_ROUND;
    for (uint32_t round = 0; round < (uint32_t)n_act; round += step) {  // uniform in the launch's workgroups of this pair
        if (threadIdx.x == 0) n_moving = 0;
        __syncthreads();
        // the workgroups take the slots of a round 16 at a time in turn, so that few slots spread over all of them
        const uint32_t end = min((uint32_t)n_act, round + step);
        for (uint32_t slot = round + blockIdx.x * STEP_WAVES + wave; slot < end; slot += gridDim.x * STEP_WAVES) {  // uniform in the wave
            const u64 kf = st.keys_f[base + slot];
            const u64 kb = a.out_keys[base + slot];
            const int32_t u = st.cur_u[base + slot];
            const int32_t sid = st.seed_id[base + slot];
            const int32_t v = key_index(kf);
            int32_t u_next = -1;
            if (kb != 0) {
                const int64_t qrow = min(max(v, 0), a.src_rows - 1);
                u_next = resolve_tile<CT, DP>(a, tgt, kb, O::load(src + qrow * O::ROW_BYTES, h), c, h).idx;
            }
            const bool converged = st.mode != 2 && u_next == u;
            if (lane == 0) {
                if (converged || st.mode != 0) {
                    st.seed_i[base + sid] = u;
                    st.seed_j[base + sid] = v;
                    st.seed_iter[base + sid] = converged ? st.t : -1;
                } else {
                    moving[atomicAdd(&n_moving, 1)] = make_int2(u_next, sid);  // a round gives a workgroup at most STEP_ROUND slots
                }
                st.keys_f[base + slot] = 0;  // both tables start the next searches empty
                a.out_keys[base + slot] = 0;
            }
        }
        __syncthreads();
        if (threadIdx.x == 0) first_pos = n_moving ? atomicAdd(&st.next_active[b], n_moving) : 0;
        __syncthreads();
        for (int i = threadIdx.x; i < n_moving; i += STEP_WAVES * 64) {
            st.next_u[base + first_pos + i] = moving[i].x;
            st.next_seed_id[base + first_pos + i] = moving[i].y;
        }
        __syncthreads();  // the next round empties the list
    }
}

// One resident wave per hardware slot: the grid is exactly what the chip holds at once
// (workgroups per CU from the occupancy calculator x CUs), split evenly between the pairs, so
// there is no partial last round and the per-wave start-up cost and the final key merges are
// paid once per slot.  Two waves per SIMD are what the widest variant fits and what measured
// best for the narrower ones too, so the widest variant's occupancy sizes every launch.
template <int CT, int DP>
static int search_wgs_per_pair(int batch) {
    static DeviceCache resident_wgs;  // workgroups of the widest variant the current device holds at once
    const long long resident = resident_wgs.get([](int dev) -> long long {
        int per_cu = 0;
        hipDeviceProp_t prop;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu,
                                                         search_kernel<CT, DP, SEARCH_R, search_ring<CT, DP>(), search_g_limit<CT, DP>()>,
                                                         SEARCH_WAVES * 64, 0) != hipSuccess ||
            hipGetDeviceProperties(&prop, dev) != hipSuccess)
            return -1;
        return (long long)(per_cu > 0 ? per_cu : 1) * prop.multiProcessorCount;
    });
    if (resident <= 0) return 0;
    int wgs = (int)resident / batch;
    if (wgs >= 8) wgs &= ~7;  // a multiple of 8 per pair keeps the XCD renumbering a bijection
    return wgs < 1 ? 1 : wgs;
}

// Tiles per chunk if the launch used row groups of G*R blocks.
template <int CT, int DP, int G>
static int search_chunk_tiles(const SearchArgs& a, int batch) {
    const int n_waves = search_wgs_per_pair<CT, DP>(batch) * SEARCH_WAVES;
    const int row_groups = (a.nq + 32 * SEARCH_R * G - 1) / (32 * SEARCH_R * G);
    const int chunks = n_waves / row_groups > 0 ? n_waves / row_groups : 1;
    return a.m_tiles / chunks;
}

template <int CT, int DP, int G>
static hipError_t launch_search_g(const SearchArgs& a, int batch, hipStream_t s) {
    int wgs = search_wgs_per_pair<CT, DP>(batch);
    if (wgs == 0) return hipErrorUnknown;
    const int64_t max_units = (int64_t)((a.nq + 32 * SEARCH_R * G - 1) / (32 * SEARCH_R * G)) *
                              ((a.m_tiles + SEARCH_MIN_TILES - 1) / SEARCH_MIN_TILES);
    const int64_t need = (max_units + SEARCH_WAVES - 1) / SEARCH_WAVES;
    if (need < wgs) wgs = (int)(need > 0 ? need : 1);
    return launch_detail(TK_SEARCH, G, search_kernel<CT, DP, SEARCH_R, search_ring<CT, DP>(), G>, dim3(wgs, batch), dim3(SEARCH_WAVES * 64), 0, s, a);
}

template <int CT, int DP>
static hipError_t launch_search_t(const SearchArgs& a, int batch, hipStream_t s) {
    // Wider row groups (more query blocks per loaded candidate tile) pay off while the chunks
    // stay long -- with many waves per pair (few pairs) short chunks would mostly pay
    // start-up -- and while the resident query fragments fit the register file.
    constexpr int G_LIMIT = search_g_limit<CT, DP>();
    if constexpr (G_LIMIT >= 4)
        if (search_chunk_tiles<CT, DP, 4>(a, batch) >= SEARCH_WIDE_MIN_TILES) return launch_search_g<CT, DP, 4>(a, batch, s);
    if constexpr (G_LIMIT >= 2)
        if (search_chunk_tiles<CT, DP, 2>(a, batch) >= SEARCH_WIDE_MIN_TILES) return launch_search_g<CT, DP, 2>(a, batch, s);
    return launch_search_g<CT, DP, 1>(a, batch, s);
}

hipError_t launch_search(const SearchArgs& a, int batch, int compute, int dp, hipStream_t s) {
    if (a.nq <= 0 || batch <= 0) return hipSuccess;
    if (compute == FNN_F16) {
        if (dp == 16) return launch_search_t<CT_F16, 16>(a, batch, s);
        if (dp == 24) return launch_search_t<CT_F16, 24>(a, batch, s);
        if (dp == 32) return launch_search_t<CT_F16, 32>(a, batch, s);
        // rows of the two-term representation (three copies of the channels)
        if (dp == 48) return launch_search_t<CT_F16, 48>(a, batch, s);
        if (dp == 64) return launch_search_t<CT_F16, 64>(a, batch, s);
        if (dp == 80) return launch_search_t<CT_F16, 80>(a, batch, s);
        if (dp == 96) return launch_search_t<CT_F16, 96>(a, batch, s);
    } else if (compute == FNN_BF16) {
        if (dp == 16) return launch_search_t<CT_BF16, 16>(a, batch, s);
        if (dp == 24) return launch_search_t<CT_BF16, 24>(a, batch, s);
        if (dp == 32) return launch_search_t<CT_BF16, 32>(a, batch, s);
    } else {
        if (dp == 8) return launch_search_t<CT_F32, 8>(a, batch, s);
        if (dp == 16) return launch_search_t<CT_F32, 16>(a, batch, s);
        if (dp == 24) return launch_search_t<CT_F32, 24>(a, batch, s);
        if (dp == 32) return launch_search_t<CT_F32, 32>(a, batch, s);
    }
    return hipErrorInvalidValue;
}

// ---- fused first search: launch shape ------------------------------------------------------
// Workgroups of the staged kernel that the current device holds at once (0: unknown).
static int first_search_resident_wgs() {
    static DeviceCache resident_wgs;
    const long long resident = resident_wgs.get([](int dev) -> long long {
        int per_cu = 0;
        hipDeviceProp_t prop;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, search_first_kernel<CT_F16, FIRST_G, true>, SEARCH_WAVES * 64, 0) != hipSuccess ||
            hipGetDeviceProperties(&prop, dev) != hipSuccess)
            return -1;
        return (long long)(per_cu > 0 ? per_cu : 1) * prop.multiProcessorCount;
    });
    return resident > 0 ? (int)resident : 0;
}
static int first_search_wgs_per_pair(int batch) {
    int wgs = first_search_resident_wgs() / batch;
    if (wgs >= 8) wgs &= ~7;
    return wgs < 1 ? 1 : wgs;
}

bool first_search_applies(int64_t nq, int64_t m, int batch) {
    // at least one full quad of row groups, so that the four waves of a workgroup all have queries ...
    if (nq < (int64_t)SEARCH_WAVES * 32 * SEARCH_R * FIRST_G || nq > 0x7FFFFFFF) return false;
    // ... and chunks of at least FIRST_MIN_CHUNK tiles: one pair alone spreads over so many workgroups
    // that a chunk would be a few turns long and mostly start-up (measured: a single 512x384 pair is
    // 1.5 % slower with the staged kernel, two pairs are 2.5 % faster)
    const int64_t row_groups = (nq + 32 * SEARCH_R * FIRST_G - 1) / (32 * SEARCH_R * FIRST_G);
    const int64_t quads = (row_groups + SEARCH_WAVES - 1) / SEARCH_WAVES;
    const int64_t chunks = first_search_wgs_per_pair(batch) / quads > 0 ? first_search_wgs_per_pair(batch) / quads : 1;
    return (m + 31) / 32 / chunks >= FIRST_MIN_CHUNK;
}

template <int CT, bool RAWT>
static hipError_t launch_search_first_t(const FirstSearchArgs& a, int batch, hipStream_t s) {
    if (first_search_resident_wgs() <= 0) return hipErrorUnknown;
    int wgs = first_search_wgs_per_pair(batch);
    const int row_groups = (a.s.nq + 32 * SEARCH_R * FIRST_G - 1) / (32 * SEARCH_R * FIRST_G);
    const int quads = (row_groups + SEARCH_WAVES - 1) / SEARCH_WAVES;
    const int64_t max_units = (int64_t)quads * ((a.s.m_tiles + FIRST_TURN - 1) / FIRST_TURN);
    if (max_units < wgs) wgs = (int)(max_units > 0 ? max_units : 1);
    return launch_detail(TK_SEARCH, 100 + FIRST_G, search_first_kernel<CT, FIRST_G, RAWT>, dim3(wgs, batch), dim3(SEARCH_WAVES * 64), 0, s, a);
}

hipError_t launch_search_first(const FirstSearchArgs& a, int batch, int compute, hipStream_t s) {
    if (a.s.nq <= 0 || batch <= 0) return hipSuccess;
    const bool raw = a.raw_tgt.map[0] != nullptr;  // else the candidates are the prepared map s.tgt itself
    if (compute == FNN_F16) return raw ? launch_search_first_t<CT_F16, true>(a, batch, s) : launch_search_first_t<CT_F16, false>(a, batch, s);
    if (compute == FNN_BF16) return raw ? launch_search_first_t<CT_BF16, true>(a, batch, s) : launch_search_first_t<CT_BF16, false>(a, batch, s);
    return hipErrorInvalidValue;
}

hipError_t launch_resolve_raw(const FirstSearchArgs& a, int batch, int compute, int32_t* out_idx, float* out_score, int32_t* clear_count,
                              hipStream_t s) {
    if (a.s.nq <= 0 || batch <= 0) return hipSuccess;
    int wgs = (a.s.nq + 3) / 4;
    const int cap = 2048 / batch > 64 ? 2048 / batch : 64;
    if (wgs > cap) wgs = cap;
    if (compute == FNN_F16) return launch(TK_RESOLVE, resolve_raw_kernel<CT_F16>, dim3(wgs, batch), dim3(256), 0, s, a, out_idx, out_score, clear_count);
    if (compute == FNN_BF16) return launch(TK_RESOLVE, resolve_raw_kernel<CT_BF16>, dim3(wgs, batch), dim3(256), 0, s, a, out_idx, out_score, clear_count);
    return hipErrorInvalidValue;
}

template <int CT, int DP>
static hipError_t launch_resolve_t(const SearchArgs& a, int batch, int32_t* out_idx, float* out_score, int32_t* clear_count,
                                   hipStream_t s) {
    int wgs = (a.nq + 3) / 4;
    const int cap = 2048 / batch > 64 ? 2048 / batch : 64;  // measured best: more waves only add dispatch time
    if (wgs > cap) wgs = cap;
    return launch(TK_RESOLVE, resolve_kernel<CT, DP>, dim3(wgs, batch), dim3(256), 0, s, a, out_idx, out_score, clear_count);
}

hipError_t launch_resolve(const SearchArgs& a, int batch, int compute, int dp, int32_t* out_idx, float* out_score,
                          int32_t* clear_count, hipStream_t s) {
    if (a.nq <= 0 || batch <= 0) return hipSuccess;
    if (compute == FNN_F16) {
        if (dp == 16) return launch_resolve_t<CT_F16, 16>(a, batch, out_idx, out_score, clear_count, s);
        if (dp == 24) return launch_resolve_t<CT_F16, 24>(a, batch, out_idx, out_score, clear_count, s);
        if (dp == 32) return launch_resolve_t<CT_F16, 32>(a, batch, out_idx, out_score, clear_count, s);
        if (dp == 48) return launch_resolve_t<CT_F16, 48>(a, batch, out_idx, out_score, clear_count, s);
        if (dp == 64) return launch_resolve_t<CT_F16, 64>(a, batch, out_idx, out_score, clear_count, s);
        if (dp == 80) return launch_resolve_t<CT_F16, 80>(a, batch, out_idx, out_score, clear_count, s);
        if (dp == 96) return launch_resolve_t<CT_F16, 96>(a, batch, out_idx, out_score, clear_count, s);
    } else if (compute == FNN_BF16) {
        if (dp == 16) return launch_resolve_t<CT_BF16, 16>(a, batch, out_idx, out_score, clear_count, s);
        if (dp == 24) return launch_resolve_t<CT_BF16, 24>(a, batch, out_idx, out_score, clear_count, s);
        if (dp == 32) return launch_resolve_t<CT_BF16, 32>(a, batch, out_idx, out_score, clear_count, s);
    } else {
        if (dp == 8) return launch_resolve_t<CT_F32, 8>(a, batch, out_idx, out_score, clear_count, s);
        if (dp == 16) return launch_resolve_t<CT_F32, 16>(a, batch, out_idx, out_score, clear_count, s);
        if (dp == 24) return launch_resolve_t<CT_F32, 24>(a, batch, out_idx, out_score, clear_count, s);
        if (dp == 32) return launch_resolve_t<CT_F32, 32>(a, batch, out_idx, out_score, clear_count, s);
    }
    return hipErrorInvalidValue;
}

template <int CT, int DP>
static hipError_t launch_resolve_step_t(const SearchArgs& a, const StepArgs& st, int batch, hipStream_t s) {
    int wgs = (a.nq + STEP_WAVES - 1) / STEP_WAVES;
    const int cap = STEP_MAX_WGS / batch > 16 ? STEP_MAX_WGS / batch : 16;
    if (wgs > cap) wgs = cap;
    return launch(TK_RECIP_STEP, resolve_step_kernel<CT, DP>, dim3(wgs, batch), dim3(STEP_WAVES * 64), 0, s, a, st);
}

hipError_t launch_resolve_step(const SearchArgs& a, const StepArgs& st, int batch, int compute, int dp, hipStream_t s) {
    if (a.nq <= 0 || batch <= 0) return hipSuccess;
    if (compute == FNN_F16) {
        if (dp == 16) return launch_resolve_step_t<CT_F16, 16>(a, st, batch, s);
        if (dp == 24) return launch_resolve_step_t<CT_F16, 24>(a, st, batch, s);
        if (dp == 32) return launch_resolve_step_t<CT_F16, 32>(a, st, batch, s);
        if (dp == 48) return launch_resolve_step_t<CT_F16, 48>(a, st, batch, s);
        if (dp == 64) return launch_resolve_step_t<CT_F16, 64>(a, st, batch, s);
        if (dp == 80) return launch_resolve_step_t<CT_F16, 80>(a, st, batch, s);
        if (dp == 96) return launch_resolve_step_t<CT_F16, 96>(a, st, batch, s);
    } else if (compute == FNN_BF16) {
        if (dp == 16) return launch_resolve_step_t<CT_BF16, 16>(a, st, batch, s);
        if (dp == 24) return launch_resolve_step_t<CT_BF16, 24>(a, st, batch, s);
        if (dp == 32) return launch_resolve_step_t<CT_BF16, 32>(a, st, batch, s);
    } else {
        if (dp == 8) return launch_resolve_step_t<CT_F32, 8>(a, st, batch, s);
        if (dp == 16) return launch_resolve_step_t<CT_F32, 16>(a, st, batch, s);
        if (dp == 24) return launch_resolve_step_t<CT_F32, 24>(a, st, batch, s);
        if (dp == 32) return launch_resolve_step_t<CT_F32, 32>(a, st, batch, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace fnn
