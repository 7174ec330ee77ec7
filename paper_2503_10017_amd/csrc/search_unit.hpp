// Device code of a search that the kernels of search.hip and tail.hip share: a unit of pass 1, and pass 2 for one query.
#pragma once
#include "fnn_device.hpp"
#include "fnn_kernels.hpp"
#include "query_rows.hpp"

namespace fnn {

constexpr int SEARCH_R = 4;           // 32-query blocks whose products are in flight together
// A wave keeps G groups of R query blocks resident (G = 1, 2 or 4, chosen per launch), so every
// candidate tile it loads meets G*R query blocks.
constexpr int SEARCH_WIDE_MIN_TILES = 128;  // a wave takes more groups only while its chunk stays at least this long
// Shortest chunk worth a wave.  Every chunk ends in 64-bit atomic max operations on the keys of
// the live queries, and atomics on one address are served one after the other (about 13 ns
// each here): with few live queries and few pairs, 4-tile chunks and one atomic per wave meant
// 1536 of them per key and 21-34 us per search of a 512x384 map.  8-tile chunks together with
// the workgroup-level merge in the kernel take 8-12 us (4 and 16 measured slower).
constexpr int SEARCH_MIN_TILES = 8;
constexpr int SEARCH_WAVES = 4;       // waves per workgroup
constexpr int SEARCH_P = 4;           // candidate tiles in flight per wave

// One unit of pass 1: the query blocks of slots [slot0, slot0 + 32*R*G) against the candidate
// tiles [t0, t1).  Per query the best score and the 32-candidate TILE that holds it: a lane only
// keeps a running maximum (3-input max) and, once per tile, notes the tile when the maximum
// rose -- strictly, so the lowest tile wins among equal scores.  The key carries the tile
// number in its index field; pass 2 turns it into the candidate index.  With `combine` the
// keys go to the workgroup's table in LDS (slot0 is 0 then), else to the global table.
// P candidate tiles are always in flight towards the registers; a slot is refilled as soon
// as its tile has been handed to the matrix cores.  EXACT: loads past the end of the chunk are
// skipped (for chunks that may be shorter than the ring); otherwise they re-read the chunk's
// last tile, which keeps the loop free of branches around the loads.
// LIVE_LIST: a.q_idx is written while the kernel runs, see query_rows.
template <int CT, int DP, int R, int P, int G, bool EXACT, bool LIVE_LIST = false>
__device__ __forceinline__ void search_unit(const SearchArgs& a, const char* src, const char* tgt, int64_t qbase,
                                            int n_act, int slot0, int t0, int t1, bool combine, u64* wg_keys, int c, int h) {
    using O = Ops<CT, DP>;
    using Frag = typename O::Frag;
    const float ninf = -__builtin_inff();
    // The first P loads are issued before the (dependent) query fetch so that both latencies
    // overlap.
    Frag ring[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        if (!EXACT) ring[p] = O::stream_tile(tgt + (int64_t)min(t0 + p, t1 - 1) * (32 * O::ROW_BYTES), c, h);
        else if (p == 0 || t0 + p < t1)  // uniform; a slot past the end is never used
            ring[p] = O::stream_tile(tgt + (int64_t)(t0 + p) * (32 * O::ROW_BYTES), c, h);
    }

    // blocks past the live queries of the last row group repeat the last one and are dropped; a
    // whole group of R blocks past them is skipped
    Frag q[G][R];
    float best[G][R];
    int best_tile[G][R];
    bool live[G];
#pragma unroll
    for (int g = 0; g < G; ++g) live[g] = slot0 + g * 32 * R < n_act;  // uniform
    {
        int32_t row[G * R];
        query_rows<G * R, LIVE_LIST>(a, qbase, slot0, n_act, c, row);
#pragma unroll
        for (int i = 0; i < G * R; ++i) q[i / R][i % R] = O::load(src + (int64_t)row[i] * O::ROW_BYTES, h);
    }
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int r = 0; r < R; ++r) {
            arrived(q[g][r]);
            best[g][r] = ninf;
            best_tile[g][r] = 0x7FFFFFFF;
        }

    int tb = t0;
    if constexpr (!EXACT && G < 4 && O::ROW_BYTES <= 64) {
        // Whole trips of the ring over whole tiles with every group live: a product is followed by the maxima of the one before it
        // (see coarse_kernel; here the matrix instructions are most of the time: one 512x384 pair 195.9 -> 193.3 us, two pairs with squared distance
        // 317.4 -> 311.1; with four groups 16 pairs 1313 -> 1324; wider rows gain nothing and spill).
        const int whole = live[G - 1] ? min(t1, a.m / 32) : t0;  // uniform
        constexpr int BLOCKS = G * R;
        static_assert(BLOCKS * P % 2 == 0, "a trip starts on acc[0]");
        f32x16 acc[2];
        if (tb + P <= whole) acc[0] = O::mma(ring[0], q[0][0]);
        for (; tb + P <= whole; tb += P) {
#pragma unroll
            for (int p = 0; p < P; ++p) {
#pragma unroll
                for (int i = 0; i < BLOCKS; ++i) {
                    const int n = p * BLOCKS + i, g = i / R, r = i % R;
                    if (i + 1 < BLOCKS) acc[(n + 1) & 1] = O::mma(ring[p], q[(i + 1) / R][(i + 1) % R]);
                    else acc[(n + 1) & 1] = O::mma(ring[(p + 1) % P], q[0][0]);  // past the last trip: of a tile that the loop below takes again
                    if (i + 2 == BLOCKS) ring[p] = O::stream_tile(tgt + (int64_t)min(tb + p + P, t1 - 1) * (32 * O::ROW_BYTES), c, h);
                    __builtin_amdgcn_sched_barrier(0);
                    const float top = fold16(best[g][r], acc[n & 1]);
                    if (top > best[g][r]) best_tile[g][r] = tb + p;
                    best[g][r] = top;
                    asm volatile("" : "+v"(best[g][r]));
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
    }
    for (; tb < t1; tb += P) {
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const int t = tb + p;
            if (__builtin_expect(t < t1, 1)) {  // uniform
                const Frag cur = ring[p];
                if (!EXACT) ring[p] = O::stream_tile(tgt + (int64_t)min(t + P, t1 - 1) * (32 * O::ROW_BYTES), c, h);
                else if (t + P < t1) ring[p] = O::stream_tile(tgt + (int64_t)(t + P) * (32 * O::ROW_BYTES), c, h);
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    if (__builtin_expect(live[g], 1)) {
                        f32x16 acc[R];
#pragma unroll
                        for (int r = 0; r < R; ++r) acc[r] = O::mma(cur, q[g][r]);
                        if (__builtin_expect(t * 32 + 32 > a.m, 0)) {  // only the last tile of the map can be partial
                            // candidate t*32 + tile_row(v, h) lies past the map; tested against one
                            // lane-dependent bound so that no per-register constants stay resident
                            const int bound = a.m - t * 32 - 4 * h;
#pragma unroll
                            for (int r = 0; r < R; ++r)
#pragma unroll
                                for (int v = 0; v < 16; ++v)
                                    if (tile_row(v, 0) >= bound) acc[r][v] = ninf;
                        }
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            const float top = fold16(best[g][r], acc[r]);
                            if (top > best[g][r]) best_tile[g][r] = t;
                            best[g][r] = top;
                        }
                    }
                }
            }
        }
    }

#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float ob = __shfl_xor(best[g][r], 32);
            const int ot = __shfl_xor(best_tile[g][r], 32);
            if (ob > best[g][r] || (ob == best[g][r] && ot < best_tile[g][r])) {
                best[g][r] = ob;
                best_tile[g][r] = ot;
            }
            const int slot = slot0 + (g * R + r) * 32 + c;
            if (h == 0 && slot < n_act) {
                const u64 key = pack_key(best[g][r], best_tile[g][r]);
                if (combine) atomicMax(&wg_keys[slot], key);
                else atomicMax(&a.out_keys[qbase + slot], key);
            }
        }
}

// Candidate tiles a wave keeps in flight when a pair has at most 32*R live queries (NB = blocks
// that hold one).  Such a search is bound by streaming the candidate map, not by arithmetic,
// and what limits a stream is the number of bytes on their way: the registers that the resident
// query blocks of the wide variants would occupy hold a longer ring instead.  Rows wider than
// 96 bytes keep the ordinary ring (their fragments leave no room).
template <int CT, int DP, int NB>
constexpr int stream_ring() {
    constexpr int frag_regs = Ops<CT, DP>::ROW_BYTES / 8;
    constexpr int fit = (NB <= 2 ? 96 : 72) / frag_regs;
    constexpr int base = Ops<CT, DP>::ROW_BYTES > 128 ? 2 : SEARCH_P;
    return frag_regs > 12 ? base : (fit > 16 ? 16 : (fit < base ? base : fit));
}

// Candidate tiles in flight: rows wider than 128 bytes (the two-term fp16 representation) take
// a shorter ring so that ring, query fragments and accumulators still fit the register file.
template <int CT, int DP>
constexpr int search_ring() {
    return Ops<CT, DP>::ROW_BYTES > 128 ? 2 : SEARCH_P;
}
template <int CT, int DP>
constexpr int search_g_limit() {
    // a query fragment is ROW_BYTES / 8 registers per lane and G*R of them are resident
    constexpr int frag_regs = Ops<CT, DP>::ROW_BYTES / 8;
    return frag_regs <= 6 ? 4 : (frag_regs <= 12 ? 2 : 1);
}

// Pass 2: one wave per query recomputes the 32 scores of the winning tile with the same
// matrix instruction (the query replicated into every column, so each score has the bits
// pass 1 saw) and picks the lowest candidate that attains the maximum.
template <int CT, int DP>
__device__ __forceinline__ Resolved resolve_tile(const SearchArgs& a, const char* tgt, u64 key, const typename Ops<CT, DP>::Frag& qf,
                                                 int c, int h) {
    using O = Ops<CT, DP>;
    const int tile = max(0, min(key_index(key), a.m_tiles - 1));
    const typename O::Frag cand = O::load(tgt + ((int64_t)tile * 32 + c) * O::ROW_BYTES, h);
    return lowest_at_maximum(O::mma(cand, qf), tile, a.m, h);
}

}  // namespace fnn
