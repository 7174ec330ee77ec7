// The whole FastNN iteration of one image pair in one workgroup (paper section 3.2.5, "FastNN
// Algorithm", steps 1-4), for pairs so small that the ordinary sequence -- four launches per
// iteration, enqueued for every iteration the caller allows -- is launches and nothing else: a 64x48
// pair with 48 seeds took 150 us at ten allowed iterations (43 launches at 2.5 us of host and 1.6 us
// of device time and up), of which its arithmetic is 2 us.  Here the searches of a pair follow one
// another behind workgroup barriers, and the loop really ends when no seed is left.
//
// What bounds it: the latency of a search (first tiles, LDS merge, winning tiles), then the
// arithmetic of the one compute unit that a pair occupies; walk_applies() says up to which size the host chooses it.
// The rows that a search finds stay in LDS as the next one's queries, and that one's first tiles are loaded meanwhile:
// 64x48 with 48 seeds 37.0 -> 32.1 us a call, and 46.7 -> 43.7 before that (another, slower machine) when one block of queries is multiplied alone.
#include "fnn_device.hpp"
#include "fnn_kernels.hpp"
#include "trace.hpp"

namespace fnn {

constexpr int WALK_WAVES = 16;
constexpr int WALK_THREADS = WALK_WAVES * 64;
constexpr int WALK_MAX_SEEDS = 96;  // see walk_applies()
static_assert(WALK_MAX_SEEDS <= WALK_THREADS, "the compaction handles one slot per thread");

// Query blocks R that a wave multiplies with each loaded tile, tiles it keeps in flight and queries that it resolves at a
// time: 128 registers (four waves per SIMD) hold the query fragments, the results and the ring.  Two blocks share
// a tile's load; one block alone (at most 32 live seeds) is half the products, leaves room for a longer ring, and
// its 32 queries are two for each wave.
template <int CT, int DP, int R>
struct WalkShape {
    static constexpr int FRAG_REGS = Ops<CT, DP>::ROW_BYTES / 8;
    static constexpr int P = FRAG_REGS <= 6 ? (R == 1 ? 6 : 4) : 2;
    static constexpr bool AHEAD = FRAG_REGS <= 12;  // a search's first tiles are loaded while the one before it ends
    static constexpr int Q = FRAG_REGS <= 8 ? 2 : 1;  // (four at a time spill beside the ring)
};
template <int CT, int DP>
constexpr int walk_blocks() { return Ops<CT, DP>::ROW_BYTES / 8 <= 8 ? 2 : 1; }

// Row j of a prepared map as its fragments hold it, lane half h's half of it, into a row in LDS.
template <int CT, int DP>
__device__ __forceinline__ void store_row(char* row, int h, const typename Ops<CT, DP>::Frag& f) {
    using O = Ops<CT, DP>;
    if constexpr (O::ROW_BYTES == 48) {
        O::store_tile(row, 0, h, f);
    } else {
#pragma unroll
        for (int i = 0; i < O::NV; ++i) reinterpret_cast<uint4*>(row + h * O::LANE_BYTES)[i] = f.v[i];
    }
}

// How the 16 waves share a search: R query blocks against one chunk of the tiles each (never more units than waves).
template <int R>
struct WalkSplit {
    int m_tiles, groups, per_chunk, chunks;
    __device__ __forceinline__ WalkSplit(int m, int n_act) {
        m_tiles = (m + 31) / 32;
        groups = (n_act + 32 * R - 1) / (32 * R);
        chunks = max(1, WALK_WAVES / groups);
        per_chunk = (m_tiles + chunks - 1) / chunks;
        chunks = (m_tiles + per_chunk - 1) / per_chunk;
    }
};

// The first tiles of this wave's chunk.
template <int CT, int DP, int R>
struct WalkRing {
    static constexpr int P = WalkShape<CT, DP, R>::P;
    typename Ops<CT, DP>::Frag tile[P];
    __device__ __forceinline__ void fill(const char* tgt, int m, int n_act, int wave, int c, int h) {
        const WalkSplit<R> split(m, n_act);
        const int t0 = wave / split.groups * split.per_chunk, t1 = min(t0 + split.per_chunk, split.m_tiles);
#pragma unroll
        for (int p = 0; p < P; ++p)  // a wave without a chunk reads the last tile and drops it
            tile[p] = Ops<CT, DP>::stream_tile(tgt + (int64_t)max(min(t0 + p, t1 - 1), 0) * (32 * Ops<CT, DP>::ROW_BYTES), c, h);
    }
};

// Nearest candidate of every live slot: the query of a slot is row at[slot] (at: NULL, row `slot`) of `rows` in LDS, the answers
// go to found[slot], the candidates' rows to found_rows, also in LDS, where the next search finds its queries.
// Two passes as in the search of its own (search.hip): a unit of pass 1 is R query blocks against one
// chunk of the tiles, shared among the 16 waves and merged in LDS; pass 2 recomputes each query's
// winning tile, Q queries of a wave at a time so that their loads overlap.  (Tracking the candidate
// itself in pass 1 needs no second pass but 40 more vector instructions per product: 229 us instead
// of 142 us per call for a 128x96 pair with 192 seeds.)
// A search waits for two things from memory only, its first tiles and the winning ones, and the first tiles are asked for
// while the search before it names its winners (`next`, or NULL).  `keys` are empty on entry; next_keys are emptied.
template <int CT, int DP, int R>
__device__ __forceinline__ void walk_search(const char* rows, const int32_t* at, const char* tgt, int m, int n_act, u64* keys, int32_t* found,
                                            char* found_rows, WalkRing<CT, DP, R>& ring, u64* next_keys, const char* next, int next_m) {
    using O = Ops<CT, DP>;
    using Frag = typename O::Frag;
    constexpr int P = WalkShape<CT, DP, R>::P, Q = WalkShape<CT, DP, R>::Q;
    const int lane = threadIdx.x & 63, c = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const float ninf = -__builtin_inff();
    for (int s = threadIdx.x; s < n_act; s += WALK_THREADS) next_keys[s] = 0;

    auto query = [&](int slot) {  // slots past the last live one repeat it; their results are dropped
        const int s = min(slot, n_act - 1);
        return O::load(rows + (at ? at[s] : s) * O::ROW_BYTES, h);
    };
    const WalkSplit<R> split(m, n_act);
    const int m_tiles = split.m_tiles;
    if constexpr (!WalkShape<CT, DP, R>::AHEAD) ring.fill(tgt, m, n_act, wave, c, h);
    if (wave < split.groups * split.chunks) {
        const int slot0 = wave % split.groups * (32 * R);
        const int t0 = wave / split.groups * split.per_chunk, t1 = min(t0 + split.per_chunk, m_tiles);
        Frag q[R];
        float best[R];
        int best_tile[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            q[r] = query(slot0 + r * 32 + c);
            best[r] = ninf;
            best_tile[r] = 0x7FFFFFFF;
        }
        for (int tb = t0; tb < t1; tb += P) {
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const int t = tb + p;
                if (__builtin_expect(t < t1, 1)) {  // uniform
                    const Frag cur = ring.tile[p];
                    ring.tile[p] = O::stream_tile(tgt + (int64_t)min(t + P, t1 - 1) * (32 * O::ROW_BYTES), c, h);
                    f32x16 acc[R];
#pragma unroll
                    for (int r = 0; r < R; ++r) acc[r] = O::mma(cur, q[r]);
                    if (__builtin_expect(t * 32 + 32 > m, 0)) {  // only the last tile of the map can be partial
                        const int bound = m - t * 32 - 4 * h;
#pragma unroll
                        for (int r = 0; r < R; ++r)
#pragma unroll
                            for (int v = 0; v < 16; ++v)
                                if (tile_row(v, 0) >= bound) acc[r][v] = ninf;
                    }
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const float top = fold16(best[r], acc[r]);
                        if (top > best[r]) best_tile[r] = t;  // strictly: the lowest tile wins among equal scores
                        best[r] = top;
                    }
                }
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float ob = __shfl_xor(best[r], 32);
            const int ot = __shfl_xor(best_tile[r], 32);
            if (ob > best[r] || (ob == best[r] && ot < best_tile[r])) {
                best[r] = ob;
                best_tile[r] = ot;
            }
            const int slot = slot0 + r * 32 + c;
            if (h == 0 && slot < n_act) atomicMax(&keys[slot], pack_key(best[r], best_tile[r]));
        }
    }
    if (WalkShape<CT, DP, R>::AHEAD && next) ring.fill(next, next_m, n_act, wave, c, h);
    __syncthreads();
    for (int s0 = wave * Q; s0 < n_act; s0 += WALK_WAVES * Q) {
        Frag q[Q], cand[Q];
        int tile[Q];
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            tile[i] = min(key_index(keys[min(s0 + i, n_act - 1)]), m_tiles - 1);
            q[i] = query(s0 + i);
            cand[i] = O::load(tgt + ((int64_t)tile[i] * 32 + c) * O::ROW_BYTES, h);
        }
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const int j = lowest_at_maximum(O::mma(cand[i], q[i]), tile[i], m, h).idx;
            if (s0 + i < n_act) {
                if (lane == 0) found[s0 + i] = j;
                if (c == (j & 31)) store_row<CT, DP>(found_rows + (s0 + i) * O::ROW_BYTES, h, cand[i]);
            }
        }
    }
    __syncthreads();
}

// The seeds' rows of image 1, one thread per 8 bytes, and their indices.
template <int CT, int DP>
__device__ __forceinline__ void walk_start(const WalkArgs& a, const int32_t* seeds, const char* p1, int n_act, int32_t* u, int32_t* at, u64* keys, char* rows) {
    constexpr int ROW_BYTES = Ops<CT, DP>::ROW_BYTES, WORDS = ROW_BYTES / 8;
    for (int i = threadIdx.x; i < n_act * WORDS; i += WALK_THREADS) {
        const int slot = i / WORDS, word = i % WORDS;
        const int32_t seed = seeds[slot];
        const int64_t row = min(max(seed, 0), a.rows1 - 1);
        reinterpret_cast<uint2*>(rows + slot * ROW_BYTES)[word] = reinterpret_cast<const uint2*>(p1 + row * ROW_BYTES)[word];
        if (word == 0) {
            u[slot] = seed;
            at[slot] = slot;
            keys[slot] = 0;
        }
    }
}

// LDS (dynamic): two key tables [n_seeds], then u, v, w (U^t, V^t, U^{t+1}), the seed number and the place of its row per slot,
// the bitmap of the matched pixels of image 1 and the rank of each of its words, and the rows of V^t and U^{t+1}.
template <int CT, int DP>
__global__ __launch_bounds__(WALK_THREADS) void recip_walk_kernel(WalkArgs a) {
    using O = Ops<CT, DP>;
    extern __shared__ uint4 walk_lds[];
    __shared__ int wave_sums[17];
    char* w_rows = reinterpret_cast<char*>(walk_lds);  // whole rows of 16 bytes and more first
    char* v_rows = w_rows + a.n_seeds * O::ROW_BYTES;
    u64* keys_f = reinterpret_cast<u64*>(v_rows + a.n_seeds * O::ROW_BYTES);
    u64* keys_b = keys_f + a.n_seeds;
    int32_t* u = reinterpret_cast<int32_t*>(keys_b + a.n_seeds);
    int32_t* v = u + a.n_seeds;
    int32_t* w = v + a.n_seeds;
    int32_t* sid = w + a.n_seeds;
    int32_t* at = sid + a.n_seeds;
    uint32_t* bitmap = reinterpret_cast<uint32_t*>(at + a.n_seeds);
    int32_t* word_rank = reinterpret_cast<int32_t*>(bitmap + a.n_words);
    const int b = blockIdx.x, me = threadIdx.x;
    const int lane = me & 63, c = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(me >> 6);
    const int64_t base = (int64_t)b * a.n_seeds;
    const char* p1 = a.p1 + (int64_t)b * a.bstride1;
    const char* p2 = a.p2 + (int64_t)b * a.bstride2;

    int n_act = a.n_seeds;
    walk_start<CT, DP>(a, a.seeds + base, p1, n_act, u, at, keys_f, w_rows);
    if (me < n_act) sid[me] = me;
    for (int i = me; i < a.n_words; i += WALK_THREADS) bitmap[i] = 0;
    __syncthreads();

    auto step = [&](int t) {
        const bool last = t + 1 >= a.max_iter;
        bool survive = false;
        int32_t u_next = 0, my_sid = 0;
        if (me < n_act) {
            my_sid = sid[me];
            u_next = w[me];
            const bool converged = u_next == u[me];
            survive = !converged && !last;
            if (!survive) {
                a.seed_i[base + my_sid] = u[me];
                a.seed_j[base + my_sid] = v[me];
                a.seed_iter[base + my_sid] = converged ? t : -1;
                if (converged) atomicOr(&bitmap[(uint32_t)u_next >> 5], 1u << (u_next & 31));
            }
        }
        int kept;
        const int pos = block_scan_flag(survive, wave_sums, kept);  // its barriers also end the reads of u and sid above
        if (survive) {
            u[pos] = u_next;
            sid[pos] = my_sid;
            at[pos] = me;
        }
        n_act = kept;  // 0 after max_iter trips at the latest
        __syncthreads();
    };
    constexpr int R = walk_blocks<CT, DP>();
    int t = 0;
    if constexpr (R > 1) {
        for (; n_act > 32; ++t) {
            WalkRing<CT, DP, R> ring;
            ring.fill(p2, a.m, n_act, wave, c, h);
            walk_search<CT, DP, R>(w_rows, at, p2, a.m, n_act, keys_f, v, v_rows, ring, keys_b, p1, a.n);     // V^t = NN_2(U^t)
            walk_search<CT, DP, R>(v_rows, nullptr, p1, a.n, n_act, keys_b, w, w_rows, ring, keys_f, nullptr, 0);  // U^{t+1} = NN_1(V^t)
            step(t);
        }
    }
    if (n_act > 0) {
        WalkRing<CT, DP, 1> ring;
        ring.fill(p2, a.m, n_act, wave, c, h);
        for (; n_act > 0; ++t) {
            walk_search<CT, DP, 1>(w_rows, at, p2, a.m, n_act, keys_f, v, v_rows, ring, keys_b, p1, a.n);
            walk_search<CT, DP, 1>(v_rows, nullptr, p1, a.n, n_act, keys_b, w, w_rows, ring, keys_f, p2, a.m);
            step(t);
        }
    }

    // step 4: the matches as a set, sorted (see recip_dedup_kernel).  A converged seed's pixels are
    // read back from the outputs by the thread that handles the seed.
    __threadfence_block();
    __syncthreads();
    const int per_thread = (a.n_words + WALK_THREADS - 1) / WALK_THREADS;
    const int w0 = min(me * per_thread, a.n_words), w1 = min(w0 + per_thread, a.n_words);
    int mine = 0;
    for (int i = w0; i < w1; ++i) mine += __popc(bitmap[i]);
    int count;
    int rank = block_scan_int(mine, wave_sums, count);
    for (int i = w0; i < w1; ++i) {
        word_rank[i] = rank;
        rank += __popc(bitmap[i]);
    }
    __syncthreads();
    if (me < a.n_seeds && a.seed_iter[base + me] >= 0) {
        const uint32_t i = (uint32_t)a.seed_i[base + me];
        const int pos = word_rank[i >> 5] + __popc(bitmap[i >> 5] & ((1u << (i & 31)) - 1u));
        a.pairs[(base + pos) * 2 + 0] = (int32_t)i;
        a.pairs[(base + pos) * 2 + 1] = a.seed_j[base + me];
    }
    if (me >= count && me < a.n_seeds) {
        a.pairs[(base + me) * 2 + 0] = -1;
        a.pairs[(base + me) * 2 + 1] = -1;
    }
    if (me == 0) a.n_pairs[b] = count;
}

// The same walk with a workgroup for every 32 seeds of a pair: seeds do not meet before the final sort, which is
// recip_dedup_kernel's here.  A group sweeps the whole map on its own compute unit, so this is for small maps
// (groups_apply()), where the searches of the ordinary sequence are launches and latency too.
constexpr int GROUP_SEEDS = 32;
template <int CT, int DP>
__global__ __launch_bounds__(WALK_THREADS) void recip_groups_kernel(WalkArgs a) {
    using O = Ops<CT, DP>;
    __shared__ __attribute__((aligned(16))) char v_rows[GROUP_SEEDS * O::ROW_BYTES], w_rows[GROUP_SEEDS * O::ROW_BYTES];
    __shared__ u64 keys_f[GROUP_SEEDS], keys_b[GROUP_SEEDS];
    __shared__ int32_t u[GROUP_SEEDS], v[GROUP_SEEDS], w[GROUP_SEEDS], sid[GROUP_SEEDS], at[GROUP_SEEDS];  // as in recip_walk_kernel
    __shared__ int live;
    const int b = blockIdx.y, first = blockIdx.x * GROUP_SEEDS, me = threadIdx.x;
    const int lane = me & 63, c = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(me >> 6);
    const int64_t base = (int64_t)b * a.n_seeds;
    const char* p1 = a.p1 + (int64_t)b * a.bstride1;
    const char* p2 = a.p2 + (int64_t)b * a.bstride2;

    int n_act = min(GROUP_SEEDS, a.n_seeds - first);
    WalkRing<CT, DP, 1> ring;
    ring.fill(p2, a.m, n_act, wave, c, h);
    walk_start<CT, DP>(a, a.seeds + base + first, p1, n_act, u, at, keys_f, w_rows);
    if (me < n_act) sid[me] = first + me;
    __syncthreads();
    for (int t = 0; n_act > 0; ++t) {  // uniform; 0 after max_iter trips at the latest
        walk_search<CT, DP, 1>(w_rows, at, p2, a.m, n_act, keys_f, v, v_rows, ring, keys_b, p1, a.n);     // V^t = NN_2(U^t)
        walk_search<CT, DP, 1>(v_rows, nullptr, p1, a.n, n_act, keys_b, w, w_rows, ring, keys_f, p2, a.m);  // U^{t+1} = NN_1(V^t)
        if (me < 64) {  // the first wave; all of its reads come before its writes
            const bool last = t + 1 >= a.max_iter;
            bool survive = false;
            int32_t u_next = 0, my_sid = 0;
            if (me < n_act) {
                my_sid = sid[me];
                u_next = w[me];
                const bool converged = u_next == u[me];
                survive = !converged && !last;
                if (!survive) {
                    a.seed_i[base + my_sid] = u[me];
                    a.seed_j[base + my_sid] = v[me];
                    a.seed_iter[base + my_sid] = converged ? t : -1;
                }
            }
            const u64 stay = __ballot(survive);
            if (survive) {
                const int pos = __popcll(stay & ((1ull << me) - 1ull));
                u[pos] = u_next;
                sid[pos] = my_sid;
                at[pos] = me;
            }
            if (me == 0) live = __popcll(stay);
        }
        __syncthreads();
        n_act = live;  // written again behind the barriers of the next searches
    }
}

static size_t walk_lds_bytes(int64_t n, int64_t n_seeds, int row_bytes) {
    return (size_t)n_seeds * (2 * row_bytes + 2 * sizeof(u64) + 5 * sizeof(int32_t)) + (size_t)((n + 31) / 32) * 2 * sizeof(int32_t);
}

// Where one workgroup per pair is no slower than the launch sequence, however long the seeds keep
// moving.  Both sides in microseconds per call, one pair, fp16, 24 channels: a call of the walk takes 10, and
// every iteration with live seeds 8 + 2.1 per block of 32 seeds + 0.018 per product of 32x32 scores and
// search (query blocks are multiplied in twos); an iteration without live seeds takes nothing.  The sequence took 13 + 18
// (one or two blocks) to 21 for every allowed iteration when the walk came, 13 + 16 to 18 now.  With
// every seed live for all ten allowed iterations, and with all of them settled in the first:
//     1 block  x 175 tiles  walk 161 / 23, sequence 159 / 151 (before the walk: 186 / 189)
//     2 blocks x 175 tiles  walk 182 / 26, sequence 176 / 155 (195 / 192)
//     3 blocks x  87 tiles  walk 196 / 27, sequence 190 / 154 (214 / 193)
//     8 blocks x  64 tiles  walk 343 / 42, sequence 189 / 154 (222 / 187): past the line
//    31 blocks x  31 tiles  walk 940 / 103, sequence 195 / 152 (231 / 191): past the line
// A fragment of 32 channels takes half as much again per product (2 blocks x 120 tiles: 184 against 199 before).
// Wide rows and fp32 products leave room for one block at a time (96 channels, 24 tiles: 210 against 236;
// fp32 products of 32 channels: 266 against 286; two blocks x 2 tiles: 303 against 223).
// The 64x48 pair with 48 seeds (2 blocks x 96 tiles) takes 23 to 154 against 189 to 194.  With a few allowed
// iterations the sequence is short as well: at most 100 products for each.
// Those are figures of the sequence in launches.  With its late iterations in one launch (what it takes with a workspace of fnn_workspace_bytes()) it is
// the faster one beyond some 60 tiles.  Walk / sequence, replayed from a graph, settled at once and live for all ten iterations:
//     30 seeds   16 tiles  22 / 24,  92 / 98    64  24 / 25, 107 / 104    96  25 / 25, 116 / 102    175  28 / 25, 140 / 106
//     60 seeds   32 tiles  24 / 25, 113 / 105   64  25 / 25, 124 / 106    96  26 / 25, 136 / 106    175  30 / 26, 165 / 113
//     90 seeds   32 tiles  27 / 26              64  30 / 27, 168 / 124    87  31 / 27, 186 / 121
//     60 seeds, 32 channels, 64 tiles  26 / 25, 134 / 104    96  28 / 25, 152 / 105    120  29 / 25, 165 / 108
// The line still is the one against launches: on this side of it up to 14 % is given away where seeds settle and up to half where none ever does.
bool walk_applies(int64_t n, int64_t m, int64_t n_seeds, int32_t max_iter, int compute, int dp) {
    if (n_seeds < 1 || n_seeds > WALK_MAX_SEEDS || n < 1 || m < 1) return false;
    const int64_t blocks = (n_seeds + 31) / 32, tiles = ((n > m ? n : m) + 31) / 32;
    const bool costly = compute == FNN_F32 || dp > 32;
    if (blocks * tiles * (costly ? 5 : 1) > 100 * (int64_t)max_iter) return false;
    if (costly) return blocks == 1 && tiles <= 24;
    return (blocks + 1) / 2 * 2 * tiles <= (dp > 24 ? 240 : 350);
}

// Where a workgroup per 32 seeds is no slower than the launch sequence, however long the seeds keep moving.  Microseconds per
// call (replayed from a graph, fp16, 24 channels), groups / sequence, with every seed live for all ten allowed iterations, for
// two, and with all of them settled in the first:
//     200 seeds, 1 pair     145 tiles  129 / 184,  40 / 48,  29 / 86    220 tiles  150 / 187,  44 / 48,  32 / 86    320 tiles  180 / 195,  51 / 49,  36 / 87
//     60 seeds, 4 pairs     210 tiles  147 / 171,  45 / 45,  32 / 85    320 tiles  179 / 174,  52 / 46,  36 / 85
//     256 seeds, 32 pairs   145 tiles  191 / 284,  62 / 69,  46 / 104   220 tiles  251 / 293,  75 / 74,  55 / 109
// and with 32 channels
//     200 seeds, 1 pair     145 tiles  151 / 190,  43 / 49,  30 / 87    210 tiles  186 / 193,  51 / 49,  34 / 88
//     256 seeds, 32 pairs   145 tiles  227 / 305,  68 / 75,  50 / 108
// Those are figures of the sequence in launches.  With its late iterations in one launch it takes the same whatever the number of blocks while they are few, and
// (groups / sequence, settled at once, live for three and for all ten iterations)
//     200 seeds, 1 pair     145 tiles  29 / 31,  63 / 76,  130 / 166    224 tiles  32 / 33,  72 / 81,  151 / 176    280 tiles  34 / 34,  79 / 85,  169 / 186
//     120 seeds, 1 pair     180 tiles  30 / 28,  66 / 62,  138 / 130    224 tiles  31 / 28,  71 / 64,  150 / 135    280 tiles  34 / 29,  78 / 68,  168 / 144
//     60 seeds, 4 pairs     180 tiles  30 / 27,  67 / 56,  138 / 114    210 tiles  32 / 27,  70 / 56,  148 / 114    280 tiles  34 / 28,  79 / 58,  168 / 119
//     200 seeds, 4 pairs    145 tiles  29 / 33,  63 / 78,  130 / 169    210 tiles  32 / 34,  71 / 82,  149 / 179    280 tiles  36 / 36,  81 / 89,  170 / 194
//     256 seeds, 32 pairs   100 tiles  41 / 42,  82 / 96,  157 / 204    145 tiles  46 / 45, 101 / 105, 207 / 225    210 tiles  54 / 51, 128 / 119, 272 / 253
// and with 32 channels
//     200 seeds, 1 pair     145 tiles  30 / 31,  71 / 75,  151 / 162    180 tiles  32 / 32,  78 / 78,  170 / 169
//     60 seeds, 4 pairs     145 tiles  30 / 26,  71 / 54,  151 / 110    180 tiles  32 / 27,  78 / 55,  170 / 113
//     256 seeds, 32 pairs   100 tiles  41 / 42,  90 / 96,  187 / 202    145 tiles  50 / 48, 120 / 108, 259 / 229
// So the lines hold for pairs of 200 seeds and more (of many pairs within 8 %, with 32 channels 13 %); with 120 seeds and fewer the sequence is faster well before
// them, by up to a fifth where seeds settle and up to half where none does.
// A full chip sweeps a tile at two thirds of the speed of a quarter of it, and more than one workgroup per compute unit would walk
// in turns.  fp32 products and two-term rows take several times as long per tile.  Past 256 seeds, and on maps that need no prepared
// copy, the sequence runs as before.
bool groups_apply(int64_t n, int64_t m, int64_t n_seeds, int batch, int32_t max_iter, int compute, int dp) {
    if (n_seeds < 1 || n_seeds > 256 || n < 1 || m < 1 || max_iter < 1 || compute == FNN_F32 || dp > 32) return false;
    const int64_t groups = (n_seeds + GROUP_SEEDS - 1) / GROUP_SEEDS * batch, tiles = ((n > m ? n : m) + 31) / 32;
    if (groups > 256) return false;
    if (groups > 64) return tiles <= (dp > 24 ? 145 : 210);
    return tiles <= (dp > 24 ? 180 : 280);
}
template <int CT, int DP>
static hipError_t launch_groups_t(const WalkArgs& a, int batch, hipStream_t s) {
    const unsigned groups = (a.n_seeds + GROUP_SEEDS - 1) / GROUP_SEEDS;
    return launch(TK_RECIP_GROUPS, recip_groups_kernel<CT, DP>, dim3(groups, batch), dim3(WALK_THREADS), 0, s, a);
}
hipError_t launch_groups(const WalkArgs& a, int batch, int compute, int dp, hipStream_t s) {
    if (compute == FNN_F16) {
        if (dp == 16) return launch_groups_t<CT_F16, 16>(a, batch, s);
        if (dp == 24) return launch_groups_t<CT_F16, 24>(a, batch, s);
        if (dp == 32) return launch_groups_t<CT_F16, 32>(a, batch, s);
    } else if (compute == FNN_BF16) {
        if (dp == 16) return launch_groups_t<CT_BF16, 16>(a, batch, s);
        if (dp == 24) return launch_groups_t<CT_BF16, 24>(a, batch, s);
        if (dp == 32) return launch_groups_t<CT_BF16, 32>(a, batch, s);
    }
    return hipErrorInvalidValue;
}

template <int CT, int DP>
static hipError_t launch_walk_t(const WalkArgs& a, int batch, hipStream_t s) {
    return launch(TK_RECIP_WALK, recip_walk_kernel<CT, DP>, dim3(batch), dim3(WALK_THREADS), walk_lds_bytes(a.n, a.n_seeds, Ops<CT, DP>::ROW_BYTES), s, a);
}

hipError_t launch_walk(const WalkArgs& a, int batch, int compute, int dp, hipStream_t s) {
    if (compute == FNN_F16) {
        if (dp == 16) return launch_walk_t<CT_F16, 16>(a, batch, s);
        if (dp == 24) return launch_walk_t<CT_F16, 24>(a, batch, s);
        if (dp == 32) return launch_walk_t<CT_F16, 32>(a, batch, s);
        if (dp == 48) return launch_walk_t<CT_F16, 48>(a, batch, s);
        if (dp == 64) return launch_walk_t<CT_F16, 64>(a, batch, s);
        if (dp == 80) return launch_walk_t<CT_F16, 80>(a, batch, s);
        if (dp == 96) return launch_walk_t<CT_F16, 96>(a, batch, s);
    } else if (compute == FNN_BF16) {
        if (dp == 16) return launch_walk_t<CT_BF16, 16>(a, batch, s);
        if (dp == 24) return launch_walk_t<CT_BF16, 24>(a, batch, s);
        if (dp == 32) return launch_walk_t<CT_BF16, 32>(a, batch, s);
    } else {
        if (dp == 8) return launch_walk_t<CT_F32, 8>(a, batch, s);
        if (dp == 16) return launch_walk_t<CT_F32, 16>(a, batch, s);
        if (dp == 24) return launch_walk_t<CT_F32, 24>(a, batch, s);
        if (dp == 32) return launch_walk_t<CT_F32, 32>(a, batch, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace fnn
