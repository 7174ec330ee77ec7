// The late iterations of a FastNN walk (paper section 3.2.5, steps 2-3) in one launch.
//
// From the third iteration on a handful of seeds still move, and what an iteration costs is its four launches: with ten
// allowed iterations 24 to 28 of them found no seed left (1.5 us each), and a search of a hundred queries or fewer took 12 to 16 us with
// its resolve pass.  Here a group of workgroups takes a pair of images through all iterations that are left; between the steps
// they meet at a barrier of their own (1.7 us among 256 workgroups, bare), and the launch ends when no seed is left.
//
// While many seeds move (more than TAIL_FEW), an iteration has the four steps of the launches.  A few of them every workgroup
// keeps in its own LDS, all the same; its waves name the candidates themselves, not the tiles that hold them, so a search needs no resolve pass, and what
// the workgroups hand each other is one key per query: a barrier for each search.
//
// Who takes part.  A workgroup announces itself when it starts, and a search of many seeds is dealt to those that had done so when it began; the
// first search of few seeds fixes who takes part in the rest, and who comes later leaves.  Nobody waits for a workgroup that is not running yet, so it
// does not matter how many of them the device holds at once, or what else it is running: one workgroup alone would walk to the end.
//
// What the workgroups hand each other is read and written with relaxed atomics of device scope only, which pass the caches that are not
// shared; a workgroup waits until its stores have arrived (s_waitcnt) before it reports.  There is no fence: on this part one writes
// back an XCD's whole L2.  The language does not promise that this is enough; it rests on three properties of gfx950 and its compiler:
//   - such a load or store is an instruction with the sc1 bit, and such a read-modify-write is performed for the whole device, so each acts where all XCDs see
//     it (tests/test_kernel_scratch.py looks for the bit in the built kernels: a plain access is one of a map or of a final result);
//   - s_waitcnt with all counts at 0 returns when the wave's earlier stores and read-modify-writes have acted, and the compiler moves no access over the
//     empty asm statements on either side of it;
//   - a wave issues its loads in the order of the program, and none ahead of the s_barrier behind which its workgroup's word has been seen.
#include "fnn_device.hpp"
#include "fnn_kernels.hpp"
#include "search_unit.hpp"
#include "trace.hpp"

namespace fnn {

namespace {

template <typename T>
__device__ __forceinline__ T shared_load(const T* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T>
__device__ __forceinline__ void shared_store(T* p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ uint32_t shared_add(uint32_t* p, uint32_t v) {
    return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Every store and atomic of this wave has arrived where the other XCDs see it.
__device__ __forceinline__ void stores_arrived() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0);
    asm volatile("" ::: "memory");
}

// What the takers of a phase read: its number (phase & 3: search forward, its resolve pass, search back, its resolve pass with the
// bookkeeping), how many they are, and the live seeds.  No live seeds: the walk has ended.  0: not begun.
struct Phase {
    uint32_t number, takers, live;
    __device__ __forceinline__ static u64 pack(uint32_t number, uint32_t takers, uint32_t live) {
        return (u64)number << 42 | (u64)takers << 32 | live;
    }
    __device__ __forceinline__ explicit Phase(u64 w) : number((uint32_t)(w >> 42)), takers((uint32_t)(w >> 32) & 1023u), live((uint32_t)w) {}
};
static_assert(TAIL_MOST_WGS < 1024 && TAIL_MOST_ITERATIONS <= (1 << 22) / 4, "the fields of a phase word");

}  // namespace

constexpr int TAIL_WAVES = 8;    // two for every SIMD
constexpr int TAIL_THREADS = TAIL_WAVES * 64;
static_assert(TAIL_FEW == TAIL_THREADS, "a thread for each of few seeds");
constexpr int TAIL_ROUND = 256;  // queries that a workgroup resolves before it hands its moving seeds on


// Pass 1 of few queries with the candidates named: R blocks of queries, rows at[slot] of `src` from slot0 on, against the tiles [t0, t1).
// A lane keeps the 16 scores of its query's best tile (16 moves, where any lane of the wave has found a better one), and looks for
// the candidate when the last one is done.  Scores count from low[slot] on, which some candidate exceeds.  The keys are those that the resolve pass would leave, also where no score is more than minus infinity (the first such
// in the last tile of the map) or none is a number (the last pixel).  Bound by latency: the
// queries' rows, the tiles.  (Keeping the tile, and multiplying it again for every query of the workgroup, as a variant of this kernel: 512x384 193 -> 215 us, squared
// distance of two pairs 312 -> 336, 16 pairs 1251 -> 1249; both ways in one kernel spilled and were slower than either.)
template <int CT, int DP, int R, int P>
__device__ __forceinline__ void named_unit(const int32_t* at, const char* src, int src_rows, const char* tgt, int n_act, int slot0, int t0, int t1, int m, const float* low,
                                           u64* keys, int c, int h) {
    using O = Ops<CT, DP>;
    using Frag = typename O::Frag;
    const float ninf = -__builtin_inff();
    const int last = (m - 1) / 32;
    asm volatile("" : "+v"(c), "+v"(h));  // else what hangs on the lane is kept from search to search, and spills the tiles
    Frag ring[P];
#pragma unroll
    for (int p = 0; p < P; ++p)
        if (p == 0 || t0 + p < t1) ring[p] = O::stream_tile(tgt + (int64_t)(t0 + p) * (32 * O::ROW_BYTES), c, h);  // uniform
    Frag q[R];
    float best[R], least[R];
    int best_tile[R];
    f32x16 kept[R];
#pragma unroll
    for (int r = 0; r < R; ++r) q[r] = O::load(src + (int64_t)min(max(at[min(slot0 + r * 32 + c, n_act - 1)], 0), src_rows - 1) * O::ROW_BYTES, h);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        arrived(q[r]);
        best[r] = least[r] = low[min(slot0 + r * 32 + c, n_act - 1)];
        best_tile[r] = last;
#pragma unroll
        for (int v = 0; v < 16; ++v) kept[r][v] = 0.0f;
    }
    for (int tb = t0; tb < t1; tb += P) {
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const int t = tb + p;
            if (__builtin_expect(t < t1, 1)) {  // uniform
                const Frag cur = ring[p];
                if (t + P < t1) ring[p] = O::stream_tile(tgt + (int64_t)(t + P) * (32 * O::ROW_BYTES), c, h);
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
                    const bool rose = top > best[r];  // strictly: the lowest tile wins among equal scores
                    if (__any(rose)) {
                        best_tile[r] = rose ? t : best_tile[r];
#pragma unroll
                        for (int v = 0; v < 16; ++v) kept[r][v] = rose ? acc[r][v] : kept[r][v];
                        best[r] = top;
                    }
                }
            }
        }
    }
    // Where no score was more than minus infinity, the last tile of the map stands for them all.  (Kept in the loop, in each of the ring's places, that makes the
    // kernel 63 KB of code instead of 55.)
    if (t1 > last) {  // uniform
        bool none = false;
#pragma unroll
        for (int r = 0; r < R; ++r) none = none || best[r] == ninf;
        if (__builtin_expect(__any(none), 0)) {
            const Frag tile = O::stream_tile(tgt + (int64_t)last * (32 * O::ROW_BYTES), c, h);
            const int bound = m - last * 32 - 4 * h;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const f32x16 x = O::mma(tile, q[r]);
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (best[r] == ninf) kept[r][v] = tile_row(v, 0) >= bound ? ninf : x[v];
            }
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        int row = 64;
#pragma unroll
        for (int v = 15; v >= 0; --v)
            if (kept[r][v] == best[r]) row = tile_row(v, h);
        const u64 key = pack_key(best[r], min(best_tile[r] * 32 + row, m - 1));
        const u64 least_key = least[r] == ninf ? 0 : (u64)order_bits(least[r]) << 32 | 0xFFFFFFFFu;  // nothing above the bound: not a candidate of this unit
        const u64 other = shfl_xor_u64(key, 32);
        const int slot = slot0 + r * 32 + c;
        const u64 most = other > key ? other : key;
        if (h == 0 && slot < n_act && most > least_key) atomicMax(&keys[slot], most);
    }
}
template <int CT, int DP, int R>
constexpr int named_ring() {
    constexpr int frag_regs = Ops<CT, DP>::ROW_BYTES / 8, fit = (R == 2 ? 36 : 60) / frag_regs;
    return fit > 12 ? 12 : (fit < 2 ? 2 : fit);
}

// grid: workgroups of a pair, pairs.
template <int CT, int DP, int G>
__global__ __launch_bounds__(TAIL_THREADS) __attribute__((amdgpu_waves_per_eu(2)))
void recip_tail_kernel(TailArgs ta) {
    using O = Ops<CT, DP>;
    constexpr int R = SEARCH_R, P = search_ring<CT, DP>();
    __shared__ u64 published;
    __shared__ int2 moving[TAIL_ROUND];  // (U^{t+1}, seed number)
    __shared__ int n_moving, first_pos;
    __shared__ uint32_t my_id, lost;
    // few seeds: U^t and V^t, the seed number of every slot, and the keys of a search
    __shared__ int32_t few_at[2][TAIL_FEW], few_sid[TAIL_FEW];
    __shared__ u64 few_keys[TAIL_FEW];
    __shared__ float few_low[TAIL_FEW];
    __shared__ int wave_sums[17];
    const int lane = threadIdx.x & 63, c = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int b = blockIdx.y;
    const int64_t base = (int64_t)b * ta.n_seeds;
    const uint32_t n_first = (uint32_t)min(max(ta.n_active[b], 0), ta.n_seeds);
    // (beside a thousand seeds and fewer the others would cost the barriers more than they take off the searches: one 640x480 pair 371 -> 376 us)
    const uint32_t most = n_first <= 2 * (uint32_t)TAIL_FEW ? ta.few_wgs : gridDim.x;
    if (n_first == 0 || blockIdx.x >= most) return;
    TailControl& ctl = ta.control[b];
    const char* p1 = ta.p1 + (int64_t)b * ta.bstride1;
    const char* p2 = ta.p2 + (int64_t)b * ta.bstride2;

    auto publish = [&](u64 word) {  // by lanes 0..15 of a wave
        if (lane < TAIL_COPIES) shared_store(&ctl.phase[lane].word, word);
    };
    if (wave == 0) {
        uint32_t id = 0;
        if (lane == 0) id = shared_add(&ctl.registered, 1u);
        id = __builtin_amdgcn_readfirstlane(id);
        if (lane == 0) my_id = id;
        if (lane == 0) lost = 0;
        if (id == 0) {
            // the first to come opens the first search; it gives the others a few microseconds to appear, and some more while they are few
            uint32_t takers = 1;
            for (int i = 0; i < 64 && (takers < most / 4 || (i < 8 && takers < most)); ++i) {
                uint32_t seen = 0;
                if (lane == 0) seen = shared_load(&ctl.registered);
                takers = __builtin_amdgcn_readfirstlane(seen);
            }
            publish(Phase::pack(0, min(max(takers, 1u), most), n_first));
        }
    }
    __syncthreads();
    const uint32_t id = my_id;

    // ---- many seeds ----
    u64 last = 0;
    for (;;) {  // ends when few are left: a phase waits for running workgroups only, and every four phases are an iteration
        if (threadIdx.x == 0) {
            u64 word;
            uint64_t polls = 0;
            while ((word = shared_load(&ctl.phase[id % TAIL_COPIES].word)) == last && ++polls < ta.most_polls) __builtin_amdgcn_s_sleep(1);
            published = word == last ? 0 : word;  // given up (see tail_most_polls): leave
        }
        __syncthreads();
        last = published;
        const Phase phase(last);
        if (phase.live == 0) return;               // uniform
        if (phase.live <= (uint32_t)TAIL_FEW) break;  // an iteration of few seeds begins (the words of one with many say so to its end)
        if (id >= phase.takers) {                  // came after this phase began
            __syncthreads();                       // `published` has been read by all
            continue;
        }
        const int kind = phase.number & 3, t = ta.t0 + (int)(phase.number >> 2), half = (ta.half + (int)(phase.number >> 2)) & 1;
        const bool forward = kind < 2;
        const int n_act = (int)min(phase.live, (uint32_t)ta.n_seeds);
        const int takers = (int)phase.takers;
        SearchArgs a;
        a.src_rows = forward ? ta.rows1 : ta.rows2;
        a.q_idx = forward ? ta.cur_u[half] : ta.v;
        a.q_keys = nullptr;
        a.nq = ta.n_seeds;
        a.m = forward ? ta.m : ta.n;
        a.m_tiles = (a.m + 31) / 32;
        a.out_keys = ta.keys;
        const char* src = forward ? p1 : p2;
        const char* tgt = forward ? p2 : p1;

        if ((kind & 1) == 0) {
            const int gw = (int)id * TAIL_WAVES + wave, n_waves = takers * TAIL_WAVES;
            // as in search_kernel
            const int row_groups = (n_act + 32 * R * G - 1) / (32 * R * G);
            int chunks = max(1, n_waves / row_groups);
            const int tiles_per_chunk = max((a.m_tiles + chunks - 1) / chunks, SEARCH_MIN_TILES);
            chunks = (a.m_tiles + tiles_per_chunk - 1) / tiles_per_chunk;
            const int64_t units = (int64_t)row_groups * chunks;
            for (int64_t unit = gw; unit < units; unit += n_waves) {
                const int chunk = (int)(unit / row_groups), slot0 = (int)(unit % row_groups) * 32 * R * G;
                const int tile0 = chunk * tiles_per_chunk, tile1 = min(tile0 + tiles_per_chunk, a.m_tiles);
                search_unit<CT, DP, R, P, G, false, true>(a, src, tgt, base, n_act, slot0, tile0, tile1, false, nullptr, c, h);
            }
        } else {
            // query k of this workgroup is slot id + k takers; wave k % TAIL_WAVES takes it
            const bool final_one = t + 1 >= ta.max_iter;
            const int mine = n_act > (int)id ? (n_act - (int)id - 1) / takers + 1 : 0;
            for (int round = 0; round < mine; round += TAIL_ROUND) {  // uniform in the workgroup
                if (threadIdx.x == 0) n_moving = 0;
                __syncthreads();
                const int end = min(mine, round + TAIL_ROUND);
                for (int k = round + wave; k < end; k += TAIL_WAVES) {  // uniform in the wave
                    const int64_t slot = id + (int64_t)k * takers;
                    const int32_t u = shared_load(ta.cur_u[half] + base + slot);
                    int32_t v = 0, sid = 0;
                    if (!forward) {
                        v = shared_load(ta.v + base + slot);
                        sid = shared_load(ta.seed_id[half] + base + slot);
                    }
                    const u64 key = shared_load(ta.keys + base + slot);
                    stores_arrived();  // read before it is cleared for the next search
                    if (lane == 0) shared_store(ta.keys + base + slot, (u64)0);
                    const int64_t row = min(max(forward ? u : v, 0), a.src_rows - 1);
                    const int32_t idx = resolve_tile<CT, DP>(a, tgt, key, O::load(src + row * O::ROW_BYTES, h), c, h).idx;
                    if (lane == 0) {
                        if (forward) {
                            shared_store(ta.v + base + slot, idx);
                        } else if (idx == u || final_one) {
                            ta.seed_i[base + sid] = u;
                            ta.seed_j[base + sid] = v;
                            ta.seed_iter[base + sid] = idx == u ? t : -1;
                        } else {
                            moving[atomicAdd(&n_moving, 1)] = make_int2(idx, sid);
                        }
                    }
                }
                __syncthreads();
                if (!forward && n_moving > 0) {  // uniform
                    if (threadIdx.x == 0) first_pos = (int)shared_add(&ctl.moving, (uint32_t)n_moving);
                    __syncthreads();
                    for (int i = threadIdx.x; i < n_moving; i += TAIL_THREADS) {
                        shared_store(ta.cur_u[half ^ 1] + base + first_pos + i, moving[i].x);
                        shared_store(ta.seed_id[half ^ 1] + base + first_pos + i, moving[i].y);
                    }
                    __syncthreads();
                }
            }
        }

        // report; the last of all opens the next phase
        stores_arrived();
        __syncthreads();
        if (wave == 0) {
            const uint32_t group = id % TAIL_COPIES, groups = min(phase.takers, (uint32_t)TAIL_COPIES);
            const uint32_t of_group = (phase.takers - group + TAIL_COPIES - 1) / TAIL_COPIES;
            uint32_t is_last = 0;
            if (lane == 0 && shared_add(&ctl.arrived[group].count, 1u) + 1 == of_group) is_last = shared_add(&ctl.groups_arrived, 1u) + 1 == groups;
            if (__builtin_amdgcn_readfirstlane(is_last)) {
                uint32_t takers_next = phase.takers, live_next = phase.live;
                if (lane == 0) {
                    if (kind == 3) live_next = shared_load(&ctl.moving);
                    if (kind & 1) takers_next = shared_load(&ctl.registered);  // a search is dealt to all that are there, and resolved by the same
                }
                takers_next = min((uint32_t)__builtin_amdgcn_readfirstlane(takers_next), most);
                live_next = __builtin_amdgcn_readfirstlane(live_next);
                if (kind == 3 && t + 1 >= ta.max_iter) live_next = 0;
                if (kind == 3 && live_next <= (uint32_t)TAIL_FEW) takers_next = min(takers_next, ta.few_wgs);
                stores_arrived();
                if (lane < TAIL_COPIES) shared_store(&ctl.arrived[lane].count, 0u);
                if (lane == 0) shared_store(&ctl.groups_arrived, 0u);
                if (lane == 0) shared_store(&ctl.moving, 0u);
                stores_arrived();
                // (the walk's end is not phase 0 either: a word of zeros would mean that it has not begun)
                publish(Phase::pack(phase.number + 1, takers_next, live_next));
            }
        }
    }

    // ---- few seeds ----
    const Phase phase(last);
    const uint32_t takers = phase.takers;
    if (id >= takers) return;
    int n_act = (int)phase.live, t = ta.t0 + (int)(phase.number >> 2);
    {
        const int half = (ta.half + (int)(phase.number >> 2)) & 1;
        if ((int)threadIdx.x < n_act) {
            few_at[0][threadIdx.x] = shared_load(ta.cur_u[half] + base + threadIdx.x);
            few_sid[threadIdx.x] = shared_load(ta.seed_id[half] + base + threadIdx.x);
            few_low[threadIdx.x] = -__builtin_inff();
        }
    }
    u64* table = ta.few_keys + (int64_t)b * 3 * TAIL_KEY_COPIES * TAIL_FEW;
    const uint32_t group = id % TAIL_COPIES, groups = min(takers, (uint32_t)TAIL_COPIES), of_group = (takers - group + TAIL_COPIES - 1) / TAIL_COPIES;
    const int gw = (int)id * TAIL_WAVES + wave, n_waves = (int)takers * TAIL_WAVES;
    // A search, out (V^t = NN_2(U^t)) and back (U^{t+1} = NN_1(V^t)) in turn.
    for (uint32_t searches = 0; n_act > 0;) {  // uniform; 0 after max_iter iterations at the latest
        const bool forward = (searches & 1) == 0;
        const int32_t* at = few_at[forward ? 0 : 1];
        const char* src = forward ? p1 : p2;
        const char* tgt = forward ? p2 : p1;
        const int src_rows = forward ? ta.rows1 : ta.rows2, m = forward ? ta.m : ta.n, m_tiles = (m + 31) / 32;
        // The keys of three searches take turns: while one fills, the one before it has been read by all, and is emptied for the next.
        u64* keys = table + searches % 3 * TAIL_KEY_COPIES * TAIL_FEW;
        for (uint32_t k = id; k < TAIL_KEY_COPIES; k += takers) shared_store(table + ((searches + 1) % 3 * TAIL_KEY_COPIES + k) * TAIL_FEW + threadIdx.x, (u64)0);
        if ((int)threadIdx.x < n_act) few_keys[threadIdx.x] = 0;
        __syncthreads();
        // A wave takes one or two blocks of queries and the more tiles for it.  Taking four and a few tiles (three of a 512x384 map, and the map once more for
        // every 128 queries) it waited for that many rows of queries and named that many winners for little work between.  This split, the bound that
        // scores start from (few_low), the copies of the keys and twice to four times as many workgroups, together, the launch in us: one 512x384 pair 53.8 -> 36.7, two with squared
        // distance 54.5 -> 46.3, four raw pairs 79.5 -> 66, four of two-term rows 112.5 -> 96 (so with two blocks; three blocks of narrow rows one by one).  One of them taken back, whole calls, features of
        // 1, 4 and 32 pixels, one 512x384 pair 162, 178 and 203 us: without the bound 163, 181 and 208, with one copy of the keys 165, 181 and 206, with a workgroup for 48 tiles 164, 182 and 216; four raw
        // pairs 391, 430 and 523: without the bound 394, 435 and 534, the other two the same.  Bound by
        // the loads of the tiles: a compute unit takes 236 ns for eight waves' 1.5 KB each, whatever they multiply them with; four blocks of narrow rows per
        // load cost more in registers and code than that saves (36.7 -> 40.0, 46.3 -> 47.6).  Products in fp32 cost more than the loads: an odd number of blocks is taken one
        // by one there, where by twos half of a pair is padding (whole calls, features of 4 pixels, 24 channels, by twos / one by one: 16 pairs of 256x192 433 / 418 us, four of 320x240
        // 241 / 232, of 512x384 with every 16th pixel a seed 366 / 360; features of 1 pixel the same).
        const int blocks = (n_act + 31) / 32, together = blocks == 1 || (blocks == 3 && O::ROW_BYTES <= 64) || (CT == CT_F32 && blocks % 2) ? 1 : 2, groups_of = (blocks + together - 1) / together;
        const int chunks = max(1, min(n_waves / groups_of, m_tiles));
#pragma unroll 1
        for (int unit = gw; unit < groups_of * chunks; unit += n_waves) {  // uniform in the wave
            const int chunk = unit / groups_of, slot0 = unit % groups_of * together * 32;
            const int tile0 = (int)((int64_t)m_tiles * chunk / chunks), tile1 = (int)((int64_t)m_tiles * (chunk + 1) / chunks);
            if (together == 1) named_unit<CT, DP, 1, named_ring<CT, DP, 1>()>(at, src, src_rows, tgt, n_act, slot0, tile0, tile1, m, few_low, few_keys, c, h);
            else named_unit<CT, DP, 2, named_ring<CT, DP, 2>()>(at, src, src_rows, tgt, n_act, slot0, tile0, tile1, m, few_low, few_keys, c, h);
        }
        __syncthreads();
        if ((int)threadIdx.x < n_act) {
            const u64 key = few_keys[threadIdx.x];
            if (key != 0) atomicMax(&keys[id % TAIL_KEY_COPIES * TAIL_FEW + threadIdx.x], key);
        }
        // the barrier: counts go on from search to search, and so does the number of the last search that is complete
        ++searches;
        stores_arrived();
        __syncthreads();
        if (wave == 0) {
            uint32_t is_last = 0;
            if (lane == 0 && shared_add(&ctl.few_arrived[group].count, 1u) + 1 == searches * of_group)
                is_last = shared_add(&ctl.few_groups_arrived, 1u) + 1 == searches * groups;
            if (__builtin_amdgcn_readfirstlane(is_last)) {
                if (lane < TAIL_COPIES) shared_store(&ctl.few_complete[lane].count, searches);
            } else if (lane == 0) {
                uint64_t polls = 0;
                while (shared_load(&ctl.few_complete[group].count) < searches && ++polls < ta.most_polls) __builtin_amdgcn_s_sleep(1);
                if (polls >= ta.most_polls) lost = 1;
            }
        }
        __syncthreads();
        if (lost) return;
        const bool here = (int)threadIdx.x < n_act;
        u64 key = 0;
        if (here) {
            u64 of[TAIL_KEY_COPIES];
#pragma unroll
            for (int k = 0; k < TAIL_KEY_COPIES; ++k) of[k] = shared_load(&keys[k * TAIL_FEW + threadIdx.x]);
#pragma unroll
            for (int k = 0; k < TAIL_KEY_COPIES; ++k) key = of[k] > key ? of[k] : key;
        }
        const int32_t found = here ? min(max(key_index(key), 0), m - 1) : 0;
        // What the next search finds is no worse than the way back to where this one began: the same product.
        // (compared as an integer, which sends what is not a number the same way as infinities)
        const float score = key_score(key);
        const bool number = (__float_as_uint(score) & 0x7FFFFFFFu) < __float_as_uint(1e30f);
        const float low = number ? score - 1e-3f * __builtin_fabsf(score) - 1e-30f : -__builtin_inff();
        if (forward) {
            few_at[1][threadIdx.x] = found;
            few_low[threadIdx.x] = low;
            continue;  // (read behind the next barrier)
        }
        const int32_t u = here ? few_at[0][threadIdx.x] : 0, v = here ? few_at[1][threadIdx.x] : 0, sid = here ? few_sid[threadIdx.x] : 0;
        const bool converged = found == u, moves = here && !converged && t + 1 < ta.max_iter;
        if (here && !moves && id == 0) {
            ta.seed_i[base + sid] = u;
            ta.seed_j[base + sid] = v;
            ta.seed_iter[base + sid] = converged ? t : -1;
        }
        int kept;
        const int pos = block_scan_flag(moves, wave_sums, kept);  // its barriers also end the reads of the slots above
        if (moves) {
            few_at[0][pos] = found;
            few_sid[pos] = sid;
            few_low[pos] = low;
        }
        n_act = kept;
        ++t;
        __syncthreads();
    }
}

// Workgroups per pair: one for every compute unit, dealt to the pairs.  When few seeds are left no more go on than leave two workgroups a tile and a half for every
// wave, or one dearer one: more would only make the barriers longer.  Whole calls of one pair in us, features of 4 pixels, with a workgroup for 48 / 24 / 12 tiles (and 32 at least): 160x120
// 67.2 / 67.3 / 65.0, 256x192 91.8 / 88.7 / 88.9, 320x240 102.2 / 99.2 / 99.3, 512x384 195.4 / 191 / 190; for 24 / 12 / 6 dearer ones: 256x192, fp32 products 177.1 / 173.1 /
// 169.8, two-term rows 126.5 / 123.9 / 123.9; 512x384 and 1024x768 of those the same.  (The keys of a query were one word, which took 13 ns for every workgroup; then a workgroup for 48
// tiles was best.)
static int tail_wgs_per_pair(int batch) { return TAIL_MOST_WGS / batch < 1 ? 1 : TAIL_MOST_WGS / batch; }
static int tail_few_wgs_per_pair(const TailArgs& a, int batch, int compute, int dp) {
    const int tiles = ((a.n > a.m ? a.n : a.m) + 31) / 32, per_wg = compute == FNN_F32 || dp > 32 ? 6 : 12;
    const int enough = tiles / per_wg > 32 ? tiles / per_wg : 32, wgs = tail_wgs_per_pair(batch);
    return wgs < enough ? wgs : enough;
}

// Groups of query blocks per wave while many seeds move: four would leave the named search no registers, and two of rows of 96 bytes spill 17 of them (fp32 products
// of 24 channels, two 512x384 pairs of 768 seeds that hardly settle 729 us with two, 690 with one).  Wider rows spill a few as they are, 20 of 96 two-term channels: half the
// query blocks cost more than that (two-term rows of four pairs that hardly settle 1627 us, 1880 with two blocks and no spill).
template <int CT, int DP>
constexpr int tail_groups() { return Ops<CT, DP>::ROW_BYTES > 64 ? 1 : (search_g_limit<CT, DP>() > 2 ? 2 : search_g_limit<CT, DP>()); }

template <int CT, int DP>
static hipError_t launch_tail_t(TailArgs a, int batch, hipStream_t s) {
    a.few_wgs = tail_few_wgs_per_pair(a, batch, CT, DP);
    return launch(TK_RECIP_TAIL, recip_tail_kernel<CT, DP, tail_groups<CT, DP>()>, dim3(tail_wgs_per_pair(batch), batch), dim3(TAIL_THREADS), 0, s, a);
}
hipError_t launch_tail(const TailArgs& a, int batch, int compute, int dp, hipStream_t s) {
    if (compute == FNN_F16) {
        if (dp == 16) return launch_tail_t<CT_F16, 16>(a, batch, s);
        if (dp == 24) return launch_tail_t<CT_F16, 24>(a, batch, s);
        if (dp == 32) return launch_tail_t<CT_F16, 32>(a, batch, s);
        if (dp == 48) return launch_tail_t<CT_F16, 48>(a, batch, s);
        if (dp == 64) return launch_tail_t<CT_F16, 64>(a, batch, s);
        if (dp == 80) return launch_tail_t<CT_F16, 80>(a, batch, s);
        if (dp == 96) return launch_tail_t<CT_F16, 96>(a, batch, s);
    } else if (compute == FNN_BF16) {
        if (dp == 16) return launch_tail_t<CT_BF16, 16>(a, batch, s);
        if (dp == 24) return launch_tail_t<CT_BF16, 24>(a, batch, s);
        if (dp == 32) return launch_tail_t<CT_BF16, 32>(a, batch, s);
    } else {
        if (dp == 8) return launch_tail_t<CT_F32, 8>(a, batch, s);
        if (dp == 16) return launch_tail_t<CT_F32, 16>(a, batch, s);
        if (dp == 24) return launch_tail_t<CT_F32, 24>(a, batch, s);
        if (dp == 32) return launch_tail_t<CT_F32, 32>(a, batch, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace fnn
