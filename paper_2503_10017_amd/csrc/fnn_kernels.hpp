// Host-side declarations of the kernel launchers that the C entry points are built from.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <mutex>

#include "../../include/fnn.h"

namespace fnn {

typedef unsigned long long u64;

// A launch shape that depends on the device (how many workgroups of a kernel it holds, how much
// LDS it grants): computed once per device by the first call made with that device current, under
// a lock, so that host threads and devices may make their first calls concurrently.
struct DeviceCache {
    static constexpr int MAX_DEVICES = 64;
    std::mutex mu;
    bool filled[MAX_DEVICES] = {};
    long long value[MAX_DEVICES] = {};
    // compute(device) returns the value, negative = failed (reported, not cached)
    template <typename F>
    long long get(F&& compute) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess) return -1;
        if (dev < 0 || dev >= MAX_DEVICES) return compute(dev);
        std::lock_guard<std::mutex> lock(mu);
        if (!filled[dev]) {
            const long long v = compute(dev);
            if (v < 0) return v;
            value[dev] = v;
            filled[dev] = true;
        }
        return value[dev];
    }
};

// Padded channel count of a prepared map: 16-bit formats use one K=16 matrix instruction,
// a K=16 and a K=8 one (24 channels, no padding for the paper's d = 24) or two K=16 ones;
// fp32 uses K=2 instructions on channel pairs.
constexpr int padded_d(int d, int compute) {
    if (compute == FNN_F32) return (d + 7) / 8 * 8;
    return d <= 16 ? 16 : (d <= 24 ? 24 : (d + 15) / 16 * 16);
}
// Channels of a prepared row that carry data: the descriptor plus, for the L2 score, the
// norm terms and their unit partners (two 16-bit halves each, or one fp32 value each).
inline int l2_extra_channels(int compute) { return compute == FNN_F32 ? 2 : 4; }
// ... or, for the two-term fp16 representation (FNN_FLAG_SPLIT), three copies of the descriptor's
// channels: [hi, hi, lo] in image 1 and [hi, lo, hi] in image 2.
inline int effective_d(int d, int compute, bool l2, bool split = false) {
    return split ? 3 * d : (l2 ? d + l2_extra_channels(compute) : d);
}
constexpr int64_t MAX_SLOTS = 2147483647LL - 64;  // most queries or seeds of a pair
constexpr int MAX_ROW_CHANNELS = 96;  // widest prepared row (16-bit formats; fp32 rows hold at most 32)
inline int elem_size(int dtype) { return dtype == FNN_F32 ? 4 : 2; }
inline int64_t round_up(int64_t x, int64_t a) { return (x + a - 1) / a * a; }

// ---- prepare: convert / pad the caller's maps into the workspace ------------------------
struct PrepSide {
    const void* src[FNN_MAX_BATCH];  // device pointers, one per pair
    int64_t n;                       // valid pixels
    int64_t n_pad;                   // rows written per pair (multiple of 32; rows >= n are zero)
    int32_t segment_major;           // 1: rows are stored in the dense kernel's segment-major order
    int64_t row_stride;              // source row stride, elements
    int32_t dtype;                   // source storage format
    int32_t vector_rows;             // set by the launcher: rows may be copied whole in 16-byte pieces
    int32_t second_image;            // L2 score: 0 = rows [x, 1.., -|x|^2/2..], 1 = rows [x, -|x|^2/2.., 1..]
    void* dst;                       // [batch][n_pad][dp] in the compute format
};
// Small initialisations that ride along with the prepare launch instead of costing launches
// of their own: clearing key tables / bitmaps, and step 1 of the FastNN iteration (U^0).
struct PrepExtra {
    u64* zero_ptr;          // range of 64-bit words to clear (NULL: none)
    int64_t zero_count;
    u64* zero_more;         // a second one
    int64_t zero_more_count;
    const int32_t* seeds;   // [batch][n_seeds] (NULL: no seed initialisation)
    int32_t* cur_u;         // [batch][n_seeds] <- seeds
    int32_t* seed_id;       // [batch][n_seeds] <- 0, 1, 2, ...
    int32_t* seed_iter;     // [batch][n_seeds] <- -1 (NULL: not written)
    int32_t* n_active;      // [batch] <- n_seeds
    int32_t n_seeds;
};
struct PrepArgs {
    PrepExtra extra;
    PrepSide side[2];
    int32_t n_sides;  // 1 or 2
    int32_t batch;
    int32_t d;
    int32_t dp;
    int32_t compute;
    int32_t normalize;  // divide every descriptor by its Euclidean norm first (FNN_FLAG_NORMALIZE)
    int32_t l2;         // append the norm channels of the L2 score (FNN_FLAG_L2)
    int32_t split;      // rows hold the two-term fp16 representation (FNN_FLAG_SPLIT); d is the source's
};
hipError_t launch_prep(const PrepArgs& a, hipStream_t s);
// "no neighbour": idx = -1, score = -inf (score may be NULL)
hipError_t launch_fill_i32f32(int32_t* idx, float* score, int64_t count, hipStream_t s);

// ---- one-directional search ------------------------------------------------------------
// What a search in two steps (coarse.hip) found out about the contrast of a pair.  A pair is given up where its queries need so many cells again
// that 8-bit scores do not pay.
struct SearchVote {
    u64 tally;          // of some waves of step 1, while it ran: queries that a cell leaves in doubt (24 bits), of how many (24), by how many waves (16)
    u64 again, of;      // of step 2: cells that queries had to be multiplied with, of how many
    uint32_t given_up;  // in step 1
    uint32_t reserved;
};
struct SearchArgs {
    const char* src;        // prepared map the queries are rows of, [batch][*][dp]
    int64_t src_bstride;    // bytes per pair
    int32_t src_rows;       // rows per pair in src (row indices are clamped to it)
    const int32_t* q_idx;   // [batch][nq] rows of src, or NULL
    const u64* q_keys;      // [batch][nq] keys whose index field names the row, or NULL
    const int32_t* nq_active;  // [batch] or NULL
    int32_t nq;
    const char* tgt;        // prepared candidate map [batch][m_tiles*32][dp]
    int64_t tgt_bstride;
    int32_t m;              // valid candidates
    int32_t m_tiles;
    u64* out_keys;          // [batch][nq], must hold 0 (or earlier partial results)
};
// Pass 1: out_keys receive (best score, tile of 32 candidates holding it).
hipError_t launch_search(const SearchArgs& a, int batch, int compute, int dp, hipStream_t s);

// The first searches of a call whose maps are still the caller's fp32 arrays (24 channels, a
// 16-bit compute format, every query live): the candidates are read from the caller's map,
// rounded on the way, staged through LDS once per workgroup, and written to the prepared map
// `s.tgt` as a by-product, so no separate prepare pass over that map is needed.
struct RawMaps {
    const float* map[FNN_MAX_BATCH];  // caller's map of every pair (16-byte aligned rows)
    int64_t row_stride;               // floats per row (a multiple of 4)
};
struct FirstSearchArgs {
    SearchArgs s;      // s.tgt: prepared candidate map to WRITE; s.nq_active is ignored (all nq queries are live)
    RawMaps raw_tgt;   // candidates
    RawMaps raw_src;   // queries, when raw_queries != 0 (else they are rows of the prepared map s.src)
    int32_t raw_queries;
};
// true if this shape should take the staged first search: enough queries to fill the workgroups'
// four waves and, with `batch` pairs sharing the device, chunks of m candidates long enough
bool first_search_applies(int64_t nq, int64_t m, int batch);
hipError_t launch_search_first(const FirstSearchArgs& a, int batch, int compute, hipStream_t s);
// launch_resolve with the queries still in the caller's fp32 map
hipError_t launch_resolve_raw(const FirstSearchArgs& a, int batch, int compute, int32_t* out_idx, float* out_score, int32_t* clear_count,
                              hipStream_t s);
// ---- tiles of the dense mode ------------------------------------------------------------------
constexpr int DENSE_J = 4;      // candidate tiles resident per wave
constexpr int DENSE_WAVES = 4;  // waves per workgroup
constexpr int DENSE_TILES_PER_GROUP = DENSE_J * DENSE_WAVES;

// What a sample of a pair's pixels says of the dense mode's 8-bit scores: the cells that may hold a sample's best partner, both ways, and so which way
// of the pair is the fastest.  It is decided once, at the end of the samples' launch: where every workgroup of the later launches did these sums for itself, they took 5 to 10 us
// longer each where workgroups are many.
enum DenseWay { DENSE_ONE_STEP, DENSE_SINGLES, DENSE_GROUPS };  // in the call's own format; in 8 bits, a maximum for every candidate; one for three
enum { MARKS_ROWS, MARKS_SINGLES, MARKS_GROUPS, DENSE_MARKS, PAIR_WAY = DENSE_MARKS, DENSE_RECORD };  // the words of a pair's record
struct DenseJudge {
    const int32_t* marked;      // [batch][DENSE_RECORD] (NULL: every pair in one step).  (With the ways in an array of their own dense_kernel keeps 284 bytes of scratch for rows of 32
                                // channels instead of 276, and one step of such rows took up to 4 % longer.)
    __device__ __forceinline__ DenseWay way(int b) const { return marked ? (DenseWay)marked[DENSE_RECORD * b + PAIR_WAY] : DENSE_ONE_STEP; }
};
struct DenseCosts {
    int64_t pairs;
    int64_t each[DENSE_MARKS];  // what a mark costs
    int64_t singles, groups;    // ... beside the marks, over one step
    int64_t least_groups;       // what the candidates' first round costs in groups, whatever is marked
    int64_t margin;             // a pair that gains no more than this goes the way of the others
    // over one step, of p pairs together
    __device__ __forceinline__ void costs(const int32_t (&m)[DENSE_MARKS], int64_t p, int64_t (&of)[3]) const {
        const int64_t rows = m[MARKS_ROWS] * each[MARKS_ROWS], marks = m[MARKS_GROUPS] * each[MARKS_GROUPS], least = p * least_groups;
        of[DENSE_ONE_STEP] = 0;
        of[DENSE_SINGLES] = p * singles + rows + m[MARKS_SINGLES] * each[MARKS_SINGLES];
        of[DENSE_GROUPS] = p * groups + rows + (marks > least ? marks : least);
    }
    __device__ __forceinline__ static int cheapest(const int64_t (&of)[3]) {
        const int two = of[DENSE_GROUPS] < of[DENSE_SINGLES] ? DENSE_GROUPS : DENSE_SINGLES;
        return (two == DENSE_GROUPS ? of[DENSE_GROUPS] : of[DENSE_SINGLES]) < 0 ? two : DENSE_ONE_STEP;
    }
    // the way of a pair from its marks and those of the call's pairs together
    __device__ __forceinline__ DenseWay way(const int32_t (&marked)[DENSE_MARKS], const int32_t (&all)[DENSE_MARKS]) const {
        int64_t of[3];
        costs(all, pairs, of);
        const int common = cheapest(of);
        costs(marked, 1, of);
        const int own = cheapest(of);
        const int64_t with_others = common == DENSE_GROUPS ? of[DENSE_GROUPS] : (common == DENSE_SINGLES ? of[DENSE_SINGLES] : 0);
        const int64_t alone = own == DENSE_GROUPS ? of[DENSE_GROUPS] : (own == DENSE_SINGLES ? of[DENSE_SINGLES] : 0);
        return (DenseWay)(with_others - alone > margin ? own : common);
    }
};

// ---- pass 1 in 8 bits, for searches large enough (coarse.hip) -------------------------------
// Pixels of a map are taken SEG_PIXELS at a time: one scale and one set of bounds for each segment.  A query's scores
// are bounded per CELL, a whole segment or half of one.
constexpr int SEG_TILES = 32;
constexpr int SEG_PIXELS = 32 * SEG_TILES;
constexpr int DENSE_SB_PIXELS = 4096;  // the dense mode sweeps so many queries at a time: one or two segments of its maps
constexpr int DENSE_CELL_PIXELS = 1024;  // ... past so many candidates
constexpr int DENSE_CELL_GROUPS = 384;   // ... of which it keeps a maximum each, or one for so many groups
constexpr int COARSE_ROW_BYTES = 32;  // one K=32 matrix instruction
struct SegInfo {
    float scale;     // a row is about scale * its 8-bit row
    float residual;  // at most this far from it, in any of the segment's rows
    float length;    // the longest 8-bit row, scaled
    float reserved;
};
// The 8-bit image of a batch of prepared maps.  Rows past the map repeat its last row.
struct CoarseMap {
    char* rows;           // [batch][n_segs * SEG_PIXELS][COARSE_ROW_BYTES]
    uint32_t* row_bound;  // [batch][n_segs * SEG_PIXELS] length and residual of every row over its segment's scale (two bf16, rounded up)
    SegInfo* seg;         // [batch][n_segs]
    int32_t n_segs;
};
struct QuantiseSide {
    const char* prepared;  // [batch] prepared maps, bstride bytes apart: read, or (raw) written on the way
    int64_t bstride;
    int64_t n;             // valid pixels (gather: rows listed)
    int64_t n_pad;         // prepared rows per pair (raw)
    const float* raw[FNN_MAX_BATCH];  // the caller's fp32 rows of 24 channels, 16-byte aligned (raw_rows)
    int64_t raw_stride;    // floats
    const int32_t* gather; // [batch][n] rows of the source to take, in this order (NULL: all of them)
    int64_t gather_rows;   // rows of that source; the list's entries are clamped to it
    CoarseMap out;
};
struct QuantiseArgs {
    PrepExtra extra;       // side jobs that ride along where there is no prepare launch
    QuantiseSide side[2];
    int32_t batch;
    int32_t raw_rows;
    int32_t normalize;     // (raw_rows, rows that are not two-term) rows are divided by their norm first
    int32_t seg_pixels;    // SEG_PIXELS, 2048 or 4096
    uint32_t* lower;       // bounds to clear
    int64_t lower_count;
    int32_t split_d;       // channels of a two-term row's descriptor (0: rows are not two-term)
};
hipError_t launch_quantise(const QuantiseArgs& a, int compute, int dp, hipStream_t s);

struct CoarseArgs {
    CoarseMap src, tgt;
    int32_t src_listed;    // src holds the queries themselves, in the order of their slots
    uint16_t* upper;       // [batch][cells][slab] bf16: no score of the cell lies above it
    uint32_t* lower;       // [batch][slot_pitch] order_bits: some score lies at or above it (0 on entry)
    int32_t slab;          // slots that one launch takes (a multiple of 64)
    int64_t slot_pitch;    // queries of a pair, rounded up to whole 64s
    int32_t n_cells;       // of a pair
    int32_t cell_shift;    // a cell is 2^cell_shift workgroups of the second step
    const uint64_t* mask;  // launch_refine: the slots that need a cell, instead of the bounds: [n_cells][slab / 64] of every pair, slot_pitch words
                           // apart.  Of a pair's candidates in groups: twice as many cells, the bits of every 1024 slots in the order of mask_candidate()
    DenseJudge judge;      // launch_refine: pairs to leave alone
    int32_t side;          // ... and whose slots they are: image 1's (queries) or 2's (candidates)
    int32_t second_round;  // ... of the candidates in groups: pairs without them are left alone
    int32_t range;         // (the launchers set these) queries that a workgroup of the second step looks at, or fewer
    int32_t first_slot;
    int32_t min_live;      // fewer live queries of a pair than this: its cells are refined for every query
    SearchVote* vote;      // [batch] (0 on entry), or NULL: scores in 8 bits whatever the maps hold
    const SearchVote* earlier;  // [batch] of a search of the same maps, or NULL: pairs that it gives up begin with step 2, for every query
    float even;            // (vote) cells that a query may have to be multiplied with before one step is faster, over those that it need not
};
// What launch_search does: the queries' list and live count, the prepared maps and the keys are those of `a`.
hipError_t launch_coarse_search(const SearchArgs& a, const CoarseArgs& ca, int batch, int compute, int dp, hipStream_t s);
// The second step alone, for the slots [first_slot, first_slot + slab) and cells of SEG_TILES << cell_shift tiles, from the table
// `mask`; its keys name units of DENSE_J tiles.
hipError_t launch_refine(const SearchArgs& a, const CoarseArgs& ca, int batch, int compute, int dp, hipStream_t s);
// Nanoseconds of the device that a search of `nq` queries per pair against maps of m pixels gains in two steps (very negative where
// it has to run in one), and what the 8-bit maps of `rows` pixels cost
double coarse_gain(int64_t nq, int64_t m, int batch, int compute, int dp, int d, bool l2);
double coarse_cells_again(double cells, int d, bool l2);
bool coarse_votes(int compute, int dp);  // whether the searches of such rows should
double coarse_cost(int64_t rows, int compute, int dp);
constexpr double COARSE_LEAST_GAIN = 3000.0;  // of a call
// See CoarseArgs.even: three cells in seven.  (Of a search of 16-bit rows, 46 ns a block in one step, some 17 of 26 are still to do in 8 bits when the
// votes are in, and the second step takes 58 for every block it is left with.)
constexpr float COARSE_EVEN = 0.75f;
// Fewer queries per pair than this spread the second step thin: a call with so few runs in one
inline int64_t coarse_least_queries(int compute, int dp) { return compute == FNN_F32 || dp > 32 ? 256 : 2048; }
// Live queries of a pair below which its part of a later search goes straight to the second step
inline int coarse_min_live(int compute, int dp) { return compute == FNN_F32 || dp > 32 ? 64 : 512; }
// Slots per launch that keep the table of upper bounds small
int64_t coarse_slab(int64_t nq, int64_t n_segs, int batch);
int coarse_cells(int64_t nq, int64_t n_segs, int batch, int compute);  // cells of a segment

// Pass 2: out_keys become (best score, lowest candidate index); optionally also stored to
// out_idx / out_score (either may be NULL).  Queries without any candidate get -1 / -inf.
// clear_count, if not NULL, is int32[batch] to set to 0.
hipError_t launch_resolve(const SearchArgs& a, int batch, int compute, int dp, int32_t* out_idx, float* out_score,
                          int32_t* clear_count, hipStream_t s);

// ---- the paper's blocked schedules with a materialised score block (contrast experiment) ----
struct BlockedArgs {
    const char* src;        // prepared query map (one pair)
    int32_t src_rows;
    const int32_t* q_idx;   // [nq] or NULL
    int32_t nq;
    const char* tgt;        // prepared candidate map
    int32_t m;
    float* dists;           // [block_rows][ld] score block in device memory
    int64_t ld;             // columns of the score block (multiple of 32)
    int32_t* out_idx;       // [nq]
    float* out_score;       // [nq] (required: it holds the running best between blocks)
    int32_t half_accumulate;  // FNN_FLAG_HALF_ACCUMULATE: fp16 products and fp16 sums on the vector ALU
};
// block_cols == 0: Algorithm 2 (whole B per block of A); otherwise Algorithm 1 (double loop).
hipError_t run_blocked(const BlockedArgs& a, int compute, int d, int dp, int block_rows, int block_cols, hipStream_t s);

// ---- reciprocal iteration bookkeeping ----------------------------------------------------
struct RecipState {
    int32_t* cur_u[2];   // [batch][n_seeds] ping-pong: U^t of the seeds still moving
    int32_t* seed_id[2]; // [batch][n_seeds] which seed sits in each slot
    int32_t* n_active[2];  // [batch] seeds still moving; the half not in use is 0 when an iteration's bookkeeping starts
    u64* keys_f;         // [batch][n_seeds] result of the search into image 2 (V^t)
    u64* keys_b;         // [batch][n_seeds] result of the search back into image 1 (U^{t+1})
    uint32_t* bitmap;    // [batch][n_words] one bit per pixel of image 1, for the final sort
    int32_t* word_rank;  // [batch][n_words] rank of the first bit of each bitmap word (before the sort: n_active[1])
    int64_t n_words;
};
struct StepArgs {
    const int32_t* cur_u;     // U^t per slot
    const int32_t* seed_id;
    int32_t* next_u;          // U^{t+1} of the survivors, compacted
    int32_t* next_seed_id;
    int32_t* next_active;     // [batch] their number (0 on entry)
    u64* keys_f;              // V^t per slot (index field); cleared for the next search
    int32_t t;
    int32_t mode;
    int32_t* seed_i;
    int32_t* seed_j;
    int32_t* seed_iter;
};
// Pass 2 of the search back (its arguments are `a`; the keys are cleared afterwards) and the
// bookkeeping of iteration t.  mode 0: ordinary iteration; 1: last iteration (survivors are
// reported as unconverged); 2: no iteration at all (max_iter == 0; no search back was made):
// every seed is reported unconverged with (U^0, V^0).
hipError_t launch_resolve_step(const SearchArgs& a, const StepArgs& st, int batch, int compute, int dp, hipStream_t s);
hipError_t launch_recip_dedup(const RecipState& st, int32_t n_seeds, int batch,
                              const int32_t* seed_i, const int32_t* seed_j, const int32_t* seed_iter,
                              int32_t* pairs, int32_t* n_pairs, hipStream_t s);

// The whole iteration of a small pair in one workgroup, on prepared maps; all outputs included.
struct WalkArgs {
    const char* p1;        // prepared maps of both images
    const char* p2;
    int64_t bstride1, bstride2;  // bytes per pair
    int32_t rows1;         // rows per pair of image 1 (the seeds are clamped to them)
    int32_t n, m;          // valid pixels
    int32_t n_words;       // ceil(n / 32)
    const int32_t* seeds;  // [batch][n_seeds]
    int32_t n_seeds;
    int32_t max_iter;      // at least 1
    int32_t* seed_i;
    int32_t* seed_j;
    int32_t* seed_iter;
    int32_t* pairs;
    int32_t* n_pairs;
};
// true if a pair is small enough that one workgroup beats the launch sequence
bool walk_applies(int64_t n, int64_t m, int64_t n_seeds, int32_t max_iter, int compute, int dp);
hipError_t launch_walk(const WalkArgs& a, int batch, int compute, int dp, hipStream_t s);
// true if one workgroup per 32 seeds beats the launch sequence; the outputs of the sort (pairs, n_pairs) are launch_recip_dedup's
bool groups_apply(int64_t n, int64_t m, int64_t n_seeds, int batch, int32_t max_iter, int compute, int dp);
hipError_t launch_groups(const WalkArgs& a, int batch, int compute, int dp, hipStream_t s);

// The iterations from t0 on in one launch (tail.hip), for all seeds that still move.
constexpr int TAIL_FEW = 512;        // seeds of a pair that every workgroup can keep
constexpr int TAIL_MOST_WGS = 256;   // of a pair
constexpr int TAIL_COPIES = 16;      // of the words that many workgroups read or count in, each in a cache line of its own
constexpr int TAIL_KEY_COPIES = 8;   // of few seeds' keys: additions to one word are served one after the other
constexpr int TAIL_MOST_ITERATIONS = 1 << 20;
struct TailControl {                 // of a pair; 0 on entry
    struct alignas(128) Word { u64 word; };
    struct alignas(128) Count { uint32_t count; };
    Word phase[TAIL_COPIES];         // see tail.hip
    Count arrived[TAIL_COPIES];
    Count few_arrived[TAIL_COPIES], few_complete[TAIL_COPIES];
    alignas(128) uint32_t groups_arrived;
    alignas(128) uint32_t few_groups_arrived;
    alignas(128) uint32_t registered;
    alignas(128) uint32_t moving;
};
struct TailArgs {
    const char* p1;                  // prepared maps of both images
    const char* p2;
    int64_t bstride1, bstride2;
    int32_t rows1, rows2;            // rows per pair (indices are clamped to them)
    int32_t n, m;                    // valid pixels
    int32_t n_seeds;
    int32_t* cur_u[2];               // [batch][n_seeds] see RecipState
    int32_t* seed_id[2];
    int32_t half;                    // of the two that holds the live seeds of iteration t0
    const int32_t* n_active;         // [batch] their number
    u64* keys;                       // [batch][n_seeds] 0 on entry
    int32_t* v;                      // [batch][n_seeds] scratch
    u64* few_keys;                   // [batch][3][TAIL_KEY_COPIES][TAIL_FEW] 0 on entry
    TailControl* control;
    int32_t t0, max_iter;            // t0 < max_iter <= TAIL_MOST_ITERATIONS
    uint64_t most_polls;             // looks at a word before a wait is given up
    uint32_t few_wgs;                // workgroups of a pair that go on when few seeds are left, at most
    int32_t* seed_i;
    int32_t* seed_j;
    int32_t* seed_iter;
};
hipError_t launch_tail(const TailArgs& a, int batch, int compute, int dp, hipStream_t s);
// A wait of recip_tail_kernel lasts one phase at most: a search of all seeds that are left, or its resolve pass, by the workgroups that take part, which
// may be a single one (the others came later, and wait until it is done).  A workgroup alone takes 0.2 us at most for a block of 32x32 scores (the dearest
// products, of 32 fp32 channels, 600 ns of one of its four SIMDs; fewer bytes than that has time to load) and 2 us for a query of the resolve pass; a look takes 0.13 us (at one
// word, by 1, 16 and 256 workgroups).  Twenty times that, and never less than 2^26 looks (9 s): a wait that is longer means that two calls share a workspace
// unordered and have overwritten each other's words.
inline uint64_t tail_most_polls(int64_t n, int64_t m, int64_t n_seeds) {
    const uint64_t tiles = (uint64_t)((n > m ? n : m) + 31) / 32, blocks = (uint64_t)((n_seeds + 31) / 32) * tiles;
    return ((uint64_t)1 << 26) + 32 * blocks + 320 * (uint64_t)n_seeds;
}

// ---- dense mutual nearest neighbours -----------------------------------------------------
struct DenseArgs {
    const char* d1;        // prepared queries, segment-major, [batch][n_sb*32*DENSE_S][dp]
    int64_t d1_bstride;
    const char* d2;        // prepared candidates, natural order, [batch][m_tiles*32][dp]
    int64_t d2_bstride;
    int32_t n, m;
    int32_t n_sb;          // super-blocks of queries (32*DENSE_S pixels each)
    int32_t m_tiles;       // 32-pixel tiles of candidates
    u64* row_keys;         // [batch][n] zero-initialised; (best score, group of DENSE_J tiles)
    u64* col_keys;         // [batch][m] zero-initialised; (best score, run of DENSE_S queries)
    int32_t sb_per_wg;     // super-blocks swept by one workgroup
    int32_t groups_per_wg; // candidate groups (DENSE_WAVES x DENSE_J tiles) per workgroup
    // pass 2: pixels bucketed by their winning unit
    int32_t row_units;     // groups of DENSE_J candidate tiles
    int32_t col_units;     // runs of DENSE_S queries (n_sb * 32)
    int64_t rows_cap;      // list positions for the queries: round_up(n, 32) + 32 * row_units
    int64_t cols_cap;      // list positions for the candidates: round_up(m, 32) + 32 * col_units
    int32_t* unit_counts;  // [batch][row_units + col_units] zero-initialised
    int32_t* unit_cursor;  // [batch][row_units + col_units] next free list position (after the fill: end) of a bucket
    int32_t* lists;        // [batch][rows_cap + cols_cap] pixels grouped by unit, buckets start on multiples of 32
    int32_t* chunk_unit;   // [batch][(rows_cap + cols_cap) / 32] unit of every chunk of 32 list positions
    int32_t* chunk_totals; // [batch][2] chunks in use per side
    DenseJudge judge;      // launch_dense_pass1: takes the pairs that are DENSE_ONE_STEP
};
// Pass 1 (both maxima with coarse locations) and pass 2 (exact indices and scores into
// nn12/s12/nn21/s21; s12, s21 may be NULL).
hipError_t launch_dense(const DenseArgs& a, int batch, int compute, int dp, int32_t* nn12, float* s12, int32_t* nn21,
                        float* s21, hipStream_t s);

// Pass 1 alone.
hipError_t launch_dense_pass1(const DenseArgs& a, int batch, int compute, int dp, hipStream_t s);

// Of pairs that turn out alike: the prepared rows of image 1 in the order that the dense kernels sweep.
struct DenseSwept {
    const char* from;  // [batch] prepared maps in natural order
    int64_t from_bstride;
    char* to;          // [batch][n_pad][row_bytes], or NULL: not in this launch
    int64_t n_pad;     // a multiple of DENSE_SB_PIXELS
    int32_t row_bytes; // a multiple of 16
};
// Pass 1 in 8 bits (dense_coarse.hip), on maps quantised in segments of seg_pixels: the largest 8-bit score of every query in
// every cell of candidates, and of every candidate, or group of candidates, in every cell of queries.
struct DenseCoarseArgs {
    CoarseMap map[2];      // images 1 and 2
    int32_t n_tiles[2];    // tiles of each that hold a pixel
    int32_t seg_pixels;    // 2048 or 4096
    int32_t first_sb;      // the runs of DENSE_SB_PIXELS of image 1 that this launch takes
    int32_t n_sb;
    int32_t cell_runs;     // runs of DENSE_CELL_PIXELS candidates in a cell: 1, 2 or 4
    int32_t grouped;       // pairs may keep the maxima of groups of candidates, whose cells are half segments of queries instead of whole ones (DENSE_GROUPS)
    int32_t n_cells;       // of image 2
    int32_t n_col_cells;   // of image 1, those that hold a pixel: half segments where `grouped`, else whole ones
    int32_t cells_per_wg;  // (set by the launcher)
    uint16_t* best[2];     // [batch][n_cells][n_sb * 4096] of the queries; [map[0].n_segs][pixels of map[1]], or [2 map[0].n_segs][its groups], of the candidates,
                           // pairs map[0].n_segs * pixels apart
    uint64_t* mask[2];     // [batch][the same cells], a bit for every query and every candidate: cells that may hold its best partner; of the
                           // candidates, pairs (map[0].n_segs << grouped) * pixels bits apart
    float* least;          // [batch][groups of map[1]] the second round's limit: see select_groups
    int64_t pixels[2];
    float* sample_upper[2];  // [batch][cells of the other image][DENSE_SAMPLES]
    float* sample_group;     // (grouped) [batch][n_col_cells][DENSE_SAMPLES]
    uint32_t* sample_lower;  // [batch][2][DENSE_SAMPLES] order_bits (0 on entry)
    uint32_t* sample_best;   // (grouped) [batch][DENSE_SAMPLES] order_bits (0 on entry)
    int32_t* marked;         // [batch][DENSE_RECORD] (0 on entry): see DenseJudge
    uint32_t* filed;         // workgroups that have counted their marks (0 on entry)
    DenseJudge judge;
    DenseSwept swept;
};
constexpr int DENSE_SAMPLES = 128;  // pixels of either image
// Counts the marks of the samples.
hipError_t launch_dense_sample(const DenseCoarseArgs& a, const DenseCosts& costs, int batch, hipStream_t s);
hipError_t launch_dense_coarse(DenseCoarseArgs a, int batch, hipStream_t s);
// From best[side] to mask[side] for one or both sides.  0: the queries of this launch's runs; 1: the candidates, once every run is done.
// Groups of candidates take two rounds, the second with what the first left in their keys (col_keys, NULL: the first).
hipError_t launch_dense_select(const DenseCoarseArgs& a, int first_side, int sides, const u64* col_keys, int batch, hipStream_t s);
int dense_cell_runs(int64_t n, int64_t m);
bool dense_grouped(int64_t n, int compute, int dp);  // whether the candidates' maxima may be those of groups
int dense_seg_pixels(int64_t n);
DenseCosts dense_costs(const DenseCoarseArgs& a, int batch, int compute, int dp, bool l2);
// Nanoseconds that a call gains this way
double dense_coarse_gain(int64_t n, int64_t m, int batch, int compute, int dp, int d, bool l2);

// Pass 2 for keys that launch_refine left in row_keys and col_keys (units of DENSE_J tiles of the other map), both maps in natural order.
hipError_t launch_dense_resolve(const DenseArgs& a, int batch, int compute, int dp, int32_t* nn12, float* s12, int32_t* nn21, float* s21,
                                hipStream_t s);

struct DenseFinalArgs {
    int32_t n, m;
    const int32_t* nn12;
    const int32_t* nn21;
    int32_t* pairs;       // [batch][min(n,m)][2]
    int32_t* n_pairs;     // [batch]
    int32_t* block_counts;  // [batch][ceil(max(n,m)/1024)] scratch
};
hipError_t launch_dense_final(const DenseFinalArgs& a, int batch, hipStream_t s);

// ---- matches as pixel coordinates, confidence filter -------------------------------------
struct PixelArgs {
    const int32_t* pairs;    // [batch][max_pairs][2] flat pixel ids (i in image 1, j in image 2)
    const int32_t* n_pairs;  // [batch]
    int64_t max_pairs;
    int64_t n, m;            // pixels per image
    int32_t width1, width2;
    const float* conf1;      // [batch][n] or NULL
    const float* conf2;      // [batch][m] or NULL
    float min_conf1, min_conf2;
    int32_t* out_xy;         // [batch][max_pairs][4]
    int32_t* out_count;      // [batch]
};
hipError_t launch_pairs_to_pixels(const PixelArgs& a, int batch, hipStream_t s);

}  // namespace fnn
