// C entry points of libfnn (see include/fnn.h): argument checks, workspace carving and the
// fixed kernel sequences.  Nothing here synchronises with the device or allocates memory.
#include <hip/hip_runtime.h>
#include <string.h>

#include "dense_perm.hpp"
#include "fnn_kernels.hpp"

using namespace fnn;

namespace {

constexpr int64_t MAX_PIXELS = MAX_SLOTS;
constexpr int64_t MAX_DENSE_PIXELS = 1LL << 30;  // keeps the padded bucket lists of the dense mode within int32
constexpr size_t WS_ALIGN = 256;

struct Carver {
    char* base;
    size_t used;
    void* take(size_t bytes) {
        void* p = base ? base + used : nullptr;
        used += (bytes + WS_ALIGN - 1) / WS_ALIGN * WS_ALIGN;
        return p;
    }
};

bool valid_dtype(int32_t t) { return t == FNN_F32 || t == FNN_F16 || t == FNN_BF16; }

struct MapsLayout {
    void* p1;
    void* p2;
    int64_t n_pad, m_pad;
    int64_t bstride1, bstride2;  // bytes per pair
    int dp;
};

MapsLayout carve_maps(Carver& cv, int batch, int64_t n, int64_t m, int d, int compute, int64_t n_align = 32) {
    MapsLayout L;
    L.dp = padded_d(d, compute);
    L.n_pad = round_up(n, n_align);
    L.m_pad = round_up(m, 32);
    const int es = elem_size(compute);
    L.bstride1 = L.n_pad * L.dp * es;
    L.bstride2 = L.m_pad * L.dp * es;
    L.p1 = cv.take((size_t)batch * L.bstride1);
    L.p2 = cv.take((size_t)batch * L.bstride2);
    return L;
}

struct NearestLayout {
    MapsLayout maps;
    u64* keys;
};
NearestLayout carve_nearest(Carver& cv, int batch, int64_t n, int64_t m, int d, int64_t nq, int compute) {
    NearestLayout L;
    L.maps = carve_maps(cv, batch, n, m, d, compute);
    L.keys = (u64*)cv.take((size_t)batch * nq * sizeof(u64));
    return L;
}

struct RecipLayout {
    MapsLayout maps;
    RecipState st;
    int64_t zero_words;  // 64-bit words from keys_f to the end of the bitmap
};
RecipLayout carve_recip(Carver& cv, int batch, int64_t n, int64_t m, int d, int64_t n_seeds, int compute) {
    RecipLayout L;
    L.maps = carve_maps(cv, batch, n, m, d, compute);
    const size_t per = (size_t)batch * n_seeds;
    // keys_f, keys_b and the bitmap are adjacent so that one range clears all three
    const size_t z0 = cv.used;
    L.st.keys_f = (u64*)cv.take(per * sizeof(u64));
    L.st.keys_b = (u64*)cv.take(per * sizeof(u64));
    L.st.n_words = (n + 31) / 32;
    L.st.bitmap = (uint32_t*)cv.take((size_t)batch * L.st.n_words * sizeof(uint32_t));
    L.zero_words = (int64_t)((cv.used - z0) / sizeof(u64));
    L.st.cur_u[0] = (int32_t*)cv.take(per * sizeof(int32_t));
    L.st.cur_u[1] = (int32_t*)cv.take(per * sizeof(int32_t));
    L.st.seed_id[0] = (int32_t*)cv.take(per * sizeof(int32_t));
    L.st.seed_id[1] = (int32_t*)cv.take(per * sizeof(int32_t));
    L.st.n_active[0] = (int32_t*)cv.take((size_t)batch * sizeof(int32_t));
    L.st.word_rank = (int32_t*)cv.take((size_t)batch * L.st.n_words * sizeof(int32_t));
    L.st.n_active[1] = L.st.word_rank;  // the sort writes its ranks after the last iteration (n > 0, so a word per pair is there)
    return L;
}

// Room for the two-step search behind the layouts above.  A caller's workspace that ends before it is searched in one step.
struct CoarseLayout {
    CoarseMap map[2];      // images 1 and 2 (fnn_nearest: the queries and the candidates)
    uint16_t* upper;
    uint32_t* lower;       // [searches][batch][slot_pitch]
    int64_t lower_count;   // words of one search
    SearchVote* votes;     // [searches][batch], behind them
    int64_t zero_words;    // 32-bit words that start at 0, from `lower` on
    int64_t slot_pitch;
    int64_t slab;
};
CoarseMap carve_coarse_map(Carver& cv, int batch, int64_t pixels, int segment = SEG_PIXELS) {
    CoarseMap M;
    M.n_segs = (int32_t)((pixels + segment - 1) / segment);
    const size_t rows = (size_t)batch * M.n_segs * segment;
    M.rows = (char*)cv.take(rows * COARSE_ROW_BYTES);
    M.row_bound = (uint32_t*)cv.take(rows * sizeof(uint32_t));
    M.seg = (SegInfo*)cv.take((size_t)batch * M.n_segs * sizeof(SegInfo));
    return M;
}
// both_searched: image 1 is a map of candidates too
CoarseLayout carve_coarse(Carver& cv, int batch, int64_t rows1, int64_t rows2, bool both_searched, int64_t nq, int searches, int compute) {
    CoarseLayout L;
    L.map[0] = carve_coarse_map(cv, batch, rows1);
    L.map[1] = carve_coarse_map(cv, batch, rows2);
    const int64_t segs = both_searched && L.map[0].n_segs > L.map[1].n_segs ? L.map[0].n_segs : L.map[1].n_segs;
    int64_t cells = 0;
    for (int i = both_searched ? 0 : 1; i < 2; ++i) {
        const int64_t of_map = (int64_t)L.map[i].n_segs * coarse_cells(nq, L.map[i].n_segs, batch, compute);
        if (of_map > cells) cells = of_map;
    }
    L.slot_pitch = round_up(nq, 64);
    L.slab = coarse_slab(nq, segs, batch);
    L.lower_count = batch * L.slot_pitch;
    L.zero_words = searches * (L.lower_count + batch * (int64_t)(sizeof(SearchVote) / sizeof(uint32_t)));
    L.lower = (uint32_t*)cv.take((size_t)L.zero_words * sizeof(uint32_t));
    L.votes = reinterpret_cast<SearchVote*>(L.lower ? L.lower + searches * L.lower_count : nullptr);
    L.upper = (uint16_t*)cv.take((size_t)batch * cells * L.slab * sizeof(uint16_t));
    return L;
}
// vote: whether the pairs of this search may be given up
CoarseArgs coarse_args(const CoarseLayout& L, int batch, int src, int search, bool vote) {
    CoarseArgs ca;
    memset(&ca, 0, sizeof(ca));
    ca.src = L.map[src];
    ca.tgt = L.map[src ^ 1];
    ca.upper = L.upper;
    ca.lower = L.lower + search * L.lower_count;
    ca.slab = (int32_t)L.slab;
    ca.slot_pitch = L.slot_pitch;
    if (vote) ca.vote = L.votes + (int64_t)search * batch;
    ca.even = COARSE_EVEN;
    return ca;
}
// Queries of fnn_nearest that are few beside their map are taken out of it, in the order of their slots.
bool list_queries(const int32_t* q_idx, int64_t nq, int64_t n) { return q_idx && nq <= n / 2; }
constexpr int RECIP_COARSE_SEARCHES = 4;  // out and back, of the first two iterations

// Searches of a call that run in two steps, if its workspace allows: none or the one of fnn_nearest, none, the first two or the
// first four of the iteration.  About half the seeds live to see the second iteration; if few do, two launches are wasted.
int nearest_coarse_searches(int batch, int64_t n, int64_t m, int64_t nq, bool listed, int compute, int dp, int d, bool l2) {
    if (nq < coarse_least_queries(compute, dp)) return 0;
    const double gain = coarse_gain(nq, m, batch, compute, dp, d, l2) - coarse_cost(batch * (m + (listed ? nq : n)), compute, dp);
    return gain > COARSE_LEAST_GAIN ? 1 : 0;
}
int recip_coarse_searches(int batch, int64_t n, int64_t m, int64_t n_seeds, int compute, int dp, int d, bool l2) {
    if (n_seeds < coarse_least_queries(compute, dp)) return 0;
    const double first = coarse_gain(n_seeds, m, batch, compute, dp, d, l2) + coarse_gain(n_seeds, n, batch, compute, dp, d, l2);
    const double second = coarse_gain(n_seeds / 2, m, batch, compute, dp, d, l2) + coarse_gain(n_seeds / 2, n, batch, compute, dp, d, l2);
    const double gain = first + (second > 0.0 ? second : 0.0) - coarse_cost(batch * (n + m), compute, dp);
    return gain <= COARSE_LEAST_GAIN ? 0 : (second > 2.0 * COARSE_LEAST_GAIN ? RECIP_COARSE_SEARCHES : 2);
}

// The iteration from which on the rest are one launch (recip_tail_kernel), -1: none.  The first two are the ones with many seeds, whose searches the
// launches share out better; a walk that begins with few seeds is one launch altogether.  Whole calls in us with launches only / the tail from iteration
// 0 / 1 / 2 / 3: one 512x384 pair, features of 1 and of 4 pixels, 192 seeds 163 / 84 / 104 / 112 and 180 / 91 / 112 / 128, 352 183 / 104 / 106 / 130 and
// 185 / 109 / 111 / 131, 768 181 / 132 / 119 / 122 and 193 / 157 / 143 / 134, 3072 236 / 249 / 206 / 183 and 267 / 277 / 236 / 204; 320x240, 300 seeds 149 / 88 / 84 / 86, 1200
// 153 / 157 / 121 / 102; 160x120, 1200 seeds 142 / 208 / 135 / 86.  Where very many seeds are left, the launches also have the wider search; from 2 / 3 on, features of 1, 4 and
// 32 pixels, and of 4 and 32 in maps that have nothing in common: 12 pairs of 512x384, 3072 seeds 968 / 981, 1096 / 1127, 1341 / 1394, 1199 / 1201, 2209 / 2213; 24 of them 1840 / 1836,
// 2066 / 2100, 2588 / 2723, 2327 / 2315, 4432 / 4550; 48 3659 / 3656, 4097 / 4118, 5101 / 5498, 4629 / 4616, 8901 / 9487; four of 1024x768, 12288 seeds 3396 / 3366, 3849 / 3975,
// 5124 / 5301, 4351 / 4364, 8221 / 8224; one, 49152 seeds 3162 / 3171, 3500 / 3514, 4621 / 4643, 4038 / 4059, 7922 / 7918; 64 of 256x192, 3072 seeds 1417 / 1433, 1593 / 1596, 1974 / 1995,
// 1864 / 1838, 3855 / 3759; 48 of 160x120, 4800 seeds 1048 / 1073, 1151 / 1173, 1428 / 1417, 1360 / 1344, 3066 / 2836.  So the line lies where the last kind begins to lose more than the
// others gain, between 48 x 3072 and 64 x 3072.
// Two maps that have nothing in common and features of 32 pixels keep hundreds of seeds moving for many iterations.  In launches only / so: one 512x384 pair 410 / 351, 16 pairs 3084 /
// 3008, 1024x768 2455 / 2336, 16 256x192 pairs 496 / 444; with every fourth pixel a seed, 320x240 316 / 299, four of them 703 / 698, 400x300 505 / 483, but 64 160x120 pairs 985 / 1042: the price
// of what such calls gain where features of 4 pixels let seeds settle (195 / 139, 380 / 331, 294 / 232, 552 / 481).
int first_late_iteration(int batch, int64_t n_seeds, int32_t max_iter, bool coarse) {
    const int from = batch * n_seeds > 147456 ? 3 : (n_seeds > TAIL_FEW || coarse ? 2 : (n_seeds > TAIL_FEW / 2 ? 1 : 0));
    const int least = from > 2 ? from + 2 : 4;  // (with a single iteration left, four launches are as good)
    return max_iter >= least && max_iter <= TAIL_MOST_ITERATIONS ? from : -1;
}

struct DenseLayout {
    MapsLayout maps;
    u64* row_keys;
    u64* col_keys;
    int32_t* unit_counts;
    int64_t zero_words;  // 64-bit words from row_keys to the end of unit_counts
    int32_t row_units, col_units;
    int64_t rows_cap, cols_cap;
    int32_t* unit_cursor;
    int32_t* lists;
    int32_t* chunk_unit;
    int32_t* chunk_totals;
    int32_t* block_counts;
    int64_t blocks_per_pair;
};
DenseLayout carve_dense(Carver& cv, int batch, int64_t n, int64_t m, int d, int compute) {
    DenseLayout L;
    L.maps = carve_maps(cv, batch, n, m, d, compute, 32 * DENSE_S);
    // the two key tables and the bucket counters are adjacent so that one range clears them all
    const size_t z0 = cv.used;
    L.row_keys = (u64*)cv.take((size_t)batch * (n + m) * sizeof(u64));
    L.col_keys = L.row_keys ? L.row_keys + (size_t)batch * n : nullptr;
    L.row_units = (int32_t)((L.maps.m_pad / 32 + DENSE_J - 1) / DENSE_J);
    L.col_units = (int32_t)(L.maps.n_pad / DENSE_S);
    const size_t units = (size_t)batch * ((size_t)L.row_units + L.col_units);
    L.unit_counts = (int32_t*)cv.take(units * sizeof(int32_t));
    L.zero_words = (int64_t)((cv.used - z0) / sizeof(u64));
    L.unit_cursor = (int32_t*)cv.take(units * sizeof(int32_t));
    L.rows_cap = round_up(n, 32) + 32 * (int64_t)L.row_units;
    L.cols_cap = round_up(m, 32) + 32 * (int64_t)L.col_units;
    L.lists = (int32_t*)cv.take((size_t)batch * (L.rows_cap + L.cols_cap) * sizeof(int32_t));
    L.chunk_unit = (int32_t*)cv.take((size_t)batch * ((L.rows_cap + L.cols_cap) / 32) * sizeof(int32_t));
    L.chunk_totals = (int32_t*)cv.take((size_t)batch * 2 * sizeof(int32_t));
    const int64_t most = n > m ? n : m;
    L.blocks_per_pair = (most + 1023) / 1024;
    L.block_counts = (int32_t*)cv.take((size_t)batch * (L.blocks_per_pair + 1) * sizeof(int32_t));
    return L;
}

// Room for the dense mode's 8-bit pass behind its own layout.
struct DenseCoarseLayout {
    DenseCoarseArgs args;  // of the first group of pairs
    int32_t group;         // pairs that share the tables of scores, one group after the other
    int32_t n_sb;  // runs of DENSE_SB_PIXELS of image 1
    int32_t slab;  // ... per launch
    int64_t sample_words;  // 32-bit words that start at 0, from args.sample_lower on
    char* swept;   // image 1 of a group as the dense kernels read it
};
DenseCoarseLayout carve_dense_coarse(Carver& cv, int batch, int64_t n, int64_t m, const MapsLayout& maps, int compute) {
    DenseCoarseLayout L;
    memset(&L, 0, sizeof(L));
    DenseCoarseArgs& a = L.args;
    a.seg_pixels = dense_seg_pixels(n);
    a.map[0] = carve_coarse_map(cv, batch, round_up(n, DENSE_SB_PIXELS), a.seg_pixels);
    a.map[1] = carve_coarse_map(cv, batch, round_up(m, DENSE_SB_PIXELS), a.seg_pixels);
    a.n_tiles[0] = (int32_t)((n + 31) / 32);
    a.n_tiles[1] = (int32_t)((m + 31) / 32);
    a.cell_runs = dense_cell_runs(n, m);
    a.grouped = dense_grouped(n, compute, maps.dp) ? 1 : 0;
    const int64_t cell = DENSE_CELL_PIXELS * a.cell_runs, col_cell = a.seg_pixels >> a.grouped;
    a.n_cells = (int32_t)((m + cell - 1) / cell);
    a.n_col_cells = (int32_t)((n + col_cell - 1) / col_cell);
    // Tables of scores: the candidates' of as many pairs at a time as 512 MB hold (all of a pair's), their queries' a run of 128 MB at a time.  (Groups
    // of four 512x384 pairs instead of eight cost 1 %.)
    const size_t pixels2 = (size_t)a.map[1].n_segs * a.seg_pixels;
    const size_t cols = a.map[0].n_segs * pixels2 * sizeof(uint16_t);  // one for every candidate and segment; groups in half segments need three quarters of that
    static_assert(2 * DENSE_CELL_GROUPS <= DENSE_CELL_PIXELS, "the groups' table fits in the other's place");
    const int64_t together = cols > 0 && cols < ((size_t)512 << 20) ? (int64_t)(((size_t)512 << 20) / cols) : 1;
    const int64_t groups = (batch + together - 1) / together;
    L.group = (int32_t)((batch + groups - 1) / groups);
    const int64_t per_sb = L.group * a.n_cells * (int64_t)DENSE_SB_PIXELS * (int64_t)sizeof(uint16_t);
    int64_t slab = ((int64_t)128 << 20) / (per_sb > 0 ? per_sb : 1);
    if (slab < 1) slab = 1;
    L.n_sb = (int32_t)((n + DENSE_SB_PIXELS - 1) / DENSE_SB_PIXELS);
    const int64_t launches = (L.n_sb + slab - 1) / slab;
    L.slab = launches > 0 ? (int32_t)((L.n_sb + launches - 1) / launches) : 1;
    a.best[0] = (uint16_t*)cv.take((size_t)per_sb * L.slab);
    a.best[1] = (uint16_t*)cv.take((size_t)L.group * cols);
    a.mask[0] = (uint64_t*)cv.take((size_t)per_sb * L.slab / 16);
    a.mask[1] = (uint64_t*)cv.take((size_t)L.group * ((size_t)a.map[0].n_segs << a.grouped) * pixels2 / 8);
    if (a.grouped) a.least = (float*)cv.take((size_t)L.group * (pixels2 / DENSE_CELL_PIXELS * DENSE_CELL_GROUPS) * sizeof(float));
    L.swept = (char*)cv.take((size_t)L.group * maps.bstride1);
    a.pixels[0] = n;
    a.pixels[1] = m;
    a.sample_upper[0] = (float*)cv.take((size_t)batch * a.n_cells * DENSE_SAMPLES * sizeof(float));
    a.sample_upper[1] = (float*)cv.take((size_t)batch * a.n_col_cells * DENSE_SAMPLES * sizeof(float));
    if (a.grouped) a.sample_group = (float*)cv.take((size_t)batch * a.n_col_cells * DENSE_SAMPLES * sizeof(float));
    const size_t zeros = cv.used;
    a.sample_lower = (uint32_t*)cv.take((size_t)batch * 2 * DENSE_SAMPLES * sizeof(uint32_t));
    if (a.grouped) a.sample_best = (uint32_t*)cv.take((size_t)batch * DENSE_SAMPLES * sizeof(uint32_t));
    a.marked = (int32_t*)cv.take((size_t)batch * DENSE_RECORD * sizeof(int32_t));
    a.filed = (uint32_t*)cv.take(sizeof(uint32_t));
    L.sample_words = (int64_t)((cv.used - zeros) / sizeof(uint32_t));
    return L;
}

// Room for the late iterations in one launch, behind everything else: a workspace that ends before it has them launched one by one.
struct TailLayout {
    TailControl* control;
    u64* few_keys;
    int64_t zero_words;  // 64-bit words that start at 0, from `control` on
};
TailLayout carve_tail(Carver& cv, int batch) {
    TailLayout L;
    const size_t z0 = cv.used;
    L.control = (TailControl*)cv.take((size_t)batch * sizeof(TailControl));
    L.few_keys = (u64*)cv.take((size_t)batch * 3 * TAIL_KEY_COPIES * TAIL_FEW * sizeof(u64));
    L.zero_words = (int64_t)((cv.used - z0) / sizeof(u64));
    return L;
}

bool shape_ok(int32_t batch, int64_t n, int64_t m, int32_t d, int64_t nq) {
    return batch >= 1 && batch <= FNN_MAX_BATCH && n >= 0 && m >= 0 && n <= MAX_PIXELS && m <= MAX_PIXELS &&
           d >= 1 && d <= FNN_MAX_D && nq >= 0 && nq <= MAX_PIXELS;
}

// Checks a host array of `batch` maps that must share shape and format.
int32_t check_maps(int32_t batch, const fnn_map* maps) {
    if (!maps) return FNN_E_NULL;
    for (int b = 0; b < batch; ++b) {
        const fnn_map& mp = maps[b];
        if (!valid_dtype(mp.dtype)) return FNN_E_DTYPE;
        if (mp.n < 0 || mp.n > MAX_PIXELS || mp.d < 1 || mp.d > FNN_MAX_D || mp.row_stride < mp.d) return FNN_E_SHAPE;
        if (mp.n != maps[0].n || mp.d != maps[0].d || mp.dtype != maps[0].dtype || mp.row_stride != maps[0].row_stride)
            return FNN_E_SHAPE;
        if (mp.n > 0 && !mp.data) return FNN_E_NULL;
    }
    return FNN_OK;
}

int32_t check_opts(const fnn_opts* o) {
    if (!o) return FNN_E_NULL;
    if (!valid_dtype(o->compute)) return FNN_E_DTYPE;
    if (o->max_iter < 0) return FNN_E_RANGE;
    if (o->flags & ~(FNN_FLAG_NORMALIZE | FNN_FLAG_HALF_ACCUMULATE | FNN_FLAG_L2 | FNN_FLAG_SPLIT)) return FNN_E_RANGE;
    for (int i = 0; i < 5; ++i)
        if (o->reserved[i] != 0) return FNN_E_RANGE;
    return FNN_OK;
}

// Channels the prepared rows must hold for this call (descriptor + L2 norm channels), or
// -1 when they do not fit the widest row the kernels take.
int32_t row_channels(int32_t d, const fnn_opts* o) {
    const bool split = (o->flags & FNN_FLAG_SPLIT) != 0;
    const int32_t de = effective_d(d, o->compute, (o->flags & FNN_FLAG_L2) != 0, split);
    return de <= (split ? MAX_ROW_CHANNELS : FNN_MAX_D) ? de : -1;
}
// FNN_FLAG_SPLIT is defined for fp16 products and the dot-product score only.
bool split_unsupported(const fnn_opts* o) {
    return (o->flags & FNN_FLAG_SPLIT) && (o->compute != FNN_F16 || (o->flags & FNN_FLAG_L2));
}

int32_t check_workspace(const void* ws, size_t have, size_t need) {
    if (need == 0) return FNN_OK;
    if (!ws || ((uintptr_t)ws % WS_ALIGN) != 0 || have < need) return FNN_E_WORKSPACE;
    return FNN_OK;
}

void fill_prep_side(PrepSide& sd, int32_t batch, const fnn_map* maps, int64_t n_pad, void* dst, int second_image) {
    memset(&sd, 0, sizeof(sd));
    sd.second_image = second_image;
    for (int b = 0; b < batch; ++b) sd.src[b] = maps[b].data;
    sd.n = maps[0].n;
    sd.n_pad = n_pad;
    sd.row_stride = maps[0].row_stride;
    sd.dtype = maps[0].dtype;
    sd.dst = dst;
}

// A batch of caller maps that already has the layout the kernels read: stored in the compute
// format, dp channels per row, rows packed, whole 32-pixel tiles, 16-byte aligned, and the
// pairs equally spaced in memory (one stacked array).  Such maps are used where they are.
bool direct_layout(int32_t batch, const fnn_map* maps, const fnn_opts* opts, int dp, const char** base, int64_t* bstride) {
    const fnn_map& m0 = maps[0];
    if (opts->flags != 0) return false;
    for (int b = 0; b < batch; ++b)
        if (maps[b].dtype != opts->compute || maps[b].d != dp || maps[b].row_stride != dp || maps[b].n != m0.n) return false;
    if (m0.n <= 0 || m0.n % 32 != 0 || ((uintptr_t)m0.data % 16) != 0) return false;
    const int64_t bytes = m0.n * dp * elem_size(opts->compute);
    int64_t stride = 0;
    if (batch > 1) {
        stride = (const char*)maps[1].data - (const char*)m0.data;
        if (stride < bytes || stride % 16 != 0) return false;
        for (int b = 2; b < batch; ++b)
            if ((const char*)maps[b].data != (const char*)m0.data + (int64_t)b * stride) return false;
    }
    *base = (const char*)m0.data;
    *bstride = stride;
    return true;
}

// Caller maps that the fused first searches can read where they are (they round the fp32 rows
// themselves and write the prepared copy as a by-product): plain fp32 rows of 24 channels that
// start on 16-byte boundaries, a 16-bit compute format, no options, enough queries.
bool raw_rows(int32_t batch, const fnn_map* maps) {
    for (int i = 0; i < batch; ++i)
        if (maps[i].dtype != FNN_F32 || maps[i].d != 24 || maps[i].row_stride % 4 != 0 || maps[i].n <= 0 ||
            ((uintptr_t)maps[i].data % 16) != 0)
            return false;
    return true;
}
bool raw_options(const fnn_opts* opts) {
    return opts->flags == 0 && (opts->compute == FNN_F16 || opts->compute == FNN_BF16);
}
// Maps that the quantise launch reads where they are, and prepares on the way: the same, and with two-term rows, or with rows that are to be normalised.
bool raw_quantise(int32_t batch, const fnn_map* a, const fnn_map* b, const fnn_opts* opts) {
    const bool normalised = opts->flags == FNN_FLAG_NORMALIZE && opts->compute != FNN_F32;
    return (raw_options(opts) || opts->flags == FNN_FLAG_SPLIT || normalised) && raw_rows(batch, a) && raw_rows(batch, b);
}
bool raw_first_search(int32_t batch, const fnn_map* a, const fnn_map* b, const fnn_opts* opts, int64_t n_queries) {
    return raw_options(opts) && first_search_applies(n_queries, a[0].n, batch) && first_search_applies(n_queries, b[0].n, batch) &&
           raw_rows(batch, a) && raw_rows(batch, b);
}
void fill_raw(RawMaps& r, int32_t batch, const fnn_map* maps) {
    memset(&r, 0, sizeof(r));
    for (int i = 0; i < batch; ++i) r.map[i] = (const float*)maps[i].data;
    r.row_stride = maps[0].row_stride;
}

// Prepares the maps that are not used in place (skip_a / skip_b) and runs the side jobs.
hipError_t prep_both(int32_t batch, const fnn_map* a, const fnn_map* b, const MapsLayout& L, int d, const fnn_opts* opts,
                     hipStream_t s, const PrepExtra& extra, bool first_segment_major = false, bool skip_a = false,
                     bool skip_b = false) {
    const int compute = opts->compute;
    PrepArgs pa;
    memset(&pa, 0, sizeof(pa));
    pa.extra = extra;
    int sides = 0;
    if (!skip_a) {
        fill_prep_side(pa.side[sides], batch, a, L.n_pad, L.p1, 0);
        pa.side[sides].segment_major = first_segment_major ? 1 : 0;
        ++sides;
    }
    if (!skip_b) {
        fill_prep_side(pa.side[sides], batch, b, L.m_pad, L.p2, 1);
        ++sides;
    }
    pa.n_sides = sides;
    pa.batch = batch;
    pa.d = d;
    pa.dp = L.dp;
    pa.compute = compute;
    pa.normalize = (opts->flags & FNN_FLAG_NORMALIZE) ? 1 : 0;
    pa.l2 = (opts->flags & FNN_FLAG_L2) ? 1 : 0;
    pa.split = (opts->flags & FNN_FLAG_SPLIT) ? 1 : 0;
    return launch_prep(pa, s);
}

// One side of the quantise launch; raw: the caller's fp32 maps are read, else the prepared ones at `prepared`.
void fill_quantise_side(QuantiseSide& sd, int32_t batch, const fnn_map* maps, bool raw, const char* prepared, int64_t bstride, int64_t n_pad,
                        const CoarseMap& out) {
    sd.prepared = prepared;
    sd.bstride = bstride;
    sd.n = maps[0].n;
    sd.n_pad = n_pad;
    if (raw)
        for (int b = 0; b < batch; ++b) sd.raw[b] = (const float*)maps[b].data;
    sd.raw_stride = maps[0].row_stride;
    sd.out = out;
}

// The pairs of a group: see dense_two_steps.
hipError_t dense_group(const DenseCoarseLayout& C, const DenseLayout& L, const SearchArgs& rows, const SearchArgs& cols, DenseCoarseArgs da, DenseArgs sweep,
                       bool at_once, int pairs, int compute, hipStream_t s) {
    CoarseArgs ca;
    memset(&ca, 0, sizeof(ca));
    ca.judge = sweep.judge = da.judge;
    hipError_t e = hipSuccess;
    const DenseSwept none = {}, swept = {rows.src, rows.src_bstride, C.swept, L.maps.n_pad, (int32_t)(L.maps.bstride1 / L.maps.n_pad)};
    for (int sb = 0; sb < C.n_sb; sb += C.slab) {
        da.first_sb = sb;
        da.n_sb = C.n_sb - sb < C.slab ? C.n_sb - sb : C.slab;
        da.swept = sb == 0 ? swept : none;
        e = launch_dense_coarse(da, pairs, s);
        if (e == hipSuccess) e = launch_dense_select(da, 0, at_once ? 2 : 1, nullptr, pairs, s);
        ca.mask = da.mask[0];
        ca.slab = da.n_sb * DENSE_SB_PIXELS;
        ca.n_cells = da.n_cells;
        ca.slot_pitch = (int64_t)da.n_cells * (ca.slab / 64);
        ca.cell_shift = da.cell_runs == 4 ? 2 : (da.cell_runs == 2 ? 1 : 0);
        ca.first_slot = sb * DENSE_SB_PIXELS;
        ca.side = 0;
        if (e == hipSuccess) e = launch_refine(rows, ca, pairs, compute, L.maps.dp, s);
        if (e != hipSuccess) return e;
    }
    if (!at_once) e = launch_dense_select(da, 1, 1, nullptr, pairs, s);
    ca.mask = da.mask[1];
    ca.slab = da.map[1].n_segs * da.seg_pixels;
    ca.n_cells = da.map[0].n_segs;
    ca.slot_pitch = (int64_t)(da.map[0].n_segs << da.grouped) * (ca.slab / 64);
    ca.cell_shift = da.seg_pixels == 4096 ? 2 : 1;
    ca.first_slot = 0;
    ca.side = 1;
    if (e == hipSuccess) e = launch_refine(cols, ca, pairs, compute, L.maps.dp, s);
    if (da.grouped) {
        if (e == hipSuccess) e = launch_dense_select(da, 1, 1, cols.out_keys, pairs, s);
        ca.second_round = 1;
        if (e == hipSuccess) e = launch_refine(cols, ca, pairs, compute, L.maps.dp, s);
    }
    sweep.d1 = C.swept;
    if (e == hipSuccess) e = launch_dense_pass1(sweep, pairs, compute, L.maps.dp, s);
    return e;
}

// Both directions of the dense mode from its 8-bit maps to the keys: pass 1 range by range of image 1, the second step for the queries
// of a range at once, for the candidates when every range is done; a group of pairs after the other.  Pairs whose samples say that this would be the slower way are swept
// by the dense kernels of `sweep` instead.
hipError_t dense_two_steps(const DenseCoarseLayout& C, const DenseLayout& L, int batch, int64_t n, int64_t m, int compute, bool l2, DenseArgs sweep, hipStream_t s) {
    SearchArgs rows;
    memset(&rows, 0, sizeof(rows));
    rows.src = (const char*)L.maps.p1;
    rows.src_bstride = L.maps.bstride1;
    rows.src_rows = (int32_t)L.maps.n_pad;
    rows.nq = (int32_t)n;
    rows.tgt = (const char*)L.maps.p2;
    rows.tgt_bstride = L.maps.bstride2;
    rows.m = (int32_t)m;
    rows.m_tiles = (int32_t)(L.maps.m_pad / 32);
    rows.out_keys = L.row_keys;
    SearchArgs cols = rows;
    cols.src = rows.tgt;
    cols.src_bstride = rows.tgt_bstride;
    cols.src_rows = (int32_t)L.maps.m_pad;
    cols.nq = (int32_t)m;
    cols.tgt = rows.src;
    cols.tgt_bstride = rows.src_bstride;
    cols.m = (int32_t)n;
    cols.m_tiles = (int32_t)((n + 31) / 32);
    cols.out_keys = L.col_keys;

    DenseCoarseArgs da = C.args;
    hipError_t e = launch_dense_sample(da, dense_costs(da, batch, compute, L.maps.dp, l2), batch, s);
    da.judge = {da.marked};
    // a launch that leaves every pair alone costs its workgroups' start: no more of them than fill the chip a few times
    auto wgs = [&]() { return (int64_t)C.group * sweep.n_sb * ((sweep.m_tiles + DENSE_TILES_PER_GROUP * sweep.groups_per_wg - 1) / (DENSE_TILES_PER_GROUP * sweep.groups_per_wg)); };
    while (wgs() > 4096) sweep.groups_per_wg *= 2;
    const bool at_once = C.slab >= C.n_sb;  // both sides' marks in one launch
    for (int b0 = 0; b0 < batch && e == hipSuccess; b0 += C.group) {
        const int pairs = batch - b0 < C.group ? batch - b0 : C.group;
        e = dense_group(C, L, rows, cols, da, sweep, at_once, pairs, compute, s);
        const int step = C.group;
        rows.src += step * rows.src_bstride;
        rows.tgt += step * rows.tgt_bstride;
        rows.out_keys += step * n;
        cols.src += step * cols.src_bstride;
        cols.tgt += step * cols.tgt_bstride;
        cols.out_keys += step * m;
        for (CoarseMap& map : da.map) {
            map.rows += (int64_t)step * map.n_segs * da.seg_pixels * COARSE_ROW_BYTES;
            map.row_bound += (int64_t)step * map.n_segs * da.seg_pixels;
            map.seg += (int64_t)step * map.n_segs;
        }
        da.judge.marked += DENSE_RECORD * step;
        sweep.d2 += step * sweep.d2_bstride;
        sweep.row_keys += step * n;
        sweep.col_keys += step * m;
    }
    return e;
}

#define FNN_TRY(expr)                        \
    do {                                     \
        if ((expr) != hipSuccess) return FNN_E_HIP; \
    } while (0)

}  // namespace

// ---- scratch of fnn_reciprocal_static ----------------------------------------------------------
// One array per device (every device that loads the library holds its own copy at its own
// address, for the life of the process).  In host code the array's name is only a handle: the
// memory is reached through the address that hipGetSymbolAddress returns for the current device,
// looked up once per device and kept.
static __device__ __align__(256) unsigned char scratch[FNN_STATIC_SCRATCH_BYTES];

static struct StaticScratch {
    std::mutex mu;
    void* ptr[DeviceCache::MAX_DEVICES] = {};
} g_static_scratch;

// Address of the current device's scratch array, or NULL (a HIP call failed).  Allocates nothing.
static void* static_scratch_for_current_device() {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= DeviceCache::MAX_DEVICES) return nullptr;
    std::lock_guard<std::mutex> lock(g_static_scratch.mu);
    if (!g_static_scratch.ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
            (void)hipGetLastError();
            return nullptr;
        }
        g_static_scratch.ptr[dev] = p;
    }
    return g_static_scratch.ptr[dev];
}

#pragma GCC visibility push(default)
extern "C" {

const char* fnn_status_string(int32_t status) {
    switch (status) {
        case FNN_OK: return "ok";
        case FNN_E_NULL: return "a required pointer is NULL";
        case FNN_E_SHAPE: return "shape out of range or inconsistent";
        case FNN_E_DTYPE: return "unknown storage or compute format";
        case FNN_E_RANGE: return "option out of range";
        case FNN_E_WORKSPACE: return "workspace missing, misaligned or too small";
        case FNN_E_HIP: return "a HIP call or kernel launch failed";
        case FNN_E_UNSUPPORTED: return "request not supported by this build";
        default: return "unknown status";
    }
}

size_t fnn_workspace_bytes_opts(int32_t batch, int64_t n, int64_t m, int32_t d, int64_t n_queries,
                                const fnn_opts* opts) {
    if (!shape_ok(batch, n, m, d, n_queries) || check_opts(opts) != FNN_OK || split_unsupported(opts)) return 0;
    const int32_t de = row_channels(d, opts);
    if (de < 0) return 0;
    const int32_t compute = opts->compute;
    size_t most = 0;
    const int dp = padded_d(de, compute);
    const bool l2 = (opts->flags & FNN_FLAG_L2) != 0;
    {
        Carver cv{nullptr, 0};
        carve_nearest(cv, batch, n, m, de, n_queries, compute);
        most = cv.used;
        // the queries' own rows, or their whole map, whichever the call may need
        for (int listed = 0; listed < 2; ++listed) {
            if (!nearest_coarse_searches(batch, n, m, n_queries, listed != 0, compute, dp, d, l2)) continue;
            Carver with = cv;
            carve_coarse(with, batch, listed ? n_queries : n, m, false, n_queries, 1, compute);
            if (with.used > most) most = with.used;
        }
    }
    {
        Carver cv{nullptr, 0};
        carve_recip(cv, batch, n, m, de, n_queries, compute);
        if (recip_coarse_searches(batch, n, m, n_queries, compute, dp, d, l2))
            carve_coarse(cv, batch, n, m, true, n_queries, RECIP_COARSE_SEARCHES, compute);
        carve_tail(cv, batch);
        if (cv.used > most) most = cv.used;
    }
    {
        Carver cv{nullptr, 0};
        const DenseLayout D = carve_dense(cv, batch, n, m, de, compute);
        if (n <= MAX_DENSE_PIXELS && m <= MAX_DENSE_PIXELS && dense_coarse_gain(n, m, batch, compute, dp, d, l2) > 0.0)
            carve_dense_coarse(cv, batch, n, m, D.maps, compute);
        if (cv.used > most) most = cv.used;
    }
    return most + WS_ALIGN;
}

size_t fnn_workspace_bytes(int32_t batch, int64_t n, int64_t m, int32_t d, int64_t n_queries, int32_t compute) {
    fnn_opts o;
    memset(&o, 0, sizeof(o));
    o.compute = compute;
    return fnn_workspace_bytes_opts(batch, n, m, d, n_queries, &o);
}

int32_t fnn_nearest(int32_t batch, const fnn_map* src, const int32_t* q_idx, int64_t nq, const int32_t* nq_active,
                    const fnn_map* tgt, const fnn_opts* opts, int32_t* out_idx, float* out_score, void* workspace,
                    size_t workspace_bytes, void* stream) {
    if (batch < 1 || batch > FNN_MAX_BATCH) return FNN_E_SHAPE;
    int32_t st = check_maps(batch, src);
    if (st != FNN_OK) return st;
    st = check_maps(batch, tgt);
    if (st != FNN_OK) return st;
    st = check_opts(opts);
    if (st != FNN_OK) return st;
    if ((opts->flags & FNN_FLAG_HALF_ACCUMULATE) || split_unsupported(opts)) return FNN_E_UNSUPPORTED;
    const int64_t n = src[0].n, m = tgt[0].n;
    const int32_t d = src[0].d;
    if (tgt[0].d != d || nq < 0 || nq > MAX_PIXELS) return FNN_E_SHAPE;
    const int32_t de = row_channels(d, opts);
    if (de < 0) return FNN_E_SHAPE;
    if (!q_idx && nq > n) return FNN_E_SHAPE;
    if (nq > 0 && n == 0) return FNN_E_SHAPE;
    if (nq > 0 && !out_idx) return FNN_E_NULL;
    if (nq == 0) return FNN_OK;

    Carver cv{(char*)workspace, 0};
    NearestLayout L = carve_nearest(cv, batch, n, m, de, nq, opts->compute);
    st = check_workspace(workspace, workspace_bytes, cv.used);
    if (st != FNN_OK) return st;
    hipStream_t s = (hipStream_t)stream;

    PrepExtra extra;
    memset(&extra, 0, sizeof(extra));
    extra.zero_ptr = L.keys;  // the key table starts empty
    extra.zero_count = (int64_t)batch * nq;
    const char *p1 = (const char*)L.maps.p1, *p2 = (const char*)L.maps.p2;
    int64_t bs1 = L.maps.bstride1, bs2 = L.maps.bstride2;
    const bool direct1 = direct_layout(batch, src, opts, L.maps.dp, &p1, &bs1);
    const bool direct2 = direct_layout(batch, tgt, opts, L.maps.dp, &p2, &bs2);
    // With every query live and enough of them, the search runs in the kernel that stages the
    // candidate tiles through LDS; fp32 maps of the paper's shape are then read where they are (no
    // prepare pass: the search leaves the prepared candidates behind for the resolve pass).
    const bool staged_shape = !nq_active && first_search_applies(nq, m, batch);
    const bool fused = staged_shape && raw_options(opts) && raw_rows(batch, src) && raw_rows(batch, tgt);
    const bool staged = fused || (staged_shape && L.maps.dp == 24 && opts->compute != FNN_F32);
    // ... or, where that is faster and the workspace has the room, in two steps, the first in 8 bits
    const bool listed = list_queries(q_idx, nq, n);
    CoarseLayout C = carve_coarse(cv, batch, listed ? nq : n, m, false, nq, 1, opts->compute);
    const bool coarse = !nq_active && cv.used <= workspace_bytes &&
                        nearest_coarse_searches(batch, n, m, nq, listed, opts->compute, L.maps.dp, d, (opts->flags & FNN_FLAG_L2) != 0);
    const bool raw = coarse && raw_quantise(batch, src, tgt, opts);
    const bool prepared = raw || (coarse && direct1 && direct2);  // the quantise launch is the first, and takes the side jobs
    if (!prepared) FNN_TRY(prep_both(batch, src, tgt, L.maps, d, opts, s, extra, false, direct1 || fused, direct2 || fused));
    SearchArgs sa;
    memset(&sa, 0, sizeof(sa));
    sa.src = p1;
    sa.src_bstride = bs1;
    sa.src_rows = (int32_t)L.maps.n_pad;
    sa.q_idx = q_idx;
    sa.nq_active = nq_active;
    sa.nq = (int32_t)nq;
    sa.tgt = p2;
    sa.tgt_bstride = bs2;
    sa.m = (int32_t)m;
    sa.m_tiles = (int32_t)(L.maps.m_pad / 32);
    sa.out_keys = L.keys;
    if (coarse) {
        QuantiseArgs qa;
        memset(&qa, 0, sizeof(qa));
        if (prepared) qa.extra = extra;
        fill_quantise_side(qa.side[0], batch, src, raw, p1, bs1, L.maps.n_pad, C.map[0]);
        fill_quantise_side(qa.side[1], batch, tgt, raw, p2, bs2, L.maps.m_pad, C.map[1]);
        if (listed) {
            qa.side[0].gather = q_idx;
            qa.side[0].gather_rows = n;
            qa.side[0].n = nq;
            if (raw) {  // the prepared copy of image 1 holds the listed rows only
                qa.side[0].n_pad = nq;
                sa.q_idx = nullptr;
                sa.src_rows = (int32_t)nq;
            }
        }
        qa.batch = batch;
        qa.raw_rows = raw ? 1 : 0;
        qa.normalize = (opts->flags & FNN_FLAG_NORMALIZE) ? 1 : 0;
        qa.seg_pixels = SEG_PIXELS;
        qa.lower = C.lower;
        qa.lower_count = C.zero_words;
        qa.split_d = (opts->flags & FNN_FLAG_SPLIT) ? d : 0;
        FNN_TRY(launch_quantise(qa, opts->compute, L.maps.dp, s));
        CoarseArgs ca = coarse_args(C, batch, 0, 0, coarse_votes(opts->compute, L.maps.dp));
        ca.src_listed = listed ? 1 : 0;
        FNN_TRY(launch_coarse_search(sa, ca, batch, opts->compute, L.maps.dp, s));
    } else if (staged) {
        FirstSearchArgs first;
        memset(&first, 0, sizeof(first));
        first.s = sa;
        if (fused) {
            first.s.src_rows = (int32_t)n;  // query rows are clamped to the caller's map, which has no padding rows
            fill_raw(first.raw_tgt, batch, tgt);
            fill_raw(first.raw_src, batch, src);
            first.raw_queries = 1;
        }
        FNN_TRY(launch_search_first(first, batch, opts->compute, s));
        if (fused) {
            FNN_TRY(launch_resolve_raw(first, batch, opts->compute, out_idx, out_score, nullptr, s));
            return FNN_OK;
        }
    } else {
        FNN_TRY(launch_search(sa, batch, opts->compute, L.maps.dp, s));
    }
    FNN_TRY(launch_resolve(sa, batch, opts->compute, L.maps.dp, out_idx, out_score, nullptr, s));
    return FNN_OK;
}

size_t fnn_blocked_workspace_bytes(int64_t n, int64_t m, int32_t d, int32_t block_rows, int32_t block_cols,
                                   int32_t compute) {
    if (!shape_ok(1, n, m, d, 0) || !valid_dtype(compute) || block_rows < 1 || block_cols < 0) return 0;
    Carver cv{nullptr, 0};
    carve_maps(cv, 1, n, m, d, compute);
    const int64_t ld = block_cols > 0 ? round_up(block_cols, 32) : round_up(m, 32);
    cv.take((size_t)block_rows * ld * sizeof(float));
    return cv.used + WS_ALIGN;
}

int32_t fnn_nearest_blocked(const fnn_map* src, const int32_t* q_idx, int64_t nq, const fnn_map* tgt,
                            const fnn_opts* opts, int32_t block_rows, int32_t block_cols, int32_t* out_idx,
                            float* out_score, void* workspace, size_t workspace_bytes, void* stream) {
    int32_t st = check_maps(1, src);
    if (st != FNN_OK) return st;
    st = check_maps(1, tgt);
    if (st != FNN_OK) return st;
    st = check_opts(opts);
    if (st != FNN_OK) return st;
    if ((opts->flags & FNN_FLAG_HALF_ACCUMULATE) && opts->compute != FNN_F16) return FNN_E_UNSUPPORTED;
    if (opts->flags & (FNN_FLAG_L2 | FNN_FLAG_SPLIT)) return FNN_E_UNSUPPORTED;
    const int64_t n = src[0].n, m = tgt[0].n;
    const int32_t d = src[0].d;
    if (tgt[0].d != d || nq < 0 || nq > MAX_PIXELS || block_rows < 1 || block_cols < 0) return FNN_E_SHAPE;
    if ((!q_idx && nq > n) || (nq > 0 && n == 0)) return FNN_E_SHAPE;
    if (nq > 0 && (!out_idx || !out_score)) return FNN_E_NULL;
    if (nq == 0) return FNN_OK;

    Carver cv{(char*)workspace, 0};
    MapsLayout L = carve_maps(cv, 1, n, m, d, opts->compute);
    const int64_t ld = block_cols > 0 ? round_up(block_cols, 32) : round_up(m, 32);
    float* dists = (float*)cv.take((size_t)block_rows * ld * sizeof(float));
    st = check_workspace(workspace, workspace_bytes, cv.used);
    if (st != FNN_OK) return st;
    hipStream_t s = (hipStream_t)stream;

    PrepExtra extra;
    memset(&extra, 0, sizeof(extra));
    FNN_TRY(prep_both(1, src, tgt, L, d, opts, s, extra));
    if (m == 0) {
        FNN_TRY(launch_fill_i32f32(out_idx, out_score, nq, s));
        return FNN_OK;
    }
    BlockedArgs ba;
    memset(&ba, 0, sizeof(ba));
    ba.src = (const char*)L.p1;
    ba.src_rows = (int32_t)L.n_pad;
    ba.q_idx = q_idx;
    ba.nq = (int32_t)nq;
    ba.tgt = (const char*)L.p2;
    ba.m = (int32_t)m;
    ba.dists = dists;
    ba.ld = ld;
    ba.out_idx = out_idx;
    ba.out_score = out_score;
    ba.half_accumulate = (opts->flags & FNN_FLAG_HALF_ACCUMULATE) ? 1 : 0;
    FNN_TRY(run_blocked(ba, opts->compute, d, L.dp, block_rows, (int)(block_cols > 0 ? ld : 0), s));
    return FNN_OK;
}

// The FastNN iteration.  use_static: the workspace is the library's own scratch array of the
// current device (looked up only after every argument check has passed).
static int32_t reciprocal_impl(int32_t batch, const fnn_map* d1, const fnn_map* d2, const int32_t* seeds, int64_t n_seeds,
                               const fnn_opts* opts, int32_t* seed_i, int32_t* seed_j, int32_t* seed_iter, int32_t* pairs,
                               int32_t* n_pairs, void* workspace, size_t workspace_bytes, bool use_static, void* stream) {
    if (batch < 1 || batch > FNN_MAX_BATCH) return FNN_E_SHAPE;
    int32_t st = check_maps(batch, d1);
    if (st != FNN_OK) return st;
    st = check_maps(batch, d2);
    if (st != FNN_OK) return st;
    st = check_opts(opts);
    if (st != FNN_OK) return st;
    if ((opts->flags & FNN_FLAG_HALF_ACCUMULATE) || split_unsupported(opts)) return FNN_E_UNSUPPORTED;
    const int64_t n = d1[0].n, m = d2[0].n;
    const int32_t d = d1[0].d;
    if (d2[0].d != d || n_seeds < 0 || n_seeds > MAX_PIXELS) return FNN_E_SHAPE;
    const int32_t de = row_channels(d, opts);
    if (de < 0) return FNN_E_SHAPE;
    if (n_seeds > 0 && (n == 0 || m == 0)) return FNN_E_SHAPE;
    if (!n_pairs) return FNN_E_NULL;
    if (n_seeds > 0 && (!seeds || !seed_i || !seed_j || !seed_iter || !pairs)) return FNN_E_NULL;

    if (use_static) {
        Carver need{nullptr, 0};
        carve_recip(need, batch, n, m, de, n_seeds, opts->compute);
        if (need.used > FNN_STATIC_SCRATCH_BYTES) return FNN_E_WORKSPACE;  // before the device is touched
        workspace = static_scratch_for_current_device();
        if (!workspace) return FNN_E_HIP;
        workspace_bytes = FNN_STATIC_SCRATCH_BYTES;
    }
    Carver cv{(char*)workspace, 0};
    RecipLayout L = carve_recip(cv, batch, n, m, de, n_seeds, opts->compute);
    st = check_workspace(workspace, workspace_bytes, cv.used);
    if (st != FNN_OK) return st;
    hipStream_t s = (hipStream_t)stream;
    const int compute = opts->compute;
    const int32_t ns = (int32_t)n_seeds;

    if (ns == 0) {
        // nothing to match: only the counts are defined
        RecipState none = L.st;
        none.n_words = 0;
        FNN_TRY(launch_recip_dedup(none, 0, batch, seed_i, seed_j, seed_iter, pairs, n_pairs, s));
        return FNN_OK;
    }

    // the prepare launch also clears the key tables and the sort bitmap and sets U^0 = seeds (a small
    // pair's own workgroup keeps all of that in LDS)
    const char *p1 = (const char*)L.maps.p1, *p2 = (const char*)L.maps.p2;
    int64_t bs1 = L.maps.bstride1, bs2 = L.maps.bstride2;
    const bool direct1 = direct_layout(batch, d1, opts, L.maps.dp, &p1, &bs1);
    const bool direct2 = direct_layout(batch, d2, opts, L.maps.dp, &p2, &bs2);
    const bool one_group = walk_applies(n, m, n_seeds, opts->max_iter, compute, L.maps.dp);
    const bool walk = one_group || (!(direct1 && direct2) && groups_apply(n, m, n_seeds, batch, opts->max_iter, compute, L.maps.dp));
    PrepExtra extra;
    memset(&extra, 0, sizeof(extra));
    if (!walk) {
        extra.zero_ptr = L.st.keys_f;
        extra.zero_count = L.zero_words;
        extra.seeds = seeds;
        extra.cur_u = L.st.cur_u[0];
        extra.seed_id = L.st.seed_id[0];
        extra.n_active = L.st.n_active[0];
        extra.n_seeds = ns;
    }
    // fp32 maps of the paper's shape: no prepare pass; the first forward and the first backward
    // search read the caller's maps and leave the prepared copies behind for the later searches
    const bool fused = !walk && raw_first_search(batch, d1, d2, opts, n_seeds);
    // the same LDS-staged kernel serves the first two searches on prepared 24-channel maps
    const bool staged = fused || (L.maps.dp == 24 && opts->compute != FNN_F32 && first_search_applies(n_seeds, n, batch) &&
                                  first_search_applies(n_seeds, m, batch));
    // ... and large ones run in two steps, the first in 8 bits, where the workspace has the room
    Carver behind = cv;
    CoarseLayout C = carve_coarse(behind, batch, n, m, true, n_seeds, RECIP_COARSE_SEARCHES, compute);
    const int coarse_searches = walk || behind.used > workspace_bytes ? 0 : recip_coarse_searches(batch, n, m, n_seeds, compute, L.maps.dp, d,
                                                                                                  (opts->flags & FNN_FLAG_L2) != 0);
    const bool coarse = coarse_searches > 0;
    if (coarse) cv = behind;
    // the late iterations are one launch
    const TailLayout T = carve_tail(cv, batch);
    const int tail_from = walk || cv.used > workspace_bytes ? -1 : first_late_iteration(batch, n_seeds, opts->max_iter, coarse);
    const bool tail = tail_from >= 0;
    if (tail) {
        extra.zero_more = (u64*)T.control;
        extra.zero_more_count = T.zero_words;
        extra.seed_iter = seed_iter;  // a seed that the late iterations give up is none that the final sort looks at
    }
    const bool raw = coarse && raw_quantise(batch, d1, d2, opts);
    const bool prepared = raw || (coarse && direct1 && direct2);  // the quantise launch is the first, and takes the side jobs
    if (!prepared) FNN_TRY(prep_both(batch, d1, d2, L.maps, d, opts, s, extra, false, direct1 || fused, direct2 || fused));
    if (coarse) {
        QuantiseArgs qa;
        memset(&qa, 0, sizeof(qa));
        if (prepared) qa.extra = extra;
        fill_quantise_side(qa.side[0], batch, d1, raw, p1, bs1, L.maps.n_pad, C.map[0]);
        fill_quantise_side(qa.side[1], batch, d2, raw, p2, bs2, L.maps.m_pad, C.map[1]);
        qa.batch = batch;
        qa.raw_rows = raw ? 1 : 0;
        qa.normalize = (opts->flags & FNN_FLAG_NORMALIZE) ? 1 : 0;
        qa.seg_pixels = SEG_PIXELS;
        qa.lower = C.lower;
        qa.lower_count = C.zero_words;
        qa.split_d = (opts->flags & FNN_FLAG_SPLIT) ? d : 0;
        FNN_TRY(launch_quantise(qa, compute, L.maps.dp, s));
    }

    if (walk) {
        WalkArgs wa;
        memset(&wa, 0, sizeof(wa));
        wa.p1 = p1;
        wa.p2 = p2;
        wa.bstride1 = bs1;
        wa.bstride2 = bs2;
        wa.rows1 = (int32_t)L.maps.n_pad;
        wa.n = (int32_t)n;
        wa.m = (int32_t)m;
        wa.n_words = (int32_t)L.st.n_words;
        wa.seeds = seeds;
        wa.n_seeds = ns;
        wa.max_iter = opts->max_iter;
        wa.seed_i = seed_i;
        wa.seed_j = seed_j;
        wa.seed_iter = seed_iter;
        wa.pairs = pairs;
        wa.n_pairs = n_pairs;
        if (one_group) {
            FNN_TRY(launch_walk(wa, batch, compute, L.maps.dp, s));
        } else {
            FNN_TRY(launch_groups(wa, batch, compute, L.maps.dp, s));
            FNN_TRY(launch_recip_dedup(L.st, ns, batch, seed_i, seed_j, seed_iter, pairs, n_pairs, s));
        }
        return FNN_OK;
    }

    SearchArgs fwd;  // queries in image 1 -> candidates in image 2
    memset(&fwd, 0, sizeof(fwd));
    fwd.src = p1;
    fwd.src_bstride = bs1;
    fwd.src_rows = (int32_t)L.maps.n_pad;
    fwd.nq = ns;
    fwd.tgt = p2;
    fwd.tgt_bstride = bs2;
    fwd.m = (int32_t)m;
    fwd.m_tiles = (int32_t)(L.maps.m_pad / 32);
    fwd.out_keys = L.st.keys_f;

    SearchArgs bwd;  // queries in image 2 (named by the index field of keys_f) -> image 1
    memset(&bwd, 0, sizeof(bwd));
    bwd.src = p2;
    bwd.src_bstride = bs2;
    bwd.src_rows = (int32_t)L.maps.m_pad;
    bwd.q_keys = L.st.keys_f;
    bwd.nq = ns;
    bwd.tgt = p1;
    bwd.tgt_bstride = bs1;
    bwd.m = (int32_t)n;
    bwd.m_tiles = (int32_t)(L.maps.n_pad / 32);
    bwd.out_keys = L.st.keys_b;

    StepArgs step;  // bookkeeping of an iteration, in the launch that resolves its search back
    memset(&step, 0, sizeof(step));
    step.keys_f = L.st.keys_f;
    step.seed_i = seed_i;
    step.seed_j = seed_j;
    step.seed_iter = seed_iter;

    int which = 0;
    auto take_state = [&](int w) {  // the searches and the bookkeeping read half w of the ping-pong state
        which = w;
        fwd.q_idx = L.st.cur_u[w];
        fwd.nq_active = bwd.nq_active = L.st.n_active[w];
        step.cur_u = L.st.cur_u[w];
        step.seed_id = L.st.seed_id[w];
        step.next_u = L.st.cur_u[w ^ 1];
        step.next_seed_id = L.st.seed_id[w ^ 1];
        step.next_active = L.st.n_active[w ^ 1];  // emptied by the resolve pass of the search forward
    };
    take_state(0);
    // search number k of the call (out 0, back 0, out 1, ...): the first few may run in two steps
    auto search = [&](const SearchArgs& a, int k) -> hipError_t {
        if (k >= coarse_searches) return launch_search(a, batch, compute, L.maps.dp, s);
        const bool votes = coarse_votes(compute, L.maps.dp);
        CoarseArgs ca = coarse_args(C, batch, k & 1, k, votes && k < 2);
        if (votes && k >= 1) ca.earlier = C.votes + (int64_t)(k >= 2 ? k - 2 : 0) * batch;
        ca.min_live = k < 2 ? 0 : coarse_min_live(compute, L.maps.dp);
        return launch_coarse_search(a, ca, batch, compute, L.maps.dp, s);
    };
    // the iterations from t0 on, for the seeds of the half that take_state() chose
    auto late_iterations = [&](int t0) -> hipError_t {
        TailArgs ta;
        memset(&ta, 0, sizeof(ta));
        ta.p1 = p1;
        ta.p2 = p2;
        ta.bstride1 = bs1;
        ta.bstride2 = bs2;
        ta.rows1 = fwd.src_rows;
        ta.rows2 = bwd.src_rows;
        ta.n = (int32_t)n;
        ta.m = (int32_t)m;
        ta.n_seeds = ns;
        for (int w = 0; w < 2; ++w) {
            ta.cur_u[w] = L.st.cur_u[w];
            ta.seed_id[w] = L.st.seed_id[w];
        }
        ta.half = which;
        ta.n_active = L.st.n_active[which];
        ta.keys = L.st.keys_f;  // empty, like keys_b, of which the tail keeps V^t in the first half
        ta.v = (int32_t*)L.st.keys_b;
        ta.few_keys = T.few_keys;
        ta.control = T.control;
        ta.t0 = t0;
        ta.max_iter = opts->max_iter;
        ta.most_polls = tail_most_polls(n, m, ns);
        ta.seed_i = seed_i;
        ta.seed_j = seed_j;
        ta.seed_iter = seed_iter;
        return launch_tail(ta, batch, compute, L.maps.dp, s);
    };
    const bool fuse_first = fused && !coarse, stage_first = staged && !coarse;
    if (tail_from == 0) {
        FNN_TRY(late_iterations(0));
    } else if (fuse_first) {
        FirstSearchArgs first;  // V^0 = NN_2(U^0): queries and candidates still raw; writes the prepared image 2
        first.s = fwd;
        first.s.src_rows = (int32_t)n;  // query rows are clamped to the caller's map, which has no padding rows
        fill_raw(first.raw_tgt, batch, d2);
        fill_raw(first.raw_src, batch, d1);
        first.raw_queries = 1;
        FNN_TRY(launch_search_first(first, batch, compute, s));
        FNN_TRY(launch_resolve_raw(first, batch, compute, nullptr, nullptr, step.next_active, s));
    } else if (stage_first) {
        FirstSearchArgs first;
        memset(&first, 0, sizeof(first));
        first.s = fwd;
        FNN_TRY(launch_search_first(first, batch, compute, s));
        FNN_TRY(launch_resolve(fwd, batch, compute, L.maps.dp, nullptr, nullptr, step.next_active, s));
    } else {
        FNN_TRY(search(fwd, 0));  // V^0 = NN_2(U^0)
        FNN_TRY(launch_resolve(fwd, batch, compute, L.maps.dp, nullptr, nullptr, step.next_active, s));
    }
    if (opts->max_iter == 0) {
        step.mode = 2;
        FNN_TRY(launch_resolve_step(bwd, step, batch, compute, L.maps.dp, s));
    }
    for (int t = 0; t < opts->max_iter && tail_from != 0; ++t) {
        const bool last = (t == opts->max_iter - 1);
        if (stage_first && t == 0) {
            FirstSearchArgs first;  // U^1 = NN_1(V^0): queries from the prepared image 2; if raw, writes the prepared image 1
            memset(&first, 0, sizeof(first));
            first.s = bwd;
            if (fuse_first) fill_raw(first.raw_tgt, batch, d1);
            FNN_TRY(launch_search_first(first, batch, compute, s));
        } else {
            FNN_TRY(search(bwd, 2 * t + 1));  // U^{t+1} = NN_1(V^t)
        }
        step.t = t;
        step.mode = last ? 1 : 0;
        FNN_TRY(launch_resolve_step(bwd, step, batch, compute, L.maps.dp, s));
        if (last) break;
        take_state(which ^ 1);
        if (t + 1 == tail_from) {
            FNN_TRY(late_iterations(t + 1));
            break;
        }
        FNN_TRY(search(fwd, 2 * t + 2));  // V^{t+1} = NN_2(U^{t+1})
        FNN_TRY(launch_resolve(fwd, batch, compute, L.maps.dp, nullptr, nullptr, step.next_active, s));
    }
    FNN_TRY(launch_recip_dedup(L.st, ns, batch, seed_i, seed_j, seed_iter, pairs, n_pairs, s));
    return FNN_OK;
}

int32_t fnn_reciprocal(int32_t batch, const fnn_map* d1, const fnn_map* d2, const int32_t* seeds, int64_t n_seeds,
                       const fnn_opts* opts, int32_t* seed_i, int32_t* seed_j, int32_t* seed_iter, int32_t* pairs,
                       int32_t* n_pairs, void* workspace, size_t workspace_bytes, void* stream) {
    return reciprocal_impl(batch, d1, d2, seeds, n_seeds, opts, seed_i, seed_j, seed_iter, pairs, n_pairs, workspace,
                           workspace_bytes, false, stream);
}

int32_t fnn_reciprocal_static(int32_t batch, const fnn_map* d1, const fnn_map* d2, const int32_t* seeds, int64_t n_seeds,
                              const fnn_opts* opts, int32_t* seed_i, int32_t* seed_j, int32_t* seed_iter, int32_t* pairs,
                              int32_t* n_pairs, void* stream) {
    return reciprocal_impl(batch, d1, d2, seeds, n_seeds, opts, seed_i, seed_j, seed_iter, pairs, n_pairs, nullptr, 0,
                           true, stream);
}

int32_t fnn_mutual_dense(int32_t batch, const fnn_map* d1, const fnn_map* d2, const fnn_opts* opts, int32_t* nn12,
                         float* s12, int32_t* nn21, float* s21, int32_t* pairs, int32_t* n_pairs, void* workspace,
                         size_t workspace_bytes, void* stream) {
    if (batch < 1 || batch > FNN_MAX_BATCH) return FNN_E_SHAPE;
    int32_t st = check_maps(batch, d1);
    if (st != FNN_OK) return st;
    st = check_maps(batch, d2);
    if (st != FNN_OK) return st;
    st = check_opts(opts);
    if (st != FNN_OK) return st;
    if ((opts->flags & FNN_FLAG_HALF_ACCUMULATE) || split_unsupported(opts)) return FNN_E_UNSUPPORTED;
    const int64_t n = d1[0].n, m = d2[0].n;
    const int32_t d = d1[0].d;
    if (d2[0].d != d) return FNN_E_SHAPE;
    if (n > MAX_DENSE_PIXELS || m > MAX_DENSE_PIXELS) return FNN_E_SHAPE;
    const int32_t de = row_channels(d, opts);
    if (de < 0) return FNN_E_SHAPE;
    if (!n_pairs) return FNN_E_NULL;
    if ((n > 0 && !nn12) || (m > 0 && !nn21)) return FNN_E_NULL;
    if (n > 0 && m > 0 && !pairs) return FNN_E_NULL;

    Carver cv{(char*)workspace, 0};
    DenseLayout L = carve_dense(cv, batch, n, m, de, opts->compute);
    st = check_workspace(workspace, workspace_bytes, cv.used);
    if (st != FNN_OK) return st;
    hipStream_t s = (hipStream_t)stream;

    PrepExtra extra;
    memset(&extra, 0, sizeof(extra));
    extra.zero_ptr = L.row_keys;  // both key tables and the bucket counters start empty
    extra.zero_count = L.zero_words;
    DenseFinalArgs fa;
    fa.n = (int32_t)n;
    fa.m = (int32_t)m;
    fa.nn12 = nn12;
    fa.nn21 = nn21;
    fa.pairs = pairs;
    fa.n_pairs = n_pairs;
    fa.block_counts = L.block_counts;

    DenseArgs da;
    memset(&da, 0, sizeof(da));
    da.d1 = (const char*)L.maps.p1;
    da.d1_bstride = L.maps.bstride1;
    da.d2 = (const char*)L.maps.p2;
    da.d2_bstride = L.maps.bstride2;
    da.n = (int32_t)n;
    da.m = (int32_t)m;
    da.n_sb = (int32_t)(L.maps.n_pad / (32 * DENSE_S));
    da.m_tiles = (int32_t)(L.maps.m_pad / 32);
    da.row_keys = L.row_keys;
    da.col_keys = L.col_keys;
    da.row_units = L.row_units;
    da.col_units = L.col_units;
    da.rows_cap = L.rows_cap;
    da.cols_cap = L.cols_cap;
    da.unit_counts = L.unit_counts;
    da.unit_cursor = L.unit_cursor;
    da.lists = L.lists;
    da.chunk_unit = L.chunk_unit;
    da.chunk_totals = L.chunk_totals;

    // Workgroup tile: one query super-block (32 KB of LDS keys) x up to 8 candidate groups (of
    // DENSE_WAVES x DENSE_J tiles).  Larger tiles mean fewer merges into the global key
    // tables; small problems shrink the tile until the grid covers the chip a few times.
    const int64_t groups_total = (da.m_tiles + DENSE_TILES_PER_GROUP - 1) / DENSE_TILES_PER_GROUP;
    const int64_t sb_per_wg = 1;
    int64_t groups_per_wg = 8;
    auto wg_count = [&]() {
        return ((da.n_sb + sb_per_wg - 1) / sb_per_wg) * ((groups_total + groups_per_wg - 1) / groups_per_wg) * batch;
    };
    while (groups_per_wg > 1 && wg_count() < 1024) groups_per_wg >>= 1;
    da.sb_per_wg = (int32_t)sb_per_wg;
    da.groups_per_wg = (int32_t)groups_per_wg;

    // Large maps: 8-bit scores first, then, where the workspace has the room, the second step of the searches in both directions
    DenseCoarseLayout C = carve_dense_coarse(cv, batch, n, m, L.maps, opts->compute);
    const bool l2 = (opts->flags & FNN_FLAG_L2) != 0;
    if (cv.used <= workspace_bytes && dense_coarse_gain(n, m, batch, opts->compute, L.maps.dp, d, l2) > 0.0) {
        const bool raw = raw_quantise(batch, d1, d2, opts);
        if (!raw) FNN_TRY(prep_both(batch, d1, d2, L.maps, d, opts, s, extra));
        QuantiseArgs qa;
        memset(&qa, 0, sizeof(qa));
        if (raw) qa.extra = extra;
        fill_quantise_side(qa.side[0], batch, d1, raw, (const char*)L.maps.p1, L.maps.bstride1, L.maps.n_pad, C.args.map[0]);
        fill_quantise_side(qa.side[1], batch, d2, raw, (const char*)L.maps.p2, L.maps.bstride2, L.maps.m_pad, C.args.map[1]);
        qa.batch = batch;
        qa.raw_rows = raw ? 1 : 0;
        qa.normalize = (opts->flags & FNN_FLAG_NORMALIZE) ? 1 : 0;
        qa.seg_pixels = C.args.seg_pixels;
        qa.lower = C.args.sample_lower;
        qa.lower_count = C.sample_words;
        qa.split_d = (opts->flags & FNN_FLAG_SPLIT) ? d : 0;
        FNN_TRY(launch_quantise(qa, opts->compute, L.maps.dp, s));
        FNN_TRY(dense_two_steps(C, L, batch, n, m, opts->compute, l2, da, s));
        FNN_TRY(launch_dense_resolve(da, batch, opts->compute, L.maps.dp, nn12, s12, nn21, s21, s));
        FNN_TRY(launch_dense_final(fa, batch, s));
        return FNN_OK;
    }
    if (n > 0 && m > 0) FNN_TRY(prep_both(batch, d1, d2, L.maps, d, opts, s, extra, true));
    if (n > 0 && m > 0) FNN_TRY(launch_dense(da, batch, opts->compute, L.maps.dp, nn12, s12, nn21, s21, s));
    else if (n > 0) FNN_TRY(launch_fill_i32f32(nn12, s12, (int64_t)batch * n, s));
    else if (m > 0) FNN_TRY(launch_fill_i32f32(nn21, s21, (int64_t)batch * m, s));

    FNN_TRY(launch_dense_final(fa, batch, s));
    if (n == 0 && m == 0) {
        // no kernel ran: n_pairs still has to be defined
        FNN_TRY(launch_recip_dedup(RecipState{}, 0, batch, nullptr, nullptr, nullptr, pairs, n_pairs, s));
    }
    return FNN_OK;
}

int32_t fnn_pairs_to_pixels(int32_t batch, const int32_t* pairs, const int32_t* n_pairs, int64_t max_pairs, int64_t n,
                            int32_t width1, int64_t m, int32_t width2, const float* conf1, const float* conf2,
                            float min_conf1, float min_conf2, int32_t* out_xy, int32_t* out_count, void* stream) {
    if (batch < 1 || batch > FNN_MAX_BATCH || max_pairs < 0 || max_pairs > MAX_PIXELS || n < 0 || m < 0 ||
        n > MAX_PIXELS || m > MAX_PIXELS || width1 < 1 || width2 < 1)
        return FNN_E_SHAPE;
    if (!n_pairs || !out_count) return FNN_E_NULL;
    if (max_pairs > 0 && (!pairs || !out_xy)) return FNN_E_NULL;
    PixelArgs pa;
    memset(&pa, 0, sizeof(pa));
    pa.pairs = pairs;
    pa.n_pairs = n_pairs;
    pa.max_pairs = max_pairs;
    pa.n = n;
    pa.m = m;
    pa.width1 = width1;
    pa.width2 = width2;
    pa.conf1 = conf1;
    pa.conf2 = conf2;
    pa.min_conf1 = min_conf1;
    pa.min_conf2 = min_conf2;
    pa.out_xy = out_xy;
    pa.out_count = out_count;
    FNN_TRY(launch_pairs_to_pixels(pa, batch, (hipStream_t)stream));
    return FNN_OK;
}

}  // extern "C"
#pragma GCC visibility pop
