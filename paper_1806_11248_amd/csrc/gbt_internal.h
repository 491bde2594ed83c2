// Internal declarations shared by the translation units of libgbt.
// Not part of the ABI; include/gbt.h is.
#pragma once

#include <hip/hip_runtime.h>
#include <mutex>
#include <stdint.h>
#include <stdio.h>

#include <math.h>

#include <algorithm>
#include <vector>

#include "gbt.h"

struct ProfSpan {
    int cls;
    double bytes;       // HBM bytes this library's design moves in the launch
    double alg_bytes;   // bytes the method itself needs (see gbt_profile); < 0: the same as `bytes`
    int level;          // depth of the nodes whose histograms the launch builds, -1: not a histogram launch
    double row_features;   // rows * features accumulated into those histograms
    hipEvent_t start, stop;
};

struct gbt_ctx {
    int device;
    hipStream_t stream;
    int num_cu;
    size_t lds_per_block;   // largest dynamic LDS a workgroup may ask for
    size_t lds_max;         // the most LDS one workgroup can be given (a kernel with one workgroup per CU and no static LDS)
    char *pinned;           // host staging for job tables and small read-backs
    size_t pinned_bytes;
    int hist_block;         // threads per histogram workgroup
    int hist_block_auto;    // 1: hist_block is the default, which a launch of few workgroups may double
    int hist_runtime_bits;  // 1: unpack with run-time shifts even where a compile-time kernel exists
    int part_fused;         // 1: one-launch record partition where it applies
    int lossguide_batch;    // open leaves a round of loss-guided growth expands at once (1: only the one whose turn it is)
    int plan;               // 1: depth-wise levels are planned on the device where that applies (paths 1 and 3, sparse rows)
    int part_nomove;        // partition + histogram path, depth-wise: 1: the last histogram level is built without moving rows; 2: the last two
    int part_cycle;         // same path: above the last two levels, rows are moved every third level only (keep, keep with two histograms, move three levels)
    int part_ids;           // 1: rows wider than 64 words are not moved: id lists are partitioned and the histogram kernel gathers
    int order_rows;         // 1: a caller's row order is made from the finished tree, so that it does not restrict the partition form
    int hist_fix;           // 1: the root histogram kernel also converts the gradient pairs where that applies
    int part_hist;          // 1: and the children's histograms in the same pass where that applies
    int hist_lds_kb;        // 0, or a cap on the LDS histogram of one workgroup (more workgroups per CU)
    int hist_lds_auto;      // 1: hist_lds_kb is the default, which a shape of two to four feature tiles may double to save a tile
    int hist_jobs_per_cu;   // histogram workgroups to aim for per compute unit and launch
    int move_max_words;     // rows of more 32-bit words than this are never moved: only their ids are partitioned
    int hist_merge_ratio;   // weight of the merges into HBM in the cutting of rows into histogram jobs (96: as measured)
    int hist8;              // 1: the root histogram of 8-bit symbols with at most 16 features takes kernels_hist8.hip
    int hist8_stagger;      // its workgroups on one compute unit get unequal shares of rows: spread in 1/256ths
    int sparse_jobs_per_cu; // row pieces per compute unit and launch of the sparse-row histogram kernel
    int quantise_sort;      // 1: cuts from sorted columns also where selection applies
    int quantise_work;      // key reads one workgroup of the selection may spend on a column (0: by the column's length)
    int quantise_late;      // 1: columns go to the sort only where their selection has reached that, not by their sample
    int sparse_tiled;       // 1: keep the sparse-row LDS histogram under hist_lds_kb even where all ids would fit
    char *part_static;      // this device's copy of the static partition scratch (gbt_partition_static), or NULL
    size_t up_off;          // next free byte of the upload ring (first half of `pinned`)
    char err[512];
    bool profiling;
    std::vector<ProfSpan> *spans;       // recorded, not yet read
    std::vector<hipEvent_t> *free_events;
};

// Brackets a launch group with events when profiling is on (no-ops otherwise).
// bytes: what the design moves; alg_bytes: what the method needs (< 0: the same); level, row_features: for
// launches that build histograms (see ProfSpan).  Returns the span's index for gbt_prof_patch, -1 when off.
int gbt_prof_begin(gbt_ctx *ctx, int cls, double bytes, double alg_bytes = -1.0, int level = -1,
                   double row_features = 0.0);
void gbt_prof_end(gbt_ctx *ctx);
// Figures of a span that are only known after its launch has been waited for (rows of the built children).
void gbt_prof_patch(gbt_ctx *ctx, int span, double alg_bytes, double row_features);

#define GBT_STAGING_BYTES (8u << 20)

// ---- error plumbing -------------------------------------------------------
int32_t gbt_fail(gbt_ctx *ctx, int32_t code, const char *fmt, ...);

#define GBT_HIP(ctx, call)                                                                  \
    do {                                                                                    \
        hipError_t e_ = (call);                                                             \
        if (e_ != hipSuccess)                                                               \
            return gbt_fail((ctx), GBT_EHIP, "%s: %s (%s:%d)", #call, hipGetErrorString(e_), \
                            __FILE__, __LINE__);                                            \
    } while (0)

#define GBT_REQUIRE(ctx, cond, code, ...) \
    do {                                  \
        if (!(cond)) return gbt_fail((ctx), (code), __VA_ARGS__); \
    } while (0)

static constexpr inline size_t gbt_align(size_t x, size_t a = 256) { return (x + a - 1) / a * a; }

// ---- job descriptors (host-built, read by kernels) --------------------------
// One workgroup of the histogram kernel: rows [row_begin, row_begin+n_rows) of
// the level's row-id buffer (or of the matrix itself when there is no row-id
// buffer), features [f0, f0+ft), accumulated into the histogram at hist_off.
struct HistJob {
    uint64_t hist_off;   // offset of the node's histogram in int64 units
    uint32_t row_begin;
    uint32_t n_rows;
    uint32_t f0, ft;
    uint32_t pad0;   // 1: this is the only job of its (node, feature tile): it may store its bins instead of adding them
    uint32_t pad1;
};

// One node for the split kernel.
struct EvalNode {
    uint64_t hist_off;
    int64_t Gq, Hq;
    // sibling subtraction folded into the evaluation: when parent_off != GBT_NO_HIST the node's histogram
    // does not exist yet; the kernel makes it as parent - built (int64 units, like hist_off), stores it
    // at hist_off and evaluates it in the same pass
    uint64_t parent_off, built_off;
};
#define GBT_NO_HIST (~0ull)

// One segment for the partition kernels.
struct PartJob {
    uint32_t seg_begin, seg_len;
    uint32_t feature, bin;
    uint32_t default_left;
    uint32_t tile_begin;   // index of the segment's first tile in the level's tile arrays
    uint32_t n_tiles;
    uint32_t pad;          // partition + histogram pass: the child to build (1 left, 0 right, 2 none)
    uint64_t hist_off;     // same pass: that child's histogram in the pool (int64 units)
};

// One parent segment for the two-level row count: the rows still lie in the parent's order, its split
// (index 0) tells each row's child, and the children's splits (1: left child, 2: right child; has[] = 0
// for a child that is not split) tell the row's side there.
struct CountJob {
    uint32_t seg_begin, seg_len;
    uint32_t tile_begin, n_tiles;
    // the splits below the segment in heap order: 0 the segment's own, 1 and 2 its left / right child's,
    // 3..6 the grandchildren's (left to right); has[p]: node p splits (0 always does)
    uint32_t feature[7], bin[7], default_left[7];
    uint32_t has[7];
    uint32_t pad;
};

// One segment for the histogram pass over rows that were not moved at the segment's own split: the
// split tells each row's child (0 left, 1 right), the child's split (if it has one) the row's side there.
// Of each splitting child's two children one histogram is built (build[c]: 1 the left, 0 the right)
// into hist_off[c]; cursor word 2 * job + c counts the child's left rows.
struct Hist2Job {
    uint32_t seg_begin, seg_len;
    uint32_t tile_begin, n_tiles;   // in spans of rows_per_span rows
    uint32_t feature[3], bin[3], default_left[3];
    uint32_t has[2], build[2];
    uint32_t pad;
    uint64_t hist_off[2];
};

// One segment for the pass that puts rows in order again after two levels in place (gbt_launch_move3): the splits
// below the segment in heap order as in CountJob (0 the segment's own, 1 and 2 its children's, 3..6 the
// grandchildren's; has[p] = 0: node p does not split and its rows are dropped), and the row range of each
// grandchild in the destination, inside which its left rows are stored from the front and its right rows from the
// back.  Cursor word 4 * job + g counts grandchild g's left (low half) and right (high half) rows.
struct Move3Job {
    uint32_t seg_begin, seg_len;
    uint32_t tile_begin, n_tiles;   // in spans of rows_per_span rows
    uint32_t feature[7], bin[7], default_left[7];
    uint32_t has[7];
    uint32_t node_begin[4], node_len[4];
};
static_assert(sizeof(Move3Job) % 4 == 0 && sizeof(Move3Job) / 4 <= 64, "staged into LDS by the first wave");

// One leaf segment for the final gather.
struct LeafSeg {
    uint32_t seg_begin;
    uint32_t node;
    uint32_t buf;   // which of the two row-id buffers holds the segment
    uint32_t len;
};

struct DevTree {   // one tree's arrays inside the predict workspace (offsets in bytes)
    int32_t n_nodes;
    int32_t pad;   // the tree's depth (steps of its longest root-to-leaf walk)
    uint64_t feature, bin, default_left, left, right, threshold, weight;
};

// ---- growth planned on the device (kernels_plan.hip) -------------------------
enum { PLAN_BAD_ROWS = 1, PLAN_BAD_JOBS = 2 };
struct PlanLevel {           // one depth of the tree
    uint32_t n_nodes;        // nodes of this depth; their ids are consecutive, from first_node
    uint32_t first_node;
    uint32_t n_splits;       // of them split: jobs of the partition ...
    uint32_t n_tiles;        // ... and its tiles
    uint32_t n_hist_jobs;    // jobs that build this depth's histograms
    uint32_t bad;            // PLAN_BAD_*: a partition counted more left rows than the node has, more jobs than the launch has
    uint64_t built_rows;     // rows of the nodes whose histogram is built
};
struct PlanNode {
    uint32_t begin, len;
    int64_t Gq, Hq;
    double gain;
    int32_t feature, bin, default_left, left;   // feature -1: a leaf; the right child is left + 1
    float threshold;
    uint32_t pad;
};
struct PlanJob {             // what the children of partition job k need of its node's split
    uint32_t node, pad;
    int64_t GLq, HLq;
};
// How the rows of a level's built nodes are cut into histogram jobs: pieces of at most rows_per_job rows of a node, a job
// per piece and column tile.  Short pieces spread the rows over the chip, long ones merge fewer histograms into HBM (two
// 64-bit atomics per bin).  Both sides in rows a compute unit could have added instead:
//   adding   the busiest compute unit's share: the longest piece, or the average job times the jobs of a compute unit;
//   merging  jobs * merge (hist_rule; a node of one piece stores its bins: a quarter of that).
// With equal pieces and fewer jobs than compute units the best length is sqrt(rows * tiles * merge); the candidates are
// that length times 2^(-1) .. 2^(7/8), because what decides near it is how the number of jobs falls on the compute units
// (5M x 30 bytes, us per round with a fixed number of jobs per launch: 250 jobs 1790, 300 2012, 500 1987, 560 2184).
struct PlanHistRule {
    int64_t pieces_max, min_rows, max_rows;
    double merge;            // see above, per job; more than 0
    int num_cu;
    int tiles, ft, width;    // feature (or bin id) tiles: `tiles` tiles of ft of the `width` columns (ids)
    int exclusive_ok;        // a node of one piece stores its bins
};
constexpr int kPieceCandidates = 16;
__host__ __device__ inline int64_t gbt_clamp_rows(const PlanHistRule &r, double rows) {
    const int64_t v = rows > 1e18 ? (int64_t)1e18 : (int64_t)rows;
    return v < r.min_rows ? r.min_rows : v > r.max_rows ? r.max_rows : v;
}
// candidate c for `rows` rows in all
__host__ __device__ inline int64_t gbt_piece_candidate(const PlanHistRule &r, int64_t rows, int c) {
    // 2^((c - 8) / 8)
    constexpr double step[8] = {1.0, 1.0905077326652577, 1.189207115002721, 1.2968395546510096,
                                1.4142135623730951, 1.5422108254079407, 1.681792830507429, 1.8340080864093424};
    double v = sqrt((double)rows * r.tiles * r.merge) * step[c & 7] * (c < 8 ? 0.5 : 1.0);
    const double least = (double)((rows + r.pieces_max - 1) / r.pieces_max);
    return gbt_clamp_rows(r, v < least ? least : v);
}
// what cutting at `length` rows costs: pieces in all, those of nodes of one piece, the longest node
__host__ __device__ inline double gbt_piece_cost(const PlanHistRule &r, int64_t rows, int64_t length, int64_t pieces, int64_t single,
                                                 int64_t longest) {
    const double jobs = (double)pieces * r.tiles, most = (double)(longest < length ? longest : length);
    const double per_cu = (double)(((int64_t)pieces * r.tiles + r.num_cu - 1) / r.num_cu);
    const double share = jobs > 0.0 ? per_cu * (double)rows * r.tiles / jobs : 0.0;
    const double merged = (double)(pieces - single) + 0.25 * (double)single;
    return (share > most ? share : most) + merged * r.tiles * r.merge;
}
// The most jobs `splits` built children of a matrix of n rows can be cut into: the size of the launch that takes them, which
// plan_children_kernel holds its own count against.
inline int64_t gbt_plan_jobs_max(const PlanHistRule &r, int64_t n, int64_t splits) {
    const int64_t built = n / 2 + 1;
    // By the shortest candidate length: b / (length(b) - 1) grows with the b rows built (length is the square root, rounded
    // down, and at least min_rows), so that of the most rows bounds them all; without the 1, fewer rows whose length rounds
    // down by more can make a few pieces more.
    const int64_t shortest = std::max<int64_t>({1, r.min_rows, gbt_piece_candidate(r, built, 0) - 1});
    int64_t pieces = std::min(r.pieces_max, built / shortest + 2);
    pieces = std::max(pieces, (built + r.max_rows - 1) / r.max_rows);
    return (pieces + splits) * r.tiles;
}
// Where the job of column tile `tile` of row piece `piece` stands among a launch's pieces * tiles jobs.  Workgroups are
// dealt to the eight dies in turn, and each die has an L2 of its own: the tiles of a piece, which read the same rows, pairs
// and ids, stand eight apart and meet in one L2.
__host__ __device__ inline uint32_t gbt_job_place(uint32_t piece, uint32_t tile, uint32_t pieces, uint32_t tiles) {
    const uint32_t group = piece & ~7u, wide = pieces - group < 8u ? pieces - group : 8u;
    return group * tiles + tile * wide + (piece - group);
}
struct PlanView {            // device addresses unless noted
    PlanLevel *levels;
    PlanNode *nodes;
    const gbt_split *recs;   // the evaluation's records, node-major
    uint32_t *win;           // scratch: the winning chunk of every node of a level
    PartJob *pjobs;
    PlanJob *pinfo;
    EvalNode *enodes;
    HistJob *hjobs;
    unsigned long long *cursors;
    int cursors_per_job;
    int64_t *pool;
    int64_t hist_len;
    const float *cuts;
    int F, B;
    double inv_sg, inv_sh, lambda, min_gain;
    char *tree;              // the tree as the walks read it: a DevTree, then its arrays at `arrays`' offsets
    DevTree arrays;
    uint32_t *hint;          // host memory: splits of each level, written when they are known
};
// sums: n_sums partial totals of the pairs (int64[2] each)
hipError_t gbt_launch_plan_root(hipStream_t s, const PlanView &v, const int64_t *sums, int n_sums, int64_t n, int n_levels);
hipError_t gbt_launch_plan_split(hipStream_t s, const PlanView &v, int depth, int chunks, uint32_t tile_rows);
// n_left: left rows of split k at n_left[k * stride] (NULL: not counted yet, the children's row counts come later).
// jobs_max: what the job table and the launch behind it hold; a level that needs more gets no jobs and PLAN_BAD_JOBS
hipError_t gbt_launch_plan_children(hipStream_t s, const PlanView &v, int depth, int64_t max_splits, const uint32_t *n_left,
                                    int stride, bool with_hist, const PlanHistRule &rule, uint32_t jobs_max);
hipError_t gbt_launch_plan_rank(hipStream_t s, const PlanView &v, int n_levels, uint32_t *count, uint32_t *rank);
hipError_t gbt_launch_plan_finish(hipStream_t s, const PlanView &v, int n_levels, int last, const uint32_t *counted,
                                  PlanLevel *levels_out, PlanNode *nodes_out, uint32_t cap);

#define GBT_PART_TILE 2048   // rows per partition workgroup
#define GBT_PART_BLOCK 256

// ---- kernel launchers (each returns the hipGetLastError of its launches) ---
// DEVICE COUNTS.  Where a launcher takes n_jobs_dev / n_nodes_dev / counts_dev, the number of jobs (nodes) is not known to
// the host: the host's number is the most there can be, workgroups past the device's one leave at once.  counts_dev holds
// two words, the jobs and their tiles; the partition's cursors are then cleared by the caller.
hipError_t gbt_launch_fill_u64(hipStream_t s, uint64_t *p, uint64_t v, int64_t count);
hipError_t gbt_launch_iota_u32(hipStream_t s, uint32_t *p, int64_t count);
hipError_t gbt_launch_stream_read(hipStream_t s, const void *buf, int64_t bytes, uint32_t *sink);
// Reductions over rows store one partial result of 16 bytes per workgroup into `slots` (device memory, or host memory that
// the device can address: room for gbt_red_slots_max() of them); *n_slots receives their number.
//   bounds  uint32[4]: bits of the largest |g|, of the largest |h|, 1 if some h < 0, bits of the smallest |h|
//   sums    int64[2]
int gbt_red_slots_max();
hipError_t gbt_launch_absmax(hipStream_t s, const float *gpair, int64_t n, void *slots, int *n_slots);
// slots (may be NULL): the sums of gq
hipError_t gbt_launch_to_fixed(hipStream_t s, const float *gpair, int64_t n, double sg, double sh,
                               int32_t *gq, void *slots, int *n_slots);
hipError_t gbt_launch_sum_gq(hipStream_t s, const int32_t *gq, const uint32_t *row_idx, int64_t n_rows, void *slots, int *n_slots);
// bounds (may be NULL): slots for the bounds of these pairs
hipError_t gbt_launch_gradients(hipStream_t s, int objective, const float *margin, const float *label,
                                int64_t n, float *gpair, void *bounds = nullptr, int *n_slots = nullptr);
hipError_t gbt_launch_subtract_one(hipStream_t s, const int64_t *parent, const int64_t *child,
                                   int64_t *out, int64_t count);
hipError_t gbt_launch_export(hipStream_t s, const int64_t *hist, int64_t count, double inv_sg,
                             double inv_sh, double *out);

// packed: a bit stream whose row r starts at bit r*stride_bits (the canonical packed matrix has
// stride_bits = F*bits; the word-aligned working copy of the grow loop 32*ceil(F*bits/32));
// n_words: readable 32-bit words of `packed`; row_idx NULL: job rows are matrix rows.
hipError_t gbt_launch_hist(gbt_ctx *ctx, const uint32_t *packed, int bits, int64_t stride_bits, int64_t n_words,
                           int64_t n, int B, uint32_t missing, const uint32_t *row_idx, const int32_t *gq,
                           int64_t *hist_pool, const HistJob *jobs, int n_jobs, int max_ft,
                           // every row's rounded h equals hq_uniform: kernels that have a form for it (symbol widths
                           // other than 8 bits) count rows instead of summing h; jobs then hold at most
                           // gbt_histw_max_rows(true) rows
                           bool uniform_h = false, int32_t hq_uniform = 0, int block = 0,   // threads (0: ctx->hist_block)
                           const uint32_t *n_jobs_dev = nullptr);   // see DEVICE COUNTS
// Most whole symbols of `bits` bits in 16 bytes that start at the first one's byte: a register window of kernels_histw.hip.
#define GBT_HISTW_WINDOWS 4   // of a row that a tile may have
constexpr int gbt_histw_window(int bits) {
    const int first = bits % 8 == 0 ? 0 : bits % 4 == 0 ? 4 : bits % 2 == 0 ? 6 : 7;   // the first one's bit, at most
    const int e = (128 - first) / bits;
    return e < 32 ? e : 32;
}
// What a tile of ft of the F columns costs a row, in slots (an element's field, address and atomic).
//   bytes        every slot of a window of sixteen, used or not (hist_b8_kernel)
//   other widths a lane takes a window's share of a row, which costs it about ten slots beside its columns; where all windows are
//                full nothing asks whether a column is there, a third less.  (Of four full windows the lanes meet more often in
//                a bank, those of 31 or 32 columns the most.)  Not less than the line of 128 bytes that a tile reads of a longer
//                row, dearer the further the rows are apart; and where rows are gathered (gathered: the bytes of their matrix) from
//                past the last cache, that line comes from HBM for every tile.
// us of a root, general pairs: 1M x 100 x 6 bits in two tiles of 50 118, four of 25 88, five of 20 (full) 53; 1M x 52 x 9 bits, three of
// 18 84, four of 13 (full) 53; 500,000 x 1000 x 6 bits, 13 of 77 310, 25 of 40 (full) 242, 50 of 20 (full, a line each) 342.  A round
// that gathers, equal hessians: 10M x 50 x 9 bits (560 MB), four tiles of 13 3514, two of 25 3096; a third of its rows 1166 and (20) 1208.
constexpr double kLastCacheBytes = 256e6;
inline double gbt_tile_cost(int ft, int F, int bits, double gathered) {
    const int E = gbt_histw_window(bits), windows = ft <= E ? 1 : ft <= 2 * E ? 2 : GBT_HISTW_WINDOWS;
    if (bits == 8) return (ft + E - 1) / E * E;
    const double full = windows == 1 ? 0.67 : windows == 2 ? 0.69 : E > 24 ? 0.85 : 0.74, row_bytes = (double)F * bits / 8.0;
    const double slots = ft == windows * E ? windows * (10 + E) * full : windows * (10 + (ft + windows - 1) / windows);
    const double line = 35.0 * std::min(1.0, row_bytes / 256.0) + 10.0 * std::min(1.0, row_bytes / 1500.0);
    return (slots > line ? slots : line) + (gathered > kLastCacheBytes ? 30.0 : 0.0);
}
// Columns of a tile, ft_max at most (the last tile has what is left, and is waited for as long as for the others): of the even splits,
// and of tiles of one, two or four full windows, those that cost a row least.  us of a root, 666,666 x 150 x 3 bits: tiles of 128 and 22
// columns 103, of 64 56, of 32 64.  Over 104 shapes of 1 to 10 bits, 40 to 2000 columns, what is taken is 1.03 times as slow as
// the best of some fifteen tiles on average, 1.13 at most.
// Bytes: more tiles than needed cost a pass over the pairs each, and are taken where they save a fifth of the slots (with full
// windows only, 1M x 50 77 instead of 69 us).
inline int gbt_tile_columns(int F, int bits, int ft_max, double gathered) {
    int best = 0;
    double best_cost = 0.0;
    auto consider = [&](int ft) {
        if (ft > ft_max) return;
        const int tiles = (F + ft - 1) / ft;
        const double whole = gbt_tile_cost(ft, F, bits, gathered), last = gbt_tile_cost(F - (tiles - 1) * ft, F, bits, gathered);
        const double cost = (tiles - 1) * whole + (last > whole ? last : whole);
        if (best && (bits == 8 ? cost * 5.0 > best_cost * 4.0 : cost >= best_cost)) return;
        best = ft;
        best_cost = cost;
    };
    const int nt_min = (F + ft_max - 1) / ft_max, E = gbt_histw_window(bits);
    for (int nt = nt_min; nt <= nt_min + 8 && nt <= F; ++nt) consider((F + nt - 1) / nt);
    for (int windows = 1; bits != 8 && windows <= GBT_HISTW_WINDOWS; windows *= 2) consider(windows * E);
    return best;
}
int gbt_histw_max_rows(bool uniform_h);
hipError_t gbt_launch_histw(gbt_ctx *ctx, const uint32_t *packed, int bits, int64_t stride_bits, int64_t n_words,
                            int64_t n, int B, uint32_t missing, const uint32_t *row_idx, const int32_t *gq,
                            int64_t *hist_pool, const HistJob *jobs, int n_jobs, int max_ft, bool uniform_h,
                            int32_t hq_uniform, int block, const uint32_t *n_jobs_dev = nullptr);
// Largest feature tile whose LDS histogram fits, and the per-job row count to aim for.
int gbt_hist_feature_tile(const gbt_ctx *ctx, int F, int B, int64_t n_rows = 0);   // n_rows: rows of the matrix the tiles are for (0: unknown)

// out receives n_nodes * n_chunks records (node-major); gbt_eval_chunks picks n_chunks.
int gbt_eval_chunks(int F, int n_nodes, size_t record_budget_bytes);
constexpr int kEvalGroups = 8192;   // workgroups an evaluation of many nodes is cut into, about
// the most records of any F features and at most n_nodes nodes (fewer than one more chunk per node than fill kEvalGroups)
inline int64_t gbt_eval_records_max(int64_t n_nodes) { return kEvalGroups + n_nodes; }
// `out` may be host memory the device can address (the pinned staging): the records are then where the
// host reads them when the launch has finished, without a copy.  tail: n 64-bit words copied from src to
// dst (again possibly such host memory) by the same launch, and src cleared behind the copy if `clear`
// (the row cursors of the partition that ran before, returned and made ready for the next one).
// clear_slot >= 0: the launch also zeroes the histograms that the evaluated nodes' children would
// accumulate into if their parents split: pool slots clear_slot + 2 i and clear_slot + 2 i + 1 for node
// i, as far as they lie below clear_slot_end (a slot is F * B * 2 values).
struct EvalTail {
    unsigned long long *src, *dst;
    int n, clear;
    int64_t clear_slot, clear_slot_end;
    int src_stride = 1;   // word i is src[i * src_stride]
    int skip_store = 0;   // 1: a histogram made by subtraction is evaluated but not stored (nothing below these nodes
                          // will subtract from it: their children are leaves)
};
// The cursors of the passes that partition in one launch lie one per 128-byte line (index * kCursorStride): atomics on
// words of one line take turns as if they were one address, 12 ns each.  (10M sparse rows, 9766 tiles with two cursors of
// a node side by side: 240 us per level of atomics alone, whatever the tiles did meanwhile.)
constexpr int kCursorStride = 16;
hipError_t gbt_launch_eval(hipStream_t s, int64_t *hist_pool, const EvalNode *nodes, int n_nodes,
                           const int32_t *nb, int F, int B, int n_chunks, double inv_sg, double inv_sh,
                           double lambda, double mcw, gbt_split *out, EvalTail tail = EvalTail{nullptr, nullptr, 0, 0, -1, 0},
                           const uint32_t *n_nodes_dev = nullptr);

// Row ids in one launch, order not kept: tiles of tile_rows = gbt_partition_ids_tile() rows, a cursor of 64 bits per job (the caller
// clears them), [ right rows : left rows ].  src NULL: a segment's ids are its places.
int gbt_partition_ids_tile(const gbt_ctx *ctx, int64_t n);
hipError_t gbt_launch_partition_ids(hipStream_t s, const uint32_t *packed, int bits, int64_t stride_bits, int64_t n, uint32_t missing,
                                    const uint32_t *src, uint32_t *dst, int tile_rows, const PartJob *jobs, int n_jobs, int total_tiles,
                                    unsigned long long *cursor, int cursor_stride, const uint32_t *counts_dev);
hipError_t gbt_launch_partition(hipStream_t s, const uint32_t *packed, int bits, int64_t stride_bits, int64_t n,
                                uint32_t missing, const uint32_t *src, uint32_t *dst,
                                const PartJob *jobs, int n_jobs, int total_tiles, uint64_t *masks,
                                uint32_t *tile_left, uint32_t *n_left_out, const uint32_t *counts_dev = nullptr,
                                // one job only: dst == src, the ids are copied to `ids` by the first pass and come back
                                // from there; n_left_host also receives n_left
                                uint32_t *ids = nullptr, uint32_t *n_left_host = nullptr);

// A set of rows in some order: symbols (row p starts at bit p*stride_bits), fixed-point gradient
// pairs and original row ids (NULL: the id of position p is p).  The *_rw members are the same
// addresses for a set that may be written.
struct GbtRows {
    const uint32_t *sym;
    int64_t stride_bits, n_words;
    const int32_t *gq;
    const uint32_t *id;
    uint32_t *sym_rw;
    int32_t *gq_rw;
    uint32_t *id_rw;
};
// Stable partition of the jobs' segments of `src` into `dst` (records move, see kernels_partition.hip).
// ids_only: move the row ids alone (the segments' children will not be read again).
hipError_t gbt_launch_partition_records(hipStream_t s, const GbtRows &src, const GbtRows &dst, int bits, int row_bits,
                                        int64_t n, uint32_t missing, int what, const PartJob *jobs,
                                        int n_jobs, int total_tiles, uint64_t *masks, uint32_t *tile_left,
                                        uint32_t *n_left_out, const uint32_t *counts_dev = nullptr);
// `what` above: move whole records, move only the ids, or only count the left rows of every job
enum { GBT_PART_RECORDS = 0, GBT_PART_IDS = 1, GBT_PART_COUNT = 2 };
// The same move of whole records in one launch for a caller that does not need the row order
// (and no ids): rows narrow enough (gbt_partition_fused_ok), tiles of gbt_partition_fused_tile(dst, n)
// rows (PartJob.tile_begin / n_tiles count those).  cursor: one word per job, cleared by the
// launcher; after the launch its low half is the job's n_left.  Inside a child the rows of one
// tile keep their order, the tiles' order is arbitrary.
bool gbt_partition_fused_ok(const GbtRows &dst);
int gbt_partition_fused_tile(const GbtRows &dst, int64_t n);   // n: rows of the matrix
hipError_t gbt_launch_partition_fused(hipStream_t s, const GbtRows &src, const GbtRows &dst, int bits, int row_bits,
                                      int64_t n, uint32_t missing, const PartJob *jobs, int n_jobs, int total_tiles,
                                      unsigned long long *cursor, int cursor_stride, const uint32_t *counts_dev = nullptr);
// The root histogram straight from the fp32 gradient pairs (8-bit symbols, one feature tile of at
// most 16 features, jobs that cover rows [0, n) exactly once: gbt_hist_fix_ok): rounds each pair to
// fixed point with the given scales, stores it to gq_out and adds the totals into sums_out[2].
bool gbt_hist_fix_ok(int bits, int64_t stride_bits, int max_ft, int n_ftiles);
hipError_t gbt_launch_hist_fix(gbt_ctx *ctx, const uint32_t *packed, int64_t stride_bits, int64_t n_words, int64_t n,
                               int B, uint32_t missing, const float *gpair, double sg, double sh, int32_t *gq_out,
                               int64_t *sums_out, int64_t *hist_pool, const HistJob *jobs, int n_jobs, int max_ft);
// The histogram of ALL n rows of a packed matrix with 8-bit symbols and F <= 16 features (kernels_hist8.hip).
// The pairs come as fixed-point gq (gpair == NULL), or as fp32 gpair, which the kernel rounds itself:
// mode 1 through fp64, mode 2 in fp32 (only where gbt_fix32_ok(sg, sh)); gq_out (may be NULL) receives the
// rounded pairs; sums (may be NULL) int64[gbt_hist8_max_jobs()][2] receives one pair of partial totals per
// workgroup ([0, *n_jobs_out) are written; their sum is the total of all rows).  uniform_h: every
// row's rounded h equals hq_uniform (the caller has checked that all fp32 h are equal).  hist_out must be zero.
// A launch that asks for more dynamic LDS than the default limit of a launch first raises the kernel's limit.
// That limit is one value per kernel for the whole process, so the raise and the launch it serves happen under
// one process-wide lock: a concurrent launch of the same kernel from another context cannot lower it in between.
// Declare the guard before the attribute call and keep it alive until the kernel has been launched.
std::recursive_mutex &gbt_lds_mutex();
struct GbtLdsGuard {
    bool needed;
    std::unique_lock<std::recursive_mutex> lock;
    explicit GbtLdsGuard(size_t lds) : needed(lds > 64u * 1024u) {
        if (needed) lock = std::unique_lock<std::recursive_mutex>(gbt_lds_mutex());
    }
};

struct Hist8Pairs {
    const float *gpair;
    const int32_t *gq;
    int32_t *gq_out;
    double sg, sh;
    int mode;
    int uniform_h;
    int32_t hq_uniform;
    int64_t *sums;
};
bool gbt_hist8_ok(int bits, int F, int n_ftiles, int64_t n, int64_t n_words);
bool gbt_fix32_ok(double sg, double sh);
int gbt_hist8_max_jobs();
// filter (may be NULL): only the rows on one side of a split are added -- the histogram of one child of the root
// with the rows staying in the matrix; hist_out must have been cleared; *lefts (device, cleared by the caller)
// receives the number of rows that go left.  Pairs as fixed point (p.gq) or fp32 with mode 2.
struct Hist8Filter {
    int feature, bin, default_left;
    int take_left;               // 1: the left rows are added, 0: the right rows
    unsigned long long *lefts;
};
hipError_t gbt_launch_hist8(gbt_ctx *ctx, const uint32_t *packed, int64_t n, int F, int B, uint32_t missing,
                            const Hist8Pairs &p, int64_t *hist_out, int *n_jobs_out = nullptr,
                            const Hist8Filter *filter = nullptr);
hipError_t gbt_launch_hist8_records(gbt_ctx *ctx, const uint32_t *records, int F, int B, uint32_t missing,
                                    const PartJob *jobs, int n_jobs, int n_spans, uint32_t rows_per_span, int64_t *pool,
                                    int32_t hq_uniform);
// Partition and the histogram of one child of every job in one pass (8-bit symbols, at most 16
// features, the bins of all features in one LDS tile: gbt_part_hist_ok).  No ids, order inside a
// child not kept.  Rows travel as records of gbt_part_hist_record_words(F) words (symbols, padding,
// the fixed-point pair in the last 7 bytes); src_records == NULL: the source is the packed matrix
// (rows of F bytes) with the pairs in gq.  PartJob.tile_begin / n_tiles count spans of rows_per_span
// rows (a multiple of gbt_part_hist_tile()); PartJob.pad / hist_off name the child to build, whose
// histogram must have been cleared.
// dst_records == NULL: nothing is moved (the children's rows stay interleaved in the parent's segment);
// the histogram is built and the low word of each cursor counts the left rows.
// The cursors (one 64-bit word per job) are cleared here unless the caller says they are zero already.
bool gbt_part_hist_ok(const gbt_ctx *ctx, int bits, int F, int B);
// Rows of 8-bit symbols, row p at byte p * stride_bytes of `rows`.  levels = 1: counts[2 * j + c] = rows
// of job j's child c that go left at that child's split; levels = 2: counts[4 * j + t] the same for
// grandchild t (heap position 3 + t).  Rows that reach a node without a split on their way are not
// counted.  counts is cleared here.
int gbt_count2_tile();
hipError_t gbt_launch_count2(hipStream_t s, const uint8_t *rows, int64_t stride_bytes, uint32_t missing,
                             const CountJob *jobs, int n_jobs, int n_tiles, uint32_t *counts, int levels = 1,
                             bool records_ok = false);   // records_ok: rows are records of the partition + histogram pass
// The histogram pass over record segments that stay in place for a second level (Hist2Job); 8-bit symbols,
// at most 16 features, two LDS histograms per workgroup (gbt_hist2_ok).  cursor: 2 words per job, cleared
// here unless the caller says they are zero; the built children's histograms must have been cleared.
bool gbt_hist2_ok(const gbt_ctx *ctx, int F, int B);
hipError_t gbt_launch_hist2(gbt_ctx *ctx, const uint32_t *records, int F, int B, uint32_t missing,
                            const Hist2Job *jobs, int n_jobs, int n_spans, uint32_t rows_per_span,
                            unsigned long long *cursor, int64_t *hist_pool, bool cursors_are_zero = false,
                            int hq_uniform = -1);   // >= 0: every row has this hessian (fixed point): bins count rows
// The pass that moves the records of segments whose rows stayed in place for two levels to their grandchildren's
// children (Move3Job); records of at most 16 byte symbols.  dst_rows: rows the destination holds (a store past it
// is skipped).  cursor: 4 words per job, cleared here unless the caller says they are zero.
int gbt_move3_tile();
hipError_t gbt_launch_move3(gbt_ctx *ctx, const uint32_t *src_records, uint32_t *dst_records, int64_t dst_rows, int F,
                            uint32_t missing, const Move3Job *jobs, int n_jobs, int n_spans, uint32_t rows_per_span,
                            unsigned long long *cursor, bool cursors_are_zero = false);
// The same over two levels of splits (the segment's own and its children's: Move3Job entries 0..2, targets 0 and 1)
// with the rows taken from the caller's packed matrix and pair array (gq, or fp32 pairs rounded with sg, sh as in
// gbt_launch_part_hist) and written as records: for a segment whose rows stayed in the matrix at its split.
hipError_t gbt_launch_move2_first(gbt_ctx *ctx, const uint32_t *packed, int64_t packed_words, const int32_t *gq,
                                  const float *gpair_fp32, double sg, double sh, uint32_t *dst_records, int64_t dst_rows, int F,
                                  uint32_t missing, const Move3Job *jobs, int n_jobs, int n_spans, uint32_t rows_per_span,
                                  unsigned long long *cursor, bool cursors_are_zero = false);
int gbt_part_hist_tile();
int gbt_part_hist_record_words(int F);
hipError_t gbt_launch_part_hist(gbt_ctx *ctx, const uint32_t *packed, int64_t packed_words, const int32_t *gq,
                                const uint32_t *src_records, uint32_t *dst_records, int F, int B, uint32_t missing,
                                const PartJob *jobs, int n_jobs, int n_spans, uint32_t rows_per_span,
                                unsigned long long *cursor, int64_t *hist_pool, bool cursors_are_zero = false,
                                // first level only: the pairs are these fp32 pairs (not gq), rounded in the pass with
                                // the scales sg, sh, for which gbt_fix32_ok must hold
                                const float *gpair_fp32 = nullptr, double sg = 1.0, double sh = 1.0,
                                // >= 0: every row has this hessian (fixed point): bins count rows instead of adding hessians
                                int hq_uniform = -1);
// LeafSeg.buf: 0/1 = id buffers buf0/buf1, 2 = the id of position p is p.
hipError_t gbt_launch_leaf_gather(hipStream_t s, const uint32_t *buf0, const uint32_t *buf1,
                                  const LeafSeg *segs, int n_segs, int64_t n, uint32_t *row_idx_out,
                                  int32_t *leaf_of_row);

// Row ids in leaf order from each row's leaf: a stable sort of the positions 0..n-1 by
// rank_tbl[leaf[row]] (n_nodes table entries, ranks below n_ranks).  key_tmp / val_tmp: two buffers of
// n words each, touched only when n_ranks > 256; ws: gbt_order_ws(n) bytes.
size_t gbt_order_ws(int64_t n);
hipError_t gbt_launch_order_rows(hipStream_t s, const int32_t *leaf, const uint32_t *rank_tbl, uint32_t n_nodes,
                                 uint32_t n_ranks, int64_t n, uint32_t *key_tmp[2], uint32_t *val_tmp[2], char *ws,
                                 uint32_t *row_idx_out);

// sparse rows (kernels_sparse.hip): rowptr + global bin ids of ent_bytes = 2 or 4 bytes each, see there
int64_t gbt_sparse_scan_tiles(int64_t n);
hipError_t gbt_launch_sparse_rowptr(hipStream_t s, const uint16_t *sym, int64_t n, int F, uint32_t missing,
                                    uint32_t *rowptr, uint64_t *tile_ws, uint64_t *total_dev);
hipError_t gbt_launch_sparse_fill(hipStream_t s, const uint16_t *sym, int64_t n, int F, int B, uint32_t missing,
                                  const uint32_t *rowptr, void *ent, int ent_bytes, int64_t nnz, int64_t capacity);
int gbt_sparse_hist_tile(const gbt_ctx *ctx, int64_t bins);
// HistJob.f0 / ft: the job's range of global bin ids
hipError_t gbt_launch_sparse_hist(gbt_ctx *ctx, const uint32_t *rowptr, const void *ent, int ent_bytes, const int32_t *gq,
                                  int64_t *pool, const HistJob *jobs, int n_jobs, int max_glen, bool tiled,
                                  // >= 0 (16-bit entries only): every row has this hessian; jobs of at most
                                  // gbt_sparse_hist_max_rows() rows, and HistJob.pad0 as for the dense kernels
                                  int hq_uniform, const uint32_t *n_jobs_dev = nullptr);
int gbt_sparse_hist_max_rows();

// Unordered partition of sparse rows, one launch per level (PartJob as for the dense forms; tiles of
// tile_rows = gbt_sparse_part_tile() rows).  cursor: two 64-bit words per job, cleared here; afterwards the low
// word of cursor[2 * j] is job j's number of left rows.  move == false: only that count.
// Rows of a tile, 128 to 1024: as many as leave the average tile's entries an eighth of room in the staging window, for a tile that
// does not fit reads and copies its rows in place (rows that do not fit 128 at a time are read in place anyway); and 512 or 256 on
// few rows, where they are short of tiles.  Not fewer: a node's tiles take turns on its cursors, 12 ns for an atomic.
// us per tree with tiles of 1024 rows and as few as fit: 5M x 50 with 17.5 entries a row, depth 6 2684 and 1267; 1M x 200 with 40,
// depth 7 1801 and 1188, with 80, depth 6 2859 and 1757; 2M x 40 with 14, depth 8 1551 and 799; 400,000 x 300 with 15 (32-bit ids),
// depth 6 902 and 646.  With 128, 256, 512 and 1024 rows, depth 6, two entries a row: 5,000 rows 211, 209, 211, 220; 25,000 225, 220,
// 218, 228; 50,000 239, 228, 221, 228; 100,000 281, 244, 229, 234; 200,000 335, 284, 248, 243; ten entries: 100,000 277, 246, 240, 249;
// 200,000 332, 288, 261, 264.
int gbt_sparse_part_tile(const gbt_ctx *ctx, int64_t n, int64_t nnz, int ent_bytes);
hipError_t gbt_launch_sparse_partition(hipStream_t s, const uint32_t *src_rowptr, const void *src_ent, int ent_bytes,
                                       const int32_t *src_gq, uint32_t *dst_rowptr, void *dst_ent,
                                       int32_t *dst_gq, int B, bool move, int tile_rows, const PartJob *jobs, int n_jobs,
                                       int n_tiles, unsigned long long *cursor, int cursor_stride,
                                       const uint32_t *counts_dev = nullptr);
// nnz: entries of all rows (-1: only the row pointers say); depth: of the trees, on average
hipError_t gbt_launch_sparse_walk(hipStream_t s, const char *ws, const DevTree *trees, int n_trees,
                                  const uint32_t *rowptr, const void *ent, int ent_bytes, int64_t n, int64_t nnz, int F, int B, double eta,
                                  float *margin, int32_t *leaf_out, int max_nodes, bool compact_ok, double depth);

hipError_t gbt_launch_compress(hipStream_t s, const uint16_t *sym, int64_t n_elems, int bits,
                               uint32_t *packed, int64_t n_words);

hipError_t gbt_launch_predict(hipStream_t s, const char *ws, const DevTree *trees, int n_trees,
                              const uint32_t *packed, int bits, uint32_t missing, const float *X,
                              int64_t n, int F, double eta, float *margin, int32_t *leaf_out, int max_nodes,
                              bool compact_ok, uint32_t *node_rows = nullptr,
                              const float *margin_src = nullptr);   // leaf_out != NULL: store each row's leaf id instead of updating margin
// node_rows, margin_src (one tree, and only where gbt_predict_counts_ok): count the rows that end in every node into
// node_rows[node * kNodeRowsStride] (zeroed by the caller); margin[r] = margin_src[r] + eta * weight
constexpr int kNodeRowsStride = 32;   // words between two nodes' row counters (gbt_launch_predict's node_rows)
bool gbt_predict_counts_ok(bool packed, int bits, int F, int64_t n, int max_nodes, bool compact_ok);
// compact_ok: every split node has right == left + 1, feature < 2^20 and bin < 4096

// Many trees on raw floats in one pass over the rows (kernels_misc.hip).  A node is 8 bytes: values are compared as
// integers in the floats' order (NaN the largest), "right" iff value + a >= thr with a = the node's default_left, and
// meta = a | the left child's byte offset from the group's first node (bits 4..17: a left child stands at an even place,
// so that the right one is 8 | that) | feature << 18; a leaf leads to itself (thr = the largest integer, a = 1, bit 3 as
// its own place has it).  wts: eta * weight of every node.  tree_off[t] = first node of
// tree t in nodes / wts, an odd place of its group (tree_off[n_trees] = all places + 1); group_end[g] = one past the last tree of group g; no group has
// more than cap_nodes nodes; gbt_predict_batch_tile_bytes(F) + 8 * cap_nodes bytes of LDS per workgroup.
struct gbt_batch_node {
    int32_t thr;
    uint32_t meta;
};
constexpr int kBatchNodesMax = 1 << 15, kBatchColsMax = 1 << 14;   // what the fields of meta hold
int gbt_predict_batch_rows(int F);
size_t gbt_predict_batch_tile_bytes(int F);
hipError_t gbt_launch_predict_raw_batched(hipStream_t s, const gbt_batch_node *nodes, const double *wts,
                                          const int32_t *tree_off, const int32_t *tree_depth,
                                          const int32_t *group_end, int n_groups, int cap_nodes, const float *X,
                                          int64_t n, int F, float *margin);

// Four consecutive words with ONE load instruction at 4-byte alignment (rows of packed symbols start at any byte).
typedef uint32_t gbt_u32x4 __attribute__((ext_vector_type(4), aligned(4)));
template <int N>
__device__ __forceinline__ void load_words(uint32_t (&x)[N], const uint32_t *p) {
    static_assert(N >= 1 && N <= 5, "a 16-byte window and the word behind it");
    if (N >= 4) {
        const gbt_u32x4 v = *(const gbt_u32x4 *)p;
        x[0] = v.x;
        x[1] = v.y;
        x[2] = v.z;
        x[3] = v.w;
        if (N == 5) x[N - 1] = p[4];
    } else {
#pragma unroll
        for (int k = 0; k < N; ++k) x[k] = p[k];
    }
}
// The job whose tile range contains `tile` (jobs are sorted by tile_begin, the first begins at or before it).  A wave looks
// at 64 of them at once, so that up to 64 jobs cost one load and up to 4096 two; a bisection of 128 jobs is seven loads one
// behind the other, two or three microseconds in front of everything a workgroup does.  Every lane of the wave must call.
template <typename Job>
__device__ __forceinline__ int gbt_find_job(const Job *jobs, int n_jobs, uint32_t tile) {
    const int lane = (int)(threadIdx.x & 63u);
    int lo = 0, n = n_jobs;   // the job is one of [lo, lo + n)
    while (n > 1) {
        const int step = (n + 63) >> 6, at = lane * step;
        const bool before = at < n && jobs[lo + at].tile_begin <= tile;
        const int k = __popcll(__ballot(before)) - 1;   // the last of the 64 that begins at or before the tile
        lo += (k < 0 ? 0 : k) * step;
        n = n - (k < 0 ? 0 : k) * step < step ? n - (k < 0 ? 0 : k) * step : step;
    }
    return __builtin_amdgcn_readfirstlane(lo);
}
constexpr int kHShift = 30;                        // width of the h field
constexpr uint32_t kHMask = (1u << kHShift) - 1u;


// order statistics by selection (kernels_select.hip): keys, segments and tiles as kernels_quantise.hip lays them out,
// `collected` a second buffer of n_values words; cuts, nb and present (values that are not missing) per feature, but for
// those whose mode is kSelSorted (some is iff *A.flag is not zero): theirs are still to be found
struct SelArrays;
bool gbt_select_ok(int F, int64_t n_values, int B);
size_t gbt_select_layout(int F, int64_t n_values, int B, char *base, SelArrays *A);   // bytes; base, A may be NULL
hipError_t gbt_launch_select(gbt_ctx *ctx, const uint32_t *keys, uint32_t *collected, const uint64_t *seg_off,
                             const uint32_t *blk_off, int F, int64_t n_values, int B, const SelArrays &A, float *cuts,
                             int32_t *nb, uint32_t *present);
// ... and, for a dense matrix, the bit stream from the key columns: gbt_launch_bin_table once the cuts are there, then
// gbt_launch_bin_columns (cols: gbt_bin_columns_bytes scratch bytes)
size_t gbt_bin_columns_bytes(int64_t n, int F);
bool gbt_bin_columns_ok(int64_t n, int F, int bits);
hipError_t gbt_launch_bin_table(gbt_ctx *ctx, int F, int B, const SelArrays &A, const float *cuts, const int32_t *nb);
hipError_t gbt_launch_bin_columns(gbt_ctx *ctx, const uint32_t *keys, void *cols, const uint64_t *seg_off, const uint32_t *blk_off,
                                  int64_t n, int F, int B, const SelArrays &A, const float *cuts, const int32_t *nb,
                                  uint32_t missing, int bits, uint32_t *packed, int64_t n_words);
// quantise
hipError_t gbt_quantise_run(gbt_ctx *ctx, const float *X, const int64_t *indptr, const int32_t *indices,
                            const float *values, int64_t n, int F, int64_t n_values, int B, float *cuts,
                            int32_t *nb, uint16_t *sym, int32_t *max_value, int32_t *missing_sym,
                            char *ws, size_t ws_bytes, int32_t *status, uint32_t *packed = nullptr,
                            int64_t packed_cap_words = 0, int32_t *bits_out = nullptr);
size_t gbt_quantise_ws(int64_t n, int F, int64_t n_values, int B);
