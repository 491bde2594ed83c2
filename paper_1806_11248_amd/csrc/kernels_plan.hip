// Depth-wise growth planned on the device (Alg. 1's loop over the levels of a tree).
//
// Between the passes over the rows (histograms, partition) a level needs a few decisions on small tables: which node
// splits where, which rows a tile of the partition takes, which child's histogram is built and how its rows are cut
// into jobs.  Made on the host they cost two waits and three or four small copies per level (about 100 us, more than
// the passes themselves below a million rows).  Here they are two small launches per level, so that a whole tree is
// enqueued without a wait:
//   plan_split     after the evaluation: merges a node's chunk records, decides, numbers the children, writes the
//                  partition's jobs.  One workgroup: everything it does is a prefix sum over the level's nodes.
//   plan_children  after the partition has counted the left rows: the children's rows, which one is built, its
//                  histogram jobs, the evaluation table of the next level; clears the histograms that are added into.
//                  Every workgroup forms the same prefix sums over the splits (a few thousand at most) and writes its
//                  share of the jobs, so that the clearing and the table need one launch, not two.
// The passes themselves are launched over the most nodes, tiles or jobs the level can have; the workgroups past the
// real count (which they read from the level's entry) leave at once.
// The decisions are those of the host loop, value for value: gains and sums are compared and added in the same types.
#include "gbt_internal.h"
#include "wave_scan.h"

namespace {

constexpr int kSplitBlock = 1024;
constexpr int kChildBlock = 256;

// Inclusive prefix sum over the workgroup; total in *sum.  tmp: one word per wave.
template <int BLOCK>
__device__ __forceinline__ int64_t block_scan(int64_t x, int64_t *tmp, int64_t *sum) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t incl = wave_scan_i64(x);
    __syncthreads();   // (tmp may still be read by the scan before)
    if (lane == 63) tmp[wave] = incl;
    __syncthreads();
    int64_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < BLOCK / 64; ++w) {
        if (w < wave) before += tmp[w];
        all += tmp[w];
    }
    *sum = all;
    return before + incl;
}

__device__ __forceinline__ void set_leaf(const PlanView &v, uint32_t id, int64_t Gq, int64_t Hq) {
    char *t = v.tree;
    const DevTree T = v.arrays;
    ((int32_t *)(t + T.feature))[id] = -1;
    ((int32_t *)(t + T.bin))[id] = 0;
    ((int32_t *)(t + T.default_left))[id] = 0;
    ((int32_t *)(t + T.left))[id] = -1;
    ((int32_t *)(t + T.right))[id] = -1;
    const double G = (double)Gq * v.inv_sg, H = (double)Hq * v.inv_sh;
    ((double *)(t + T.weight))[id] = H + v.lambda > 0.0 ? -G / (H + v.lambda) : 0.0;
}

__global__ __launch_bounds__(64) void plan_root_kernel(PlanView v, const int64_t *__restrict__ sums, int n_sums, uint32_t n_rows,
                                                       int n_levels) {
    int64_t G = 0, H = 0;
    for (int i = threadIdx.x; i < n_sums; i += 64) {
        G += sums[2 * i];
        H += sums[2 * i + 1];
    }
    G = last_lane_i64(wave_scan_i64(G));
    H = last_lane_i64(wave_scan_i64(H));
    for (int d = threadIdx.x; d < n_levels; d += 64) {
        PlanLevel l{};
        if (d == 0) l.n_nodes = 1;
        v.levels[d] = l;
    }
    if (threadIdx.x == 0) {
        PlanNode nd{};
        nd.len = n_rows;
        nd.Gq = G;
        nd.Hq = H;
        nd.feature = -1;
        nd.left = -1;
        v.nodes[0] = nd;
        v.enodes[0] = EvalNode{0, nd.Gq, nd.Hq, GBT_NO_HIST, GBT_NO_HIST};
        set_leaf(v, 0, nd.Gq, nd.Hq);
        DevTree head = v.arrays;
        head.n_nodes = 1;
        head.pad = 0;
        *(DevTree *)v.tree = head;
    }
}

__global__ __launch_bounds__(kSplitBlock) void plan_split_kernel(PlanView v, int d, int chunks, uint32_t tile_rows) {
    __shared__ int64_t tmp[kSplitBlock / 64];
    const uint32_t n = v.levels[d].n_nodes, first = v.levels[d].first_node;
    const uint32_t first_child = first + n;
    // the best of each node's chunks: a group of lanes per node (largest gain, the earliest chunk on equal gains)
    int gs = 1;
    while (gs < chunks && gs < 64) gs <<= 1;
    const int sub = threadIdx.x / gs, lane_in = threadIdx.x % gs;
    for (uint32_t i0 = 0; i0 < n; i0 += (uint32_t)(kSplitBlock / gs)) {
        const uint32_t i = i0 + (uint32_t)sub;
        double gain = -INFINITY;
        uint32_t at = 0xffffffffu;
        if (i < n)
            for (int c = lane_in; c < chunks; c += gs) {
                const gbt_split *r = v.recs + (size_t)i * chunks + c;
                if (r->valid && (at == 0xffffffffu || r->gain > gain)) {
                    gain = r->gain;
                    at = (uint32_t)c;
                }
            }
        for (int o = gs >> 1; o > 0; o >>= 1) {
            const int64_t gb = __double_as_longlong(gain);
            const int lo = __shfl_xor((int)(gb & 0xffffffff), o), hi = __shfl_xor((int)(gb >> 32), o);
            const double g2 = __longlong_as_double((int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo));
            const uint32_t a2 = (uint32_t)__shfl_xor((int)at, o);
            if (a2 != 0xffffffffu && (at == 0xffffffffu || g2 > gain || (g2 == gain && a2 < at))) {
                gain = g2;
                at = a2;
            }
        }
        if (i < n && lane_in == 0) {
            uint32_t w = 0xffffffffu;
            if (at != 0xffffffffu && gain > v.min_gain && v.nodes[first + i].len > 0) {
                const gbt_split *r = v.recs + (size_t)i * chunks + at;
                if (r->feature >= 0 && r->feature < v.F && r->bin >= 0 && r->bin < v.B) w = at;
            }
            v.win[i] = w;
        }
    }
    __syncthreads();
    // jobs in node order: one prefix sum carries the number of splits (low half) and of tiles (high half)
    int64_t carry = 0;
    for (uint32_t i0 = 0; i0 < n; i0 += kSplitBlock) {
        const uint32_t i = i0 + threadIdx.x;
        const uint32_t w = i < n ? v.win[i] : 0xffffffffu;
        const bool ok = w != 0xffffffffu;
        uint32_t begin = 0, len = 0, tiles = 0;
        if (ok) {
            begin = v.nodes[first + i].begin;
            len = v.nodes[first + i].len;
            tiles = (len + tile_rows - 1) / tile_rows;
        }
        const int64_t x = ok ? (int64_t)(((uint64_t)tiles << 32) | 1u) : 0;
        int64_t all;
        const int64_t excl = carry + block_scan<kSplitBlock>(x, tmp, &all) - x;
        if (ok) {
            const gbt_split r = v.recs[(size_t)i * chunks + w];
            const uint32_t k = (uint32_t)excl, id = first + i, lc = first_child + 2u * k;
            PartJob j;
            j.seg_begin = begin;
            j.seg_len = len;
            j.feature = (uint32_t)r.feature;
            j.bin = (uint32_t)r.bin;
            j.default_left = (uint32_t)r.default_left;
            j.tile_begin = (uint32_t)((uint64_t)excl >> 32);
            j.n_tiles = tiles;
            j.pad = 2;
            j.hist_off = 0;
            v.pjobs[k] = j;
            v.pinfo[k] = PlanJob{id, 0, r.GLq, r.HLq};
            for (int c = 0; c < v.cursors_per_job; ++c) v.cursors[((size_t)k * v.cursors_per_job + c) * kCursorStride] = 0ull;
            PlanNode &nd = v.nodes[id];
            nd.gain = r.gain;
            nd.feature = r.feature;
            nd.bin = r.bin;
            nd.default_left = r.default_left;
            nd.left = (int32_t)lc;
            nd.threshold = r.bin < v.B - 1 ? v.cuts[(size_t)r.feature * (v.B - 1) + r.bin] : INFINITY;
            const DevTree T = v.arrays;
            ((int32_t *)(v.tree + T.feature))[id] = r.feature;
            ((int32_t *)(v.tree + T.bin))[id] = r.bin;
            ((int32_t *)(v.tree + T.default_left))[id] = r.default_left;
            ((int32_t *)(v.tree + T.left))[id] = (int32_t)lc;
            ((int32_t *)(v.tree + T.right))[id] = (int32_t)lc + 1;
        }
        carry += all;
    }
    if (threadIdx.x == 0) {
        const uint32_t ns = (uint32_t)carry;
        v.levels[d].n_splits = ns;
        v.levels[d].n_tiles = (uint32_t)((uint64_t)carry >> 32);
        DevTree *head = (DevTree *)v.tree;
        head->n_nodes = (int32_t)(first_child + 2u * ns);
        if (ns) head->pad = d + 1;
        // (a hint for the host, which may have stopped enqueuing levels by then: it is read without waiting)
        __hip_atomic_store(v.hint + d, ns, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// The cheapest of the candidate piece lengths (gbt_piece_cost); sixteen threads count the pieces of one candidate.  Levels of
// more than kPieceNodes splits take the middle candidate: their nodes are one piece each nearly everywhere.
constexpr uint32_t kPieceNodes = 2048;
__device__ uint32_t pick_piece(const PlanHistRule &rule, int64_t rows, uint32_t ns, const uint32_t *s_small, double *s_cost) {
    if (ns > kPieceNodes) return (uint32_t)gbt_piece_candidate(rule, rows, kPieceCandidates / 2);
    static_assert(kChildBlock == 16 * kPieceCandidates, "sixteen threads per candidate");
    const int c = threadIdx.x >> 4;
    const uint32_t length = (uint32_t)gbt_piece_candidate(rule, rows, c);
    uint32_t pieces = 0, single = 0, longest = 0;
    for (uint32_t k = threadIdx.x & 15; k < ns; k += 16) {
        const uint32_t s = s_small[k], p = (s + length - 1) / length;
        pieces += p;
        single += p == 1 ? 1u : 0u;
        longest = longest > s ? longest : s;
    }
    for (int o = 8; o > 0; o >>= 1) {
        pieces += (uint32_t)__shfl_xor((int)pieces, o);
        single += (uint32_t)__shfl_xor((int)single, o);
        const uint32_t l = (uint32_t)__shfl_xor((int)longest, o);
        longest = longest > l ? longest : l;
    }
    if ((threadIdx.x & 15) == 0) s_cost[c] = gbt_piece_cost(rule, rows, length, pieces, rule.exclusive_ok ? single : 0, longest);
    __syncthreads();
    int best = 0;
    for (int k = 1; k < kPieceCandidates; ++k)
        if (s_cost[k] < s_cost[best]) best = k;
    return (uint32_t)gbt_piece_candidate(rule, rows, best);
}

__global__ __launch_bounds__(kChildBlock) void plan_children_kernel(PlanView v, int d, const uint32_t *__restrict__ n_left,
                                                                    int stride, int with_hist, PlanHistRule rule, uint32_t pieces_max) {
    __shared__ int64_t tmp[kChildBlock / 64];
    __shared__ uint32_t s_small[kPieceNodes];
    __shared__ double s_cost[kPieceCandidates];
    __shared__ uint32_t s_off[kChildBlock], s_begin[kChildBlock], s_len[kChildBlock], s_slot[kChildBlock], s_pieces[kChildBlock];
    const uint32_t ns = v.levels[d].n_splits;
    const uint32_t first_child = v.levels[d].first_node + v.levels[d].n_nodes;
    const bool lead = blockIdx.x == 0;
    auto left_rows = [&](uint32_t k, uint32_t len) -> uint32_t {
        const uint32_t l = n_left ? n_left[(size_t)k * stride] : 0u;
        return l < len ? l : len;
    };
    uint32_t rpj = 1;
    int64_t built = 0, pieces = 0;
    if (with_hist) {
        int64_t mine = 0;
        for (uint32_t k = threadIdx.x; k < ns; k += kChildBlock) {
            const uint32_t len = v.pjobs[k].seg_len, l = left_rows(k, len), small = l <= len - l ? l : len - l;
            mine += small;
            if (k < kPieceNodes) s_small[k] = small;
        }
        (void)block_scan<kChildBlock>(mine, tmp, &built);   // (its barriers also complete s_small)
        rpj = pick_piece(rule, built, ns, s_small, s_cost);
        mine = 0;
        for (uint32_t k = threadIdx.x; k < ns; k += kChildBlock) {
            const uint32_t len = v.pjobs[k].seg_len, l = left_rows(k, len);
            mine += ((l <= len - l ? l : len - l) + rpj - 1) / rpj;
        }
        (void)block_scan<kChildBlock>(mine, tmp, &pieces);
    }
    // (the host's bound holds for every rule and number of rows; were it short, nothing is written past the table)
    const bool fits = (uint32_t)pieces <= pieces_max;
    // Whose nodes: with fewer splits than workgroups a split's node is shared by `shares` of them, else every `lanes`-th is one
    // workgroup's own.  (Every workgroup looking at every node took 0.07 us a node: 1672 splits 122 us.)
    const uint32_t shares = ns < gridDim.x ? gridDim.x / (ns > 0 ? ns : 1u) : 1u, lanes = gridDim.x / shares;
    const uint32_t lane = blockIdx.x / shares, share = blockIdx.x % shares;   // (a lane past the last: a workgroup too many)
    int64_t carry = 0;
    uint32_t bad = 0;
    for (uint32_t k0 = 0; k0 < ns; k0 += kChildBlock) {
        const uint32_t k = k0 + threadIdx.x;
        uint32_t mine = 0;   // pieces of this thread's node
        if (k < ns) {
            const PartJob j = v.pjobs[k];
            const PlanJob info = v.pinfo[k];
            const PlanNode nd = v.nodes[info.node];
            const uint32_t l = left_rows(k, j.seg_len), r = j.seg_len - l;
            if (n_left && n_left[(size_t)k * stride] > j.seg_len) bad = 1;
            const uint32_t lid = first_child + 2u * k, rid = lid + 1u;
            const bool left_small = l <= r;
            const uint32_t small = left_small ? l : r;
            if (with_hist) {
                mine = (small + rpj - 1) / rpj;
                s_begin[threadIdx.x] = left_small ? j.seg_begin : j.seg_begin + l;
                s_len[threadIdx.x] = small;
                s_slot[threadIdx.x] = left_small ? lid : rid;
                s_pieces[threadIdx.x] = mine;
            }
            if (lead) {
                const int64_t GR = nd.Gq - info.GLq, HR = nd.Hq - info.HLq;
                PlanNode c{};
                c.feature = -1;
                c.left = -1;
                c.threshold = INFINITY;
                c.begin = j.seg_begin;
                c.len = n_left ? l : 0u;
                c.Gq = info.GLq;
                c.Hq = info.HLq;
                v.nodes[lid] = c;
                c.begin = j.seg_begin + l;
                c.len = n_left ? r : 0u;
                c.Gq = GR;
                c.Hq = HR;
                v.nodes[rid] = c;
                set_leaf(v, lid, info.GLq, info.HLq);
                set_leaf(v, rid, GR, HR);
                if (with_hist) {
                    const uint64_t hl = (uint64_t)v.hist_len, par = info.node * hl, blt = (left_small ? lid : rid) * hl;
                    v.enodes[2u * k] = EvalNode{lid * hl, info.GLq, info.HLq, left_small ? GBT_NO_HIST : par,
                                                left_small ? GBT_NO_HIST : blt};
                    v.enodes[2u * k + 1u] = EvalNode{rid * hl, GR, HR, left_small ? par : GBT_NO_HIST,
                                                     left_small ? blt : GBT_NO_HIST};
                }
            }
        }
        if (!with_hist) continue;
        int64_t all;
        const int64_t incl = block_scan<kChildBlock>((int64_t)mine, tmp, &all);
        s_off[threadIdx.x] = (uint32_t)(carry + incl) - mine;
        __syncthreads();
        const uint32_t here = !fits || lane >= lanes ? 0u : ns - k0 < (uint32_t)kChildBlock ? ns - k0 : (uint32_t)kChildBlock;
        for (uint32_t q = (lane + lanes - k0 % lanes) % lanes; q < here; q += lanes) {
            const uint32_t len = s_len[q];
            const bool exclusive = rule.exclusive_ok && len <= rpj && len > 0;
            if (!exclusive) {   // its jobs add into the histogram (or it has none)
                ulonglong2 *z = (ulonglong2 *)(v.pool + (int64_t)s_slot[q] * v.hist_len);
                for (int64_t i = share * kChildBlock + threadIdx.x; i < v.hist_len / 2; i += shares * kChildBlock)
                    z[i] = make_ulonglong2(0ull, 0ull);
            }
            for (uint32_t t = share * kChildBlock + threadIdx.x; t < s_pieces[q] * (uint32_t)rule.tiles; t += shares * kChildBlock) {
                const uint32_t piece = t / (uint32_t)rule.tiles, tile = t - piece * (uint32_t)rule.tiles;
                HistJob h;
                h.hist_off = (uint64_t)s_slot[q] * (uint64_t)v.hist_len;
                h.row_begin = s_begin[q] + piece * rpj;
                h.n_rows = len - piece * rpj < rpj ? len - piece * rpj : rpj;
                h.f0 = tile * (uint32_t)rule.ft;
                h.ft = (uint32_t)rule.width - h.f0 < (uint32_t)rule.ft ? (uint32_t)rule.width - h.f0 : (uint32_t)rule.ft;
                h.pad0 = exclusive ? 1u : 0u;
                h.pad1 = 0;
                v.hjobs[gbt_job_place(s_off[q] + piece, tile, (uint32_t)pieces, (uint32_t)rule.tiles)] = h;
            }
        }
        carry += all;
        __syncthreads();   // (the tables are rewritten)
    }
    if (lead && bad) v.levels[d + 1].bad = PLAN_BAD_ROWS;
    if (lead && threadIdx.x == 0) {
        PlanLevel &nx = v.levels[d + 1];
        nx.first_node = first_child;
        nx.n_nodes = 2u * ns;
        nx.n_hist_jobs = fits ? (uint32_t)(pieces * rule.tiles) : 0u;
        if (!fits) nx.bad = PLAN_BAD_JOBS;
        nx.built_rows = (uint64_t)built;
    }
}

// rank[id] of every leaf: its place in the tree's left-to-right order.  Leaves are counted from the deepest level up,
// then handed out from the root down.  One workgroup; n_levels levels.
__global__ __launch_bounds__(kSplitBlock) void plan_rank_kernel(PlanView v, int n_levels, uint32_t *count, uint32_t *rank) {
    const int32_t *left = (const int32_t *)(v.tree + v.arrays.left);
    for (int d = n_levels - 1; d >= 0; --d) {
        const uint32_t f = v.levels[d].first_node, n = v.levels[d].n_nodes;
        for (uint32_t i = threadIdx.x; i < n; i += kSplitBlock) {
            const int32_t l = left[f + i];
            count[f + i] = l < 0 ? 1u : count[l] + count[l + 1];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) rank[0] = 0;
    __syncthreads();
    for (int d = 0; d < n_levels; ++d) {
        const uint32_t f = v.levels[d].first_node, n = v.levels[d].n_nodes;
        for (uint32_t i = threadIdx.x; i < n; i += kSplitBlock) {
            const int32_t l = left[f + i];
            if (l < 0) continue;
            const uint32_t r = rank[f + i];
            rank[l] = r;
            rank[l + 1] = r + count[l];
        }
        __syncthreads();
    }
}

// What the host reads: the levels and the nodes, stored into its memory.  counted (may be NULL): row counts of the
// nodes whose partition was left to the walk (the children of depth `last`), one per kNodeRowsStride words.
__global__ __launch_bounds__(256) void plan_finish_kernel(PlanView v, int n_levels, int last, const uint32_t *__restrict__ counted,
                                                          PlanLevel *levels_out, PlanNode *nodes_out, uint32_t cap) {
    const uint32_t n = (uint32_t)((const DevTree *)v.tree)->n_nodes;
    const uint32_t deferred_from = counted ? v.levels[last].first_node + v.levels[last].n_nodes : 0xffffffffu;
    for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < n && i < cap; i += gridDim.x * 256u) {
        PlanNode nd = v.nodes[i];
        if (i >= deferred_from) nd.len = counted[(size_t)i * kNodeRowsStride];
        nodes_out[i] = nd;
    }
    if (blockIdx.x == 0)
        for (int d = threadIdx.x; d < n_levels; d += 256) levels_out[d] = v.levels[d];
}

}  // namespace

hipError_t gbt_launch_plan_root(hipStream_t s, const PlanView &v, const int64_t *sums, int n_sums, int64_t n, int n_levels) {
    plan_root_kernel<<<1, 64, 0, s>>>(v, sums, n_sums, (uint32_t)n, n_levels);
    return hipGetLastError();
}
hipError_t gbt_launch_plan_split(hipStream_t s, const PlanView &v, int depth, int chunks, uint32_t tile_rows) {
    plan_split_kernel<<<1, kSplitBlock, 0, s>>>(v, depth, chunks, tile_rows);
    return hipGetLastError();
}
hipError_t gbt_launch_plan_children(hipStream_t s, const PlanView &v, int depth, int64_t max_splits, const uint32_t *n_left,
                                    int stride, bool with_hist, const PlanHistRule &rule, uint32_t jobs_max) {
    // workgroups: enough to clear what the level may have to clear at a few kilobytes each
    const int64_t clear = with_hist ? max_splits * v.hist_len : 0;
    const int64_t grid = std::min<int64_t>(256, std::max<int64_t>(1, (clear + 2047) / 2048));
    plan_children_kernel<<<(unsigned)grid, kChildBlock, 0, s>>>(v, depth, n_left, stride, with_hist ? 1 : 0, rule, jobs_max / (uint32_t)rule.tiles);
    return hipGetLastError();
}
hipError_t gbt_launch_plan_rank(hipStream_t s, const PlanView &v, int n_levels, uint32_t *count, uint32_t *rank) {
    plan_rank_kernel<<<1, kSplitBlock, 0, s>>>(v, n_levels, count, rank);
    return hipGetLastError();
}
hipError_t gbt_launch_plan_finish(hipStream_t s, const PlanView &v, int n_levels, int last, const uint32_t *counted,
                                  PlanLevel *levels_out, PlanNode *nodes_out, uint32_t cap) {
    const unsigned grid = (unsigned)std::min<int64_t>(64, std::max<int64_t>(1, (cap + 255) / 256));
    plan_finish_kernel<<<grid, 256, 0, s>>>(v, n_levels, last, counted, levels_out, nodes_out, cap);
    return hipGetLastError();
}
