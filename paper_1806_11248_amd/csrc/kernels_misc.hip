// Small streaming kernels around the tree builder: fills, fixed-point
// conversion of the gradient pairs, node totals, gradients (Eq. 1-2), sibling
// subtraction, export, bit packing (Sec. 2.2), prediction (Sec. 2.4) and the
// final leaf gather.  All are bandwidth-trivial next to the histogram kernel.
#include "gbt_internal.h"

namespace {

constexpr int kBlock = 256;

inline int grid_for(int64_t count, int per_block, int cap = 1 << 20) {
    int64_t g = (count + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (int)g;
}

__global__ void fill_u64_kernel(uint64_t *p, uint64_t v, int64_t count) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void iota_u32_kernel(uint32_t *p, int64_t count) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = (uint32_t)i;
}

// Reductions over all rows leave one partial result of 16 bytes per workgroup (at most kRedGroups of kRedBlock threads: as
// many waves as are resident); whoever reads them (the host, from its own memory; plan_root_kernel) puts them together.
// One atomic per workgroup on one address, some 12 ns each whatever the kernel does meanwhile, was what these launches
// waited for: 10M pairs, absmax 78 us, to_fixed 61; 1M rows, gradients with bounds 15.6 us.
constexpr int kRedBlock = 1024, kRedGroups = 512;
inline int red_grid(int64_t count, int per_thread) { return grid_for(count, kRedBlock * per_thread, kRedGroups); }

// max |g| and max |h| as raw float bits (non-negative floats order like their
// bit patterns; NaN sorts above +inf, so a non-finite input is detected).
// Word 2 becomes non-zero if any h is negative, word 3 is the smallest |h| as bits.
// A thread takes kStreamBatch 16-byte loads (two pairs each) that are all issued before the
// first is used, so that enough bytes are in flight to cover the HBM latency.
constexpr int kStreamBatch = 4;
// The pointers must be 16-byte aligned; `head` pairs (0 or 1) in front of them are taken singly,
// which is how a caller's pointer that is only 8-byte aligned is served.
// The workgroup's (largest |g|, largest |h|, is some h negative, smallest |h|) to out[blockIdx.x]; every thread must call.
__device__ __forceinline__ void store_bounds(uint32_t mg, uint32_t mh, uint32_t neg, uint32_t lh, uint4 *out) {
    for (int o = 32; o > 0; o >>= 1) {
        const uint32_t a = __shfl_xor(mg, o), b = __shfl_xor(mh, o), c = __shfl_xor(lh, o);
        mg = a > mg ? a : mg;
        mh = b > mh ? b : mh;
        lh = c < lh ? c : lh;
        neg |= __shfl_xor(neg, o);
    }
    __shared__ uint4 red[kRedBlock / 64];
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = make_uint4(mg, mh, neg, lh);
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < (int)(blockDim.x >> 6); ++w) {
            mg = max(mg, red[w].x);
            mh = max(mh, red[w].y);
            neg |= red[w].z;
            lh = min(lh, red[w].w);
        }
        out[blockIdx.x] = make_uint4(mg, mh, neg, lh);
    }
}

__global__ __launch_bounds__(kRedBlock) void absmax_kernel(const float2 *gp, int64_t n, int head, uint4 *out) {
    uint32_t mg = 0, mh = 0, neg = 0, lh = 0xffffffffu;
    if (head && blockIdx.x == 0 && threadIdx.x == 1) {
        const float2 v = gp[-1];
        mg = __float_as_uint(v.x) & 0x7fffffffu;
        mh = __float_as_uint(v.y) & 0x7fffffffu;
        lh = mh;
        neg = v.y < 0.0f ? 1u : 0u;
    }
    const float4 *gp4 = (const float4 *)gp;
    const int64_t n4 = n >> 1;   // whole 16-byte pieces
    auto take = [&](const float4 &v) {
        const uint32_t a0 = __float_as_uint(v.x) & 0x7fffffffu, b0 = __float_as_uint(v.y) & 0x7fffffffu;
        const uint32_t a1 = __float_as_uint(v.z) & 0x7fffffffu, b1 = __float_as_uint(v.w) & 0x7fffffffu;
        mg = max(mg, max(a0, a1));
        mh = max(mh, max(b0, b1));
        lh = min(lh, min(b0, b1));
        neg |= (v.y < 0.0f || v.w < 0.0f) ? 1u : 0u;
    };
    // a workgroup takes contiguous chunks of kStreamBatch * kRedBlock pieces; whole chunks need no conditional load
    const int64_t chunk = (int64_t)kStreamBatch * kRedBlock, n_whole = n4 / chunk;
    for (int64_t c = blockIdx.x; c < n_whole; c += gridDim.x) {
        float4 v[kStreamBatch];
#pragma unroll
        for (int k = 0; k < kStreamBatch; ++k) v[k] = gp4[c * chunk + k * kRedBlock + threadIdx.x];
#pragma unroll
        for (int k = 0; k < kStreamBatch; ++k) take(v[k]);
    }
    for (int64_t i = n_whole * chunk + (int64_t)blockIdx.x * kRedBlock + threadIdx.x; i < n4; i += (int64_t)gridDim.x * kRedBlock)
        take(gp4[i]);
    if ((n & 1) && blockIdx.x == 0 && threadIdx.x == 0) {   // the odd last pair
        const float2 v = gp[n - 1];
        mg = max(mg, __float_as_uint(v.x) & 0x7fffffffu);
        mh = max(mh, __float_as_uint(v.y) & 0x7fffffffu);
        lh = min(lh, __float_as_uint(v.y) & 0x7fffffffu);
        neg |= v.y < 0.0f ? 1u : 0u;
    }
    store_bounds(mg, mh, neg, lh, out);
}

__device__ inline int64_t wave_sum_i64(int64_t v) {
    for (int o = 32; o > 0; o >>= 1) {
        int lo = __shfl_xor((int)(v & 0xffffffff), o);
        int hi = __shfl_xor((int)(v >> 32), o);
        v += (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
    }
    return v;
}

// The workgroup's (g, h) to sums[blockIdx.x]; every thread must call.
__device__ inline void store_sums(int64_t g, int64_t h, longlong2 *sums) {
    __shared__ int64_t red[2][kRedBlock / 64];
    g = wave_sum_i64(g);
    h = wave_sum_i64(h);
    if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = g;
        red[1][threadIdx.x >> 6] = h;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < (int)(blockDim.x >> 6); ++w) {
            g += red[0][w];
            h += red[1][w];
        }
        sums[blockIdx.x] = make_longlong2(g, h);
    }
}

// gp and gq must be 16-byte aligned; `head` pairs (0 or 1) in front of BOTH are taken singly.
__global__ __launch_bounds__(kRedBlock) void to_fixed_kernel(const float2 *gp, int64_t n, int head, double sg, double sh,
                                                             int2 *gq, longlong2 *sums) {
    int64_t g = 0, h = 0;
    if (head && blockIdx.x == 0 && threadIdx.x == 1) {
        const float2 v = gp[-1];
        int2 q;
        q.x = __double2int_rn((double)v.x * sg);
        q.y = __double2int_rn((double)v.y * sh);
        gq[-1] = q;
        g = q.x;
        h = q.y;
    }
    const float4 *gp4 = (const float4 *)gp;
    int4 *gq4 = (int4 *)gq;
    const int64_t n4 = n >> 1;   // whole 16-byte pieces (two pairs)
    auto take = [&](int64_t at, const float4 &v) {
        int4 q;
        q.x = __double2int_rn((double)v.x * sg);
        q.y = __double2int_rn((double)v.y * sh);
        q.z = __double2int_rn((double)v.z * sg);
        q.w = __double2int_rn((double)v.w * sh);
        gq4[at] = q;
        g += (int64_t)q.x + q.z;
        h += (int64_t)q.y + q.w;
    };
    const int64_t chunk = (int64_t)kStreamBatch * kRedBlock, n_whole = n4 / chunk;
    for (int64_t c = blockIdx.x; c < n_whole; c += gridDim.x) {
        float4 v[kStreamBatch];
#pragma unroll
        for (int k = 0; k < kStreamBatch; ++k) v[k] = gp4[c * chunk + k * kRedBlock + threadIdx.x];
#pragma unroll
        for (int k = 0; k < kStreamBatch; ++k) take(c * chunk + k * kRedBlock + threadIdx.x, v[k]);
    }
    for (int64_t i = n_whole * chunk + (int64_t)blockIdx.x * kRedBlock + threadIdx.x; i < n4; i += (int64_t)gridDim.x * kRedBlock)
        take(i, gp4[i]);
    if ((n & 1) && blockIdx.x == 0 && threadIdx.x == 0) {   // the odd last pair
        const float2 v = gp[n - 1];
        int2 q;
        q.x = __double2int_rn((double)v.x * sg);
        q.y = __double2int_rn((double)v.y * sh);
        gq[n - 1] = q;
        g += q.x;
        h += q.y;
    }
    if (sums) store_sums(g, h, sums);
}

// One pair per load: for a source and a destination whose 16-byte alignments differ.
__global__ __launch_bounds__(kRedBlock) void to_fixed_pairs_kernel(const float2 *gp, int64_t n, double sg, double sh,
                                                                   int2 *gq, longlong2 *sums) {
    int64_t g = 0, h = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const float2 v = gp[i];
        int2 q;
        q.x = __double2int_rn((double)v.x * sg);
        q.y = __double2int_rn((double)v.y * sh);
        gq[i] = q;
        g += q.x;
        h += q.y;
    }
    if (sums) store_sums(g, h, sums);
}

__global__ __launch_bounds__(kRedBlock) void sum_gq_kernel(const int2 *gq, const uint32_t *row_idx, int64_t n_rows, longlong2 *sums) {
    int64_t g = 0, h = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_rows;
         i += (int64_t)gridDim.x * blockDim.x) {
        int64_t r = row_idx ? (int64_t)row_idx[i] : i;
        int2 q = gq[r];
        g += q.x;
        h += q.y;
    }
    store_sums(g, h, sums);
}

// Eq. 1 and Eq. 2 (logistic) and the squared-error pair, one instance per
// thread.  Evaluated in fp64 and rounded once so that the fp32 pair does not
// depend on a fast-math exp.
__device__ __forceinline__ float2 gradient_pair(int objective, float margin, float label) {
    double m = margin, y = label, g, h;
    if (objective == GBT_OBJ_LOGISTIC) {
        double p = 1.0 / (1.0 + exp(-m));
        g = p - y;
        h = p * (1.0 - p);
    } else {
        g = m - y;
        h = 1.0;
    }
    return make_float2((float)g, (float)h);
}
// A thread takes four consecutive instances at a time (16-byte loads, two 16-byte stores) where the three
// arrays are 16-byte aligned; the launcher says so.  The last n mod 4 instances are taken singly.
// bounds (may be NULL): what absmax_kernel leaves for these pairs, reduced on the way so that the pairs need not be read
// again for them.
__global__ __launch_bounds__(kRedBlock) void gradients_kernel(int objective, const float *__restrict__ margin,
                                                           const float *__restrict__ label, int64_t n,
                                                           float2 *__restrict__ gp, int vec, uint4 *bounds, int nt) {
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, nthreads = (int64_t)gridDim.x * blockDim.x;
    uint32_t mg = 0, mh = 0, neg = 0, lh = 0xffffffffu;
    auto note = [&](const float2 &v) {
        const uint32_t a = __float_as_uint(v.x) & 0x7fffffffu, b = __float_as_uint(v.y) & 0x7fffffffu;
        mg = max(mg, a);
        mh = max(mh, b);
        lh = min(lh, b);
        neg |= v.y < 0.0f ? 1u : 0u;
    };
    int64_t done = 0;
    if (vec) {
        const int64_t n4 = n >> 2;
        const float4 *m4 = (const float4 *)margin, *y4 = (const float4 *)label;
        float4 *o4 = (float4 *)gp;
        for (int64_t i = tid; i < n4; i += nthreads) {
            typedef float f4v __attribute__((ext_vector_type(4)));
            const float4 m = m4[i], y = y4[i];
            const float2 a = gradient_pair(objective, m.x, y.x), b = gradient_pair(objective, m.y, y.y);
            const float2 c = gradient_pair(objective, m.z, y.z), d = gradient_pair(objective, m.w, y.w);
            // nt: non-temporal stores.  Written the ordinary way, the last few hundred MB of an array much larger than
            // the memory-side cache are still waiting there when the kernel ends, and their write-back then competes
            // with whatever streams next (measured: the root histogram launch right behind takes 0.52 ms instead of
            // 0.48 on 115M rows).  Pairs that fit the cache are better left in it for the launch that reads them.
            if (nt) {
                const f4v s0 = {a.x, a.y, b.x, b.y}, s1 = {c.x, c.y, d.x, d.y};
                __builtin_nontemporal_store(s0, (f4v *)&o4[2 * i]);
                __builtin_nontemporal_store(s1, (f4v *)&o4[2 * i + 1]);
            } else {
                o4[2 * i] = make_float4(a.x, a.y, b.x, b.y);
                o4[2 * i + 1] = make_float4(c.x, c.y, d.x, d.y);
            }
            note(a);
            note(b);
            note(c);
            note(d);
        }
        done = n4 << 2;
    }
    for (int64_t i = done + tid; i < n; i += nthreads) {
        const float2 v = gradient_pair(objective, margin[i], label[i]);
        gp[i] = v;
        note(v);
    }
    if (bounds) store_bounds(mg, mh, neg, lh, bounds);
}

__global__ void subtract_one_kernel(const int64_t *p, const int64_t *c, int64_t *o, int64_t count) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        o[i] = p[i] - c[i];
}

__global__ void export_kernel(const int64_t *hist, int64_t count, double inv_sg, double inv_sh,
                              double *out) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        out[i] = (double)hist[i] * ((i & 1) ? inv_sh : inv_sg);
}

// Sec. 2.2: one thread assembles one 32-bit word of the bit stream from the
// elements that overlap it (no atomics; the trailing pad word comes out zero).
__global__ void compress_kernel(const uint16_t *sym, int64_t n_elems, int bits, uint32_t *packed,
                                int64_t n_words) {
    for (int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; w < n_words;
         w += (int64_t)gridDim.x * blockDim.x) {
        int64_t bit0 = w * 32;
        int64_t e = bit0 / bits;
        uint32_t word = 0;
        for (; e < n_elems; ++e) {
            int64_t pos = e * bits - bit0;   // may be negative for the first element
            if (pos >= 32) break;
            uint32_t s = sym[e];
            word |= pos >= 0 ? (s << pos) : (s >> (-pos));
        }
        packed[w] = word;
    }
}

__device__ inline uint32_t load_symbol(const uint32_t *packed, uint64_t elem, int bits, uint32_t mask) {
    uint64_t bp = elem * (uint64_t)bits;
    const uint32_t *w = packed + (bp >> 5);
    uint64_t v = (uint64_t)w[0] | ((uint64_t)w[1] << 32);
    return (uint32_t)(v >> (bp & 31)) & mask;
}

// Sec. 2.4: one instance per thread, trees in order, walking from the root.
__global__ void predict_kernel(const char *ws, const DevTree *trees, int n_trees,
                               const uint32_t *packed, int bits, uint32_t missing, const float *X,
                               int64_t n, int F, double eta, float *margin, int32_t *leaf_out) {
    const uint32_t mask = (1u << bits) - 1u;
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n;
         r += (int64_t)gridDim.x * blockDim.x) {
        double m = margin ? margin[r] : 0.0;
        for (int t = 0; t < n_trees; ++t) {
            DevTree T = trees[t];
            const int32_t *feature = (const int32_t *)(ws + T.feature);
            const int32_t *bin = (const int32_t *)(ws + T.bin);
            const int32_t *dl = (const int32_t *)(ws + T.default_left);
            const int32_t *left = (const int32_t *)(ws + T.left);
            const int32_t *right = (const int32_t *)(ws + T.right);
            const float *thr = (const float *)(ws + T.threshold);
            const double *weight = (const double *)(ws + T.weight);
            int node = 0;
            // a well-formed tree ends in fewer than n_nodes steps; the bound keeps a
            // malformed one from spinning
            for (int step = 0; step < T.n_nodes; ++step) {
                int f = feature[node];
                if (f < 0) break;
                bool go_left;
                if (packed) {
                    uint32_t s = load_symbol(packed, (uint64_t)r * F + f, bits, mask);
                    go_left = (s == missing) ? (dl[node] != 0) : ((int)s <= bin[node]);
                } else {
                    float x = X[r * F + f];
                    go_left = (x != x) ? (dl[node] != 0) : (x < thr[node]);
                }
                node = go_left ? left[node] : right[node];
            }
            m = (double)(float)(m + eta * weight[node]);
            if (leaf_out) leaf_out[r] = node;   // leaf mode: the caller passes one tree
        }
        if (margin) margin[r] = (float)m;
    }
}

// Same walk with the tree's nodes staged in LDS (32 bytes per node): the per-level
// node fetches then cost an LDS read instead of a dependent global load.
struct LdsNode {
    int32_t feature, bin, left, right;
    float thr;
    int32_t dl;
    double weight;
};
__global__ __launch_bounds__(256) void predict_lds_kernel(const char *ws, const DevTree *trees, int n_trees,
                                                          const uint32_t *packed, int bits, uint32_t missing,
                                                          const float *X, int64_t n, int F, double eta,
                                                          float *margin, int rows_per_block, int32_t *leaf_out) {
    extern __shared__ LdsNode nodes[];
    const uint32_t mask = (1u << bits) - 1u;
    const int64_t r0 = (int64_t)blockIdx.x * rows_per_block;
    const int64_t r1 = r0 + rows_per_block < n ? r0 + rows_per_block : n;
    for (int t = 0; t < n_trees; ++t) {
        const DevTree T = trees[t];
        __syncthreads();   // the previous tree's walks are done
        for (int i = threadIdx.x; i < T.n_nodes; i += 256) {
            LdsNode nd;
            nd.feature = ((const int32_t *)(ws + T.feature))[i];
            nd.bin = ((const int32_t *)(ws + T.bin))[i];
            nd.left = ((const int32_t *)(ws + T.left))[i];
            nd.right = ((const int32_t *)(ws + T.right))[i];
            nd.thr = ((const float *)(ws + T.threshold))[i];
            nd.dl = ((const int32_t *)(ws + T.default_left))[i];
            nd.weight = ((const double *)(ws + T.weight))[i];
            nodes[i] = nd;
        }
        __syncthreads();
        for (int64_t r = r0 + threadIdx.x; r < r1; r += 256) {
            const uint64_t rowbit = (uint64_t)r * (uint64_t)F * (uint64_t)bits;
            int node = 0;
            for (int step = 0; step < T.n_nodes; ++step) {
                const LdsNode nd = nodes[node];
                if (nd.feature < 0) break;
                bool go_left;
                if (packed) {
                    const uint64_t bp = rowbit + (uint64_t)nd.feature * (uint64_t)bits;
                    const uint32_t *w = packed + (bp >> 5);
                    const uint32_t sh = (uint32_t)(bp & 31);
                    uint32_t v = w[0] >> sh;
                    if (sh + (uint32_t)bits > 32u) v |= w[1] << (32u - sh);
                    const uint32_t s = v & mask;
                    go_left = (s == missing) ? (nd.dl != 0) : ((int)s <= nd.bin);
                } else {
                    const float x = X[r * F + nd.feature];
                    go_left = (x != x) ? (nd.dl != 0) : (x < nd.thr);
                }
                node = go_left ? nd.left : nd.right;
            }
            if (leaf_out) leaf_out[r] = node;
            else margin[r] = (float)((double)margin[r] + eta * nodes[node].weight);
        }
    }
}

// Rows of at most 128 bits: the whole row is fetched once (five words, funnel-shifted to the
// row's first bit) and every level's symbol is cut out of registers, so a tree walk costs one
// row fetch instead of one dependent gather per level.
__device__ __forceinline__ uint32_t pick4(const uint32_t (&W)[4], int i) {
    return i == 0 ? W[0] : (i == 1 ? W[1] : (i == 2 ? W[2] : W[3]));
}
// Nodes are staged as 8 bytes: x = left child id | default_left << 31 (the right child is
// left + 1, which the caller has checked), y = feature << 12 | bin.  A leaf is staged as a
// node that sends every row to itself (left = own id, default left, bin 0xfff >= any symbol),
// so every row takes exactly T.pad steps (the tree's depth) and the walks of the kPredRows rows
// a thread handles at once run side by side instead of one divergent loop after the other.
constexpr int kPredRows = 4;
constexpr size_t kWalkLds = 96u * 1024u;   // the most LDS a walk takes
__device__ __forceinline__ void stage_compact(const char *ws, const DevTree &T, uint2 *cnodes, double *lweight, int max_nodes) {
    const int n = T.n_nodes < max_nodes ? T.n_nodes : max_nodes;
    for (int i = threadIdx.x; i < n; i += 256) {
        const int32_t f = ((const int32_t *)(ws + T.feature))[i];
        uint2 c;
        if (f < 0) {
            c.x = (uint32_t)i | 0x80000000u;
            c.y = 0xfffu;
        } else {
            c.x = (uint32_t)((const int32_t *)(ws + T.left))[i] |
                  (((const int32_t *)(ws + T.default_left))[i] ? 0x80000000u : 0u);
            c.y = ((uint32_t)f << 12) | (uint32_t)((const int32_t *)(ws + T.bin))[i];
        }
        cnodes[i] = c;
        lweight[i] = ((const double *)(ws + T.weight))[i];
    }
}
// The rows that end in each node, counted per workgroup in LDS and then into node_rows[node * kNodeRowsStride] (one
// counter per 128-byte line: atomics on one line take turns).
__device__ __forceinline__ void flush_counts(const uint32_t *lcount, int max_nodes, uint32_t *node_rows) {
    __syncthreads();
    for (int i = threadIdx.x; i < max_nodes; i += 256) {
        const uint32_t c = lcount[i];
        if (c) atomicAdd(&node_rows[(size_t)i * kNodeRowsStride], c);
    }
}

// Q rows of a thread are walked side by side: kPredRows, or one where the matrix has too few rows to fill the chip.
// COUNT: with node_rows, where a workgroup takes many blocks.  The form without it takes one and has no loop over them (100M rows
// of four 5-bit symbols, depth 5: 586 us with the loop, 539 without).
template <int Q, bool COUNT>
__global__ __launch_bounds__(256) void predict_window_kernel(const char *ws, const DevTree *trees, int n_trees,
                                                             const uint32_t *packed, int64_t n_words, int bits,
                                                             uint32_t missing, int64_t n, int F, double eta,
                                                             float *margin, int rows_per_block, int max_nodes,
                                                             int32_t *leaf_out, uint32_t *node_rows,
                                                             const float *margin_src) {
    extern __shared__ uint2 cnodes[];
    double *lweight = (double *)(cnodes + max_nodes);
    uint32_t *lcount = (uint32_t *)(lweight + max_nodes);   // only there when node_rows is given
    if (COUNT)
        for (int i = threadIdx.x; i < max_nodes; i += 256) lcount[i] = 0;
    const uint32_t mask = (1u << bits) - 1u;
    const int64_t n_blocks = (n + rows_per_block - 1) / rows_per_block;
    for (int t = 0; t < n_trees; ++t) {
        const DevTree T = trees[t];
        __syncthreads();
        stage_compact(ws, T, cnodes, lweight, max_nodes);
        __syncthreads();
        const int depth = T.pad;
        for (int64_t blk = blockIdx.x; blk < (COUNT ? n_blocks : (int64_t)blockIdx.x + 1); blk += gridDim.x) {   // (uncounted: one block)
        const int64_t r0 = blk * rows_per_block;
        const int64_t r1 = r0 + rows_per_block < n ? r0 + rows_per_block : n;
        for (int64_t rb = r0 + threadIdx.x; rb < r1; rb += 256 * Q) {
            uint32_t W[Q][4];
            float m[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                // rows past the end repeat the last row (their result is dropped)
                const int64_t r = rb + 256 * q < r1 ? rb + 256 * q : r1 - 1;
                const uint64_t rowbit = (uint64_t)r * (uint64_t)F * (uint64_t)bits;
                const int64_t w0 = (int64_t)(rowbit >> 5);
                const uint32_t sh = (uint32_t)(rowbit & 31);
                uint32_t w[5];
#pragma unroll
                for (int k = 0; k < 5; ++k) w[k] = packed[w0 + k < n_words ? w0 + k : n_words - 1];
#pragma unroll
                for (int k = 0; k < 4; ++k) W[q][k] = __builtin_amdgcn_alignbit(w[k + 1], w[k], sh);
                m[q] = leaf_out ? 0.f : margin_src[r];
            }
            uint32_t node[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) node[q] = 0;
            for (int step = 0; step < depth; ++step) {
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    const uint2 c = cnodes[node[q]];
                    const int pos = (int)(c.y >> 12) * bits, wd = pos >> 5;
                    const uint32_t lo = pick4(W[q], wd), hi = wd < 3 ? pick4(W[q], wd + 1) : 0u;
                    const uint32_t s = __builtin_amdgcn_alignbit(hi, lo, (uint32_t)(pos & 31)) & mask;
                    const bool go_left = (s == missing) ? (c.x >> 31) != 0 : (s <= (c.y & 0xfffu));
                    node[q] = (c.x & 0x7fffffffu) + (go_left ? 0u : 1u);
                }
            }
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int64_t r = rb + 256 * q;
                if (r < r1) {
                    if (leaf_out) leaf_out[r] = (int32_t)node[q];
                    else margin[r] = (float)((double)m[q] + eta * lweight[node[q]]);
                    if (COUNT) atomicAdd(&lcount[node[q]], 1u);
                }
            }
        }
        }
    }
    if (COUNT) flush_counts(lcount, max_nodes, node_rows);
}

// Rows of any width: every level's symbol is fetched from the matrix, one dependent access per level (the rows a thread
// walks side by side keep Q of them in flight).  Nodes as above, with bit 30 of x set on a leaf: it keeps its rows
// whatever symbol the matrix holds for them.
// 1M x 28 bytes, depth 6: 37 us with one row at a time and a branch per step, 23 us so.
template <int Q>
__global__ __launch_bounds__(256) void predict_gather_kernel(const char *ws, const DevTree *trees, int n_trees,
                                                             const uint32_t *packed, int bits, uint32_t missing, int64_t n,
                                                             int F, double eta, float *margin, int rows_per_block,
                                                             int max_nodes, int32_t *leaf_out, uint32_t *node_rows,
                                                             const float *margin_src) {
    extern __shared__ uint2 cnodes[];
    double *lweight = (double *)(cnodes + max_nodes);
    uint32_t *lcount = (uint32_t *)(lweight + max_nodes);   // only there when node_rows is given
    if (node_rows)
        for (int i = threadIdx.x; i < max_nodes; i += 256) lcount[i] = 0;
    const uint32_t mask = (1u << bits) - 1u;
    const uint64_t stride_bits = (uint64_t)F * (uint64_t)bits;
    const int64_t n_blocks = (n + rows_per_block - 1) / rows_per_block;
    struct __attribute__((packed, aligned(4))) Pair4 {   // a symbol lies in one word or two; the stream ends in a pad word
        uint32_t lo, hi;
    };
    for (int t = 0; t < n_trees; ++t) {
        const DevTree T = trees[t];
        __syncthreads();
        stage_compact(ws, T, cnodes, lweight, max_nodes);
        __syncthreads();
        for (int i = threadIdx.x; i < T.n_nodes && i < max_nodes; i += 256)   // (a thread's own nodes)
            if (cnodes[i].y == 0xfffu && cnodes[i].x == ((uint32_t)i | 0x80000000u)) cnodes[i].x |= 0x40000000u;
        __syncthreads();
        const int depth = T.pad;
        for (int64_t blk = blockIdx.x; blk < n_blocks; blk += gridDim.x) {
            const int64_t r0 = blk * rows_per_block;
            const int64_t r1 = r0 + rows_per_block < n ? r0 + rows_per_block : n;
            for (int64_t rb = r0 + threadIdx.x; rb < r1; rb += 256 * Q) {
                uint64_t rowbit[Q];
                float m[Q];
                uint32_t node[Q];
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    const int64_t r = rb + 256 * q < r1 ? rb + 256 * q : r1 - 1;   // past the end: the last row again
                    rowbit[q] = (uint64_t)r * stride_bits;
                    m[q] = leaf_out ? 0.f : margin_src[r];
                    node[q] = 0;
                }
                for (int step = 0; step < depth; ++step) {
                    uint2 c[Q];
                    Pair4 w[Q];
                    uint32_t sh[Q];
#pragma unroll
                    for (int q = 0; q < Q; ++q) {
                        c[q] = cnodes[node[q]];
                        const uint64_t bp = rowbit[q] + (uint64_t)((c[q].y >> 12) * (uint32_t)bits);
                        w[q] = *(const Pair4 *)(packed + (bp >> 5));
                        sh[q] = (uint32_t)(bp & 31);
                    }
#pragma unroll
                    for (int q = 0; q < Q; ++q) {
                        const uint32_t sy = __builtin_amdgcn_alignbit(w[q].hi, w[q].lo, sh[q]) & mask;
                        bool stay = (sy == missing) ? (c[q].x >> 31) != 0 : (sy <= (c[q].y & 0xfffu));
                        stay |= (c[q].x & 0x40000000u) != 0;
                        node[q] = (c[q].x & 0x3fffffffu) + (stay ? 0u : 1u);
                    }
                }
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    const int64_t r = rb + 256 * q;
                    if (r < r1) {
                        if (leaf_out) leaf_out[r] = (int32_t)node[q];
                        else margin[r] = (float)((double)m[q] + eta * lweight[node[q]]);
                        if (node_rows) atomicAdd(&lcount[node[q]], 1u);
                    }
                }
            }
        }
    }
    if (node_rows) flush_counts(lcount, max_nodes, node_rows);
}

// Rows wider than the register window, up to kStagedRowBits bits: a wave's 64 consecutive rows are one contiguous
// piece of the bit stream, which the wave fetches linearly into an LDS window of its own; every level's symbol is
// then cut out of LDS instead of being gathered from memory, one dependent access per level.  Nodes as in
// predict_window_kernel.  wave_words: words of a wave's window (64 rows and one word of slack).
constexpr int kStagedRowBits = 1024, kGatheredRowBits = 320;   // (see walk_form)
__global__ __launch_bounds__(256) void predict_staged_kernel(const char *ws, const DevTree *trees, int n_trees,
                                                             const uint32_t *packed, int64_t n_words, int bits,
                                                             uint32_t missing, int64_t n, int F, double eta,
                                                             float *margin, int rows_per_block, int max_nodes,
                                                             int32_t *leaf_out, int wave_words, uint32_t *node_rows,
                                                             const float *margin_src) {
    extern __shared__ uint2 cnodes[];
    double *lweight = (double *)(cnodes + max_nodes);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t *st = (uint32_t *)(lweight + max_nodes) + (size_t)wave * wave_words;
    uint32_t *lcount = (uint32_t *)(lweight + max_nodes) + (size_t)4 * wave_words;   // only there when node_rows is given
    if (node_rows)
        for (int i = threadIdx.x; i < max_nodes; i += 256) lcount[i] = 0;
    const uint32_t mask = (1u << bits) - 1u;
    const uint64_t stride_bits = (uint64_t)F * (uint64_t)bits;
    const int64_t n_blocks = (n + rows_per_block - 1) / rows_per_block;
    for (int t = 0; t < n_trees; ++t) {
        const DevTree T = trees[t];
        __syncthreads();
        stage_compact(ws, T, cnodes, lweight, max_nodes);
        __syncthreads();
        const int depth = T.pad;
        for (int64_t blk = blockIdx.x; blk < n_blocks; blk += gridDim.x) {
        const int64_t r0 = blk * rows_per_block;
        const int64_t r1 = r0 + rows_per_block < n ? r0 + rows_per_block : n;
        for (int64_t rw = r0 + (int64_t)wave * 64; rw < r1; rw += 256) {   // rw: the wave's first row
            const int64_t rend = rw + 64 < r1 ? rw + 64 : r1;
            const uint64_t bit0 = (uint64_t)rw * stride_bits, bit1 = (uint64_t)rend * stride_bits;
            const int64_t word0 = (int64_t)(bit0 >> 5);
            const uint32_t nw = (uint32_t)(((bit1 + 31) >> 5) - (uint64_t)word0) + 1u;   // + the word a last symbol may reach into
            for (uint32_t w = lane; w < nw; w += 64) st[w] = packed[word0 + w < n_words ? word0 + w : n_words - 1];
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const int64_t r = rw + lane;
            if (r < r1) {
                const uint32_t rowbit = (uint32_t)((uint64_t)r * stride_bits - ((uint64_t)word0 << 5));
                uint32_t node = 0;
                for (int step = 0; step < depth; ++step) {
                    const uint2 c = cnodes[node];
                    const uint32_t pos = rowbit + (c.y >> 12) * (uint32_t)bits;
                    const uint32_t lo = st[pos >> 5], hi = st[(pos >> 5) + 1];
                    const uint32_t sy = __builtin_amdgcn_alignbit(hi, lo, pos & 31u) & mask;
                    const bool go_left = (sy == missing) ? (c.x >> 31) != 0 : (sy <= (c.y & 0xfffu));
                    node = (c.x & 0x7fffffffu) + (go_left ? 0u : 1u);
                }
                if (leaf_out) leaf_out[r] = (int32_t)node;
                else margin[r] = (float)((double)margin_src[r] + eta * lweight[node]);
                if (node_rows) atomicAdd(&lcount[node], 1u);
            }
            __builtin_amdgcn_wave_barrier();   // the window is refilled only after every lane has left it
        }
        }
    }
    if (node_rows) flush_counts(lcount, max_nodes, node_rows);
}

// The same walk for 8-bit symbols (rows of at most 16 bytes, any byte alignment): a node is staged
// as a v_perm selector that cuts its feature's byte out of one half of the row, so a step is two
// permutes and a handful of compares.
//   y = 0x0C0C0C00 | (feature & 7)                       (selector: byte -> bits 0..7, zeros above)
//   x = left child id (20 bits) | bin << 20 | (feature >= 8) << 28 | default_left << 29
// A leaf is staged as (own id, bin 255, feature 0, default left): every row stays on it.
// MISS: the matrix has a missing symbol (it is < 256).
// A workgroup takes blocks of rows_per_block rows, blockIdx.x, blockIdx.x + gridDim.x, ...
// node_rows (may be NULL; one tree only): the rows that end in each node are counted, per workgroup in LDS and
// then into node_rows[node * kNodeRowsStride] (one counter per 128-byte line: atomics on one line take turns).
// margin_src: where a row's margin is read from (margin itself, or with one tree another array: out = src + step).
template <bool MISS, int Q>
__global__ __launch_bounds__(256) void predict_b8_kernel(const char *ws, const DevTree *trees, int n_trees,
                                                         const uint32_t *packed, int64_t n_words, uint32_t missing,
                                                         int64_t n, int F, double eta, float *margin,
                                                         int rows_per_block, int max_nodes, int32_t *leaf_out,
                                                         uint32_t *node_rows, const float *margin_src) {
    extern __shared__ uint2 cnodes[];
    double *lweight = (double *)(cnodes + max_nodes);
    uint32_t *lcount = (uint32_t *)(lweight + max_nodes);   // only there when node_rows is given
    if (node_rows)
        for (int i = threadIdx.x; i < max_nodes; i += 256) lcount[i] = 0;
    const int64_t n_blocks = (n + rows_per_block - 1) / rows_per_block;
    for (int t = 0; t < n_trees; ++t) {
        const DevTree T = trees[t];
        __syncthreads();
        for (int i = threadIdx.x; i < T.n_nodes && i < max_nodes; i += 256) {
            const int32_t f = ((const int32_t *)(ws + T.feature))[i];
            uint2 c;
            if (f < 0) {
                c.x = (uint32_t)i | (255u << 20) | (1u << 29);
                c.y = 0x0C0C0C00u;
            } else {
                const int32_t bin = ((const int32_t *)(ws + T.bin))[i];   // a bin >= 255 admits every symbol
                c.x = (uint32_t)((const int32_t *)(ws + T.left))[i] |
                      ((uint32_t)(bin < 255 ? bin : 255) << 20) | ((uint32_t)((f >> 3) & 1) << 28) |
                      (((const int32_t *)(ws + T.default_left))[i] ? (1u << 29) : 0u);
                c.y = 0x0C0C0C00u | (uint32_t)(f & 7);
            }
            cnodes[i] = c;
            lweight[i] = ((const double *)(ws + T.weight))[i];
        }
        __syncthreads();
        const int depth = T.pad;
        for (int64_t blk = blockIdx.x; blk < n_blocks; blk += gridDim.x) {
        const int64_t r0 = blk * rows_per_block;
        const int64_t r1 = r0 + rows_per_block < n ? r0 + rows_per_block : n;
        for (int64_t rb = r0 + threadIdx.x; rb < r1; rb += 256 * Q) {
            uint32_t W[Q][4];
            float m[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int64_t r = rb + 256 * q < r1 ? rb + 256 * q : r1 - 1;   // past the end: the last row again
                const uint64_t byte0 = (uint64_t)r * (uint64_t)F;
                const int64_t w0 = (int64_t)(byte0 >> 2);
                const uint32_t a = (uint32_t)(byte0 & 3);
                uint32_t w[5];
                if (w0 + 4 < n_words) {   // (all but the last rows of the matrix) one 16-byte load and one word
                    load_words(w, packed + w0);
                } else {
#pragma unroll
                    for (int k = 0; k < 5; ++k) w[k] = packed[w0 + k < n_words ? w0 + k : n_words - 1];
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) W[q][k] = __builtin_amdgcn_alignbyte(w[k + 1], w[k], a);
                m[q] = leaf_out ? 0.f : margin_src[r];
            }
            uint32_t node[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) node[q] = 0;
            for (int step = 0; step < depth; ++step) {
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    const uint2 c = cnodes[node[q]];
                    const uint32_t lo = __builtin_amdgcn_perm(W[q][1], W[q][0], c.y);
                    const uint32_t hi = __builtin_amdgcn_perm(W[q][3], W[q][2], c.y);
                    const uint32_t sy = (c.x & (1u << 28)) ? hi : lo;
                    bool go_left = sy <= ((c.x >> 20) & 0xffu);
                    if (MISS) go_left = (sy == missing) ? (c.x & (1u << 29)) != 0 : go_left;
                    node[q] = (c.x & 0xfffffu) + (go_left ? 0u : 1u);
                }
            }
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int64_t r = rb + 256 * q;
                if (r < r1) {
                    if (leaf_out) leaf_out[r] = (int32_t)node[q];
                    else margin[r] = (float)((double)m[q] + eta * lweight[node[q]]);
                    if (node_rows) atomicAdd(&lcount[node[q]], 1u);
                }
            }
        }
        }
    }
    if (node_rows) flush_counts(lcount, max_nodes, node_rows);
}

// Final row order and leaf ids: every position of [0, n) lies in exactly one
// leaf segment; segments are sorted by seg_begin.
// Each workgroup takes a chunk of positions; the search starts from the segment of the chunk's
// first position (found once) and only walks forward.
constexpr int kGatherChunk = 256 * 16;
__global__ __launch_bounds__(256) void leaf_gather_kernel(const uint32_t *buf0, const uint32_t *buf1,
                                                          const LeafSeg *segs, int n_segs, int64_t n,
                                                          uint32_t *row_idx_out, int32_t *leaf_of_row) {
    const int64_t p0 = (int64_t)blockIdx.x * kGatherChunk;
    __shared__ int first_seg;
    if (threadIdx.x == 0) {
        int lo = 0, hi = n_segs;   // last segment with seg_begin <= p0
        while (hi - lo > 1) {
            int mid = (lo + hi) >> 1;
            if ((int64_t)segs[mid].seg_begin <= p0) lo = mid; else hi = mid;
        }
        first_seg = lo;
    }
    __syncthreads();
    int cur = first_seg;
    for (int k = 0; k < kGatherChunk / 256; ++k) {
        const int64_t p = p0 + (int64_t)k * 256 + threadIdx.x;
        if (p >= n) break;
        while (cur + 1 < n_segs && (int64_t)segs[cur + 1].seg_begin <= p) ++cur;
        const LeafSeg s = segs[cur];
        const uint32_t r = s.buf == 2 ? (uint32_t)p : (s.buf ? buf1 : buf0)[p];
        row_idx_out[p] = r;
        if (leaf_of_row && (int64_t)r < n) leaf_of_row[r] = (int32_t)s.node;
    }
}

}  // namespace

hipError_t gbt_launch_fill_u64(hipStream_t s, uint64_t *p, uint64_t v, int64_t count) {
    if (count <= 0) return hipSuccess;
    fill_u64_kernel<<<grid_for(count, kBlock * 4, 4096), kBlock, 0, s>>>(p, v, count);
    return hipGetLastError();
}
hipError_t gbt_launch_iota_u32(hipStream_t s, uint32_t *p, int64_t count) {
    if (count <= 0) return hipSuccess;
    iota_u32_kernel<<<grid_for(count, kBlock * 4, 8192), kBlock, 0, s>>>(p, count);
    return hipGetLastError();
}
// A plain streaming read of `n16` 16-byte pieces: what HBM delivers to a kernel that only reads (the yardstick
// beside the histogram kernels' achieved bandwidth).  sink is written only if the xor of everything read
// equals a magic word, which keeps the loads alive.
namespace {
__global__ __launch_bounds__(kBlock) void stream_read_kernel(const uint4 *__restrict__ p, int64_t n16, uint32_t *sink) {
    uint32_t acc = 0;
    const int64_t chunk = (int64_t)kStreamBatch * kBlock, n_whole = n16 / chunk;
    for (int64_t c = blockIdx.x; c < n_whole; c += gridDim.x) {
        uint4 v[kStreamBatch];
#pragma unroll
        for (int k = 0; k < kStreamBatch; ++k) v[k] = p[c * chunk + k * kBlock + threadIdx.x];
#pragma unroll
        for (int k = 0; k < kStreamBatch; ++k) acc ^= v[k].x ^ v[k].y ^ v[k].z ^ v[k].w;
    }
    for (int64_t i = n_whole * chunk + (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n16; i += (int64_t)gridDim.x * kBlock) {
        const uint4 v = p[i];
        acc ^= v.x ^ v.y ^ v.z ^ v.w;
    }
    if (acc == 0x9E3779B9u) *sink = acc;
}
}  // namespace
hipError_t gbt_launch_stream_read(hipStream_t s, const void *buf, int64_t bytes, uint32_t *sink) {
    const int64_t n16 = bytes / 16;
    if (n16 <= 0) return hipSuccess;
    stream_read_kernel<<<grid_for(n16, kBlock * kStreamBatch, 4096), kBlock, 0, s>>>((const uint4 *)buf, n16, sink);
    return hipGetLastError();
}

int gbt_red_slots_max() { return kRedGroups; }
hipError_t gbt_launch_absmax(hipStream_t s, const float *gpair, int64_t n, void *slots, int *n_slots) {
    *n_slots = 0;
    if (n <= 0) return hipSuccess;
    const int head = (int)(((uintptr_t)gpair >> 3) & 1u);   // pairs before the first 16-byte boundary
    *n_slots = red_grid(n, 2 * kStreamBatch);
    absmax_kernel<<<*n_slots, kRedBlock, 0, s>>>((const float2 *)gpair + head, n - head, head, (uint4 *)slots);
    return hipGetLastError();
}
hipError_t gbt_launch_to_fixed(hipStream_t s, const float *gpair, int64_t n, double sg, double sh,
                               int32_t *gq, void *slots, int *n_slots) {
    if (n_slots) *n_slots = 0;
    if (n <= 0) return hipSuccess;
    const int head = (int)(((uintptr_t)gpair >> 3) & 1u);
    const bool pairs = head != (int)(((uintptr_t)gq >> 3) & 1u);
    const int grid = red_grid(n, pairs ? 4 : 2 * kStreamBatch);
    if (n_slots) *n_slots = grid;
    if (pairs)
        to_fixed_pairs_kernel<<<grid, kRedBlock, 0, s>>>((const float2 *)gpair, n, sg, sh, (int2 *)gq, (longlong2 *)slots);
    else
        to_fixed_kernel<<<grid, kRedBlock, 0, s>>>((const float2 *)gpair + head, n - head, head, sg, sh, (int2 *)gq + head,
                                                   (longlong2 *)slots);
    return hipGetLastError();
}
hipError_t gbt_launch_sum_gq(hipStream_t s, const int32_t *gq, const uint32_t *row_idx, int64_t n_rows, void *slots, int *n_slots) {
    *n_slots = 0;
    if (n_rows <= 0) return hipSuccess;
    *n_slots = red_grid(n_rows, 4);
    sum_gq_kernel<<<*n_slots, kRedBlock, 0, s>>>((const int2 *)gq, row_idx, n_rows, (longlong2 *)slots);
    return hipGetLastError();
}
hipError_t gbt_launch_gradients(hipStream_t s, int objective, const float *margin, const float *label,
                                int64_t n, float *gpair, void *bounds, int *n_slots) {
    if (n_slots) *n_slots = 0;
    if (n <= 0) return hipSuccess;
    const int vec = ((((uintptr_t)margin | (uintptr_t)label | (uintptr_t)gpair) & 15u) == 0) ? 1 : 0;
    const int grid = bounds ? red_grid(n, 4) : grid_for(n, kBlock * 4, 8192);
    if (bounds) *n_slots = grid;
    gradients_kernel<<<grid, bounds ? kRedBlock : kBlock, 0, s>>>(objective, margin, label, n, (float2 *)gpair, vec,
                                                                 (uint4 *)bounds,
                                                                 (size_t)n * sizeof(float2) > ((size_t)192 << 20) ? 1 : 0);
    return hipGetLastError();
}
hipError_t gbt_launch_subtract_one(hipStream_t s, const int64_t *parent, const int64_t *child,
                                   int64_t *out, int64_t count) {
    if (count <= 0) return hipSuccess;
    subtract_one_kernel<<<grid_for(count, kBlock * 4, 4096), kBlock, 0, s>>>(parent, child, out, count);
    return hipGetLastError();
}
hipError_t gbt_launch_export(hipStream_t s, const int64_t *hist, int64_t count, double inv_sg,
                             double inv_sh, double *out) {
    if (count <= 0) return hipSuccess;
    export_kernel<<<grid_for(count, kBlock * 4, 4096), kBlock, 0, s>>>(hist, count, inv_sg, inv_sh, out);
    return hipGetLastError();
}
hipError_t gbt_launch_compress(hipStream_t s, const uint16_t *sym, int64_t n_elems, int bits,
                               uint32_t *packed, int64_t n_words) {
    if (n_words <= 0) return hipSuccess;
    compress_kernel<<<grid_for(n_words, kBlock * 4, 16384), kBlock, 0, s>>>(sym, n_elems, bits, packed,
                                                                            n_words);
    return hipGetLastError();
}
// ---------------------------------------------------------------------------
// Sec. 2.4 for many trees on raw floats: the rows are read from HBM once.  A workgroup stages a tile of R rows in LDS,
// then takes the trees in groups that fit LDS beside it (8-byte nodes, converted on the host; the leaf weights stay in
// global memory, one gather per walk against one node per step): one row per thread, four trees of a group walked side
// by side (independent chains hide the LDS latency), every walk a fixed number of steps (the tree's depth) because a
// leaf is staged as a node that leads to itself.  The margin stays in a register and is rounded to fp32 after every
// tree, in tree order, like the one-tree kernels.
// Bound: LDS reads (a node and a value per step) and the instructions around them, not HBM.  Two things follow.
//  - The tile is feature-major, word (feature, row) at feature * R + row: whatever features the lanes of a wave ask
//    for, lane l always reads bank l mod 64, so a value read never conflicts (row-major, odd stride: about five ways).
//  - Values are staged as integers in the floats' order with NaN as the largest one, and a node carries its threshold
//    the same way: "right" is (value + a >= threshold), where a = 1 on a node whose missing values go left (NaN wraps
//    to the smallest integer): one add and one compare instead of two compares and the mask arithmetic between them.
//    A tile without a NaN needs neither the add nor the bit that it adds.
//  - A node names its left child by the byte offset that the next read takes, so that a step is six or eight vector
//    instructions; ids and a base to add per tree made it eleven, and vector issue, not LDS, was what took the time.
//  - What waits for memory is asked for ahead: the next group's nodes while this one is walked, four leaves' weights behind
//    the next four walks.
// 1M x 28 rows, 100 trees of depth 6 (6*10^8 steps): 0.44 ms row-major, 0.262 feature-major, 0.238 with fewer instructions
// (82 instead of 107 million vector instructions, on 80 % of the cycles before) and the weights behind, 0.208 with the nodes ahead.
// ---------------------------------------------------------------------------
namespace {
constexpr int kBatchTrees = 4;   // 2, 3, 6 and 8 take the same time within 3 %

struct __attribute__((packed, aligned(4))) Float4a4 {
    float v[4];
};

__device__ __forceinline__ int float_key(float x) {
    const int b = __float_as_int(x + 0.0f);   // -0 and +0 compare equal as floats
    return x != x ? 0x7fffffff : b ^ ((b >> 31) & 0x7fffffff);
}

template <int R>
__global__ __launch_bounds__(R) void predict_raw_batched_kernel(
    const gbt_batch_node *__restrict__ nodes_g, const double *__restrict__ wts_g,
    const int32_t *__restrict__ tree_off, const int32_t *__restrict__ tree_depth,
    const int32_t *__restrict__ group_end, int n_groups, int cap_nodes, const float *__restrict__ X, int64_t n, int F,
    float *__restrict__ margin) {
    extern __shared__ char smem[];   // the group's nodes, then the tile
    gbt_batch_node *nd = (gbt_batch_node *)smem;
    int *xs = (int *)(smem + (size_t)cap_nodes * 8);
    bool nan = false;
    const int64_t r0 = (int64_t)blockIdx.x * R;
    const int rows = n - r0 < R ? (int)(n - r0) : R;
    // A group's nodes are asked for while the trees of the group before are walked, the first group's while the tile is fetched
    // (kAhead per thread; of a larger group the rest is fetched when it is needed).
    constexpr int kAhead = 1536 / R;
    gbt_batch_node ahead[kAhead];
    auto fetch = [&](int n0, int n1, int first, gbt_batch_node (&a)[kAhead]) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            const int i = first + (int)threadIdx.x + k * R;
            a[k] = nodes_g[n0 + (i < n1 - n0 ? i : n1 - n0 - 1)];
        }
    };
    // (a group's first tree stands at its second place)
    int t_begin = 0, n0 = tree_off[0] - 1, n1 = tree_off[group_end[0]] - 1;
    fetch(n0, n1, 0, ahead);
    // (the vote on missing values goes through the nodes' place: a word of static LDS would cost a compute unit its fourth workgroup)
    int *vote = (int *)smem;
    if (threadIdx.x == 0) *vote = 0;
    __syncthreads();
    {   // the tile is one contiguous piece of X, taken in chunks of four features of a row: chunk tid + R k by thread
        // tid in step k, four chunks in flight per thread; (row, chunk) advance without divisions
        const int C = (F + 3) >> 2, total = rows * C;
        const float *src = X + r0 * F;
        const int dq = R / C, dr = R % C;
        int row = (int)threadIdx.x / C, c = (int)threadIdx.x % C;
        for (int i0 = threadIdx.x; i0 < total; i0 += 4 * R) {
            float v[4][4];
            int at[4], nf[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const bool on = i0 + k * R < total;
                const int f = 4 * c;
                nf[k] = on ? (F - f < 4 ? F - f : 4) : 0;
                at[k] = f * R + row;
                const float *p = src + (int64_t)row * F + f;
                if (nf[k] == 4) {
                    const Float4a4 q = *(const Float4a4 *)p;
#pragma unroll
                    for (int j = 0; j < 4; ++j) v[k][j] = q.v[j];
                } else {
#pragma unroll
                    for (int j = 0; j < 3; ++j) v[k][j] = j < nf[k] ? p[j] : 0.0f;
                    v[k][3] = 0.0f;
                }
                row += dq;
                c += dr;
                if (c >= C) {
                    c -= C;
                    ++row;
                }
            }
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (j < nf[k]) {
                        nan |= v[k][j] != v[k][j];
                        xs[at[k] + j * R] = float_key(v[k][j]);
                    }
        }
    }
    const bool live = (int)threadIdx.x < rows;
    float m = live ? margin[r0 + threadIdx.x] : 0.0f;
    typedef const unsigned long long __attribute__((address_space(3))) lds_u64;
    typedef const int __attribute__((address_space(3))) lds_i32;
    // LDS addresses as numbers: nothing is added to an offset before it is read
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_i32 *)smem;
    const uint32_t xrow = lds0 + (uint32_t)cap_nodes * 8u + 4u * (live ? threadIdx.x : 0u);
    if (nan) *vote = 1;
    __syncthreads();
    const bool any_nan = *vote != 0;
    // the weights of four trees' leaves are added behind the next four trees' walks: their gather takes as long as a walk
    double w[kBatchTrees];
    int n_w = 0;
    auto add_weights = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < kBatchTrees; ++k)
            if (k < n_w) m = (float)((double)m + w[k]);
    };
    auto place = [&](int count, int first, const gbt_batch_node (&a)[kAhead]) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            const int i = first + (int)threadIdx.x + k * R;
            gbt_batch_node q = a[k];
            if (!any_nan) q.thr -= (int)(q.meta & 1u);   // then value >= thr, nothing added on either side
            q.meta += lds0;   // (a multiple of 16, and small: the launch has no other LDS)
            if (i < count) nd[i] = q;
        }
    };
    for (int g = 0; g < n_groups; ++g) {
        const int t_end = group_end[g];
        __syncthreads();   // the row tile is complete; the previous group's walks are done
        place(n1 - n0, 0, ahead);
        for (int first = kAhead * R; first < n1 - n0; first += kAhead * R) {
            fetch(n0, n1, first, ahead);
            place(n1 - n0, first, ahead);
        }
        __syncthreads();
        const int g0 = n0;   // this group's first node
        const double *wts = wts_g + g0;
        if (g + 1 < n_groups) {
            n0 = n1;
            n1 = tree_off[group_end[g + 1]] - 1;
            fetch(n0, n1, 0, ahead);
        }
        for (int t = t_begin; t < t_end; t += kBatchTrees) {
            uint32_t at[kBatchTrees];   // LDS address of the node a walk has reached
            int depth = 0;
#pragma unroll
            for (int k = 0; k < kBatchTrees; ++k) {
                const int tk = t + k < t_end ? t + k : t_end - 1;   // past the group: the last tree again, unused
                at[k] = lds0 + 8u * (uint32_t)(tree_off[tk] - g0);
                const int dk = tree_depth[tk];
                depth = dk > depth ? dk : depth;
            }
            auto step = [&](bool with_nan) __attribute__((always_inline)) {
                // the four walks' LDS reads are issued together: first the nodes, then the values
                uint2 q[kBatchTrees];   // x: threshold, y: meta
                int x[kBatchTrees];
#pragma unroll
                for (int k = 0; k < kBatchTrees; ++k) {
                    const unsigned long long v = *(const lds_u64 *)(uintptr_t)at[k];
                    q[k] = make_uint2((uint32_t)v, (uint32_t)(v >> 32));
                }
#pragma unroll
                for (int k = 0; k < kBatchTrees; ++k) {
                    uint32_t f = q[k].y >> 18;
                    asm("" : "+v"(f));   // (a shift and a shift with add; the compiler makes shift, mask, add of the two shifts)
                    x[k] = *(const lds_i32 *)(uintptr_t)(xrow + f * (uint32_t)(R * 4));
                }
#pragma unroll
                for (int k = 0; k < kBatchTrees; ++k) {
                    const int v = with_nan ? (int)((uint32_t)x[k] + (q[k].y & 1u)) : x[k];
                    at[k] = (q[k].y & 0x3fff8u) | (v >= (int)q[k].x ? 8u : 0u);
                }
            };
            if (any_nan)
                for (int d = 0; d < depth; ++d) step(true);
            else
                for (int d = 0; d < depth; ++d) step(false);
            add_weights();
#pragma unroll
            for (int k = 0; k < kBatchTrees; ++k) w[k] = *(const double *)((const char *)wts + (at[k] - lds0));
            n_w = t_end - t;
        }
        t_begin = t_end;
    }
    add_weights();
    if (live) margin[r0 + threadIdx.x] = m;
}

// Rows of a tile: 256 while two workgroups of a compute unit find room for it beside their nodes, then fewer.  1M rows and 100
// trees of depth 6, the call in us with 64, 128 and 256 rows: 28 columns 612, 472, 403; 64 columns 848, 688, 570; 95 columns
// 1092, 1011, 958; 128 columns 1434, 1148, does not fit; 200 columns 2214, 1975, does not fit (the lines at 64 and 128 columns
// are not the best ones: at 65 columns 128 rows take 730 and 256 take 588).
inline int batch_rows(int F) { return F <= 64 ? 256 : F <= 128 ? 128 : 64; }

template <int R>
hipError_t launch_batched(hipStream_t s, const gbt_batch_node *nodes, const double *wts, const int32_t *tree_off,
                          const int32_t *tree_depth, const int32_t *group_end, int n_groups, int cap_nodes, size_t lds, const float *X,
                          int64_t n, int F, float *margin) {
    GbtLdsGuard lds_guard(lds);
    if (lds_guard.needed) {
        hipError_t e = hipFuncSetAttribute((const void *)predict_raw_batched_kernel<R>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    predict_raw_batched_kernel<R><<<(unsigned)((n + R - 1) / R), R, lds, s>>>(nodes, wts, tree_off, tree_depth, group_end,
                                                                            n_groups, cap_nodes, X, n, F, margin);
    return hipGetLastError();
}
}  // namespace

int gbt_predict_batch_rows(int F) { return batch_rows(F); }
size_t gbt_predict_batch_tile_bytes(int F) { return (size_t)batch_rows(F) * F * 4; }

hipError_t gbt_launch_predict_raw_batched(hipStream_t s, const gbt_batch_node *nodes, const double *wts,
                                          const int32_t *tree_off, const int32_t *tree_depth,
                                          const int32_t *group_end, int n_groups, int cap_nodes, const float *X,
                                          int64_t n, int F, float *margin) {
    if (n <= 0 || n_groups <= 0) return hipSuccess;
    const size_t lds = gbt_predict_batch_tile_bytes(F) + (size_t)cap_nodes * 8;
    switch (batch_rows(F)) {
        case 256: return launch_batched<256>(s, nodes, wts, tree_off, tree_depth, group_end, n_groups, cap_nodes, lds, X, n, F, margin);
        case 128: return launch_batched<128>(s, nodes, wts, tree_off, tree_depth, group_end, n_groups, cap_nodes, lds, X, n, F, margin);
        default: return launch_batched<64>(s, nodes, wts, tree_off, tree_depth, group_end, n_groups, cap_nodes, lds, X, n, F, margin);
    }
}

// LDS of a walk over packed symbols with compact nodes: 16 bytes per node, a row counter per node if it counts, the rows'
// windows of the staged form.
namespace {
enum { WALK_B8, WALK_WINDOW, WALK_STAGED, WALK_GATHER };
int staged_wave_words(int bits, int F) { return (int)((64 * (int64_t)F * bits + 31) / 32) + 2; }
// Rows staged through LDS, a wave's 64 at a time, where a row is wider than 40 bytes: a narrower one lies in a cache line or
// two that the gathers of its levels all hit.  us per call, gathered and staged, one tree of depth 3, 6 and 9, 10M rows: of 28
// bytes 99 and 188, 133 and 196, 181 and 219; of 33 116 and 211, 164 and 219, 224 and 243; of 40 138 and 243, 205 and 251, 279
// and 275; of 57 202 and 317, 355 and 326, 514 and 355; of 112 424 and 554, 826 and 560, 1230 and 979 (below depth 5 the
// gathers are the shorter way for wider rows as well; 200,000 rows take the same time either way).
int walk_form(int bits, int F, int max_nodes, bool counts, size_t *lds) {
    const int64_t row_bits = (int64_t)F * bits;
    *lds = (size_t)max_nodes * (16 + (counts ? 4 : 0));
    if (row_bits <= 128) return bits == 8 && F <= 16 && max_nodes <= (1 << 20) ? WALK_B8 : WALK_WINDOW;   // (node ids of 20 bits)
    if (row_bits > kGatheredRowBits && row_bits <= kStagedRowBits) {
        const size_t staged = *lds + (size_t)4 * staged_wave_words(bits, F) * 4;
        if (staged <= kWalkLds) {
            *lds = staged;
            return WALK_STAGED;
        }
    }
    return WALK_GATHER;
}
// Trees that a walk over packed symbols keeps in LDS.  Every workgroup stages the whole tree, and past 80 KB a compute unit
// holds one workgroup: larger trees are read from the caches, but where rows are many and their own reads few.  us per call,
// from LDS and from the caches, 3071, 4095 and 4801 nodes: 100,000 rows of 28 bytes 47 and 43, 52 and 44, 57 and 47; 1M of 14 symbols of 9
// bits 78 and 60, 88 and 61, 96 and 65; 1M of 13 bytes 60 and 61, 67 and 62, 74 and 66; 4M of 13 bytes 106 and 140, 143 and 143, 157 and 151;
// 10M of 13 bytes 169 and 296, 212 and 297, 234 and 314; of 28 212 and 330, 246 and 332, 270 and 347.
constexpr int kWalkNodes = 3072;
constexpr int64_t kWalkManyRows = 6 << 20;
bool walk_from_lds(int bits, int F, int max_nodes, int64_t n) {
    if (max_nodes <= kWalkNodes) return true;
    const int64_t row_bits = (int64_t)F * bits;
    const bool few_reads = row_bits <= 128 ? bits == 8 && F <= 16 : row_bits <= kGatheredRowBits || row_bits > kStagedRowBits;
    return n >= kWalkManyRows && few_reads && (size_t)max_nodes * 20 <= kWalkLds;
}
// Rows that a thread gathers for side by side, and rows of a block.  The more rows a compute unit walks at once, the more often a
// row's lines leave the caches between two levels: rows past 32 bytes are walked one by one, wide ones in longer blocks from 768k
// rows on; past 3M rows nothing is kept between levels, and short blocks that follow each other closely share DRAM pages.  us per
// call, depth 8, (4 rows, blocks of 1024), (1, 1024), (1, 4096) and (2, 256): 1M x 40 bytes 51, 46, 64, 52; 500,000 x 132 92, 52,
// 67, 63; 1M x 132 147, 77, 70, 83; 1M x 300 166, 129, 115, 128; 2M x 132 262, 228, 104, 124; 2M x 300 301, 281, 191, 217; 5M x 132
// 611, 479, 353, 261; 5M x 200 682, 591, 528, 395 (of depth 10, 2047 nodes, 785, 560, 694, 648); 5M x 40 121, 107, 95, 114 and 95
// with (2, 4096); 1M x 28 44, 44, 63, 53.
// Past 1024 nodes short blocks would mostly stage nodes: there LDS for two workgroups of a compute unit bounds the rows at once
// (6M x 180, 2047 nodes: 445 so, 603 with (1, 1024), 991 with (4, 4096)).
void gathered_rows(int64_t row_bits, int64_t n, int max_nodes, int *side_by_side, int *rows_per_block, size_t *lds) {
    if (row_bits <= 256) return;
    *side_by_side = 1;
    if (row_bits <= kStagedRowBits) {
        if (*rows_per_block == 4096) *side_by_side = 2;
    } else if (n <= (int64_t)3 << 20) {
        *rows_per_block = n <= (int64_t)704 * 1024 ? 1024 : 4096;
    } else if (max_nodes <= 1024) {
        *side_by_side = 2;
        *rows_per_block = 256;
    } else {
        *rows_per_block = 4096;
        *lds = std::max(*lds, (size_t)64 * 1024);
    }
}
template <typename K, typename... A>
hipError_t launch_walk(K kernel, int64_t grid, size_t lds, hipStream_t s, A... args) {
    GbtLdsGuard lds_guard(lds);
    if (lds_guard.needed) {
        hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    kernel<<<(unsigned)grid, 256, lds, s>>>(args...);
    return hipGetLastError();
}
}  // namespace

// Can the walk also count the rows per node, and read the margins from another array?  The forms that keep the tree in LDS do.
bool gbt_predict_counts_ok(bool packed, int bits, int F, int64_t n, int max_nodes, bool compact_ok) {
    return packed && compact_ok && walk_from_lds(bits, F, max_nodes, n);
}

hipError_t gbt_launch_predict(hipStream_t s, const char *ws, const DevTree *trees, int n_trees,
                              const uint32_t *packed, int bits, uint32_t missing, const float *X,
                              int64_t n, int F, double eta, float *margin, int32_t *leaf_out, int max_nodes,
                              bool compact_ok, uint32_t *node_rows, const float *margin_src) {
    if (n <= 0) return hipSuccess;
    if (margin_src == margin) margin_src = nullptr;
    if ((node_rows || margin_src) && !(n_trees == 1 && gbt_predict_counts_ok(packed != nullptr, bits, F, n, max_nodes, compact_ok)))
        return hipErrorInvalidValue;   // (the caller asks gbt_predict_counts_ok first)
    size_t lds = 0;
    const int form = walk_form(bits, F, max_nodes, node_rows != nullptr, &lds);
    if (packed && compact_ok && walk_from_lds(bits, F, max_nodes, n) && lds <= kWalkLds) {
        // A workgroup stages the tree and walks a block of rows.  Where blocks of 4096 rows would leave compute units
        // without a workgroup they are shorter, down to one row per thread (1M x 28 bytes: 37 us with 245 workgroups, 23 us
        // with 977 and four rows per thread side by side; 50,000 x 22 bytes 36 -> 7 us).
        const bool few = n <= (int64_t)256 * 1024;
        int rows_per_block = few ? 256 : n < (int64_t)4096 * 1024 ? 1024 : 4096;
        int side_by_side = few ? 1 : kPredRows;   // rows of a thread
        if (form == WALK_GATHER && !few) gathered_rows((int64_t)F * bits, n, max_nodes, &side_by_side, &rows_per_block, &lds);
        int64_t grid = (n + rows_per_block - 1) / rows_per_block;
        // counting: few enough workgroups that their counts meet rarely in HBM, each taking many blocks
        if (node_rows && grid > 2048) grid = 2048;
        const int64_t n_words = (n * (int64_t)F * bits + 31) / 32 + 1;
        const float *src = margin_src ? margin_src : margin;
        switch (form) {
            case WALK_B8: {
                const bool miss = missing < 256u;
                auto k = miss ? (few ? predict_b8_kernel<true, 1> : predict_b8_kernel<true, kPredRows>)
                              : (few ? predict_b8_kernel<false, 1> : predict_b8_kernel<false, kPredRows>);
                return launch_walk(k, grid, lds, s, ws, trees, n_trees, packed, n_words, missing, n, F, eta, margin,
                                   rows_per_block, max_nodes, leaf_out, node_rows, src);
            }
            case WALK_WINDOW: {
                auto k = node_rows ? (few ? predict_window_kernel<1, true> : predict_window_kernel<kPredRows, true>)
                                   : (few ? predict_window_kernel<1, false> : predict_window_kernel<kPredRows, false>);
                return launch_walk(k, grid, lds, s, ws, trees, n_trees, packed, n_words, bits, missing, n, F, eta, margin,
                                   rows_per_block, max_nodes, leaf_out, node_rows, src);
            }
            case WALK_STAGED:
                return launch_walk(predict_staged_kernel, grid, lds, s, ws, trees, n_trees, packed, n_words, bits, missing, n, F,
                                   eta, margin, rows_per_block, max_nodes, leaf_out, staged_wave_words(bits, F), node_rows, src);
            default: {
                auto k = side_by_side == 1 ? predict_gather_kernel<1> : side_by_side == 2 ? predict_gather_kernel<2> : predict_gather_kernel<kPredRows>;
                return launch_walk(k, grid, lds, s, ws, trees, n_trees, packed, bits, missing, n, F, eta, margin,
                                   rows_per_block, max_nodes, leaf_out, node_rows, src);
            }
        }
    }
    const size_t lds_full = (size_t)max_nodes * sizeof(LdsNode);
    if (lds_full <= kWalkLds) {
        // Blocks as above, but raw floats past 128 MB are read in blocks of 4096 rows from 768k rows on (1536k of 96 and more columns): the more rows a compute unit
        // walks at once, the more often a row's line is fetched again.  us per call with 1024 and 4096, depth 6: 1M x 28 53 and 57, 2M x
        // 28 155 and 78, 3.9M x 28 251 and 151, 500,000 x 64 49 and 65, 1M x 64 102 and 72, 1M x 100 112 and 110, 2M x 100 222 and 181,
        // 500,000 x 200 65 and 96, 2M x 200 235 and 214, two trees of depth 3 over 1M x 216 133 and 152, 3.9M x 4 54 and 65.
        const bool wide = X && n > (int64_t)(F < 96 ? 768 : 1536) * 1024 && n * (int64_t)F * 4 > (int64_t)128 << 20;
        const int rows_per_block = n <= (int64_t)256 * 1024 ? 256 : n < (int64_t)4096 * 1024 && !wide ? 1024 : 4096;
        return launch_walk(predict_lds_kernel, (n + rows_per_block - 1) / rows_per_block, lds_full, s, ws, trees, n_trees,
                           packed, bits, missing, X, n, F, eta, margin, rows_per_block, leaf_out);
    }
    predict_kernel<<<grid_for(n, kBlock, 1 << 16), kBlock, 0, s>>>(ws, trees, n_trees, packed, bits,
                                                                    missing, X, n, F, eta, margin, leaf_out);
    return hipGetLastError();
}
hipError_t gbt_launch_leaf_gather(hipStream_t s, const uint32_t *buf0, const uint32_t *buf1,
                                  const LeafSeg *segs, int n_segs, int64_t n, uint32_t *row_idx_out,
                                  int32_t *leaf_of_row) {
    if (n <= 0 || n_segs <= 0) return hipSuccess;
    const int64_t grid = (n + kGatherChunk - 1) / kGatherChunk;
    leaf_gather_kernel<<<(unsigned)grid, 256, 0, s>>>(buf0, buf1, segs, n_segs, n, row_idx_out, leaf_of_row);
    return hipGetLastError();
}
