// Feature quantile generation (Sec. 2.1) on the GPU: exact per-feature order statistics, then cuts, then binning.
//
//   1. keys: every feature's values become one contiguous segment of uint32 keys in the floats' order (dense input: an
//      LDS-tiled transpose, a missing value becomes the largest key; CSR input: counted, offset and scattered by
//      column);
//   2. order statistics and cuts by selection (kernels_select.hip).  With more than 1024 bins, for many short columns
//      (gbt_select_ok) and for columns whose values lie too close together, by a segmented LSD radix sort (here): four
//      8-bit passes, each a per-tile digit histogram, offsets from the tile histograms and a stable scatter (ranks from
//      wave ballots, tiles and waves in order), then one wave per feature walks the sorted segment;
//   3. bin: symbol = number of cuts <= x.  Packed and dense, all columns by selection: column by column with the selection's
//      cells, then packed from the columns (kernels_select.hip).  Otherwise from the values: by bisection over the feature's
//      cuts, or for packed CSR rows in two levels with the upper one in LDS.
#include "gbt_internal.h"
#include "quantise_common.h"

#include <string.h>

#include <initializer_list>
#include <vector>

namespace {

constexpr int kSortBlock = 256;
constexpr int kKeysPerWave = kSortTile / (kSortBlock / 64);   // 1024
constexpr int kRounds = kKeysPerWave / 64;            // 16

// ---- 1a. dense input: transpose into per-feature key segments -------------
// Bound: HBM (each value read once, each key written once).  A thread issues its loads together, past the edge from the
// last element (read, not stored): one load per thread and turn left too little in flight to cover the memory's latency.
// The whole call (cuts, binning, packing) before and after: 115M x 13 8.54 -> 8.20 ms, 3M x 64 2.07 -> 1.63 ms, 500K x 801
// 3.68 -> 3.57 ms; 50K x 5 the same within its noise.
constexpr int kTrRows = 64, kTrCols = 64;
__global__ __launch_bounds__(256) void dense_keys_kernel(const float *__restrict__ X, int64_t n, int F,
                                                         uint32_t *__restrict__ keys) {
    __shared__ uint32_t tile[kTrRows][kTrCols + 1];
    const int64_t r0 = (int64_t)blockIdx.x * kTrRows;
    const int f0 = blockIdx.y * kTrCols;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;   // 64 x 4
    const float *src = X + r0 * F + (f0 + tx < F ? f0 + tx : F - 1);
    const int last = n - r0 < kTrRows ? (int)(n - r0) - 1 : kTrRows - 1;
    float x[kTrRows / 4];
#pragma unroll
    for (int k = 0; k < kTrRows / 4; ++k) {
        const int i = ty + 4 * k;
        x[k] = src[(int64_t)(i < last ? i : last) * F];
    }
#pragma unroll
    for (int k = 0; k < kTrRows / 4; ++k) tile[ty + 4 * k][tx] = float_key(x[k]);
    __syncthreads();
    for (int j = ty; j < kTrCols; j += 4) {
        const int f = f0 + j;
        const int64_t r = r0 + tx;
        if (f < F && r < n) keys[(int64_t)f * n + r] = tile[tx][j];
    }
}

// Few features (F <= 64): a tile of 256 whole rows is one contiguous piece of X; it is read linearly
// (every lane busy, whole lines), kept in LDS with an odd row stride, and written out column by column.
constexpr int kTrNarrowRows = 256, kTrNarrowPer = 8;
__global__ __launch_bounds__(256) void dense_keys_narrow_kernel(const float *__restrict__ X, int64_t n, int F,
                                                                uint32_t *__restrict__ keys) {
    extern __shared__ uint32_t ntile[];   // [kTrNarrowRows][F | 1]
    const int stride = F | 1;
    const int64_t r0 = (int64_t)blockIdx.x * kTrNarrowRows;
    const int rows = n - r0 < kTrNarrowRows ? (int)(n - r0) : kTrNarrowRows;
    const float *src = X + r0 * F;
    const int total = rows * F, dr = 256 / F, df = 256 - dr * F;   // 256 elements on: dr rows and df features
    int r = threadIdx.x / F, f = threadIdx.x - r * F;
    for (int i = threadIdx.x; i < total; i += 256 * kTrNarrowPer) {
        float x[kTrNarrowPer];
#pragma unroll
        for (int k = 0; k < kTrNarrowPer; ++k) x[k] = src[i + 256 * k < total ? i + 256 * k : total - 1];
#pragma unroll
        for (int k = 0; k < kTrNarrowPer; ++k) {
            if (i + 256 * k < total) ntile[r * stride + f] = float_key(x[k]);
            r += dr;
            f += df;
            if (f >= F) {
                f -= F;
                ++r;
            }
        }
    }
    __syncthreads();
    if ((int)threadIdx.x < rows) {
        uint32_t *out = keys + r0 + threadIdx.x;
#pragma unroll 4
        for (int j = 0; j < F; ++j) out[(int64_t)j * n] = ntile[threadIdx.x * stride + j];
    }
}

// ---- 1b. CSR input: count, offset, scatter by column -----------------------
// A fixed number of workgroups take equal runs of whole chunks of the stored values, the same run in both kernels, so the
// first leaves a table of counts per (column, workgroup) whose prefix sums are where the second writes: no atomics on HBM
// (one per chunk and column took turns on each column's address, some 12 ns each).  10M x 50 rows of 10 entries: count
// 0.26 -> 0.09 ms, scatter 1.09 -> 0.43 ms (that one also by writing whole runs, see there).
// More than kCsrLdsCols columns: an atomic per value.
constexpr int kCsrChunk = 4096;   // (24 KB staged: six workgroups of 256 per compute unit, one's barriers under another's loads)
constexpr int kCsrLdsCols = 4096;
constexpr int kCsrBlock = 256;
constexpr int kCsrPer = kCsrChunk / kCsrBlock;

// chunks [*c0, *c1) of workgroup blockIdx.x
__device__ inline void csr_run(int64_t nnz, int64_t *c0, int64_t *c1) {
    const int64_t chunks = (nnz + kCsrChunk - 1) / kCsrChunk;
    *c0 = chunks * blockIdx.x / gridDim.x;
    *c1 = chunks * (blockIdx.x + 1) / gridDim.x;
}

__global__ __launch_bounds__(kCsrBlock) void csr_count_kernel(const int32_t *__restrict__ indices, int64_t nnz, int F,
                                                              uint32_t *__restrict__ table) {
    extern __shared__ uint32_t lc[];   // F
    for (int i = threadIdx.x; i < F; i += kCsrBlock) lc[i] = 0;
    __syncthreads();
    int64_t c0, c1;
    csr_run(nnz, &c0, &c1);
    for (int64_t c = c0; c < c1; ++c) {
        const int64_t i0 = c * kCsrChunk + threadIdx.x;
        int f[kCsrPer];
#pragma unroll
        for (int k = 0; k < kCsrPer; ++k) f[k] = i0 + k * kCsrBlock < nnz ? indices[i0 + k * kCsrBlock] : -1;
#pragma unroll
        for (int k = 0; k < kCsrPer; ++k)
            if (f[k] >= 0 && f[k] < F) atomicAdd(&lc[f[k]], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < F; i += kCsrBlock) table[(int64_t)i * gridDim.x + blockIdx.x] = lc[i];
}

// table[f][w] becomes the first slot of workgroup w in column f; counts[f] the column's length.  A wave per column.
__global__ __launch_bounds__(64) void csr_offsets_kernel(uint32_t *__restrict__ table, int W, uint32_t *__restrict__ counts) {
    uint32_t *t = table + (int64_t)blockIdx.x * W;
    const int lane = threadIdx.x;
    uint32_t run = 0;
    for (int w0 = 0; w0 < W; w0 += 64) {
        const uint32_t v = w0 + lane < W ? t[w0 + lane] : 0u;
        uint32_t x = v;
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = (uint32_t)__shfl_up((int)x, o);
            if (lane >= o) x += y;
        }
        if (w0 + lane < W) t[w0 + lane] = run + x - v;
        run += (uint32_t)__shfl((int)x, 63);
    }
    if (lane == 0) counts[blockIdx.x] = run;
}

// The direct form's count.
__global__ __launch_bounds__(256) void csr_count_direct_kernel(const int32_t *__restrict__ indices, int64_t nnz, int F,
                                                               uint32_t *__restrict__ counts) {
    const int64_t i0 = (int64_t)blockIdx.x * kCsrChunk;
    const int64_t i1 = i0 + kCsrChunk < nnz ? i0 + kCsrChunk : nnz;
    for (int64_t i = i0 + threadIdx.x; i < i1; i += 256) {
        const int f = indices[i];
        if (f >= 0 && f < F) atomicAdd(&counts[f], 1u);
    }
}

// Scatter.  A chunk's keys are put in column order inside LDS and copied out from there: consecutive threads hold
// consecutive keys of a column's run, so a run goes to HBM as whole lines.
inline size_t csr_scatter_lds(int F) { return (size_t)kCsrChunk * 6 + (size_t)F * 12; }
__global__ __launch_bounds__(kCsrBlock) void csr_scatter_kernel(const int32_t *__restrict__ indices,
                                                                const float *__restrict__ values, int64_t nnz, int F,
                                                                const uint64_t *__restrict__ seg_off,
                                                                const uint32_t *__restrict__ table,
                                                                uint32_t *__restrict__ keys) {
    extern __shared__ uint32_t stage[];                        // kCsrChunk keys in column order
    uint32_t *lc = stage + kCsrChunk;                          // F: keys of a column in this chunk
    uint32_t *start = lc + F;                                  // F: the run's first place in `stage`
    uint32_t *cur = start + F;                                 // F: the column's next slot in its segment
    uint16_t *col = (uint16_t *)(cur + F);                     // kCsrChunk: column of a staged key
    __shared__ uint32_t wsum[kCsrBlock / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int i = tid; i < F; i += kCsrBlock) {
        cur[i] = table[(int64_t)i * gridDim.x + blockIdx.x];
        lc[i] = 0;
    }
    int64_t c0, c1;
    csr_run(nnz, &c0, &c1);
    const int per = (F + kCsrBlock - 1) / kCsrBlock, f0 = tid * per, f1 = f0 + per < F ? f0 + per : F;
    for (int64_t c = c0; c < c1; ++c) {
        const int64_t i0 = c * kCsrChunk + tid;
        int f[kCsrPer];
        uint32_t key[kCsrPer], rank[kCsrPer];
#pragma unroll
        for (int k = 0; k < kCsrPer; ++k) {
            const int64_t i = i0 + k * kCsrBlock;
            f[k] = i < nnz ? indices[i] : -1;
            key[k] = i < nnz ? float_key(values[i]) : 0u;
            if (f[k] >= F) f[k] = -1;
        }
        __syncthreads();   // the chunk before has been copied out, its counts cleared
#pragma unroll
        for (int k = 0; k < kCsrPer; ++k) rank[k] = f[k] >= 0 ? atomicAdd(&lc[f[k]], 1u) : 0u;
        __syncthreads();
        // exclusive prefix of the counts: a piece of columns per thread, a scan over the pieces
        uint32_t sum = 0;
        for (int j = f0; j < f1; ++j) sum += lc[j];
        uint32_t x = sum;
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = (uint32_t)__shfl_up((int)x, o);
            if (lane >= o) x += y;
        }
        if (lane == 63) wsum[wave] = x;
        __syncthreads();
        uint32_t at = x - sum, total = 0;
        for (int w = 0; w < kCsrBlock / 64; ++w) {
            at += w < wave ? wsum[w] : 0u;
            total += wsum[w];
        }
        for (int j = f0; j < f1; ++j) {
            start[j] = at;
            at += lc[j];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kCsrPer; ++k)
            if (f[k] >= 0) {
                const uint32_t d = start[f[k]] + rank[k];
                stage[d] = key[k];
                col[d] = (uint16_t)f[k];
            }
        __syncthreads();
        for (uint32_t i = tid; i < total; i += kCsrBlock) {
            const uint32_t j = col[i];
            keys[seg_off[j] + cur[j] + (i - start[j])] = stage[i];
        }
        __syncthreads();
        for (int j = f0; j < f1; ++j) {
            cur[j] += lc[j];
            lc[j] = 0;
        }
    }
}

// More columns than the counters in LDS: a global slot per value.
__global__ __launch_bounds__(256) void csr_scatter_direct_kernel(const int32_t *__restrict__ indices,
                                                                 const float *__restrict__ values, int64_t nnz, int F,
                                                                 const uint64_t *__restrict__ seg_off,
                                                                 uint32_t *__restrict__ cursor,
                                                                 uint32_t *__restrict__ keys) {
    const int64_t i0 = (int64_t)blockIdx.x * kCsrChunk;
    const int64_t i1 = i0 + kCsrChunk < nnz ? i0 + kCsrChunk : nnz;
    for (int64_t i = i0 + threadIdx.x; i < i1; i += 256) {
        const int f = indices[i];
        if (f < 0 || f >= F) continue;
        const uint32_t slot = atomicAdd(&cursor[f], 1u);
        keys[seg_off[f] + slot] = float_key(values[i]);
    }
}

// seg_off / blk_off / chk_off [f] = exclusive prefix of the segments' lengths, tiles and scan chunks (kScanChunk tiles
// each), by one workgroup: a piece of features per thread, then a scan over the pieces.  With `mode` only the features to
// be sorted (kSelSorted) have tiles.  dear[0..1] (may be NULL) are cleared for the selection.
__global__ __launch_bounds__(1024) void offsets_kernel(const uint32_t *counts, int F, int64_t fixed_len,
                                                       const uint32_t *__restrict__ mode, uint64_t *seg_off,
                                                       uint32_t *blk_off, uint32_t *chk_off, int scan_chunk,
                                                       unsigned long long *dear) {
    __shared__ uint64_t so[1024];
    __shared__ uint32_t bo[1024], co[1024];
    const int tid = threadIdx.x, per = (F + 1023) / 1024, f0 = tid * per, f1 = f0 + per < F ? f0 + per : F;
    auto tiles_of = [&](int f, uint64_t len) {
        return mode && mode[f] != kSelSorted ? 0u : (uint32_t)((len + kSortTile - 1) / kSortTile);
    };
    uint64_t o = 0;
    uint32_t b = 0, c = 0;
    for (int f = f0; f < f1; ++f) {
        const uint64_t len = counts ? (uint64_t)counts[f] : (uint64_t)fixed_len;
        const uint32_t tiles = tiles_of(f, len);
        o += len;
        b += tiles;
        c += (tiles + (uint32_t)scan_chunk - 1) / (uint32_t)scan_chunk;
    }
    so[tid] = o;
    bo[tid] = b;
    co[tid] = c;
    __syncthreads();
    for (int d = 1; d < 1024; d <<= 1) {
        const uint64_t po = tid >= d ? so[tid - d] : 0;
        const uint32_t pb = tid >= d ? bo[tid - d] : 0, pc = tid >= d ? co[tid - d] : 0;
        __syncthreads();
        so[tid] += po;
        bo[tid] += pb;
        co[tid] += pc;
        __syncthreads();
    }
    o = so[tid] - o;
    b = bo[tid] - b;
    c = co[tid] - c;
    for (int f = f0; f < f1; ++f) {
        seg_off[f] = o;
        blk_off[f] = b;
        chk_off[f] = c;
        const uint64_t len = counts ? (uint64_t)counts[f] : (uint64_t)fixed_len;
        const uint32_t tiles = tiles_of(f, len);
        o += len;
        b += tiles;
        c += (tiles + (uint32_t)scan_chunk - 1) / (uint32_t)scan_chunk;
    }
    if (tid == 1023) {
        seg_off[F] = so[1023];
        blk_off[F] = bo[1023];
        chk_off[F] = co[1023];
        if (dear) dear[0] = dear[1] = 0;   // (and SelArrays::mix behind it)
    }
}

// ---- 2a. segmented radix sort ----------------------------------------------
// One count per key into a 256-bin LDS histogram.  Sorted or low-cardinality data gives a whole wave
// the same digit, which as 64 atomics on one address would take 64 turns: that case is one add.
__device__ inline void count_digit(uint32_t *h, uint32_t d, bool live) {
    const uint64_t act = __ballot(live);
    if (act == 0) return;
    const uint32_t lead = (uint32_t)__builtin_amdgcn_readlane((int)d, (int)__builtin_ctzll(act));
    if (__ballot(live && d == lead) == act) {
        if ((threadIdx.x & 63) == (uint32_t)__builtin_ctzll(act)) atomicAdd(&h[lead], (uint32_t)__popcll(act));
    } else if (live) {
        atomicAdd(&h[d], 1u);
    }
}

// A segment's keys sit in one of the two key buffers (bit 0 of its flag word: 0 = keys_a); a pass in which all keys
// of a segment have the same digit is the identity for it and moves nothing (bit 1, set by scan_chunks_kernel, read
// by sort_scatter_kernel), so after the pass the segment is still where it was (flip_kernel).
constexpr uint32_t kSegInB = 1u, kSegSkip = 2u;

__global__ __launch_bounds__(kSortBlock) void sort_hist_kernel(const uint32_t *__restrict__ keys_a,
                                                               const uint32_t *__restrict__ keys_b,
                                                               const uint32_t *__restrict__ seg_flags,
                                                               const uint64_t *__restrict__ seg_off,
                                                               const uint32_t *__restrict__ blk_off, int F,
                                                               int shift, uint32_t *__restrict__ tile_hist) {
    __shared__ uint32_t h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t blk = blockIdx.x;
    const int f = find_segment(blk_off, F, blk);
    const uint32_t *__restrict__ keys = (seg_flags[f] & kSegInB) ? keys_b : keys_a;
    const uint64_t base = seg_off[f], len = seg_off[f + 1] - base;
    const uint64_t t0 = (uint64_t)(blk - blk_off[f]) * kSortTile;
    if (t0 + kSortTile <= len) {   // a whole tile: all loads are issued before the first count
        uint32_t k[kSortTile / kSortBlock];
#pragma unroll
        for (int j = 0; j < kSortTile / kSortBlock; ++j) k[j] = keys[base + t0 + (uint64_t)j * kSortBlock + threadIdx.x];
#pragma unroll
        for (int j = 0; j < kSortTile / kSortBlock; ++j) count_digit(h, (k[j] >> shift) & 255u, true);
    } else {
        for (int i0 = 0; i0 < kSortTile; i0 += kSortBlock) {   // uniform trip count: count_digit uses ballots
            const uint64_t p = t0 + i0 + threadIdx.x;
            const bool live = p < len;
            count_digit(h, live ? (keys[base + p] >> shift) & 255u : 0u, live);
        }
    }
    __syncthreads();
    tile_hist[(uint64_t)blk * 256 + threadIdx.x] = h[threadIdx.x];
}

// tile_hist[blk][d] becomes the position (inside the segment) of the first key of tile blk
// with digit d.  Three launches, thread d owns digit d everywhere:
//   partial : one workgroup per chunk of kScanChunk tiles adds up the chunk's counts;
//   chunks  : one workgroup per segment turns the chunk totals into chunk start positions
//             (exclusive over chunks, then offset by the exclusive scan over the digits);
//   apply   : one workgroup per chunk walks its tiles from the chunk's start position.
constexpr int kScanChunk = 128;

__global__ __launch_bounds__(256) void scan_partial_kernel(const uint32_t *__restrict__ blk_off,
                                                           const uint32_t *__restrict__ chk_off, int F,
                                                           const uint32_t *__restrict__ tile_hist,
                                                           uint32_t *__restrict__ chunk_tot) {
    const uint32_t chunk = blockIdx.x;
    const int f = find_segment(chk_off, F, chunk), d = threadIdx.x;
    const uint32_t b0 = blk_off[f] + (chunk - chk_off[f]) * kScanChunk;
    const uint32_t b1 = b0 + kScanChunk < blk_off[f + 1] ? b0 + kScanChunk : blk_off[f + 1];
    uint32_t run = 0;
    for (uint32_t b = b0; b < b1; ++b) run += tile_hist[(uint64_t)b * 256 + d];
    chunk_tot[(uint64_t)chunk * 256 + d] = run;
}

__global__ __launch_bounds__(256) void scan_chunks_kernel(const uint32_t *__restrict__ chk_off,
                                                          const uint64_t *__restrict__ seg_off,
                                                          uint32_t *__restrict__ seg_flags,
                                                          uint32_t *__restrict__ chunk_tot) {
    const int f = blockIdx.x, d = threadIdx.x;
    const uint32_t c0 = chk_off[f], c1 = chk_off[f + 1];
    uint32_t run = 0;
    for (uint32_t c = c0; c < c1; ++c) {
        const uint32_t v = chunk_tot[(uint64_t)c * 256 + d];
        chunk_tot[(uint64_t)c * 256 + d] = run;
        run += v;
    }
    __shared__ uint32_t tot[256];
    tot[d] = run;
    if (d == 0) seg_flags[f] &= ~kSegSkip;
    __syncthreads();
    // every key of the segment has digit d: at most one thread sees that
    if (run > 0 && (uint64_t)run == seg_off[f + 1] - seg_off[f]) seg_flags[f] |= kSegSkip;
    for (int o = 1; o < 256; o <<= 1) {
        uint32_t v = d >= o ? tot[d - o] : 0;
        __syncthreads();
        tot[d] += v;
        __syncthreads();
    }
    const uint32_t base = tot[d] - run;   // keys of this segment with a smaller digit
    for (uint32_t c = c0; c < c1; ++c) chunk_tot[(uint64_t)c * 256 + d] += base;
}

__global__ __launch_bounds__(256) void scan_apply_kernel(const uint32_t *__restrict__ blk_off,
                                                         const uint32_t *__restrict__ chk_off, int F,
                                                         uint32_t *__restrict__ tile_hist,
                                                         const uint32_t *__restrict__ chunk_tot) {
    const uint32_t chunk = blockIdx.x;
    const int f = find_segment(chk_off, F, chunk), d = threadIdx.x;
    const uint32_t b0 = blk_off[f] + (chunk - chk_off[f]) * kScanChunk;
    const uint32_t b1 = b0 + kScanChunk < blk_off[f + 1] ? b0 + kScanChunk : blk_off[f + 1];
    uint32_t run = chunk_tot[(uint64_t)chunk * 256 + d];
    for (uint32_t b = b0; b < b1; ++b) {
        const uint32_t c = tile_hist[(uint64_t)b * 256 + d];
        tile_hist[(uint64_t)b * 256 + d] = run;
        run += c;
    }
}

// Stable scatter of one tile.  The tile's keys are first put in digit order inside LDS (ranks from
// per-wave digit counts and, inside a round of 64 keys, from ballots), then copied out: consecutive
// threads hold consecutive keys of a digit's run, so the run goes to HBM as whole lines instead of
// 64 separate 4-byte stores per wave instruction.
__global__ __launch_bounds__(kSortBlock) void sort_scatter_kernel(uint32_t *__restrict__ keys_a,
                                                                  uint32_t *__restrict__ keys_b,
                                                                  const uint32_t *__restrict__ seg_flags,
                                                                  const uint64_t *__restrict__ seg_off,
                                                                  const uint32_t *__restrict__ blk_off, int F,
                                                                  int shift,
                                                                  const uint32_t *__restrict__ tile_hist) {
    __shared__ uint32_t cnt[kSortBlock / 64][256];   // per wave: running local position per digit
    __shared__ uint32_t local_start[256];            // first local position of each digit's run
    __shared__ uint32_t run_base[256];               // position in the segment of each digit's run
    __shared__ uint32_t stage[kSortTile];
    static_assert(kSortBlock == 256, "one thread per digit below");
    const uint32_t blk = blockIdx.x;
    const int f = find_segment(blk_off, F, blk);
    const uint32_t flags = seg_flags[f];
    if (flags & kSegSkip) return;   // (the whole workgroup: one segment per tile)
    const uint32_t *__restrict__ src = (flags & kSegInB) ? keys_b : keys_a;
    uint32_t *__restrict__ dst = (flags & kSegInB) ? keys_a : keys_b;
    const uint64_t base = seg_off[f], len = seg_off[f + 1] - base;
    const uint64_t t0 = (uint64_t)(blk - blk_off[f]) * kSortTile;
    const uint32_t tile_keys = len - t0 < (uint64_t)kSortTile ? (uint32_t)(len - t0) : (uint32_t)kSortTile;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int i = threadIdx.x; i < (kSortBlock / 64) * 256; i += kSortBlock) (&cnt[0][0])[i] = 0;
    __syncthreads();

    // the wave's 1024 keys, 64 per round, kept in registers
    uint32_t key[kRounds];
    const uint64_t w0 = t0 + (uint64_t)wave * kKeysPerWave;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const uint64_t p = w0 + (uint64_t)r * 64 + lane;
        key[r] = p < len ? src[base + p] : 0;
        if (p < len) atomicAdd(&cnt[wave][(key[r] >> shift) & 255u], 1u);
    }
    __syncthreads();
    // thread d: the tile's digit-d keys are [local_start[d], local_start[d] + total) inside the tile,
    // wave w's share of them starts at cnt[w][d]
    {
        const int d = threadIdx.x;
        uint32_t total = 0;
        for (int w = 0; w < kSortBlock / 64; ++w) total += cnt[w][d];
        // exclusive scan of the totals over the 256 digits
        uint32_t x = total;
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = (uint32_t)__shfl_up((int)x, o);
            if (lane >= o) x += y;
        }
        __shared__ uint32_t wave_tot[kSortBlock / 64];
        if (lane == 63) wave_tot[wave] = x;
        __syncthreads();
        uint32_t before = 0;
        for (int w = 0; w < wave; ++w) before += wave_tot[w];
        const uint32_t start = before + x - total;
        local_start[d] = start;
        run_base[d] = tile_hist[(uint64_t)blk * 256 + d];
        uint32_t run = start;
        for (int w = 0; w < kSortBlock / 64; ++w) {
            const uint32_t c = cnt[w][d];
            cnt[w][d] = run;
            run += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const uint64_t p = w0 + (uint64_t)r * 64 + lane;
        const bool live = p < len;
        const uint32_t dgt = (key[r] >> shift) & 255u;
        // lanes of this round with the same digit
        uint64_t peers = __ballot(live);
        for (int b = 0; b < 8; ++b) {
            const uint64_t m = __ballot((dgt >> b) & 1u);
            peers &= ((dgt >> b) & 1u) ? m : ~m;
        }
        volatile uint32_t *wc = cnt[wave];   // touched by this wave only from here on
        const uint32_t below = (uint32_t)__popcll(peers & ((1ull << lane) - 1ull));
        uint32_t first = 0;
        if (live) first = wc[dgt];            // every peer reads the same count ...
        __builtin_amdgcn_wave_barrier();
        if (live && below == 0) wc[dgt] = first + (uint32_t)__popcll(peers);   // ... before the leader bumps it
        __builtin_amdgcn_wave_barrier();
        if (live) stage[first + below] = key[r];   // first + below < tile_keys
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < tile_keys; i += kSortBlock) {
        const uint32_t k = stage[i];
        const uint32_t d = (k >> shift) & 255u;
        dst[base + run_base[d] + (i - local_start[d])] = k;
    }
}

// after a pass: the segments that were scattered have changed buffers
__global__ void flip_kernel(uint32_t *seg_flags, int F) {
    const int f = blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= F) return;
    const uint32_t fl = seg_flags[f];
    seg_flags[f] = (fl & kSegSkip) ? (fl & kSegInB) : ((fl & kSegInB) ^ kSegInB);
}

// ---- 2b. cuts of a sorted segment ----------------------------------------------------------------
// First index in [lo, hi) with a[i] > v (hi if there is none), found by a whole wave: 64 probes per step cut the
// range by 65, so 1.15e8 keys take five dependent rounds of loads instead of 27.  Every lane passes the same
// arguments and gets the same result.
__device__ inline uint64_t upper_bound_wave(const uint32_t *a, uint64_t lo, uint64_t hi, uint32_t v, int lane) {
    while (hi - lo > 64) {
        const uint64_t span = hi - lo;   // probes lo + span * (l + 1) / 65 are distinct and inside [lo, hi)
        const bool gt = a[lo + span * (uint64_t)(lane + 1) / 65] > v;
        const uint64_t m = __ballot(gt);
        if (m == 0) {
            lo = lo + span * 64 / 65 + 1;   // the last probe is still <= v
        } else {
            const int first = __builtin_ctzll(m);
            const uint64_t new_hi = lo + span * (uint64_t)(first + 1) / 65;   // > v: the answer is at or before it
            if (first > 0) lo = lo + span * (uint64_t)first / 65 + 1;         // the probe before it is <= v
            hi = new_hi;
        }
    }
    const bool gt = lo + (uint64_t)lane < hi && a[lo + (uint64_t)lane] > v;
    const uint64_t m = __ballot(gt);
    return m ? lo + (uint64_t)__builtin_ctzll(m) : hi;
}

// One wave per feature (with `mode`: of those that were sorted).  Wave-uniform control flow throughout; lane 0 writes.
__global__ __launch_bounds__(64) void cuts_kernel(const uint32_t *__restrict__ keys_a, const uint32_t *__restrict__ keys_b,
                                                  const uint32_t *__restrict__ seg_flags,
                                                  const uint64_t *__restrict__ seg_off, const uint32_t *__restrict__ mode,
                                                  int F, int B, float *__restrict__ cuts, int32_t *__restrict__ nb,
                                                  uint32_t *__restrict__ present) {
    const int f = blockIdx.x, lane = threadIdx.x;
    if (f >= F || (mode && mode[f] != kSelSorted)) return;
    const uint32_t *v = ((seg_flags[f] & kSegInB) ? keys_b : keys_a) + seg_off[f];
    const uint64_t len = seg_off[f + 1] - seg_off[f];
    float *c = cuts + (int64_t)f * (B - 1);
    for (int k = lane; k < B - 1; k += 64) c[k] = __uint_as_float(0x7f800000u);   // +inf
    // present values = keys below the missing key
    const uint64_t m = len == 0 ? 0 : upper_bound_wave(v, 0, len, kMissingKey - 1u, lane);
    if (lane == 0) present[f] = (uint32_t)m;
    if (m == 0) {
        if (lane == 0) nb[f] = 1;
        return;
    }
    // distinct values, counted up to B+1; the first B-1 after the smallest are
    // written as tentative cuts
    int d = 0, nc = 0;
    uint64_t pos = 0;
    while (pos < m && d <= B) {
        const uint32_t key = v[pos];
        if (d >= 1 && d <= B - 1 && lane == 0) c[d - 1] = key_float(key);
        ++d;
        pos = upper_bound_wave(v, pos + 1, m, key, lane);
    }
    if (d <= B) {
        nc = d - 1;
    } else {
        // the B-1 order statistics, fetched 64 at a time, then thinned by lane 0 in order
        __shared__ uint32_t pick[4096];
        const uint32_t vmin = v[0];
        uint32_t prev = 0;
        for (int k0 = 1; k0 < B; k0 += 4096) {
            const int cnt = B - k0 < 4096 ? B - k0 : 4096;
            for (int j = lane; j < cnt; j += 64) pick[j] = v[(uint64_t)(k0 + j) * m / (uint64_t)B];
            __syncthreads();
            if (lane == 0) {
                for (int j = 0; j < cnt; ++j) {
                    const uint32_t key = pick[j];
                    if (key == vmin) continue;
                    if (nc > 0 && key == prev) continue;
                    c[nc++] = key_float(key);
                    prev = key;
                }
            }
            __syncthreads();
        }
        nc = __shfl(nc, 0);
        for (int k = nc + lane; k < B - 1; k += 64) c[k] = __uint_as_float(0x7f800000u);
    }
    if (lane == 0) nb[f] = nc + 1;
}

// ---- 3. binning -------------------------------------------------------------
__device__ inline uint32_t bin_of(const float *c, int ncut, float x) {
    int lo = 0, hi = ncut;   // number of cuts <= x
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (c[mid] <= x) lo = mid + 1; else hi = mid;
    }
    return (uint32_t)lo;
}

// LDS_CUTS: the cut table (F * (B-1) floats) and nb are staged in LDS first, so the bisection's
// dependent reads stay on the CU (the table is 13 KB for 13 x 256 bins).  The feature of an element
// is carried along instead of a 64-bit modulo per element.
template <bool LDS_CUTS>
__global__ __launch_bounds__(256) void bin_dense_kernel(const float *__restrict__ X, int64_t n_elems, int F, int B,
                                                        const float *__restrict__ cuts, const int32_t *__restrict__ nb,
                                                        uint32_t missing, uint16_t *__restrict__ sym,
                                                        uint32_t *__restrict__ max_out) {
    extern __shared__ float lcuts[];
    int32_t *lnb = (int32_t *)(lcuts + (LDS_CUTS ? F * (B - 1) : 0));
    if (LDS_CUTS) {
        for (int i = threadIdx.x; i < F * (B - 1); i += 256) lcuts[i] = cuts[i];
        for (int i = threadIdx.x; i < F; i += 256) lnb[i] = nb[i];
        __syncthreads();
    }
    const float *ct = LDS_CUTS ? lcuts : cuts;
    const int32_t *nbt = LDS_CUTS ? lnb : nb;
    uint32_t mx = 0;
    const int64_t stride = (int64_t)gridDim.x * 256;
    const int step_f = (int)(stride % F);
    int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    int f = (int)(e % F);
    for (; e < n_elems; e += stride) {
        const float x = X[e];
        const uint32_t s = (x != x) ? missing : bin_of(ct + f * (B - 1), nbt[f] - 1, x);
        sym[e] = (uint16_t)s;
        mx = s > mx ? s : mx;
        f += step_f;
        f = f >= F ? f - F : f;
    }
    for (int o = 32; o > 0; o >>= 1) {
        const uint32_t t = (uint32_t)__shfl_xor((int)mx, o);
        mx = t > mx ? t : mx;
    }
    __shared__ uint32_t wmax[4];
    if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0) atomicMax(max_out, max(max(wmax[0], wmax[1]), max(wmax[2], wmax[3])));
}

__global__ void fill_u16_kernel(uint16_t *p, uint16_t v, int64_t count) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void bin_csr_kernel(const int64_t *__restrict__ indptr, const int32_t *__restrict__ indices,
                               const float *__restrict__ values, int64_t n, int64_t nnz, int F, int B,
                               const float *__restrict__ cuts, const int32_t *__restrict__ nb, uint32_t missing,
                               uint16_t *__restrict__ sym, uint32_t *__restrict__ max_out) {
    uint32_t mx = 0;
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n;
         r += (int64_t)gridDim.x * blockDim.x) {
        int64_t a = indptr[r], b = indptr[r + 1];
        if (a < 0) a = 0;
        if (b > nnz) b = nnz;
        bool any_missing = (b - a) < F;
        for (int64_t i = a; i < b; ++i) {
            const int f = indices[i];
            if (f < 0 || f >= F) continue;
            const float x = values[i];
            const uint32_t s = (x != x) ? missing : bin_of(cuts + (int64_t)f * (B - 1), nb[f] - 1, x);
            sym[r * F + f] = (uint16_t)s;
            mx = s > mx ? s : mx;
        }
        if (any_missing) mx = missing > mx ? missing : mx;
    }
    for (int o = 32; o > 0; o >>= 1) {
        const uint32_t t = (uint32_t)__shfl_xor((int)mx, o);
        mx = t > mx ? t : mx;
    }
    if ((threadIdx.x & 63) == 0) atomicMax(max_out, mx);
}

// ---- 3b. binning and packing in one pass (Sec. 2.1 -> Sec. 2.2) ------------------
// The symbols of a tile of elements are binned into LDS and leave as words of the bit stream: the uint16 symbol
// matrix never exists.  A tile holds a multiple of 32 elements, so it starts on a word boundary whatever the width;
// one thread assembles one word from the LDS symbols that overlap it.
constexpr int kPackTile = 4096;   // elements per tile of the dense form

__device__ inline void pack_tile(const uint16_t *lsym, int tile_elems, int bits, uint32_t *out) {
    const int nw = (tile_elems * bits + 31) >> 5;
    for (int w = threadIdx.x; w < nw; w += 256) {
        const int bit0 = w * 32;
        uint32_t word = 0;
        for (int e = bit0 / bits; e < tile_elems; ++e) {
            const int pos = e * bits - bit0;   // may be negative for the first element
            if (pos >= 32) break;
            const uint32_t sv = lsym[e];
            word |= pos >= 0 ? (sv << pos) : (sv >> (-pos));
        }
        out[w] = word;
    }
}

template <bool LDS_CUTS>
__global__ __launch_bounds__(256) void bin_pack_dense_kernel(const float *__restrict__ X, int64_t n_elems, int F, int B,
                                                             const float *__restrict__ cuts,
                                                             const int32_t *__restrict__ nb, uint32_t missing, int bits,
                                                             uint32_t *__restrict__ packed, int64_t n_words) {
    extern __shared__ float lcuts[];
    int32_t *lnb = (int32_t *)(lcuts + (LDS_CUTS ? F * (B - 1) : 0));
    __shared__ uint16_t lsym[kPackTile];
    if (LDS_CUTS) {
        for (int i = threadIdx.x; i < F * (B - 1); i += 256) lcuts[i] = cuts[i];
        for (int i = threadIdx.x; i < F; i += 256) lnb[i] = nb[i];
        __syncthreads();
    }
    const float *ct = LDS_CUTS ? lcuts : cuts;
    const int32_t *nbt = LDS_CUTS ? lnb : nb;
    const int64_t n_tiles = (n_elems + kPackTile - 1) / kPackTile;
    const int step_f = 256 % F;
    for (int64_t t = blockIdx.x; t < n_tiles; t += gridDim.x) {
        const int64_t e0 = t * kPackTile;
        const int tile_elems = n_elems - e0 < kPackTile ? (int)(n_elems - e0) : kPackTile;
        int f = (int)((e0 + threadIdx.x) % F);
        float x[kPackTile / 256];
#pragma unroll
        for (int j = 0; j < kPackTile / 256; ++j) {
            const int i = j * 256 + (int)threadIdx.x;
            x[j] = i < tile_elems ? X[e0 + i] : 0.0f;
        }
#pragma unroll
        for (int j = 0; j < kPackTile / 256; ++j) {
            const int i = j * 256 + (int)threadIdx.x;
            if (i < tile_elems)
                lsym[i] = (uint16_t)((x[j] != x[j]) ? missing : bin_of(ct + f * (B - 1), nbt[f] - 1, x[j]));
            f += step_f;
            f = f >= F ? f - F : f;
        }
        __syncthreads();
        pack_tile(lsym, tile_elems, bits, packed + e0 / 32 * bits);   // kPackTile * bits / 32 words per tile
        __syncthreads();
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) packed[n_words - 1] = 0;   // the pad word (Sec. 2.2 layout)
}

// CSR input: a tile of rows (a multiple of 32) is laid out in LDS as missing symbols, the stored values of those rows
// are binned into their places, and the tile is packed.  A row is taken by 2^log_lanes neighbouring lanes (about as many
// as a row has entries), so no lane has to search for the row of its entry and a wave's loads are one piece of the CSR
// arrays.  The cuts are searched in two levels: every 2^cut_log-th one in LDS (all of them where they fit: 51 KB for
// 50 x 255), then the few between two of those.
// UNEVEN (rows can have more entries than four turns of their lanes): a tile with such a row gives every row more lanes, up to
// what takes all rows in one turn; otherwise its longest row holds up the whole workgroup.  5M x 50, one row in a hundred full,
// the others with one entry: the call 1.87 ms without this, 0.84 with it.  The look costs 0.3 us a tile, so where no row can be
// that long it is left out.
// 10M x 50 rows of 10 entries: 0.84 ms; 1.99 ms with a bisection for the row, one through global memory for the cut and
// a word of the stream at a time.  Instruction issue is what remains (90 MB of words written, 0.9 GB read).
constexpr int kCsrPackBlock = 1024;
constexpr int kCsrPackRows = 4;   // rows side by side: their loads and searches overlap
template <int BITS, bool UNEVEN>
__global__ __launch_bounds__(kCsrPackBlock) __attribute__((amdgpu_waves_per_eu(8))) void bin_pack_csr_kernel(
    const int64_t *__restrict__ indptr, const int32_t *__restrict__ indices, const float *__restrict__ values, int64_t n,
    int64_t nnz, int F, int B, const float *__restrict__ cuts, const int32_t *__restrict__ nb, uint32_t missing, int tile_rows,
    int log_lanes, int cut_log, int step0, uint32_t *__restrict__ packed, int64_t n_words) {
    extern __shared__ uint32_t dyn[];
    uint16_t *lrow = (uint16_t *)dyn;                        // tile_rows * F symbols (a multiple of 32)
    float *tops = (float *)(dyn + ((size_t)tile_rows * F) / 2);   // F x n_top, padded with +inf
    const int n_top = 2 * step0 - 1;
    int32_t *lcut = (int32_t *)(tops + (size_t)F * n_top);   // F: cuts of a feature
    uint32_t *lptr = (uint32_t *)(lcut + F);                 // tile_rows + 1 row pointers, relative to the tile's first
    for (int i = threadIdx.x; i < F * n_top; i += kCsrPackBlock) {
        const int f = i / n_top, at = ((i - f * n_top + 1) << cut_log) - 1;
        tops[i] = at < B - 1 ? cuts[(int64_t)f * (B - 1) + at] : __uint_as_float(0x7f800000u);
    }
    for (int i = threadIdx.x; i < F; i += kCsrPackBlock) lcut[i] = nb[i] - 1;
    const int64_t n_tiles = (n + tile_rows - 1) / tile_rows;
    __shared__ uint32_t longest;   // row of the tile, if it takes more than four turns
    if (UNEVEN) {
        if (threadIdx.x == 0) longest = 0;
        __syncthreads();
    }
    const uint32_t two = missing | (missing << 16);
    // Entries of a tile (rows may repeat a column).  A lane whose row has ended moves on with the others of its turn: twice
    // this and a lane count more has to fit 32 bits.
    constexpr uint32_t kMost = (1u << 31) - 128u;
    for (int64_t t = blockIdx.x; t < n_tiles; t += gridDim.x) {
        const int64_t r0 = t * tile_rows;
        const int rows = n - r0 < tile_rows ? (int)(n - r0) : tile_rows;
        const int elems = rows * F;
        int64_t a0 = indptr[r0];
        a0 = a0 < 0 ? 0 : a0 > nnz ? nnz : a0;
        for (int i = threadIdx.x; i < (elems + 1) / 2; i += kCsrPackBlock) dyn[i] = two;
        for (int i = threadIdx.x; i <= rows; i += kCsrPackBlock) {
            int64_t p = indptr[r0 + i];
            p = p < a0 ? a0 : p > nnz ? nnz : p;
            lptr[i] = p - a0 < (int64_t)kMost ? (uint32_t)(p - a0) : kMost;
            if (UNEVEN && i < rows) {
                const int64_t len = indptr[r0 + i + 1] - p;
                if (len > (4 << log_lanes)) atomicMax(&longest, len < (int64_t)kMost ? (uint32_t)len : kMost);
            }
        }
        __syncthreads();
        int ll = log_lanes;   // (in scalar registers, as what follows from it)
        if (UNEVEN) {
            const uint32_t most = (uint32_t)__builtin_amdgcn_readfirstlane((int)longest);
            while (ll < 6 && most > (4u << ll) && (rows << (ll + 1)) <= kCsrPackRows * kCsrPackBlock) ++ll;
        }
        const int lanes = 1 << ll, sub = threadIdx.x & (lanes - 1), groups = kCsrPackBlock >> ll;
        const int32_t *ip = indices + a0;
        const float *vp = values + a0;
        constexpr int U = kCsrPackRows;
        for (int rb = threadIdx.x >> ll; rb < rows; rb += U * groups) {
            uint32_t at[U], end[U];
            bool more = false;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int r = rb + u * groups;
                at[u] = r < rows ? lptr[r] + sub : 0;
                end[u] = r < rows ? lptr[r + 1] : 0;
                more |= at[u] < end[u];
            }
            while (more) {
                int f[U], base[U], pos[U];
                float x[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    f[u] = at[u] < end[u] ? ip[at[u]] : -1;
                    x[u] = at[u] < end[u] ? vp[at[u]] : 0.0f;
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    f[u] = (unsigned)f[u] < (unsigned)F ? f[u] : -1;
                    base[u] = pos[u] = (f[u] < 0 ? 0 : f[u]) * n_top;
                }
                for (int step = step0; step > 0; step >>= 1) {   // pos - base: tops at or below x
#pragma unroll
                    for (int u = 0; u < U; ++u) pos[u] += tops[pos[u] + step - 1] <= x[u] ? step : 0;
                }
                more = false;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (f[u] >= 0) {
                        const int ncut = lcut[f[u]];
                        int lo = (pos[u] - base[u]) << cut_log;
                        if (cut_log) {
                            const float *c = cuts + (int64_t)f[u] * (B - 1);
                            int hi = lo + (1 << cut_log) - 1;
                            hi = hi < B - 1 ? hi : B - 1;
                            while (lo < hi) {
                                const int mid = (lo + hi) >> 1;
                                if (c[mid] <= x[u]) lo = mid + 1; else hi = mid;
                            }
                        }
                        lo = lo < ncut ? lo : ncut;   // (x = +inf lies at or above the padding)
                        lrow[(rb + u * groups) * F + f[u]] = (uint16_t)(x[u] == x[u] ? (uint32_t)lo : missing);
                    }
                    at[u] += lanes;
                    more |= at[u] < end[u];
                }
            }
        }
        __syncthreads();
        if (UNEVEN && threadIdx.x == 0) longest = 0;
        uint32_t *out = packed + ((r0 * F) >> 5) * BITS;   // r0 * F is a multiple of 32
        const int nw = (int)(((int64_t)elems * BITS + 31) >> 5);
        for (int g = threadIdx.x; g < (elems + 31) >> 5; g += kCsrPackBlock) {
            const uint4 *src = (const uint4 *)(dyn + 16 * g);
            const uint4 q[4] = {src[0], src[1], src[2], src[3]};
            const uint32_t s[16] = {q[0].x, q[0].y, q[0].z, q[0].w, q[1].x, q[1].y, q[1].z, q[1].w,
                                    q[2].x, q[2].y, q[2].z, q[2].w, q[3].x, q[3].y, q[3].z, q[3].w};
            uint32_t w[BITS];
            pack_group<BITS>(w, [&](int j) -> uint32_t {
                const uint32_t v = (j & 1) ? s[j >> 1] >> 16 : s[j >> 1] & 0xffffu;
                return 32 * g + j < elems ? v : 0u;
            });
#pragma unroll
            for (int i = 0; i < BITS; ++i)
                if (g * BITS + i < nw) out[(int64_t)g * BITS + i] = w[i];
        }
        __syncthreads();
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) packed[n_words - 1] = 0;
}

// Does any element lack a value?  A row with fewer than F stored entries, or a stored NaN.
__global__ void csr_any_missing_kernel(const int64_t *__restrict__ indptr, const float *__restrict__ values, int64_t n,
                                       int64_t nnz, int F, uint32_t *__restrict__ flag) {
    bool any = false;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x, i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t r = i0; r < n; r += stride) {
        int64_t a = indptr[r], b = indptr[r + 1];
        a = a < 0 ? 0 : a;
        b = b > nnz ? nnz : b;
        any |= (b - a) < F;
    }
    for (int64_t i = i0; i < nnz; i += stride) {
        const float x = values[i];
        any |= x != x;
    }
    if (__ballot(any) != 0 && (threadIdx.x & 63) == 0) atomicOr(flag, 1u);
}

// workgroups of the CSR count and scatter: six per compute unit, at least a chunk each
constexpr int kCsrWorkgroups = 1536;
int csr_workgroups(int num_cu, int64_t nnz) {
    const int64_t chunks = (nnz + kCsrChunk - 1) / kCsrChunk;
    const int most = 6 * num_cu < kCsrWorkgroups ? 6 * num_cu : kCsrWorkgroups;
    return (int)(chunks < 1 ? 1 : chunks < most ? chunks : most);
}

struct QLayout {
    size_t keys_a, keys_b, tile_hist, chunk_tot, seg_off, blk_off, chk_off, counts, cursor, seg_flags, present, misc, select, csr_table, total;
    int64_t max_tiles, max_chunks;
};
QLayout q_layout(int64_t n, int F, int64_t n_values, int B) {
    QLayout L;
    L.max_tiles = n_values / kSortTile + F + 1;
    size_t o = 0;
    L.keys_a = o;    o += gbt_align((size_t)n_values * 4 + 4);
    // (behind the selection, a dense matrix's columns of symbols)
    const bool select = gbt_select_ok(F, n_values, B);
    const size_t cols = select && n_values >= n * (int64_t)F ? gbt_bin_columns_bytes(n, F) : 0;
    L.keys_b = o;    o += gbt_align(cols > (size_t)n_values * 4 + 4 ? cols : (size_t)n_values * 4 + 4);
    L.tile_hist = o; o += gbt_align((size_t)L.max_tiles * 256 * 4);
    L.max_chunks = L.max_tiles / 128 + F + 1;
    L.chunk_tot = o; o += gbt_align((size_t)L.max_chunks * 256 * 4);
    L.seg_off = o;   o += gbt_align((size_t)(F + 1) * 8);
    L.blk_off = o;   o += gbt_align((size_t)(F + 1) * 4);
    L.chk_off = o;   o += gbt_align((size_t)(F + 1) * 4);
    L.counts = o;    o += gbt_align((size_t)F * 4);
    L.cursor = o;    o += gbt_align((size_t)F * 4);
    L.seg_flags = o; o += gbt_align((size_t)F * 4);
    L.present = o;   o += gbt_align((size_t)F * 4);
    L.misc = o;      o += 256;
    L.select = o;    o += select ? gbt_select_layout(F, n_values, B, nullptr, nullptr) : 0;
    L.csr_table = o; o += F > kCsrLdsCols ? 0 : gbt_align((size_t)F * kCsrWorkgroups * 4);
    L.total = o;
    return L;
}

inline int grid_for(int64_t count, int per_block, int cap) {
    int64_t g = (count + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (int)g;
}

}  // namespace

size_t gbt_quantise_ws(int64_t n, int F, int64_t n_values, int B) {
    return q_layout(n, F, n_values, B).total;
}

#define Q_HIP(call)                        \
    do {                                   \
        hipError_t e_ = (call);            \
        if (e_ != hipSuccess) return e_;   \
    } while (0)

// Small results to the host with one wait: through the pinned staging as far as they fit there.
struct ReadBack {
    void *to;
    const void *from;
    size_t bytes;
};
static hipError_t read_back(gbt_ctx *ctx, std::initializer_list<ReadBack> what) {
    const size_t room = GBT_STAGING_BYTES / 2;
    char *pin = ctx->pinned + room;
    size_t at = 0;
    for (const ReadBack &r : what) {
        const bool fits = at + r.bytes <= room;
        hipError_t e = hipMemcpyAsync(fits ? (void *)(pin + at) : r.to, r.from, r.bytes, hipMemcpyDeviceToHost, ctx->stream);
        if (e != hipSuccess) return e;
        if (fits) at += gbt_align(r.bytes, 16);
    }
    hipError_t e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) return e;
    at = 0;
    for (const ReadBack &r : what)
        if (at + r.bytes <= room) {
            memcpy(r.to, pin + at, r.bytes);
            at += gbt_align(r.bytes, 16);
        }
    return hipSuccess;
}

hipError_t gbt_quantise_run(gbt_ctx *ctx, const float *X, const int64_t *indptr, const int32_t *indices,
                            const float *values, int64_t n, int F, int64_t n_values, int B, float *cuts,
                            int32_t *nb, uint16_t *sym, int32_t *max_value, int32_t *missing_sym, char *ws,
                            size_t ws_bytes, int32_t *status, uint32_t *packed, int64_t packed_cap_words,
                            int32_t *bits_out) {
    (void)ws_bytes;
    *status = GBT_OK;
    hipStream_t s = ctx->stream;
    const QLayout L = q_layout(n, F, n_values, B);
    uint32_t *keys_a = (uint32_t *)(ws + L.keys_a), *keys_b = (uint32_t *)(ws + L.keys_b);
    uint32_t *tile_hist = (uint32_t *)(ws + L.tile_hist);
    uint64_t *seg_off = (uint64_t *)(ws + L.seg_off);
    uint32_t *blk_off = (uint32_t *)(ws + L.blk_off);
    uint32_t *chk_off = (uint32_t *)(ws + L.chk_off);
    uint32_t *chunk_tot = (uint32_t *)(ws + L.chunk_tot);
    uint32_t *counts = (uint32_t *)(ws + L.counts), *cursor = (uint32_t *)(ws + L.cursor);
    uint32_t *misc = (uint32_t *)(ws + L.misc);
    uint32_t *seg_flags = (uint32_t *)(ws + L.seg_flags);
    uint32_t *present = (uint32_t *)(ws + L.present);
    const bool dense = X != nullptr;

    const bool select = gbt_select_ok(F, n_values, B) && !ctx->quantise_sort;
    SelArrays A{};
    if (select) gbt_select_layout(F, n_values, B, ws + L.select, &A);

    // 1. key segments
    if (dense) {
        offsets_kernel<<<1, 1024, 0, s>>>(nullptr, F, n, nullptr, seg_off, blk_off, chk_off, kScanChunk, A.dear);
        if (n > 0 && F <= 64) {
            const size_t lds = (size_t)kTrNarrowRows * (F | 1) * 4;   // at most 65 KB
            GbtLdsGuard lds_guard(lds);
            if (lds_guard.needed) {
                Q_HIP(hipFuncSetAttribute((const void *)dense_keys_narrow_kernel,
                                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
            }
            dense_keys_narrow_kernel<<<(unsigned)((n + kTrNarrowRows - 1) / kTrNarrowRows), 256, lds, s>>>(X, n, F,
                                                                                                           keys_a);
        } else if (n > 0) {
            dim3 grid((unsigned)((n + kTrRows - 1) / kTrRows), (unsigned)((F + kTrCols - 1) / kTrCols));
            dense_keys_kernel<<<grid, 256, 0, s>>>(X, n, F, keys_a);
        }
    } else {
        if (F <= kCsrLdsCols) {
            const int W = csr_workgroups(ctx->num_cu, n_values);
            uint32_t *table = (uint32_t *)(ws + L.csr_table);
            const size_t lds = csr_scatter_lds(F);
            GbtLdsGuard lds_guard(lds);
            if (lds_guard.needed)
                Q_HIP(hipFuncSetAttribute((const void *)csr_scatter_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
            csr_count_kernel<<<W, kCsrBlock, (size_t)F * 4, s>>>(indices, n_values, F, table);
            csr_offsets_kernel<<<F, 64, 0, s>>>(table, W, counts);
            offsets_kernel<<<1, 1024, 0, s>>>(counts, F, 0, nullptr, seg_off, blk_off, chk_off, kScanChunk, A.dear);
            csr_scatter_kernel<<<W, kCsrBlock, lds, s>>>(indices, values, n_values, F, seg_off, table, keys_a);
        } else {
            Q_HIP(gbt_launch_fill_u64(s, (uint64_t *)counts, 0, (int64_t)(gbt_align((size_t)F * 4) / 8)));
            Q_HIP(gbt_launch_fill_u64(s, (uint64_t *)cursor, 0, (int64_t)(gbt_align((size_t)F * 4) / 8)));
            const int csr_grid = (int)((n_values + kCsrChunk - 1) / kCsrChunk);
            if (n_values > 0) csr_count_direct_kernel<<<csr_grid, 256, 0, s>>>(indices, n_values, F, counts);
            offsets_kernel<<<1, 1024, 0, s>>>(counts, F, 0, nullptr, seg_off, blk_off, chk_off, kScanChunk, A.dear);
            if (n_values > 0)
                csr_scatter_direct_kernel<<<csr_grid, 256, 0, s>>>(indices, values, n_values, F, seg_off, cursor, keys_a);
        }
    }
    Q_HIP(hipGetLastError());
    // 2. the cuts: by selection where that applies, else (all of them, or the features it leaves) from the sorted segments
    std::vector<int32_t> hnb((size_t)F);
    std::vector<uint32_t> hp((size_t)F);   // values that are not missing
    bool done = false;                     // by selection, every feature: keys_a is as it was made
    const uint32_t *to_sort = nullptr;     // the modes of the features, or all are to be sorted
    if (select) {
        Q_HIP(gbt_launch_select(ctx, keys_a, keys_b, seg_off, blk_off, F, n_values, B, A, cuts, nb, present));
        if (dense && packed) Q_HIP(gbt_launch_bin_table(ctx, F, B, A, cuts, nb));
        uint32_t failed = 0;
        Q_HIP(read_back(ctx, {{&failed, A.flag, 4}, {hnb.data(), nb, (size_t)F * 4}, {hp.data(), present, (size_t)F * 4}}));
        done = failed == 0;
        if (!done) {
            to_sort = A.mode;
            offsets_kernel<<<1, 1024, 0, s>>>(dense ? nullptr : counts, F, dense ? n : 0, to_sort, seg_off, blk_off, chk_off, kScanChunk, nullptr);
        }
    }
    if (!done) {
        uint32_t n_tiles = 0, n_chunks = 0;
        Q_HIP(read_back(ctx, {{&n_tiles, blk_off + F, 4}, {&n_chunks, chk_off + F, 4}}));
        if ((int64_t)n_tiles > L.max_tiles || (int64_t)n_chunks > L.max_chunks) {
            *status = gbt_fail(ctx, GBT_EINVAL, "gbt_quantise: inconsistent input (tile count)");
            return hipSuccess;
        }
        // four stable 8-bit passes between the two key buffers; a segment skips the passes whose digit is the same
        // for all its keys (small integers stored as floats: the low mantissa bytes) and stays where it is
        Q_HIP(gbt_launch_fill_u64(s, (uint64_t *)seg_flags, 0, (int64_t)(gbt_align((size_t)F * 4) / 8)));
        for (int pass = 0; pass < 4 && n_tiles > 0; ++pass) {
            const int shift = pass * 8;
            sort_hist_kernel<<<n_tiles, kSortBlock, 0, s>>>(keys_a, keys_b, seg_flags, seg_off, blk_off, F, shift, tile_hist);
            scan_partial_kernel<<<n_chunks, 256, 0, s>>>(blk_off, chk_off, F, tile_hist, chunk_tot);
            scan_chunks_kernel<<<F, 256, 0, s>>>(chk_off, seg_off, seg_flags, chunk_tot);
            scan_apply_kernel<<<n_chunks, 256, 0, s>>>(blk_off, chk_off, F, tile_hist, chunk_tot);
            sort_scatter_kernel<<<n_tiles, kSortBlock, 0, s>>>(keys_a, keys_b, seg_flags, seg_off, blk_off, F, shift, tile_hist);
            flip_kernel<<<(F + 255) / 256, 256, 0, s>>>(seg_flags, F);
        }
        Q_HIP(hipGetLastError());
        cuts_kernel<<<F, 64, 0, s>>>(keys_a, keys_b, seg_flags, seg_off, to_sort, F, B, cuts, nb, present);
        Q_HIP(hipGetLastError());
        Q_HIP(read_back(ctx, {{hnb.data(), nb, (size_t)F * 4}, {hp.data(), present, (size_t)F * 4}}));
    }
    int32_t miss = 1;
    for (int f = 0; f < F; ++f) miss = hnb[f] > miss ? hnb[f] : miss;
    if (miss > 65535) {
        *status = gbt_fail(ctx, GBT_EUNSUPPORTED, "gbt_quantise: %d bins do not fit a 16-bit symbol", miss);
        return hipSuccess;
    }

    if (packed) {
        // 3b. symbols straight into the bit stream.  Its width follows from the largest symbol, which is known
        //     without binning: the largest present value of a feature falls into its last bin, and the missing
        //     symbol (max_f nb[f]) occurs iff some element has no value.
        uint64_t tot = 0;
        for (int f = 0; f < F; ++f) tot += hp[f];
        bool any_missing = tot < (uint64_t)n * (uint64_t)F;
        if (!dense && !any_missing && n > 0) {   // as many values as elements; a row may still have fewer than F (and another more)
            Q_HIP(gbt_launch_fill_u64(s, (uint64_t *)misc, 0, 1));
            csr_any_missing_kernel<<<grid_for(n > n_values ? n : n_values, 256 * 8, 4096), 256, 0, s>>>(
                indptr, values, n, n_values, F, misc);
            Q_HIP(hipGetLastError());
            uint32_t fl = 0;
            Q_HIP(read_back(ctx, {{&fl, misc, 4}}));
            any_missing = fl != 0;
        }
        const int32_t mx = n == 0 ? 0 : (any_missing ? miss : miss - 1);
        const int bits = gbt_bits((uint32_t)mx);
        if (bits > GBT_MAX_BITS) {
            *status = gbt_fail(ctx, GBT_EUNSUPPORTED, "gbt_quantise_packed: symbols need %d bits", bits);
            return hipSuccess;
        }
        const int64_t n_words = gbt_packed_words(n, F, bits);
        if (n_words > packed_cap_words) {
            *status = gbt_fail(ctx, GBT_ENOMEM, "gbt_quantise_packed: %lld words needed for %d-bit symbols, %lld given",
                               (long long)n_words, bits, (long long)packed_cap_words);
            return hipSuccess;
        }
        const int64_t n_elems = n * (int64_t)F;
        if (dense && done && gbt_bin_columns_ok(n, F, bits)) {
            Q_HIP(gbt_launch_bin_columns(ctx, keys_a, keys_b, seg_off, blk_off, n, F, B, A, cuts, nb, (uint32_t)miss, bits,
                                         packed, n_words));
        } else if (dense) {
            const size_t cut_bytes = ((size_t)F * (B - 1) + (size_t)F) * 4;
            const int grid = grid_for(n_elems, kPackTile, 8192);
            if (cut_bytes <= 48u * 1024u)
                bin_pack_dense_kernel<true><<<grid, 256, cut_bytes, s>>>(X, n_elems, F, B, cuts, nb, (uint32_t)miss, bits,
                                                                         packed, n_words);
            else
                bin_pack_dense_kernel<false><<<grid, 256, 0, s>>>(X, n_elems, F, B, cuts, nb, (uint32_t)miss, bits,
                                                                  packed, n_words);
        } else {
            int tile_rows = 256;
            while (tile_rows >= 32 && (size_t)tile_rows * F * 2 + 8 + ((size_t)tile_rows + 1) * 8 > 48u * 1024u) tile_rows -= 32;
            if (tile_rows < 32) {
                *status = gbt_fail(ctx, GBT_EUNSUPPORTED, "gbt_quantise_packed: CSR rows of %d features do not fit the "
                                   "packing tile; use gbt_quantise and gbt_compress", F);
                return hipSuccess;
            }
            // the cuts kept in LDS, a power of two less one per feature: at most 56 KB of them
            int cut_log = 0, step0 = 1;
            auto steps_of = [&](int cl) {
                int st = 1;
                while (2 * st - 1 < (B - 1) >> cl) st *= 2;
                return st;
            };
            for (;; ++cut_log) {
                step0 = steps_of(cut_log);
                if (step0 == 1 || (size_t)F * (2 * step0 - 1) * 4 <= 56u * 1024u) break;
            }
            int log_lanes = 0;   // lanes per row: at least a row's average number of entries, where that is below 64
            while (log_lanes < 6 && ((int64_t)n << log_lanes) < n_values) ++log_lanes;
            const size_t lds = (size_t)tile_rows * F * 2 + (size_t)F * (2 * step0 - 1) * 4 + (size_t)F * 4 + ((size_t)tile_rows + 1) * 4;
            Q_HIP(with_bits(bits, [&](auto bc) {
                constexpr int BITS = decltype(bc)::value;
                const auto fn = F > (4 << log_lanes) ? bin_pack_csr_kernel<BITS, true> : bin_pack_csr_kernel<BITS, false>;
                GbtLdsGuard lds_guard(lds);
                if (lds_guard.needed) {
                    hipError_t e = hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
                    if (e != hipSuccess) return e;
                }
                fn<<<grid_for(n, tile_rows, 2 * ctx->num_cu), kCsrPackBlock, lds, s>>>(
                    indptr, indices, values, n, n_values, F, B, cuts, nb, (uint32_t)miss, tile_rows, log_lanes, cut_log, step0,
                    packed, n_words);
                return hipGetLastError();
            }));
        }
        Q_HIP(hipGetLastError());
        Q_HIP(hipStreamSynchronize(s));
        *max_value = mx;
        *missing_sym = miss;
        *bits_out = bits;
        return hipSuccess;
    }

    // 3. symbols
    Q_HIP(gbt_launch_fill_u64(s, (uint64_t *)misc, 0, 1));
    if (n > 0) {
        if (dense) {
            const size_t cut_bytes = ((size_t)F * (B - 1) + (size_t)F) * 4;
            if (cut_bytes <= 60u * 1024u) {
                GbtLdsGuard lds_guard(cut_bytes);
                if (lds_guard.needed) {
                    Q_HIP(hipFuncSetAttribute((const void *)bin_dense_kernel<true>,
                                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)cut_bytes));
                }
                bin_dense_kernel<true><<<grid_for(n * (int64_t)F, 4096, 8192), 256, cut_bytes, s>>>(
                    X, n * (int64_t)F, F, B, cuts, nb, (uint32_t)miss, sym, misc);
            } else {
                bin_dense_kernel<false><<<grid_for(n * (int64_t)F, 1024, 16384), 256, 0, s>>>(
                    X, n * (int64_t)F, F, B, cuts, nb, (uint32_t)miss, sym, misc);
            }
        } else {
            fill_u16_kernel<<<grid_for(n * (int64_t)F, 2048, 16384), 256, 0, s>>>(sym, (uint16_t)miss,
                                                                                   n * (int64_t)F);
            bin_csr_kernel<<<grid_for(n, 256, 16384), 256, 0, s>>>(indptr, indices, values, n, n_values, F, B, cuts,
                                                                   nb, (uint32_t)miss, sym, misc);
        }
    }
    Q_HIP(hipGetLastError());
    Q_HIP(hipMemcpyAsync(ctx->pinned + GBT_STAGING_BYTES / 2, misc, 4, hipMemcpyDeviceToHost, s));
    Q_HIP(hipStreamSynchronize(s));
    uint32_t mx;
    memcpy(&mx, ctx->pinned + GBT_STAGING_BYTES / 2, 4);
    *max_value = (int32_t)mx;
    *missing_sym = miss;
    return hipSuccess;
}
