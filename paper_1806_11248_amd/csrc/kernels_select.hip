// Exact order statistics of every feature (Sec. 2.1) by selection instead of a sort.
//
// B - 1 cuts need B order statistics of a feature (or, with at most B distinct values, those values), not its sorted
// values.  A segment of keys (quantise_common.h) is read twice:
//
//   sample   4096 keys of the segment, sorted in LDS, say where its values lie: the key space is divided into cells,
//            every interval of equal top 11 bits into 2^j equal ones with j by the interval's share of the sample (up to
//            8192 cells for all of them, at least one each): the cell of a key is one table read, a shift and an add;
//   count    first reading: keys per cell, in LDS, one workgroup per run of tiles.  In a column of few distinct values
//            (by the sample) a cell also keeps one of its keys and whether it has met another;
//   pick     the cells that hold a wanted rank (or every non-empty cell, where those are no more than B): a slot each;
//   collect  second reading: the keys of those cells, some 5 % of the segment.  A key that the sample shows to be
//            frequent in its cell is counted by difference and not collected; a column of categories, each in a cell
//            of its own, is not read again at all;
//   distinct, order  the slots' keys sorted, counted or marked in LDS, and the statistics read off;
//   cuts     statistics thinned to strictly increasing cuts.
//
// A column whose values lie so close together that one workgroup would have to read much of it is left to the sort (mode
// kSelSorted): by its sample as a rule, else as soon as distinct or order meets such a cell.
//
// Bound, 115M x 13 of which 8 are categories (a kernel that only reads gets 5.9 TB/s): count reads 6 GB at 3.5 TB/s, held up by
// LDS (conflicts of the counters on 40 % of a compute unit's cycles); collect reads 2.3 GB at 2.0 TB/s, its waves waiting three
// quarters of their time (98 scalar registers leave one workgroup on a compute unit, with two barriers a step).
// The sort it replaces (four 8-bit digits) reads and writes every key up to four times.  115M x 13: sort and cuts 24.6 ms, selection 3.2 ms (count 1.7, collect 1.15); 10M x 50 rows of 10 entries: 2.6 and
// 0.45 ms; 500K x 800 columns of 64 bins: 1.6 ms.
//
// A dense matrix is then binned column by column from the same keys with the same cells (most cells hold no cut: one
// table read gives the symbol) and packed from the columns: 115M x 13 3.76 -> 2.8 ms, 500K x 800 8.1 -> 1.3 ms against
// a bisection over each element's cuts.
#include "gbt_internal.h"
#include "quantise_common.h"

#include <algorithm>

namespace {

constexpr int kSelBlock = 1024;
constexpr int kSegBits = 11, kSegs = 1 << kSegBits, kSegShift = 32 - kSegBits;
constexpr int kSelBinsMax = 1024;
constexpr int kCellsMax = 16384, kSampleMax = 4096;
constexpr uint32_t kDiscreteCells = 4096;   // at most, of a discrete feature
constexpr int kSmallSlot = 256;        // collected keys up to which a wave ranks a slot by comparing all with all
constexpr int kMidSlot = 8192;         // ... and up to which a workgroup of 256 threads takes one
constexpr int kMidBits = 12, kBigBits = 14;   // counters of those workgroups (16 and 64 KB of LDS)
constexpr int kMarkBits = 19;          // bits of the mark table (64 KB of LDS)
constexpr uint32_t kKindDiscrete = 1, kKindNoCollect = 2;   // bits of SelArrays::kind
constexpr int kKindHotShift = 8;       // above: 1 + where a discrete feature's frequent key stands in the sample (0: there is none)
constexpr uint16_t kNoSlot = 0xffff;

// Exclusive prefix sum over the workgroup's threads; *total receives the sum.  tmp: one word per wave.
__device__ inline uint32_t block_scan(uint32_t x, uint32_t *tmp, uint32_t *total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    uint32_t s = x;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)s, o);
        if (lane >= o) s += y;
    }
    __syncthreads();   // the words of the scan before are read
    if (lane == 63) tmp[wave] = s;
    __syncthreads();
    uint32_t before = 0, all = 0;
    for (int w = 0; w < waves; ++w) {
        before += w < wave ? tmp[w] : 0u;
        all += tmp[w];
    }
    *total = all;
    return before + s - x;
}

__device__ inline uint32_t cell_of(const uint32_t *seg, uint32_t key) {
    const uint32_t t = seg[key >> kSegShift];
    return (t & 0xffffffu) + ((key & ((1u << kSegShift) - 1u)) >> (t >> 24));
}

// LDS words that lanes of one wave exchange: what was written before is there to be read behind it.
__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Key reads that one workgroup may spend on a feature's distinct values or on one slot; beyond it the feature is sorted.  A
// workgroup reads 2 to 3 keys per ns where they are few distinct ones, which meet on few LDS words (9M collected keys of 108
// values: 3.1 ms), or come from HBM; 4 to 6 where the whole matrix's keys fit the 256 MB cache (kCachedKeys).  The sort takes
// about 0.5 ms of launches and 16 ns per 1000 keys, of all features that go there together; the workgroups work side by
// side.  So the limit follows from `dear`, the keys of all features that would be sorted for their own sake: 8 columns of
// 10M dates in 64 bins, 1.3 ms, sorted 2.1; 30 columns of 3M narrow normals in 16 bins, 1.6 and 2.3.
constexpr uint64_t kCachedKeys = 1ull << 25;
// Tiles per workgroup of the count from which on (`many`) frequent keys are looked for and runs are of equal work: 3 and 1 us of the
// sample kernel, which 0.6M keys (the call 220 us) do not gain back.  The host says so: kernels that look up the number of keys wait
// for it (20,000 x 13, categories and numbers, collect 8.7 us and so 8.4).
constexpr int64_t kManyTiles = 8;
__device__ inline uint64_t work_limit(uint64_t tuned, const uint64_t *seg_off, int F, int f, uint64_t dear, bool discrete) {
    const uint64_t len = seg_off[f + 1] - seg_off[f], reads = (1ull << 20) + (len > dear ? len : dear) / 32;
    return tuned ? tuned : discrete || seg_off[F] > kCachedKeys ? reads : reads * 5 / 2;
}
constexpr uint32_t kSlotReads = 12u << 10;   // what a slot costs sel_distinct_kernel beside its keys (100 slots: 0.45 ms)

// Bits of the first count of sel_order_kernel<*, most> over a slot of L collected keys: counters for twice the keys, and no
// more bits left than a second count takes.
__device__ inline int order_bits(uint32_t L, int shift, int most) {
    int nb = 33 - __builtin_clz(L | 1u);
    nb = nb < kSegShift - most ? kSegShift - most : nb > most ? most : nb;
    return nb > shift ? shift : nb;
}

// The first k with floor(k m / B) >= rank.
__device__ inline uint64_t first_k(uint64_t rank, uint64_t m, uint32_t B) { return (rank * B + m - 1) / m; }

// ---- sample ---------------------------------------------------------------------------------------------------
// One workgroup per feature: 4096 keys at jittered even steps, sorted (bitonic), then the cells.  Also clears the cell
// counts, and says which features are to be sorted: where values lie so close together that many share a cell (months as
// 201501.0, dates, ids above 10^7: a cell is never less than 128 neighbouring floats, and 2048 in a discrete feature), one
// workgroup would read most of the column in sel_distinct_kernel or sel_order_kernel.
// One column of 10M such months, the whole call: 0.78 ms sorted, 3.34 by selection, 0.85 with this.  The look at the sample
// takes 3 us of the kernel's 47.
template <typename Less>
__device__ inline int sample_bound(const uint32_t *v, int lo, int hi, Less &&less) {   // first j in [lo, hi) without less(v[j])
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (less(v[mid])) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// (With 80 scalar registers or fewer two workgroups fit a compute unit: 512 columns of 30,000 in 72 us, with 88 in 96.)
__global__ __launch_bounds__(kSelBlock) __attribute__((amdgpu_num_sgpr(80))) void sel_sample_kernel(
    const uint32_t *__restrict__ keys, const uint64_t *__restrict__ seg_off, int B, SelArrays A, uint64_t work_tuned, bool many) {
    __shared__ uint32_t v[kSampleMax];
    __shared__ uint32_t per_seg[kSegs];   // sampled keys of an interval, then its first cell and shift
    __shared__ uint64_t heads[kSampleMax / 64];   // bits: a cell's first sampled key
    __shared__ uint32_t tmp[kSelBlock / 64];
    __shared__ uint32_t n_mixed, sum_other;     // cells of several values, and their sampled keys besides the frequent one
    __shared__ uint32_t max_other, max_order;   // the dearest cell: such keys, and key reads of sel_order_kernel
    __shared__ uint32_t longest;                // the most frequent key: how often << 12 | where (discrete features)
    static_assert(kSampleMax <= 1 << 12, "a place in the sample has 12 bits");
    const int f = blockIdx.x, tid = threadIdx.x;
    const uint64_t len = seg_off[f + 1] - seg_off[f];
    const uint32_t *p = keys + seg_off[f];
    const int S = (int)(len < (uint64_t)A.sample_cap ? len : (uint64_t)A.sample_cap);
    int P = 64;
    while (P < S) P <<= 1;
    for (int j = tid; j < P; j += kSelBlock) {
        uint32_t k = kMissingKey;
        if (j < S) {
            const uint64_t a = len * (uint64_t)j / (uint64_t)S, b = len * (uint64_t)(j + 1) / (uint64_t)S;
            uint32_t h = (uint32_t)j * 2654435761u + (uint32_t)f * 40503u;
            h = (h ^ (h >> 15)) * 2246822519u;
            h ^= h >> 13;
            k = p[a + (uint64_t)h % (b - a)];   // (b > a: S <= len)
        }
        v[j] = k;
    }
    for (int i = tid; i < kSegs; i += kSelBlock) per_seg[i] = 0;
    __syncthreads();
    for (int size = 2; size <= P; size <<= 1)
        for (int d = size >> 1; d > 0; d >>= 1) {
            for (int i = tid; i < P / 2; i += kSelBlock) {
                const int lo = ((i & ~(d - 1)) << 1) | (i & (d - 1)), hi = lo + d;
                const bool up = (lo & size) == 0;
                const uint32_t x = v[lo], y = v[hi];
                if ((x > y) == up) {
                    v[lo] = y;
                    v[hi] = x;
                }
            }
            // (with d <= 64 the 64 comparisons of a wave stay inside 128 words of its own)
            if (d > 64 || (d == 1 && size >= 128)) __syncthreads(); else wave_sync();
        }
    __syncthreads();
    uint32_t mine = 0, fresh = 0;
    for (int j = tid; j < A.sample_cap; j += kSelBlock) {
        const uint32_t k = j < P ? v[j] : kMissingKey;
        if (k != kMissingKey) {
            atomicAdd(&per_seg[k >> kSegShift], 1u);
            ++mine;
            fresh += j == 0 || v[j - 1] != k ? 1u : 0u;
        }
    }
    uint32_t present, distinct;
    block_scan(mine, tmp, &present);   // (and a barrier behind the counts)
    block_scan(fresh, tmp, &distinct);
    __syncthreads();
    // Few distinct keys, seen eight times each on average: a coarser division separates them (and leaves LDS for more
    // than one copy of the counters, which such a column needs: its keys meet on few addresses).
    const bool discrete = distinct * 8 <= present && present > 0;
    // cells per interval: at least 2^least where the sample has seen the interval, as fine as fits `cap`
    const uint32_t budget = discrete ? kDiscreteCells / 4 : (uint32_t)A.cap / 2, limit = discrete ? kDiscreteCells : (uint32_t)A.cap;
    uint32_t first = 0, total = 0;
    int bits[kSegs / kSelBlock];
    static_assert(kSegs % kSelBlock == 0, "a whole number of intervals per thread");
    constexpr int PER = kSegs / kSelBlock;
    for (int least = 6; least >= 0; --least) {
        uint32_t sum = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const uint32_t c = per_seg[tid * PER + i];
            const uint32_t want = c ? (uint32_t)((uint64_t)c * budget / present) : 0u;
            int b = want > 0 ? 31 - __builtin_clz(want) : 0;
            if (c && b < least) b = least;
            bits[i] = b;
            sum += 1u << b;
        }
        first = block_scan(sum, tmp, &total);
        if (total <= limit) break;   // with least = 0 the sum is at most budget + kSegs <= limit
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        per_seg[tid * PER + i] = first | ((uint32_t)(kSegShift - bits[i]) << 24);
        first += 1u << bits[i];
    }
    if (tid == 0) n_mixed = sum_other = max_other = max_order = longest = 0;
    __syncthreads();
    uint32_t *rep = A.rep + (uint64_t)f * kDiscreteCells;
    if (discrete)
        for (uint32_t c = tid; c < total; c += kSelBlock) rep[c] = kMissingKey;
    // The cells of the sampled keys, which are neighbours in v.  (Cells are aligned: keys of one share their top bits.)
    for (int j = tid; j < P; j += kSelBlock) {   // (P is a multiple of 64: a wave takes a whole word)
        const uint32_t k = v[j], shift = per_seg[k >> kSegShift] >> 24;
        const uint64_t m = __ballot(k != kMissingKey && (j == 0 || v[j - 1] >> shift != k >> shift));
        if ((tid & 63) == 0) heads[j >> 6] = m;
    }
    __syncthreads();   // (and `rep` is clear)
    if (discrete && many)
        for (int j = tid; j < (int)present; j += kSelBlock) {
            const uint32_t k = v[j];
            if (j > 0 && v[j - 1] == k) continue;
            const int end = sample_bound(v, j, (int)present, [&](uint32_t x) { return x <= k; });
            atomicMax(&longest, (uint32_t)(end - j) << 12 | (uint32_t)j);
        }
    uint32_t used = (tid & 63) < P / 64 ? (uint32_t)__popcll(heads[tid & 63]) : 0u;   // every wave adds them up
    for (int o = 32; o > 0; o >>= 1) used += (uint32_t)__shfl_xor((int)used, o);
    // What the feature would cost.  In no more cells than bins the distinct values are counted by one workgroup; otherwise a
    // workgroup takes a cell, and only one with a share of the feature that shows in S / 128 sampled keys can be dear.
    const int least_keys = used > (uint32_t)B ? S / 128 : 2;
    const float per_key = (float)len / (float)(S > 0 ? S : 1), per_rank = (float)B / (float)(present > 0 ? present : 1);
    for (int j = tid; j < P; j += kSelBlock) {
        if (!((heads[j >> 6] >> (j & 63)) & 1u)) continue;
        const uint32_t k = v[j], shift = per_seg[k >> kSegShift] >> 24, same = k >> shift;
        uint32_t mid = k;
        const int quick = j + (least_keys > 2 ? least_keys : 2) - 1;
        if (quick < P && v[quick] >> shift == same) {
            int w = j >> 6, end = (int)present;   // the next cell's first key, in this word or one of the next three, or bisected
            uint64_t m = heads[w] & (~1ull << (j & 63));
            for (int i = 0; i < 3 && !m && w + 1 < P / 64; ++i) m = heads[++w];
            if (m) {
                end = 64 * w + (int)__builtin_ctzll(m);
            } else if (64 * (w + 1) < (int)present) {
                end = sample_bound(v, 64 * (w + 1), (int)present, [&](uint32_t x) { return x >> shift == same; });
            }
            if (v[end - 1] != k) {
                mid = v[(j + end) >> 1];   // the frequent key, if there is one: not collected
                const int m0 = sample_bound(v, j, end, [&](uint32_t x) { return x < mid; });
                const int m1 = sample_bound(v, m0, end, [&](uint32_t x) { return x <= mid; });
                const uint32_t other = (uint32_t)(end - j - (m1 - m0));
                const uint32_t reads = shift > (uint32_t)kMarkBits ? other << (shift - kMarkBits) : other;
                atomicAdd(&n_mixed, 1u);
                atomicAdd(&sum_other, reads);
                atomicMax(&max_other, reads);
                const float L = per_key * (float)other;
                const int rest = (int)shift - order_bits(L < 2e9f ? (uint32_t)L : 2000000000u, (int)shift, kBigBits);
                const float cost = rest > 0 ? L * (2.0f + (float)(end - j) * per_rank) : L;
                atomicMax(&max_order, cost < 4e9f ? (uint32_t)cost : 4000000000u);
            }
        }
        if (discrete) rep[cell_of(per_seg, k)] = mid;
    }
    __syncthreads();
    if (tid == 0) {
        float cost = (float)max_order;
        if (used <= (uint32_t)B) {
            const float all = per_key * (float)sum_other + (float)n_mixed * (float)kSlotReads;
            if (distinct > (uint32_t)B) {   // it stops behind the slot that brings the one value too many
                const float part = all * (float)B / (float)distinct + per_key * (float)max_other;
                cost += part < all ? part : all;
            } else {
                cost = all;
            }
        }
        const uint32_t hot = (longest >> 12) * 8u >= present ? (longest & 4095u) + 1u : 0u;
        A.kind[f] = discrete ? kKindDiscrete | hot << kKindHotShift : 0u;
        A.cost[f] = cost < 4e9f ? (uint32_t)cost : 4000000000u;
        const bool dear = A.cost[f] > work_limit(work_tuned, seg_off, gridDim.x, f, 0, discrete);
        if (dear) atomicAdd(A.dear, (unsigned long long)len);
        if (many) atomicOr(&A.mix[0], (discrete ? 2u : 1u) | (dear ? 4u : 0u));
        A.n_cells[f] = total;
    }
    // what the next kernels read (behind the last barrier: none waits for these stores)
    for (int j = tid; j < A.sample_cap; j += kSelBlock) A.sample[(uint64_t)f * A.sample_cap + j] = j < P ? v[j] : kMissingKey;
    for (int i = tid; i < kSegs; i += kSelBlock) A.seg[(uint64_t)f * kSegs + i] = per_seg[i];
    for (uint32_t c = tid; c < total; c += kSelBlock) A.counts[(uint64_t)f * A.cap + c] = 0;
    if (discrete)
        for (uint32_t c = tid; c < total; c += kSelBlock) A.mixed[(uint64_t)f * kDiscreteCells + c] = 0;
    if (f == 0 && tid == 0) {   // (*A.dear and A.mix are cleared with the offsets: this kernel adds to them)
        A.n_work[0] = A.n_work[1] = A.n_work[2] = 0;
        A.flag[0] = 0;
    }
}

// ---- count ------------------------------------------------------------------------------------------------------
typedef uint32_t sel_u32x4 __attribute__((ext_vector_type(4), aligned(4)));   // a segment starts at any word

// Workgroup b of the grid takes a run of tiles, whatever features they belong to: an equal one, or one of equal work where a
// feature's tiles weigh what the kernel says (0: nothing to do there).  A table of 115M rows with 8 columns of categories and 5
// of numbers, equal runs and runs of equal work: count 1.69 and 1.46 ms, collect 1.14 and 0.89, the whole call 7.96 and 7.41.
// The shares cost 7 us a launch, so not where all features are of one kind (`mix`, a bit per kind, left empty where there are
// fewer than kManyTiles); and up to a feature per thread.
struct TileShares {
    uint32_t tmp[kSelBlock / 64], edge[2];
    int first;
    unsigned long long active[kSelBlock / 64];   // bits: features of any weight
};
struct TileRun {
    uint32_t t, end;
    int f;
    const unsigned long long *active = nullptr;   // NULL: every feature
    __device__ TileRun(const uint32_t *blk_off, int F) { equal(blk_off, F); }
    template <typename Weight>
    __device__ TileRun(const uint32_t *blk_off, int F, uint32_t mix, TileShares *sh, Weight &&weight) {
        const uint32_t nt = blk_off[F];
        if ((mix & (mix - 1u)) == 0u || F > kSelBlock) {
            equal(blk_off, F);
            return;
        }
        const int me = (int)threadIdx.x;
        const uint32_t w = me < F ? weight(me) : 0u, t0 = me < F ? blk_off[me] : 0u;
        const uint32_t work = w ? w * (blk_off[me + 1] - t0) : 0u;
        const unsigned long long m = __ballot(work != 0u);
        if ((me & 63) == 0) sh->active[me >> 6] = m;
        if (me == 0) sh->edge[0] = sh->edge[1] = nt;
        uint32_t total;
        const uint32_t before = block_scan(work, sh->tmp, &total);
        for (int k = 0; k < 2; ++k) {
            const uint32_t p = (uint32_t)((uint64_t)total * (blockIdx.x + k) / gridDim.x);
            if (p >= before && p - before < work) {   // one thread, or none behind the last tile
                sh->edge[k] = t0 + (p - before) / w;
                if (k == 0) sh->first = me;
            }
        }
        __syncthreads();
        t = sh->edge[0];
        end = sh->edge[1];
        f = t < end ? sh->first : 0;
        active = sh->active;
    }
    __device__ void equal(const uint32_t *blk_off, int F) {
        const uint64_t nt = blk_off[F];
        t = (uint32_t)(nt * blockIdx.x / gridDim.x);
        end = (uint32_t)(nt * (blockIdx.x + 1) / gridDim.x);
        f = t < end ? find_segment(blk_off, F, t) : 0;
    }
    // the next piece of one segment: keys [k0, k1) of segment f; false: none left
    __device__ bool next(const uint32_t *blk_off, const uint64_t *seg_off, uint64_t *k0, uint64_t *k1) {
        if (t >= end) return false;
        if (active && blk_off[f + 1] <= t) {
            int i = (f + 1) >> 6;
            if (i >= kSelBlock / 64) return false;
            unsigned long long m = active[i] & (~0ull << ((f + 1) & 63));
            while (!m && ++i < kSelBlock / 64) m = active[i];
            if (!m) return false;
            f = 64 * i + (int)__builtin_ctzll(m);
            t = blk_off[f] > t ? blk_off[f] : t;
            if (t >= end) return false;
        }
        while (blk_off[f + 1] <= t) ++f;
        const uint32_t te = end < blk_off[f + 1] ? end : blk_off[f + 1];
        const uint64_t len = seg_off[f + 1] - seg_off[f];
        *k0 = (uint64_t)(t - blk_off[f]) * kSortTile;
        *k1 = (uint64_t)(te - blk_off[f]) * kSortTile;
        if (*k1 > len) *k1 = len;
        t = te;
        return true;
    }
};

// every key of a piece of a segment, four 16-byte loads in flight per thread
template <typename Fn>
__device__ inline void for_each_key(const uint32_t *p, uint64_t k0, uint64_t k1, Fn &&fn) {
    constexpr uint64_t STEP = 4ull * kSelBlock;
    uint64_t i = k0 + 4ull * threadIdx.x;
    for (; i + 3 * STEP + 4 <= k1; i += 4 * STEP) {
        sel_u32x4 q[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) q[j] = *(const sel_u32x4 *)(p + i + j * STEP);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c) fn(q[j][c]);
    }
    for (; i < k1; i += STEP)
        for (int c = 0; c < 4; ++c)
            if (i + c < k1) fn(p[i + c]);
}

// (80 scalar registers: as for sel_sample_kernel.  1M x 28, 34.4 us, with 89 38.4.)
__global__ __launch_bounds__(kSelBlock) __attribute__((amdgpu_num_sgpr(80))) void sel_count_kernel(const uint32_t *__restrict__ keys,
                                                              const uint64_t *__restrict__ seg_off,
                                                              const uint32_t *__restrict__ blk_off, int F, SelArrays A,
                                                              uint64_t work_tuned, bool many) {
    extern __shared__ uint32_t cnt[];   // cap words: the counters, as many copies as fit (a lane adds to one of them);
                                        // a discrete feature's keys and marks in front of them
    __shared__ uint32_t seg[kSegs];
    __shared__ TileShares shares;
    // (a discrete feature's key: one more read, and lanes that meet on few counters)
    TileRun run(blk_off, F, many ? A.mix[0] : 0u, &shares, [&](int f) __attribute__((always_inline)) -> uint32_t {
        const bool discrete = A.kind[f] & kKindDiscrete;
        return A.cost[f] > work_limit(work_tuned, seg_off, F, f, *A.dear, discrete) ? 0u : discrete ? 3u : 2u;
    });
    uint64_t k0, k1;
    while (run.next(blk_off, seg_off, &k0, &k1)) {
        const int f = run.f;
        const uint32_t nc = A.n_cells[f], kind = A.kind[f];
        const bool discrete = kind & kKindDiscrete;
        if (A.cost[f] > work_limit(work_tuned, seg_off, F, f, *A.dear, discrete)) continue;
        uint32_t *rep = cnt, *counters = discrete ? cnt + nc : cnt;   // rep: key of a cell
        uint32_t copies = ((uint32_t)A.cap - (discrete ? nc : 0u)) / nc;
        copies = copies < 1 ? 1 : copies > 8 ? 8 : copies;
        __syncthreads();   // the piece before has been merged
        for (int i = threadIdx.x; i < kSegs; i += kSelBlock) seg[i] = A.seg[(uint64_t)f * kSegs + i];
        for (uint32_t i = threadIdx.x; i < nc * copies; i += kSelBlock) counters[i] = 0;
        if (discrete)
            for (uint32_t i = threadIdx.x; i < nc; i += kSelBlock) rep[i] = A.rep[(uint64_t)f * kDiscreteCells + i];
        __syncthreads();
        const uint32_t *p = keys + seg_off[f];
        uint32_t *mine = counters + (threadIdx.x % copies) * nc;
        if (discrete) {
            uint8_t *mixed = A.mixed + (uint64_t)f * kDiscreteCells;
            auto add = [&](uint32_t k, uint32_t times) __attribute__((always_inline)) {
                const uint32_t c = cell_of(seg, k);
                uint32_t r = rep[c];
                if (r != k) {
                    if (r == kMissingKey) r = atomicCAS(&rep[c], kMissingKey, k);
                    if (r != kMissingKey && r != k) mixed[c] = 1;   // (any thread, any number of times)
                }
                atomicAdd(&mine[c], times);
            };
            // The frequent key (none: kMissingKey) is counted in a register: lanes that hold it would take turns on one counter.  The
            // table of TileRun, count: 1.46 ms without, 1.32 with it.  An eighth of the sample: below it few lanes of a copy meet.
            const uint32_t at = kind >> kKindHotShift, hot = at ? A.sample[(uint64_t)f * A.sample_cap + at - 1u] : kMissingKey;
            uint32_t times = 0;
            for_each_key(p, k0, k1, [&](uint32_t k) {
                if (k == hot) ++times;
                else if (k != kMissingKey) add(k, 1u);
            });
            if (hot != kMissingKey) {
                for (int o = 32; o > 0; o >>= 1) times += (uint32_t)__shfl_xor((int)times, o);
                if ((threadIdx.x & 63) == 0 && times) add(hot, times);
            }
        } else {
            for_each_key(p, k0, k1, [&](uint32_t k) {
                if (k != kMissingKey) atomicAdd(&mine[cell_of(seg, k)], 1u);
            });
        }
        __syncthreads();
        for (uint32_t c = threadIdx.x; c < nc; c += kSelBlock) {
            uint32_t sum = 0;
            for (uint32_t j = 0; j < copies; ++j) sum += counters[j * nc + c];
            if (!sum) continue;
            atomicAdd(&A.counts[(uint64_t)f * A.cap + c], sum);
            if (discrete) {   // the workgroups' keys of a cell have to agree
                const uint32_t r = atomicCAS(&A.rep[(uint64_t)f * kDiscreteCells + c], kMissingKey, rep[c]);
                if (r != kMissingKey && r != rep[c]) A.mixed[(uint64_t)f * kDiscreteCells + c] = 1;
            }
        }
    }
}

// ---- pick -------------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kSelBlock) void sel_pick_kernel(const uint64_t *__restrict__ seg_off, SelArrays A, int B,
                                                             uint32_t *__restrict__ present, uint64_t work_tuned, bool many) {
    __shared__ uint32_t seg[kSegs];
    __shared__ uint32_t cell[kSelBinsMax];   // of a slot
    __shared__ uint32_t tmp[kSelBlock / 64];
    const int f = blockIdx.x, tid = threadIdx.x;
    if (A.cost[f] > work_limit(work_tuned, seg_off, gridDim.x, f, *A.dear, A.kind[f] & kKindDiscrete)) {
        if (tid == 0) {
            A.n_slots[f] = 0;
            A.mode[f] = kSelSorted;
            A.flag[0] = 1;
            if (many) atomicOr(&A.mix[1], 2u);
        }
        return;
    }
    const uint32_t nc = A.n_cells[f];
    constexpr int PER = kCellsMax / kSelBlock;
    for (int i = tid; i < kSegs; i += kSelBlock) seg[i] = A.seg[(uint64_t)f * kSegs + i];
    uint32_t c[PER], sum = 0, ne = 0;
    const uint32_t per = (nc + kSelBlock - 1) / kSelBlock, c0 = tid * per;
    const uint32_t *cn = A.counts + (uint64_t)f * A.cap;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        c[i] = (uint32_t)i < per && c0 + i < nc ? cn[c0 + i] : 0u;
        sum += c[i];
        ne += c[i] ? 1u : 0u;
    }
    uint32_t m, n_used;
    const uint32_t start0 = block_scan(sum, tmp, &m);
    block_scan(ne, tmp, &n_used);
    const bool order = n_used > (uint32_t)B, discrete = A.kind[f] & kKindDiscrete;
    bool collect = !discrete;
    // which cells: those with a wanted rank, or all that hold anything
    uint32_t sel = 0, n_sel = 0, sel_keys = 0, start = start0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        if (c[i]) {
            bool want = true;
            if (order) {
                const uint64_t k = first_k(start, m, (uint32_t)B);
                want = k < (uint64_t)B && k * m / (uint64_t)B < (uint64_t)start + c[i];
            }
            if (want) {
                sel |= 1u << i;
                ++n_sel;
                sel_keys += c[i];
            }
            start += c[i];
        }
    }
    uint32_t n_slots, n_keys;
    uint32_t slot = block_scan(n_sel, tmp, &n_slots);
    uint32_t off = block_scan(sel_keys, tmp, &n_keys);
    (void)n_keys;
    start = start0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        if ((uint32_t)i < per && c0 + i < nc) {
            const bool on = (sel >> i) & 1u;
            A.slot_of[(uint64_t)f * A.cap + c0 + i] = on ? (uint16_t)slot : kNoSlot;
            if (on) {
                SelSlot s;
                s.start = start;
                s.cnt = c[i];
                s.off = off;
                s.heavy = s.key_lo = s.shift = 0;
                A.slots[(uint64_t)f * B + slot] = s;
                A.cursor[(uint64_t)f * B + slot] = 0;
                cell[slot] = c0 + i;
                ++slot;
                off += c[i];
            }
            start += c[i];
        }
    }
    __syncthreads();
    // a thread per slot: where its cell lies, and the key that is not collected
    const uint32_t *sample = A.sample + (uint64_t)f * A.sample_cap;
    for (uint32_t s = tid; s < n_slots; s += kSelBlock) {
        const uint32_t ci = cell[s];
        int lo = 0, hi = kSegs;   // the interval of the cell: the last one that starts at or before it
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if ((seg[mid] & 0xffffffu) <= ci) lo = mid; else hi = mid;
        }
        const uint32_t shift = seg[lo] >> 24, key_lo = ((uint32_t)lo << kSegShift) + ((ci - (seg[lo] & 0xffffffu)) << shift);
        uint32_t heavy = kMissingKey;
        if (discrete) {
            heavy = A.rep[(uint64_t)f * kDiscreteCells + ci];
            collect = collect || A.mixed[(uint64_t)f * kDiscreteCells + ci];
        } else {
            // the middle one of the sample's keys in the cell: the frequent key, if there is one
            const uint32_t last = key_lo + ((1u << shift) - 1u);
            int a = 0, b = A.sample_cap;
            while (a < b) {
                const int mid = (a + b) >> 1;
                if (sample[mid] < key_lo) a = mid + 1; else b = mid;
            }
            int e = a;
            b = A.sample_cap;
            while (e < b) {
                const int mid = (e + b) >> 1;
                if (sample[mid] <= last) e = mid + 1; else b = mid;
            }
            if (e > a) heavy = sample[(a + e) >> 1];
        }
        SelSlot *o = A.slots + (uint64_t)f * B + s;
        o->heavy = heavy;
        o->key_lo = key_lo;
        o->shift = shift;
    }
    collect = __syncthreads_or(collect ? 1 : 0) != 0;
    if (tid == 0) {
        A.kind[f] = (discrete ? kKindDiscrete : 0u) | (collect ? 0u : kKindNoCollect);
        A.n_slots[f] = n_slots;
        if (many) atomicOr(&A.mix[1], n_slots && collect ? 1u : 2u);
        A.mode[f] = order ? kSelOrder : kSelDistinct;
        present[f] = m;
    }
}

// ---- collect ----------------------------------------------------------------------------------------------------
constexpr int kCollectPer = 16;   // keys per thread and step
// (64 vector and 80 scalar registers at most, so that two workgroups fit a compute unit and one reads while the other waits at a
// barrier: 115M rows of 5 columns of numbers and 8 of categories 0.885 -> 0.578 ms, 1M x 28 numbers 59 -> 44 us.)
__global__ __launch_bounds__(kSelBlock) __attribute__((amdgpu_num_sgpr(80), amdgpu_waves_per_eu(8))) void sel_collect_kernel(const uint32_t *__restrict__ keys,
                                                                const uint64_t *__restrict__ seg_off,
                                                                const uint32_t *__restrict__ blk_off, int F, int B,
                                                                SelArrays A, uint32_t *__restrict__ out, bool many) {
    extern __shared__ uint32_t dyn[];
    __shared__ uint32_t seg[kSegs];
    uint32_t *heavy = dyn, *cnt = dyn + B, *base = dyn + 2 * B;
    uint16_t *slot_of = (uint16_t *)(dyn + 3 * B);   // cap
    __shared__ TileShares shares;
    TileRun run(blk_off, F, many ? A.mix[1] : 0u, &shares, [&](int f) __attribute__((always_inline)) -> uint32_t {
        return A.n_slots[f] == 0 || (A.kind[f] & kKindNoCollect) ? 0u : 1u;
    });
    uint64_t k0, k1;
    while (run.next(blk_off, seg_off, &k0, &k1)) {
        const int f = run.f;
        const uint32_t nc = A.n_cells[f], ns = A.n_slots[f];
        if (ns == 0 || (A.kind[f] & kKindNoCollect)) continue;   // nothing to look for, or every cell has one key only
        __syncthreads();
        for (int i = threadIdx.x; i < kSegs; i += kSelBlock) seg[i] = A.seg[(uint64_t)f * kSegs + i];
        for (uint32_t i = threadIdx.x; i < nc; i += kSelBlock) slot_of[i] = A.slot_of[(uint64_t)f * A.cap + i];
        for (uint32_t i = threadIdx.x; i < ns; i += kSelBlock) {
            heavy[i] = A.slots[(uint64_t)f * B + i].heavy;
            cnt[i] = 0;
        }
        __syncthreads();
        const uint32_t *p = keys + seg_off[f];
        uint32_t *o = out + seg_off[f];
        for (uint64_t t0 = k0; t0 < k1; t0 += (uint64_t)kCollectPer * kSelBlock) {
            uint32_t k[kCollectPer], at[kCollectPer];   // at: slot << 16 | rank inside this step, ~0: not collected
            const uint64_t i0 = t0 + 4ull * threadIdx.x;
            if (t0 + (uint64_t)kCollectPer * kSelBlock <= k1) {
#pragma unroll
                for (int j = 0; j < kCollectPer / 4; ++j) {
                    const sel_u32x4 q = *(const sel_u32x4 *)(p + i0 + (uint64_t)j * 4 * kSelBlock);
#pragma unroll
                    for (int c = 0; c < 4; ++c) k[4 * j + c] = q[c];
                }
            } else {
#pragma unroll
                for (int j = 0; j < kCollectPer; ++j) {
                    const uint64_t i = i0 + (uint64_t)(j / 4) * 4 * kSelBlock + (j & 3);
                    k[j] = i < k1 ? p[i] : kMissingKey;
                }
            }
#pragma unroll
            for (int j = 0; j < kCollectPer; ++j) {
                at[j] = 0xffffffffu;
                if (k[j] != kMissingKey) {
                    const uint32_t s = slot_of[cell_of(seg, k[j])];
                    if (s != kNoSlot && heavy[s] != k[j]) at[j] = (s << 16) | atomicAdd(&cnt[s], 1u);
                }
            }
            __syncthreads();
            for (uint32_t s = threadIdx.x; s < ns; s += kSelBlock) {
                const uint32_t c = cnt[s];
                if (c) {
                    base[s] = A.slots[(uint64_t)f * B + s].off + atomicAdd(&A.cursor[(uint64_t)f * B + s], c);
                    cnt[s] = 0;
                }
            }
            __syncthreads();
#pragma unroll
            for (int j = 0; j < kCollectPer; ++j)
                if (at[j] != 0xffffffffu) o[base[at[j] >> 16] + (at[j] & 0xffffu)] = k[j];
        }
    }
}
static_assert(kSegs + kDiscreteCells / 4 <= kDiscreteCells, "one cell per interval and the budget");
static_assert(kCollectPer * kSelBlock <= 65536, "a rank inside a step has 16 bits");

// ---- distinct -----------------------------------------------------------------------------------------------------
// One workgroup per feature whose non-empty cells are no more than B: its distinct values, counted up to B + 1.  At most
// B of them: all but the smallest are the cuts.  More: the feature is an ordinary one after all (every non-empty cell
// has a slot, so nothing is missing for the order statistics).
__global__ __launch_bounds__(kSelBlock) void sel_distinct_kernel(const uint64_t *__restrict__ seg_off, int B, SelArrays A,
                                                                 const uint32_t *__restrict__ collected,
                                                                 float *__restrict__ cuts, int32_t *__restrict__ nb,
                                                                 uint64_t work_tuned) {
    extern __shared__ uint32_t dyn[];
    uint32_t *mark = dyn;                               // 2^kMarkBits bits
    uint32_t *ext = dyn + (1 << kMarkBits) / 32;        // B + 1 distinct keys of the slots with collected keys, in order
    uint32_t *ext_at = ext + B + 1;                     // B: first one of a slot
    uint32_t *dcnt = ext_at + B;                        // B: distinct keys of a slot
    __shared__ uint32_t tmp[kSelBlock / 64];
    __shared__ uint32_t n_ext;
    const int f = blockIdx.x, tid = threadIdx.x;
    if (A.mode[f] != kSelDistinct) return;
    const uint32_t ns = A.n_slots[f];
    float *c = cuts + (int64_t)f * (B - 1);
    if (ns == 0) {
        for (int k = tid; k < B - 1; k += kSelBlock) c[k] = __uint_as_float(0x7f800000u);
        if (tid == 0) nb[f] = 1;
        return;
    }
    if (tid == 0) n_ext = 0;
    const SelSlot *slots = A.slots + (uint64_t)f * B;
    const uint32_t *cur = A.cursor + (uint64_t)f * B;
    for (uint32_t s = tid; s < ns; s += kSelBlock) dcnt[s] = cur[s] ? 0u : 1u;
    __syncthreads();
    const uint64_t work_max = work_limit(work_tuned, seg_off, gridDim.x, f, *A.dear, A.kind[f] & kKindDiscrete);
    uint64_t work = 0;
    bool many = false;
    for (uint32_t s = 0; s < ns && !many; ++s) {
        if (dcnt[s]) continue;   // one value, the heavy key (uniform: dcnt is the same for all threads here)
        const SelSlot sl = slots[s];
        const uint32_t L = cur[s];
        const uint32_t *k = collected + seg_off[f] + sl.off;
        const uint32_t span = 1u << sl.shift, win = span < (1u << kMarkBits) ? span : (1u << kMarkBits);
        work += (uint64_t)L * (span / win);
        if (work > work_max) {
            if (tid == 0) {
                A.mode[f] = kSelSorted;
                A.flag[0] = 1;
            }
            return;
        }
        const uint32_t words = (win + 31) / 32;
        const bool has_heavy = sl.heavy != kMissingKey && sl.cnt > L;
        uint32_t found = 0;
        for (uint32_t w0 = 0; w0 < span && !many; w0 += win) {
            for (uint32_t i = tid; i < words; i += kSelBlock) mark[i] = 0;
            __syncthreads();
            for (uint32_t i = tid; i < L; i += kSelBlock) {
                const uint32_t d = k[i] - sl.key_lo - w0;
                if (d < win) atomicOr(&mark[d >> 5], 1u << (d & 31u));
            }
            if (tid == 0 && has_heavy) {
                const uint32_t d = sl.heavy - sl.key_lo - w0;
                if (d < win) atomicOr(&mark[d >> 5], 1u << (d & 31u));
            }
            __syncthreads();
            const uint32_t per = (words + kSelBlock - 1) / kSelBlock, i0 = tid * per;
            uint32_t mine = 0;
            for (uint32_t i = i0; i < i0 + per && i < words; ++i) mine += (uint32_t)__popc(mark[i]);
            uint32_t total;
            uint32_t at = n_ext + block_scan(mine, tmp, &total);
            if (n_ext + total > (uint32_t)B) {   // (the same for all threads: n_ext changes behind a barrier)
                many = true;
            } else {
                for (uint32_t i = i0; i < i0 + per && i < words; ++i)
                    for (uint32_t b = mark[i]; b; b &= b - 1) ext[at++] = sl.key_lo + w0 + i * 32 + (uint32_t)__builtin_ctz(b);
                __syncthreads();
                if (tid == 0) n_ext += total;
                found += total;
            }
            __syncthreads();
        }
        if (tid == 0) {
            ext_at[s] = n_ext - found;
            dcnt[s] = found;
        }
        __syncthreads();
    }
    // number of distinct values before each slot
    uint32_t d = 0;
    if (!many) {
        uint32_t mine = 0;
        const uint32_t per = (ns + kSelBlock - 1) / kSelBlock, s0 = tid * per;
        for (uint32_t s = s0; s < s0 + per && s < ns; ++s) mine += dcnt[s];
        uint32_t at = block_scan(mine, tmp, &d);
        if (d > (uint32_t)B) {
            many = true;
        } else {
            for (uint32_t s = s0; s < s0 + per && s < ns; ++s) {
                const bool pure = cur[s] == 0;
                for (uint32_t j = 0; j < dcnt[s]; ++j, ++at)
                    if (at > 0) c[at - 1] = key_float(pure ? slots[s].heavy : ext[ext_at[s] + j]);
            }
            for (int k = (int)d - 1 + tid; k < B - 1; k += kSelBlock) c[k] = __uint_as_float(0x7f800000u);
            if (tid == 0) nb[f] = (int32_t)d;
        }
    }
    if (many && tid == 0) A.mode[f] = kSelOrder;
}

// ---- order --------------------------------------------------------------------------------------------------------
// The slots of the features that take order statistics, listed by size: up to kSmallSlot collected keys (a wave ranks
// them), up to kMidSlot (a workgroup of 256), more (of 1024).
__global__ __launch_bounds__(kSelBlock) void sel_list_kernel(int F, int B, SelArrays A) {
    __shared__ uint32_t n[3], base[3];
    if (threadIdx.x < 3) n[threadIdx.x] = 0;
    __syncthreads();
    const uint64_t g = (uint64_t)blockIdx.x * kSelBlock + threadIdx.x;
    int cls = -1;
    uint32_t at = 0;
    if (g < (uint64_t)F * B) {
        const int f = (int)(g / (uint64_t)B);
        if ((uint32_t)(g % (uint64_t)B) < A.n_slots[f] && A.mode[f] == kSelOrder) {
            const uint32_t L = A.cursor[g];
            cls = L <= (uint32_t)kSmallSlot ? 0 : L <= (uint32_t)kMidSlot ? 1 : 2;
            at = atomicAdd(&n[cls], 1u);
        }
    }
    __syncthreads();
    if (threadIdx.x < 3) base[threadIdx.x] = n[threadIdx.x] ? atomicAdd(&A.n_work[threadIdx.x], n[threadIdx.x]) : 0u;
    __syncthreads();
    if (cls >= 0) A.work[(uint64_t)cls * F * B + base[cls] + at] = (uint32_t)g;
}

// A wave per slot: every collected key's rank by comparison with all of them.
__global__ __launch_bounds__(256) void sel_order_small_kernel(const uint64_t *__restrict__ seg_off, int B, SelArrays A,
                                                              const uint32_t *__restrict__ present,
                                                              const uint32_t *__restrict__ collected) {
    __shared__ uint32_t raw[4][kSmallSlot], srt[4][kSmallSlot];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t n_work = A.n_work[0];
    for (uint32_t wi = blockIdx.x * 4 + w; wi < n_work; wi += gridDim.x * 4) {
        const uint32_t g = A.work[wi];
        const int f = (int)(g / (uint32_t)B);
        const SelSlot sl = A.slots[g];
        const uint32_t L = A.cursor[g];
        const uint32_t *k = collected + seg_off[f] + sl.off;
        uint32_t key[kSmallSlot / 64], rank[kSmallSlot / 64];
        uint32_t below = 0;
        wave_sync();   // the slot before has been read
#pragma unroll
        for (int j = 0; j < kSmallSlot / 64; ++j) {
            const uint32_t i = j * 64 + lane;
            key[j] = i < L ? k[i] : kMissingKey;
            rank[j] = 0;
            raw[w][i] = key[j];
            below += (uint32_t)__popcll(__ballot(i < L && key[j] < sl.heavy));
        }
        wave_sync();
        const uint32_t *rw = raw[w];
        for (uint32_t i0 = 0; i0 < L; i0 += 4) {   // (the words behind the last key hold kMissingKey: below no key)
#pragma unroll
            for (uint32_t c = 0; c < 4; ++c) {
                const uint32_t i = i0 + c, x = rw[i];
#pragma unroll
                for (int j = 0; j < kSmallSlot / 64; ++j)
                    rank[j] += (x < key[j] || (x == key[j] && i < (uint32_t)(j * 64 + lane))) ? 1u : 0u;
            }
        }
        uint32_t *sw = srt[w];
#pragma unroll
        for (int j = 0; j < kSmallSlot / 64; ++j)
            if (j * 64 + lane < (int)L) sw[rank[j]] = key[j];
        wave_sync();
        const uint64_t m = present[f];
        const uint32_t eq = sl.cnt - L;
        uint64_t k_end = first_k((uint64_t)sl.start + sl.cnt, m, (uint32_t)B);
        if (k_end > (uint64_t)B) k_end = (uint64_t)B;
        for (uint64_t q = first_k(sl.start, m, (uint32_t)B) + lane; q < k_end; q += 64) {
            const uint32_t r = (uint32_t)(q * m / (uint64_t)B - sl.start);
            A.pick[(uint64_t)f * B + q] = r < below ? sw[r] : r < below + eq ? sl.heavy : sw[r - eq];
        }
    }
}

// A workgroup per larger slot: the keys counted by their top bits inside the cell (about as many counters as keys), the
// wanted ranks found in the running sum; where bits are left, once more inside every bucket that holds a wanted rank.
template <int BLOCK, int BITS>
__global__ __launch_bounds__(BLOCK) void sel_order_kernel(const uint64_t *__restrict__ seg_off, int F, int B, SelArrays A,
                                                          const uint32_t *__restrict__ present,
                                                          const uint32_t *__restrict__ collected, int cls,
                                                          uint64_t work_tuned) {
    static_assert(2 * BITS >= kSegShift + 1, "two levels reach the last bit");
    extern __shared__ uint32_t dyn[];
    uint32_t *cnt = dyn;                     // 2^BITS
    uint32_t *bucket = dyn + (1 << BITS);    // B: buckets to look into
    uint32_t *bstart = bucket + B;           // B: rank of a bucket's smallest key
    __shared__ uint32_t tmp[BLOCK / 64];
    __shared__ uint32_t n_buckets;
    const int tid = threadIdx.x;
    const uint32_t n_work = A.n_work[cls];
    const uint32_t *work = A.work + (uint64_t)cls * F * B;
    for (uint32_t wi = blockIdx.x; wi < n_work; wi += gridDim.x) {
        const uint32_t g = work[wi];
        const int f = (int)(g / (uint32_t)B);
        const SelSlot sl = A.slots[g];
        const uint32_t L = A.cursor[g], eq = sl.cnt - L;
        const uint32_t *k = collected + seg_off[f] + sl.off;
        const uint64_t m = present[f];
        uint32_t *pick = A.pick + (uint64_t)f * B;
        const int nb1 = order_bits(L, (int)sl.shift, BITS);
        const int rest = (int)sl.shift - nb1;
        auto count = [&](uint32_t lo, int bits, int drop, uint32_t len) {   // keys in [lo, lo + len) by (key - lo) >> drop
            for (uint32_t i = tid; i < (1u << bits); i += BLOCK) cnt[i] = 0;
            __syncthreads();
            for (uint32_t i = tid; i < L; i += BLOCK) {
                const uint32_t d = k[i] - lo;
                if (d < len) atomicAdd(&cnt[d >> drop], 1u);
            }
            if (tid == 0 && eq) {
                const uint32_t d = sl.heavy - lo;
                if (d < len) atomicAdd(&cnt[d >> drop], eq);
            }
            __syncthreads();
        };
        // the ranks that fall into a count: whole keys are picked, buckets listed
        auto take = [&](uint32_t lo, int bits, int drop, uint32_t rank0) {
            const uint32_t n = 1u << bits, per = (n + BLOCK - 1) / BLOCK, i0 = tid * per;
            uint32_t mine = 0;
            for (uint32_t i = i0; i < i0 + per && i < n; ++i) mine += cnt[i];
            uint32_t all;
            uint64_t pos = (uint64_t)rank0 + block_scan(mine, tmp, &all);
            if (mine) {
                uint64_t q = first_k(pos, m, (uint32_t)B);   // the first wanted rank at or behind pos: nothing to do below it
                uint64_t want = q < (uint64_t)B ? q * m / (uint64_t)B : ~0ull;
                for (uint32_t i = i0; i < i0 + per && i < n; ++i) {
                    const uint32_t c = cnt[i];
                    if (want < pos + c) {
                        if (drop == 0) {
                            for (; want < pos + c; want = q < (uint64_t)B ? q * m / (uint64_t)B : ~0ull) pick[q++] = lo + i;
                        } else {
                            const uint32_t b = atomicAdd(&n_buckets, 1u);
                            bucket[b] = i;
                            bstart[b] = (uint32_t)pos;
                            q = first_k(pos + c, m, (uint32_t)B);
                            want = q < (uint64_t)B ? q * m / (uint64_t)B : ~0ull;
                        }
                    }
                    pos += c;
                }
            }
            __syncthreads();
        };
        const uint64_t work_max = work_limit(work_tuned, seg_off, F, f, *A.dear, A.kind[f] & kKindDiscrete);
        if (L > work_max) {   // (the sample did not show this many)
            if (tid == 0) {
                A.mode[f] = kSelSorted;
                A.flag[0] = 1;
            }
            continue;
        }
        if (tid == 0) n_buckets = 0;
        __syncthreads();
        count(sl.key_lo, nb1, rest, 1u << sl.shift);
        take(sl.key_lo, nb1, rest, sl.start);
        if (rest > 0) {
            const uint32_t nbk = n_buckets;   // (at most the slot's ranks, so at most B)
            if ((uint64_t)nbk * L > work_max) {
                if (tid == 0) {
                    A.mode[f] = kSelSorted;
                    A.flag[0] = 1;
                }
            } else {
                for (uint32_t b = 0; b < nbk; ++b) {
                    const uint32_t lo = sl.key_lo + (bucket[b] << rest), r0 = bstart[b];
                    count(lo, rest, 0, 1u << rest);
                    take(lo, rest, 0, r0);
                }
            }
        }
        __syncthreads();
    }
}

// ---- cuts -----------------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void sel_cuts_kernel(int B, SelArrays A, float *__restrict__ cuts, int32_t *__restrict__ nb) {
    __shared__ uint32_t tmp[4];
    const int f = blockIdx.x, tid = threadIdx.x;
    if (A.mode[f] != kSelOrder) return;   // written by sel_distinct_kernel, or left to the sort
    const uint32_t *pick = A.pick + (uint64_t)f * B;
    float *c = cuts + (int64_t)f * (B - 1);
    const uint32_t vmin = pick[0];
    const int per = (B + 255) / 256, k0 = tid * per;
    uint32_t mine = 0;
    for (int k = k0; k < k0 + per && k < B; ++k) mine += k > 0 && pick[k] != vmin && pick[k] != pick[k - 1] ? 1u : 0u;
    uint32_t nc;
    uint32_t at = block_scan(mine, tmp, &nc);
    for (int k = k0; k < k0 + per && k < B; ++k)
        if (k > 0 && pick[k] != vmin && pick[k] != pick[k - 1]) c[at++] = key_float(pick[k]);
    for (int k = (int)nc + tid; k < B - 1; k += 256) c[k] = __uint_as_float(0x7f800000u);
    if (tid == 0) nb[f] = (int32_t)nc + 1;
}

// ---- symbols of whole columns -------------------------------------------------------------------------------------
// The symbol of a key is the number of cuts at or below it.  Most cells hold no cut: their keys' symbol is one table
// read behind the cell; in the others (bit 15) the cuts up to the next cell's are bisected: one or two of them as a rule,
// most of a column's where its values are neighbours as floats (100,000 x 200 ids of 200 values above 10^7, the whole call:
// 1.69 ms one cut after the other, 0.45 bisected).  slot_of is free by now.
__global__ __launch_bounds__(kSelBlock) void sel_bins_kernel(int B, SelArrays A, const float *__restrict__ cuts,
                                                             const int32_t *__restrict__ nb) {
    __shared__ uint32_t seg[kSegs];
    __shared__ uint32_t ck[kSelBinsMax];
    if (A.flag[0]) return;   // some feature is to be sorted: its cuts are not there, and the table is not used
    const int f = blockIdx.x;
    const uint32_t nc = A.n_cells[f];
    const int ncut = nb[f] - 1;
    for (int i = threadIdx.x; i < kSegs; i += kSelBlock) seg[i] = A.seg[(uint64_t)f * kSegs + i];
    for (int i = threadIdx.x; i < ncut; i += kSelBlock) ck[i] = float_key(cuts[(int64_t)f * (B - 1) + i]);
    __syncthreads();
    for (uint32_t c = threadIdx.x; c < nc; c += kSelBlock) {
        int lo = 0, hi = kSegs;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if ((seg[mid] & 0xffffffu) <= c) lo = mid; else hi = mid;
        }
        const uint32_t shift = seg[lo] >> 24, key_lo = ((uint32_t)lo << kSegShift) + ((c - (seg[lo] & 0xffffffu)) << shift);
        int b = 0, e = ncut;   // cuts at or below the cell's first key
        while (b < e) {
            const int mid = (b + e) >> 1;
            if (ck[mid] <= key_lo) b = mid + 1; else e = mid;
        }
        const bool inside = b < ncut && ck[b] - key_lo < (1u << shift);
        A.slot_of[(uint64_t)f * A.cap + c] = (uint16_t)(b | (inside ? 0x8000 : 0));
    }
}

template <typename T>
__global__ __launch_bounds__(kSelBlock) void col_bins_kernel(const uint32_t *__restrict__ keys,
                                                             const uint64_t *__restrict__ seg_off,
                                                             const uint32_t *__restrict__ blk_off, int F, int B, SelArrays A,
                                                             const float *__restrict__ cuts, const int32_t *__restrict__ nb,
                                                             uint32_t missing, T *__restrict__ sym, int64_t stride) {
    extern __shared__ uint32_t dyn[];
    __shared__ uint32_t seg[kSegs];
    uint32_t *ck = dyn;                             // B
    uint16_t *first = (uint16_t *)(dyn + B);        // cap + 1
    TileRun run(blk_off, F);
    uint64_t k0, k1;
    while (run.next(blk_off, seg_off, &k0, &k1)) {
        const int f = run.f;
        const uint32_t nc = A.n_cells[f];
        const uint32_t ncut = (uint32_t)nb[f] - 1u;
        __syncthreads();
        for (int i = threadIdx.x; i < kSegs; i += kSelBlock) seg[i] = A.seg[(uint64_t)f * kSegs + i];
        for (uint32_t i = threadIdx.x; i < nc; i += kSelBlock) first[i] = A.slot_of[(uint64_t)f * A.cap + i];
        if (threadIdx.x == 0) first[nc] = (uint16_t)ncut;
        for (uint32_t i = threadIdx.x; i < ncut; i += kSelBlock) ck[i] = float_key(cuts[(int64_t)f * (B - 1) + i]);
        __syncthreads();
        const uint32_t *p = keys + seg_off[f];
        T *o = sym + (int64_t)f * stride;
        auto symbol = [&](uint32_t k) -> uint32_t {
            if (k == kMissingKey) return missing;
            const uint32_t c = cell_of(seg, k);
            uint32_t b = first[c];
            if (b & 0x8000u) {
                b &= 0x7fffu;
                for (uint32_t e = first[c + 1] & 0x7fffu; b < e;) {
                    const uint32_t mid = (b + e) >> 1;
                    if (ck[mid] <= k) b = mid + 1; else e = mid;
                }
            }
            return b;
        };
        auto store4 = [&](uint64_t i, const uint32_t (&v)[4]) {   // i: a multiple of four, the column starts on a line
            if (sizeof(T) == 1) {
                *(uint32_t *)(o + i) = v[0] | (v[1] << 8) | (v[2] << 16) | (v[3] << 24);
            } else {
                uint2 w;
                w.x = v[0] | (v[1] << 16);
                w.y = v[2] | (v[3] << 16);
                *(uint2 *)(o + i) = w;
            }
        };
        constexpr uint64_t STEP = 4ull * kSelBlock;
        uint64_t i = k0 + 4ull * threadIdx.x;
        for (; i + 3 * STEP + 4 <= k1; i += 4 * STEP) {
            sel_u32x4 q[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) q[j] = *(const sel_u32x4 *)(p + i + j * STEP);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t v[4] = {symbol(q[j][0]), symbol(q[j][1]), symbol(q[j][2]), symbol(q[j][3])};
                store4(i + j * STEP, v);
            }
        }
        for (; i < k1; i += STEP) {
            uint32_t v[4] = {0, 0, 0, 0};   // (what lies behind the last row is padding of the column)
            for (int c = 0; c < 4; ++c)
                if (i + c < k1) v[c] = symbol(p[i + c]);
            store4(i, v);
        }
    }
}

// Columns of symbols into the row-major bit stream: a tile of 2^log_rows rows (at least 32, so that it starts on a
// word) through LDS, columns at an odd stride of words; a thread packs 32 symbols in a row.
// Bound: HBM (symbols read once, written once) with enough loads in flight: with one word per thread and turn the whole
// call took 8.23 ms (115M x 13), 3.57 (500K x 801) and 1.62 (3M x 64); with eight 8.04, 3.38 and 1.57.
template <int BITS>
__global__ __launch_bounds__(256) void pack_columns_kernel(const void *__restrict__ cols, int64_t stride, int64_t n, int F,
                                                           int log_rows, uint32_t *__restrict__ packed, int64_t n_words) {
    using T = typename std::conditional<(BITS <= 8), uint8_t, uint16_t>::type;
    extern __shared__ uint32_t tile[];
    const T *sym = (const T *)cols;
    constexpr int PER = 4 / sizeof(T);   // symbols per word
    const int log_w = log_rows - (sizeof(T) == 1 ? 2 : 1), W = 1 << log_w, WS = W + 1;
    const int64_t r0 = (int64_t)blockIdx.x << log_rows;
    const int rows = n - r0 < ((int64_t)1 << log_rows) ? (int)(n - r0) : 1 << log_rows;
    const int need = (rows + PER - 1) / PER;   // words of a column that hold rows of this tile
    const int words = F << log_w;
    for (int i = threadIdx.x; i < words; i += 256 * 8) {   // eight loads in flight (past the edge the last word again)
        uint32_t v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int j = i + 256 * k < words ? i + 256 * k : words - 1, f = j >> log_w, w = j & (W - 1);
            v[k] = *(const uint32_t *)(sym + (int64_t)f * stride + r0 + (int64_t)(w < need ? w : need - 1) * PER);
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int j = i + 256 * k;
            if (j < words) tile[(j >> log_w) * WS + (j & (W - 1))] = v[k];
        }
    }
    __syncthreads();
    const int elems = rows * F, groups = (elems + 31) >> 5, nw = (int)(((int64_t)elems * BITS + 31) >> 5);
    uint32_t *out = packed + ((r0 * F) >> 5) * BITS;
    const uint32_t row_bytes = sizeof(T), col_bytes = (uint32_t)WS * 4u, back = col_bytes * (uint32_t)F - row_bytes;
    for (int g = threadIdx.x; g < groups; g += 256) {
        uint32_t e = 32u * (uint32_t)g;
        const uint32_t r = e / (uint32_t)F;
        uint32_t f = e - r * (uint32_t)F, at = f * col_bytes + r * row_bytes;
        uint32_t w[BITS];
        const bool whole = 32 * g + 32 <= elems;
        pack_group<BITS>(w, [&](int j) -> uint32_t {
            const uint32_t v = whole || 32 * g + j < elems ? *(const T *)((const char *)tile + at) : 0u;
            at += col_bytes;
            ++f;
            const bool wrap = f == (uint32_t)F;
            f = wrap ? 0u : f;
            at -= wrap ? back : 0u;
            return v;
        });
        if (whole) {
#pragma unroll
            for (int i = 0; i < BITS; ++i) out[(int64_t)g * BITS + i] = w[i];
        } else {
#pragma unroll
            for (int i = 0; i < BITS; ++i)
                if (g * BITS + i < nw) out[(int64_t)g * BITS + i] = w[i];
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) packed[n_words - 1] = 0;   // the pad word (Sec. 2.2 layout)
}

int cells_cap(int F, int64_t n_values) {
    int64_t avg = n_values / F, cap = 8192;   // at least kSegs + cap / 2, and twice a discrete feature's kDiscreteCells
    while (cap < avg / 4 && cap < kCellsMax) cap <<= 1;
    return (int)cap;
}
int sample_cap(int F, int64_t n_values) {
    int64_t avg = n_values / F, cap = 256;
    while (cap < avg && cap < kSampleMax) cap <<= 1;
    return (int)cap;
}

}  // namespace

// Where selection is the shorter way.  Up to 1024 bins: a wanted rank per cell is rare then (1024 of some 6000 cells that
// hold anything).  A column costs it some 0.3 us besides its values (cells, counters and slots, however few they are) and
// about a hundred KB of workspace, the sort some 0.1 us and 2 KB; but a few columns spend their time on launches, of which
// the sort has twice as many.  Dense matrices of normal values, the whole call in us by selection and by sort:
//   rows x columns        16 bins        64           256          1024
//     1000 x  256      173   197     183   234     206   333     617   617
//     1000 x 1000      341   232      -     -      458   398    1940   688
//     4000 x  700      358   267     377   328     452   466     731   949
//     5000 x 1900       -     -      790   749     990  1101      -     -
//     8000 x 1000      475   428     504   593     609   870    1043  1739
//     8000 x 4000     1583  1123    2169  1708    2925  2500    6850  6650
//    12000 x 3500     1461  1391    1582  2138    1995  3022    7252  7476
//    16000 x 1000      507   611     547   896     674  1249    1181  2228
//    16000 x 10000    4770  5185    7465  7941   15095 15562   31594 31913
// (with more than 3640 columns, 1920 of more than 255 bins, the symbols are bisected either way).  And the workspace: beyond
// 8 GB the selection's arrays may take a sixteenth of what the keys take.
bool gbt_select_ok(int F, int64_t n_values, int B) {
    if (B > kSelBinsMax) return false;
    // (the most a column can take, so that a larger matrix of as many columns never needs less)
    const int64_t column = (int64_t)(kSampleMax + kSegs + kCellsMax + kDiscreteCells) * 4 + kDiscreteCells + kCellsMax * 2 +
                           (int64_t)B * (int64_t)(sizeof(SelSlot) + 20);
    if (F * column > std::max((int64_t)8 << 30, n_values / 2)) return false;
    const int64_t len = n_values / F;   // of a column, on average
    if (len >= 14000) return true;
    if (len >= 3584 + (1 << 17) / B) return F <= 3640;   // (the widest matrix of 8-bit symbols that is packed from columns)
    return F <= 256 + (len > B ? 2 * std::min(B, 512) : 0);
}

size_t gbt_select_layout(int F, int64_t n_values, int B, char *base, SelArrays *A) {
    const int cap = cells_cap(F, n_values), sc = sample_cap(F, n_values);
    size_t o = 0;
    auto take = [&](size_t bytes) {
        char *p = base + o;
        o += gbt_align(bytes);
        return p;
    };
    SelArrays a;
    a.cap = cap;
    a.sample_cap = sc;
    a.sample = (uint32_t *)take((size_t)F * sc * 4);
    a.seg = (uint32_t *)take((size_t)F * kSegs * 4);
    a.n_cells = (uint32_t *)take((size_t)F * 4);
    a.counts = (uint32_t *)take((size_t)F * cap * 4);
    a.rep = (uint32_t *)take((size_t)F * kDiscreteCells * 4);
    a.mixed = (uint8_t *)take((size_t)F * kDiscreteCells);
    a.kind = (uint32_t *)take((size_t)F * 4);
    a.slot_of = (uint16_t *)take((size_t)F * cap * 2);
    a.slots = (SelSlot *)take((size_t)F * B * sizeof(SelSlot));
    a.n_slots = (uint32_t *)take((size_t)F * 4);
    a.cursor = (uint32_t *)take((size_t)F * B * 4);
    a.pick = (uint32_t *)take((size_t)F * B * 4);
    a.mode = (uint32_t *)take((size_t)F * 4);
    a.work = (uint32_t *)take((size_t)F * B * 12);
    a.n_work = (uint32_t *)take(12);
    a.flag = (uint32_t *)take(4);
    a.cost = (uint32_t *)take((size_t)F * 4);
    a.dear = (unsigned long long *)take(16);
    a.mix = (uint32_t *)(a.dear + 1);
    if (A) *A = a;
    return o;
}

hipError_t gbt_launch_select(gbt_ctx *ctx, const uint32_t *keys, uint32_t *collected, const uint64_t *seg_off,
                             const uint32_t *blk_off, int F, int64_t n_values, int B, const SelArrays &A, float *cuts,
                             int32_t *nb, uint32_t *present) {
    hipStream_t s = ctx->stream;
    const size_t lds_count = (size_t)A.cap * 4;
    const size_t lds_collect = (size_t)B * 12 + (size_t)A.cap * 2;
    const size_t lds_distinct = (size_t)(1 << kMarkBits) / 8 + (size_t)(3 * B + 1) * 4;
    const size_t lds_big = (size_t)(1 << kBigBits) * 4 + (size_t)B * 8, lds_mid = (size_t)(1 << kMidBits) * 4 + (size_t)B * 8;
    const uint64_t work = (uint64_t)ctx->quantise_work, by_sample = ctx->quantise_late ? ~0ull : work;   // 0: by lengths
    GbtLdsGuard guard(lds_distinct);
    hipError_t e = hipSuccess;
    auto raise = [&](const void *fn, size_t lds) {
        if (e == hipSuccess && lds > 64u * 1024u)
            e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    };
    raise((const void *)sel_distinct_kernel, lds_distinct);
    raise((const void *)sel_order_kernel<1024, kBigBits>, lds_big);
    if (e != hipSuccess) return e;
    // two workgroups of 1024 threads per compute unit, and no more than there are tiles to share out
    const int64_t tiles = n_values / kSortTile + F;
    const int grid = (int)(tiles < 2 * ctx->num_cu ? (tiles > 0 ? tiles : 1) : 2 * ctx->num_cu);
    const bool many = n_values >= kManyTiles * kSortTile * 2 * ctx->num_cu;
    sel_sample_kernel<<<F, kSelBlock, 0, s>>>(keys, seg_off, B, A, by_sample, many);
    sel_count_kernel<<<grid, kSelBlock, lds_count, s>>>(keys, seg_off, blk_off, F, A, by_sample, many);
    sel_pick_kernel<<<F, kSelBlock, 0, s>>>(seg_off, A, B, present, by_sample, many);
    sel_collect_kernel<<<grid, kSelBlock, lds_collect, s>>>(keys, seg_off, blk_off, F, B, A, collected, many);
    sel_distinct_kernel<<<F, kSelBlock, lds_distinct, s>>>(seg_off, B, A, collected, cuts, nb, work);
    const uint64_t all = (uint64_t)F * B;
    auto at_most = [&](uint64_t n, int per_cu) { return (unsigned)(n < (uint64_t)per_cu * ctx->num_cu ? n : (uint64_t)per_cu * ctx->num_cu); };
    sel_list_kernel<<<(unsigned)((all + kSelBlock - 1) / kSelBlock), kSelBlock, 0, s>>>(F, B, A);
    sel_order_small_kernel<<<at_most((all + 3) / 4, 8), 256, 0, s>>>(seg_off, B, A, present, collected);
    sel_order_kernel<256, kMidBits><<<at_most(all, 8), 256, lds_mid, s>>>(seg_off, F, B, A, present, collected, 1, work);
    sel_order_kernel<1024, kBigBits><<<at_most(all, 2), 1024, lds_big, s>>>(seg_off, F, B, A, present, collected, 2, work);
    sel_cuts_kernel<<<F, 256, 0, s>>>(B, A, cuts, nb);
    return hipGetLastError();
}

// ---- binning and packing of a dense matrix whose columns lie as keys -------------------------------------------------
namespace {
// log2 of the rows per tile of pack_columns_kernel: up to 1024 while the tile takes at most 40 KB of LDS (four
// workgroups per compute unit), 32 rows at up to 128 KB for wide matrices; 0: too wide
int pack_log_rows(int F, int sym_bytes) {
    auto lds = [&](int lr) { return (size_t)F * (((size_t)sym_bytes << lr) + 4); };
    for (int lr = 10; lr >= 6; --lr)
        if (lds(lr) <= 40u * 1024u) return lr;
    return lds(6) <= 128u * 1024u ? 6 : lds(5) <= 128u * 1024u ? 5 : 0;
}
int64_t col_stride(int64_t n) { return (n + 63) / 64 * 64; }

template <typename T>
hipError_t bin_pack_columns(gbt_ctx *ctx, const uint32_t *keys, void *cols, const uint64_t *seg_off, const uint32_t *blk_off,
                            int64_t n, int F, int B, const SelArrays &A, const float *cuts, const int32_t *nb, uint32_t missing,
                            int bits, uint32_t *packed, int64_t n_words) {
    hipStream_t s = ctx->stream;
    const int64_t stride = col_stride(n), tiles = n / kSortTile * F + F;
    const int grid = (int)(tiles < 2 * ctx->num_cu ? tiles : 2 * ctx->num_cu);
    const int lr = pack_log_rows(F, sizeof(T));
    const size_t lds = (size_t)F * (((size_t)sizeof(T) << lr) + 4);
    col_bins_kernel<T><<<grid, kSelBlock, (size_t)B * 4 + (size_t)(A.cap + 1) * 2, s>>>(keys, seg_off, blk_off, F, B, A, cuts, nb, missing,
                                                                                 (T *)cols, stride);
    return with_bits(bits, [&](auto bc) {
        constexpr int BITS = decltype(bc)::value;
        GbtLdsGuard guard(lds);
        if (guard.needed) {
            hipError_t e = hipFuncSetAttribute((const void *)pack_columns_kernel<BITS>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
        }
        pack_columns_kernel<BITS><<<(unsigned)((n + ((int64_t)1 << lr) - 1) >> lr), 256, lds, s>>>(cols, stride, n, F, lr, packed, n_words);
        return hipGetLastError();
    });
}
}  // namespace

size_t gbt_bin_columns_bytes(int64_t n, int F) { return (size_t)col_stride(n) * (size_t)F * 2; }
bool gbt_bin_columns_ok(int64_t n, int F, int bits) { return n > 0 && pack_log_rows(F, bits <= 8 ? 1 : 2) > 0; }

hipError_t gbt_launch_bin_table(gbt_ctx *ctx, int F, int B, const SelArrays &A, const float *cuts, const int32_t *nb) {
    sel_bins_kernel<<<F, kSelBlock, 0, ctx->stream>>>(B, A, cuts, nb);
    return hipGetLastError();
}

hipError_t gbt_launch_bin_columns(gbt_ctx *ctx, const uint32_t *keys, void *cols, const uint64_t *seg_off, const uint32_t *blk_off,
                                  int64_t n, int F, int B, const SelArrays &A, const float *cuts, const int32_t *nb,
                                  uint32_t missing, int bits, uint32_t *packed, int64_t n_words) {
    return bits <= 8 ? bin_pack_columns<uint8_t>(ctx, keys, cols, seg_off, blk_off, n, F, B, A, cuts, nb, missing, bits, packed, n_words)
                     : bin_pack_columns<uint16_t>(ctx, keys, cols, seg_off, blk_off, n, F, B, A, cuts, nb, missing, bits, packed, n_words);
}
