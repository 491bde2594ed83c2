// BuildPartialHistograms (Alg. 1) for symbol widths other than 8 bits (compile-time width; 8 bits in the uniform form), any
// feature tile, rows given as a range or as a list of row ids.
//
// A row's slice of the bit stream, of up to four register windows of E = gbt_histw_window(BITS) whole symbols, is taken by
// as many neighbouring lanes, a window each: sixteen bytes from the byte of the first symbol on, in any alignment.  What
// decides, in the order the counters showed it (500,000 x 2000 x 6 bits, uniform, us of the root launch and of the round):
//   one row per lane, bins of a column side by side in LDS                           583    4820
//     (16 LDS clocks an atomic, of them 8 bank conflicts and 4 on one address; 10 vector instructions an element, which the
//     compiler makes of predicated slots and of an address it forms anew for each)
//   columns side by side in LDS, lanes that start at different columns, so that an instruction meets the banks of many;
//   an element is a field, a multiply-add and an atomic with its own offset           491    4400
//     (7 LDS clocks, 5 vector instructions: the L1 is what is busy, for it takes the dwords of scattered lanes one by one)
//   a row's windows in neighbouring lanes, whose sixteen bytes the L1 takes as one    333    3606
// So: word (symbol, column) of the table is symbol * fs + column, fs a multiple of 16 where that leaves two workgroups on a
// compute unit; a lane begins at column `start` of its window and goes on from the window's first column behind its last (a
// second load, placed that far back, brings those).  Symbols that are no bin, the missing one among them, have rows of the
// table that nothing reads: B + 1 rows, or one for each symbol where those are fewer.
// The words of a lane's next row are requested before the present ones are added, its pair one row ahead, a listed row's id
// two rows ahead.
//
// Two forms of the accumulated LDS word, as in kernels_hist8.hip:
//   general     [ g : 34 | h : 30 ], returning atomics in groups of four whose returned words are tested
//               together for a carry out of h or a wrap of g, side counter per bin;
//   uniform h   [ g : 46 | rows : 18 ], non-returning atomics, nothing tested (at most 2^18 - 1 rows per job),
//               8 bytes of LDS per bin instead of 12.
#include "gbt_internal.h"
#include "hist_common.h"
#include "hist_merge.h"

#include <type_traits>

namespace {

typedef unsigned long long __attribute__((address_space(3))) ldsw_u64;
typedef uint32_t __attribute__((address_space(3))) ldsw_u32;
// the 64-bit word `word` words behind the LDS byte address `addr`
__device__ __forceinline__ unsigned long long ldsw_add_rtn(uint32_t addr, int word, unsigned long long v) {
    return __hip_atomic_fetch_add((ldsw_u64 *)(uintptr_t)addr + word, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void ldsw_add(uint32_t addr, int word, unsigned long long v) {
    (void)__hip_atomic_fetch_add((ldsw_u64 *)(uintptr_t)addr + word, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

constexpr int kWRowsShift = 18;
constexpr uint32_t kWRowsMask = (1u << kWRowsShift) - 1u;

// One returned word: the exact carry test and the tight wrap test, then the bookkeeping (see hist_common.h).
// side_addr: LDS byte address of the bin's side counter.
__device__ __forceinline__ void pkw_check(uint32_t side_addr, unsigned long long old, unsigned long long addv, uint32_t hq) {
    uint32_t olo = (uint32_t)old, ohi = (uint32_t)(old >> 32);
    if ((pk_near_carry(old) < hq) | (pk_near_wrap(old, addv) < pk_reach(addv))) {
        asm volatile("" : "+v"(olo), "+v"(ohi));
        const uint32_t carry = ((olo & kHMask) + hq) >> kHShift;
        const uint32_t alo = (uint32_t)addv, ahi = (uint32_t)(addv >> 32);
        const uint32_t nlo = olo + alo;
        const uint32_t nhi = ohi + ahi + (nlo < olo ? 1u : 0u);
        const int32_t ovf = (int32_t)((ohi ^ nhi) & (ahi ^ nhi));
        const int32_t delta = ovf < 0 ? ((int32_t)nhi < 0 ? 1 : -1) : 0;
        if (carry != 0 || delta != 0)
            (void)__hip_atomic_fetch_add((ldsw_u32 *)(uintptr_t)side_addr, (uint32_t)(delta * 65536 + (int32_t)carry),
                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
}

typedef uint32_t w_u32x4 __attribute__((ext_vector_type(4), aligned(1)));
typedef uint32_t w_u32x2 __attribute__((ext_vector_type(2), aligned(1)));

// BITS: of a symbol.  CLAMP: a symbol may be larger than the last row of the LDS table and is counted there.
// SHORT: a row's columns are at most kShortBits bits, one window, which one load of eight bytes holds wherever it begins; it is turned to
// the lane's column in registers.  Wide symbols have such tiles, for their bins fill the LDS, and read little else than what the L1
// has to look up for them: with two loads of sixteen bytes and with this, root of 1M x 150 columns of 4096 bins 1661 and 948 us (a tile
// per column), of 462,962 x 324 of 2048 976 and 677, of 1M x 20 of 4096 122 and 88.  (Narrower symbols have tiles of more than 57 bits.)
constexpr int kShortBits = 57, kShortFrom = 10;
template <int BITS, bool LIST, bool UNI, bool CLAMP, bool SHORT>
__global__ __launch_bounds__(kHistBlock) void hist_bits_kernel(
    const uint32_t *__restrict__ packed, int64_t n_words, int64_t stride_bits, int64_t n, int B, int rows_lds, int fs,
    uint32_t missing, const uint32_t *__restrict__ row_idx, const int2 *__restrict__ gq,
    int64_t *__restrict__ pool, const HistJob *__restrict__ jobs, int32_t hq_uniform,
    const uint32_t *__restrict__ n_jobs_dev) {
    if (n_jobs_dev && blockIdx.x >= *n_jobs_dev) return;
    constexpr int E = gbt_histw_window(BITS);       // most elements of a window
    // Atomics in flight per lane.  Those that return hold two registers each until they are tested: in groups of four a compute unit
    // takes more waves (1M x 300 x 4 bits, root: 292 us in groups of 16, 225 of 8, 202 of 4; 3M x 50 x 9 bits 132, 131, 117).
    constexpr int G = UNI ? (E < 16 ? E : 16) : 4;
    constexpr uint32_t MASK = (1u << BITS) - 1u;
    extern __shared__ unsigned long long lds[];
    const HistJob job = jobs[blockIdx.x];
    const int ft = (int)job.ft;
    const int n_acc = rows_lds * fs;
    unsigned long long *main_ = lds;
    uint32_t *side = (uint32_t *)(lds + n_acc);
    for (int i = threadIdx.x; i < n_acc; i += (int)blockDim.x) {
        main_[i] = 0;
        if (!UNI) side[i] = 0;
    }
    __syncthreads();

    const uint32_t lds_base = (uint32_t)(uintptr_t)(ldsw_u64 *)main_;
    const uint32_t side_base = lds_base + 8u * (uint32_t)n_acc;
    const uint32_t fs8 = 8u * (uint32_t)fs, top = (uint32_t)rows_lds - 1u;
    // a row's windows (one, two or four) to neighbouring lanes; each begins at another of its columns than its neighbours'
    // and goes on from its first one behind its last
    const int log_win = ft <= E ? 0 : ft <= 2 * E ? 1 : 2, win = (int)threadIdx.x & ((1 << log_win) - 1);
    const int c0 = __umul24(ft, win) >> log_win, cnt = ((int)(__umul24(ft, win) + ft) >> log_win) - c0;   // this lane's columns
    const int most = (ft + (1 << log_win) - 1) >> log_win;                            // of any lane
    const int turn = (int)((threadIdx.x & 63) >> log_win), start = turn - (int)__umul24(SmallDiv((uint32_t)cnt)((uint32_t)turn), cnt);
    const int until = cnt - start;   // slots before its first column
    const int n_step = (int)(blockDim.x >> log_win);
    using Words = std::conditional_t<SHORT, w_u32x2, w_u32x4>;
    const int64_t last_at = n_words * 4 - (int64_t)sizeof(Words);   // the last byte from which they can be read (the launcher has made sure of one)
    const char *bytes = (const char *)packed;
    uint32_t keep[4];   // the bits that come before the first column
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int k = (int)__umul24(until, BITS) - 32 * j;
        keep[j] = (uint32_t)((0xffffffffull << std::min(std::max(k, 0), 32)) >> 32);
    }

    auto row_id = [&](uint32_t i) __attribute__((always_inline)) -> uint64_t {
        const uint64_t pos = (uint64_t)job.row_begin + i;
        return LIST ? (uint64_t)row_idx[pos] : pos;
    };
    const uint64_t lane_bit = ((uint64_t)job.f0 + (uint32_t)(SHORT ? c0 : c0 + start)) * BITS;
    const int back = (int)__umul24(cnt, BITS);   // from the first slot's bit to where the window's first column would follow its last
    // Sixteen bytes from the byte of bit `at` on.  What lies outside the buffer holds no bit that is used: the sixteen bytes
    // nearest to it are read, and put in their places when they are used.
    auto byte_in = [&](int64_t at) __attribute__((always_inline)) {
        const int64_t byte = at >> 3;
        return byte < 0 ? (int64_t)0 : byte > last_at ? last_at : byte;
    };
    auto aligned = [&](const w_u32x4 &v, int64_t at, int off, uint32_t (&W)[4]) __attribute__((always_inline)) {
        uint32_t x[4] = {v[0], v[1], v[2], v[3]};
        if (__builtin_expect(off != 0, 0)) {
            unsigned __int128 y = ((unsigned __int128)(((uint64_t)x[3] << 32) | x[2]) << 64) | (((uint64_t)x[1] << 32) | x[0]);
            y = off > 15 || off < -15 ? 0 : off > 0 ? y >> (8 * off) : y << (-8 * off);
#pragma unroll
            for (int j = 0; j < 4; ++j) x[j] = (uint32_t)(y >> (32 * j));
        }
        const uint32_t sh = (uint32_t)at & 7u;
#pragma unroll
        for (int j = 0; j < 3; ++j) W[j] = BITS % 8 == 0 ? x[j] : __builtin_amdgcn_alignbit(x[j + 1], x[j], sh);
        W[3] = BITS % 8 == 0 ? x[3] : x[3] >> sh;
    };
    auto turned = [&](const w_u32x2 &v, int64_t at, int off, uint32_t (&W)[4]) __attribute__((always_inline)) {
        uint64_t y = (((uint64_t)v[1] << 32) | v[0]) >> (8 * off + (int)(at & 7));
        y &= (1ull << back) - 1ull;
        y = (y >> (start * BITS)) | (y << (until * BITS));
        W[0] = (uint32_t)y;
        W[1] = (uint32_t)(y >> 32);
        W[2] = W[3] = 0;
    };
    Words wa, wb;   // the window on its way: from the lane's start on, and from its first column on (in its place); SHORT: the one
    int64_t at = 0;
    int offa = 0, offb = 0;
    auto issue = [&](uint64_t r) __attribute__((always_inline)) {
        at = (int64_t)(r * (uint64_t)stride_bits + lane_bit);
        const int64_t a = byte_in(at);
        wa = *(const Words *)(bytes + a);
        offa = (int)((at >> 3) - a);
        if constexpr (!SHORT) {
            const int64_t b = byte_in(at - back);
            wb = *(const Words *)(bytes + b);
            offb = (int)(((at - back) >> 3) - b);
        }
    };
    // (an opaque base: one register and an instruction's own offset, not sums made anew for every slot)
    uint32_t base = lds_base + 8u * (uint32_t)(c0 + start), base2 = base - 8u * (uint32_t)cnt;
    asm volatile("" : "+v"(base), "+v"(base2));
    auto add = [&](const uint32_t (&W)[4], unsigned long long addv, uint32_t hq, auto full) __attribute__((always_inline)) {
        // (Compared where it is needed: a mask per slot, kept, takes all scalar registers.  A lane's own columns by one comparison, the
        // most of any lane by the group: with both asked for each slot it took eleven instructions and not six, 666,666 x 260 x 9 bits,
        // root, 222 and 194 us, 2M x 124 x 2 bits 143 and 118.  SHORT has few columns of many slots, and is 4 % slower so.)
        int n = most, mine = cnt;
        asm volatile("" : "+s"(n));
        if constexpr (!SHORT) asm volatile("" : "+v"(mine));
#pragma unroll
        for (int g0 = 0; g0 < E; g0 += G) {
            if (!full && g0 >= n) break;
            uint32_t addr[G];
            unsigned long long old[G];
#pragma unroll
            for (int jj = 0; jj < G; ++jj) {
                const int j = g0 + jj;
                if (j < E && (!SHORT || j < n)) {
                    const int pos = j * BITS, wd = pos >> 5, off = pos & 31;
                    uint32_t sv;
                    if (off + BITS <= 32)
                        sv = (W[wd] >> off) & MASK;
                    else
                        sv = __builtin_amdgcn_alignbit(W[wd < 3 ? wd + 1 : 3], W[wd], (uint32_t)off) & MASK;
                    if (CLAMP) sv = min(sv, top);
                    addr[jj] = __umul24(sv, fs8) + (j >= until ? base2 : base);
                    if (full || (SHORT ? j + 1 < n || j < cnt : __builtin_expect(j < mine, 1))) {
                        if (UNI) ldsw_add(addr[jj], j, addv);
                        else old[jj] = ldsw_add_rtn(addr[jj], j, addv);
                    } else if (!UNI) {
                        old[jj] = 0;
                    }
                }
            }
            if (!UNI) {
                // the returned words of the group tested together: the smallest distance of any of them
                // from an event decides whether the per-word bookkeeping runs at all
                uint32_t near_carry = 0xffffffffu, near_wrap = 0xffffffffu;
#pragma unroll
                for (int jj = 0; jj < G; ++jj)
                    if (g0 + jj < E && (full || g0 + jj < n)) {
                        near_carry = min(near_carry, pk_near_carry(old[jj]));
                        near_wrap = min(near_wrap, pk_near_wrap(old[jj], addv));
                    }
                if (near_carry < hq || near_wrap < pk_reach(addv)) {
#pragma unroll
                    for (int jj = 0; jj < G; ++jj)
                        if (g0 + jj < E && (full || g0 + jj < n))
                            pkw_check(side_base + ((addr[jj] + 8u * (g0 + jj) - lds_base) >> 1), old[jj], addv, hq);
                }
            }
        }
    };

    const uint32_t nrows = job.n_rows, step = (uint32_t)n_step;
    uint32_t i = threadIdx.x >> log_win;
    if (i < nrows) {
        uint64_t r = row_id(i);
        uint64_t r1 = i + step < nrows ? row_id(i + step) : 0;
        bool ok_row = r < (uint64_t)n;   // a malformed row id is skipped, never dereferenced (row 0 is read in its place)
        int2 q = gq[ok_row ? r : 0];
        issue(ok_row ? r : 0);
        for (;;) {
            const bool more = i + step < nrows;
            const uint64_t r2 = i + 2 * step < nrows ? row_id(i + 2 * step) : 0;
            const bool ok_next = more && r1 < (uint64_t)n;
            const uint64_t next = ok_next ? r1 : 0;
            const int2 q1 = gq[next];
            const unsigned long long addv =
                UNI ? ((unsigned long long)(long long)q.x << kWRowsShift) + 1ull : pack_pair(q);
            const uint32_t hq = (uint32_t)q.y;
            uint32_t W[4];
            if constexpr (SHORT) {
                turned(wa, at, offa, W);
            } else {
                uint32_t V[4];
                aligned(wa, at, offa, W);
                aligned(wb, at - back, offb, V);
#pragma unroll
                for (int j = 0; j < 4; ++j) W[j] = (W[j] & keep[j]) | (V[j] & ~keep[j]);
            }
            issue(next);
            if (ok_row) {
                if (!SHORT && most == E && ft == E << log_win) add(W, addv, hq, std::integral_constant<bool, !SHORT>());
                else add(W, addv, hq, std::false_type());
            }
            if (!more) break;
            i += step;
            r1 = r2;
            q = q1;
            ok_row = ok_next;
        }
    }
    __syncthreads();
    int64_t *out = pool + job.hist_off + (uint64_t)job.f0 * (uint64_t)B * 2u;
    // (pad0: the only job of its (node, tile))
    merge_bins(ft, B, out, (int)blockDim.x, job.pad0 == 1u, [&](uint32_t t, uint32_t b, int64_t &g, int64_t &h) __attribute__((always_inline)) {
        if (b > MASK || b == missing) return;   // (a table of fewer rows than bins: the symbols cannot hold them)
        const uint32_t idx = b * (uint32_t)fs + t;
        const unsigned long long wv = main_[idx];
        if (UNI) {
            const int64_t rows = (int64_t)(wv & kWRowsMask);
            g = ((int64_t)wv - rows) >> kWRowsShift;
            h = (int64_t)((uint64_t)(uint32_t)rows * (uint32_t)hq_uniform);
        } else {
            const uint32_t sc = side[idx];
            const int64_t carry = (int64_t)(sc & 0xffffu), wr = (int64_t)((int32_t)sc >> 16);
            g = ((int64_t)wv >> kHShift) + wr * ((int64_t)1 << (64 - kHShift)) - carry;
            h = (int64_t)(wv & kHMask) + (carry << kHShift);
        }
    });
}

struct WArgs {
    hipStream_t s;
    int n_jobs, block, max_ft;
    size_t lds;
    const uint32_t *packed;
    int64_t n_words, stride_bits, n;
    int B, rows_lds, fs;
    uint32_t missing;
    const uint32_t *row_idx;
    const int2 *gq;
    int64_t *pool;
    const HistJob *jobs;
    int32_t hq_uniform;
    const uint32_t *n_jobs_dev;
};
template <int BITS, bool LIST, bool UNI, bool CLAMP, bool SHORT>
hipError_t launch_w(const WArgs &a) {
    auto *const kernel = hist_bits_kernel<BITS, LIST, UNI, CLAMP, SHORT>;
    GbtLdsGuard lds_guard(a.lds);
    if (lds_guard.needed) {
        hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)a.lds);
        if (e != hipSuccess) return e;
    }
    kernel<<<a.n_jobs, a.block, a.lds, a.s>>>(a.packed, a.n_words, a.stride_bits, a.n, a.B, a.rows_lds, a.fs, a.missing, a.row_idx, a.gq,
                                              a.pool, a.jobs, a.hq_uniform, a.n_jobs_dev);
    return hipGetLastError();
}
template <int BITS, bool CLAMP, bool SHORT>
hipError_t pick_w2(const WArgs &a, bool uni) {
    if (a.row_idx) return uni ? launch_w<BITS, true, true, CLAMP, SHORT>(a) : launch_w<BITS, true, false, CLAMP, SHORT>(a);
    return uni ? launch_w<BITS, false, true, CLAMP, SHORT>(a) : launch_w<BITS, false, false, CLAMP, SHORT>(a);
}
template <int BITS, bool CLAMP>
hipError_t pick_w1(const WArgs &a, bool uni) {
    if constexpr (BITS >= kShortFrom) {
        if (a.max_ft * BITS <= kShortBits) return pick_w2<BITS, CLAMP, true>(a, uni);
    }
    return pick_w2<BITS, CLAMP, false>(a, uni);
}
template <int BITS>
hipError_t pick_w(const WArgs &a, bool uni) {
    return a.rows_lds < (1 << BITS) ? pick_w1<BITS, true>(a, uni) : pick_w1<BITS, false>(a, uni);
}
}  // namespace

int gbt_histw_max_rows(bool uniform_h) { return uniform_h ? (int)kWRowsMask : 1 << 21; }

hipError_t gbt_launch_histw(gbt_ctx *ctx, const uint32_t *packed, int bits, int64_t stride_bits, int64_t n_words,
                            int64_t n, int B, uint32_t missing, const uint32_t *row_idx, const int32_t *gq,
                            int64_t *hist_pool, const HistJob *jobs, int n_jobs, int max_ft, bool uniform_h,
                            int32_t hq_uniform, int block, const uint32_t *n_jobs_dev) {
    if (n_jobs <= 0) return hipSuccess;
    // rows of the LDS table: the symbols, or the bins and one row for what is no bin; a stride that keeps a column in its banks
    // where that leaves two workgroups on a compute unit
    const int rows_lds = std::min(1 << bits, B + 1);
    auto lds_of = [&](int fs) { return (size_t)rows_lds * fs * (uniform_h ? 8 : 12); };
    int fs = (max_ft + 15) / 16 * 16;
    if (lds_of(fs) > ctx->lds_per_block / 2) fs = max_ft | 1;
    if (lds_of(fs) > ctx->lds_per_block) fs = max_ft;
    const size_t lds = lds_of(fs);
    const WArgs a{ctx->stream, n_jobs, block, max_ft, lds, packed, n_words, stride_bits, n, B, rows_lds, fs, missing, row_idx,
                  (const int2 *)gq, hist_pool, jobs, hq_uniform, n_jobs_dev};
    switch (bits) {
        case 1: return pick_w<1>(a, uniform_h);
        case 2: return pick_w<2>(a, uniform_h);
        case 3: return pick_w<3>(a, uniform_h);
        case 4: return pick_w<4>(a, uniform_h);
        case 5: return pick_w<5>(a, uniform_h);
        case 6: return pick_w<6>(a, uniform_h);
        case 7: return pick_w<7>(a, uniform_h);
        case 8: return pick_w<8>(a, uniform_h);
        case 9: return pick_w<9>(a, uniform_h);
        case 10: return pick_w<10>(a, uniform_h);
        case 11: return pick_w<11>(a, uniform_h);
        case 12: return pick_w<12>(a, uniform_h);
        case 13: return pick_w<13>(a, uniform_h);
        case 14: return pick_w<14>(a, uniform_h);
        case 15: return pick_w<15>(a, uniform_h);
        case 16: return pick_w<16>(a, uniform_h);
        default: return hipErrorInvalidValue;
    }
}
