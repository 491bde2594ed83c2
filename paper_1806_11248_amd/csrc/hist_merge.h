// The merge of a workgroup's bins into the node's histogram in HBM, shared by the histogram kernels.
#ifndef GBT_HIST_MERGE_H
#define GBT_HIST_MERGE_H
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace {

// i / d for i < 2^21, d < 2^16: (i + 1/2) / d is at least 1 / 2d from a whole number, and v_rcp_f32 (1 ulp) with one rounding is off by
// less than i / d * 2^-22.  (A division of whole numbers takes some twenty-five instructions, and a workgroup of 1024 threads issues
// one of its own sixteen times before a short job has begun: see merge_bins.)
struct SmallDiv {
    float inv;
    __device__ explicit SmallDiv(uint32_t d) : inv(__builtin_amdgcn_rcpf((float)d)) {}
    __device__ uint32_t operator()(uint32_t i) const { return (uint32_t)__builtin_fmaf((float)i, inv, 0.5f * inv); }
};

// A tile of ft columns of B bins, out[(t * B + b) * 2] its g and the next word its h: adds what bin(t, b, g, h) yields, or,
// where this workgroup is the only one (`exclusive`), stores it, zeros included.  block: a multiple of 64.
// Bound: 64-bit atomics on HBM, which are retired by the line and not by the word, and take turns on a line.  So (1) a lane
// takes one WORD of the histogram, g or h, and sixteen neighbouring lanes a line of 128 bytes, wherever in its column that begins: an
// instruction covers four whole lines, where a lane per bin took two instructions of eight half-filled ones; (2) every workgroup
// starts at another place, so that those of one node, which end together, do not all queue at the same lines.  Root of 1M x 28
// bytes of 256 bins, 230 workgroups (1.65M atomics): 24 us a lane per bin, 12.5 with (1), 9.5 with both.  With lines counted from the
// column's first bin, which is a line's first only where B is a multiple of eight, 255 bins took 39 us a call, and so
// 36 (256 bins 33).
// (3) The four lines of an instruction belong to four columns (of tiles that have them): where the bins of a column lie in one LDS
// bank, eight of them meet there and not 32.
// Small tables: a launch of few short jobs takes what one workgroup has to issue, so groups of lanes are counted in scalar registers
// and nothing is divided: 5,000 x 19 x 6 bits, us a launch, 5.4 with two divisions here and one in the windows' kernel, 4.8 without
// (4.6 a lane per bin); 5,000 x 4 bytes 4.95 and 4.75; rounds of 5,000 to 120,000 rows x 4 to 60 columns 1.02 times as fast.
template <typename Bin>
__device__ __forceinline__ void merge_bins(int ft, int B, int64_t *out, int block, bool exclusive, Bin &&bin) {
    const uint32_t lead = (uint32_t)((uintptr_t)out >> 4) & 7u;   // bins of a line before the tile's first
    const uint32_t per_col = lead | ((uint32_t)B & 7u) ? ((uint32_t)B + 14u) >> 3 : (uint32_t)B >> 3;   // lines a column can touch
    const uint32_t units = (uint32_t)ft * per_col;
    const SmallDiv by_cols((uint32_t)ft);
    const uint32_t lane = threadIdx.x & 63u, waves = (uint32_t)block >> 6;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (!exclusive) {
        const uint32_t groups = (units + 3u) >> 2, first = __umulhi(blockIdx.x * 2654435761u, groups);
        for (uint32_t q = wave; q < groups; q += waves) {
            const uint32_t group = q + first < groups ? q + first : q + first - groups;
            const uint32_t unit = 4u * group + (lane >> 4), c = by_cols(unit), t = unit - __umul24(c, (uint32_t)ft);
            const uint32_t b = 8u * c + ((lane >> 1) & 7u) - ((lead + __umul24(t, (uint32_t)B)) & 7u);
            if (unit >= units || b >= (uint32_t)B) continue;
            int64_t g = 0, h = 0;
            bin(t, b, g, h);
            const int64_t v = (lane & 1u) ? h : g;
            if (v != 0) atomicAdd((unsigned long long *)(out + 2u * (__umul24(t, (uint32_t)B) + b) + (lane & 1u)), (unsigned long long)v);
        }
        return;
    }
    for (uint32_t q = wave; 8u * q < units; q += waves) {
        const uint32_t unit = 8u * q + (lane >> 3), c = by_cols(unit), t = unit - __umul24(c, (uint32_t)ft);
        const uint32_t b = 8u * c + (lane & 7u) - ((lead + __umul24(t, (uint32_t)B)) & 7u);
        if (unit >= units || b >= (uint32_t)B) continue;
        int64_t g = 0, h = 0;
        bin(t, b, g, h);
        *(longlong2 *)(out + 2u * (__umul24(t, (uint32_t)B) + b)) = make_longlong2(g, h);
    }
}

// The same for one column of n bins, many of them empty in a short job, as sparse rows have it.  Bound there: the wait for every
// word of LDS, so four are asked for together (all are read, for a branch around a read waits for it).  Trees of 50,000 rows of a
// fiftieth of 20 and of 100 columns x 256 bins, us a launch: by merge_bins 6.4 and 7.0, so 5.7 and 6.0 (a lane per bin that
// skips empty ones 4.6 and 5.7, which takes 2.5 times as long where few are empty).
template <typename Bin>
__device__ __forceinline__ void merge_ids(uint32_t n, int64_t *out, int block, bool exclusive, Bin &&bin) {
    constexpr uint32_t kDeep = 4;
    const uint32_t lead = (uint32_t)((uintptr_t)out >> 4) & 7u, groups = (lead + n + 31u) >> 5;   // of four lines
    const uint32_t first = __umulhi(blockIdx.x * 2654435761u, groups);
    const uint32_t lane = threadIdx.x & 63u, waves = (uint32_t)block >> 6;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (exclusive) {
        for (uint32_t i = threadIdx.x; i < n; i += (uint32_t)block) {
            int64_t g, h;
            bin(i, g, h);
            *(longlong2 *)(out + 2u * i) = make_longlong2(g, h);
        }
        return;
    }
    for (uint32_t q0 = wave; q0 < groups; q0 += kDeep * waves) {
        uint32_t i[kDeep];
        int64_t g[kDeep], h[kDeep];
#pragma unroll
        for (uint32_t j = 0; j < kDeep; ++j) {
            const uint32_t q = q0 + j * waves, group = q + first < groups ? q + first : q + first - groups;
            i[j] = 32u * group + (lane >> 1) - lead;
            i[j] = q < groups && i[j] < n ? i[j] : ~0u;
            bin(i[j] == ~0u ? 0u : i[j], g[j], h[j]);
        }
#pragma unroll
        for (uint32_t j = 0; j < kDeep; ++j) {
            const int64_t v = i[j] == ~0u ? 0 : (lane & 1u) ? h[j] : g[j];
            if (v != 0) atomicAdd((unsigned long long *)(out + 2u * i[j] + (lane & 1u)), (unsigned long long)v);
        }
    }
}

}  // namespace
#endif
