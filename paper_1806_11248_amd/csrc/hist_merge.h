// The merge of a workgroup's bins into the node's histogram in HBM, shared by the histogram kernels.
#ifndef GBT_HIST_MERGE_H
#define GBT_HIST_MERGE_H
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace {

// i / d where i * d < 2^32 (a workgroup's bins in units of eight: under 2^13, tiles of under 2^15 columns): a multiplication
// with ceil(2^32 / d), which is off by less than i * d / 2^32.  (A division by a number that is not known takes some twenty
// instructions, for every word of a merge.)
struct SmallDiv {
    uint32_t d, inv;
    __device__ explicit SmallDiv(uint32_t by) : d(by), inv(by > 1u ? 0xffffffffu / by + 1u : 0u) {}
    __device__ uint32_t operator()(uint32_t i) const { return d > 1u ? __umulhi(i, inv) : i; }
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
// (3) The four lines of an instruction belong to four columns (of tiles that have them):
// where the bins of a column lie in one LDS bank, eight of them meet there and not 32.
template <typename Bin>
__device__ __forceinline__ void merge_bins(int ft, int B, int64_t *out, int block, bool exclusive, Bin &&bin) {
    const uint32_t lead = (uint32_t)((uintptr_t)out >> 4) & 7u;   // bins of a line before the tile's first
    const uint32_t per_col = lead | ((uint32_t)B & 7u) ? ((uint32_t)B + 14u) >> 3 : (uint32_t)B >> 3, units = (uint32_t)ft * per_col;   // lines a column can touch, in all
    const SmallDiv by_cols((uint32_t)ft);
    if (!exclusive) {
        const uint32_t groups = (units + 3u) >> 2, first = (blockIdx.x * 2654435761u >> 8) % groups;
        for (uint32_t k = threadIdx.x; k < 64u * groups; k += (uint32_t)block) {
            uint32_t group = (k >> 6) + first;
            group = group >= groups ? group - groups : group;
            const uint32_t unit = 4u * group + ((k >> 4) & 3u), c = by_cols(unit), t = unit - c * (uint32_t)ft;
            const uint32_t b = 8u * c + ((k >> 1) & 7u) - ((lead + t * (uint32_t)B) & 7u);
            if (unit >= units || b >= (uint32_t)B) continue;
            int64_t g = 0, h = 0;
            bin(t, b, g, h);
            const int64_t v = (k & 1u) ? h : g;
            if (v != 0) atomicAdd((unsigned long long *)(out + 2u * (t * (uint32_t)B + b) + (k & 1u)), (unsigned long long)v);
        }
        return;
    }
    for (uint32_t k = threadIdx.x; k < 8u * units; k += (uint32_t)block) {
        const uint32_t unit = k >> 3, c = by_cols(unit), t = unit - c * (uint32_t)ft;
        const uint32_t b = 8u * c + (k & 7u) - ((lead + t * (uint32_t)B) & 7u);
        if (b >= (uint32_t)B) continue;
        int64_t g = 0, h = 0;
        bin(t, b, g, h);
        *(longlong2 *)(out + 2u * (t * (uint32_t)B + b)) = make_longlong2(g, h);
    }
}

}  // namespace
#endif
