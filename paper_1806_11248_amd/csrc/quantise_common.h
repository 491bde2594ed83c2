// What the two ways to a feature's order statistics share (kernels_quantise.hip: sort; kernels_select.hip: selection).
#ifndef GBT_QUANTISE_COMMON_H
#define GBT_QUANTISE_COMMON_H
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace {

constexpr int kSortTile = 4096;   // keys per tile: the unit of blk_off (a segment's first tile)
constexpr uint32_t kMissingKey = 0xffffffffu;

// Order-preserving image of a float; a missing value is the largest key.
__device__ inline uint32_t float_key(float x) {
    if (x != x) return kMissingKey;
    x = x + 0.0f;   // -0.0 -> +0.0: the two compare equal and must share a key
    uint32_t u = __float_as_uint(x);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ inline float key_float(uint32_t k) {
    uint32_t u = (k & 0x80000000u) ? (k & 0x7fffffffu) : ~k;
    return __uint_as_float(u);
}

__device__ inline int find_segment(const uint32_t *blk_off, int F, uint32_t blk) {
    int lo = 0, hi = F;   // last f with blk_off[f] <= blk and a non-empty tile range
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (blk_off[mid] <= blk) lo = mid; else hi = mid;
    }
    return lo;
}

// 32 symbols of BITS bits are BITS whole words of the stream: fn(j) yields symbol j, j = 0..31 in order.  Shifts and word
// numbers are compile-time constants (a word at a time, with its element and bit position computed, took three times
// the instructions).
template <int BITS, typename Fn>
__device__ __forceinline__ void pack_group(uint32_t (&w)[BITS], Fn &&fn) {
#pragma unroll
    for (int i = 0; i < BITS; ++i) w[i] = 0;
#pragma unroll
    for (int j = 0; j < 32; ++j) {
        const int bit = j * BITS, i = bit >> 5, at = bit & 31;
        const uint32_t v = fn(j);
        w[i] |= v << at;
        if (at + BITS > 32) w[i + 1] |= v >> (32 - at);
    }
}

// Calls fn(std::integral_constant<int, bits>) for bits = 1..16.
template <typename Fn>
inline hipError_t with_bits(int bits, Fn &&fn) {
    switch (bits) {
#define GBT_BITS_CASE(k) \
    case k: return fn(std::integral_constant<int, k>());
        GBT_BITS_CASE(1) GBT_BITS_CASE(2) GBT_BITS_CASE(3) GBT_BITS_CASE(4) GBT_BITS_CASE(5) GBT_BITS_CASE(6)
        GBT_BITS_CASE(7) GBT_BITS_CASE(8) GBT_BITS_CASE(9) GBT_BITS_CASE(10) GBT_BITS_CASE(11) GBT_BITS_CASE(12)
        GBT_BITS_CASE(13) GBT_BITS_CASE(14) GBT_BITS_CASE(15) GBT_BITS_CASE(16)
#undef GBT_BITS_CASE
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

enum : uint32_t {
    kSelOrder = 0,      // more than B distinct values: order statistics
    kSelDistinct = 1,   // at most B, perhaps
    kSelSorted = 2      // the feature's values lie too close together for selection: its cuts come from the sort
};
// Selection (kernels_select.hip).  Device arrays, all inside the quantise workspace.
struct SelSlot {
    uint32_t start;    // rank of the cell's smallest key
    uint32_t cnt;      // keys in the cell
    uint32_t off;      // where the cell's collected keys start inside the segment's part of the second key buffer
    uint32_t heavy;    // a key of the cell that is counted, not collected (kMissingKey: none)
    uint32_t key_lo;   // the cell holds the keys [key_lo, key_lo + 2^shift)
    uint32_t shift;
};
struct SelArrays {
    uint32_t *sample;    // [F][sample_cap] sorted sample of a segment
    uint32_t *seg;       // [F][2048] first cell of a key's top 11 bits | (shift << 24)
    uint32_t *n_cells;   // [F]
    uint32_t *counts;    // [F][cap] keys per cell
    uint32_t *rep;       // [F][kDiscreteCells] a discrete feature's cells: a key of the cell (kMissingKey: none seen yet) ...
    uint8_t *mixed;      // [F][kDiscreteCells] ... and whether the cell holds another one as well
    uint32_t *kind;      // [F] bit 0: discrete (few distinct keys in the sample), bit 1: nothing of it has to be collected;
                         // until the pick, bits 8 up: 1 + the place of its frequent key in the sample
    uint16_t *slot_of;   // [F][cap] the slot of a cell that is looked into, 0xffff: none
    SelSlot *slots;      // [F][B]
    uint32_t *n_slots;   // [F]
    uint32_t *cursor;    // [F][B] keys collected per slot
    uint32_t *pick;      // [F][B] the order statistics floor(k m / B), k = 0..B-1
    uint32_t *mode;      // [F] kSelOrder / kSelDistinct / kSelSorted
    uint32_t *work;      // [3][F * B] slots by the number of collected keys ...
    uint32_t *n_work;    // [3] ... and how many
    uint32_t *flag;      // [1] not zero: some feature's mode is kSelSorted
    uint32_t *cost;      // [F] key reads of the workgroup that would spend most on the feature, by its sample
    unsigned long long *dear;   // [1] keys of the features whose cost is more than sorting them alone
    uint32_t *mix;              // [2] behind it: kinds of features the count meets (1 numbers, 2 discrete, 4 some dear) and the collection (1 work, 2 none)
    int cap, sample_cap;
};
#endif
