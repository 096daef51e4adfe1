// nucleus.hpp -- what the partial row sort of the top-p sampler (nucleus.hip)
// and the draw on its result (rows.hip) share.
#pragma once

#include "tile.hpp"

namespace ls {

// Sort key of a value's bits: its IEEE 754 totalOrder code, unsigned.
__device__ __forceinline__ uint32_t nuc_key(uint32_t bits) {
    return bits ^ ((bits >> 31) ? 0xFFFFFFFFu : 0x80000000u);
}
__device__ __forceinline__ uint32_t nuc_bits(uint32_t key) {
    return key ^ ((key >> 31) ? 0x80000000u : 0xFFFFFFFFu);
}

// A row's map from keys to bins, monotone: the sampled range [lo, hi] is cut
// into cells of 2^shift keys, and cell c into 2^sub bins from bin `base` on
// (map[c] = base | sub << 16); keys below lo go to the first bin.
constexpr int kNucCells = 2048;
constexpr int kNucBins = 4096;
struct NucRow {
    uint32_t lo, hi, shift;
    uint32_t key_min;  // keys from here up are gathered and sorted
    uint32_t groups;   // groups they form
    uint32_t direct;   // the cells are the bins
    uint32_t pad[2];
};

// Where the draw finds the source index of a sorted element: the row's list
// (keys and their source indices; `stride` words from row to row), where group g
// of rows[r].groups has the same places as in the sorted row, from groups[r
// (slots + 1) + g].x to the next one's, in no particular order; or, with keys
// null, the row x.
struct NucSource {
    const uint32_t* x;
    const uint32_t* keys;
    const uint32_t* idx;
    const NucRow* rows;
    const uint2* groups;
    uint32_t stride, slots;
};

}  // namespace ls
