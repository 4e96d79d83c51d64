// The tiles of the 4-cycle apex lists (c4.hip, k_c4_lists): plain arithmetic
// over host integers, checked on the host over every accepted graph size.
#pragma once

#include <stdint.h>

namespace gpm {

constexpr int kListTile = 1024;    // ids per step of a workgroup
constexpr int kListTiles = 2048;   // tiles at most
constexpr int kClassBits = 21;     // a tile's size of one class; three classes to a 64-bit word

// Ids per tile of n ids: a multiple of kListTile, at most kListTiles tiles.
constexpr int32_t list_tile(int32_t n) {
    const int64_t t = ((int64_t)n + kListTiles - 1) / kListTiles;
    return (int32_t)((t + kListTile - 1) / kListTile * kListTile);
}
// A whole tile of one class has to stay below the next class's bits, also on
// the largest graph: with 1,024 tiles a tile of 2^21 ids carried into them.
static_assert(list_tile(INT32_MAX - 1) < (1 << kClassBits), "a class fills its bits");

// One id of class k (0, 1, 2), and the ids of class k in a word of sizes.
constexpr uint64_t one_of_class(int k) { return 1ull << (kClassBits * k); }
constexpr uint32_t ids_of_class(uint64_t sizes, int k) {
    return (uint32_t)(sizes >> (kClassBits * k)) & ((1u << kClassBits) - 1u);
}

}  // namespace gpm
