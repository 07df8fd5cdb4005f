// Grids of more workgroups than one dimension of a launch holds (fewer than 2^32
// threads): the workgroups are dealt to rows of a two-dimensional grid.  The host
// part is plain C++ so that the CPU tests compile it.
#pragma once

#include <cstdint>

namespace gl {

// Workgroups (of up to 1024 threads) per row of the grid: far below the limit, so that
// sizes in daily use, from a million rows of 16 lanes on, take the same way as the largest.
constexpr int64_t kFoldRow = 1 << 16;

struct Fold {
    uint32_t x, y;  // y > 1: the last row may have workgroups beyond the last, which return
};

inline Fold fold_blocks(int64_t blocks) {
    if (blocks <= kFoldRow) return {(uint32_t)(blocks > 0 ? blocks : 1), 1u};
    return {(uint32_t)kFoldRow, (uint32_t)((blocks + kFoldRow - 1) / kFoldRow)};
}

// Number of the workgroup at place (x, y) of a grid of that many per row.
#ifdef __HIPCC__
__host__ __device__
#endif
inline int64_t folded(uint32_t x, uint32_t y, uint32_t row) { return (int64_t)y * row + x; }

}  // namespace gl
