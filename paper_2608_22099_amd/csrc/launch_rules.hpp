// Limits of the launches, as plain host arithmetic (no HIP, so that they can be
// checked without a GPU).
#pragma once

#include <climits>
#include <cstdint>

namespace bandlu {

// A launch holds fewer than 2^32 threads: workgroups of `threads` that fit one.
constexpr int64_t max_groups(int64_t threads) { return int64_t(UINT32_MAX) / threads; }

// Tiled band Cholesky (pbtrf_tile.hip): the window's tiles fill LDS at 12 tile
// rows, and its 32-bit row and column numbers run up to 13 tiles past n.
constexpr int kCholTileThreads = 512;
constexpr int64_t kCholTileMaxKd = 144;
constexpr int64_t kCholTileMaxN = INT_MAX - 16 * 14;
constexpr bool chol_tile_fits(int64_t n, int64_t kd) {
    return n > 0 && n <= kCholTileMaxN && kd <= kCholTileMaxKd;
}

}  // namespace bandlu
