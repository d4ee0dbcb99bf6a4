// Limits of the launches, as plain host arithmetic (no HIP, so that they can be
// checked without a GPU).
#pragma once

#include <climits>
#include <cstdint>

namespace bandlu {

// A launch holds fewer than 2^32 threads (of more it runs the remainder, without
// an error): workgroups of `threads` that fit one.
constexpr int64_t max_groups(int64_t threads) { return int64_t(UINT32_MAX) / threads; }

// Tiled band Cholesky (pbtrf_tile.hip): the window's tiles fill LDS at 12 tile
// rows, and its 32-bit row and column numbers run up to 13 tiles past n.
constexpr int kCholTileThreads = 512;
constexpr int64_t kCholTileMaxKd = 144;
constexpr int64_t kCholTileMaxN = INT_MAX - 16 * 14;
constexpr bool chol_tile_fits(int64_t n, int64_t kd) {
    return n > 0 && n <= kCholTileMaxN && kd <= kCholTileMaxKd;
}

// Small systems in batches: the tiles of one or two panels are mostly padding and
// only two of their workgroups fit a CU (one for kd > 48), where eight of the
// column kernel's do.  Measured (us, column kernel / tiles): n = 4, kd = 2: 51 / 198
// for 16384 systems, 14 / 16 for 512; n = 12, kd = 8: 28 / 34 for 2048; n = 20, kd = 4:
// 190 / 291 for 16384; n = 40, kd = 2: 1297 / 1453 for 65536; n = 50, kd = 49: 261 / 336
// for 4096; and the other way n = 32, kd = 12: 46 / 30 for 1024.
// With the chip full, a system costs about 5.6 ns and 5.6 for each panel in tiles
// (another 5.6 for kd > 16, 14.6 instead for kd > 48), and 0.41 (kd = 0) or 0.48 +
// 0.013 kd for each column by columns.  Smaller batches leave the tiles' few workgroups a CU less far behind:
// `percent` is where the two met from 640 to 16384 systems, over n = 9..128 and
// kd = 0..64.  One matrix of up to 8 columns is at launch latency either way.
constexpr bool chol_columns(int64_t n, int64_t kd, int64_t batch) {
    if (n <= 8) return true;
    if (batch <= 512 || n > 256 || kd > 64) return false;
    const int64_t percent = batch < 1024    ? 66
                            : batch < 1536  ? 72
                            : batch < 2048  ? 77
                            : batch < 4096  ? 82
                            : batch < 8192  ? 90
                            : batch < 16384 ? 95
                                            : 100;
    const int64_t panels = (n + 15) / 16;
    const int64_t by_columns = n * (kd == 0 ? 410 : 480 + 13 * kd);
    const int64_t by_tiles = kd > 48 ? 14600 * (panels + 1) : 5600 * (panels + (kd > 16 ? 2 : 1));
    return by_columns * 100 <= by_tiles * percent;
}

// L^T pass (getrs_lt.hip): halves of 2^nbs rows that stage rows n-2 .. 0, n >= 2
// (both sides of the kernel count their barriers by it).
constexpr int lt_halves(int n, int nbs) { return int((unsigned(n - 1) + (1u << nbs) - 1) >> nbs); }

}  // namespace bandlu
