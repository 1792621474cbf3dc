// Rules of the dispatch that are sums over what the host knows of a call.  Plain C++: the CPU tests hold them against
// the measurements that they rest on.
#pragma once

#include <cstdint>

namespace ocean {

// ---- products in tiles of 64 entries of a row of B (tiles.hpp), or numbered one by one ----
constexpr int64_t TILE_MIN_ENTRIES = 8;   // that B has where its rows are walked in tiles (tiles.hpp)
// Whether the dense-range kernel walks its rows in tiles of 64 entries of a row of B: where these have 32 on average.  (60 000 rows
// in blocks of 1000 columns, fp64, whole call, one by one and in tiles: rows of B of 24 entries 416 and 426 us, of 36 488 and 484,
// of 50 564 and 535, of 78 811 and 675; fp32 400 and 398, 445 and 435, 512 and 481, 787 and 610.)
constexpr bool dspan_in_tiles(int64_t b_nnz, int64_t products, int64_t a_nnz)
{
    return b_nnz >= TILE_MIN_ENTRIES && b_nnz < 0xffffffffLL && products >= 32 * a_nnz;
}

// Whether rows that are accumulated in n_win column windows (`rows` of them, `products` products, `entries` entries of A) are walked
// in tiles: where what a pass finds of a row of B fills half a tile on average.  A pass has as many windows as hold 8192
// entries of C, one at least and sixteen at most; a row of B's entries lie all over the windows.
// Numeric stage one by one and in tiles, fp64, rows of B of equal length with columns anywhere, us (entries per pass): 1 window, rows
// of 223 000 products 284 and 389 (16), 273 and 273 (32), 277 and 223 (48), 334 and 205 (64); 4 windows, 260 000 649 and 1370 (4),
// 523 and 842 (8), 430 and 532 (16), 383 and 433 (24), 393 and 381 (32); 8 windows, 59 000 1258 and 1778 (7), 791 and 892 (18),
// 753 and 765 (26), 644 and 645 (35); 64 windows, 16 000 1.31 times (8), 1.12 (16), 0.95 (32); 128 windows 1.17 (16), 1.10 (24),
// 1.06 (32).  Power-law matrices are in favour of tiles by 0.77 to 1.02 from 41 entries per pass on: their products lie in long rows.
constexpr bool heavy_in_tiles(double products, double rows, double entries, int n_win)
{
    double share = 8192.0 * rows / products;   // of the columns, in a pass
    if (share > 16.0 / n_win) share = 16.0 / n_win;
    if (share < 1.0 / n_win) share = 1.0 / n_win;
    if (share > 1.0) share = 1.0;
    return products * share >= 32.0 * entries;
}

}  // namespace ocean
