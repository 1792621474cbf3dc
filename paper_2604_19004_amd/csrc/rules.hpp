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

// Whether rows that are accumulated in column windows (`rows` of them, `products` products, `entries` entries of A) are walked in
// tiles: where what a pass finds of a row of B fills half a tile on average.  A pass has as many windows as hold 8192
// entries of C, one at least and sixteen at most; the entries of a row of B lie all over `windows` windows.
// Numeric stage one by one and in tiles, fp64, rows of B of equal length with columns anywhere, us (entries per pass): 1 window, rows
// of 223 000 products 284 and 389 (16), 273 and 273 (32), 277 and 223 (48), 334 and 205 (64); 4 windows, 260 000 649 and 1370 (4),
// 523 and 842 (8), 430 and 532 (16), 383 and 433 (24), 393 and 381 (32); 8 windows, 59 000 1258 and 1778 (7), 791 and 892 (18),
// 753 and 765 (26), 644 and 645 (35); 64 windows, 16 000 1.31 times (8), 1.12 (16), 0.95 (32); 128 windows 1.17 (16), 1.10 (24),
// 1.06 (32).  Columns in blocks of 8000 of 800 000 (1.5 windows), rows of 100 000 866 and 764 (67), of 60 000 1352 and 1496 (20).  Power-law matrices are in favour of tiles by 0.77 to 1.02 from 41 entries per pass on: their products lie in long rows.
constexpr bool heavy_in_tiles(double products, double rows, double entries, double windows)
{
    double share = 8192.0 * rows / products;   // of the columns, in a pass
    if (share > 16.0 / windows) share = 16.0 / windows;
    if (share < 1.0 / windows) share = 1.0 / windows;
    if (share > 1.0) share = 1.0;
    return products * share >= 32.0 * entries;
}

// Whether rows of the 4096-slot bin may go through n_win column windows (in tiles), too; those of the 8192-slot bin always cost less there
// than in hash tables.  12 000 rows of 3040 products, fp64, symbolic workflow, whole call hashed and in windows, 1 / 16 / 64 windows: rows
// of B of 8 entries 810 -> 999, 1142 -> 1175, 1378 -> 3102 us; of 16 783 -> 844, 1362 -> 969, 1614 -> 2232; of 32 775 -> 721, 1814 -> 1440,
// 2065 -> 1709; of 256 1069 -> 802, 1804 -> 1290, 4317 -> 3715; numeric stage of 20 000 rows of 3000, 32 windows, of 64 847 -> 918, of 250
// 856 -> 803, of 1000 886 -> 799.  R-MAT of scale 14 642 -> 619 us, of scale 18 (16 windows) 13.03 -> 12.86 ms.  With 64 windows rows
// of equal length gain, the power-law matrix does not (scale 20 105.6 and 105.8): there the tables stay.
constexpr bool middle_in_windows(int n_win, int64_t products, int64_t a_nnz)
{
    return n_win <= 32 && products >= (n_win <= 16 ? 32 : 128) * a_nnz;
}

// Whether the symbolic pass marks its bitmaps in tiles (from the mean entries of a row of B per entry of A).  Call in us one by one
// and in tiles, rows of B of equal length with columns anywhere: 65 536 columns, rows of 6000 products 332 and 503 (2 entries),
// 202 and 189 (8), 194 and 156 (12), 202 and 141 (16), rows of 24 000 434 and 714 (2), 258 and 277 (8), 187 and 177 (12);
// 2^20 columns, where a compute unit has one workgroup, 6000 217 and 287 (8), 237 and 215 (16), 226 and 201 (24), 100 000 373 and
// 535 (8), 312 and 398 (16), 303 and 323 (24), 271 and 287 (32), 215 and 204 (48); 2^22 columns, four windows, 100 000 742 and
// 1472 (8), 671 and 824 (24), 564 and 676 (32), 419 and 412 (48).
constexpr bool symbolic_in_tiles(int64_t b_nnz, int64_t b_cols, int64_t products, int64_t a_nnz)
{
    return b_nnz >= TILE_MIN_ENTRIES && products >= (b_cols <= 1 << 18 ? 10 : b_cols <= 1 << 20 ? 20 : 40) * a_nnz;
}

// Products up to which a row is counted by a workgroup of 512 threads, in a launch of its own behind that of the larger ones (a
// workgroup of 1024, drawn from a counter).  The largest row decides how long a launch takes, so where none stands out (by 65536
// products, or by twice a compute unit's share of all products and 2^19) every row goes with the smaller workgroups, of which the
// chip works on twice as many.  Call in us with all rows in the smaller ones, split at 32768, at 65536 and at 524288: one row of 4 M
// products beside 4000 of 10 000 535, 394, 392, 393; 250 rows of 1.5 M (rows of B of 1000) 280, 215, 214, 212; 64 of 256 000 beside
// 40 000 of 2500 244, 275, 268, 244; 1000 of 300 000 (32) 416, 458, 457, 417; 2000 of 60 000 (64) 164, 178, 164, 162; R-MAT (16)
// of scale 13 144, 151, 158, 144, 14 177, 184, 189, 178, 16 440, 446, 451, 529, 17 883, 818, 830, 955, 18 1980, 1664, 1730, 2066.
constexpr int64_t symbolic_few_products(int64_t products, int64_t max_row, int n_cu)
{
    const int64_t share = 2 * products / n_cu < 1 << 19 ? 2 * products / n_cu : 1 << 19;
    return max_row <= (share > 65536 ? share : 65536) ? max_row : 32768;
}

// ---- the copy of B with its rows in column order (order.hip) ----
// Entries from which a row of more than 128 is ordered by a bitmap over the columns, 262 144 at a time, instead of a network: the
// bitmap is cleared and counted whatever the row, and beyond four turns of it is not worth it at 4096 entries, where both end.
// (Figures at the kernels.)
constexpr int SORT_BITMAP_LEAST = 129, SORT_BITMAP_NONE = 4097;
constexpr int sort_bitmap_from(int64_t cols)
{
    return cols > 1 << 20 ? SORT_BITMAP_NONE : cols / 384 > SORT_BITMAP_LEAST ? (int)(cols / 384) : SORT_BITMAP_LEAST;
}

}  // namespace ocean
