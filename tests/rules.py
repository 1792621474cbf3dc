"""The dispatch's rules (csrc/rules.hpp) as the host applies them, compiled for the CPU."""
import ctypes
import functools
import os
import subprocess
import tempfile

import numpy as np

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_19004_amd", "csrc")
SOURCE = """
#include "rules.hpp"
extern "C" int heavy_in_tiles(double products, double rows, double entries, double windows) { return ocean::heavy_in_tiles(products, rows, entries, windows); }
extern "C" int middle_in_windows(int n_win, int64_t products, int64_t a_nnz) { return ocean::middle_in_windows(n_win, products, a_nnz); }
extern "C" int symbolic_in_tiles(int64_t b_nnz, int64_t b_cols, int64_t products, int64_t a_nnz) { return ocean::symbolic_in_tiles(b_nnz, b_cols, products, a_nnz); }
extern "C" int64_t symbolic_few_products(int64_t products, int64_t max_row, int n_cu) { return ocean::symbolic_few_products(products, max_row, n_cu); }
extern "C" int sort_bitmap_from(int64_t cols) { return ocean::sort_bitmap_from(cols); }
"""


@functools.lru_cache(maxsize=None)
def load():
    with tempfile.TemporaryDirectory() as d:
        src, lib = os.path.join(d, "rules.cpp"), os.path.join(d, "rules.so")
        with open(src, "w") as f:
            f.write(SOURCE)
        subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, src, "-o", lib], check=True)
        so = ctypes.CDLL(lib)
    so.heavy_in_tiles.argtypes = [ctypes.c_double] * 4
    so.middle_in_windows.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_int64]
    so.symbolic_in_tiles.argtypes = [ctypes.c_int64] * 4
    so.sort_bitmap_from.argtypes = [ctypes.c_int64]
    so.symbolic_few_products.argtypes, so.symbolic_few_products.restype = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int], ctypes.c_int64
    return so


def heavy_in_tiles(st, B):
    """Whether the rows of a call's column windows are walked in tiles, from its statistics and B (whose rows are all looked at here,
    and sampled by the library)."""
    lengths = np.diff(B.row_ptr)
    some = lengths > 0
    first, last = B.col_idx[B.row_ptr[:-1][some]] >> 14, B.col_idx[B.row_ptr[1:][some] - 1] >> 14
    spread = float((lengths[some] * (np.abs(last - first) + 1.0)).sum() / lengths[some].sum())

    def tiles_from(bin_):
        rows, products, entries = (sum(st[k][b] for b in range(bin_, 11)) for k in ("rows_per_bin", "bin_products", "bin_nnz_a"))
        return rows > 0 and bool(load().heavy_in_tiles(products, rows, entries, spread))
    middle = load().middle_in_windows((B.cols + 16383) >> 14, st["products"], round(st["products"] / st["er"]))
    return bool(middle and tiles_from(7)) or tiles_from(8)
