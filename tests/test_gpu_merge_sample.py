"""What the upper-bound workflow reserves for placed rows: an eighth more than the columns counted for 512 rows promise, or, where
they were not all counted or say nothing about the others, every product; and a pass repeated because the counted rows misled."""
import numpy as np
import pytest

from oracle import spgemm as O
from test_gpu_placed_rows import _csr, ob  # noqa: F401
from test_gpu_spgemm import check_result

pytestmark = pytest.mark.gpu


def _counted(rows):
    """The rows whose columns are counted (k_row_products)."""
    turn = np.arange(512, dtype=np.uint64)
    part = rows // 512
    return (turn * part + ((turn * 2654435769 & 0xffffffff) >> 8) % part).astype(np.int64)


# `entries` entries a row, each naming a row of B of 8 entries; a merging row names 8 rows of B four times each
@pytest.mark.parametrize("length, counted", [(32, True), (33, False)])
def test_long_rows_of_b(ob, length, counted):  # noqa: F811
    """A row of B longer than a lane walks: nothing is promised."""
    rng = np.random.default_rng(length)
    B = _csr(64, 600, [np.sort(rng.choice(600, length, replace=False)) for _ in range(64)], rng, np.float64)
    lists = [np.resize(rng.permutation(64)[:1], 4) for _ in range(9000)]
    A = _csr(9000, 64, lists, rng, np.float64)
    C, st = ob.spgemm(ob.to_device(A), ob.to_device(B), workflow=ob.WF_UPPER_BOUND)
    check_result(C, O.multiply_rows(A, B), A, f"rows of B of {length}")
    products = 9000 * 4 * length
    assert st["stage_ms"]["binning"] == 0.0
    assert st["temp_slots"] == (int(products / 4 * 1.125 + 4096.0) if counted else products)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("rows, entries, merging, expect", [
    (2048, 32, "all", "counted"), (2049, 32, "all", "counted"), (9001, 32, "all", "counted"), (2047, 32, "all", "products"),
    (2048, 33, "all", "products"), (4096, 32, "counted", "counted"), (4096, 32, "others", "products"), (4096, 32, "none", "products"),
    (70001, 1, "one", "products")])
def test_reservation(ob, rows, entries, merging, expect, dtype):  # noqa: F811
    rng = np.random.default_rng(rows + entries)
    n = 8 * 64
    columns = rng.permutation(n).reshape(64, 8)   # disjoint, in no order
    if dtype == np.float64:
        columns = np.sort(columns, axis=1)
    B = _csr(64, n, list(columns), rng, dtype)
    lists = [rng.permutation(64)[:entries] for _ in range(rows)]
    merge = {"all": range(rows), "counted": _counted(rows), "others": np.setdiff1d(np.arange(rows), _counted(rows) if rows >= 512 else []),
             "none": [], "one": []}[merging]
    for r in merge:
        lists[r] = np.resize(rng.permutation(64)[:8], entries)
    if merging == "one":
        lists[5] = np.resize(rng.permutation(64)[:8], 9)   # more than 8 times the average, and few enough to be placed still
    A = _csr(rows, 64, lists, rng, dtype)
    products = 8 * sum(len(x) for x in lists)
    dA, dB = ob.to_device(A), ob.to_device(B)
    ref = O.multiply_rows(A, B)
    for _ in range(2):
        C, st = ob.spgemm(dA, dB, workflow=ob.WF_UPPER_BOUND)
        check_result(C, ref, A, f"{rows} {entries} {merging}")
        assert st["stage_ms"]["binning"] == 0.0
        had = st["temp_slots"] if st["nnz_c"] <= st["temp_slots"] else st["nnz_c"]   # (reserved again if too little)
        trimmed = had - st["nnz_c"] > had // 8 and had - st["nnz_c"] > 65536
        assert C.col_idx.untyped_storage().nbytes() // 4 == (st["nnz_c"] if trimmed else had)
        assert trimmed == (merging in ("all", "others") and expect == "products")
        assert st["temp_slots"] == (int(products / 4 * 1.125 + 4096.0) if expect == "counted" else products)
