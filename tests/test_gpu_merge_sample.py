"""What is reserved for placed rows.  Upper-bound workflow: an eighth more than the columns counted for 512 rows promise, or, where
they were not all counted or say nothing about the others, every product; and a pass repeated because the counted rows misled.
The other workflows: what the columns of sampled rows promise."""
import numpy as np
import pytest

from oracle import hll as ohll
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


def _count(cols):
    """Different columns as they are counted: by 17 bits of their hashes (linear counting)."""
    places = 1 << 17
    return np.rint(-places * np.log1p(-np.unique(ohll.hash32(cols) >> (32 - 17)).size / places))


def _promised(ob, A, B, prod):
    """What the counted rows of a sample promise, four standard errors and a 64th more."""
    sampled = ob.sample_rows(A.rows)
    counted = sampled[np.arange(512) * sampled.size // 512]
    p, c = np.zeros(512), np.zeros(512)
    for i, r in enumerate(counted):
        entries = A.col_idx[A.row_ptr[r]:A.row_ptr[r + 1]]
        p[i] = c[i] = prod[r]
        if 0 < entries.size <= 256:
            c[i] = min(p[i], _count(np.concatenate([B.col_idx[B.row_ptr[k]:B.row_ptr[k + 1]] for k in entries])))
    per = c.sum() / p.sum()
    error = np.sqrt(max(0.0, ((c - per * p) ** 2).sum())) / c.sum()
    return int(prod.sum() * per * (1 + 1 / 64 + 4 * error) + 4096)


# entries of A of a row, rows of B, their entries, columns; numbers of columns for which sketches say an eighth too little
@pytest.mark.parametrize("entries, k, length, n, all_counted", [(34, 2000, 60, 1500, True), (40, 1000, 30, 400, True), (20, 1000, 20, 300, True),
                                                                (2, 40, 1000, 3500, True), (0, 1000, 8, 5000, True), (257, 2000, 9, 1500, False)])
def test_sample_counts_columns(ob, entries, k, length, n, all_counted):  # noqa: F811
    """No pass is repeated for an error that all rows' sketches have in common."""
    rng = np.random.default_rng(n)
    B = _csr(k, n, [[]] + [np.sort(rng.choice(n, length, replace=False)) for _ in range(k - 1)], rng, np.float64)
    lists = [rng.choice(k, entries or int(rng.integers(0, 65)), replace=False) for _ in range(4000)]
    lists[7] = []
    if entries == 0:                                     # half of the rows merge four times over
        lists = [np.resize(x[: (len(x) + 3) // 4], len(x)) if r % 2 else x for r, x in enumerate(lists)]
    A = _csr(len(lists), k, lists, rng, np.float64)
    C, st = ob.spgemm(ob.to_device(A), ob.to_device(B), tuned_min_products=0.0)
    check_result(C, O.multiply_rows(A, B), A, f"{entries} entries, {n} columns")
    assert st["stage_ms"]["binning"] == 0.0 and st["sampled_rows"] > 512
    prod = O.row_products(A, B)
    promised = _promised(ob, A, B, prod)
    slots = C.col_idx.untyped_storage().nbytes() // 4
    if all_counted:
        assert st["nnz_c"] < slots < prod.sum() and abs(slots - promised) <= 2
    else:                                                # a bound was reserved, and C trimmed
        assert promised > prod.sum() and slots == st["nnz_c"]


@pytest.mark.parametrize("validate", [1, 0])
def test_upper_bound_counts_columns_of_large_rows(ob, validate):  # noqa: F811
    """50 million products in rows of more than 128: counted, and sorted straight to C or not; an A out of range is refused."""
    rng = np.random.default_rng(11)
    B = _csr(2000, 1500, [np.sort(rng.choice(1500, 25, replace=False)) for _ in range(2000)], rng, np.float32)
    A = _csr(170000, 2000, list(rng.integers(0, 2000, (170000, 12))), rng, np.float32)
    dA, dB = ob.to_device(A), ob.to_device(B)
    C, st = ob.spgemm(dA, dB, workflow=ob.WF_UPPER_BOUND, validate_inputs=validate)
    check_result(C, O.multiply_rows(A, B), A, "counted")
    assert st["stage_ms"]["binning"] == 0.0 and abs(st["temp_slots"] - _promised(ob, A, B, O.row_products(A, B))) <= 2
    assert st["nnz_c"] < st["temp_slots"] == C.col_idx.untyped_storage().nbytes() // 4
    if validate:
        dA.col_idx[12345] = 2000
        with pytest.raises(ob.OceanError):
            ob.spgemm(dA, dB, workflow=ob.WF_UPPER_BOUND)
