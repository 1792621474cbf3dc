"""Rows that are written to their place in C as they are sorted (placed.hip) against the CPU oracle and the general path:
numbers of rows at the edges of the units and of the placing turns, every size of sort alone and all sizes in one matrix, rows of
B in no order and with repeated columns, a reservation that turns out too small, and one of which little is used.  A call went
this way when it shows no binning stage."""
import numpy as np
import pytest

from oracle import spgemm as O
from paper_2604_19004_amd.workloads import CSR
from test_gpu_spgemm import check_result

pytestmark = pytest.mark.gpu

CLASSES = (32, 64, 96, 128, 192, 256, 384, 512, 768, 1024, 1536, 2048)


@pytest.fixture(scope="module")
def ob():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2604_19004_amd import binding
    binding.load()
    return binding


def _csr(rows, cols, lists, rng, dtype):
    ptr = np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int64)
    idx = np.concatenate([np.asarray(x, dtype=np.int64) for x in lists]).astype(np.int32)
    return CSR(rows, cols, ptr, idx, rng.uniform(-1, 1, idx.size).astype(dtype))


def _b(rng, n, dtype, order):
    """An empty row, then rows of 1 .. 64 entries at random columns and 64 rows of those lengths on 80 columns."""
    lists = [[]]
    for low, span in ((0, n), (n - 80, 80)):
        for length in range(1, 65):
            cols = low + rng.choice(span, length, replace=order == "repeated")
            lists.append(cols if order == "unsorted" else np.sort(cols))
    return _csr(len(lists), n, lists, rng, dtype)


def _row(rng, total, most=64):
    """Entries of A whose rows of B have `total` entries together."""
    row = []
    longest = max(1, min(64, -(-total // 30)))
    while total > 0 and len(row) < most:
        step = min(total, int(rng.integers(max(1, longest // 2), longest + 1)))
        row.append(step + 64 * int(rng.integers(0, 2)))
        total -= step
    return row


def _check(ob, A, B, label, placed=True, **options):
    dA, dB = ob.to_device(A), ob.to_device(B)
    ref = O.multiply_rows(A, B)
    C, st = ob.spgemm(dA, dB, **options)
    check_result(C, ref, A, f"{label} {options}")
    assert (st["stage_ms"]["binning"] == 0.0) == placed, (label, st["stage_ms"])
    with_products = O.row_products(A, B) > 0
    assert st["nnz_c"] == ref.col_idx.size == sum(st["bin_nnz_c"])
    assert sum(st["rows_per_bin"]) == int(with_products.sum())
    assert sum(st["bin_products"]) == st["products"]
    assert sum(st["bin_nnz_a"]) == int(np.diff(A.row_ptr)[with_products].sum())
    return C, st


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("order", ["sorted", "unsorted", "repeated"])
@pytest.mark.parametrize("cap", CLASSES)
def test_each_size_of_sort(ob, cap, order, dtype):
    rng = np.random.default_rng(cap)
    B = _b(rng, 5000, dtype, order)
    smaller = ([0] + list(CLASSES))[CLASSES.index(cap)] + 1
    most = 32 if cap == 32 else 64
    for rows in (1, 5, 33, 300):
        lists = [_row(rng, int(rng.integers(smaller, cap + 1)), most) for _ in range(rows)]
        lists[0] = _row(rng, cap, most)
        if rows > 1:
            lists[-1] = [0, 0, 0]                      # entries, but no products
            lists[rows // 2] = []
        A = _csr(rows, B.rows, lists, rng, dtype)
        C, st = _check(ob, A, B, f"{cap} products, {rows} rows", workflow=ob.WF_UPPER_BOUND)
        general, st = ob.spgemm(ob.to_device(A), ob.to_device(B), workflow=ob.WF_UPPER_BOUND, compact_in_place=0)
        assert st["stage_ms"]["binning"] > 0.0
        for x, y in ((C.row_ptr, general.row_ptr), (C.col_idx, general.col_idx)):
            assert bool((x == y).all())


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("most", [512, 1024, 1536, 2048])
def test_all_sizes_in_one_matrix(ob, most, dtype):
    rng = np.random.default_rng(most)
    B = _b(rng, 30000, dtype, "sorted")
    lists = [_row(rng, int(rng.choice([0, 1, 60, 130, 190, 250, 380, 500, 700, 1000, 1500, 2000]) % (most + 1))) for _ in range(3001)]
    lists[7] = _row(rng, most)
    A = _csr(len(lists), B.rows, lists, rng, dtype)
    for wf in (ob.WF_UPPER_BOUND, ob.WF_AUTO):
        _check(ob, A, B, f"up to {most} products", workflow=wf)
    # a row with an entry more than the sort takes, or a product: the general way; the same entries without a product are none
    for extra, placed in (([1] * 65, False), ([0] * 65, True), (_row(rng, 2048) + [1], False)):
        A = _csr(len(lists) + 1, B.rows, lists + [extra], rng, dtype)
        assert O.row_products(A, B)[-1] == {65: 65 * (extra[0] > 0)}.get(len(extra), 2049)
        _check(ob, A, B, f"a row of {len(extra)} entries", placed=placed, workflow=ob.WF_UPPER_BOUND)


def _wide_row(rng, entries, total):
    """`entries` entries of A whose rows of B have `total` entries together."""
    row = np.full(entries, total // entries) + (np.arange(entries) < total % entries)
    return rng.permutation(row) + 64 * rng.integers(0, 2, entries) * (row > 0)


# 2 and 7 entries a row: 64 entries are as many as a group of two lanes takes; 9: of four lanes
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("short", [2, 7, 9])
@pytest.mark.parametrize("products", [800, 1500, 2048])
def test_rows_of_64_entries_among_short_ones(ob, products, short, dtype):
    rng = np.random.default_rng(products + short)
    B = _b(rng, 5000, dtype, "sorted")
    lists = [_wide_row(rng, short, 30 * short) for _ in range(4096)]
    for unit in range(4):                               # at each place of a unit of four rows
        lists[400 * unit + unit] = _wide_row(rng, 64, products - unit)
    lists[2001:2004] = [_wide_row(rng, 64, products) for _ in range(3)]
    A = _csr(len(lists), B.rows, lists, rng, dtype)
    for wf in (ob.WF_UPPER_BOUND, ob.WF_AUTO):
        _check(ob, A, B, f"64 entries, {products} products", workflow=wf)
    lists[9] = _wide_row(rng, 65, products)             # an entry more than the sort takes
    A = _csr(len(lists), B.rows, lists, rng, dtype)
    _check(ob, A, B, "65 entries", placed=False, workflow=ob.WF_UPPER_BOUND)


# more than 64 and 128 entries a row on average: groups of 32 and 64 lanes
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("entries", [100, 300])
@pytest.mark.parametrize("products", [257, 800, 2048])
def test_sorted_rows_among_long_ones_without_products(ob, products, entries, dtype):
    rng = np.random.default_rng(products + entries)
    B = _b(rng, 5000, dtype, "sorted")
    lists = [[0] * entries for _ in range(1500)]        # of B's empty row: in no sort class, and none is needed
    for r in range(0, 1500, 7):
        lists[r] = _row(rng, products - r % 5)
    lists[640:644] = [_wide_row(rng, 64, products) for _ in range(4)]
    A = _csr(len(lists), B.rows, lists, rng, dtype)
    assert A.row_ptr[-1] > (128 if entries == 300 else 64) * A.rows
    for wf in (ob.WF_UPPER_BOUND, ob.WF_AUTO):
        _check(ob, A, B, f"{products} products among rows of {entries} entries", workflow=wf)


# units of 32, 16, 8 and 4 rows: around a wave of counts, the 1024 of a turn and several turns
@pytest.mark.parametrize("units", [1, 63, 64, 65, 1023, 1024, 1025, 5000])
@pytest.mark.parametrize("rows_per_unit, products", [(32, 20), (16, 60), (8, 150), (4, 300)])
def test_numbers_of_units(ob, rows_per_unit, products, units):
    rng = np.random.default_rng(units)
    B = _b(rng, 900, np.float64, "sorted")
    for rows in {units * rows_per_unit, units * rows_per_unit - rows_per_unit + 1}:
        lists = [_row(rng, int(p), 32) for p in rng.integers(0, products + 1, rows)]
        lists[0] = _row(rng, products, 32)
        A = _csr(rows, B.rows, lists, rng, np.float64)
        _check(ob, A, B, f"{units} units", workflow=ob.WF_UPPER_BOUND)


def test_sample_that_promises_too_little(ob):
    """The sampled rows' products fall on few columns and nobody else's do: C needs more than was reserved."""
    rng = np.random.default_rng(4)
    rows, n = 20000, 100000
    lists = [np.sort(rng.choice(n, 32, replace=False)) for _ in range(200)] + [np.arange(32) for _ in range(200)]
    B = _csr(400, n, lists, rng, np.float64)
    sampled = np.zeros(rows, bool)
    sampled[ob.sample_rows(rows)] = True
    A = _csr(rows, 400, [rng.choice(200, 6, replace=False) + 200 * sampled[r] for r in range(rows)], rng, np.float64)
    C, st = _check(ob, A, B, "misled sample", tuned_min_products=0.0)
    assert st["sampled_rows"] == sampled.sum() and st["products"] / st["sampled_cr"] * 1.5 < st["nnz_c"]


@pytest.mark.parametrize("columns, kept", [(40, False), (1000, True)])
def test_what_c_keeps_of_the_reservation(ob, columns, kept):
    rng = np.random.default_rng(columns)
    B = _csr(500, columns, [np.sort(rng.choice(columns, 8, replace=False)) for _ in range(500)], rng, np.float32)
    A = _csr(30000, 500, [rng.choice(500, 7, replace=False) for _ in range(30000)], rng, np.float32)
    C, st = _check(ob, A, B, "reservation")
    slots = C.col_idx.untyped_storage().nbytes() // 4
    # (where the columns of 512 rows were counted C keeps what they promise, which the bound below covers: the trim has its
    # cases in test_gpu_merge_sample)
    assert slots == (st["products"] if kept else st["temp_slots"])
    assert slots <= st["nnz_c"] * 8 // 7 + 65536


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("span", [600, 1024, 1025, 2048, 2049, 4096, 4097])
def test_dense_ranges(ob, span, dtype):
    """Rows whose columns lie in a window of exactly `span` columns, up to the accumulator's 4096 and one more; then the
    same rows of B in no order."""
    rng = np.random.default_rng(span)
    windows, per, rows = 5, 70, 700
    n = windows * span + 3
    lists = []
    for w in range(windows):
        for _ in range(per):
            inner = 1 + rng.choice(span - 2, 38, replace=False)
            lists.append(3 + w * span + np.sort(np.concatenate([[0], inner, [span - 1]])))
    B = _csr(len(lists), n, lists, rng, dtype)
    a_lists = [per * int(rng.integers(0, windows)) + rng.choice(per, int(rng.integers(52, per + 1)), replace=False) for _ in range(rows)]
    a_lists[0] = a_lists[rows // 3] = []
    A = _csr(rows, B.rows, a_lists, rng, dtype)
    nb = len(ob.bin_layout()[0])
    C, st = _check(ob, A, B, f"{span} columns", placed=span <= 4096, tuned_min_products=0.0)
    if span <= 4096:
        assert st["rows_per_bin"][nb] == rows - 2
    mixed = _csr(len(lists), n, [rng.permutation(x) for x in lists], rng, dtype)
    mixed.val[:] = B.val
    C, st = ob.spgemm(ob.to_device(A), ob.to_device(mixed), tuned_min_products=0.0)
    check_result(C, O.multiply_rows(A, mixed), A, f"{span} columns, rows of B in no order")
    assert st["stage_ms"]["binning"] > 0.0


def test_ranges_of_rows_that_merge_much(ob):
    """A band of 25 diagonals, 625 products on 49 columns a row: sorted takes 0.8 of what the dense accumulator over the ranges
    does."""
    n, w = 100000, 25
    rng = np.random.default_rng(w)
    cols = np.arange(n)[:, None] + np.arange(w) - w // 2
    inside = (cols >= 0) & (cols < n)
    A = CSR(n, n, np.concatenate([[0], np.cumsum(inside.sum(1))]).astype(np.int64), cols[inside].astype(np.int32),
            rng.uniform(-1, 1, int(inside.sum())))
    dA = ob.to_device(A)
    C, st = ob.spgemm(dA, dA)
    check_result(C, O.multiply_rows(A, A), A, "band of 25")
    assert st["dense_range_rows"] == st["sampled_rows"] and st["rows_per_bin"][len(ob.bin_layout()[0])] == 0
    assert st["stage_ms"]["binning"] == 0.0
