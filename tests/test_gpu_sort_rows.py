"""The sorting kernel of rows with few products (k_numeric_sort) against the CPU oracle at the edges of its size classes:
rows with one product less and more than a class holds, with as many entries of A as a class takes and one more, with
columns that never and with columns that always merge, and matrices whose column ids just fit or no longer fit beside a
product's number in a 32-bit key.  The hash kernels run the same rows with force_hash_kernels."""
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


def _matrix(rng, rows, n, dtype):
    ptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
    idx = np.concatenate(rows).astype(np.int32)
    return CSR(len(rows), n, ptr, idx, rng.uniform(-1, 1, idx.size).astype(dtype))


def _case(seed, n, dtype, shuffle_b):
    """B: 64 rows of every length 1 .. 64 at random columns, 64 of them inside 96 columns at the end of the range, and an
    empty row.  A: for every class, rows whose products number cap - 1, cap and cap + 1, built from few long and from many
    short rows of B; rows of 63, 64 and 65 entries (empty rows of B among them); empty rows."""
    rng = np.random.default_rng(seed)
    b_rows = [np.zeros(0, np.int64)]
    for low, span in ((0, n), (n - min(n, 96), min(n, 96))):
        for length in range(1, 65):
            cols = low + np.sort(rng.choice(span, length, replace=False))
            b_rows.append(rng.permutation(cols) if shuffle_b else cols)
    a_rows = [[], [0], [0, 0, 0]]
    for cap in CLASSES:
        for total in (cap - 1, cap, cap + 1):
            for base in (0, 64):             # scattered columns, columns that merge
                for longest in (64, max(1, min(64, -(-cap // 40)))):
                    row, left = [], total
                    while left > 0:
                        step = min(left, int(rng.integers(max(1, longest // 2), longest + 1)))
                        row.append(base + step)
                        left -= step
                    a_rows.append(row)
    for ne in (63, 64, 65):
        for filler in (0, 1):                # empty rows of B, rows of one entry
            a_rows.append([filler] * (ne - 3) + [70, 64, 128])
    a_rows = [a_rows[i] for i in rng.permutation(len(a_rows))]
    B = _matrix(rng, b_rows, n, dtype)
    A = _matrix(rng, a_rows, len(b_rows), dtype)
    return A, B


@pytest.mark.parametrize("shuffle_b", [False, True])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
# 2^(32 - bits) columns are one too many for the class whose products are numbered in `bits` bits
@pytest.mark.parametrize("n", [100, (1 << 21) - 1, 1 << 21, (1 << 24) - 1, 1 << 27])
def test_sorted_rows_at_the_edges_of_the_classes(ob, n, dtype, shuffle_b):
    A, B = _case(n % 1000 + 7 * shuffle_b, n, dtype, shuffle_b)
    ref = O.multiply_rows(A, B)
    dA, dB = ob.to_device(A), ob.to_device(B)
    for kw in (dict(workflow=ob.WF_UPPER_BOUND), dict(workflow=ob.WF_SYMBOLIC), dict(workflow=ob.WF_HLL),
               dict(workflow=ob.WF_HLL, estimate_scale=0.4), dict(workflow=ob.WF_UPPER_BOUND, esc_short_rows=1),
               dict(workflow=ob.WF_SYMBOLIC, force_hash_kernels=1), dict(workflow=ob.WF_UPPER_BOUND, force_hash_kernels=1)):
        Cd, st = ob.spgemm(dA, dB, **kw)
        check_result(Cd, ref, A, f"n={n} {kw}")
        assert sum(st["rows_per_bin"]) == int((O.row_products(A, B) > 0).sum())


# Rows per class from which its smallest tables are worth a launch, and columns that fill the largest table that is cheaper
# than sorting (tables ask for 1.5 slots per entry: 32, 64, 256 and 1024 slots).
MANY = {64: (420000, 20), 96: (330000, 20), 128: (240000, 20), 192: (112000, 20), 256: (84000, 20), 384: (56000, 40), 512: (42000, 40),
        768: (34000, 160), 1024: (19000, 160), 1536: (28000, 600), 2048: (7000, 600)}


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("width", [10, None], ids=["10 columns", "largest table"])
def test_classes_whose_products_fall_on_few_columns(ob, width, dtype):
    """Classes of so many rows on few columns that nearly all of them go to hash tables, and among them one row in thirty
    whose products hardly merge, which is sorted.  Rows repeat, so the oracle multiplies each kind once."""
    rng = np.random.default_rng(width or 1)
    n = 5000
    b_rows, kinds, per_kind = [], [], []
    for cap, (many, widest) in MANY.items():
        columns = width or widest
        step = max(1, -(-cap // 60))                 # entries of B's rows, 60 of A's rows at most
        first = len(b_rows)
        for at in range(64):                         # few columns: the same ones over and over
            b_rows.append(np.sort((at * step + np.arange(min(step, columns))) % columns) * (n // columns))
        for at in range(64):                         # hardly any merge
            b_rows.append(np.sort(rng.choice(n, step, replace=False)))
        length = min(step, columns)
        for low, share in ((0, 29), (64, 1)):
            entries = min(64, cap // (length if low == 0 else step))
            for kind in range(3):
                kinds.append(first + low + (np.arange(entries) + 7 * kind) % 64)
                per_kind.append(many * share // 90 + 1)
    order = rng.permutation(np.repeat(np.arange(len(kinds)), per_kind))
    B = _matrix(rng, b_rows, n, dtype)
    head = _matrix(rng, kinds, len(b_rows), dtype)
    ref = O.multiply_rows(head, B)

    def repeated(ptr, *arrays):
        lengths = np.diff(ptr)[order]
        out = np.concatenate([[0], np.cumsum(lengths)])
        at = np.repeat(ptr[:-1][order] - out[:-1], lengths) + np.arange(out[-1])
        return (out, *(x[at] for x in arrays))
    a_ptr, a_col, a_val = repeated(head.row_ptr, head.col_idx, head.val)
    c_ptr, c_col, c_val, c_abs = repeated(ref.row_ptr, ref.col_idx, ref.val, ref.absval)
    A = CSR(order.size, len(b_rows), a_ptr, a_col, a_val)
    whole = type(ref)(0, A.rows, c_ptr, c_col, c_val, c_abs)
    dA, dB = ob.to_device(A), ob.to_device(B)
    for kw in (dict(workflow=ob.WF_SYMBOLIC), dict(workflow=ob.WF_HLL), dict(workflow=ob.WF_HLL, estimate_scale=0.6)):
        Cd, st = ob.spgemm(dA, dB, **kw)
        check_result(Cd, whole, A, f"{width} columns {kw}")
