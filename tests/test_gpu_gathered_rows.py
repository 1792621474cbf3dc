"""Placed rows most of whose products lie in a window of a few hundred columns (part_products in placed.hip): every number of
entries, rests from none to more than half of the products, windows at both ends of the columns, columns in no order, repeated
ones, products of -0 and products that are no numbers, against the CPU oracle."""
import numpy as np
import pytest

from oracle import spgemm as O
from paper_2604_19004_amd.workloads import CSR
from test_gpu_spgemm import check_result

pytestmark = pytest.mark.gpu

LENGTH = 30                        # entries of a row of B
OUTSIDE = (0, 1, 3, 8, 15, 20)     # of them outside the window


@pytest.fixture(scope="module")
def ob():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2604_19004_amd import binding
    binding.load()
    return binding


def _csr(rows, cols, lists, values):
    ptr = np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int64)
    idx = np.concatenate([np.asarray(x, dtype=np.int64) for x in lists]).astype(np.int32)
    return CSR(rows, cols, ptr, idx, values(idx.size))


def _matrices(rng, n, start, width, order, values):
    lists = []
    for outside in OUTSIDE:
        for _ in range(64):
            cols = np.concatenate([start + rng.choice(width, LENGTH - outside, replace=order == "repeated"), rng.choice(n, outside, replace=False)])
            lists.append(cols if order == "unsorted" else np.sort(cols))
    B = _csr(len(lists), n, lists, values)
    # every number of entries from 9 (270 products) on, of every kind of row; every fifth row has some of another kind as well
    rows = []
    for entries in range(9, 65):
        for kind in range(len(OUTSIDE)):
            row = 64 * kind + rng.permutation(64)[:entries]
            if entries % 5 == 0:
                row[: entries // 3] = rng.integers(0, len(lists), entries // 3)
            rows.append(np.sort(row))
    A = _csr(len(rows), len(lists), rows, values)
    return A, B


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("order", ["sorted", "unsorted", "repeated"])
@pytest.mark.parametrize("start, width, n", [(0, 60, 20000), (9000, 128, 20000), (19750, 250, 20000), (40, 200, 300), (100, 500, 700)])
def test_rows_that_gather(ob, start, width, n, order, dtype):
    rng = np.random.default_rng(start + width)
    A, B = _matrices(rng, n, start, width, order, lambda k: rng.choice(np.array([-1.5, -0.0, 0.0, 0.25, 3.0], dtype=dtype), k) + rng.integers(0, 2, k).astype(dtype) * rng.uniform(-1, 1, k).astype(dtype))
    ref = O.multiply_rows(A, B)
    for options in (dict(workflow=ob.WF_UPPER_BOUND, dense_range=0), dict(workflow=ob.WF_UPPER_BOUND), dict()):
        C, st = ob.spgemm(ob.to_device(A), ob.to_device(B), **options)
        check_result(C, ref, A, f"{start} {width} {options}")
        if "dense_range" in options:
            assert st["stage_ms"]["binning"] == 0.0, st["stage_ms"]


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_infinities_and_nan_among_rows_that_gather(ob, dtype):
    rng = np.random.default_rng(11)
    A, B = _matrices(rng, 20000, 5000, 128, "sorted", lambda k: rng.choice(np.array([1.0, -2.0, 0.5, 0.0], dtype=dtype), k))
    B.val[rng.choice(B.val.size, 40, replace=False)] = rng.choice([np.inf, -np.inf, np.nan], 40)
    with np.errstate(invalid="ignore"):
        ref = O.multiply_rows(A, B)
    C, st = ob.spgemm(ob.to_device(A), ob.to_device(B), workflow=ob.WF_UPPER_BOUND, dense_range=0)
    assert st["stage_ms"]["binning"] == 0.0
    assert np.array_equal(C.row_ptr.cpu().numpy(), ref.row_ptr) and np.array_equal(C.col_idx.cpu().numpy(), ref.col_idx)
    assert np.array_equal(C.val.cpu().numpy().astype(np.float64), ref.val.astype(np.float64), equal_nan=True)   # (sums of few small numbers: exact)
