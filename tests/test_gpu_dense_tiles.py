"""The dense-range kernel where it walks the products in tiles of 64 entries of a row of B, and where it does not, against the
CPU oracle: rows of B shorter than a lane's four entries (among them B's first), at and around a tile's length, rows of A
of more entries than the kernel takes at a time, and products that are -0, +0, underflow to them or are no numbers."""
import numpy as np
import pytest

from oracle import spgemm as O
from paper_2604_19004_amd.workloads import CSR
from test_gpu_spgemm import check_result

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ob():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2604_19004_amd import binding
    binding.load()
    return binding


def _csr(rows, cols, rng, dtype):
    ptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
    idx = np.concatenate(rows).astype(np.int32)
    return CSR(len(rows), cols, ptr, idx, rng.uniform(-1, 1, idx.size).astype(dtype))


LENGTHS = {"tiles": [1, 2, 3, 4, 5, 60, 61, 63, 64, 65, 67, 68, 127, 128, 129, 200], "no tiles": [1, 2, 3, 4, 5, 7, 8, 15, 16, 17]}


@pytest.mark.parametrize("kind", LENGTHS)
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("span", [900, 2000, 4096])
def test_tiles_of_dense_rows(ob, span, dtype, kind):
    rng = np.random.default_rng(span)
    lengths = LENGTHS[kind]
    n, low = span + 40, 17
    # (the first rows of B are the shortest, so that tiles end among its first entries)
    b_rows = [low + np.sort(rng.choice(span, length, replace=False)) for length in lengths for _ in range(40)]
    entries = [520, 600, 255, 256, 257, 300, 511, 512, 513] * 8
    a_rows = [np.sort(rng.choice(len(b_rows), min(e, len(b_rows)), replace=False)) for e in entries]
    B = _csr(b_rows, n, rng, dtype)
    A = _csr(a_rows, len(b_rows), rng, dtype)
    A.val[::7] = 0.0
    if dtype == np.float64:   # (the oracle's sums of float32 products are in 64 bits, where nothing underflows)
        A.val[1::7] = -np.finfo(dtype).tiny
        B.val[3::11] = np.finfo(dtype).tiny
    ref = O.multiply_rows(A, B)
    dA, dB = ob.to_device(A), ob.to_device(B)
    nb = len(ob.bin_layout()[0])
    for kw in (dict(workflow=ob.WF_SYMBOLIC), dict(workflow=ob.WF_UPPER_BOUND), dict(tuned_min_products=0.0)):
        C, st = ob.spgemm(dA, dB, dense_range=2, **kw)
        check_result(C, ref, A, f"{kind} {span} {kw}")
        assert (kind == "tiles") == (st["products"] >= 32 * A.col_idx.size)
        if kw.get("workflow") == ob.WF_SYMBOLIC:
            assert st["rows_per_bin"][nb] > 0 and st["overflow_rows"] == 0
    # out of column order the ranges are guesses: products beyond them are noticed
    mixed = _csr([rng.permutation(r) for r in b_rows], n, rng, dtype)
    C, st = ob.spgemm(dA, ob.to_device(mixed), dense_range=2, workflow=ob.WF_UPPER_BOUND)
    check_result(C, O.multiply_rows(A, mixed), A, f"{kind} {span}, rows of B in no order")


@pytest.mark.parametrize("kind", LENGTHS)
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("span", [900, 2000, 4096])
def test_infinities_and_nan_among_dense_rows(ob, span, dtype, kind):
    """A column's accumulator tells by -0 that it has no product: infinities, their differences and NaN are products like others."""
    rng = np.random.default_rng(span + 1)
    b_rows = [17 + np.sort(rng.choice(span, length, replace=False)) for length in LENGTHS[kind] for _ in range(40)]
    B = _csr(b_rows, span + 40, rng, dtype)
    A = _csr([np.sort(rng.choice(len(b_rows), min(e, len(b_rows)), replace=False)) for e in (520, 256, 300, 513) * 8], len(b_rows), rng, dtype)
    A.val[:] = rng.choice(np.array([1.0, -2.0, 0.5, 0.0, -0.0], dtype=dtype), A.val.size)
    B.val[:] = rng.choice(np.array([1.0, -1.0, 0.25, -0.0], dtype=dtype), B.val.size)
    B.val[rng.choice(B.val.size, 30, replace=False)] = rng.choice([np.inf, -np.inf, np.nan], 30)
    with np.errstate(invalid="ignore"):
        ref = O.multiply_rows(A, B)
    nb = len(ob.bin_layout()[0])
    for kw in (dict(workflow=ob.WF_SYMBOLIC, dense_range=2), dict(workflow=ob.WF_UPPER_BOUND, dense_range=2), dict(tuned_min_products=0.0)):
        C, st = ob.spgemm(ob.to_device(A), ob.to_device(B), **kw)
        assert st["rows_per_bin"][nb] > 0
        assert np.array_equal(C.row_ptr.cpu().numpy(), ref.row_ptr) and np.array_equal(C.col_idx.cpu().numpy(), ref.col_idx)
        val = C.val.cpu().numpy().astype(np.float64)
        assert np.array_equal(val, ref.val.astype(np.float64), equal_nan=True)   # (sums of few small numbers: exact)
        assert np.isnan(val).any() and np.isinf(val).any() and not np.any(np.signbit(val) & (val == 0))
