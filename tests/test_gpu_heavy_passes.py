"""Rows whose output exceeds the hash tables, at the edges of the passes that accumulate them: pieces of a few entries among
B's first, windows of about as many products as a ranked pass may have entries, stretches of more entries than one pass
takes, more entries of A than one chunk holds, and products of -0 or that underflow to it, against the CPU oracle."""
import numpy as np
import pytest

from oracle import spgemm as O
from paper_2604_19004_amd.workloads import CSR

pytestmark = pytest.mark.gpu

WIN, CAP, CHUNK = 16384, 8192, 512   # columns of a window, entries of a ranked pass, entries of A of a chunk


@pytest.fixture(scope="module")
def ob():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2604_19004_amd import binding
    binding.load()
    return binding


def _csr(rows, cols, lists, values):
    ptr = np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int64)
    idx = np.concatenate([np.asarray(x, dtype=np.int32) for x in lists])
    return CSR(rows, cols, ptr, idx, values(idx.size))


def _check(ob, A, B, **options):
    ref = O.multiply_rows(A, B)
    C, st = ob.spgemm(ob.to_device(A), ob.to_device(B), **options)
    assert sum(st["rows_per_bin"][8:11]) > 0, "no row reaches the kernel under test"
    assert np.array_equal(C.row_ptr.cpu().numpy(), ref.row_ptr) and np.array_equal(C.col_idx.cpu().numpy(), ref.col_idx)
    val = C.val.cpu().numpy()
    # sums of up to a few thousand terms in any order: (terms - 1) * 2^-53 of sum |a b|, and one rounding to the result's type
    tol = 1e-12 if val.dtype == np.float64 else 2e-7
    # (a product of 4 bytes that underflows is off by up to the smallest subnormal number; the oracle multiplies in 64 bits)
    lost = 0.0 if val.dtype == np.float64 else float(np.finfo(np.float32).smallest_subnormal) * int(np.diff(A.row_ptr).max())
    assert np.all(np.abs(val.astype(np.float64) - ref.val) <= tol * ref.absval + lost)
    return val


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("first", [(1, 1, 1), (2, 1, 0), (3, 0, 1), (0, 2, 5), (63, 64, 65)])
def test_pieces_among_the_first_entries_of_b(ob, first, dtype):
    rng = np.random.default_rng(sum(first))
    cols = 18 * WIN + 77   # (more windows than a stretch has)
    lists = [np.sort(rng.choice(cols, n, replace=False)) for n in first]
    lists += [np.sort(rng.choice(cols, int(n), replace=False)) for n in rng.integers(1, 900, 60)]
    lists += [np.sort(5 * WIN + rng.choice(WIN, 3000, replace=False)) for _ in range(4)]   # (a dense window)
    B = _csr(len(lists), cols, lists, lambda n: rng.uniform(-1, 1, n).astype(dtype))
    k = len(lists)
    rows = [list(range(k)), [0, 1, 2] + list(range(10, 60)), [0, 1, 2, k - 4, k - 3, k - 2, k - 1], [1] + list(range(3, 40))]
    A = _csr(len(rows), k, rows, lambda n: rng.uniform(-1, 1, n).astype(dtype))
    for workflow in (ob.WF_SYMBOLIC, ob.WF_HLL):
        _check(ob, A, B, workflow=workflow)


@pytest.mark.parametrize("products", [CAP - 1, CAP, CAP + 1, 3 * CAP + 5])
@pytest.mark.parametrize("entries", [3, CHUNK, CHUNK + 1])
def test_products_of_a_window_and_entries_of_a_row(ob, entries, products):
    """One window with `products` products of `entries` entries of A, before, between and behind others."""
    rng = np.random.default_rng(products + entries)
    cols = 20 * WIN
    lists = []
    for i in range(entries):
        n = products // entries + (i < products % entries)
        at = 3 * WIN + np.sort(rng.choice(WIN, min(n, WIN), replace=False))
        around = np.concatenate([rng.choice(3 * WIN, 9000 // entries + 1, replace=False),
                                 4 * WIN + rng.choice(16 * WIN, 30000 // entries + 1, replace=False)])
        lists.append(np.unique(np.concatenate([at, around])))
    B = _csr(entries, cols, lists, lambda n: rng.uniform(-1, 1, n))
    A = _csr(3, entries, [list(range(entries)), [], list(range(entries))], lambda n: rng.uniform(-1, 1, n))
    _check(ob, A, B, workflow=ob.WF_SYMBOLIC)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_products_of_minus_zero_are_entries(ob, dtype):
    """Every entry of C is stored, also where all its products are -0 or underflow to it, in dense windows and in ranked passes."""
    rng = np.random.default_rng(3)
    cols = 17 * WIN
    tiny = np.finfo(dtype).tiny
    lists = [np.sort(rng.choice(2 * WIN, 9000, replace=False)) for _ in range(4)] + [np.sort(rng.choice(cols, 6000, replace=False)) for _ in range(3)]
    B = _csr(len(lists), cols, lists, lambda n: rng.choice(np.array([-0.0, 0.0, tiny, -tiny, 1.0], dtype=dtype), n))
    A = _csr(2, len(lists), [list(range(7)), list(range(3, 7))], lambda n: rng.choice(np.array([-0.0, tiny, -tiny, 1.0], dtype=dtype), n))
    val = _check(ob, A, B, workflow=ob.WF_SYMBOLIC)
    assert np.count_nonzero(val == 0) > 1000 and not np.any(np.signbit(val) & (val == 0))   # (sums start from +0)
