"""Rows of many products in the symbolic pass (bitmaps marked tile by tile) against the CPU oracle: numbers of columns at which
the bitmap's size and the workgroup's change, rows at the limits between the two launches, more entries than a chunk holds, rows of B of
fewer than four entries, and a B of fewer entries than a tile's lane reads."""
import numpy as np
import pytest

import rules
from oracle import spgemm as O
from paper_2604_19004_amd.workloads import CSR

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ob():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2604_19004_amd import binding
    binding.load()
    return binding


def _csr(rows, cols, lists):
    ptr = np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int64)
    idx = np.concatenate([np.asarray(x, dtype=np.int64) for x in lists]).astype(np.int32)
    return CSR(rows, cols, ptr, idx, np.ones(idx.size))


def _counts(ob, A, B, **options):
    got, st = ob.symbolic(ob.to_device(A), ob.to_device(B), opt=ob.default_options(**options))
    assert np.array_equal(got.cpu().numpy(), O.count_rows(A, B))
    return st


@pytest.mark.parametrize("bitmap_query", [-1, 2])
@pytest.mark.parametrize("cols", [9000, 1 << 17, (1 << 17) + 1, 1 << 18, (1 << 18) + 1, (1 << 19) + 5, (1 << 20) + 7])
def test_counts_at_the_bitmap_sizes(ob, cols, bitmap_query):
    rng = np.random.default_rng(cols)
    lists = [np.sort(rng.choice(cols, n, replace=False)) for n in (1, 2, 0, 3, 1)]
    lists += [np.sort(rng.choice(cols, int(n), replace=False)) for n in rng.integers(1, 130, 700)]
    lists += [np.sort(rng.choice(cols, n, replace=False)) for n in (8192, 4096, 4097, 63, 64, 65)]
    B = _csr(len(lists), cols, lists)
    k, long = len(lists), len(lists) - 6
    rows = [list(range(k)), [], [long] * 4, [long] * 4 + [0], [0, 1, 2, 3, 4, long + 2], [long + 1, 1], list(range(5, 600)), list(range(0, k, 3)) + [long, long],
            [long] * 8, [long] * 8 + [0]]
    A = _csr(len(rows), k, [np.asarray(r) for r in rows])
    prod = O.row_products(A, B)
    assert prod[2] == 32768 and prod[3] == 32769 and prod[4] > 4096 and prod[8] == 65536 and prod[9] == 65537
    apart = cols <= 1 << 18
    for n in (9, 10):   # without the last row none has more than 65536 products, and no row stands out
        part = CSR(n, A.cols, A.row_ptr[: n + 1], A.col_idx[: A.row_ptr[n]], A.val[: A.row_ptr[n]])
        st = _counts(ob, part, B, bitmap_query=bitmap_query)
        if apart:   # (both sides of the limit between the launches)
            limit = rules.load().symbolic_few_products(int(prod[:n].sum()), int(prod[:n].max()), 256)
            assert limit == (65536 if n == 9 else 32768)
            assert st["symbolic_rows_per_bin"][6] == int((prod[:n] > limit).sum()) == (0 if n == 9 else int((prod[:n] > 32768).sum()))


def test_a_matrix_of_fewer_entries_than_a_lane_reads(ob):
    B = _csr(4, 70000, [[5], [5, 69999], [], [0, 1, 2, 3]])
    rows = [[0, 1, 3] * 1500, [3] * 1200, [0] * 5000, [2], [1] * 40000]
    A = _csr(len(rows), 4, rows)
    _counts(ob, A, B)
