"""The fall-back of AUTO to two passes (the estimation workflow's output did not fit) when B's rows are out of column order:
the column ranges taken from the ends of such rows are guesses, and what the first round learned about B's order has to
outlive the check of its sorted copy.  Against the CPU oracle."""
import ctypes

import numpy as np
import pytest

from oracle import spgemm as O
from paper_2604_19004_amd import workloads as W
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


def _case(dtype, long_row):
    """B: 2048 shuffled rows of 64 entries (heavy rows of A reach tens of thousands of columns through them), 40 rows over
    2000 columns whose first and last entry lie 200 columns apart, and on request one row of 5000 entries, in order, which is
    more than the sorted copy takes.  A: 80 heavy rows, 40 rows over the narrow ones, and empty rows that keep the average
    below 64 products, so that AUTO reserves the product bound without a sample."""
    rng = np.random.default_rng(5 + long_row)
    n = 1 << 17
    heavy = W.erdos_renyi(2048, 64, seed=32, cols=n)
    b_rows = [rng.permutation(heavy.col_idx[i * 64:(i + 1) * 64]) for i in range(2048)]
    for _ in range(40):
        inner = rng.permutation(np.setdiff1d(np.arange(2000), np.arange(900, 1101)))[:60]
        b_rows.append(50000 + np.concatenate([[900], inner, [1100]]))
    if long_row:
        b_rows.append(np.sort(rng.choice(n, 5000, replace=False)))
    a_rows = [rng.choice(2048, k, replace=False) for k in [1500] * 40 + [700] * 40]
    a_rows += [2048 + rng.choice(40, 12, replace=False) for _ in range(40)]
    if long_row:
        a_rows[0][0] = len(b_rows) - 1
    a_rows += [np.zeros(0, np.int64)] * 100000

    def csr(rows, cols):
        ptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
        idx = np.concatenate(rows).astype(np.int32)
        return CSR(len(rows), cols, ptr, idx, rng.uniform(-1, 1, idx.size).astype(dtype))
    return csr(a_rows, len(b_rows)), csr(b_rows, n)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("long_row", [False, True], ids=["copy taken", "copy refused"])
def test_ranges_are_given_up_on_the_way_to_two_passes(ob, monkeypatch, dtype, long_row):
    A, B = _case(dtype, long_row)
    ref = O.multiply_rows(A, B)
    prod = np.minimum(O.row_products(A, B), B.cols)
    slab = int(prod[prod > 4096].sum()) * 4        # the output's column ids are the first request of at least the heavy rows'
    refused = []

    class RefusesTheSlabOnce(ob.TorchAllocator):
        def __init__(self, device):
            super().__init__(device)
            plain = self._alloc_cb

            def alloc(ctx, nbytes, out):
                if int(nbytes) >= slab and not refused:
                    refused.append(int(nbytes))
                    return 1
                return plain(ctx, nbytes, ctypes.cast(out, ctypes.POINTER(ctypes.c_void_p)))
            self._alloc_once = ob.ALLOC_FN(alloc)
            self.struct = ob.ocean_allocator(None, self._alloc_once, self._release_cb)

    monkeypatch.setattr(ob, "TorchAllocator", RefusesTheSlabOnce)
    Cd, st = ob.spgemm(ob.to_device(A), ob.to_device(B), dense_range=2)
    assert refused and st["fell_back"] == 1 and st["workflow"] == "symbolic"
    assert st["b_sorted_copy"] == (0 if long_row else 1)
    check_result(Cd, ref, A, f"fall-back, long row {long_row}")
