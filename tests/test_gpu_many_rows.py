"""Binning, row placement and row counting at the numbers of rows where their tiles change size, end, or have their sums
scanned beforehand, against the CPU oracle."""
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


# 256, 1024 and 2048 rows per tile up to 65536, up to 262144 and beyond; more than 4096 tiles from 8 388 609 rows on
@pytest.mark.parametrize("rows", [1, 255, 256, 257, 65536, 65537, 262143, 262145, 8388609])
def test_rows_at_the_edges_of_the_tiles(ob, rows):
    rng = np.random.default_rng(rows)
    k, n = 60, 500
    b_len = np.concatenate([[0], rng.integers(1, 60, k - 1)])
    b_ptr = np.concatenate([[0], np.cumsum(b_len)]).astype(np.int64)
    B = CSR(k, n, b_ptr, np.concatenate([np.sort(rng.choice(n, x, replace=False)) for x in b_len]).astype(np.int32),
            rng.uniform(-1, 1, int(b_ptr[-1])))
    a_len = np.where(rng.random(rows) < min(1.0, 3e5 / rows), rng.integers(0, 5, rows), 0)
    a_len[-1] = 3                                    # the last row of the last tile has entries
    a_ptr = np.concatenate([[0], np.cumsum(a_len)]).astype(np.int64)
    A = CSR(rows, k, a_ptr, rng.integers(0, k, int(a_ptr[-1])).astype(np.int32), rng.uniform(-1, 1, int(a_ptr[-1])))
    ref = O.multiply_rows(A, B)
    dA, dB = ob.to_device(A), ob.to_device(B)
    for kw in (dict(workflow=ob.WF_UPPER_BOUND), dict(workflow=ob.WF_SYMBOLIC), dict(workflow=ob.WF_HLL, estimate_scale=0.5)):
        Cd, st = ob.spgemm(dA, dB, **kw)
        check_result(Cd, ref, A, f"{rows} rows {kw}")
        assert sum(st["bin_nnz_c"]) == ref.col_idx.size or st["overflow_rows"] > 0
        assert sum(st["bin_nnz_a"]) == int(a_len[O.row_products(A, B) > 0].sum())
