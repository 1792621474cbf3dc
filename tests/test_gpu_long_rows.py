"""Sketches, merged sketches and product counts of matrices whose long rows sit side by side, at the lengths where a row
passes from the lane groups to the kernels for long rows, against the CPU oracle."""
import numpy as np
import pytest

from oracle import hll as ohll
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


def _matrix(seed, rows, long_lengths):
    """The long rows first, then short ones; square, at least as many columns as the longest row has entries."""
    rng = np.random.default_rng(seed)
    n = max(rows, max(long_lengths))
    lengths = (list(long_lengths) + rng.integers(0, 5, n).tolist())[:rows]
    lengths += [0] * (n - len(lengths))
    idx = [np.sort(rng.choice(n, length, replace=False)) for length in lengths]
    ptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    idx = np.concatenate(idx).astype(np.int32)
    return CSR(n, n, ptr, idx, rng.uniform(-1, 1, idx.size))


@pytest.mark.parametrize("m", [32, 64, 128])
@pytest.mark.parametrize("rows, long_lengths", [(1, [300]), (5, [255, 256, 257]), (4100, [256] * 9 + [1023, 1024, 1025, 4096, 4097]),
                                                (9000, [9000, 8999] + [257] * 40)])
def test_long_rows_side_by_side(ob, rows, long_lengths, m):
    A = _matrix(len(long_lengths) + m, rows, long_lengths)
    dA = ob.to_device(A)
    sk = ob.hll_sketch_rows(dA, m)
    ref_sk = ohll.sketch_rows(A, m)
    assert np.array_equal(sk.cpu().numpy(), ref_sk)
    prod, total, longest = ob.row_products(dA, dA)
    ref_prod = O.row_products(A, A)
    assert np.array_equal(prod.cpu().numpy(), ref_prod) and (total, longest) == (int(ref_prod.sum()), int(ref_prod.max()))
    est, merged = ob.hll_merge_estimate(dA, sk, m, prod=prod, B=dA, want_merged=True)
    ref_merged = ohll.merge_rows(A, ref_sk)
    assert np.array_equal(merged.cpu().numpy(), ref_merged)
    every = ob.hll_merge_estimate(dA, sk, m, rows=_all_rows(A.rows), prod=prod, B=dA)[0]   # (the path with a row list)
    assert np.array_equal(est.cpu().numpy(), every.cpu().numpy())


def _all_rows(n):
    import torch
    return torch.arange(n, dtype=torch.int64, device="cuda:0")


@pytest.mark.parametrize("m", [32, 64, 128])
def test_long_rows_of_a_large_matrix(ob, m):
    """2^20 entries and more: the long rows are merged by a launch of their own, 1024 threads a row.  Estimates bare, and
    limited by the products and the longest row of B."""
    import torch
    rng = np.random.default_rng(m)
    n = 40000
    lengths = rng.integers(0, 52, n)
    lengths[:12] = [255, 256, 257, 4095, 4096, 4097, 30000, 1024, 1023, 300, 0, 40000]      # side by side, and
    lengths[[4096, 8192, 20000, n - 1]] = [5000, 257, 256, 2000]                             # at the ends of stretches
    ptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    assert ptr[-1] >= 1 << 20 and 8 * ptr[-1] / n < 256
    idx = np.concatenate([np.sort(rng.choice(n, k, replace=False)) if k > 52 else rng.integers(0, n, k) for k in lengths]).astype(np.int32)
    A = CSR(n, n, ptr, idx, np.ones(idx.size))
    dA = ob.to_device(A)
    ref_sk = ohll.sketch_rows(A, m)
    sk = ob.hll_sketch_rows(dA, m)
    assert np.array_equal(sk.cpu().numpy(), ref_sk)
    ref_merged = ohll.merge_rows(A, ref_sk)
    est, merged = ob.hll_merge_estimate(dA, sk, m, want_merged=True)
    assert np.array_equal(merged.cpu().numpy(), ref_merged)
    np.testing.assert_allclose(est.cpu().numpy(), ohll.estimate(ref_merged), rtol=1e-12, atol=0)
    prod = torch.from_numpy(O.row_products(A, A)).cuda()
    est = ob.hll_merge_estimate(dA, sk, m, prod=prod, B=dA)[0]
    np.testing.assert_allclose(est.cpu().numpy(), ohll.estimate_rows(A, A, m), rtol=1e-12, atol=0)
