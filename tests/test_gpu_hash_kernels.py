"""The hash-table kernels on rows that are sorted by default (force_hash_kernels: no row is): the tables of every size in
each workflow, filled to the last slot, and overflowing, against the CPU oracle.  They take such rows where the rows have more
than 64 entries, the column ids leave no room for a product's number in a 32-bit key, or the products fall on few columns."""
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


@pytest.mark.parametrize("name", ["er", "laplacian", "rmat", "rect", "clustered"])
def test_workloads_in_hash_tables(ob, name):
    """(clustered: columns close together, so the tables of 512 and 1024 slots order their rows through narrow buckets)"""
    A, B, _ = W.make(name, small=True)
    ref = O.multiply_rows(A, B)
    dA, dB = ob.to_device(A), ob.to_device(B)
    for kw in (dict(workflow=ob.WF_UPPER_BOUND), dict(workflow=ob.WF_HLL), dict(workflow=ob.WF_SYMBOLIC), dict(workflow=ob.WF_AUTO)):
        Cd, st = ob.spgemm(dA, dB, force_hash_kernels=1, **kw)
        check_result(Cd, ref, A, f"{name} {kw}")
    for scale in (0.25, 0.6):      # tables and reservations too small
        Cd, st = ob.spgemm(dA, dB, workflow=ob.WF_HLL, estimate_scale=scale, force_hash_kernels=1)
        check_result(Cd, ref, A, f"{name} scale {scale}")
        assert st["overflow_rows"] > 0 or scale > 0.25 or name in ("er", "laplacian")


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("clustered", [False, True])
def test_tables_filled_to_the_last_slot(ob, clustered, dtype):
    """Rows of one entry less than, as many as and one more than a table has slots, in tables of exactly that many; scattered
    columns, and columns side by side with one far away, which leave the buckets of the ordered write-out unequal."""
    rng = np.random.default_rng(1 + clustered)
    n = 300000
    sizes = [k + d for k in (16, 32, 64, 256, 512, 1024, 2048, 4096) for d in (-1, 0, 1)] * 4
    rows = [np.concatenate([[0], n - k + 1 + np.arange(k - 1)]) if clustered else np.sort(rng.choice(n, k, replace=False))
            for k in rng.permutation(sizes)]
    ptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
    B = CSR(len(rows), n, ptr, np.concatenate(rows).astype(np.int32), rng.uniform(-1, 1, int(ptr[-1])).astype(dtype))
    # two entries of A on the same row of B: twice the products, the same keys
    a_col = np.repeat(rng.permutation(len(rows)), 2).astype(np.int32)
    A = CSR(len(rows), len(rows), np.arange(len(rows) + 1, dtype=np.int64) * 2, a_col, rng.uniform(0.5, 1, a_col.size).astype(dtype))
    ref = O.multiply_rows(A, B)
    for kw in (dict(workflow=ob.WF_SYMBOLIC, exact_load_coef=1.0), dict(workflow=ob.WF_SYMBOLIC),
               dict(workflow=ob.WF_UPPER_BOUND, bound_load_coef=1.0), dict(workflow=ob.WF_HLL, estimate_scale=0.7)):
        Cd, st = ob.spgemm(ob.to_device(A), ob.to_device(B), force_hash_kernels=1, **kw)
        check_result(Cd, ref, A, f"clustered {clustered} {kw}")
        if "exact_load_coef" in kw:
            assert st["rows_per_bin"][:9] == [8, 12, 12, 12, 12, 12, 12, 12, 4]
