"""The copy of B with its rows in column order that heavy rows get where B's are not, against the CPU oracle: rows of B at
the sizes where a wave's share, a wave's rows and a workgroup's rows end."""
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


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("n", [40000, 50000, 262144, 262145, 1 << 20, (1 << 20) + 1])
@pytest.mark.parametrize("longest", [4096, 4097])
def test_rows_of_every_length(ob, dtype, n, longest):
    """Rows of more than 4096 entries aren't sorted, and B stays as it is.  Rows from a 384th of the columns on are ordered by a bitmap
    of 2^18 columns at a time up to 2^20, shorter ones, and all beyond, by a network, in which equal columns need not stay in order."""
    rng = np.random.default_rng(longest + n)
    lengths = [0, 1, 2, 3, 63, 64, 65, 127, 128, 129, 191, 192, 193, 255, 256, 257, 511, 512, 513, 1000, 2047, 2048, 2049, 4095, longest]
    lengths += [n // 384 - 1, n // 384, n // 384 + 1]
    rows = [rng.choice(n, length, replace=False) for length in lengths * 45]   # (1260: more than one turn of the long rows' workgroups)
    for i, row in enumerate(rows):
        if i % 5 == 0 and row.size > 100:
            row[7:10] = row[50]   # (the bitmap finds a column twice)
    order = rng.permutation(len(rows))
    rows = [rows[i] for i in order]

    def csr(rows, cols):
        ptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
        idx = np.concatenate(rows).astype(np.int32)
        return CSR(len(rows), cols, ptr, idx, rng.uniform(-1, 1, idx.size).astype(dtype))
    B = csr(rows, n)
    A = csr([np.sort(rng.choice(len(rows), 60, replace=False)) for _ in range(60)] + [np.arange(len(rows))], len(rows))
    ref = O.multiply_rows(A, B)
    C, st = ob.spgemm(ob.to_device(A), ob.to_device(B), sort_b_ratio=1e-9)
    check_result(C, ref, A, f"longest {longest}")
    assert st["b_sorted_copy"] == (1 if longest == 4096 else 0)
