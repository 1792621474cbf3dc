"""Rows whose columns a bitmap counts, on both sides of the line between products in tiles and one by one (symbolic_in_tiles in
csrc/rules.hpp), at every size of the bitmap, against the CPU oracle: more entries of A than a chunk holds, rows of B of one entry
beside long ones, and chunks whose segments are runs of 16 on average beside others."""
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


def _csr(cols, lists):
    ptr = np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int64)
    idx = np.concatenate([np.asarray(x, dtype=np.int64) for x in lists]).astype(np.int32)
    return CSR(len(lists), cols, ptr, idx, np.ones(idx.size))


@pytest.mark.parametrize("bitmap_query", [-1, 2])
@pytest.mark.parametrize("tiles", [False, True])
@pytest.mark.parametrize("cols", [9000, 1 << 17, (1 << 17) + 1, (1 << 18) + 1, (1 << 19) + 5, (1 << 21) + 7])
def test_counts_both_ways(ob, cols, tiles, bitmap_query):
    rng = np.random.default_rng(cols)
    short = [np.sort(rng.choice(cols, int(n), replace=False)) for n in rng.integers(0, 6, 3200)]
    long = [np.sort(rng.choice(cols, int(n), replace=False)) for n in (400, 63, 64, 65, 1, 2, 3, 4000)]
    B = _csr(cols, short + long)
    k = len(short)
    every = list(range(k))
    some = list(range(k, B.rows))
    rows = [every, every[:1023] + some, every[:1024] + some, every[:1025] + some, [], every[:511] + some * 3, every[:512] + some * 3, every[:513], some * 9, every[5:900]]
    rows += [some * 40] * 60 if tiles else [every] * 20   # (which moves the mean over the line)
    A = _csr(B.rows, rows)
    products = int(O.row_products(A, B).sum())
    assert bool(rules.load().symbolic_in_tiles(B.col_idx.size, cols, products, A.col_idx.size)) == tiles
    got = ob.symbolic(ob.to_device(A), ob.to_device(B), opt=ob.default_options(bitmap_query=bitmap_query))[0].cpu().numpy()
    assert np.array_equal(got, O.count_rows(A, B))


def test_every_workgroup_has_one_of_a_few_rows(ob):
    """Four rows of many products beside smaller ones take about as long as one (median of many calls; 1.7 times where one workgroup
    had two of them and another none)."""
    import time

    import torch
    rng = np.random.default_rng(4)
    cols = 100000
    B = ob.to_device(_csr(cols, [np.sort(rng.choice(cols, 250, replace=False)) for _ in range(16000)]))
    small = [np.sort(rng.choice(16000, 40, replace=False)) for _ in range(4000)]
    median = []
    for rows in (1, 4):
        A = ob.to_device(_csr(16000, [np.arange(16000)] * rows + small))
        times = []
        for _ in range(30):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            st = ob.symbolic(A, B)[1]
            torch.cuda.synchronize()
            times.append(time.perf_counter() - t0)
        assert st["symbolic_rows_per_bin"][6] == rows
        median.append(sorted(times)[15])
    assert median[1] < 1.3 * median[0], median
