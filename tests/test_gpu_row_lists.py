"""Lists of so many rows that the kernels which give a row a fixed number of threads need more than 2^32 of them: a launch
holds fewer.  Rows repeat every 64, so the CPU oracle multiplies the first 64 and the rest is compared on the GPU."""
import numpy as np
import pytest

from oracle import hll as ohll
from oracle import spgemm as O
from paper_2604_19004_amd.workloads import CSR

pytestmark = pytest.mark.gpu

PERIOD = 64


@pytest.fixture(scope="module")
def ob():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2604_19004_amd import binding
    binding.load()
    return binding


TWO_PASSES = dict(workflow=3, dense_range=0)   # WF_SYMBOLIC
CASES = {                                      # rows, entries of A, entries of B, columns, options
    "sort": ((1 << 26) + 1024, 8, 33, 40, TWO_PASSES),                                     # 64 threads a row from 257 products on
    "symbolic span": ((1 << 24) + 1024, 8, 97, 600, dict(TWO_PASSES, dense_range=2)),      # 256 threads a row
    "256-slot tables": ((1 << 26) + 1024, 8, 33, 60, dict(TWO_PASSES, force_hash_kernels=1)),   # 64, both passes
    "1024-slot tables": ((1 << 24) + 1024, 2, 240, 1000, dict(TWO_PASSES, force_hash_kernels=1)),   # 256
    "dense range": ((1 << 24) + 1024, 2, 130, 300, dict(TWO_PASSES, dense_range=2)),       # 256
    "compaction": ((1 << 26) + 1024, 8, 33, 40, dict(workflow=1)),                         # 64, output of the upper bound
}


@pytest.mark.parametrize("kernel", CASES)
def test_more_rows_than_one_launch_takes(ob, kernel):
    import torch
    rows, entries, length, n, options = CASES[kernel]
    rng = np.random.default_rng(length)
    b_col = np.concatenate([np.sort(rng.choice(n, length, replace=False)) for _ in range(PERIOD)]).astype(np.int32)
    B = CSR(PERIOD, n, np.arange(PERIOD + 1, dtype=np.int64) * length, b_col, rng.uniform(-1, 1, b_col.size).astype(np.float32))
    head_col = ((np.arange(PERIOD)[:, None] + np.arange(entries)[None, :] % 2) % PERIOD).astype(np.int32).reshape(-1)
    head = CSR(PERIOD, PERIOD, np.arange(PERIOD + 1, dtype=np.int64) * entries, head_col,
               rng.uniform(-1, 1, head_col.size).astype(np.float32))
    ref = O.multiply_rows(head, B)
    per = ref.col_idx.size
    dA = ob.DeviceCSR(rows, PERIOD, torch.arange(rows + 1, dtype=torch.int64, device="cuda:0") * entries,
                      torch.from_numpy(head_col).cuda().repeat(rows // PERIOD), torch.from_numpy(head.val).cuda().repeat(rows // PERIOD))
    print(f"{kernel}: {rows} rows of {entries * length} products", flush=True)
    Cd, st = ob.spgemm(dA, ob.to_device(B), **options)
    slots, keys = ob.bin_layout()
    if kernel == "symbolic span":
        assert st["symbolic_rows_per_bin"][len(keys)] == rows
    elif kernel == "dense range":
        assert st["rows_per_bin"][len(slots)] == rows
    elif kernel.endswith("tables"):
        assert st["rows_per_bin"][slots.index(int(kernel.split("-")[0]))] > rows // 2
    assert st["nnz_c"] == per * (rows // PERIOD) and int(Cd.row_ptr[-1]) == st["nnz_c"]
    starts = Cd.row_ptr[:-1].view(-1, PERIOD)
    first = torch.arange(rows // PERIOD, device="cuda:0")[:, None] * per + torch.from_numpy(ref.row_ptr[:-1]).cuda()
    assert torch.equal(starts, first)
    col, val = Cd.col_idx[:st["nnz_c"]].view(-1, per), Cd.val[:st["nnz_c"]].view(-1, per)
    want_col, want, bound = (torch.from_numpy(x).cuda() for x in (ref.col_idx, ref.val, 1e-5 * ref.absval))
    for at in range(0, col.shape[0], 1 << 16):
        assert bool((col[at:at + (1 << 16)] == want_col).all()), f"columns from period {at} on"
        assert bool(((val[at:at + (1 << 16)].double() - want).abs() <= bound).all()), f"values from period {at} on"
    del dA, Cd, col, val, starts, first
    torch.cuda.empty_cache()


def test_more_estimates_than_one_launch_takes(ob):
    """Sketches of 64 registers merged along listed rows of 8 entries: 64 threads a row."""
    import torch
    rng = np.random.default_rng(3)
    rows, entries, n, m = (1 << 26) + 1024, 8, 5000, 64
    lengths = rng.integers(0, 60, PERIOD)
    b_ptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    B = CSR(PERIOD, n, b_ptr, np.concatenate([np.sort(rng.choice(n, k, replace=False)) for k in lengths]).astype(np.int32),
            rng.uniform(-1, 1, int(b_ptr[-1])).astype(np.float32))
    head_col = rng.integers(0, PERIOD, PERIOD * entries).astype(np.int32)
    head = CSR(PERIOD, PERIOD, np.arange(PERIOD + 1, dtype=np.int64) * entries, head_col, np.ones(head_col.size, np.float32))
    sketches = ohll.sketch_rows(B, m)
    want = torch.from_numpy(ohll.estimate(ohll.merge_rows(head, sketches))).cuda()
    dA = ob.DeviceCSR(rows, PERIOD, torch.arange(rows + 1, dtype=torch.int64, device="cuda:0") * entries,
                      torch.from_numpy(head_col).cuda().repeat(rows // PERIOD), torch.ones(rows * entries, device="cuda:0"))
    dS = torch.from_numpy(sketches).cuda()
    print(f"{rows} estimates", flush=True)
    est, _ = ob.hll_merge_estimate(dA, dS, m, rows=torch.arange(rows, dtype=torch.int64, device="cuda:0"))
    assert bool(((est.view(-1, PERIOD) - want).abs() <= 1e-12 * want).all())
    del dA, est
    torch.cuda.empty_cache()


def test_larger_sample_than_one_launch_takes(ob):
    """Every row sampled, sketches of 128 registers merged along rows of 5 entries in a matrix with one far larger row: 64
    threads a row."""
    import torch
    rng = np.random.default_rng(5)
    rows, entries, n, m = (1 << 26) + 1024, 5, 5000, 128
    lengths = np.concatenate([rng.integers(0, 4, PERIOD - 1), [300]])
    b_ptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    B = CSR(PERIOD, n, b_ptr, np.concatenate([np.sort(rng.choice(n, k, replace=False)) for k in lengths]).astype(np.int32),
            rng.uniform(-1, 1, int(b_ptr[-1])).astype(np.float32))
    head_col = rng.integers(0, PERIOD - 1, (PERIOD + 1, entries)).astype(np.int32)
    head_col[PERIOD] = head_col[PERIOD - 1]              # the matrix's last row: that of the period, and the long row of B
    head_col[PERIOD, -1] = PERIOD - 1
    head = CSR(PERIOD + 1, PERIOD, np.arange(PERIOD + 2, dtype=np.int64) * entries, head_col.reshape(-1),
               np.ones(head_col.size, np.float32))
    prod = O.row_products(head, B)
    longest = lengths[head_col].max(axis=1)
    est = np.clip(ohll.estimate(ohll.merge_rows(head, ohll.sketch_rows(B, m))), longest, np.minimum(prod, n))
    times = np.concatenate([np.full(PERIOD, rows // PERIOD), [1]])
    times[PERIOD - 1] -= 1
    assert prod[PERIOD] > 16 * (prod * times).sum() / rows
    col = torch.from_numpy(head_col[:PERIOD].reshape(-1)).cuda().repeat(rows // PERIOD)
    col[-entries:] = torch.from_numpy(head_col[PERIOD]).cuda()
    dA = ob.DeviceCSR(rows, PERIOD, torch.arange(rows + 1, dtype=torch.int64, device="cuda:0") * entries, col,
                      torch.ones(rows * entries, device="cuda:0"))
    print(f"{rows} sampled rows", flush=True)
    nnz, st = ob.symbolic(dA, ob.to_device(B), ob.default_options(assisted_symbolic=2, hll_registers=m, sample_ratio=1.0,
                                                                   sample_max=2 ** 31 - 1))
    some = est > 0
    ratio = np.divide(prod, est, where=some, out=np.zeros(est.size))
    mean = (ratio * times).sum() / times[some].sum()
    # (sums of at most 2^26 terms of equal sign in 64 bits)
    assert st["sampled_rows"] == rows
    assert abs(st["sampled_cr"] - (prod * times).sum() / (est * times).sum()) < 1e-8
    assert abs(st["cr_mean"] - mean) < 1e-8
    assert abs(st["cr_std"] ** 2 - ((ratio - mean) ** 2 * times)[some].sum() / times[some].sum()) < 1e-7
    ref = O.multiply_rows(head, B)
    want = torch.from_numpy(np.diff(ref.row_ptr).astype(np.int32)).cuda()
    assert bool((nnz[:rows - PERIOD].view(-1, PERIOD) == want[:PERIOD]).all()) and int(nnz[-1]) == int(want[PERIOD])
    del dA, nnz, col
    torch.cuda.empty_cache()
