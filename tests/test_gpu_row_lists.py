"""Lists of so many rows that the kernels which give a row a fixed number of threads need more than 2^32 of them: a launch
holds fewer.  Rows repeat every 64, so the CPU oracle multiplies the first 64 and the rest is compared on the GPU."""
import numpy as np
import pytest

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


# sorted rows: 64 lanes each from 257 products on; rows counted over their column range: 256 threads each
@pytest.mark.parametrize("kernel, rows, length, n", [("sort", (1 << 26) + 1024, 33, 40), ("span", (1 << 24) + 1024, 26, 300)])
def test_more_rows_than_one_launch_takes(ob, kernel, rows, length, n):
    import torch
    rng = np.random.default_rng(length)
    entries = 8
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
    Cd, st = ob.spgemm(dA, ob.to_device(B), workflow=ob.WF_SYMBOLIC, dense_range=2 if kernel == "span" else 0)
    if kernel == "span":
        assert st["symbolic_rows_per_bin"][len(ob.bin_layout()[1])] == rows
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
