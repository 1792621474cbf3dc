"""Rows of the 4096-slot bin, which go with the heavy rows through the column-window kernel where rows of B have 32 entries on
average and there are at most 16 windows of 16384 columns, or 128 and 32 windows, and keep their hash tables elsewhere, against the
CPU oracle."""
import numpy as np
import pytest

import rules
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
@pytest.mark.parametrize("n, length", [(n, length) for n in (16384, 16 * 16384, 16 * 16384 + 1, 32 * 16384, 32 * 16384 + 1) for length in (31, 32)] +
                         [(n, length) for n in (16 * 16384 + 1, 32 * 16384, 32 * 16384 + 1) for length in (127, 128)])
def test_rows_on_both_sides_of_the_line(ob, n, length, dtype):
    rng = np.random.default_rng(n + length)

    def csr(rows, cols):
        ptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
        idx = np.concatenate(rows).astype(np.int32)
        return CSR(len(rows), cols, ptr, idx, rng.uniform(-1, 1, idx.size).astype(dtype))
    B = csr([np.sort(rng.choice(n, length, replace=False)) for _ in range(2000)], n)
    # (rows of 1400 to 2700 entries take 4096 slots; one row is beyond 8192; short ones and an empty one between them)
    sizes = [45 * 32 // length, 60 * 32 // length, 75 * 32 // length, 84 * 32 // length, 2, 0, 30 * 32 // length] * 30 + [700]
    A = csr([np.sort(rng.choice(2000, k, replace=False)) for k in sizes], 2000)
    ref = O.multiply_rows(A, B)
    dA, dB = ob.to_device(A), ob.to_device(B)
    for kw in (dict(workflow=ob.WF_SYMBOLIC), dict(workflow=ob.WF_HLL), dict(workflow=ob.WF_UPPER_BOUND), dict(force_hash_kernels=1)):
        C, st = ob.spgemm(dA, dB, **kw)
        check_result(C, ref, A, f"n={n} length={length} {kw}")
        if kw.get("workflow") == ob.WF_SYMBOLIC:
            assert st["rows_per_bin"][ob.bin_layout()[0].index(4096)] > 0
            assert bool(rules.load().middle_in_windows((n + 16383) >> 14, st["products"], A.col_idx.size)) == (length >= (32 if n <= 1 << 18 else 128) and n <= 1 << 19)


@pytest.mark.parametrize("length", [31, 33, 63, 65])
@pytest.mark.parametrize("n", [16384, 1 << 17, (1 << 17) + 1, 1 << 18, (1 << 18) + 1])
def test_counts_on_both_sides_of_the_line(ob, n, length):
    """Rows of 820 to 3276 products, 1025 to 4096 table slots, are counted by a bitmap where rows of B have 32 entries (64 beyond 2^17
    columns), up to 2^18 columns."""
    rng = np.random.default_rng(n + length)

    def csr(rows, cols):
        ptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
        idx = np.concatenate(rows).astype(np.int32)
        return CSR(len(rows), cols, ptr, idx, rng.uniform(-1, 1, idx.size))
    B = csr([np.sort(rng.choice(n, length, replace=False)) for _ in range(2000)] + [np.sort(rng.choice(n, k, replace=False)) for k in range(1, length)], n)

    def row(products):   # of exactly so many
        last = [2000 + products % length - 1] if products % length else []
        return np.sort(np.concatenate([rng.choice(2000, products // length, replace=False), last]).astype(np.int64))
    edges = [819, 820, 3276, 3277]
    A = csr([row(k) for k in edges + [4096, 4097, 50 * length, 3, 0, 600 * length, 1100 * length] for _ in range(30)], B.rows)
    ref = O.multiply_rows(A, B)
    dA, dB = ob.to_device(A), ob.to_device(B)
    for kw in (dict(), dict(bitmap_query=2), dict(assisted_symbolic=2)):
        counts, st = ob.symbolic(dA, dB, opt=ob.default_options(**kw))
        assert np.array_equal(counts.cpu().numpy(), np.diff(ref.row_ptr)), f"{kw}"
        assert (st["er"] >= 32) == (length >= 33) and (st["er"] >= 64) == (length >= 65)
        if not kw:   # (rows of 819, 820 and 3276, 3277 products lie on both sides of the bin's ends)
            products = O.row_products(A, B)
            slots = (lambda e: e + (e + 3) // 4)(np.minimum(products, n))
            in_bin = lambda lo, hi: int(((slots > lo) & (slots <= hi)).sum())
            assert st["symbolic_rows_per_bin"][2:4] == [in_bin(256, 1024), in_bin(1024, 4096)] and sum(st["symbolic_rows_per_bin"][4:7]) == in_bin(4096, 1 << 40)
            assert [in_bin(s - 1, s) for s in (1024, 1025, 4095, 4097)] == [30] * 4
    C, _ = ob.spgemm(dA, dB, workflow=ob.WF_SYMBOLIC)
    check_result(C, ref, A, f"n={n} length={length}")


@pytest.mark.parametrize("heavy", [0, 1, 400])
def test_rows_of_both_kinds(ob, heavy):
    """Rows of the 4096-slot bin beside none, one or many rows whose pieces would not fill tiles: these few follow the others, and
    where they are most, nobody goes in tiles."""
    n = 4 * 16384
    rng = np.random.default_rng(heavy)

    def csr(rows, cols):
        ptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
        idx = np.concatenate(rows).astype(np.int32)
        return CSR(len(rows), cols, ptr, idx, rng.uniform(-1, 1, idx.size))
    B = csr([np.sort(rng.choice(n, 64, replace=False)) for _ in range(2000)] + [np.sort(rng.choice(2500, 40, replace=False)) for _ in range(300)], n)
    # (the last row has more than 8192 products, on 2500 columns, so that the window table is built)
    A = csr([np.sort(rng.choice(2000, 46, replace=False)) for _ in range(300)] + [np.sort(rng.choice(2000, 700, replace=False)) for _ in range(heavy)] + [np.arange(2000, 2300)], 2300)
    C, st = ob.spgemm(ob.to_device(A), ob.to_device(B), workflow=ob.WF_SYMBOLIC)
    assert st["er"] >= 32 and st["rows_per_bin"][7] >= 300 and sum(st["rows_per_bin"][8:11]) == heavy
    assert rules.heavy_in_tiles(st, B) == (heavy < 400)
    check_result(C, O.multiply_rows(A, B), A, f"{heavy} heavy rows")


def test_stage_of_the_order(ob):
    """Rows of the 4096-slot bin alone: putting them in order for the column-window kernel is part of the numeric stage.  (Three
    kernels, a fill and a copy, against the two kernels of the binning stage; the least of many calls.)"""
    n = 16384
    rng = np.random.default_rng(7)

    def csr(rows, cols):
        ptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
        idx = np.concatenate(rows).astype(np.int32)
        return CSR(len(rows), cols, ptr, idx, rng.uniform(-1, 1, idx.size))
    B = csr([np.sort(rng.choice(n, 40, replace=False)) for _ in range(3000)] + [np.sort(rng.choice(2500, 40, replace=False)) for _ in range(600)], n)
    # (the last row has more than 8192 products, on 2500 columns, so that the window table is built)
    A = csr([np.sort(rng.choice(3000, 60, replace=False)) for _ in range(5000)] + [np.arange(3000, 3600)], 3600)
    dA, dB = ob.to_device(A), ob.to_device(B)
    least = {}
    for hashed in (0, 1):
        calls = [ob.spgemm(dA, dB, workflow=ob.WF_SYMBOLIC, force_hash_kernels=hashed)[1] for _ in range(30)]
        assert calls[0]["rows_per_bin"][ob.bin_layout()[0].index(4096)] > 4000 and sum(calls[0]["rows_per_bin"][8:11]) == 0
        least[hashed] = min(st["stage_ms"]["binning"] for st in calls)
    assert least[0] < least[1] + 0.008, least   # ms; the order takes about 20 us
