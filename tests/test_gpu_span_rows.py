"""Rows accumulated and counted over their own column range (k_numeric_dspan, k_symbolic_span) against the CPU oracle, at
the ranges where a row passes from one size of accumulator to the next, with B's rows in column order and not."""
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


def _case(seed, n, dtype, shuffle_b):
    """Groups of 40 rows of B whose entries lie in one stretch of columns, both ends of the stretch among them; every row
    of A takes rows of one group."""
    rng = np.random.default_rng(seed)
    spans = [600, 1023, 1024, 1025, 2047, 2048, 2049, 4095, 4096, 4097, 6000]
    b_rows, a_rows = [], []
    for g, span in enumerate(spans):
        low = n - span if g % 2 else int(rng.integers(0, n - span + 1))   # (the last columns among them)
        for _ in range(40):
            inner = rng.choice(span - 2, span // 12, replace=False) + 1
            cols = low + np.sort(np.concatenate([[0, span - 1], inner]))
            b_rows.append(rng.permutation(cols) if shuffle_b else cols)
        for _ in range(30):
            a_rows.append(g * 40 + np.sort(rng.choice(40, int(rng.integers(8, 41)), replace=False)))
    a_rows = [a_rows[i] for i in rng.permutation(len(a_rows))]

    def csr(rows, cols):
        ptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
        idx = np.concatenate(rows).astype(np.int32)
        return CSR(len(rows), cols, ptr, idx, rng.uniform(-1, 1, idx.size).astype(dtype))
    return csr(a_rows, len(b_rows)), csr(b_rows, n)


@pytest.mark.parametrize("shuffle_b", [False, True])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("n", [6000, 300000])
def test_rows_over_their_own_column_range(ob, n, dtype, shuffle_b):
    A, B = _case(n + shuffle_b, n, dtype, shuffle_b)
    ref = O.multiply_rows(A, B)
    dA, dB = ob.to_device(A), ob.to_device(B)
    nb, ns = (len(x) for x in ob.bin_layout())
    for kw in (dict(workflow=ob.WF_SYMBOLIC), dict(workflow=ob.WF_SYMBOLIC, bitmap_query=1, assisted_symbolic=2),
               dict(workflow=ob.WF_UPPER_BOUND), dict(workflow=ob.WF_HLL)):
        Cd, st = ob.spgemm(dA, dB, dense_range=2, **kw)
        check_result(Cd, ref, A, f"n={n} {kw}")
        if not shuffle_b:
            assert st["rows_per_bin"][nb] > 0 and st["overflow_rows"] == 0
            if kw["workflow"] == ob.WF_SYMBOLIC:
                assert st["symbolic_rows_per_bin"][ns] == 9 * 30


@pytest.mark.parametrize("few", [199, 201])
@pytest.mark.parametrize("span, line", [(500, 1280), (513, 768), (700, 768)])
def test_rows_on_both_sides_of_the_bitmaps_line(ob, span, line, few):
    """Rows of one product less than, as many as and one more than a range of so many columns needs to be cheaper by a bitmap,
    in a matrix of as many columns: 1024 keys hold any row, so the products alone decide.  The few products are counted
    with key tables where those rows are four fifths of all, by bitmaps otherwise."""
    rng = np.random.default_rng(span)
    b_rows = [np.array([7])] * 20
    b_rows += [np.concatenate([[0], np.sort(rng.choice(span - 2, 62, replace=False)) + 1, [span - 1]]) for _ in range(20)]
    totals = [line + 1] * 50 + [line - 1, line] * (few // 2) + [line] * (few % 2)
    a_rows = [np.concatenate([rng.integers(0, 20, t % 64), rng.integers(20, 40, t // 64)]) for t in rng.permutation(totals)]

    def csr(rows, cols):
        ptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
        idx = np.concatenate(rows).astype(np.int32)
        return CSR(len(rows), cols, ptr, idx, rng.uniform(-1, 1, idx.size))
    A, B = csr(a_rows, len(b_rows)), csr(b_rows, span)
    ref = O.multiply_rows(A, B)
    Cd, st = ob.spgemm(ob.to_device(A), ob.to_device(B), workflow=ob.WF_SYMBOLIC, dense_range=2)
    check_result(Cd, ref, A, f"span {span}")
    slots, keys = ob.bin_layout()
    by_keys = few if few >= 4 * 50 else 0
    assert st["symbolic_rows_per_bin"][keys.index(1024)] == by_keys
    assert st["symbolic_rows_per_bin"][len(keys)] == 50 + few - by_keys
