"""Rows that go through column windows, on both sides of the line between products in tiles and products one by one (heavy_in_tiles
in csrc/rules.hpp), against the CPU oracle: the same rows both ways, by what other rows move the mean to.  Pieces of one entry among
B's first, windows of as many products as a pass stages and one more, stretches, more entries of A than a chunk of either
kernel holds, a B of fewer entries than a tile's lane reads, and products that are -0 or no numbers."""
import numpy as np
import pytest

import rules
from oracle import spgemm as O
from paper_2604_19004_amd.workloads import CSR

pytestmark = pytest.mark.gpu

WIN = 16384


@pytest.fixture(scope="module")
def ob():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2604_19004_amd import binding
    binding.load()
    return binding


def _csr(cols, lists, values):
    ptr = np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int64)
    idx = np.concatenate([np.asarray(x, dtype=np.int64) for x in lists]).astype(np.int32)
    return CSR(len(lists), cols, ptr, idx, values(idx.size))


def _check(ob, A, B, tiles, exact=False, **options):
    with np.errstate(invalid="ignore"):
        ref = O.multiply_rows(A, B)
    C, st = ob.spgemm(ob.to_device(A), ob.to_device(B), **options)
    assert sum(st["rows_per_bin"][8:11]) > 0, "no row reaches the kernels under test"
    if options.get("workflow") == ob.WF_SYMBOLIC and tiles is not None:
        assert rules.heavy_in_tiles(st, B) == tiles
    assert np.array_equal(C.row_ptr.cpu().numpy(), ref.row_ptr) and np.array_equal(C.col_idx.cpu().numpy(), ref.col_idx)
    val = C.val.cpu().numpy().astype(np.float64)
    if exact:
        assert np.array_equal(val, ref.val.astype(np.float64), equal_nan=True)
    else:   # sums of up to a few thousand terms in any order: (terms - 1) * 2^-53 of sum |a b|, and one rounding to the result's type
        assert np.all(np.abs(val - ref.val) <= (1e-12 if C.val.element_size() == 8 else 2e-7) * ref.absval)
    return val


def _steered(rng, cols, lists, rows, tiles, values):
    """A and B of these rows, with rows of long pieces beside them, or of pieces of a few entries, that move the mean over the line."""
    k, many = len(lists), len(rows)
    if tiles:
        lists = lists + [np.sort(rng.choice(cols, 12000, replace=False)) for _ in range(3)]
        extra = [[k, k + 1, k + 2]] * (3 + sum(len(r) for r in rows) // 64)
    else:
        lists = lists + [np.sort(rng.choice(cols, 4, replace=False)) for _ in range(3000)]
        extra = [list(range(k, k + 3000))] * (2 + sum(len(r) for r in rows) // 512)
    B = _csr(cols, lists, values)
    return _csr(B.rows, rows + extra, values), B


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("tiles", [False, True])
@pytest.mark.parametrize("entries", [3, 511, 512, 513, 1024, 1025])
@pytest.mark.parametrize("products", [8191, 8192, 8193, 25000])
def test_windows_and_chunks(ob, products, entries, tiles, dtype):
    rng = np.random.default_rng(products + entries)
    cols = 20 * WIN + 5
    lists = [np.array([0]), np.array([1, 2])]   # (pieces among B's first entries)
    for i in range(entries - 2):
        n = products // entries + (i < products % entries)
        at = 3 * WIN + rng.choice(WIN, min(n, WIN), replace=False)
        around = np.concatenate([rng.choice(3 * WIN, 9000 // entries + 1, replace=False), 4 * WIN + rng.choice(16 * WIN, 30000 // entries + 1, replace=False)])
        lists.append(np.unique(np.concatenate([at, around])))
    rows = [list(range(entries)), [], list(range(entries))]
    A, B = _steered(rng, cols, lists, rows, tiles, lambda n: rng.uniform(-1, 1, n).astype(dtype))
    for options in (dict(workflow=ob.WF_SYMBOLIC), dict(workflow=ob.WF_SYMBOLIC, bitmap_query=1), dict(workflow=ob.WF_HLL)):
        _check(ob, A, B, tiles, **options)


@pytest.mark.parametrize("tiles", [False, True])
def test_minus_zero_infinities_and_nan(ob, tiles):
    """Entries whose products are -0, infinite or no numbers, in dense windows and in ranked or sparse passes: all are stored."""
    rng = np.random.default_rng(17)
    cols = 18 * WIN
    lists = [np.sort(rng.choice(2 * WIN, 9000, replace=False)) for _ in range(4)] + [np.sort(rng.choice(cols, 6000, replace=False)) for _ in range(3)]
    A, B = _steered(rng, cols, lists, [list(range(7)), list(range(3, 7))], tiles, lambda n: rng.choice(np.array([-0.0, 0.0, 1.0, -2.0]), n))
    B.val[rng.choice(B.val.size, 300, replace=False)] = rng.choice([np.inf, -np.inf, np.nan], 300)
    for options in (dict(workflow=ob.WF_SYMBOLIC), dict(workflow=ob.WF_HLL)):
        val = _check(ob, A, B, tiles, exact=True, **options)   # (sums of few small numbers: exact)
        assert np.isnan(val).any() and np.isinf(val).any() and not np.any(np.signbit(val) & (val == 0))


def test_a_matrix_of_fewer_entries_than_a_lane_reads(ob):
    """Rows of more than 8192 products of a B of seven entries: nothing for tiles, and few columns."""
    rng = np.random.default_rng(5)
    B = _csr(70000, [[5], [5, 69999], [], [0, 1, 2, 3]], lambda n: rng.uniform(-1, 1, n))
    A = _csr(4, [[0, 1, 3] * 5000, [3] * 9000, [0] * 5, [2]], lambda n: rng.uniform(-1, 1, n))
    ref = O.multiply_rows(A, B)
    for workflow in (ob.WF_SYMBOLIC, ob.WF_HLL, ob.WF_UPPER_BOUND):
        C, _ = ob.spgemm(ob.to_device(A), ob.to_device(B), workflow=workflow)
        assert np.array_equal(C.row_ptr.cpu().numpy(), ref.row_ptr) and np.array_equal(C.col_idx.cpu().numpy(), ref.col_idx)
        assert np.all(np.abs(C.val.cpu().numpy() - ref.val) <= 1e-11 * ref.absval)   # (up to 15 000 terms)


def test_every_workgroup_has_one_of_as_many_rows(ob):
    """Equal rows, nearly one for every compute unit, take about as long as half as many (the least of many calls; 1.25 times with a
    row each, 1.7 where some workgroups have two and others none)."""
    import torch
    rng = np.random.default_rng(1)
    units = torch.cuda.get_device_properties(0).multi_processor_count
    B = _csr(2 * WIN, [np.sort(rng.choice(2 * WIN, 256, replace=False)) for _ in range(1500)], lambda n: rng.uniform(-1, 1, n))
    row = np.sort(rng.choice(1500, 400, replace=False))
    least = []
    for rows in (units // 2, units - 6):
        dA, dB = ob.to_device(_csr(1500, [row] * rows, lambda n: rng.uniform(-1, 1, n))), ob.to_device(B)
        calls = [ob.spgemm(dA, dB, workflow=ob.WF_SYMBOLIC)[1] for _ in range(30)]
        assert sum(calls[0]["rows_per_bin"][8:11]) == rows and rules.heavy_in_tiles(calls[0], B)
        least.append(min(st["stage_ms"]["numeric"] for st in calls))
    assert least[1] < 1.45 * least[0], least
