"""Rows that were to be written straight to C (placed.hip, dense ranges of numeric.hip) where that cannot be finished: a wait for a
place that runs out, by a unit or by the workgroup that gives the places, and memory that is refused.  The general way then gives
the same C and the same statistics, against the CPU oracle."""
import ctypes

import numpy as np
import pytest

from oracle import spgemm as O
from test_gpu_placed_rows import _b, _check, _csr, _row, ob  # noqa: F401
from test_gpu_spgemm import check_result

pytestmark = pytest.mark.gpu


def _ranges(rng, dtype):
    """Rows whose columns lie in windows of 900, more than 2048 products in some: accumulated over their ranges."""
    lists = [900 * w + np.sort(rng.choice(900, 40, replace=False)) for w in range(5) for _ in range(70)]
    B = _csr(len(lists), 4500, lists, rng, dtype)
    return _csr(700, B.rows, [70 * int(rng.integers(0, 5)) + rng.choice(70, int(rng.integers(52, 71)), replace=False) for _ in range(700)],
                rng, dtype), B


def _inputs(kind, dtype):
    rng = np.random.default_rng(3)
    if kind == "ranges":
        return _ranges(rng, dtype)
    B = _b(rng, 5000, dtype, "sorted")
    return _csr(1203, B.rows, [_row(rng, int(p)) for p in rng.integers(0, kind + 1, 1203)], rng, dtype), B


@pytest.fixture
def waits(ob):  # noqa: F811
    """Sets how long waits take at most, and puts the defaults back."""
    fn = ob.load().ocean_test_wait_polls
    fn.argtypes, fn.restype = [ctypes.c_int, ctypes.c_int], None
    yield fn
    fn(1 << 20, 1 << 21)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("who", ["unit", "placer"])
@pytest.mark.parametrize("kind", [32, 120, 250, 700, 2000, "ranges"])
def test_wait_that_runs_out(ob, waits, kind, who, dtype):  # noqa: F811
    A, B = _inputs(kind, dtype)
    for wf in (ob.WF_AUTO, ob.WF_UPPER_BOUND):
        if kind == "ranges" and wf == ob.WF_UPPER_BOUND:
            continue                                    # (no sample, so no ranges)
        options = dict(workflow=wf, tuned_min_products=0.0)
        waits(1 << 20, 1 << 21)
        _check(ob, A, B, f"{kind}", **options)
        waits(0 if who == "placer" else 1 << 20, 0 if who == "unit" else 1 << 21)
        _check(ob, A, B, f"{kind}, {who} gave up", placed=False, **options)


class _Refusing:
    """Allocators that count their requests and refuse those whose numbers are in `refuse`."""

    def __init__(self, ob, monkeypatch):  # noqa: F811
        outer = self
        self.sizes, self.refuse = [], set()

        class Allocator(ob.TorchAllocator):
            def __init__(self, device):
                super().__init__(device)
                plain = self._alloc_cb

                def alloc(ctx, nbytes, out):
                    outer.sizes.append(int(nbytes))
                    if len(outer.sizes) - 1 in outer.refuse:
                        return 1
                    return plain(ctx, nbytes, ctypes.cast(out, ctypes.POINTER(ctypes.c_void_p)))
                self._alloc_or_not = ob.ALLOC_FN(alloc)
                self.struct = ob.ocean_allocator(None, self._alloc_or_not, self._release_cb)

        monkeypatch.setattr(ob, "TorchAllocator", Allocator)

    def start(self, *refuse):
        self.sizes, self.refuse = [], set(refuse)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("kind", [120, 700, "ranges"])
def test_memory_that_is_refused(ob, monkeypatch, kind, dtype):  # noqa: F811
    A, B = _inputs(kind, dtype)
    memory = _Refusing(ob, monkeypatch)
    vbytes = np.dtype(dtype).itemsize
    memory.start()
    C, st = _check(ob, A, B, f"{kind}", tuned_min_products=0.0)
    slots = C.col_idx.untyped_storage().nbytes() // 4
    col = memory.sizes.index(4 * slots)
    assert memory.sizes[col + 1] == vbytes * slots
    first = col - 1 if kind == "ranges" else col         # the words for the places of the ranges come before
    for k in range(first, col + 2):
        memory.start(k)
        _check(ob, A, B, f"{kind}, request {k - col} after the columns", placed=False, tuned_min_products=0.0)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_no_memory_to_trim_c(ob, monkeypatch, dtype):  # noqa: F811
    """Every product was reserved and C has an eighth of that: it stays where it is if there is no room for a copy."""
    rng = np.random.default_rng(8)
    B = _csr(500, 12, [np.sort(rng.choice(12, 8, replace=False)) for _ in range(500)], rng, dtype)
    lists = [rng.choice(500, 7, replace=False) for _ in range(4000)]
    lists[5] = rng.choice(500, 64, replace=False)        # too large a row for what few rows say to count
    A = _csr(4000, 500, lists, rng, dtype)
    memory = _Refusing(ob, monkeypatch)
    memory.start()
    C, st = _check(ob, A, B, "trimmed", workflow=ob.WF_UPPER_BOUND)
    trimmed = memory.sizes.index(4 * st["nnz_c"])
    assert C.col_idx.untyped_storage().nbytes() == 4 * st["nnz_c"] and st["temp_slots"] == st["products"]
    for k in (trimmed, trimmed + 1):
        memory.start(k)
        C, st = ob.spgemm(ob.to_device(A), ob.to_device(B), workflow=ob.WF_UPPER_BOUND)
        check_result(C, O.multiply_rows(A, B), A, f"request {k} refused")
        assert C.col_idx.untyped_storage().nbytes() == 4 * st["products"] and st["stage_ms"]["binning"] == 0.0
