"""TorchAllocator's struct, as a C caller holds it: it works as long as it, or a pointer to it, is there, and not a call longer."""
import ctypes
import gc

import pytest

from paper_2604_19004_amd import binding


@pytest.fixture(autouse=True)
def on_the_cpu(monkeypatch):
    monkeypatch.setattr(binding, "_gpu_seen", True)   # (CPU memory does: nothing is launched)


def _take(struct, nbytes=64):
    out = (ctypes.c_void_p * 1)()
    rc = struct.alloc(struct.ctx, nbytes, out)
    return rc, out[0]


def test_the_struct_outlives_its_allocator():
    struct = binding.TorchAllocator("cpu").struct
    gc.collect()
    rc, ptr = _take(struct)
    assert rc == 0 and ptr
    struct.release(struct.ctx, ptr)


def test_a_pointer_to_the_struct_outlives_its_allocator():
    o = binding.ocean_options()
    o.allocator = ctypes.pointer(binding.TorchAllocator("cpu").struct)
    gc.collect()
    rc, ptr = _take(o.allocator.contents)
    assert rc == 0 and ptr
    o.allocator.contents.release(o.allocator.contents.ctx, ptr)


def test_blocks_belong_to_their_allocator_and_leave_with_it():
    gc.disable()   # (no cycle: what a call leaves goes at once)
    try:
        known = len(binding._allocators)
        a, b = binding.TorchAllocator("cpu"), binding.TorchAllocator("cpu")
        _, p = _take(a.struct)
        _, q = _take(b.struct)
        assert set(a.blocks) == {p} and set(b.blocks) == {q}
        b.struct.release(b.struct.ctx, q)
        assert a.take(p).numel() == 64 and not a.blocks and not b.blocks
        del a, b
        assert len(binding._allocators) == known
    finally:
        gc.enable()
