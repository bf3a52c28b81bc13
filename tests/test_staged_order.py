"""Staged snapshots and restores without a GPU (the runtime of test_table_cache.py, which sees two accesses to the same memory
that neither a stream's order nor an event keeps apart): whose memory kernels touch, and the ring of slots from call to call."""
import ctypes

import pytest

import test_table_cache

SIZES = [3001] * 200
T, L = len(SIZES), sum(SIZES)
HOST, RING = 1 << 40, 1 << 41


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    lib = test_table_cache.compile_with(test_table_cache.SOURCE, tmp_path_factory.mktemp("staged_order"))
    p, u64 = ctypes.c_void_p, ctypes.c_uint64
    lib.reft_snapshot_pack.argtypes = [p, p, p, u64, p, u64, p, p]
    lib.reft_restore.argtypes = [p, p, u64, p, u64, p, p, p]
    lib.sim_map.argtypes = [u64, u64]
    lib.sim_fail.argtypes = [ctypes.c_int64]
    lib.sim_thread.argtypes = [u64]
    lib.reft_plan_staging_slot_bytes.argtypes = [p]
    lib.reft_plan_staging_slot_bytes.restype = u64
    lib.sim_clashes.restype = lib.sim_uploads.restype = lib.sim_copies.restype = u64
    return lib


class Calls:
    """A plan and calls on it, each from or to host memory and tensors of its own."""

    def __init__(self, lib, bucket=0):
        self.lib, self.plan, self.n = lib, ctypes.c_void_p(), 0
        lib.sim_end()
        assert lib.reft_plan_create((ctypes.c_uint64 * T)(*SIZES), T, None, 0, bucket, ctypes.byref(self.plan)) == 0
        self.slot = lib.reft_plan_staging_slot_bytes(self.plan)

    def call(self, load, first, second, ring=RING, slots=2, host=None):
        self.n += 1
        host = host or HOST + (self.n << 30)
        ptrs = (ctypes.c_void_p * T)(*range((1 << 44) + (self.n << 30), (1 << 44) + (self.n << 30) + (T << 14), 1 << 14))
        self.lib.sim_call(first)
        if load:
            return self.lib.reft_restore(self.plan, host, L, ring, slots * self.slot, ptrs, first, second)
        return self.lib.reft_snapshot_pack(self.plan, ptrs, ring, slots * self.slot, host, L, first, second)

    def end(self):
        self.lib.reft_plan_destroy(self.plan)
        self.lib.sim_end()


@pytest.mark.parametrize("load", [False, True])
@pytest.mark.parametrize("pieces,copied", [([(0, L)], False), ([(-4096, L + 8192)], False), ([(0, L - 1)], True),
                                           ([(0, 4096), (L - 4096, 8192)], True), ([(0, 4096), (4096, L - 4096)], True), ([], True)])
def test_kernels_see_host_memory_of_one_piece(lib, pieces, copied, load):
    """A kernel takes the bytes across the link only where one allocation holds all of them."""
    c = Calls(lib)
    for at, n in pieces:
        lib.sim_map(HOST + at, n)
    before = lib.sim_copies()
    assert c.call(load, 1, 1, host=HOST) == 0
    assert (lib.sim_copies() > before + 1) == copied      # (the pointers' upload is a copy in any case)
    c.end()
