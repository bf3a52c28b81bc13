"""Staged snapshots and restores without a GPU (the runtime of test_table_cache.py, which sees two accesses to the same memory
that neither a stream's order nor an event keeps apart): whose memory kernels touch, and the ring of slots from call to call."""
import ctypes
import random

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
    lib.reft_snapshot_wait.argtypes = lib.reft_restore_wait.argtypes = [p]
    lib.reft_plan_staging_slot_bytes.argtypes = [p]
    lib.reft_plan_staging_slot_bytes.restype = u64
    lib.sim_clashes.restype = lib.sim_unfinished.restype = lib.sim_uploads.restype = lib.sim_copies.restype = u64
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


PER_THREAD = 2               # hipStreamPerThread: one handle, a stream of its own in every thread


@pytest.mark.parametrize("load", [False, True])
@pytest.mark.parametrize("second", [(PER_THREAD, PER_THREAD), (PER_THREAD, 5), (5, PER_THREAD), (5, 5)])
@pytest.mark.parametrize("first", [(PER_THREAD, PER_THREAD), (PER_THREAD, 4), (4, PER_THREAD), (4, 4)])
def test_threads_whose_streams_share_a_handle(lib, first, second, load):
    """One thread's calls after another's, on the same ring: one after the other, whatever their streams."""
    c = Calls(lib, 100_000)
    for i in range(4):
        lib.sim_thread(i)
        assert c.call(load, *(first if i % 2 == 0 else second)) == 0
        assert lib.sim_clashes() == 0
        assert lib.sim_races() == 0
    lib.sim_call(PER_THREAD)
    assert (lib.reft_restore_wait if load else lib.reft_snapshot_wait)(c.plan) == 0
    # tables, slots and the host's memory are free once the host knows that the last call has ended
    assert lib.sim_unfinished() == 0
    c.end()


def test_pointer_tables_of_threads_whose_streams_share_a_handle(lib):
    """A table that one thread's call has uploaded, used by another's, and overwritten once neither reads it any more."""
    p = ctypes.c_void_p
    lib.reft_pack_device.argtypes = [p, p, p, ctypes.c_uint64, p]
    c = Calls(lib)
    for i in range(400):
        lib.sim_thread(i % 3)
        lib.sim_call(PER_THREAD)
        ptrs = (ctypes.c_void_p * T)(*range((1 << 44) + (i // 5 << 30), (1 << 44) + (i // 5 << 30) + T))
        assert lib.reft_pack_device(c.plan, ptrs, HOST + (i << 30), L, PER_THREAD) == 0
        assert lib.sim_races() == 0
    c.end()


@pytest.mark.parametrize("load", [False, True])
@pytest.mark.parametrize("then", [(1, 1), (4, 5), (3, 4), (2, 2)])
@pytest.mark.parametrize("streams", [(1, 1), (1, 3)])
@pytest.mark.parametrize("copies", [1, 2, 3, 5, 6])
def test_calls_that_fail_midway(lib, copies, streams, then, load):
    """What a failed call has queued still reads and writes the slots: a later call keeps behind it."""
    c = Calls(lib, 100_000)
    assert c.call(load, *streams) == 0
    lib.sim_fail(copies + 1)                               # the pointers' upload, and then so many
    assert c.call(load, *streams) != 0
    lib.sim_fail(-1)
    assert c.call(load, *then) == 0
    assert lib.sim_clashes() == 0
    c.end()


@pytest.mark.parametrize("load", [False, True])
@pytest.mark.parametrize("calls", [[(2, 0), (6, 0)], [(6, 0), (2, 0)], [(6, 0), (2, 0), (6, 0)], [(4, 0), (4, 2), (4, 0)], [(6, 1), (3, 0), (6, 1), (2, 4)],
                                   [(2, 0), (2, 8), (2, 0), (2, 8)], [(1, 0), (4, 0), (1, 2), (8, 0), (3, 3)],
                                   [(2, 2 * i) for i in range(9)] + [(9, 0), (2, 4), (64, 0)]])
@pytest.mark.parametrize("alone", [(), (0, 2), (1,), (0, 1, 2, 3)])
def test_rings_of_other_sizes_and_places(lib, calls, alone, load):
    """Calls whose rings lie in the same memory with other numbers of slots, or in part of it; `alone`: those on one stream."""
    c = Calls(lib, 40_000)
    for i, (slots, first) in enumerate(calls):
        a = 10 + 2 * i
        assert c.call(load, a, a if i in alone else a + 1, RING + first * c.slot, slots) == 0
        assert lib.sim_clashes() == 0, i
    c.end()


@pytest.mark.parametrize("load", [False, True])
@pytest.mark.parametrize("seed", range(20))
def test_calls_in_any_order(lib, seed, load):
    """Rings anywhere in one piece of memory, one stream and two, threads that share a handle, a call in ten that fails."""
    rng = random.Random(seed)
    for bucket in (0, 20_000, 40_000, 150_000):
        c = Calls(lib, bucket)
        for i in range(25):
            first = rng.choice((None, 1, 3, 4, 5, PER_THREAD))
            second = first if rng.random() < 0.5 else rng.choice((None, 1, 3, 4, 5, PER_THREAD))
            lib.sim_thread(rng.randrange(3))
            lib.sim_fail(rng.randrange(8) if rng.random() < 0.1 else -1)
            c.call(load, first, second, RING + rng.randrange(12) * c.slot, rng.choice((1, 2, 3, 5, 8, 64)))
            lib.sim_fail(-1)
            assert lib.sim_clashes() == 0, i
        c.end()


@pytest.mark.parametrize("load", [False, True])
def test_a_failed_call_keeps_what_other_groups_wait_for(lib, load):
    """Two groups of slots under way; a call elsewhere that fails in its first group; one across the second group's slots."""
    c = Calls(lib, 40_000)
    assert c.call(load, 4, 1, RING + c.slot, 8) == 0
    lib.sim_fail(3)
    assert c.call(load, 5, 6, RING + 11 * c.slot, 1) != 0
    lib.sim_fail(-1)
    assert c.call(load, 3, 3, RING + 6 * c.slot, 5) == 0
    assert lib.sim_clashes() == 0
    c.end()
