"""Which streams of very long rows the write-burst kernel encodes, without a GPU: the host code on the runtime of
test_table_cache.py, which counts its launches."""
import ctypes

import pytest

import test_table_cache
from test_table_cache import lib  # noqa: F401  (a fixture)

test_table_cache.SOURCE = test_table_cache.SOURCE.replace(
    "uint64_t, const LaunchCfg &, const BurstCfg &, hipStream_t s) { return kernel(",
    "uint64_t, const LaunchCfg &, const BurstCfg &, hipStream_t s) { ++bursts; return kernel(", 1).replace(
    "namespace reft {", 'static uint64_t bursts;\nextern "C" uint64_t sim_bursts() { return bursts; }\nnamespace reft {', 1)


def call(lib, rows, limit, spans, **tunables):  # noqa: F811
    lib.sim_bursts.restype = ctypes.c_uint64
    lib.reft_set_tunable.argtypes = [ctypes.c_char_p, ctypes.c_uint64]
    lib.reft_get_tunable.argtypes = [ctypes.c_char_p, ctypes.POINTER(ctypes.c_uint64)]
    was = {}
    for name, value in dict(tunables, burst_min_bytes=13 << 30 if limit is None else limit).items():
        old = ctypes.c_uint64()
        assert lib.reft_get_tunable(name.encode(), ctypes.byref(old)) == 0
        was[name] = old.value
        assert lib.reft_set_tunable(name.encode(), value) == 0
    lib.sim_end()
    lib.sim_call(None)
    plan = ctypes.c_void_p()
    n = len(spans)
    try:
        assert lib.reft_plan_create((ctypes.c_uint64 * n)(*spans), n, None, 0, 0, ctypes.byref(plan)) == 0
        before = lib.sim_bursts()
        pointers = (ctypes.c_void_p * (rows * n))(*((1 << 45) + (i << 31) for i in range(rows * n)))
        assert lib.reft_parity_encode(plan, pointers, rows, 1 << 44, None) == 0, lib.reft_last_error()
        return lib.sim_bursts() - before
    finally:
        for name, value in was.items():
            lib.reft_set_tunable(name.encode(), value)
        lib.reft_plan_destroy(plan)
        lib.sim_end()


@pytest.mark.parametrize("rows,limit,spans,want", [
    (8, None, [1 << 30] * 14, 0), (7, None, [1 << 30] * 14, 0),            # written through the L2 by the stream kernel
    (8, None, [(1 << 30) + 1] * 14, 1), (7, None, [(1 << 30) + 1] * 14, 1), (6, None, [(1 << 30) + 1] * 14, 0),
    (8, None, [(1 << 30) + 1] * 12, 0),                                    # below 13 GiB
    (8, None, [1 << 16] * (14 << 14), 0),                                   # dense in small spans
    (8, 1 << 30, [1 << 30] * 14, 1), (8, 1 << 30, [(1 << 30) + 1] * 2, 1),  # where the caller has said from where on
])
def test_rows_of_many_gigabytes(lib, rows, limit, spans, want):  # noqa: F811
    assert call(lib, rows, limit, spans) == want


@pytest.mark.parametrize("tunables", [{"max_wgs": 512}, {"nontemporal": 0}])
def test_launches_that_are_not_written_through(lib, tunables):  # noqa: F811
    assert call(lib, 8, None, [1 << 30] * 14, **tunables) == 1
