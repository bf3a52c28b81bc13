"""Grid sizes and launch rules of the kernels, compiled from the library's own header as a host program."""
import ctypes
import os
import subprocess

import pytest

import paper_2310_12670_amd as reft

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2310_12670_amd", "csrc")
SOURCE = """
#include "reft_rules.hpp"
extern "C" uint32_t stream(uint64_t nunits, uint32_t waves, uint32_t cap) { return reft::stream_grid(nunits, waves, cap); }
extern "C" uint32_t link(uint64_t link_wgs, uint32_t halves, uint32_t max_wgs) { return reft::link_cap(link_wgs, halves, max_wgs); }
extern "C" uint32_t run(uint64_t nunits, uint64_t waves, uint32_t nsrc, uint64_t mean) { return reft::run_of_units(nunits, waves, nsrc, mean); }
extern "C" int span_burst(uint64_t rows, uint64_t bytes) { return reft::span_burst(rows, bytes); }
extern "C" uint64_t unit(uint32_t kib, uint64_t w, uint64_t n) { return kib == 1 ? reft::unit_of_wave<1>(w, n) : reft::unit_of_wave<2>(w, n); }
extern "C" uint64_t contig_rows(uint64_t rows) { return reft::contig_burst_min_rows(rows); }
extern "C" uint64_t contig_bytes(uint64_t bytes) { return reft::contig_burst_min_bytes(bytes); }
"""
GiB = 1 << 30


@pytest.fixture(scope="module")
def grid(tmp_path_factory):
    d = tmp_path_factory.mktemp("grid")
    (d / "grid.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-shared", "-fPIC", "-O1", "-I", CSRC, "-o", str(d / "grid.so"), str(d / "grid.cpp")], check=True)
    lib = ctypes.CDLL(str(d / "grid.so"))
    lib.stream.argtypes = [ctypes.c_uint64, ctypes.c_uint32, ctypes.c_uint32]
    lib.stream.restype = ctypes.c_uint32
    lib.link.argtypes = [ctypes.c_uint64, ctypes.c_uint32, ctypes.c_uint32]
    lib.link.restype = ctypes.c_uint32
    lib.run.argtypes = [ctypes.c_uint64, ctypes.c_uint64, ctypes.c_uint32, ctypes.c_uint64]
    lib.run.restype = ctypes.c_uint32
    lib.span_burst.argtypes = [ctypes.c_uint64, ctypes.c_uint64]
    lib.unit.argtypes = [ctypes.c_uint32, ctypes.c_uint64, ctypes.c_uint64]
    lib.unit.restype = ctypes.c_uint64
    for f in (lib.contig_rows, lib.contig_bytes):
        f.argtypes = [ctypes.c_uint64]
        f.restype = ctypes.c_uint64
    return lib


@pytest.mark.parametrize("waves", [1, 4])
@pytest.mark.parametrize("unit", [1024, 2048, 4096])
@pytest.mark.parametrize("nbytes", [1, 1023, 1024, 5 << 20, 32 * GiB, 64 * GiB - 1024, 64 * GiB - 1, 64 * GiB, 64 * GiB + 1,
                                    128 * GiB - 2048, 128 * GiB, 256 * GiB, 288 * 10**9, 1 << 45])
def test_stream_launch_fits_a_dispatch(grid, nbytes, unit, waves):
    """Fewer than 2^32 work-items whatever the stream's length, and a wave per unit where they are."""
    units = -(-nbytes // unit)
    g = grid.stream(units, waves, 0)
    assert 1 <= g and g * 64 * waves < 1 << 32
    assert g == min(-(-units // waves), (2**32 - 1) // (64 * waves))


@pytest.mark.parametrize("waves", [1, 4])
@pytest.mark.parametrize("cap", [1, 7, 48, 1 << 20])
def test_stream_cap(grid, cap, waves):
    for units in (1, 5, 100, 1 << 30, 1 << 35):
        assert grid.stream(units, waves, cap) == min(-(-units // waves), cap, (2**32 - 1) // (64 * waves))


@pytest.mark.parametrize("halves", [3, 4])
def test_link_cap_keeps_to_max_wgs(grid, halves):
    """Direct snapshot: half as many again as link_wgs; direct restore: twice; "max_wgs" bounds both."""
    for link in (1, 2, 16, 32, 1 << 20):
        for most in (1, 4, 16, 33, 4096, 1 << 20):
            assert grid.link(link, halves, most) == min(link * halves // 2, most)


def test_packed_decode_goes_by_the_callers_burst_limits(grid):
    """reft_reconstruct takes "burst_min_rows" and "burst_min_bytes" as they are set, raised or lowered;
    only at their defaults does it have limits of its own."""
    rows, size = reft.reft_get_tunable("burst_min_rows"), reft.reft_get_tunable("burst_min_bytes")
    assert grid.contig_rows(rows) == 5 and grid.contig_bytes(size) == 8 << 20
    for r in (1, 2, 5, 6, 8, 9, 32, 1 << 40):
        assert grid.contig_rows(r) == r
    for b in (0, 1, 8 << 20, 9 << 20, 1 << 30, (2 << 30) + 1, 4 << 30, 1 << 62):
        assert grid.contig_bytes(b) == b


def test_burst_kernel_over_spans_is_asked_for(grid):
    """By default the calls over span tables take the stream kernel; either value set brings the burst kernel back."""
    rows, size = reft.reft_get_tunable("burst_min_rows"), reft.reft_get_tunable("burst_min_bytes")
    assert not grid.span_burst(rows, size)
    assert grid.span_burst(rows - 1, size) and grid.span_burst(rows, size + 1) and grid.span_burst(1, 0)


def test_runs_leave_every_wave_eight(grid):
    """1 to 16 units together; one at a time from five sources on, with many waves and in short spans."""
    for waves in (4, 16, 256, 384, 896, 4096):
        for units in (1, 100, 30720, 1 << 22, 1 << 36):
            for nsrc in (1, 2, 4, 5, 16):
                for mean in (10_000, 1 << 18, 1 << 30):
                    n = grid.run(units, waves, nsrc, mean)
                    assert n == 1 or (2 <= n <= 16 and n * 8 * waves <= units)
                    if nsrc > 4 or waves > (896 if nsrc == 1 else 384) or mean < 1 << 18:
                        assert n == 1
    assert grid.run(30720, 16, 1, 1 << 20) == 16 and grid.run(30720, 512, 1, 1 << 20) == 7


@pytest.mark.parametrize("kib", [1, 2])
def test_every_unit_has_one_wave(grid, kib):
    """The order of units is a permutation inside 32 KiB, each XCD on its own bits; what is left stays in order."""
    for n in (1, 31, 32, 33, 63, 64, 65, 1000, 4097):
        units = [grid.unit(kib, w, n) for w in range(n)]
        assert sorted(units) == list(range(n))
        assert all(u // 32 == w // 32 for w, u in enumerate(units)) and units[n // 32 * 32:] == list(range(n // 32 * 32, n))
        own = 0b10011 if kib == 1 else 0b01011
        for x in range(8):
            assert len({u & own for u in units[x:n // 32 * 32:8]}) <= 1
    for n in (1 << 33, (1 << 40) + 5):                # beyond 32 bits
        at = n // 32 * 32 - 64
        assert sorted(grid.unit(kib, w, n) for w in range(at, n)) == list(range(at, n))
