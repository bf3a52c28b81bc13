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
extern "C" uint32_t crowd_waves(uint32_t nsrc, uint64_t mean, bool packed) { return reft::crowd_waves(nsrc, mean, packed); }
extern "C" uint32_t crowd_lds(uint32_t waves) { return reft::crowd_lds(waves); }
extern "C" uint64_t units_of(uint64_t n, uint64_t head) { return reft::units_of(n, head); }
extern "C" uint32_t align_of(uint64_t L, uint64_t T) { return reft::align_of(L, T); }
extern "C" uint32_t grid_of(uint64_t L, uint64_t T) { return reft::grid_of(L, T); }
extern "C" uint64_t first_number(uint64_t least, uint64_t off, uint64_t align) { return reft::first_number(least, off, align); }
extern "C" uint64_t head_of(uint64_t off, uint64_t grid) { return reft::head_of(off, grid); }
extern "C" uint64_t first_unit_at(uint64_t r, uint64_t head) { return reft::first_unit_at(r, head); }
extern "C" uint64_t last_unit_at(uint64_t r, uint64_t head) { return reft::last_unit_at(r, head); }
extern "C" void piece_of(uint64_t j, uint64_t head, uint32_t lead, int64_t lo, int64_t hi, int64_t *st)
{
    const reft::Piece p = reft::piece_of(j, head, lead, lo, hi);
    st[0] = p.s;
    st[1] = p.t;
}
extern "C" uint64_t unit_bytes(uint64_t L, uint64_t T) { return reft::unit_bytes(L, T); }
extern "C" uint64_t small_units_of(uint64_t n) { return reft::units_of(n, reft::kSmallUnit, reft::kSmallUnit); }
extern "C" uint64_t small_first_at(uint64_t r) { return reft::first_unit_at(r, reft::kSmallUnit, reft::kSmallUnit); }
extern "C" uint64_t small_last_at(uint64_t r) { return reft::last_unit_at(r, reft::kSmallUnit, reft::kSmallUnit); }
extern "C" void small_piece_of(uint64_t j, int64_t lo, int64_t hi, int64_t *st)
{
    const reft::Piece p = reft::piece_of(j, reft::kSmallUnit, 0, lo, hi, reft::kSmallUnit);
    st[0] = p.s;
    st[1] = p.t;
}
extern "C" int32_t lane_place(int32_t at, int32_t len) { return reft::lane_place(at, len); }
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
    lib.crowd_waves.argtypes = [ctypes.c_uint32, ctypes.c_uint64, ctypes.c_bool]
    lib.crowd_lds.argtypes = [ctypes.c_uint32]
    lib.crowd_waves.restype = lib.crowd_lds.restype = ctypes.c_uint32
    lib.first_number.argtypes = [ctypes.c_uint64] * 3
    lib.first_number.restype = ctypes.c_uint64
    for f in (lib.units_of, lib.first_unit_at, lib.last_unit_at, lib.grid_of, lib.align_of, lib.head_of):
        f.argtypes = [ctypes.c_uint64, ctypes.c_uint64]
        f.restype = ctypes.c_uint64
    lib.unit_bytes.argtypes = [ctypes.c_uint64, ctypes.c_uint64]
    for f in (lib.small_units_of, lib.small_first_at, lib.small_last_at):
        f.argtypes = [ctypes.c_uint64]
    for f in (lib.unit_bytes, lib.small_units_of, lib.small_first_at, lib.small_last_at):
        f.restype = ctypes.c_uint64
    lib.small_piece_of.argtypes = [ctypes.c_uint64, ctypes.c_int64, ctypes.c_int64, ctypes.POINTER(ctypes.c_int64)]
    lib.piece_of.argtypes = [ctypes.c_uint64, ctypes.c_uint64, ctypes.c_uint32, ctypes.c_int64, ctypes.c_int64, ctypes.POINTER(ctypes.c_int64)]
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
    for b in (0, 1, 8 << 20, 9 << 20, 1 << 30, 2 << 30, (2 << 30) + 1, 4 << 30, (13 << 30) - 1, (13 << 30) + 1, 1 << 62):
        assert grid.contig_bytes(b) == b


def test_runs_leave_every_wave_eight(grid):
    """1 to 16 units together; one at a time from five sources on, with many waves and in short spans."""
    most = {1: 896, 2: 768, 3: 384, 4: 384}
    for waves in (4, 16, 256, 384, 385, 512, 768, 769, 896, 897, 4096):
        for units in (1, 100, 30720, 1 << 22, 1 << 36):
            for nsrc in (1, 2, 3, 4, 5, 16):
                for mean in (10_000, (1 << 18) - 1, 1 << 18, 1 << 30):
                    n = grid.run(units, waves, nsrc, mean)
                    assert n == 1 or (2 <= n <= 16 and n * 8 * waves <= units)
                    if nsrc > 4 or waves > most[nsrc] or mean < 1 << 18:
                        assert n == 1
                    elif units == 1 << 36:
                        assert n == 16
    assert grid.run(30720, 16, 1, 1 << 20) == 16 and grid.run(30720, 512, 1, 1 << 20) == 7


def test_waves_that_share_a_compute_unit(grid):
    """As swept, the more sources the fewer; and LDS for no more of them, in blocks as the device hands it out."""
    swept = [24, 32, 24, 16, 15, 14, 13, 12, 12, 11, 11, 10, 9, 9, 8, 8]
    assert [grid.crowd_waves(k, 1 << 20, False) for k in range(1, 17)] == swept
    assert [grid.crowd_waves(k, (1 << 20) - 1, False) for k in range(1, 17)] == [24, 28] + swept[2:]
    assert [grid.crowd_waves(k, 65535, False) for k in (1, 2, 3)] == [32, 28, 24]
    assert [grid.crowd_waves(k, 1 << 16, True) for k in (1, 2, 3, 8)] == [32, 28, 24, 12]
    assert grid.crowd_lds(32) == 0
    for waves in {28, *swept} - {32}:
        asked = grid.crowd_lds(waves)
        assert asked <= 64 << 10 and waves - 3 <= (160 << 10) // (-(-asked // 1280) * 1280) <= waves


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


@pytest.mark.parametrize("mean", [1 << 16, 70_001, 300_000, 1 << 20, 3 << 20])
def test_units_that_are_spread_have_the_numbers_of_their_kib(grid, mean):
    """From a mean of 64 KiB on, where a launch spreads them: modulo 8, from 256 KiB on modulo the 32 KiB inside which they
    change places."""
    sizes = [mean + (-1) ** i * (7 * i % 61) * 100 for i in range(96)]
    sizes[-1] += 96 * mean - sum(sizes)
    mask, align = grid.grid_of(sum(sizes), len(sizes)), grid.align_of(sum(sizes), len(sizes))
    assert mask == 1023 and grid.grid_of(96 * 65536 - 1, 96) == 0 and align == (31 if mean >= 1 << 18 else 7)
    assert grid.align_of((5 << 20) - 1, 2) == grid.grid_of((5 << 20) - 1, 2) == 0 and grid.align_of(5 << 20, 2) == 31
    off = number = 0
    for n in sizes:
        number = grid.first_number(number, off, align)
        for j in (0, 1, grid.units_of(n, grid.head_of(off, mask)) - 1):
            start = off if j == 0 else off + grid.head_of(off, mask) + (j - 1) * 1024
            assert (number + j - start // 1024) & align == 0
        number += grid.units_of(n, grid.head_of(off, mask))
        off += n


def moved(grid, n, head, lead, lo, hi, once):
    """How often each byte of a span of n bytes is written by the units that a launch over its bytes lo .. hi - 1
    has, as the kernel's lanes do it."""
    count = [0] * n
    st = (ctypes.c_int64 * 2)()
    low, high = max(lo, 0), min(hi, n)
    for j in range(grid.first_unit_at(low, head), grid.last_unit_at(high - 1, head) + 1):
        assert j < grid.units_of(n, head)
        grid.piece_of(j, head, 0 if once else lead, low, high, st)
        a, b = st
        if a >= b:
            continue
        size = b - a
        assert size < 1024 + 128
        if not once and b - low >= 16:
            start, size = (b - 16, 16) if size < 16 else (a, size)
            at = [start + grid.lane_place(16 * x, size) for x in range(-(-size // 16))]
            assert all(start <= x and x + 16 <= b for x in at)
            places = [x + i for x in at for i in range(16)]
        else:
            places = range(a, b)                       # 16 bytes a lane, what is left one byte a lane
        for x in places:
            assert low <= x < high
            count[x] += 1
    return count


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 100, 127, 128, 129, 1023, 1024, 1025, 1040, 1151, 1152, 1153, 2047, 2048,
                               2049, 2200, 5000])
def test_units_cover_a_span(grid, n):
    cuts = sorted({x for x in (0, 1, 5, 15, 16, 100, 127, 128, 500, 1008, 1023, 1024, 1025, 1100, 2040, n - 17, n - 1, n)
                   if 0 <= x <= n})
    for head, lead in [(1024, x) for x in (0, 1, 15, 16, 64, 127)] + [(1, 0), (1, 127), (17, 3), (600, 120), (1023, 127)]:
        for lo in cuts:
            for hi in cuts:
                if lo < hi:
                    for once in (False, True):
                        count = moved(grid, n, head, lead, -70 if lo == 0 else lo, hi + 90 if hi == n else hi, once)
                        assert not any(count[:lo]) and not any(count[hi:])
                        assert all(c == 1 if once else c >= 1 for c in count[lo:hi])


def moved_in_steps(grid, n, head, lead, lo, hi, once, steps, before):
    """The same where a wave takes `steps` units of a span together (the span's first unit is the before-th of one)."""
    count = [0] * n
    st, en = (ctypes.c_int64 * 2)(), (ctypes.c_int64 * 2)()
    low, high = max(lo, 0), min(hi, n)
    first, last = grid.first_unit_at(low, head), grid.last_unit_at(high - 1, head)
    j = first
    while j <= last:
        end = min((j + before) // steps * steps + steps - before, last + 1)
        grid.piece_of(j, head, 0 if once else lead, low, high, st)
        grid.piece_of(end - 1, head, 0 if once else lead, low, high, en)
        j, a, b = end, st[0], en[1]
        if a >= b:
            continue
        twice, size = not once and b - low >= 16, b - a
        assert size < 1024 * steps + 128
        if twice and size < 16:
            size = 16
        start, places = b - size, []
        if size >= 16:
            chunks = min(-(-size // 1024), steps)
            for x in range(chunks * 64):
                place = start + grid.lane_place(16 * x, size)
                assert start <= place and place + 16 <= b
                if 16 * x + (0 if twice else 15) < size:
                    places.append(place)
            if size > steps * 1024:
                places += [start + grid.lane_place(steps * 1024 + 16 * x, size) for x in range(64) if 16 * x < size - steps * 1024]
        places = [x + i for x in places for i in range(16)]
        if not twice:
            places += range(a + (size & ~15), a + size)
        for x in places:
            assert low <= x < high
            count[x] += 1
    return count


def moved_small(grid, n, lo, hi, once):
    """The same for units of 256 bytes, 16 lanes each."""
    count = [0] * n
    st = (ctypes.c_int64 * 2)()
    low, high = max(lo, 0), min(hi, n)
    for j in range(grid.small_first_at(low), grid.small_last_at(high - 1) + 1):
        assert j < grid.small_units_of(n)
        grid.small_piece_of(j, low, high, st)
        a, b = st
        if a >= b:
            continue
        twice, size = not once and b - low >= 16, b - a
        assert size <= 256
        whole, k = size & ~15, 16 if twice and size < 16 else size
        for me in range(16):
            at = 16 * me
            place = b - k + (grid.lane_place(at, k) if twice else at)
            mine = list(range(place, place + 16)) if at + (0 if twice else 15) < k else []
            if not twice and me < size - whole:
                mine.append(a + whole + me)
            for x in mine:
                assert low <= x < high
                count[x] += 1
    return count


def cuts_of(n):
    return sorted({x for x in (0, 1, 5, 15, 16, 100, 127, 128, 255, 256, 257, 271, 272, 500, 1008, 1024, 1025, 1100, 2040, 4096,
                               n - 17, n - 1, n) if 0 <= x <= n})


@pytest.mark.parametrize("n", [1, 15, 16, 17, 129, 1023, 1024, 1025, 1151, 1153, 2048, 2200, 4095, 4097, 4224, 5000])
@pytest.mark.parametrize("steps", [2, 4])
def test_steps_of_units_cover_a_span(grid, n, steps):
    for head, lead, before in [(1024, 0, 0), (1024, 127, 1), (1, 0, 0), (1, 127, 3), (17, 3, 2), (600, 120, 1), (1023, 127, 0)]:
        cuts = cuts_of(n)
        for lo in cuts:
            for hi in cuts[::2] + [n]:
                if lo < hi:
                    for once in (False, True):
                        count = moved_in_steps(grid, n, head, lead, -70 if lo == 0 else lo, hi + 90 if hi == n else hi, once, steps,
                                               before % steps)
                        assert not any(count[:lo]) and not any(count[hi:])
                        assert all(c == 1 if once else c >= 1 for c in count[lo:hi])


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 100, 239, 240, 241, 255, 256, 257, 270, 272, 273, 511, 512, 513, 1000])
def test_small_units_cover_a_span(grid, n):
    for lo in cuts_of(n):
        for hi in cuts_of(n):
            if lo < hi:
                for once in (False, True):
                    count = moved_small(grid, n, -70 if lo == 0 else lo, hi + 90 if hi == n else hi, once)
                    assert not any(count[:lo]) and not any(count[hi:])
                    assert all(c == 1 if once else c >= 1 for c in count[lo:hi])


def test_small_units_have_an_entry_each(grid):
    """At most 4 a span, which is what the look-up table has room for."""
    assert grid.unit_bytes(511 * 1000, 1000) == 256 and grid.unit_bytes(512 * 1000, 1000) == 1024
    for sizes in ([511] * 999, [1] * 998 + [509_000], [257, 765] * 500):
        assert grid.unit_bytes(sum(sizes), len(sizes)) == 256
        assert sum(grid.small_units_of(n) for n in sizes) <= 4 * len(sizes)
