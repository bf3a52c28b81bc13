"""Every byte of a staged call's runs is moved once, whatever the order in which a launch deals its units: the launches that the
host code queues, without a GPU (the runtime of test_table_cache.py), each dealt step by step as the stream kernel deals it, in
every order and with one and two units a step, as if it were long enough to be spread, onto tensors that lie anywhere."""
import ctypes
import random

import pytest

import test_table_cache

MODEL = test_table_cache.SOURCE + r"""
#include "reft_rules.hpp"
using namespace reft;

// Bytes of the launch's range that no unit moves, or that one moves outside of it.  Where tensors are written (or a slot is, in
// plain stream order), unit 0 of a span begins at place + its offset in the stream, or at a place of its own.
template <uint32_t U>
static uint64_t not_moved(const Launch &l, int order, uint64_t place, bool own_places)
{
    const PlanTables &pt = l.pt;
    const StreamRange &r = l.range;
    std::vector<bool> moved(r.hi - r.lo);
    uint64_t wrong = 0;
    const uint64_t first_step = r.first / U, n = r.last / U - first_step + 1;
    if (first_step % 32) order = 0;
    for (uint64_t w = 0; w < n; ++w) {
        const uint64_t step = order == kFar || order == kFarUnturned ? unit_of_wave<U>(w, n) : order == kNear ? near_step_of_wave(w, n)
                              : order == kPairs ? pair_step_of_wave(w, n) : w;
        uint64_t u = (first_step + step) * U, end = u + U;
        if (u < r.first) u = r.first;
        if (end > r.last + 1) end = r.last + 1;
        for (bool turns = end - u == U; u < end; turns = false) {
            const uint64_t i = std::upper_bound(pt.unit_off, pt.unit_off + pt.T + 1, u) - pt.unit_off - 1;
            const uint64_t b = pt.off[i], e = pt.off[i + 1], u0 = pt.unit_off[i], u1 = pt.unit_off[i + 1];
            const uint64_t head = head_of(b, pt.grid), ref = (own_places ? place * (2 * i + 1) : place + b) + head;
            const bool wide = order && order != kFarUnturned && u1 - u0 > kTurned;
            const uint32_t lead = (uint32_t)(0 - ref) & ((wide ? kMaxLead : kLineLead) - 1);
            const uint32_t turn = wide && b >= r.lo && e <= r.hi ? turn_of(u0, (ref + lead - kUnit) / kUnit) : 0;
            if (turns && end <= u1) {
                u = turned<U>(u, u0, u1, turn);
                end = u + U;
            }
            for (const uint64_t part = end < u1 ? end : u1; u < part; ++u) {
                const int64_t lo = r.lo > b ? r.lo - b : 0, hi = (e < r.hi ? e : r.hi) - b;
                const Piece p = piece_of(u - u0, head, lead, lo, hi);
                for (int64_t x = p.s; x < p.t; ++x) {
                    const uint64_t at = b + x - r.lo;
                    if (at >= moved.size() || moved[at]) ++wrong;
                    else moved[at] = true;
                }
            }
        }
    }
    for (bool m : moved) wrong += !m;
    return wrong;
}

extern "C" uint64_t sim_launches() { return launches.size(); }
extern "C" uint64_t sim_not_moved(uint64_t i, int order, uint32_t units, uint64_t place, bool own_places)
{
    return units == 1 ? not_moved<1>(launches[i], order, place, own_places) : not_moved<2>(launches[i], order, place, own_places);
}
"""
LARGE = 5 << 20
HOST, RING = 1 << 40, 1 << 41


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    lib = test_table_cache.compile_with(MODEL, tmp_path_factory.mktemp("dealt_ranges"))
    p, u64 = ctypes.c_void_p, ctypes.c_uint64
    lib.reft_snapshot_pack_range.argtypes = [p, p, p, u64, p, u64, u64, u64, p, p]
    lib.reft_restore.argtypes = [p, p, u64, p, u64, p, p, p]
    lib.sim_not_moved.argtypes = [u64, ctypes.c_int, ctypes.c_uint32, u64, ctypes.c_bool]
    lib.sim_not_moved.restype = lib.sim_launches.restype = u64
    return lib


def check(lib, sizes, buckets, rng):
    T, L = len(sizes), sum(sizes)
    plan = ctypes.c_void_p()
    lib.sim_end()
    assert lib.reft_plan_create((ctypes.c_uint64 * T)(*sizes), T, (ctypes.c_uint64 * len(buckets))(*buckets) if buckets else None,
                                len(buckets), 0, ctypes.byref(plan)) == 0, lib.reft_last_error()
    ptrs = (ctypes.c_void_p * T)(*range(1 << 44, (1 << 44) + T))
    nb, runs = max(1, len(buckets)), 0
    for two in (0, 1):                                    # one stream, and two
        for lo, hi in [(0, nb)] + ([(1, nb)] if nb > 1 else []):
            lib.sim_call(1)
            assert lib.reft_snapshot_pack_range(plan, ptrs, RING, 1 << 34, HOST, L, lo, hi, 1, 1 + two) == 0
        assert lib.reft_restore(plan, HOST, L, RING, 1 << 34, ptrs, 1, 1 + two) == 0
    for i in range(lib.sim_launches()):
        runs += 1
        for order in range(5):
            for units in (1, 2):
                place = rng.randrange(1 << 30) if rng.random() < 0.5 else rng.randrange(1 << 30) // 512 * 512
                assert lib.sim_not_moved(i, order, units, place, rng.random() < 0.5) == 0, (sizes[:3], i, order, units, place)
    lib.reft_plan_destroy(plan)
    lib.sim_end()
    return runs


# 0, 7 and 31 unit numbers between spans; odd sizes and multiples of a KiB; a run that ends with the stream and one that does not
@pytest.mark.parametrize("sizes", [[20_001] * 300 + [LARGE], [70_001] * 70 + [LARGE], [300_001] * 20 + [LARGE], [LARGE] + [300_001] * 20,
                                   [300_001] * 10 + [0, LARGE, 0] + [70_001] * 40 + [LARGE], [1_500_000] * 9 + [LARGE, 17],
                                   [307_200] * 20 + [LARGE]])
def test_runs_in_front_of_a_copied_span(lib, sizes):
    assert check(lib, sizes, [], random.Random(len(sizes))) >= 4


@pytest.mark.parametrize("size", [70_001, 300_001, 1_500_000])
def test_buckets_that_end_where_tensors_end(lib, size):
    n = max(9, 9_000_000 // size)
    assert check(lib, [size] * 3 * n, [size * n] * 3, random.Random(size)) >= 12


@pytest.mark.parametrize("seed", range(12))
def test_drawn_streams(lib, seed):
    rng = random.Random(seed)
    mean = int(2 ** rng.uniform(14, 21))
    sizes, at, cut = [], 0, []
    while at < 12 << 20:
        sizes.append(rng.randrange(2 * mean) | 1 if rng.random() < 0.95 else rng.choice((0, 5, 1024, LARGE)))
        at += sizes[-1]
        if at - sum(cut) > 4 << 20 and rng.random() < 0.3:
            cut.append(at - sum(cut))
    if sum(cut) < at:
        cut.append(at - sum(cut))
    sizes += [LARGE]
    check(lib, sizes, [] if rng.random() < 0.5 else cut[:-1] + [cut[-1] + LARGE], rng)
