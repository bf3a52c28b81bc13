"""Which unit a wave moves where a launch deals its steps in another order, compiled from the library's own header."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2310_12670_amd", "csrc")
SOURCE = """
#include "reft_rules.hpp"
extern "C" uint64_t turned(uint32_t units, uint64_t u, uint64_t u0, uint64_t u1, uint32_t turn)
{
    return units == 1 ? reft::turned<1>(u, u0, u1, turn) : reft::turned<2>(u, u0, u1, turn);
}
extern "C" uint64_t near_step(uint64_t w, uint64_t n) { return reft::near_step_of_wave(w, n); }
extern "C" uint64_t pair_step(uint64_t w, uint64_t n) { return reft::pair_step_of_wave(w, n); }
extern "C" bool in_pairs(uint32_t nsrc, uint64_t mean, uint64_t traffic, bool odd, bool packed, bool tensors, bool windows)
{
    return reft::in_pairs(nsrc, mean, traffic, odd, packed, tensors, windows);
}
extern "C" uint32_t spread_of(uint32_t nsrc, uint64_t mean, uint64_t traffic, bool odd, bool packed, bool tensors, bool windows)
{
    return reft::spread_of(nsrc, mean, traffic, odd, packed, tensors, windows);
}
extern "C" uint32_t pair_lds(uint32_t nsrc, uint64_t mean, bool packed) { return 2 * reft::crowd_lds(reft::pair_waves(nsrc, mean, packed)); }
extern "C" bool writes_through(uint32_t nsrc, uint64_t mean, uint64_t traffic, bool odd, bool packed)
{
    return reft::writes_through(nsrc, mean, traffic, odd, packed);
}
extern "C" uint32_t through_waves(uint32_t nsrc, bool packed) { return reft::through_waves(nsrc, packed); }
extern "C" uint32_t crowd_waves(uint32_t nsrc, uint64_t mean, bool packed) { return reft::crowd_waves(nsrc, mean, packed); }
extern "C" uint32_t crowd_lds(uint32_t waves) { return reft::crowd_lds(waves); }
extern "C" uint32_t turn_of(uint64_t number, uint64_t kib) { return reft::turn_of(number, kib); }
"""


def build(tmp_path_factory, source):
    d = tmp_path_factory.mktemp("orders")
    (d / "orders.cpp").write_text(source)
    subprocess.run(["g++", "-shared", "-fPIC", "-O1", "-I", CSRC, "-o", str(d / "orders.so"), str(d / "orders.cpp")], check=True)
    return ctypes.CDLL(str(d / "orders.so"))


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    lib = build(tmp_path_factory, SOURCE)
    lib.turned.argtypes = [ctypes.c_uint32, ctypes.c_uint64, ctypes.c_uint64, ctypes.c_uint64, ctypes.c_uint32]
    lib.turned.restype = ctypes.c_uint64
    lib.turn_of.argtypes = [ctypes.c_uint64, ctypes.c_uint64]
    lib.turn_of.restype = ctypes.c_uint32
    for f in (lib.near_step, lib.pair_step):
        f.argtypes = [ctypes.c_uint64, ctypes.c_uint64]
        f.restype = ctypes.c_uint64
    lib.in_pairs.argtypes = [ctypes.c_uint32, ctypes.c_uint64, ctypes.c_uint64] + [ctypes.c_bool] * 4
    lib.in_pairs.restype = ctypes.c_bool
    lib.spread_of.argtypes = [ctypes.c_uint32, ctypes.c_uint64, ctypes.c_uint64] + [ctypes.c_bool] * 4
    lib.writes_through.argtypes = [ctypes.c_uint32, ctypes.c_uint64, ctypes.c_uint64, ctypes.c_bool, ctypes.c_bool]
    lib.writes_through.restype = ctypes.c_bool
    lib.through_waves.argtypes = [ctypes.c_uint32, ctypes.c_bool]
    lib.crowd_waves.argtypes = [ctypes.c_uint32, ctypes.c_uint64, ctypes.c_bool]
    lib.pair_lds.argtypes = [ctypes.c_uint32, ctypes.c_uint64, ctypes.c_bool]
    return lib


@pytest.mark.parametrize("per_step", [1, 2])
@pytest.mark.parametrize("first", [0, 1, 32, 77, (1 << 33) + 5])
@pytest.mark.parametrize("n", [33, 34, 35, 63, 64, 65, 1000])
def test_turned_steps_cover_a_span(rules, n, first, per_step):
    """Every whole step of the span is moved once, whatever the turn; what is no whole step is not asked for."""
    whole = [u for u in range(first, first + n) if u % per_step == 0 and u + per_step <= first + n]
    for turn in range(32):
        assert sorted(rules.turned(per_step, u, first, first + n, turn) for u in whole) == whole


@pytest.mark.parametrize("first", [0, 5, 31, 1 << 34])
@pytest.mark.parametrize("kib", [0, 9, 40, (1 << 37) + 3])
def test_turned_units_have_the_numbers_of_their_kib(rules, first, kib):
    """Modulo 32, but for those that follow behind the last one."""
    n, turn = 100, rules.turn_of(first, kib)
    for u in range(first, first + n - turn):
        assert (u - (kib + rules.turned(1, u, first, first + n, turn) - first)) % 32 == 0


@pytest.mark.parametrize("name", ["near_step", "pair_step"])
def test_orders_are_permutations(rules, name):
    """Inside 32 steps, each XCD on bits 1, 2 and 4; what is left stays in order."""
    order, waves = getattr(rules, name), 2 if name == "pair_step" else 1
    for n in (1, 31, 32, 33, 63, 64, 65, 1000, 4097):
        steps = [order(w, n) for w in range(n)]
        assert sorted(steps) == list(range(n))
        assert all(u // 32 == w // 32 for w, u in enumerate(steps)) and steps[n // 32 * 32:] == list(range(n // 32 * 32, n))
        for x in range(8):
            assert len({steps[w] & 0b10110 for w in range(n // 32 * 32) if w // waves % 8 == x}) <= 1
    for n in (1 << 33, (1 << 40) + 5):                # beyond 32 bits
        at = n // 32 * 32 - 64
        assert sorted(order(w, n) for w in range(at, n)) == list(range(at, n))
    if waves == 2:
        assert all(order(w, 64) + 1 == order(w + 1, 64) for w in range(0, 64, 2))


def test_which_order_a_launch_takes(rules):
    in_order, far, near, pairs, unturned = range(5)
    k20, k32, k64 = 20 << 10, 32 << 10, 64 << 10
    for nsrc in range(1, 17):
        for odd in (False, True):
            for packed in (False, True):
                for windows in (False, True):
                    for tensors in (False, True):
                        got, short = [[rules.spread_of(nsrc, mean, traffic, odd, packed, tensors, windows)
                                       for mean in (k20 - 1, k20, k32 - 1, k32, k64 - 1, k64)]
                                      for traffic in (512 << 20, (512 << 20) - 1)]
                        alone = nsrc == 1 and not packed
                        assert got[0] == in_order and got[1] == got[2] and (got[2] == in_order) == alone
                        # below 512 MiB of traffic: those that keep to address bits, but odd copies of short spans
                        assert short == [order if order in (in_order, pairs) or (alone and odd and i < 5) else unturned
                                         for i, order in enumerate(got)]
                        if not odd:
                            assert set(got[3:]) == {far}
                        elif packed or nsrc in (2, 3):
                            assert set(got[3:]) == {far if nsrc == 1 else pairs}
                        elif alone:
                            assert got[3:] == [near, near, far]
                        elif windows and nsrc <= 12:
                            assert set(got[3:]) == {near}
                        else:
                            assert got[3] == far and got[4] == far and got[5] == (far if tensors or windows or nsrc > 12 else near)
                        for mean, order in zip((k20 - 1, k20, k64), (got[0], got[1], got[5])):
                            assert order == in_order or (order == pairs) == rules.in_pairs(nsrc, mean, 512 << 20, odd, packed, tensors, windows)
                            assert rules.pair_lds(nsrc, mean, packed) <= 64 << 10
            for tensors in (False, True):
                for windows in (False, True):
                    for mean in (600, (4 << 10) - 1, 4 << 10, (5 << 10) - 1, 5 << 10, (11 << 10) - 1, 11 << 10, (12 << 10) - 1,
                                 12 << 10, k20 - 1, k20):
                        if not windows:
                            most = 16 if mean < 4 << 10 else 8 if mean < k20 else 3
                        elif tensors:
                            most = 16 if mean < 12 << 10 else 11 if mean < k20 else 3
                        else:
                            most = 16 if mean < 11 << 10 else 4 if mean < k20 else 3
                        assert rules.in_pairs(nsrc, mean, 512 << 20, odd, False, tensors, windows) == (
                            odd and nsrc <= most and (nsrc > 1 or 5 << 10 <= mean < k20))
                        assert rules.in_pairs(nsrc, mean, 512 << 20, odd, True, tensors, windows) == (
                            odd and 2 <= nsrc <= (8 if mean < k20 else 16))
                        for packed in (False, True):
                            assert rules.pair_lds(nsrc, mean, packed) <= 64 << 10


def test_pairs_in_longer_spans_from_some_traffic_on(rules):
    """Spans of 20 KiB and more, but for windows; in shorter ones the traffic makes no difference."""
    k20, MiB = 20 << 10, 1 << 20
    for nsrc in range(2, 17):
        for packed in (False, True):
            least = (1 if nsrc <= 3 else 160 if nsrc <= 8 else 352) if packed else 144 if nsrc == 2 else 192
            for traffic in (97 * MiB, least * MiB - 1, least * MiB, 1 << 40):
                for tensors in (False, True):
                    usual = rules.in_pairs(nsrc, k20, 1 << 40, True, packed, tensors, False)
                    assert rules.in_pairs(nsrc, k20, traffic, True, packed, tensors, False) == (usual and (least == 1 or traffic >= least * MiB))
                    for mean, windows in ((k20, True), (k20 - 1, False), (3 << 10, False), (k20 - 1, True)):
                        assert rules.in_pairs(nsrc, mean, traffic, True, packed, tensors, windows) == rules.in_pairs(
                            nsrc, mean, 1 << 40, True, packed, tensors, windows)


def test_which_launches_write_through(rules):
    """Long spans, aligned, and more than twice the cache, longer ones of few sources, and of copies with far more;
    and LDS for no more waves than those are to have."""
    for nsrc in range(1, 17):
        for packed in (False, True):
            copy = nsrc == 1
            least = 4 << 20 if copy else 1 << 20 if nsrc <= (2 if packed else 4) else 128 << 10
            most = 2 << 30 if copy else 512 << 20
            for mean in (least - 1, least):
                for traffic in (most - 1, most):
                    for odd in (False, True):
                        assert rules.writes_through(nsrc, mean, traffic, odd, packed) == (
                            mean == least and traffic == most and not odd and not (copy and packed))
            waves = rules.through_waves(nsrc, packed)
            assert 8 <= waves <= rules.crowd_waves(nsrc, 128 << 10, packed) and rules.crowd_lds(waves) <= 64 << 10
