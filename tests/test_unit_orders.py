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
