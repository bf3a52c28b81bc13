"""The pointers that a rotated unit or decode was made with the last two times: the table that a kernel gets is, word for word,
the one that a plan which has seen nothing makes of the call's own pointers, whatever came before.  Host code without a GPU, on
the runtime of test_table_cache.py, which also sees uploads into tables that a queued kernel may still read."""
import ctypes
import random

import numpy as np
import pytest

from test_table_cache import lib  # noqa: F401  (a fixture)

SIZES = [4096, 17, 0, 70_000, 333, 1 << 16, 900, 5]
T, L = len(SIZES), sum(SIZES)


class Rotated:
    def __init__(self, lib):  # noqa: F811
        self.lib = lib
        p, u32 = ctypes.c_void_p, ctypes.c_uint32
        lib.reft_parity_encode_rotated.argtypes = [p, p, u32, u32, p, p]
        lib.reft_reconstruct_rotated.argtypes = [p, p, p, u32, u32, p, p]
        lib.sim_table.argtypes = [p]
        lib.sim_table.restype = lib.sim_uploads.restype = ctypes.c_uint64
        lib.sim_end()

    def plan(self):
        plan = ctypes.c_void_p()
        assert self.lib.reft_plan_create((ctypes.c_uint64 * T)(*SIZES), T, None, 0, 0, ctypes.byref(plan)) == 0
        return plan

    def call(self, plan, shards, units, outs, k, member, decode, stream):
        """The call's table, and whether it was uploaded for it."""
        before = self.lib.sim_uploads()
        self.lib.sim_call(stream)
        s, u, o = ((ctypes.c_void_p * len(x))(*x.tolist()) for x in (shards, units, outs))
        if decode:
            rc = self.lib.reft_reconstruct_rotated(plan, s, u, k, member, o, stream)
        else:
            rc = self.lib.reft_parity_encode_rotated(plan, s, k, member, 1 << 40, stream)
        assert rc == 0, self.lib.reft_last_error()
        words = np.zeros(1 << 16, np.uint64)
        n = self.lib.sim_table(words.ctypes.data)
        assert n and self.lib.sim_races() == 0
        return words[:n].copy(), self.lib.sim_uploads() > before


def pointers(k, i):
    base = (1 << 44) + (i << 34)
    return [(base + (np.arange(n) << 21)).astype(np.uint64) for n in (k * T, k, T)]


def test_known_pointers_upload_nothing(lib):  # noqa: F811
    """Two sets in turn; not the lost member's, which may be anything; one that differs in a single word does."""
    c = Rotated(lib)
    plan = c.plan()
    for decode in (False, True):
        sets = [pointers(4, i) for i in (1, 2)]
        assert all(c.call(plan, *x, 4, 1, decode, None)[1] for x in sets)
        for _ in range(3):
            assert not any(c.call(plan, *x, 4, 1, decode, None)[1] for x in sets)
        sets[0][0][T:2 * T] += np.uint64(64)
        sets[0][1][1] = 0
        assert not c.call(plan, *sets[0], 4, 1, decode, None)[1]
        for which, at in ((0, 3),) + (((1, 0), (1, 3), (2, 0), (2, T - 1)) if decode else ()):
            sets[1][which][at] += np.uint64(16)
            assert c.call(plan, *sets[1], 4, 1, decode, None)[1]
    lib.reft_plan_destroy(plan)
    assert lib.sim_end() == 0


@pytest.mark.parametrize("seed", [1, 2, 3, 4])
def test_every_table_is_made_of_its_calls_pointers(lib, seed):  # noqa: F811
    rng = random.Random(seed)
    c = Rotated(lib)
    plan, known = c.plan(), {}
    for step in range(250):
        k = rng.choice((2, 3, 5))
        member, decode = rng.randrange(k), rng.random() < 0.5
        key = (k, rng.randrange(3) if rng.random() < 0.8 else 100 + step)
        x = known.setdefault(key, pointers(k, key[1] + 10 * k))
        if rng.random() < 0.3:
            which = rng.randrange(3)
            x[which][rng.randrange(len(x[which]))] += np.uint64(rng.choice((1, 16, 4096)))
        stream = rng.choice((None, None, 1, 2))
        got, _ = c.call(plan, *x, k, member, decode, stream)
        fresh = c.plan()
        want, _ = c.call(fresh, *x, k, member, decode, stream)
        lib.reft_plan_destroy(fresh)
        # a row of zeros that a plan keeps for itself stands behind the stream's end: its address is the plan's own
        inputs = np.concatenate(x)
        apart = got != want
        assert got.shape == want.shape
        assert not np.isin(got[apart] >> np.uint64(34), inputs >> np.uint64(34)).any()
        assert not np.isin(want[apart] >> np.uint64(34), inputs >> np.uint64(34)).any()
    lib.reft_plan_destroy(plan)
    assert lib.sim_end() == 0
