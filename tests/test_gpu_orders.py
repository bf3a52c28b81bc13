"""GPU parity of launches that deal their units in another order than the stream's (more traffic than the cache holds, spans of
20 KiB and more on average): spans of about the units that are turned, odd sizes and such as the tensors' alignment, every
call over span tables, and windows of other members' streams.  Bytes: equal to the oracle or wrong."""
import numpy as np
import pytest
import torch

import paper_2310_12670_amd as reft
from test_gpu_rotated import check_rotated
from test_gpu_stream import arena, check_all, dev, stream_kernel_only  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu
TRAFFIC = 110 << 20
# where units are not turned (but for pairs of waves and odd copies of short spans), and where they are
BOTH = pytest.mark.parametrize("traffic", [TRAFFIC, 520 << 20])


def sizes_of(kib, total, odd, seed):
    """Spans of a few bytes to either side of 31 to 35 KiB and of 63 to 66, or of `kib` KiB on average, a few small ones between."""
    rng = np.random.default_rng(seed)
    sizes = []
    while sum(sizes) < total:
        if kib == 0:
            sizes.append(int(rng.choice([31, 32, 33, 34, 35, 63, 64, 65, 66])) * 1024 + (int(rng.integers(-17, 18)) if odd else 0))
        else:
            n = int(rng.integers(kib * 512, kib * 1536))
            sizes.append(n | 1 if odd else n // 512 * 512)
        if len(sizes) % 50 == 0:
            sizes += [0, 5 if odd else 512]
    return sizes


@pytest.mark.parametrize("odd", [True, False])
@pytest.mark.parametrize("kib", [0, 21, 70])
@pytest.mark.parametrize("k", [1, 2, 3, 5, 8, 9, 13, 16])
@BOTH
def test_every_call(dev, traffic, k, kib, odd):  # noqa: F811
    check_all(dev, sizes_of(kib, traffic // (k + 1), odd, k), k, None, seed=k + kib, align=1 if odd else 16)


@pytest.mark.parametrize("odd", [True, False])
@pytest.mark.parametrize("k", [3, 8, 14, 16])
@BOTH
def test_windows(dev, traffic, k, odd):  # noqa: F811
    gen = torch.Generator(device=dev)
    gen.manual_seed(k)
    # the decode's k - 1 rows and result are what leaves the cache, the unit's k - 1 windows are a part of that
    sizes = sizes_of(300, traffic // k, odd, k)
    shards = [arena(sizes, [0] * len(sizes), dev, gen)[1] for _ in range(k)]
    check_rotated(dev, shards, sizes, losts=[0, k - 1])


@pytest.mark.parametrize("odd", [True, False])
@pytest.mark.parametrize("k", [2, 3, 4, 9])
@BOTH
def test_in_place(dev, traffic, k, odd):  # noqa: F811
    """The lost shard decoded over the parity: every byte read and written once."""
    sizes = sizes_of(70, traffic // (k + 1), odd, k)
    off = np.concatenate([[0], np.cumsum(sizes)]).tolist()
    gen = torch.Generator(device=dev)
    gen.manual_seed(k)
    shards = [arena(sizes, [0] * len(sizes), dev, gen)[1] for _ in range(k)]
    plan = reft.reft_plan_create(sizes)
    try:
        par = torch.empty(off[-1], dtype=torch.uint8, device=dev)
        reft.reft_parity_encode(plan, [t for sh in shards for t in sh], k, par)
        rows = [None if s == 1 else t for s, sh in enumerate(shards) for t in sh]
        reft.reft_reconstruct_spans(plan, rows, k, 1, par, [par[a:b] for a, b in zip(off, off[1:])])
        torch.cuda.synchronize()
        assert torch.equal(par, torch.cat(shards[1]))
    finally:
        reft.reft_plan_destroy(plan)


# more than 512 MiB of traffic, spans of 128 KiB (1 MiB with up to four sources) and more on average at multiples of 64 bytes in
# the stream, in memory at such and anywhere; of 24 shards eight (in the parity and in the decode) are added in a second pass
@pytest.mark.parametrize("align", [1, 64])
@pytest.mark.parametrize("k", [2, 3, 4, 5, 7, 8, 11, 16, 24])
def test_results_written_through(dev, k, align):  # noqa: F811
    rng = np.random.default_rng(k)
    sizes, total = [], (520 << 20) // (k + 1 if k <= 16 else k - 16 + 2)
    least = 1 << 20 if k <= 4 else 128 << 10
    while sum(sizes) < total:
        sizes.append(int(rng.integers(1, least // 16)) * 64)
        if len(sizes) % 9 == 0:
            sizes += [64, 0, 192]
    sizes += [int(rng.integers(1, 64)) for _ in range(4)]
    gen = torch.Generator(device=dev)
    gen.manual_seed(k)
    T, L = len(sizes), sum(sizes)
    assert L // T >= least

    def spans():
        return arena(sizes, rng.integers(0, 64, T) // align * align, dev, gen)

    shards = [spans()[1] for _ in range(k)]
    streams = [torch.cat(sh) for sh in shards]
    want = streams[0].clone()
    for st in streams[1:]:
        want ^= st
    plan = reft.reft_plan_create(sizes)
    try:
        flat = [t for sh in shards for t in sh]

        def guarded():
            raw = torch.full((L + 512,), 0x96, dtype=torch.uint8, device=dev)
            at = 256 + int(rng.integers(0, 64)) // align * align
            return raw, raw[at:at + L]

        def check(raw, view, expected):
            at = view.storage_offset()
            assert torch.equal(view, expected)
            assert bool((raw[:at] == 0x96).all()) and bool((raw[at + L:] == 0x96).all())

        raw, par = guarded()
        reft.reft_parity_encode(plan, flat, k, par)
        check(raw, par, want)
        raw2, packed = guarded()
        raw, par = guarded()
        reft.reft_parity_encode_pack(plan, flat, k, k - 1, par, packed)
        check(raw, par, want)
        check(raw2, packed, streams[k - 1])
        raw2, outs = spans()
        raw2.fill_(0x96)
        before = raw2.clone()
        rows = [None if s == 1 else t for s, sh in enumerate(shards) for t in sh]
        reft.reft_reconstruct_spans(plan, rows, k, 1, par, outs)
        assert torch.equal(torch.cat(outs), streams[1])
        for t in outs:
            t.fill_(0x96)
        assert torch.equal(raw2, before)
    finally:
        torch.cuda.synchronize()
        reft.reft_plan_destroy(plan)


@pytest.mark.parametrize("align", [1, 64])
def test_copies_written_through(dev, align):  # noqa: F811
    """Packed and unpacked, 1 GiB in spans of 4 MiB and more on average: whole steps of two units, and what is left of a span."""
    rng = np.random.default_rng(align)
    sizes = []
    while sum(sizes) < 1 << 30:
        sizes.append(int(rng.integers(1, 320 << 10)) * 64)
        if len(sizes) % 20 == 0:
            sizes += [0, 64]
    sizes.append(5)
    gen = torch.Generator(device=dev)
    gen.manual_seed(align)
    T, L = len(sizes), sum(sizes)
    assert L // T >= 4 << 20 and 2 * L >= 2 << 30
    shard = arena(sizes, rng.integers(0, 64, T) // align * align, dev, gen)[1]
    want = torch.cat(shard)
    plan = reft.reft_plan_create(sizes)
    try:
        raw = torch.full((L + 512,), 0x96, dtype=torch.uint8, device=dev)
        at = 256 + int(rng.integers(0, 64)) // align * align
        packed = raw[at:at + L]
        reft.reft_pack_device(plan, shard, packed)
        assert torch.equal(packed, want)
        assert bool((raw[:at] == 0x96).all()) and bool((raw[at + L:] == 0x96).all())
        raw2, outs = arena(sizes, rng.integers(0, 64, T) // align * align, dev, gen)
        raw2.fill_(0x96)
        reft.reft_unpack_device(plan, packed, outs)
        assert torch.equal(torch.cat(outs), want)
        for t in outs:
            t.fill_(0x96)
        assert bool((raw2 == 0x96).all())
    finally:
        torch.cuda.synchronize()
        reft.reft_plan_destroy(plan)


@pytest.mark.parametrize("k", [4, 7, 11, 12, 16])
@pytest.mark.parametrize("mean", [3000, 8000, 15_000])
def test_pairs_of_waves_in_short_spans(dev, k, mean):  # noqa: F811
    """More traffic than the cache holds in odd spans of less than 20 KiB on average: two waves a workgroup, in order."""
    rng = np.random.default_rng(k * mean)
    sizes = []
    while sum(sizes) < TRAFFIC // (k + 1):
        sizes.append(int(rng.integers(0, 2 * mean)) | 1)
    check_all(dev, sizes, k, None, seed=k, align=1)


# a gathered run long enough for its launch to be spread, which ends with a span in front of the stream's end: because a span
# that is copied follows, or because a bucket ends there
@pytest.mark.parametrize("two", [False, True])
@pytest.mark.parametrize("buckets", [False, True])
@pytest.mark.parametrize("size", [70_001, 300_001, 1_500_000])
def test_runs_that_end_with_a_span(dev, size, buckets, two):  # noqa: F811
    n = (56 << 20) // size
    sizes = [size] * n + ([size] * n + [5, 9 << 20] if buckets else [9 << 20, 5] + [size] * 9)
    rng = np.random.default_rng(size)
    gen = torch.Generator(device=dev)
    gen.manual_seed(size)
    T, L = len(sizes), sum(sizes)
    lists = [size * n, size * n, 5 + (9 << 20)] if buckets else [L]
    plan = reft.reft_plan_create(sizes, lists)
    try:
        a = torch.cuda.Stream()
        b = torch.cuda.Stream() if two else a
        ring = torch.empty(2 * reft.reft_plan_staging_slot_bytes(plan) + 256, dtype=torch.uint8, device=dev)[256:]
        _, tensors = arena(sizes, rng.integers(0, 512, T), dev, gen)
        want = torch.cat(tensors).cpu()
        host = torch.zeros(L, dtype=torch.uint8, pin_memory=True)
        for lo in range(len(lists)):
            host.fill_(0x33)
            ring.fill_(0x96)
            torch.cuda.synchronize()
            reft.reft_snapshot_pack_range(plan, tensors, ring, host, lo, len(lists), a, b)
            reft.reft_snapshot_wait(plan)
            begin = sum(lists[:lo])
            assert torch.equal(host[begin:], want[begin:]) and bool((host[:begin] == 0x33).all()), lo
        host.copy_(want)
        for align in (1, 512):
            raw, outs = arena(sizes, rng.integers(0, 512, T) // align * align, dev, gen)
            raw.fill_(0x96)
            ring.fill_(0x33)
            torch.cuda.synchronize()
            reft.reft_restore(plan, host, ring, outs, a, b)
            reft.reft_restore_wait(plan)
            assert torch.equal(torch.cat(outs).cpu(), want), align
            for t in outs:
                t.fill_(0x96)
            assert bool((raw == 0x96).all())
    finally:
        torch.cuda.synchronize()
        reft.reft_plan_destroy(plan)
