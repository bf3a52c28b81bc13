"""Staged snapshots and restores that share a ring of slots, queued without a host wait between them: calls on one stream, which
leave no events behind the slots, before and after calls on others; and calls of about 4 MiB, up to which one stream's bytes
go across the link by a kernel.  Bytes: equal to the tensors' or wrong."""
import itertools

import pytest
import torch

import paper_2310_12670_amd as reft

pytestmark = pytest.mark.gpu
ROUNDS = 4


@pytest.fixture(scope="module")
def streams():
    assert torch.cuda.is_available(), "these tests need the GPU"
    torch.cuda.set_device(0)
    return [None, torch.cuda.Stream(), torch.cuda.Stream()]


def spans(sizes, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return [torch.randint(0, 256, (n,), dtype=torch.uint8, device="cuda", generator=gen) for n in sizes]


# small spans alone, with slots for one run or for several, and beside a span that is copied for itself
@pytest.mark.parametrize("slots", [1, 2, 5])
@pytest.mark.parametrize("large", [0, 5 << 20])
def test_calls_that_share_a_ring(streams, slots, large):
    sizes = [33_333] * 180 + ([large] if large else []) + [7_001] * 300
    plan = reft.reft_plan_create(sizes, None, 2 << 20)
    try:
        ring = torch.empty(slots * reft.reft_plan_staging_slot_bytes(plan), dtype=torch.uint8, device="cuda")
        pairs = list(itertools.product(range(3), range(3)))
        for first in range(0, len(pairs), 3):
            # each of these after each of the others, one stream and two
            calls = [pairs[(first + i * step) % len(pairs)] for step in (1, 2, 4) for i in range(ROUNDS)]
            sets = [spans(sizes, i) for i in range(len(calls))]
            hosts = [torch.zeros(sum(sizes), dtype=torch.uint8, pin_memory=True) for _ in calls]
            torch.cuda.synchronize()
            for (a, b), tensors, host in zip(calls, sets, hosts):
                reft.reft_snapshot_pack(plan, tensors, ring, host, streams[a], streams[b])
            reft.reft_snapshot_wait(plan)
            torch.cuda.synchronize()
            for call, tensors, host in zip(calls, sets, hosts):
                assert torch.equal(host, torch.cat(tensors).cpu()), ("snapshot", call)
            outs = [[torch.zeros_like(t) for t in tensors] for tensors in sets]
            torch.cuda.synchronize()
            for (a, b), host, out in zip(calls, hosts, outs):
                reft.reft_restore(plan, host, ring, out, streams[a], streams[b])
            torch.cuda.synchronize()
            for call, tensors, out in zip(calls, sets, outs):
                assert torch.equal(torch.cat(tensors), torch.cat(out)), ("restore", call)
    finally:
        torch.cuda.synchronize()
        reft.reft_plan_destroy(plan)


@pytest.mark.parametrize("total", [(4 << 20) - 1, 4 << 20, (4 << 20) + 1])
@pytest.mark.parametrize("mean", [300, 9_999, 700_000])
@pytest.mark.parametrize("stream", [0, 1])
@pytest.mark.parametrize("pinned", [True, False])
def test_short_streams(streams, total, mean, stream, pinned):
    """On one stream, all buckets and a range of them; ordinary host memory, which a kernel cannot see, as before."""
    sizes = [mean + 7 * (i % 5) for i in range(total // (mean + 14) - 1)]
    sizes.append(total - sum(sizes))
    s = streams[stream]
    plan = reft.reft_plan_create(sizes, None, 1 << 20)
    try:
        ring = torch.empty(2 * reft.reft_plan_staging_slot_bytes(plan), dtype=torch.uint8, device="cuda")
        tensors = spans(sizes, mean)
        want = torch.cat(tensors).cpu()
        raw = torch.full((total + 512,), 0x5A, dtype=torch.uint8, pin_memory=pinned)
        host = raw[255:255 + total]
        torch.cuda.synchronize()
        reft.reft_snapshot_pack(plan, tensors, ring, host, s, s)
        reft.reft_snapshot_wait(plan)
        assert torch.equal(host, want) and bool((raw[:255] == 0x5A).all()) and bool((raw[255 + total:] == 0x5A).all())
        out = [torch.zeros_like(t) for t in tensors]
        torch.cuda.synchronize()
        reft.reft_restore(plan, host, ring, out, s, s)
        reft.reft_restore_wait(plan)
        assert torch.equal(torch.cat(out).cpu(), want)
        raw.fill_(0x5A)
        reft.reft_snapshot_pack_range(plan, tensors, ring, host, 1, 3, s, s)
        reft.reft_snapshot_wait(plan)
        lo, hi = reft.reft_plan_bucket_range(plan, 1)[0], reft.reft_plan_bucket_range(plan, 2)[1]
        assert torch.equal(host[lo:hi], want[lo:hi])
        assert bool((host[:lo] == 0x5A).all()) and bool((host[hi:] == 0x5A).all())
    finally:
        torch.cuda.synchronize()
        reft.reft_plan_destroy(plan)
