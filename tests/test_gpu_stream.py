"""GPU parity of the ragged stream kernel at the places where it can go wrong: span boundaries near
the ends of its 16-byte chunks, its KiB steps and its units, spans shorter than a chunk, empty ones,
ranges that start and end anywhere, and streams on both sides of the size at which it changes from
cached to streaming accesses, from four waves per workgroup to one, and from 1 KiB per step to more.
Bytes: equal to the oracle or wrong."""
import numpy as np
import pytest
import torch

import oracle
import paper_2310_12670_amd as reft

pytestmark = pytest.mark.gpu
CANARY = 0x96
GUARD = 512
NAMES = ("unroll", "nontemporal", "max_wgs", "burst", "burst_min_rows", "burst_min_bytes", "small_pieces", "dma_min_bytes",
         "gather_min_pieces")


@pytest.fixture(scope="module")
def dev():
    assert torch.cuda.is_available(), "these tests need the GPU"
    d = torch.device("cuda:0")
    torch.cuda.set_device(d)
    return d


@pytest.fixture(autouse=True)
def stream_kernel_only():
    saved = {n: reft.reft_get_tunable(n) for n in NAMES}
    reft.reft_set_tunable("burst", 0)
    yield
    for n, v in saved.items():
        reft.reft_set_tunable(n, v)


def arena(sizes, phases, dev, gen):
    starts, pos = [], GUARD
    for n, ph in zip(sizes, phases):
        starts.append(pos + int(ph))
        pos += (n + int(ph) + 31) // 16 * 16
    raw = torch.randint(0, 256, (pos + GUARD,), dtype=torch.uint8, device=dev, generator=gen)
    return raw, [raw[a:a + n] for a, n in zip(starts, sizes)]


def check_all(dev, sizes, k, buckets, seed, align):
    """Encode (also with pack), decode, pack, unpack and a staged snapshot and restore that gather every byte."""
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    T, L = len(sizes), sum(sizes)

    def phases():
        return rng.integers(0, 16, T) // align * align

    held = [arena(sizes, phases(), dev, gen) for _ in range(k)]
    shards = [h[1] for h in held]
    streams = [oracle.pack([oracle.as_bytes(t.cpu()) for t in sh]) for sh in shards]
    parity = oracle.encode(streams)
    plan = reft.reft_plan_create(sizes, buckets)
    try:
        def guarded(phase):
            raw = torch.full((L + 2 * GUARD + phase,), CANARY, dtype=torch.uint8, device=dev)
            return raw, raw[GUARD + phase:GUARD + phase + L]

        def check(raw, view, want, what):
            r = raw.cpu().numpy()
            at = view.storage_offset()
            assert np.array_equal(r[at:at + L], want), what
            assert np.all(r[:at] == CANARY) and np.all(r[at + L:] == CANARY), what + ": wrote outside"

        def check_spans(raw, spans, want, what):
            r = raw.cpu().numpy()
            mask = np.ones(r.shape, bool)
            for t in spans:
                mask[t.storage_offset():t.storage_offset() + t.numel()] = False
            got = np.concatenate([r[t.storage_offset():t.storage_offset() + t.numel()] for t in spans])
            assert np.array_equal(got, want), what
            assert np.all(r[mask] == CANARY), what + ": wrote outside"

        def fresh():
            raw, spans = arena(sizes, phases(), dev, gen)
            raw.fill_(CANARY)
            return raw, spans

        phase = int(rng.integers(0, 16)) // align * align
        raw, par = guarded(phase)
        reft.reft_parity_encode(plan, [t for sh in shards for t in sh], k, par)
        check(raw, par, parity, "encode")
        own = int(rng.integers(k))
        raw, par = guarded(phase)
        raw2, packed = guarded(int(rng.integers(0, 16)) // align * align)
        reft.reft_parity_encode_pack(plan, [t for sh in shards for t in sh], k, own, par, packed)
        check(raw, par, parity, "encode with pack")
        check(raw2, packed, streams[own], "pack with encode")
        lost = int(rng.integers(k))
        raw2, outs = fresh()
        rows = [None if s == lost else t for s, sh in enumerate(shards) for t in sh]
        reft.reft_reconstruct_spans(plan, rows, k, lost, par, outs)
        check_spans(raw2, outs, streams[lost], "decode")
        raw, packed = guarded(phase)
        reft.reft_pack_device(plan, shards[0], packed)
        check(raw, packed, streams[0], "pack")
        raw2, outs = fresh()
        reft.reft_unpack_device(plan, packed, outs)
        check_spans(raw2, outs, streams[0], "unpack")
        reft.reft_set_tunable("dma_min_bytes", 1 << 62)
        reft.reft_set_tunable("gather_min_pieces", 1)
        ring = torch.empty(2 * reft.reft_plan_staging_slot_bytes(plan), dtype=torch.uint8, device=dev)
        host = torch.empty(L, dtype=torch.uint8, pin_memory=True)
        reft.reft_snapshot_pack(plan, shards[0], ring, host)
        reft.reft_snapshot_wait(plan)
        assert np.array_equal(host.numpy(), streams[0]), "staged snapshot"
        raw2, outs = fresh()
        reft.reft_restore(plan, host, ring, outs)
        reft.reft_restore_wait(plan)
        check_spans(raw2, outs, streams[0], "staged restore")
        torch.cuda.synchronize()
    finally:
        torch.cuda.synchronize()
        reft.reft_plan_destroy(plan)


def boundary_sizes(rng):
    """Spans whose boundaries fall 1 .. 17 bytes around multiples of 1 KiB, with runs of spans of 0 to
    17 bytes between them."""
    cuts = set()
    for m in range(1, 48):
        for _ in range(int(rng.integers(0, 4))):
            cuts.add(1024 * m + int(rng.integers(-17, 18)))
    at = sorted(cuts)
    sizes = list(np.diff([0] + at + [1024 * 49 + int(rng.integers(0, 1024))]))
    for _ in range(6):
        i = int(rng.integers(0, len(sizes) + 1))
        sizes[i:i] = [int(x) for x in rng.integers(0, 18, int(rng.integers(1, 90)))]
    return [int(x) for x in sizes]


@pytest.mark.parametrize("unroll,max_wgs,nt", [(1, 0, 1), (1, 2, 0), (2, 3, 1), (4, 1, 1), (4, 64, 0)])
@pytest.mark.parametrize("k", [1, 2, 5, 8, 9, 12, 15, 16, 17])
def test_boundaries(dev, k, unroll, max_wgs, nt):
    reft.reft_set_tunable("unroll", unroll)
    reft.reft_set_tunable("max_wgs", max_wgs)
    reft.reft_set_tunable("nontemporal", nt)
    rng = np.random.default_rng(1000 * k + 10 * unroll + max_wgs)
    for align in (1, 4, 16):
        sizes = boundary_sizes(rng)
        if align > 1:
            sizes = [(n + align - 1) // align * align for n in sizes]
        L, buckets = sum(sizes), []
        while L:
            buckets.append(min(L, int(rng.integers(1, 9000))))
            L -= buckets[-1]
        check_all(dev, sizes, k, buckets, seed=k * 64 + unroll * 8 + align, align=align)


# the same boundaries in a stream whose spans are longer on average, so that a unit is a KiB
@pytest.mark.parametrize("unroll,max_wgs", [(1, 0), (2, 3), (4, 1), (4, 64)])
@pytest.mark.parametrize("k", [1, 2, 4, 5, 8, 9, 16, 17])
def test_boundaries_of_spans_beside_long_ones(dev, k, unroll, max_wgs):
    reft.reft_set_tunable("unroll", unroll)
    reft.reft_set_tunable("max_wgs", max_wgs)
    rng = np.random.default_rng(31 * k + unroll + max_wgs)
    for align in (1, 4, 16):
        sizes = [(n + align - 1) // align * align for n in boundary_sizes(rng)]
        sizes.insert(int(rng.integers(0, len(sizes))), 512 * (len(sizes) + 1))
        L, buckets = sum(sizes), []
        while L:
            buckets.append(min(L, int(rng.integers(1, 50_000))))
            L -= buckets[-1]
        check_all(dev, sizes, k, buckets, seed=k * 64 + unroll * 8 + align, align=align)


def tiny_sizes(rng, n, mean):
    """n spans around the ends of 16-byte chunks and of units of 256 bytes, their mean exactly `mean`."""
    edges = [0, 1, 2, 15, 16, 17, 31, 100, 239, 240, 241, 255, 256, 257, 271, 272, 273, 511, 512, 513, 767, 768, 769]
    sizes = [int(x) for x in rng.choice(edges, n - 1)]
    short = n * mean - sum(sizes)
    return sizes + [short] if short >= 0 else tiny_sizes(rng, n, mean)


# the largest mean of streams of tiny spans and the one behind it
@pytest.mark.parametrize("mean", [511, 512])
@pytest.mark.parametrize("max_wgs", [0, 2])
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 7, 8, 9, 12, 16, 17])
def test_tiny_spans(dev, k, max_wgs, mean):
    reft.reft_set_tunable("max_wgs", max_wgs)
    rng = np.random.default_rng(37 * k + max_wgs)
    for align in (1, 16):
        sizes = tiny_sizes(rng, 333, mean)
        L, buckets = sum(sizes), []
        while L:
            buckets.append(min(L, int(rng.integers(1, 20_000))))
            L -= buckets[-1]
        check_all(dev, sizes, k, buckets, seed=k, align=align)


@pytest.mark.parametrize("k", [1, 2, 8, 16])
@pytest.mark.parametrize("max_wgs", [0, 2])
def test_tiny_spans_in_place(dev, k, max_wgs):
    """Decoded over the parity, and over a survivor: every byte is read and written once only."""
    reft.reft_set_tunable("max_wgs", max_wgs)
    rng = np.random.default_rng(90 + k)
    gen = torch.Generator(device=dev)
    gen.manual_seed(90 + k)
    sizes = tiny_sizes(rng, 501, 300)
    off = np.concatenate([[0], np.cumsum(sizes)])
    L = int(off[-1])
    plan = reft.reft_plan_create(sizes)
    try:
        for lost, over in ((0, None), (0, k - 1), (k - 1, None)):
            if over == lost:
                continue
            held = [arena(sizes, rng.integers(0, 16, len(sizes)), dev, gen) for _ in range(k)]
            streams = [oracle.pack([oracle.as_bytes(t.cpu()) for t in h[1]]) for h in held]
            raw = torch.full((L + 2 * GUARD,), CANARY, dtype=torch.uint8, device=dev)
            par = raw[GUARD + 3:GUARD + 3 + L]
            par.copy_(torch.from_numpy(oracle.encode(streams)))
            outs = [par[a:b] for a, b in zip(off[:-1], off[1:])] if over is None else held[over][1]
            rows = [None if s == lost else t for s, h in enumerate(held) for t in h[1]]
            reft.reft_reconstruct_spans(plan, rows, k, lost, par, outs)
            torch.cuda.synchronize()
            assert np.array_equal(np.concatenate([t.cpu().numpy() for t in outs]), streams[lost]), (lost, over)
            r = raw.cpu().numpy()
            assert np.all(r[:GUARD + 3] == CANARY) and np.all(r[GUARD + 3 + L:] == CANARY)
    finally:
        torch.cuda.synchronize()
        reft.reft_plan_destroy(plan)


@pytest.mark.parametrize("k", [3, 17])
def test_tiny_spans_captured(dev, k):
    """The call that allocates nothing, in a graph replayed over changed contents."""
    rng = np.random.default_rng(k)
    gen = torch.Generator(device=dev)
    gen.manual_seed(k)
    sizes = tiny_sizes(rng, 400, 400)
    held = [arena(sizes, rng.integers(0, 16, len(sizes)), dev, gen) for _ in range(k)]
    spans = [t for h in held for t in h[1]]
    out = torch.empty(sum(sizes), dtype=torch.uint8, device=dev)
    plan = reft.reft_plan_create(sizes)
    try:
        s = torch.cuda.Stream()
        torch.cuda.synchronize()
        reft.reft_parity_encode_noalloc(plan, spans, k, out, s)
        s.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            reft.reft_parity_encode_noalloc(plan, spans, k, out, torch.cuda.current_stream())
        for rep in range(3):
            held[rep][0].add_(rep + 1)
            out.zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            want = oracle.encode([oracle.pack([oracle.as_bytes(t.cpu()) for t in h[1]]) for h in held])
            assert np.array_equal(out.cpu().numpy(), want), rep
        del graph
    finally:
        torch.cuda.synchronize()
        reft.reft_plan_destroy(plan)


# one launch below and one above the traffic at which the launch changes, for every number of
# sources whose rule differs, with short and with long spans
@pytest.mark.parametrize("k", [1, 2, 3, 6, 8])
@pytest.mark.parametrize("mean", [40_000, 3_000_000])
@pytest.mark.parametrize("traffic", [80 << 20, 130 << 20])
def test_sizes_around_the_launch_rule(dev, k, mean, traffic):
    rng = np.random.default_rng(k + mean + traffic)
    L = traffic // (k + 1)
    sizes = []
    while sum(sizes) < L:
        sizes.append(int(rng.integers(mean // 2, mean * 3 // 2)) | 1)
    check_all(dev, sizes, k, None, seed=k, align=1)


# uncached launches of 32 n - 1, 32 n and 32 n + 1 units of 1 KiB (one source: of 2 KiB), and a few bytes to either side
@pytest.mark.parametrize("k", [1, 15, 16])
@pytest.mark.parametrize("units,more", [(-1, 0), (0, -5), (0, 0), (0, 9), (1, 0)])
def test_units_change_places_inside_32_kib(dev, k, units, more):
    unit = 2048 if k == 1 else 1024
    L = (128 << 20) // (k + 1) // (32 * unit) * 32 * unit + units * unit + more
    sizes = [L // 3 + 1, 70_001, 16, 33, 1 << 20]
    check_all(dev, sizes + [L - sum(sizes)], k, None, seed=k, align=1)


def test_more_spans_than_one_search_step(dev):
    """Blocks of the look-up table that own several hundred spans, and wide gaps of empty ones."""
    rng = np.random.default_rng(5)
    sizes = [int(x) for x in rng.integers(0, 3, 20000)] + [100_000] + [0] * 500 + [int(x) for x in rng.integers(0, 40, 9000)]
    check_all(dev, sizes, 3, None, seed=11, align=1)


# a grid of one or three workgroups, whose waves take up to 16 units together; 17 rows end with a pass
# that accumulates into the destination
@pytest.mark.parametrize("k", [1, 2, 4, 5, 17])
@pytest.mark.parametrize("max_wgs,align", [(1, 1), (3, 1), (1, 16)])
def test_runs_of_units(dev, k, max_wgs, align):
    reft.reft_set_tunable("max_wgs", max_wgs)
    rng = np.random.default_rng(k + 10 * max_wgs)
    sizes = boundary_sizes(rng)[:6]                    # runs need a mean of 256 KiB
    for n in [int(x) for x in rng.integers(4000, 400_000, 4)] + [0, 1, 3_000_000, 2_500_001]:
        sizes.insert(int(rng.integers(0, len(sizes) + 1)), n)
    sizes = [(n + align - 1) // align * align for n in sizes]
    L = sum(sizes)
    check_all(dev, sizes, k, [1_300_003, L - 1_300_003], seed=k, align=align)


def odd_sizes(rng):
    """Boundaries around the KiB steps, then spans of several KiB at odd stream offsets (whose units
    are moved to the sources' cache lines)."""
    return boundary_sizes(rng) + [int(x) for x in rng.integers(3000, 90000, 12)]


@pytest.mark.parametrize("burst,max_wgs", [(0, 0), (1, 0), (0, 1)])
@pytest.mark.parametrize("k", [1, 2, 5, 8, 16])
def test_decode_in_place(dev, k, burst, max_wgs):
    """The lost shard decoded over the parity it comes from, and over a survivor: every byte of the
    destination is a source, so it may be read and written once only."""
    rng = np.random.default_rng(70 + k)
    gen = torch.Generator(device=dev)
    gen.manual_seed(70 + k)
    sizes = odd_sizes(rng) if max_wgs == 0 else [int(x) for x in rng.integers(1, 700_000, 7)] + [0, 900_001, 15]
    off = np.concatenate([[0], np.cumsum(sizes)])
    L = int(off[-1])
    reft.reft_set_tunable("burst", burst)
    reft.reft_set_tunable("max_wgs", max_wgs)
    reft.reft_set_tunable("burst_min_rows", 1)
    reft.reft_set_tunable("burst_min_bytes", 0)
    reft.reft_set_tunable("small_pieces", 0xffffffff)
    plan = reft.reft_plan_create(sizes)
    try:
        for align, phase, lost, over in ((1, 5, 0, None), (16, 0, k - 1, None), (1, 3, 0, k - 1), (4, 12, 0, k // 2)):
            if over == lost:
                continue
            held = [arena(sizes, rng.integers(0, 16, len(sizes)) // align * align, dev, gen) for _ in range(k)]
            streams = [oracle.pack([oracle.as_bytes(t.cpu()) for t in h[1]]) for h in held]
            raw = torch.full((L + 2 * GUARD,), CANARY, dtype=torch.uint8, device=dev)
            par = raw[GUARD + phase:GUARD + phase + L]
            par.copy_(torch.from_numpy(oracle.encode(streams)))
            outs = [par[a:b] for a, b in zip(off[:-1], off[1:])] if over is None else held[over][1]
            rows = [None if s == lost else t for s, h in enumerate(held) for t in h[1]]
            reft.reft_reconstruct_spans(plan, rows, k, lost, par, outs)
            torch.cuda.synchronize()
            got = np.concatenate([t.cpu().numpy() for t in outs])
            assert np.array_equal(got, streams[lost]), (align, over)
            r = raw.cpu().numpy()
            assert np.all(r[:GUARD + phase] == CANARY) and np.all(r[GUARD + phase + L:] == CANARY)
    finally:
        reft.reft_plan_destroy(plan)


@pytest.mark.parametrize("k,phase", [(3, 0), (5, 7), (9, 2), (17, 5)])
def test_rotated_in_place(dev, k, phase):
    """A member's unit encoded over one of the segments it covers, and the lost shard decoded over the
    units it comes from."""
    rng = np.random.default_rng(80 + k)
    gen = torch.Generator(device=dev)
    gen.manual_seed(80 + k)
    sizes = odd_sizes(rng)
    off = np.concatenate([[0], np.cumsum(sizes)])
    L = int(off[-1])
    seg = -(-L // (k - 1))
    packed = reft.reft_plan_create([L])
    plan = reft.reft_plan_create(sizes)
    try:
        # encode: shards that are one span each, the unit of member 0 over segment 0 of the last
        shards = [arena([L + seg], [phase], dev, gen)[1][0] for _ in range(k)]
        streams = [s[:L].cpu().numpy() for s in shards]
        units = [oracle.encode_rotated(streams, i) for i in range(k)]
        reft.reft_parity_encode_rotated(packed, [s[:L] for s in shards], k, 0, shards[-1][:seg])
        torch.cuda.synchronize()
        assert np.array_equal(shards[-1][:seg].cpu().numpy(), units[0])
        # decode: the units of the other members one behind the other, the tensors in the same place
        held = [arena(sizes, rng.integers(0, 16, len(sizes)), dev, gen)[1] for _ in range(k)]
        for h, s in zip(held, streams):
            for t, a in zip(h, off[:-1]):
                t.copy_(torch.from_numpy(s[a:a + t.numel()]))
        lost = k // 2
        raw = torch.zeros((k - 1) * seg + 64, dtype=torch.uint8, device=dev)
        joined = raw[phase:phase + (k - 1) * seg]
        ptrs, r = [None] * k, 0
        for i in range(k):
            if i != lost:
                joined[r * seg:(r + 1) * seg].copy_(torch.from_numpy(units[i]))
                ptrs[i] = joined[r * seg:(r + 1) * seg]
                r += 1
        outs = [joined[a:b] for a, b in zip(off[:-1], off[1:])]
        rows = [None if s == lost else t for s, h in enumerate(held) for t in h]
        reft.reft_reconstruct_rotated(plan, rows, ptrs, k, lost, outs)
        torch.cuda.synchronize()
        assert np.array_equal(joined[:L].cpu().numpy(), streams[lost])
    finally:
        reft.reft_plan_destroy(plan)
        reft.reft_plan_destroy(packed)


def test_stream_of_more_units_than_one_launch_has_waves(dev):
    """64 GiB and more: a wave per KiB would be 2^32 work-items.  Two shards whose spans are all the
    same few tensors (only the parity has its full length), every byte compared on the device."""
    if torch.cuda.mem_get_info()[0] < 72 << 30:
        pytest.skip("needs 70 GiB of free device memory")
    gen = torch.Generator(device=dev)
    gen.manual_seed(6)
    n = (1 << 30) + 1000                     # spans begin at any place of a unit, the last unit is ragged
    count = 65
    a, b = (torch.randint(0, 256, (n,), dtype=torch.uint8, device=dev, generator=gen) for _ in range(2))
    c = torch.randint(0, 256, (n,), dtype=torch.uint8, device=dev, generator=gen)
    first = [a if i % 3 else c for i in range(count)]
    raw = torch.full((n * count + 2 * GUARD,), CANARY, dtype=torch.uint8, device=dev)
    par = raw[GUARD:GUARD + n * count]
    plan = reft.reft_plan_create([n] * count)
    try:
        reft.reft_parity_encode(plan, first + [b] * count, 2, par)
        torch.cuda.synchronize()
    finally:
        reft.reft_plan_destroy(plan)
    for i in range(count):
        assert torch.equal(par[i * n:(i + 1) * n], first[i] ^ b), i
    assert (raw[:GUARD] == CANARY).all() and (raw[GUARD + n * count:] == CANARY).all()
    del raw, par
    torch.cuda.empty_cache()
