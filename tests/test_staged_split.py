"""How a staged snapshot splits into gathered runs and copies: reft_plan_staged_work against the rule
stated in plain Python (a span of at least dma_min bytes is one copy, runs of at least gather_min
pieces of smaller ones within a bucket are gathered, shorter ones copied piece by piece)."""
import numpy as np
import pytest

import paper_2310_12670_amd as reft


def split(sizes, bucket, dma_min, gather_min):
    gathers = copies = pending = at = 0
    last = -1
    for n in sizes:
        if n == 0:
            continue
        if n >= dma_min:
            gathers, copies, pending = gathers + (pending >= gather_min), copies + (pending if pending < gather_min else 1), 0
            copies += 1
        else:
            for b in range(at // bucket, (at + n - 1) // bucket + 1):
                if b != last and pending:
                    gathers, copies, pending = gathers + (pending >= gather_min), copies + (pending if pending < gather_min else 1), 0
                last = b
                pending += 1
        at += n
    gathers, copies = gathers + (pending >= gather_min), copies + (pending if pending < gather_min else 1)
    return gathers, copies


@pytest.mark.parametrize("bucket", [1000, 4096, 1 << 20, 1 << 30])
@pytest.mark.parametrize("dma_min,gather_min", [(0, 8), (1, 1), (3000, 8), (1 << 20, 8), (1 << 20, 2), (1 << 62, 1)])
def test_rule(bucket, dma_min, gather_min):
    saved = {n: reft.reft_get_tunable(n) for n in ("host_only_plans", "dma_min_bytes", "gather_min_pieces")}
    try:
        reft.reft_set_tunable("host_only_plans", 1)
        reft.reft_set_tunable("dma_min_bytes", dma_min)
        reft.reft_set_tunable("gather_min_pieces", gather_min)
        rng = np.random.default_rng(bucket + gather_min)
        for mean in (40, 900, 20000, 700000):
            sizes = [int(x) for x in rng.exponential(mean, 60)]
            if sum(sizes) // bucket > 50000:
                continue
            for i in rng.integers(0, 60, 6):
                sizes[int(i)] = 0
            sizes[0] += 1
            plan = reft.reft_plan_create(sizes, None, bucket)
            try:
                assert reft.reft_plan_staged_work(plan) == split(sizes, bucket, dma_min, gather_min)
            finally:
                reft.reft_plan_destroy(plan)
    finally:
        for n, v in saved.items():
            reft.reft_set_tunable(n, v)
