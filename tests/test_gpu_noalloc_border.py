"""Batches whose score workspace fits the non-allocating entry point's scratch
with more rows a lane than their plan's sweeps take, or just with those: accepted,
and bit for bit the allocating call."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, L, N, rho", [(14, 17560, 3000, 5), (83, 3072, 3000, 4),
                                          (170, 1280, 3900, 4), (32, 5000, 4000, 2)])
def test_noalloc_takes_batches_at_the_border(wts, n, L, N, rho):
    import torch
    d = 3
    print("case no-alloc border n", n, "L", L, flush=True)
    g = torch.Generator(device="cuda").manual_seed(n)
    Y = torch.randn((n * N, d), generator=g, device="cuda")
    B = torch.randn((L, d), generator=g, device="cuda", dtype=torch.float64)
    plan = wts.Plan(np.arange(n + 1) * N, d, "f32", L)
    assert plan.rho(wts.OP_SCORE) == rho
    assert (plan.workspace_bytes(wts.OP_SCORE) > 32 << 20) == (rho < 5)
    want = wts.anomaly_score(plan, B, Y)
    dist = torch.empty(n, dtype=torch.float64, device="cuda")
    plen = torch.empty(n, dtype=torch.int64, device="cuda")
    got = wts.anomaly_score_noalloc(plan, B, Y, dist=dist, path_len=plen)
    assert plan.status() == wts.OK
    for a, b in zip(want, got):
        assert torch.equal(a, b)
