"""The DBA update at the sizes where its workgroups' rows and cycles end (1 row
and 256 cycles up to 512 rows, 4 and 64 above) and with runs of 1 to some tens
of columns a row: means and counts bit for bit the oracle's, with and without
weights."""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, L, N, d", [
    (257, 1, 9, 1), (513, 3, 70, 2), (300, 16, 400, 3), (65, 511, 300, 8), (64, 512, 700, 1),
    (66, 513, 2000, 4), (129, 515, 130, 6), (3, 1026, 1500, 5),
])
def test_fold_matches_the_oracle(wts, n, L, N, d):
    import torch
    r = np.random.Generator(np.random.PCG64(n + L))
    cyc = [r.standard_normal((int(k), d)).astype(np.float32) for k in r.integers(max(1, N // 2), 2 * N, n)]
    cyc[-1] = cyc[-1][:1]
    X = r.standard_normal((L, d))
    w = r.uniform(0.1, 3.0, n)
    Y, off, dt = wts.pack_cycles(cyc)
    B = torch.from_numpy(X).cuda()
    plan = wts.Plan(off, d, dt, L)
    print("case fold n", n, "L", L, "N", N, "d", d, flush=True)
    for weights in (None, w):
        wt = None if weights is None else torch.from_numpy(weights).cuda()
        Bo, counts, dist = wts.dba_iterate(plan, B, Y, weights=wt)
        assert plan.status() == wts.OK
        want = oracle.dba_iterate(X, [c.astype(np.float64) for c in cyc], weights)
        np.testing.assert_array_equal(counts.cpu().numpy(), want[1])
        np.testing.assert_array_equal(dist.cpu().numpy(), want[2])
        np.testing.assert_array_equal(Bo.cpu().numpy(), want[0])
