"""Path lengths of pairs whose cost overflows to +inf: where all three
predecessors of a cell are +inf the diagonal is taken (the first of equals), off
the grid too, and the length counts the cells inside it.  Teams and one-wave
sweeps of every row count, over strips and lanes, against a plain evaluation of
that rule."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def lengths(X, Y):
    """(distance, path length) of one pair, cell by cell in the type of X and Y."""
    M, N = len(X), len(Y)
    inf = X.dtype.type(np.inf)
    r = np.full((M + 1, N + 1), inf, X.dtype)
    n = np.zeros((M + 1, N + 1), np.int64)
    r[0, 0] = 0
    with np.errstate(over="ignore"):
        cost = ((X[:, None, 0] - Y[None, :, 0]) ** 2).astype(X.dtype)
        for i in range(M):
            for j in range(N):
                dg, up, lf = r[i, j], r[i, j + 1], r[i + 1, j]
                m = min(dg, up, lf)
                k = (i, j) if dg == m else (i, j + 1) if up == m else (i + 1, j)
                r[i + 1, j + 1] = cost[i, j] + m
                n[i + 1, j + 1] = n[k] + 1
    return r[M, N], n[M, N]


@pytest.mark.parametrize("decision,big", [("fp64", 1e200), ("fp32", 1e25)])
@pytest.mark.parametrize("L", [1, 70, 300])
def test_path_lengths_of_overflowing_pairs(wts, L, decision, big):
    import torch
    r = np.random.Generator(np.random.PCG64(L))
    X = r.standard_normal((L, 1))
    cyc = [r.standard_normal((n, 1)) for n in (1, 40, 40, 90, 90, 90)]
    cyc[1][0] = cyc[2][-1] = cyc[3][45] = big      # one sample
    cyc[4][:] = cyc[5][30:] = big                  # all, and from the middle on
    t = np.float64 if decision == "fp64" else np.float32
    cyc = [c.astype(t) for c in cyc]
    want = [lengths(X.astype(t), c) for c in cyc]
    Y, off, dt = wts.pack_cycles(cyc)
    B = torch.from_numpy(X).cuda()
    for rho, grid in ((2, 0), (4, 0), (2, 64), (4, 64), (5, 0)):   # teams, then one wave a strip
        print("case overflow L", L, decision, "rho", rho, "grid", grid, flush=True)
        plan = wts.Plan(off, 1, dt, L, rho=rho, grid=grid, decision=decision)
        _, dist, plen = wts.anomaly_score(plan, B, Y)
        adist, aplen, _ = wts.dtw_align(plan, B, Y)
        assert plan.status() == wts.OK
        for d, n in ((dist, plen), (adist, aplen)):
            np.testing.assert_array_equal(d.cpu().numpy(), [float(w[0]) for w in want])
            np.testing.assert_array_equal(n.cpu().numpy(), [w[1] for w in want])
