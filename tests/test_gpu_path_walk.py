"""The path walk at the sizes where its windows and tiles end: runs to the left
longer than a window (64 columns) and longer than the tiles swept again at
once (512 steps), pairs much longer or shorter than the barycenter, single
rows and columns, for both path recoveries; bit for bit the oracle's paths,
counts and means."""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def steps(lens, levels):
    """A staircase: level k held for lens[k] samples."""
    return np.repeat(np.asarray(levels, np.float64), lens)[:, None]


def case(name):
    r = np.random.Generator(np.random.PCG64(41))
    if name == "long runs":       # one row holds 700 and more columns, another 63 .. 65
        X = steps([1, 1, 3, 1, 64], [0, 5, 9, 2, 7])
        return X, [steps([700, 63, 64, 65, 1300], [0, 5, 9, 2, 7]), steps([1, 1, 1, 1, 1], [0, 5, 9, 2, 7])]
    if name == "steep":           # far more rows than columns, and the reverse
        return r.standard_normal((1500, 3)), [r.standard_normal((n, 3)) for n in (1, 2, 40, 63, 64, 65)]
    if name == "flat":
        return r.standard_normal((66, 3)), [r.standard_normal((n, 3)) for n in (513, 2100, 64)]
    if name == "constant":        # zero cost everywhere: ties at every cell
        return np.zeros((321, 1)), [np.zeros((n, 1)) for n in (321, 640, 100)]
    return r.integers(0, 2, (1, 2)).astype(np.float64), [r.integers(0, 2, (n, 2)).astype(np.float64)
                                                         for n in (1, 64, 577)]


@pytest.mark.parametrize("walk", ["strips", "pairs"])
@pytest.mark.parametrize("rho", [2, 4, 5])
@pytest.mark.parametrize("name", ["long runs", "steep", "flat", "constant", "one row"])
def test_walk_windows(wts, name, rho, walk):
    import torch
    X, cyc = case(name)
    Y, off, dt = wts.pack_cycles(cyc)
    plan = wts.Plan(off, X.shape[1], dt, X.shape[0], rho=rho, walk=walk)
    print("case path walk", name, "rho", rho, walk, flush=True)
    B = torch.from_numpy(X).cuda()
    _, plen, paths = wts.dtw_align(plan, B, Y, paths=True)
    Bo, counts, dist = wts.dba_iterate(plan, B, Y)
    assert plan.status() == wts.OK
    Bn, K, od, _ = oracle.dba_iterate(X, cyc)
    np.testing.assert_array_equal(dist.cpu().numpy(), od)
    np.testing.assert_array_equal(counts.cpu().numpy(), K)
    np.testing.assert_array_equal(Bo.cpu().numpy(), Bn)
    for k, c in enumerate(cyc):
        np.testing.assert_array_equal(wts.path_of(plan, paths, plen, k), oracle.dtw(X, c)[2])
