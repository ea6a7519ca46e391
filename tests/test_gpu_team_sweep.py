"""The team sweep (four waves a strip, the plans of few strips) against the
one-wave sweep (a plan with a grid) and the oracle, where its groups of 16
steps, strips of 128 or 256 rows and lane edges end: values, path lengths,
paths, Sub-DTW and the medoid's matrix, bit for bit."""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

LENS = [1, 2, 15, 16, 17, 63, 64, 65, 130, 257, 700]


def plans(wts, off, d, dt, L, **kw):
    auto = wts.Plan(off, d, dt, L, **kw)
    assert L == 0 or auto.rho(wts.OP_SCORE) == 2     # few strips: swept by teams
    return {"team": auto, "team 4": wts.Plan(off, d, dt, L, rho=4, **kw),
            "one wave": wts.Plan(off, d, dt, L, rho=4, grid=64, **kw)}


@pytest.mark.parametrize("dtype,decision", [("f64", "fp64"), ("f32", "fp64"), ("f32", "fp32")])
@pytest.mark.parametrize("L", [1, 63, 127, 128, 129, 257, 513])
def test_team_and_one_wave_sweeps_agree(wts, L, dtype, decision):
    import torch
    d = L % 8 + 1
    r = np.random.Generator(np.random.PCG64(L * 7 + len(dtype)))
    ints = L % 2 == 0                                # ties decide the paths
    draw = (lambda n: r.integers(0, 3, (n, d)).astype(np.float64)) if ints else (
        lambda n: r.standard_normal((n, d)))
    X, cyc = draw(L), [draw(n).astype(np.float32 if dtype == "f32" else np.float64) for n in LENS]
    Y, off, _ = wts.pack_cycles(cyc, dtype=dtype)
    B = torch.from_numpy(X).cuda()
    print("case team sweep", L, d, dtype, decision, flush=True)
    ref = None
    for name, p in plans(wts, off, d, dtype, L, decision=decision).items():
        score = wts.anomaly_score(p, B, Y)
        dist, plen, paths = wts.dtw_align(p, B, Y, paths=True)
        out = [*score, dist, plen, *wts.subdtw(p, B, Y), *wts.dba_iterate(p, B, Y)]
        out = [t.cpu().numpy() for t in out] + [wts.path_of(p, paths, plen, k) for k in range(len(LENS))]
        assert p.status() == wts.OK
        ref = out if ref is None else ref
        for a, b in zip(ref, out):
            np.testing.assert_array_equal(a, b, err_msg=name)
    if decision == "fp64":
        os_, od, ol = oracle.score_batch(X, [c.astype(np.float64) for c in cyc])
        np.testing.assert_array_equal(ref[0], os_)
        np.testing.assert_array_equal(ref[1], od)
        np.testing.assert_array_equal(ref[2], ol)


def test_team_euclidean_scores_and_medoid(wts):
    import torch
    r = np.random.Generator(np.random.PCG64(3))
    cyc = [r.standard_normal((n, 5)) for n in LENS[4:]]
    Y, off, dt = wts.pack_cycles(cyc)
    B = torch.from_numpy(r.standard_normal((300, 5))).cuda()
    print("case team sweep l2 scores, medoid", flush=True)
    got = [[t.cpu().numpy() for t in wts.anomaly_score(p, B, Y)]
           for p in plans(wts, off, 5, dt, 300, cost="euclid").values()]
    med = [[t.cpu().numpy() for t in wts.medoid(p, Y)] for p in plans(wts, off, 5, dt, 0).values()]
    for case in (got, med):
        for other in case[1:]:
            for a, b in zip(case[0], other):
                np.testing.assert_array_equal(a, b)
    np.testing.assert_array_equal(med[0][1], oracle.medoid(cyc)[1])
