"""The two forms of the Soft-DTW backward -- a workgroup a strip and one wave a
strip -- on batches that the waves take whole (many pairs) and on batches that
the workgroups begin and hand over (wide E): gradient, row mass and swept tiles
bit for bit those of the same batch in groups of few pairs, which workgroups
take alone."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, L, d, dtype, gamma, band", [
    (1200, 257, 1, "f32", 0.05, 0.0),      # waves, narrow E: tiles passed over
    (1100, 129, 8, "f64", 2000.0, 0.4),    # waves, wide E in a band
    (700, 1500, 1, "f32", 1e6, 0.0),       # handed over: every step as likely
    (800, 1200, 3, "f64", 5000.0, 0.0),
    (700, 1400, 2, "f32", 1e6, 0.5),
    (600, 640, 6, "f32", 0.05, 0.0),       # could be handed over, and is not
])
def test_forms_of_the_backward_agree(wts, n, L, d, dtype, gamma, band):
    import torch
    r = np.random.Generator(np.random.PCG64(n + L))
    lens = r.integers(3 * L // 4, 5 * L // 4, n)
    lens[:4] = (1, 64, 65, 2 * L)
    cyc = [r.standard_normal((int(N), d)).astype(np.float32 if dtype == "f32" else np.float64)
           for N in lens]
    Y, off, _ = wts.pack_cycles(cyc, dtype=dtype)
    B = torch.from_numpy(r.standard_normal((L, d))).cuda()
    w = torch.from_numpy(r.uniform(0.5, 2.0, n)).cuda()
    print("case backward forms n", n, "L", L, "d", d, dtype, "gamma", gamma, "band", band, flush=True)

    def backward(a, b, grad, mass):
        plan = wts.Plan(off[a:b + 1] - off[a], d, dtype, L, band=band)
        y = Y[int(off[a]):int(off[b])]
        v, ck = wts.softdtw_forward(plan, B, y, gamma)
        grad, mass = wts.softdtw_backward(plan, B, y, gamma, ck, w[a:b], with_mass=True, grad=grad,
                                          mass=mass, accumulate=grad is not None)
        assert plan.status() == wts.OK
        swept = plan.bwd_tiles()
        plan.close()
        return grad, mass, swept, v

    whole = backward(0, n, None, None)
    grad = mass = None
    swept, values = np.zeros(2, np.int64), []
    for a in range(0, n, 40):
        grad, mass, t, v = backward(a, min(n, a + 40), grad, mass)
        swept += t
        values.append(v)
    assert torch.equal(whole[3], torch.cat(values))
    assert tuple(whole[2]) == tuple(swept)
    assert torch.equal(whole[0], grad) and torch.equal(whole[1], mass)
    assert bool(torch.isfinite(grad).all()) and bool((mass > 0).all())


def test_forms_of_the_cycle_gradient_agree(wts):
    import torch
    n, L, d, gamma = 1000, 150, 2, 300.0
    r = np.random.Generator(np.random.PCG64(7))
    lens = r.integers(100, 400, n)
    cyc = [r.standard_normal((int(N), d)) for N in lens]
    Y, off, dt = wts.pack_cycles(cyc)
    B = torch.from_numpy(r.standard_normal((L, d))).cuda()
    print("case backward forms, cycle gradient", flush=True)

    def grad(a, b):
        plan = wts.Plan(off[a:b + 1] - off[a], d, dt, L)
        g = wts.softdtw_grad_cycles(plan, B, Y[int(off[a]):int(off[b])], gamma)
        assert plan.status() == wts.OK
        plan.close()
        return g

    assert torch.equal(grad(0, n), torch.cat([grad(a, a + 40) for a in range(0, n, 40)]))
