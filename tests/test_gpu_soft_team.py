"""The team forward of the Soft-DTW (four waves a strip, the plans of few
strips) against the one-wave sweep (a plan with a grid), where its groups of 16
steps, strips of 128 rows and band edges end: values, and gradients and row
masses of the backward on its checkpoints, bit for bit; and the values against
the oracle."""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

LENS = [1, 2, 15, 16, 17, 63, 64, 65, 130, 257, 700]


@pytest.mark.parametrize("band", [0.0, 0.3])
@pytest.mark.parametrize("L", [1, 63, 127, 128, 129, 257, 513])
def test_team_forward_is_bitwise_the_one_wave_forward(wts, L, band):
    import torch
    d = L % 8 + 1
    r = np.random.Generator(np.random.PCG64(L * 3 + 1))
    X, cyc = r.standard_normal((L, d)), [r.standard_normal((n, d)) for n in LENS]
    dtype = "f32" if L % 2 else "f64"
    cyc = [c.astype(np.float32 if dtype == "f32" else np.float64) for c in cyc]
    Y, off, _ = wts.pack_cycles(cyc, dtype=dtype)
    B = torch.from_numpy(X).cuda()
    gv = torch.from_numpy(r.uniform(0.5, 2.0, len(cyc))).cuda()
    out = []
    for grid in (0, 64):                    # 0: teams; 64 one-wave sweepers
        print("case soft team L", L, "d", d, dtype, "band", band, "grid", grid, flush=True)
        p = wts.Plan(off, d, dtype, L, band=band, grid=grid)
        v, ck = wts.softdtw_forward(p, B, Y, 0.5)
        g, h = wts.softdtw_backward(p, B, Y, 0.5, ck, gv, with_mass=True)
        gc = wts.softdtw_grad_cycles(p, B, Y, 0.5, gv)
        assert p.status() == wts.OK
        out.append([t.cpu().numpy() for t in (v, g, h, gc)])
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)
    if band == 0.0:
        ov = oracle.softdtw_batch(X, [c.astype(np.float64) for c in cyc], 0.5, grad=False)
        np.testing.assert_allclose(out[0][0], ov, rtol=1e-4)


def test_team_forward_of_several_strips_a_workgroup(wts):
    """More strips than the launch has workgroups (four a compute unit), so that
    each takes a second one with the same LDS: lengths of every remainder of a
    group of 16 steps, short strips after long ones."""
    import torch
    r = np.random.Generator(np.random.PCG64(77))
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    L, d = 300, 3
    n = 4 * cus * 2 // 3 + 40               # 3 strips each: over twice 4 a unit
    lens = r.integers(1, 260, n)
    X, cyc = r.standard_normal((L, d)), [r.standard_normal((m, d)).astype(np.float32) for m in lens]
    Y, off, _ = wts.pack_cycles(cyc, dtype="f32")
    B = torch.from_numpy(X).cuda()
    gv = torch.from_numpy(r.uniform(0.5, 2.0, n)).cuda()
    out = []
    for grid in (0, 512):
        print("case soft team of many strips n", n, "grid", grid, flush=True)
        p = wts.Plan(off, d, "f32", L, grid=grid)
        v, ck = wts.softdtw_forward(p, B, Y, 0.5)
        g, h = wts.softdtw_backward(p, B, Y, 0.5, ck, gv, with_mass=True)
        assert p.status() == wts.OK
        out.append([t.cpu().numpy() for t in (v, g, h)])
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)
    pick = list(range(0, n, 25))
    ov = oracle.softdtw_batch(X, [cyc[k].astype(np.float64) for k in pick], 0.5, grad=False)
    np.testing.assert_allclose(out[0][0][pick], ov, rtol=1e-4)
