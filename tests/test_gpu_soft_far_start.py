"""The Soft-DTW backward of a pair whose path stays in its bottom strip for the
longest cycle a plan takes (2^24 samples): the strip above waits for its first
push for more than a second, which is no reason to give up.  Bit for bit the
backward that sweeps every tile (its strips follow each other tile by tile)."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_strip_above_waits_for_a_far_first_push(wts):
    import torch
    N, L = 1 << 24, 258                      # three strips, the bottom one of two rows
    X = np.zeros((L, 1))
    X[256:] = 1.0
    Y = torch.ones((N, 1), dtype=torch.float32, device="cuda")
    Y[:300] = 0.0                            # rows 0 .. 255 align with these, the last two with the rest
    B = torch.from_numpy(X).cuda()
    off = np.array([0, N])
    got = []
    for dense in (False, True):
        print("case far first push, dense", dense, flush=True)
        plan = wts.Plan(off, 1, "f32", L, dense_e=dense)
        v, ck = wts.softdtw_forward(plan, B, Y, 1e-3)
        grad, mass = wts.softdtw_backward(plan, B, Y, 1e-3, ck, with_mass=True)
        assert plan.status() == wts.OK
        got.append((v.cpu().numpy(), grad.cpu().numpy(), mass.cpu().numpy()))
        plan.close()
        del ck
    for a, b in zip(*got):
        np.testing.assert_array_equal(a, b)
    v, grad, mass = got[0]
    assert mass[256:].sum() > N - 300 and 256 <= mass[:256].sum() < 600
