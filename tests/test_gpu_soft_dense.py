"""The Soft-DTW backward that sweeps every tile (plan option dense_e = 1) on
batches of more strips than its workgroups-per-strip form takes: bit for bit
the default's gradient and row mass, and every tile counted as swept."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def strips(L, n):
    return n * -(-L // 128)


@pytest.mark.parametrize("L, n, d, dtype, band", [
    (129, 1300, 1, np.float32, 0.0),     # two strips, the second of one row
    (385, 700, 3, np.float64, 0.0),
    (300, 900, 8, np.float32, 0.3),
])
def test_dense_backward_of_many_strips_is_bitwise_the_default(wts, L, n, d, dtype, band):
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    n = max(n, 10 * cus // -(-L // 128) + 1)
    assert strips(L, n) > 10 * cus
    print("case dense backward: n %d, L %d, d %d, band %g" % (n, L, d, band), flush=True)
    rng = np.random.Generator(np.random.PCG64(L + n))
    lens = rng.integers(L // 2, 3 * L // 2, n)
    lens[:3] = (1, 64, 65)
    cyc = [rng.standard_normal((int(N), d)).astype(dtype) for N in lens]
    B = torch.from_numpy(rng.standard_normal((L, d))).cuda()
    Y, off, dt = wts.pack_cycles(cyc)
    out, tiles = [], []
    for dense in (False, True):
        plan = wts.Plan(off, d, dt, L, band=band, dense_e=dense)
        _, ck = wts.softdtw_forward(plan, B, Y, 1.0)
        grad, mass = wts.softdtw_backward(plan, B, Y, 1.0, ck, with_mass=True)
        torch.cuda.synchronize()
        plan.check()
        out.append((grad.cpu().numpy(), mass.cpu().numpy()))
        tiles.append(plan.bwd_tiles())
        plan.close()
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
    assert np.isfinite(out[1][0]).all() and (out[1][1] > 0).all()
    assert tiles[1][0] == tiles[1][1] > 0
    if band == 0.0:   # every 16-step tile of every strip
        assert tiles[1][1] == sum((int(N) + 63 + 15) // 16 for N in lens) * -(-L // 128)
