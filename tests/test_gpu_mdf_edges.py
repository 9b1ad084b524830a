"""Multi-direct forcing at the edges of its marker groups (28 a workgroup) and of the places its maxima are kept in:
FIXED calls equal the plain composition of interpolation and spreading bit for bit."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import as_dtype, gpu_tree, to_dev

pytestmark = pytest.mark.gpu

SHELL = synth.Sphere((0.5, 0.45, 0.55), 0.12)


@pytest.mark.parametrize("periodic", [True, False])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("n", [1, 2, 3, 27, 28, 29, 56, 57, 153, 5000, 70_001])
def test_mdf_equals_plain_composition(n, dtype, periodic):
    spec = synth.band_tree(3, 6, [SHELL], periodic=periodic, seed=2)
    t = gpu_tree(spec)
    rng = np.random.default_rng(n)
    P = np.array([0.5, 0.45, 0.55]) + 0.05 * rng.standard_normal((n, 3))
    P[::11] = P[0]                      # markers on one place
    P[5::29] = P[5::29] * 0.0 + 0.001   # next to the walls
    pos, tgt = (to_dev(as_dtype(a, dtype), dtype) for a in (P, rng.standard_normal((n, 3))))
    u0 = to_dev(as_dtype(rng.standard_normal((spec.n_leaves, 3)), dtype), dtype)
    dt, rho, iters = 0.5, 1.0, 3        # powers of two: the quotients are exact
    u, fl, fe = u0.clone(), torch.zeros_like(pos), torch.zeros_like(u0)
    for _ in range(iters):
        F = (tgt - t.interpolate(u, pos)) / dt
        f = t.spread(F, pos, mode="fixed")
        u, fl, fe = u + f / rho, fl + F, fe + f
    ug, flg, feg = t.mdf(u0, pos, tgt, iters, dt, rho, mode="fixed")
    assert torch.equal(ug, u) and torch.equal(flg, fl) and torch.equal(feg, fe)
