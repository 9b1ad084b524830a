"""The node-parallel pass of small plain calls against the per-point pass
(unsorted plans): ids, velocities, gradients and fixed-point spreading bit for
bit, atomic spreading within the oracle bound; whole and partial workgroups of
28 points and waves of 7, dense and sparse sets, walls, given host ids, points
without a host, forces that are not finite."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import as_dtype, gpu_tree, oracle_tree, spread_excess, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ot():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2605_20565_amd as m
    return m


@pytest.fixture(scope="module", params=[True, False])
def tree(request):
    spec = synth.band_tree(2, 7, [synth.Sphere((0.5, 0.45, 0.55), 0.2)], periodic=request.param, seed=2)
    return spec, oracle_tree(spec), gpu_tree(spec)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("n", [1, 6, 7, 8, 27, 28, 29, 1001, 16384])
def test_small_calls_equal_per_point_pass(ot, tree, dtype, n):
    spec, o, t = tree
    rng = np.random.default_rng(n)
    P = rng.random((n, 3))
    if n > 100:
        P[: n // 2] = 0.5 + 0.01 * rng.random((n // 2, 3))   # many points per host
        P[-4:] = [[np.nan, 0.5, 0.5], [-0.25, 0.5, 0.5], [1.5, 0.1, 0.1], [0.0, 0.0, 0.0]]
    P = as_dtype(P, dtype)
    X, F = to_dev(P, dtype), to_dev(rng.standard_normal((n, 3)), dtype)
    U = to_dev(rng.standard_normal((spec.n_leaves, 3)), dtype)

    def per_point(ops, mode="fixed"):
        plan = ot.BatchPlan(t, [0, n], [ops], dtype=dtype, mode=mode)
        ids = torch.empty(n, dtype=torch.int32, device="cuda")
        vel, gx, fo = torch.empty_like(X), torch.empty_like(X), torch.empty_like(U)
        plan.run(X, field=U if ops & 10 else None, force=F if ops & 12 else None, ids=ids if ops & 1 else None,
                 vel=vel if ops & 2 else None, field_out=fo if ops & 4 else None, grad=gx if ops & 8 else None)
        torch.cuda.synchronize()
        plan.close()
        return ids, vel, gx, fo

    ids, vel, _, fo = per_point(7)
    gx = per_point(12)[2]
    for hid in (None, ids):
        assert torch.equal(t.interpolate(U, X, ids=hid), vel)
        assert torch.equal(t.spread(F, X, mode="fixed", ids=hid), fo)
        assert torch.equal(t.grad_pos(U, F, X, ids=hid), gx)
        gf, g = t.interp_backward(U, F, X, mode="fixed", ids=hid)
        assert torch.equal(gf, fo) and torch.equal(g, gx)
        gF, g = t.spread_backward(U, F, X, ids=hid)
        assert torch.equal(gF, vel) and torch.equal(g, gx)
    i, v, f = t.track(X, field=U, force=F, mode="fixed")
    assert torch.equal(i, ids) and torch.equal(v, vel) and torch.equal(f, fo)
    acc = fo.clone()
    t.spread(F, X, mode="fixed", out=acc, accumulate=True)
    assert torch.equal(acc, fo + fo)
    fa = t.spread(F, X, mode="atomic")
    f, S, cnt, A = o.spread(F.double().cpu().numpy(), P, with_scale=True)
    assert spread_excess(fa.cpu().numpy(), f, S, A, cnt, dtype) <= 1.0
    F[n // 2, 1] = float("inf")
    assert bool(torch.isnan(t.spread(F, X, mode="fixed")).all())
