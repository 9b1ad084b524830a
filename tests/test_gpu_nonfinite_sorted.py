"""Forces that are not finite through the passes over sorted points: tiles of blocks, short ranges, plain calls that
sort.  FIXED carries them to the whole field as NaN; ATOMIC to the leaves of the point, as the per-point pass of an
unsorted plan does (a NaN or infinite value is the same whatever the order of the sum); gradients of those points are
those of the per-point pass, also beside walls, where nodes are dropped; velocities and every other gradient do not
change."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import as_dtype, gpu_tree, to_dev

pytestmark = pytest.mark.gpu

SHELL = synth.Sphere((0.5, 0.45, 0.55), 0.12)
INF, NAN = float("inf"), float("nan")
BAD = [(INF, 0.5, 0.25), (0.5, -INF, 0.25), (0.5, 0.25, INF), (NAN, 0.5, 0.25), (INF, -INF, 0.5), (0.0, INF, 0.0)]


@pytest.fixture(scope="module", params=[True, False])
def tree(request):
    spec = synth.band_tree(4, 6, [SHELL], periodic=request.param, seed=2)
    return spec, gpu_tree(spec)


def _inputs(spec, n, dtype):
    """Points in random order; every bad force at points inside, on a face and in a corner, far from each other."""
    rng = np.random.default_rng(n)
    P = np.concatenate([rng.random((n - n // 2, 3)) * 0.9999, synth.gaussian_shell_points(n // 2, [SHELL], 0.004, rng)])
    P = np.clip(P[rng.permutation(n)], 0.0, 0.9999)
    F = rng.standard_normal((n, 3))
    k = 0
    for i, bad in enumerate(BAD):
        for at in [(0.003, 0.15 * i + 0.1, 0.52), (0.15 * i + 0.1, 0.997, 0.02), (0.15 * i + 0.08, 0.3, 0.7)]:
            j = (k * 7919 + 13) % n
            P[j], F[j] = at, bad
            k += 1
    U = 1.0 + rng.random((spec.n_leaves, 3))   # of one sign: sums with one infinite component stay infinite
    return to_dev(as_dtype(P, dtype), dtype), to_dev(F, dtype), to_dev(U, dtype)


def _same(a, b):
    return torch.equal(torch.nan_to_num(a, nan=1e30, posinf=2e30, neginf=3e30),
                       torch.nan_to_num(b, nan=1e30, posinf=2e30, neginf=3e30))


def _special(a):
    return torch.where(torch.isnan(a), 1, 0) + torch.where(torch.isposinf(a), 2, 0) + torch.where(torch.isneginf(a), 4, 0)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("n", [70_000, 310_000, 1_100_000])
def test_not_finite_forces(tree, n, dtype):
    import paper_2605_20565_amd as ot
    spec, t = tree
    X, V, U = _inputs(spec, n, dtype)
    for mode in ("fixed", "atomic"):
        for ops in (6, 12):
            out = []
            for srt in (False, True):
                plan = ot.BatchPlan(t, [0, n], [ops], dtype=dtype, mode=mode, sort_points=srt)
                vel, gx, fo = torch.full_like(X, 9.0), torch.full_like(X, 9.0), torch.full_like(U, 9.0)
                kw = {"vel": vel} if ops & 2 else {"grad": gx}
                plan.run(X, field=U, force=V, field_out=fo, **kw)
                torch.cuda.synchronize()
                plan.close()
                out.append((vel, gx, fo))
            if ops == 6:
                out.append((t.track(X, field=U, force=V, ops=6, mode=mode)[1], out[0][1],
                            t.spread(V, X, mode=mode)))
            else:
                gf, gx = t.interp_backward(U, V, X, mode=mode)
                out.append((out[0][0], gx, gf))
            for vel, gx, fo in out[1:]:
                assert torch.equal(vel, out[0][0])
                assert _same(gx, out[0][1])
                if mode == "fixed":
                    assert bool(torch.isnan(fo).all())
                else:
                    assert torch.equal(_special(fo), _special(out[0][2]))
        assert int(_special(out[0][2]).count_nonzero()) > 0
