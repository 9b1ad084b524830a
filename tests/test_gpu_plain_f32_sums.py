"""FP32 atomic spreading in plain calls that sort their points is summed in FP64 and rounded once, as in sorted plans:
it differs from the fixed-point result of the same inputs (the same products, exact in FP64, rounded to the quantum)
by at most one FP32 unit in the last place plus half a quantum a product, and one more unit where it is added to a
field.  Points in random order and in host order, whose sums an unsorted call splits least; trees with sub-tables and
walls, so that the tiles of coarse and fine blocks and the ranges of sparse ones all take part."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import as_dtype, fixed_point_quantum, gpu_tree, oracle_tree, to_dev

pytestmark = pytest.mark.gpu

SHELL = synth.Sphere((0.5, 0.45, 0.55), 0.12)
TREES = {"uniform": lambda: synth.uniform_tree(4, seed=1),
         "deep_walled": lambda: synth.band_tree(3, 7, [SHELL], periodic=False, seed=2)}


@pytest.fixture(scope="module", params=sorted(TREES))
def tree(request):
    spec = TREES[request.param]()
    return spec, oracle_tree(spec), gpu_tree(spec)


@pytest.mark.parametrize("order", ["random", "host"])
@pytest.mark.parametrize("n", [30_000, 120_000, 310_000, 410_000])
def test_plain_call_rounds_once(tree, n, order):
    spec, o, t = tree
    rng = np.random.default_rng(n)
    P = np.concatenate([rng.random((n - n // 2, 3)) * 0.9999, synth.gaussian_shell_points(n // 2, [SHELL], 0.004, rng)])
    P = as_dtype(np.clip(P[rng.permutation(n)], 0.0, 0.9999), torch.float32)
    if order == "host":
        P = P[np.argsort(o.locate(P), kind="stable")]
    F = as_dtype(rng.standard_normal((n, 3)), torch.float32)
    X, V = to_dev(P, torch.float32), to_dev(F, torch.float32)
    U = to_dev(rng.standard_normal((spec.n_leaves, 3)), torch.float32)
    _, _, cnt, _ = o.spread(F, P, with_scale=True)
    half = 0.5 * fixed_point_quantum(F) * cnt[:, None]
    fixed = t.spread(V, X, mode="fixed").double().cpu().numpy()
    bound = 2.0 ** -23 * np.abs(fixed) + half
    for got in (t.spread(V, X), t.track(X, field=U, force=V)[2], t.interp_backward(U, V, X)[0]):
        assert np.all(np.abs(got.double().cpu().numpy() - fixed) <= bound)
    base = rng.standard_normal((spec.n_leaves, 3)).astype(np.float32)
    got = t.spread(V, X, out=torch.from_numpy(base).cuda(), accumulate=True).double().cpu().numpy()
    want = base + fixed
    assert np.all(np.abs(got - want) <= bound + 2.0 ** -23 * np.abs(want))
