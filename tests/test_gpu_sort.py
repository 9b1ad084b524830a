"""The pair sort behind the particle sort and the tree build, at the edges of its tiles of 2,048 keys: the particles'
order is exactly the stable order of their host ids (none counting as the last), and a shuffled tree's permutation
exactly the order of its Morton keys."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import gpu_tree, to_dev

pytestmark = pytest.mark.gpu

SHELL = synth.Sphere((0.5, 0.45, 0.55), 0.12)


@pytest.fixture(scope="module", params=[(3, 3), (4, 6), (5, 8)])   # one to three passes over the host ids
def tree(request):
    lo, hi = request.param
    spec = synth.uniform_tree(lo, seed=1) if lo == hi else synth.band_tree(lo, hi, [SHELL], periodic=False, seed=2)
    return spec, gpu_tree(spec)


@pytest.mark.parametrize("n", [1, 255, 2047, 2048, 2049, 16_385, 300_001])
def test_particle_order_is_the_stable_order_of_hosts(tree, n):
    spec, t = tree
    rng = np.random.default_rng(n)
    P = rng.random((n, 3))
    P[::7] = P[0]          # many particles of one host, in input order
    P[3::101] = 2.0        # and some without one
    X = to_dev(P, torch.float64)
    others = [to_dev(rng.standard_normal((n, 3)), torch.float64) for _ in range(3)]
    Xs, Vs, VPs, APs, ids, perm = t.particle_sort(X, *others)
    hosts = t.locate(X).cpu().numpy().astype(np.int64)
    order = np.argsort(np.where(hosts < 0, spec.n_leaves, hosts), kind="stable")
    assert np.array_equal(perm.cpu().numpy(), order)
    assert np.array_equal(ids.cpu().numpy(), hosts[order])
    assert torch.equal(Xs, X[perm.long()])
    for a, b in zip((Vs, VPs, APs), others):
        assert torch.equal(a, b[perm.long()])
