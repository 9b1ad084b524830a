"""FP64 atomic spreading: how far a field may be from the oracle's.

A leaf's sum of m contributions of random sign, added in G groups of g (m = g G) of one precision, each add rounded
(unit u = 2^-53, on average 0.41 u of the value), has a relative rms error of about 0.41 u sqrt((g + G) / 2), and the
contributions' own products add about 1 u.  Passes over points sorted by host add a leaf's points, which come from its
27 neighbours, in about 27 groups (more where a range ends between them); passes over unsorted points in a group per
workgroup that has a point near the leaf.  The bounds are 1.5 times the estimate for 60 groups, or 1.15 times it for
the workgroups that an unsorted call has (64 points each in small calls), whose estimate is closer."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import gpu_tree, oracle_tree

pytestmark = pytest.mark.gpu

U = 2.0 ** -53


def _estimate(g, G):
    return U * (1.0 + 0.41 * np.sqrt(0.5 * (g + G)))


def _inputs(level, n, order):
    spec = synth.uniform_tree(level, seed=1)
    o, t = oracle_tree(spec), gpu_tree(spec)
    rng = np.random.default_rng(n)
    P, F = rng.random((n, 3)) * 0.999, rng.standard_normal((n, 3))
    if order == "host":
        P = P[np.argsort(o.locate(P), kind="stable")]
    f = o.spread(F, P, with_scale=True)[0]

    def err(got):
        return np.linalg.norm(got.cpu().numpy() - f) / np.linalg.norm(f)
    return spec, t, torch.from_numpy(P).cuda(), torch.from_numpy(F).cuda(), err


@pytest.mark.parametrize("order", ["random", "host"])
@pytest.mark.parametrize("n", [1024, 1025, 3000, 50_000, 65_000, 100_000])
def test_sorted_plan(n, order):
    import paper_2605_20565_amd as ot
    spec, t, X, V, err = _inputs(4, n, order)
    plan = ot.BatchPlan(t, [0, n], [4], dtype=torch.float64, mode="atomic", sort_points=True)
    fo = torch.full((spec.n_leaves, 3), 9.0, dtype=torch.float64, device="cuda")
    for _ in range(2):   # the second run starts from the first one's leftovers
        plan.run(X, force=V, field_out=fo)
    assert err(fo) <= 1.5 * _estimate(27.0 * n / spec.n_leaves / 60, 60)
    plan.close()


@pytest.mark.parametrize("n", [8000, 50_000, 100_000])
def test_plain_call_on_few_leaves(n):
    spec, t, X, V, err = _inputs(3, n, "random")
    assert err(t.spread(V, X)) <= 1.15 * _estimate(64 * 27.0 / spec.n_leaves, n / 64)
