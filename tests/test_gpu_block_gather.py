"""Plans that only gather, on trees large enough for the block pass (131,072 leaves, 2 M points): velocities and
gradients of sorted plans bit for bit those of unsorted ones; on smaller trees, and in plain calls of any size, too.
Walls, tiles of root cubes and of sub-tables, sparse blocks, points without a host."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import as_dtype, gpu_tree, to_dev

pytestmark = pytest.mark.gpu

SHELL = synth.Sphere((0.5, 0.45, 0.55), 0.2)
TREES = {"large_walled": lambda: synth.band_tree(5, 8, [SHELL], periodic=False, seed=2),
         "uniform": lambda: synth.uniform_tree(6, seed=1),
         "small": lambda: synth.band_tree(3, 5, [SHELL], seed=3)}


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("name", sorted(TREES))
def test_gathers_equal_per_point_pass(name, dtype):
    import paper_2605_20565_amd as ot
    spec = TREES[name]()
    assert (spec.n_leaves >= 131072) == (name != "small")
    t = gpu_tree(spec)
    rng = np.random.default_rng(3)
    n = 2_300_001
    P = np.concatenate([rng.random((n - 1_100_002, 3)) * (1 - 1e-6),
                        synth.gaussian_shell_points(1_100_000, [SHELL], 0.004, rng),
                        np.array([[np.nan, 0.5, 0.5], [-0.25, 0.5, 0.5]])])
    X = to_dev(as_dtype(P[rng.permutation(n)], dtype), dtype)
    V, U = to_dev(rng.standard_normal((n, 3)), dtype), to_dev(rng.standard_normal((spec.n_leaves, 3)), dtype)
    for ops in (2, 3, 8, 10):
        out = []
        for srt in (False, True):
            plan = ot.BatchPlan(t, [0, 1000, n], [ops, ops], dtype=dtype, mode="fixed", sort_points=srt)
            ids = torch.full((n,), -7, dtype=torch.int32, device="cuda")
            vel, gx = torch.full_like(X, 9.0), torch.full_like(X, 9.0)
            for _ in range(2):   # the second run starts from the first one's leftovers
                plan.run(X, field=U, force=V if ops & 8 else None, ids=ids if ops & 1 else None,
                         vel=vel if ops & 2 else None, grad=gx if ops & 8 else None)
            plan.close()
            out.append((ids, vel, gx))
        for a, b in zip(*out):
            assert torch.equal(a, b)
        if ops == 3:
            ids, vel, _ = t.track(X, field=U, ops=3)
            assert torch.equal(ids, out[0][0]) and torch.equal(vel, out[0][1])
        if ops == 2:
            assert torch.equal(t.interpolate(U, X), out[0][1])
