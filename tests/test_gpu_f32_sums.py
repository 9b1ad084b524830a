"""FP32 atomic spreading in sorted plans is summed in FP64 and rounded once.  The fixed-point result of the same inputs
adds the same products (exact in FP64) rounded to its quantum and is rounded once too, so the two differ by at most one
FP32 unit in the last place (2^-23 relative) plus half a quantum a product; no order of FP32 adds would keep to that.
Sizes on both sides of the rules for short ranges and blocks."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import fixed_point_quantum, gpu_tree, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ops", [4, 6])
@pytest.mark.parametrize("n", [1, 1000, 40_000, 60_000, 310_000, 1_000_000])
def test_sorted_plan_rounds_once(n, ops):
    import paper_2605_20565_amd as ot
    spec = synth.uniform_tree(4, seed=1)   # up to 244 points a leaf
    t = gpu_tree(spec)
    rng = np.random.default_rng(n)
    F = rng.standard_normal((n, 3)).astype(np.float32)
    X, V = to_dev(rng.random((n, 3)) * 0.9999, torch.float32), to_dev(F, torch.float32)
    U = to_dev(rng.standard_normal((spec.n_leaves, 3)), torch.float32)
    out = {}
    for mode in ("fixed", "atomic"):
        plan = ot.BatchPlan(t, [0, n], [ops], dtype=torch.float32, mode=mode, sort_points=True)
        fo = torch.full((spec.n_leaves, 3), 9.0, device="cuda")
        vel = torch.empty_like(X)
        for _ in range(2):   # the second run starts from the first one's leftovers
            plan.run(X, field=U if ops & 2 else None, force=V, vel=vel if ops & 2 else None, field_out=fo)
        out[mode] = fo.double().cpu().numpy()
        plan.close()
    q = fixed_point_quantum(F.astype(np.float64))
    bound = 2.0 ** -23 * np.abs(out["fixed"]) + 0.5 * q * min(27 * n, 8 * 27 * 27 * max(1, n // spec.n_leaves) + 1000)
    assert np.all(np.abs(out["atomic"] - out["fixed"]) <= bound)
