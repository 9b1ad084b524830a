"""Trees of at most 512 leaves, whose points are not sorted to spread: plain calls, sorted plans and plans that were not
asked to sort agree bit for bit (fixed point), at both sides of the node-parallel pass's line (8,192 points)."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import as_dtype, gpu_tree, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("n", [1, 8192, 8193, 120_000, 420_000])
@pytest.mark.parametrize("level", [0, 3])
def test_routes_agree(level, n, dtype):
    import paper_2605_20565_amd as ot
    t = gpu_tree(synth.uniform_tree(level, seed=1))
    rng = np.random.default_rng(n)
    X, V = to_dev(as_dtype(rng.random((n, 3)) * 0.999, dtype), dtype), to_dev(rng.standard_normal((n, 3)), dtype)
    U = to_dev(rng.standard_normal((t.n_leaves, 3)), dtype)
    for mode in ("fixed", "atomic"):
        out = []
        for srt in (False, True):
            plan = ot.BatchPlan(t, [0, n], [7], dtype=dtype, mode=mode, sort_points=srt)
            ids, vel, fo = torch.full((n,), -7, dtype=torch.int32, device="cuda"), torch.empty_like(X), torch.empty_like(U)
            for _ in range(2):
                plan.run(X, field=U, force=V, ids=ids, vel=vel, field_out=fo)
            torch.cuda.synchronize()
            plan.close()
            out.append((ids, vel, fo))
        out.append(t.track(X, field=U, force=V, mode=mode))
        for ids, vel, fo in out[1:]:
            assert torch.equal(ids, out[0][0]) and torch.equal(vel, out[0][1])
            if mode == "fixed":
                assert torch.equal(fo, out[0][2])
            else:   # sums of n products at most, in any order
                bound = n * 2.0 ** (-24 if dtype == torch.float32 else -53) * float(V.abs().max()) * 27
                assert float((fo - out[0][2]).abs().max()) <= bound
