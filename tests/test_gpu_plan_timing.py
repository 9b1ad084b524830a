"""Timing of plans: every kind of plan that ran has a duration, also one whose ids come from the sort alone."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import gpu_tree, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ops", [1, 3, 7])
@pytest.mark.parametrize("n,sort", [(0, True), (1000, True), (120_000, True), (120_000, False)])
def test_timed_run_has_a_duration(ops, n, sort):
    import paper_2605_20565_amd as ot
    t = gpu_tree(synth.uniform_tree(4, seed=1))
    rng = np.random.default_rng(1)
    X = to_dev(rng.random((n, 3)) * 0.999, torch.float32)
    U, V = torch.ones((t.n_leaves, 3), device="cuda"), torch.ones_like(X)
    ids, vel, fo = torch.full((n,), -7, dtype=torch.int32, device="cuda"), torch.empty_like(X), torch.empty_like(U)
    plan = ot.BatchPlan(t, [0, n], [ops], mode="fixed", sort_points=sort)
    plan.set_timing(True)
    for _ in range(2):
        plan.run(X, field=U if ops & 2 else None, force=V if ops & 4 else None, ids=ids, vel=vel if ops & 2 else None,
                 field_out=fo if ops & 4 else None)
    torch.cuda.synchronize()
    assert 0.0 <= plan.last_kernel_ms() < 1000.0
    assert torch.equal(ids, t.locate(X))
    plan.close()


def test_a_failed_call_does_not_fail_the_next():
    import paper_2605_20565_amd as ot
    t = gpu_tree(synth.uniform_tree(2, seed=1))
    X = torch.rand((100, 3), device="cuda") * 0.999
    plan = ot.BatchPlan(t, [0, 100], [1])
    plan.set_timing(True)
    with pytest.raises(ot.OtError):   # nothing has run yet
        plan.last_kernel_ms()
    assert int(t.locate(X).min()) >= 0
    plan.close()
