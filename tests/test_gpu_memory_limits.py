"""A plan that fits on the device is made, also when what fits counts the memory that the library keeps for later
calls: it gives that back first.  The rest of the device is taken by tensors that nothing is written to."""
import pytest
import torch

import synth
from gpu_util import gpu_tree

pytestmark = pytest.mark.gpu

MIB = 1 << 20


def test_plan_takes_the_room_of_kept_memory():
    import paper_2605_20565_amd as ot
    t = gpu_tree(synth.uniform_tree(5, seed=1))
    n = 10_000_000
    X, V = torch.rand((n, 3), device="cuda") * 0.999, torch.randn((n, 3), device="cuda")
    out = torch.empty((t.n_leaves, 3), device="cuda")
    torch.cuda.empty_cache()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    t.spread(V, X, out=out)            # sorts in about 800 MiB, which are kept
    torch.cuda.synchronize()
    kept = before - torch.cuda.mem_get_info()[0]
    assert kept >= 600 * MIB
    filler = []
    try:
        while torch.cuda.mem_get_info()[0] > 1532 * MIB:   # (a large allocation leaves more than it says)
            filler.append(torch.empty(torch.cuda.mem_get_info()[0] - 1500 * MIB, dtype=torch.uint8, device="cuda"))
        # about 1700 MiB: more than is free, less than with what is kept
        m = 15_900_000
        plan = ot.BatchPlan(t, [0, m], [4], dtype=torch.float64, mode="fixed", sort_points=True)
        plan.close()
        # and one that does not fit is refused
        with pytest.raises(ot.OtError):
            ot.BatchPlan(t, [0, 3 * m], [4], dtype=torch.float64, mode="fixed", sort_points=True)
    finally:
        del filler
        torch.cuda.empty_cache()
    got = t.spread(V, X, mode="fixed")
    p = ot.BatchPlan(t, [0, n], [4], mode="fixed")
    p.run(X, force=V, field_out=out)
    assert torch.equal(got, out)
    p.close()
