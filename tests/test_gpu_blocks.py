"""The block pass of sorted plans (dense grids of a block's stencil nodes in
LDS) and the node-parallel pass over sorted ranges against the per-point pass
of unsorted plans: ids, velocities, gradients and fixed-point spreading bit for
bit, atomic spreading within the oracle bound.  Blocks at the edges of the tile
rules (one point fewer than a tile needs, whole tiles and one more, one host
holding several tiles' points), walls, trees several sub-tables deep and points without a host."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import as_dtype, gpu_tree, oracle_tree, spread_excess, to_dev

pytestmark = pytest.mark.gpu

SHELL = synth.Sphere((0.5, 0.45, 0.55), 0.08)

TREES = {
    # 8 cubes of 8^3 root cells
    "uniform": lambda: synth.uniform_tree(4, seed=1),
    # sub-tables of 3 and 2 levels, walls
    "deep_walled": lambda: synth.band_tree(3, 7, [SHELL], periodic=False, seed=2),
    # sub-tables of 1 level
    "shallow": lambda: synth.band_tree(4, 5, [SHELL], seed=3),
}


@pytest.fixture(scope="module")
def ot():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2605_20565_amd as m
    return m


@pytest.fixture(scope="module", params=sorted(TREES))
def tree(request):
    spec = TREES[request.param]()
    return spec, oracle_tree(spec), gpu_tree(spec)


def _points(spec, rng, n_shell):
    """Point counts per octant of the cube at the edges of the tile rules, plus points without a host."""
    counts = [191, 192, 193, 3071, 3072, 3073, 9217, 700]
    out = []
    for o, n in enumerate(counts):
        lo = 0.5 * np.array([o & 1, (o >> 1) & 1, o >> 2])
        out.append(lo + 0.5 * rng.random((n, 3)) * (1 - 1e-6))
    out.append(0.5 + 1e-3 * rng.random((7000, 3)))          # a few hosts with thousands of points
    out.append(synth.gaussian_shell_points(n_shell, [SHELL], 0.004, rng))
    out.append(np.array([[np.nan, 0.5, 0.5], [-0.25, 0.5, 0.5], [1.5, 0.1, 0.1], [0.0, 0.0, 0.0]]))
    p = np.concatenate(out)
    return p[rng.permutation(p.shape[0])]


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("ops,n_shell", [(2, 2_000_000), (4, 420_000), (4, 280_000), (4, 30_000), (7, 280_000),
                                         (7, 30_000), (8, 2_000_000), (10, 2_000_000), (12, 280_000), (12, 30_000)])
def test_block_and_range_passes_equal_per_point_pass(ot, tree, dtype, ops, n_shell):
    spec, o, t = tree
    rng = np.random.default_rng(77)
    P = as_dtype(_points(spec, rng, n_shell), dtype)
    n = P.shape[0]
    X, F = to_dev(P, dtype), to_dev(rng.standard_normal((n, 3)), dtype)
    U = to_dev(rng.standard_normal((spec.n_leaves, 3)), dtype)
    out = {}
    for mode in ("fixed", "atomic"):
        for srt in (False, True):
            plan = ot.BatchPlan(t, [0, 1000, n], [ops, ops], dtype=dtype, mode=mode, sort_points=srt)
            ids = torch.full((n,), -7, dtype=torch.int32, device="cuda")
            vel, gx = torch.full_like(X, 9.0), torch.full_like(X, 9.0)
            fo = torch.full((spec.n_leaves, 3), 9.0, dtype=dtype, device="cuda")
            for _ in range(2):   # the second run starts from the first one's leftovers
                plan.run(X, field=U if ops & 10 else None, force=F if ops & 12 else None, ids=ids if ops & 1 else None,
                         vel=vel if ops & 2 else None, field_out=fo if ops & 4 else None, grad=gx if ops & 8 else None)
            torch.cuda.synchronize()
            plan.close()
            out[mode, srt] = (ids, vel, gx, fo)
    for mode in ("fixed", "atomic"):
        for a, b in zip(out[mode, True][:3], out[mode, False][:3]):
            assert torch.equal(a, b)
    assert torch.equal(out["fixed", True][3], out["fixed", False][3])
    if ops & 4:
        f, S, cnt, A = o.spread(F.double().cpu().numpy(), P, with_scale=True)
        # plain calls sort as well: every mode, and adding to what is there
        assert torch.equal(t.spread(F, X, mode="fixed"), out["fixed", True][3])
        acc = t.spread(F, X, mode="fixed", out=out["fixed", True][3].clone(), accumulate=True)
        assert torch.equal(acc, out["fixed", True][3] + out["fixed", True][3])
        assert spread_excess(t.spread(F, X).cpu().numpy(), f, S, A, cnt, dtype) <= 1.0
        assert spread_excess(out["atomic", True][3].cpu().numpy(), f, S, A, cnt, dtype) <= 1.0


def test_sorted_call_beside_a_capture_and_inside_one(ot):
    """A plain call large enough to be sorted, made while another stream's capture is under way (the first such call
    on its tree, so it allocates) and again inside a capture, where it takes the points as they are."""
    spec = TREES["shallow"]()
    rng = np.random.default_rng(5)
    X = to_dev(as_dtype(rng.random((70_000, 3)) * 0.999, torch.float32), torch.float32)
    F = to_dev(rng.standard_normal((70_000, 3)), torch.float32)
    t = gpu_tree(spec)
    work, fo = t.workspace(), torch.empty((spec.n_leaves, 3), device="cuda")
    beside = torch.empty_like(fo)
    side, other = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    w2 = t.workspace()
    with torch.cuda.stream(side):
        graph.capture_begin(capture_error_mode="global")
        t.spread(F, X, mode="fixed", out=fo, work=work)
        with torch.cuda.stream(other):
            t.spread(F, X, mode="fixed", out=beside, work=w2)
        graph.capture_end()
    torch.cuda.synchronize()
    for _ in range(3):
        fo.fill_(9.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(fo, beside)
