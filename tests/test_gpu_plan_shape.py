"""What a plan says of its shape is what runs: tiles of the given size where the pass takes block, tile and grid, and
the pass's own shape where it does not; the tuner times such a sorted plan once."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import gpu_tree, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tree():
    return gpu_tree(synth.uniform_tree(4, seed=1))


def _shape(t, n, ops, tile, sort=True):
    import paper_2605_20565_amd as ot
    plan = ot.BatchPlan(t, [0, n], [ops], mode="fixed", block=256, tile=tile, sort_points=sort)
    s = plan.shape()
    plan.close()
    return s


# points, ops, points of the pass's own tiles (None: as given): workgroups of 28 and of 64 unsorted points, ranges of
# four steps of 56, tiles of blocks (768 points at least), tiles of points sorted by host
@pytest.mark.parametrize("n,ops,own", [(20_000, 4, 28), (20_000, 2, 64), (100_000, 4, 224), (1_000_000, 7, 1953),
                                       (310_000, 7, 768), (400_000, 2, None), (100_000, 8, None)])
def test_shape(tree, n, ops, own):
    for tile in (256, 1024):
        pts = tile if own is None else own
        tiles, groups = _shape(tree, n, ops, tile)
        assert tiles == -(-n // pts) and 1 <= groups <= max(tiles, 512)
        assert _shape(tree, n, ops, tile, sort=False)[0] == -(-n // tile)


@pytest.mark.parametrize("n,once", [(20_000, True), (100_000, True), (400_000, False)])
def test_tuner_times_fixed_shapes_once(tree, n, once):
    from paper_2605_20565_amd import tune
    rng = np.random.default_rng(1)
    X = to_dev(rng.random((n, 3)) * 0.999, torch.float32)
    U = torch.ones((tree.n_leaves, 3), device="cuda")
    ops = 7 if once else 2
    _, timings = tune.tune(tree, [0, n], [ops], X, U, X if once else None, torch.float32, "fixed", reps=1,
                           cache_path=None)
    n_sorted = sum(k.endswith("_sort") for k in timings)
    assert n_sorted == 1 if once else n_sorted > 3
    assert sum(k.endswith("_nosort") for k in timings) >= 6
