"""find_owner around the sizes at which its launch changes (2^18 and 2^20 points) and over the owners it stages in LDS:
owners are exactly those of a search among the splitters on the host, counts exactly their histogram."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import gpu_tree, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("n", [1000, (1 << 18) - 1, 1 << 18, (1 << 20) - 1, 1 << 20, (1 << 21) + 4097])
@pytest.mark.parametrize("owners", [1, 8, 32, 33, 4096])
def test_find_owner_sizes(n, owners, dtype):
    spec = synth.uniform_tree(5, seed=1)
    t = gpu_tree(spec)
    rng = np.random.default_rng(n + owners)
    P = rng.random((n, 3)) * (1 - 2.0 ** -20)
    P[::1001] = np.nan
    X = to_dev(P, dtype)
    split = t.leaf_splitters(owners)
    owner, counts = t.find_owner(split, X)
    x = X.double().cpu().numpy()
    ok = np.isfinite(x).all(axis=1)
    c = np.floor(np.where(np.isfinite(x), x, 0.0) * (1 << spec.l_max)).astype(np.int64)
    key = np.zeros(n, dtype=np.int64)
    for b in range(spec.l_max):
        for d in range(3):
            key |= ((c[:, d] >> b) & 1) << (3 * b + d)
    want = np.searchsorted(split.cpu().numpy()[1:owners], key, side="right")
    want = np.where(ok, want, -1)
    assert np.array_equal(owner.cpu().numpy(), want)
    assert np.array_equal(counts.cpu().numpy(), np.bincount(want[ok], minlength=owners))
