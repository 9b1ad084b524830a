"""Working memory of plain calls that sort their points: shared by the trees of a device, handed on between streams,
threads and trees in order, grown, and more calls at once than there are buffers.  Results are those of a plan that
does not sort, bit for bit (fixed point).  What is kept stays within its bound."""
import threading

import numpy as np
import pytest
import torch

import synth
from gpu_util import as_dtype, gpu_tree, to_dev

pytestmark = pytest.mark.gpu

SHELL = synth.Sphere((0.5, 0.45, 0.55), 0.12)


def _unsorted(t, X, V):
    import paper_2605_20565_amd as ot
    n = X.shape[0]
    plan = ot.BatchPlan(t, [0, n], [4], dtype=X.dtype, mode="fixed")
    fo = torch.empty((t.n_leaves, 3), dtype=X.dtype, device="cuda")
    plan.run(X, force=V, field_out=fo)
    torch.cuda.synchronize()
    plan.close()
    return fo


def _case(spec, n, dtype, seed):
    rng = np.random.default_rng(seed)
    return to_dev(as_dtype(rng.random((n, 3)) * 0.999, dtype), dtype), to_dev(rng.standard_normal((n, 3)), dtype)


def test_streams_of_one_thread_take_turns():
    """More streams than buffers, calls of growing and shrinking size on two trees, nothing waited for in between."""
    trees = [gpu_tree(synth.band_tree(3, 6, [SHELL], seed=2)), gpu_tree(synth.uniform_tree(4, seed=1))]
    sizes = [60_000, 200_000, 90_000, 700_000, 61_000, 330_000]
    cases = [(t, *_case(None, n, torch.float32, i)) for i, n in enumerate(sizes) for t in trees]
    want = [_unsorted(*c) for c in cases]
    work = [t.workspace() for t, _, _ in cases]
    streams = [torch.cuda.Stream() for _ in range(6)]
    torch.cuda.synchronize()
    for rep in range(4):
        got = [torch.full_like(w, 9.0) for w in want]
        torch.cuda.synchronize()
        for i, (t, X, V) in enumerate(cases):
            with torch.cuda.stream(streams[(i + rep) % len(streams)]):
                t.spread(V, X, mode="fixed", out=got[i], work=work[i])
        torch.cuda.synchronize()
        for g, w in zip(got, want):
            assert torch.equal(g, w)
    for t in trees:
        t.close()


def test_threads_with_trees_of_their_own():
    specs = [synth.band_tree(3, 6, [SHELL], seed=2), synth.uniform_tree(4, seed=1), synth.band_tree(4, 5, [SHELL], seed=3)]
    cases = [(specs[i % 3], *_case(None, 58_000 + 37_003 * i, torch.float64 if i % 2 else torch.float32, i))
             for i in range(6)]
    want = []
    for spec, X, V in cases:
        t = gpu_tree(spec)
        want.append(_unsorted(t, X, V))
        t.close()
    errors = []

    def run(k):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for rep in range(5):
                    i = (k + rep) % len(cases)
                    spec, X, V = cases[i]
                    t = gpu_tree(spec)
                    a = t.spread(V, X, mode="fixed")
                    b = t.spread(V, X, mode="fixed")
                    torch.cuda.current_stream().synchronize()
                    assert torch.equal(a, want[i]) and torch.equal(b, want[i])
                    t.close()
        except BaseException as e:   # noqa: BLE001 (shown below)
            errors.append(e)

    th = [threading.Thread(target=run, args=(k,)) for k in range(6)]
    for x in th:
        x.start()
    for x in th:
        x.join()
    assert not errors, errors


def test_kept_memory_is_bounded_for_all_trees_together():
    """Three trees in use, each with calls of about 0.5 GiB: one GiB is kept at most, a quarter of it without trees."""
    spec = synth.uniform_tree(5, seed=1)
    n = 5_000_000
    X, V = torch.rand((n, 3), device="cuda") * 0.999, torch.randn((n, 3), device="cuda")
    warm = gpu_tree(spec)   # the first call loads the kernels
    warm.spread(V[:100_000].contiguous(), X[:100_000].contiguous())
    warm.close()
    out = torch.empty((spec.n_leaves, 3), device="cuda")
    trees = [gpu_tree(spec) for _ in range(3)]
    streams = [torch.cuda.Stream() for _ in trees]
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    for t, s in zip(trees, streams):
        with torch.cuda.stream(s):
            t.spread(V, X, out=out)
        torch.cuda.synchronize()
    assert before - torch.cuda.mem_get_info()[0] <= (1 << 30) + (64 << 20)
    for t in trees:
        t.close()
    assert before - torch.cuda.mem_get_info()[0] <= (256 << 20) + (64 << 20)
