"""Sorted runs (ranges, blocks, FP64 sums of FP32 fields) at once on several streams and threads, and in graphs: each
plan works in memory of its own, clears what it needs in every run, and replays with new values in the same tensors."""
import threading

import numpy as np
import pytest
import torch

import synth
from gpu_util import as_dtype, gpu_tree, to_dev

pytestmark = pytest.mark.gpu

SHELL = synth.Sphere((0.5, 0.45, 0.55), 0.12)


@pytest.fixture(scope="module")
def tree():
    return gpu_tree(synth.band_tree(4, 6, [SHELL], periodic=False, seed=2))


def _inputs(t, n, dtype, seed):
    rng = np.random.default_rng(seed)
    X = to_dev(as_dtype(rng.random((n, 3)) * 0.999, dtype), dtype)
    return X, to_dev(rng.standard_normal((n, 3)), dtype), to_dev(rng.standard_normal((t.n_leaves, 3)), dtype)


class _Run:
    """A plan with outputs of its own, and what an unsorted plan makes of the same inputs."""

    def __init__(self, t, n, dtype, mode, seed, graph=False):
        import paper_2605_20565_amd as ot
        self.X, self.V, self.U = _inputs(t, n, dtype, seed)
        self.mode = mode
        self.vel, self.fo = torch.empty_like(self.X), torch.empty_like(self.U)
        self.plan = ot.BatchPlan(t, [0, n // 3, n], [6, 6], dtype=dtype, mode=mode, sort_points=True, graph=graph)
        self.plain = ot.BatchPlan(t, [0, n // 3, n], [6, 6], dtype=dtype, mode="fixed")

    def run(self):
        self.plan.run(self.X, field=self.U, force=self.V, vel=self.vel, field_out=self.fo)

    def check(self):
        vel, fo = torch.empty_like(self.vel), torch.empty_like(self.fo)
        self.plain.run(self.X, field=self.U, force=self.V, vel=vel, field_out=fo)
        torch.cuda.current_stream().synchronize()
        assert torch.equal(self.vel, vel)
        if self.mode == "fixed":
            assert torch.equal(self.fo, fo)
        else:
            assert float((self.fo - fo).abs().max()) <= 1e-5 * float(fo.abs().max())

    def close(self):
        self.plan.close()
        self.plain.close()


KINDS = [(120_000, torch.float32, "fixed"), (310_000, torch.float32, "fixed"), (120_000, torch.float32, "atomic"),
         (310_000, torch.float32, "atomic"), (120_000, torch.float64, "fixed"), (700_000, torch.float64, "atomic")]


def test_plans_of_one_tree_on_several_streams(tree):
    runs = [_Run(tree, *k, seed=i) for i, k in enumerate(KINDS)]
    streams = [torch.cuda.Stream() for _ in runs]
    torch.cuda.synchronize()
    for rep in range(4):
        for r in runs:
            r.vel.fill_(9.0)
            r.fo.fill_(9.0)
        torch.cuda.synchronize()
        for i, r in enumerate(runs):
            with torch.cuda.stream(streams[(i + rep) % len(streams)]):
                r.run()
        torch.cuda.synchronize()
        for r in runs:
            r.check()
    for r in runs:
        r.close()


def test_plans_of_one_tree_in_several_threads(tree):
    errors = []

    def work(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                r = _Run(tree, *KINDS[i], seed=10 + i)
                torch.cuda.current_stream().synchronize()
                for _ in range(4):
                    r.run()
                    torch.cuda.current_stream().synchronize()
                    r.check()
                r.close()
        except BaseException as e:   # noqa: BLE001 (shown below)
            errors.append(e)

    th = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for x in th:
        x.start()
    for x in th:
        x.join()
    assert not errors, errors


@pytest.mark.parametrize("kind", KINDS[:5])
@pytest.mark.parametrize("how", ["plan", "captured"])
def test_graph_replays(tree, kind, how):
    r = _Run(tree, *kind, seed=20, graph=how == "plan")
    rng = np.random.default_rng(3)
    if how == "captured":
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            r.run()
    for rep in range(4):
        r.V.copy_(to_dev(rng.standard_normal(tuple(r.V.shape)) * 10.0 ** rep, r.V.dtype))
        r.vel.fill_(9.0)
        r.fo.fill_(9.0)
        if how == "captured":
            graph.replay()
        else:
            r.run()
        torch.cuda.synchronize()
        r.check()
    r.close()
