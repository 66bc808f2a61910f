"""The handle's graph option on a handle solved directly: captured calls give the bits of
direct launches, also when the adjoint is called again after the same rollout, where the
factors kept are those of other steps than before (checkpointing); and a rollout with its
adjoint in a graph of the caller's. Replays are compared with unrelated eager work and
synchronisations between them."""

import numpy as np
import pytest
import torch

from gpu_common import make_sim, note
from paper_2203_11938_amd import workloads as W

pytestmark = pytest.mark.gpu

STEPS = 24


class Runs:
    def __init__(self, checkpoint, **kw):
        self.w = W.workload("C2", steps=STEPS, precision="fp64")
        inst = W.make_instances(self.w)[0]
        dev = torch.device("cuda:0")
        self.sim = make_sim(self.w, [inst], checkpoint_every=checkpoint, **kw)
        dt = self.sim.dtype
        self.x0 = torch.tensor(W.to_soa(inst.x0), dtype=dt, device=dev)
        self.F = torch.tensor(W.to_soa(inst.forces), dtype=dt, device=dev)
        V = self.x0.shape[1]
        self.dl = torch.linspace(-1e-3, 1e-3, STEPS * 3 * V, dtype=dt, device=dev).reshape(STEPS, 3, V)
        self.xo = torch.empty((STEPS, 3, V), dtype=dt, device=dev)
        self.out = dict(material=torch.empty((1, 3), dtype=torch.float64, device=dev),
                        forces=torch.empty((STEPS, 3, V), dtype=dt, device=dev),
                        x0=torch.empty((3, V), dtype=dt, device=dev),
                        v0=torch.empty((3, V), dtype=dt, device=dev))

    def rollout(self):
        self.sim.rollout(STEPS, self.x0, None, self.F, x_out=self.xo)

    def adjoint(self):
        for t in self.out.values():
            t.fill_(float("nan"))
        self.sim.adjoint(self.dl, out=self.out)

    def results(self, direct=True):
        self.sim.sync()
        if direct:
            assert self.sim.stats()["cg_iters_max"] == 1   # every solve direct
        return [t.cpu().numpy().copy() for t in (self.xo, *self.out.values())]


def same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b))


def between():
    a = torch.randn(512, 512, device="cuda:0")
    (a @ a).sum().item()
    torch.cuda.synchronize()


@pytest.mark.parametrize("checkpoint", [0, 7])
def test_handle_graphs_on_a_direct_handle(checkpoint):
    ref, run = Runs(checkpoint), Runs(checkpoint, graph=True)
    for k in range(4):
        for r in (ref, run):
            r.x0[2] += 0.002 * k
            r.rollout()
        for call in range(3):
            ref.adjoint()
            run.adjoint()
            between()
            assert same(ref.results(), run.results()), (k, call)
    st = run.sim.stats()
    note(f"graph, checkpoint {checkpoint}: captures {st['graph_captures']}, replays {st['graph_replays']}")
    assert st["graph_replays"] >= 3


@pytest.mark.parametrize("checkpoint", [0, 7])
def test_graphs_of_the_caller_on_a_direct_handle(checkpoint):
    ref, run = Runs(checkpoint), Runs(checkpoint)
    for r in (ref, run):       # the factors' memory is taken before the capture
        r.rollout()
        r.adjoint()
    assert same(ref.results(), run.results())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        run.rollout()
        run.adjoint()
    for k in range(3):
        for r in (ref, run):
            r.x0[2] += 0.003
        ref.rollout()
        ref.adjoint()
        g.replay()
        between()
        assert same(ref.results(), run.results()), k
    # direct calls after the replays
    for k in range(2):
        for r in (ref, run):
            r.x0[2] += 0.001
            r.rollout()
            r.adjoint()
        assert same(ref.results(), run.results()), k
