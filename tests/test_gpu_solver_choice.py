"""Which solver a handle left to the library gets: the iterative one where it needs few
iterations (loose tolerances, short steps, many small sheets), else the direct one; with
either the results meet the oracle's, and creating the handle again chooses the same."""

import numpy as np
import pytest

from gpu_common import gpu_run, make_sim, note, oracle_for, rel
from paper_2203_11938_amd import workloads as W

pytestmark = pytest.mark.gpu

STEPS = 3


@pytest.mark.parametrize("n,dt,tol,batch,direct", [
    (12, 1e-2, 1e-7, 1, True), (17, 1e-2, 1e-7, 1, True), (64, 5e-3, 1e-7, 1, True),
    (64, 1e-4, 1e-7, 1, False), (64, 1e-3, 1e-3, 1, False), (17, 1e-4, 1e-3, 1, False),
    (16, 1e-2, 1e-7, 256, False), (20, 5e-3, 1e-7, 32, True)])
def test_choice_and_results(n, dt, tol, batch, direct):
    w = W.workload("C2", n=n, steps=STEPS, precision="fp64", cg_tol=tol)
    inst = W.make_instances(w)[0]
    tgt = inst.x0[None].repeat(STEPS, axis=0) + 0.01
    outs = []
    for _ in range(2):
        s = make_sim(w, [inst] * batch, dt=dt)
        outs.append(gpu_run(s, w, [inst] * batch, [tgt] * batch))
        its = s.cg_iters()[0]
        s.close()
    note(f"{batch} of {n}x{n}, dt {dt}, tol {tol}: iterations {its.mean():.0f}")
    assert ((its == 1).all() if direct else (its > 1).all())
    for k in ("x", "forces", "x0", "v0", "material"):
        assert np.array_equal(outs[0][k], outs[1][k]), k
    import oracle
    o = oracle.Oracle(inst.tris, inst.rest, inst.pins, *inst.material.as_tuple(), dt=dt, cg_tol=1e-12)
    xo, _, _, _ = o.rollout(STEPS, inst.x0, inst.v0, inst.forces, w.loss_frames())
    # a step moves by dt dv, and dv is within about tol of its norm times sqrt(cond)
    move = np.linalg.norm(xo - inst.x0) / np.linalg.norm(xo)
    assert rel(outs[0]["x"][:, :n * n], xo) <= 100.0 * tol * move * STEPS
