"""The direct solver against the FP64 oracle at the edges of its elimination plan: sheets
of a single front, of pieces at the cut size, with borders of one row and of several
Schur tiles, a hub of the largest valence taken, a strip of narrow separators, unequal
batches, factors kept and rebuilt. Gates as for the seeded sweep: positions 1e-9, gradients 1e-6
(relative, per block). Results are the same bits in a repeated run."""

import numpy as np
import pytest

from gpu_common import gpu_run, make_sim, note, oracle_for, rel
from paper_2203_11938_amd import workloads as W

pytestmark = pytest.mark.gpu

STEPS = 4


def fan(n):
    t = 2 * np.pi * np.arange(n) / n
    rest = np.zeros((n + 1, 3))
    rest[1:, 0], rest[1:, 1] = 0.3 * np.cos(t), 0.3 * np.sin(t)
    i = np.arange(n)
    return rest, np.stack([np.zeros(n, int), 1 + i, 1 + (i + 1) % n], 1)


def strip(n):
    rest = np.zeros((2 * n, 3))
    rest[:, 0], rest[:, 1] = (np.arange(2 * n) // 2) / 32.0, (np.arange(2 * n) % 2) / 32.0
    i = 2 * np.arange(n - 1)
    return rest, np.concatenate([np.stack([i, i + 1, i + 2], 1), np.stack([i + 1, i + 3, i + 2], 1)])


def instance(mesh, seed):
    rest, tris = mesh
    g = np.random.default_rng(500 + seed)
    V = len(rest)
    pins = np.array([0, V - 1])
    mat = W.Material(*(np.array(W.Material().as_tuple()) * g.uniform(0.5, 2.0, size=3)))
    forces = g.normal(0.0, 0.05, size=(STEPS, V, 3)) * (W.SHEET_SIDE ** 2 / V)
    v0 = g.normal(0.0, 0.01, size=(V, 3))
    v0[pins] = 0.0
    return W.Instance(rest, tris, pins, mat, rest.copy(), v0, forces, np.ones(3))


CASES = {
    "4": (lambda: [W.grid_sheet(4)], 0),
    "5": (lambda: [W.grid_sheet(5)], 0),
    "9": (lambda: [W.grid_sheet(9)], 0),
    "17, recomputed": (lambda: [W.grid_sheet(17)], 2),
    "33": (lambda: [W.grid_sheet(33)], 0),
    "48": (lambda: [W.grid_sheet(48)], 0),
    "fan": (lambda: [fan(30)], 0),
    "strip": (lambda: [strip(150)], 0),
    "batch": (lambda: [W.grid_sheet(n) for n in (3, 16, 23)], 0),
}


@pytest.mark.parametrize("name", list(CASES))
def test_direct_solver_matches_oracle(name):
    build, ckpt = CASES[name]
    insts = [instance(m, k) for k, m in enumerate(build())]
    w = W.workload("C2", steps=STEPS, precision="fp64", cg_tol=1e-10)
    frames = w.loss_frames()
    refs, tgts = [], []
    for inst in insts:
        o = oracle_for(inst, w)
        xo, _, _, _ = o.rollout(STEPS, inst.x0, inst.v0, inst.forces, frames)
        tgt = np.broadcast_to(inst.x0, xo.shape)
        ref = o.gradient(STEPS, inst.x0, inst.v0, inst.forces, frames, 2.0 * (xo - tgt))
        refs.append(dict(ref, x=xo))
        tgts.append(tgt)
    s = make_sim(w, insts, checkpoint_every=ckpt)
    out = gpu_run(s, w, insts, tgts)
    again = gpu_run(s, w, insts, tgts)     # now with the factors kept
    assert out["status"] == 0 and again["status"] == 0
    assert again["stats"]["cg_iters_max"] == 1   # solved directly
    for k in ("x", "forces", "x0", "v0", "material"):
        assert np.array_equal(out[k], again[k]), k
    at = 0
    for b, (inst, ref) in enumerate(zip(insts, refs)):
        sl = slice(at, at + len(inst.rest))
        at = sl.stop
        errs = dict(x=rel(out["x"][:, sl], ref["x"]), forces=rel(out["forces"][:, sl], ref["forces"]),
                    x0=rel(out["x0"][sl], ref["x0"]), v0=rel(out["v0"][sl], ref["v0"]))
        for k in range(3):
            errs[f"mat{k}"] = abs(out["material"][b][k] - ref["material"][k]) / abs(ref["material"][k])
        note(f"direct {name} sheet {b}: " + ", ".join(f"{k} {v:.1e}" for k, v in errs.items()))
        assert errs.pop("x") < 1e-9
        assert max(errs.values()) < 1e-6, errs
    s.close()
