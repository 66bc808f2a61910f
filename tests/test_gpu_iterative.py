"""The iterative solver on handles that ask for it (a fixed matrix home), as handles left
to the library are solved directly: what its coarse space saves, the measured launch
shape, and the memory of its kept coarse operators."""

import numpy as np
import pytest

from gpu_common import as_given, gpu_run, make_sim, note, oracle_reference, rel, targets
from paper_2203_11938_amd import sim as S, workloads as W

pytestmark = pytest.mark.gpu


def test_coarse_space_cuts_the_iterative_solvers_iterations():
    """A 64x64 step takes ~1,300 iterations with block Jacobi alone and ~110 with the coarse
    level: a wrong, inaccurate or disabled coarse inverse shows up as several times more."""
    import torch
    w = W.workload("H", steps=8)
    inst = W.make_instances(w)[0]
    its = {}
    for cs in (64, 0):
        s = make_sim(w, [inst], coarse_size=cs, matrix_home="registers")
        x0 = torch.tensor(W.to_soa(inst.x0), dtype=s.dtype, device="cuda:0")
        F = torch.tensor(W.to_soa(inst.forces[:w.steps]), dtype=s.dtype, device="cuda:0")
        s.rollout(w.steps, x0, None, F, None, np.array([w.steps], np.int32))
        assert s.status() == 0
        fwd = s.cg_iters()[0]
        assert fwd.min() > 1                  # solved iteratively
        its[cs] = float(fwd.mean())
        s.close()
    note(f"64x64 sheet: iterations per solve {its[64]:.0f} with the coarse space, {its[0]:.0f} without")
    assert its[64] <= 150
    assert its[0] >= 5 * its[64]


def test_autotuned_iterative_handle_matches_oracle():
    w = W.workload("C2", steps=30)
    inst = as_given(W.make_instances(w)[0], w.precision)
    tgt = targets(w)
    s = make_sim(w, [inst], autotune=True, matrix_home="registers")
    st = s.stats()
    assert st["autotuned"] == 1 and st["autotune_candidates"] > 1 and st["autotune_ms_per_iter"] > 0
    out = gpu_run(s, w, [inst], [tgt])
    assert s.cg_iters()[0].min() > 1
    ref = oracle_reference(w, inst, tgt)
    assert rel(out["x"][-1], ref["x"][-1]) <= 1e-5
    assert rel(out["forces"], ref["forces"]) <= 1e-4
    assert rel(out["x0"], ref["x0"]) <= 1e-4
    s.close()


def test_kept_coarse_operators_and_direct_handles_memory():
    """An iterative handle keeps a segment's coarse operators, or every step's; one solved
    directly holds none of them, and factors only after an adjoint, within a fifth of the
    memory that was free."""
    import torch
    rest, tris = W.grid_sheet(64)
    sheet = S.Sheet(tris, rest, W.pin_set(64, "top2"), 1e3, 1e-4, 0.1)

    def handle(steps, **kw):
        return S.Simulator([sheet], dt=0.01, checkpoint_every=10, max_steps=steps, **kw)

    got = {}
    for steps in (100, 200):
        for kw in (dict(matrix_home="registers"), dict(matrix_home="registers", coarse_keep_all=True),
                   dict()):
            s = handle(steps, **kw)
            st = s.stats()
            got[steps, len(kw)] = st["device_bytes"]
            assert st["coarse_store_slots"] == (steps if len(kw) == 2 else 10)
            s.close()
    states = 10 * 48 * 64 * 64 + 100 * 36
    assert got[200, 0] - got[100, 0] <= states
    assert got[200, 1] - got[100, 1] <= states
    assert got[200, 2] - got[100, 2] > 100 * 4 * 384 * 384     # FP32 coarse inverses
    s = handle(20)
    before = s.stats()["device_bytes"]
    x0 = torch.tensor(W.to_soa(rest), dtype=s.dtype, device="cuda:0")
    free = torch.cuda.mem_get_info()[0]
    sizes = []
    for k in range(3):
        xo = s.rollout(20, x0)
        s.adjoint(xo)
        assert s.status() == 0
        sizes.append(s.stats()["device_bytes"] - before)
    note(f"64x64: {before / 2**20:.0f} MiB at creation, {sizes[0] / 2**20:.0f} MiB of factors")
    assert 0 < sizes[0] <= 0.2 * free and sizes == sizes[:1] * 3
    s.close()
