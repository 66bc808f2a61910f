"""The Chamfer distance's sorted search on sets that a grid over all their points would put
into a few cells: outliers far away, clusters far apart, many equal points. The bits are
those of the all-pairs search, and it is not much slower than that: the grid spans the bulk
of a set, points of one cell take their places together, and sets that are concentrated
all the same are searched plainly. Very unequal sets, whose sort would take longer than
their pairs, are not sorted at all."""

import numpy as np
import pytest

from gpu_common import note
from paper_2203_11938_amd import sim as S, workloads as W
from test_gpu_chamfer_sorted import all_pairs_bytes

pytestmark = pytest.mark.gpu


def sets(kind, ng, nm):
    g, m = (np.array(a, np.float32) for a in W.chamfer_points(ng, nm, seed=ng))
    rng = np.random.default_rng(nm)
    if kind == "outlier":
        g[7] = (900.0, 800.0, -700.0)
    elif kind == "outliers":
        for a in (g, m):
            a[::97] += rng.normal(0.0, 300.0, a[::97].shape)
    elif kind == "clusters":
        g[::2] += 1e3
        m[::2] += 1e3
    elif kind == "half equal":
        g[::2], m[::2] = 0.25, 0.25
    elif kind == "equal":
        g[:], m[:] = 0.25, 0.5
    elif kind == "non-finite":
        g[::3], m[1::2] = np.nan, np.inf
    elif kind == "nowhere finite":
        g[:] = np.nan
    return g, m


def run(g, m, size):
    import torch
    G, M = (torch.tensor(np.ascontiguousarray(a.T), device="cuda:0") for a in (g, m))
    ws = torch.empty(size, dtype=torch.uint8, device="cuda:0").fill_(0xA5)
    best = 1e9
    for k in range(4):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(5):
            ch, nn = S.chamfer(G, M, nearest=True, workspace=ws)
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / 5)
    return best, [ch.cpu().numpy().tobytes()] + [nn[k].cpu().numpy().tobytes() for k in sorted(nn)]


@pytest.mark.parametrize("ng,nm", [(30011, 30000), (13505, 13440), (65536, 2753)])
@pytest.mark.parametrize("kind", ["outlier", "outliers", "clusters", "half equal", "equal",
                                  "non-finite", "nowhere finite"])
def test_concentrated_sets(kind, ng, nm):
    g, m = sets(kind, ng, nm)
    need = S.load_library().sim_chamfer_workspace_bytes(ng, nm)
    assert need > all_pairs_bytes(ng, nm)
    fast, got = run(g, m, need)
    plain, ref = run(g, m, all_pairs_bytes(ng, nm))
    note(f"{kind} {ng} by {nm}: {1e3 * fast:.0f} us, all pairs {1e3 * plain:.0f} us")
    assert got == ref
    assert fast < 1.5 * plain       # a grid over all points: 1.3 to 11 times as long


def test_very_unequal_sets_are_not_sorted():
    lib = S.load_library()
    for ng, nm in ((2000000, 100), (100, 2000000), (1000000, 300), (500000, 1000)):
        assert lib.sim_chamfer_workspace_bytes(ng, nm) == all_pairs_bytes(ng, nm)
    assert lib.sim_chamfer_workspace_bytes(300000, 2000) > all_pairs_bytes(300000, 2000)
