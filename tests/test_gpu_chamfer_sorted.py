"""The Chamfer distance's sorted search against its all-pairs search (taken when the
workspace holds no sorted copies): the same bits for every distance, index and sum, over
set sizes around the blocks of 64, point sets that defeat the sorting (all points equal,
two clusters far apart, a line, one set inside a cell of the other's grid), repeated
points and non-finite coordinates."""

import numpy as np
import pytest

from paper_2203_11938_amd import sim as S, workloads as W

pytestmark = pytest.mark.gpu


def all_pairs_bytes(ng, nm):
    up = lambda x: (x + 255) // 256 * 256
    return up(8 * ng) + up(8 * nm) + up(8 * ((ng + 255) // 256)) + up(8 * ((nm + 255) // 256)) + 256


def sets(kind, ng, nm):
    g, m = (np.asarray(a, np.float32) for a in W.chamfer_points(ng, nm, seed=ng))
    rng = np.random.default_rng(nm)
    if kind == "equal":
        g[:], m[:] = 0.25, 0.25
    elif kind == "apart":
        m[::2] += 1e3
        g += 40.0
    elif kind == "line":
        g[:, 1:], m[:, 1:] = 0.0, 0.0
    elif kind == "inside":
        m *= 1e-4
    elif kind == "repeated":
        m[nm // 2:] = m[:nm - nm // 2]
        g[:min(ng, nm)] = m[rng.permutation(nm)[:min(ng, nm)]]
    elif kind == "non-finite":
        g[3, 0], g[ng - 1, 2] = np.nan, -np.inf
        m[5], m[nm - 2, 1] = np.nan, np.inf
    elif kind == "huge":
        g *= 3e19
    return g, m


@pytest.mark.parametrize("kind,ng,nm", [
    ("sheet", 13505, 13440), ("sheet", 65536, 2753), ("sheet", 2816, 63999),
    ("equal", 13504, 13440), ("apart", 13440, 13505), ("line", 13505, 13440),
    ("inside", 20000, 9025), ("repeated", 13440, 13505), ("non-finite", 13447, 13449),
    ("huge", 13440, 13440)])
def test_sorted_search_gives_the_same_bits(kind, ng, nm):
    import torch
    g, m = sets(kind, ng, nm)
    dev = lambda a: torch.tensor(np.ascontiguousarray(a.T), device="cuda:0")
    need = S.load_library().sim_chamfer_workspace_bytes(ng, nm)
    assert need > all_pairs_bytes(ng, nm)          # the sorted search is chosen
    out = []
    for size in (need, all_pairs_bytes(ng, nm)):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda:0").fill_(0xA5)
        ch, nn = S.chamfer(dev(g), dev(m), nearest=True, workspace=ws)
        out.append({"ch": ch.cpu().numpy().reshape(1), **{k: v.cpu().numpy() for k, v in nn.items()}})
    for k in out[0]:
        assert out[0][k].tobytes() == out[1][k].tobytes(), k
