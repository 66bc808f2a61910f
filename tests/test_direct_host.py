"""Host logic of the direct solver's elimination plan, compiled for the CPU: its tasks,
run in their order on a random symmetric positive definite matrix of the mesh's pattern,
solve the system, and each comes after those it waits for."""

import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2203_11938_amd import workloads as W

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2203_11938_amd", "csrc")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("direct") / "libdirect_check.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I" + CSRC,
                    os.path.join(HERE, "host", "direct_check.cpp"),
                    os.path.join(CSRC, "direct_prep.cpp"), "-o", out], check=True)
    return ctypes.CDLL(out)


def neighbours(nv, tris):
    """Vertices that share a triangle, and the opposite vertices of an inner edge."""
    adj = [{i} for i in range(nv)]
    edge = {}
    for a, b, c in tris:
        for u, v, w in ((a, b, c), (b, c, a), (c, a, b)):
            adj[u].add(v)
            adj[v].add(u)
            k = (min(u, v), max(u, v))
            if k in edge:
                adj[edge[k]].add(w)
                adj[w].add(edge[k])
            edge[k] = w
    return adj


def fan(n):
    """n triangles around one vertex: a hub coupled to every other vertex."""
    t = 2 * np.pi * np.arange(n) / n
    rest = np.zeros((n + 1, 3))
    rest[1:, 0], rest[1:, 1] = np.cos(t), np.sin(t)
    i = np.arange(n)
    return rest, np.stack([np.zeros(n, int), 1 + i, 1 + (i + 1) % n], 1)


def strip(n):
    """A strip n vertices long and two wide: every separator is a few vertices."""
    rest = np.zeros((2 * n, 3))
    rest[:, 0], rest[:, 1] = np.arange(2 * n) // 2, np.arange(2 * n) % 2
    i = 2 * np.arange(n - 1)
    return rest, np.concatenate([np.stack([i, i + 1, i + 2], 1), np.stack([i + 1, i + 3, i + 2], 1)])


def stacked(n):
    """All rest positions equal: the cuts have no direction to go by."""
    rest, tris = W.grid_sheet(n)
    return np.zeros_like(rest), tris


MESHES = {
    "triangle": lambda: [(np.eye(3), np.array([[0, 1, 2]]))],
    "one front": lambda: [W.grid_sheet(4)],
    "pieces at the cut size": lambda: [W.grid_sheet(n) for n in (5, 6, 8)],
    "17": lambda: [W.grid_sheet(17)],
    "33": lambda: [W.grid_sheet(33)],
    "unequal batch": lambda: [W.grid_sheet(n) for n in (2, 16, 23)],
    "fan": lambda: [fan(60)],
    "strip": lambda: [strip(150)],
    "stacked": lambda: [stacked(12)],
}


@pytest.mark.parametrize("name", list(MESHES))
def test_plan_solves_the_system(lib, name):
    sheets = MESHES[name]()
    voff = np.cumsum([0] + [len(r) for r, _ in sheets]).astype(np.int32)
    nv = int(voff[-1])
    adj = [{v + o for v in a} for (r, t), o in zip(sheets, voff) for a in neighbours(len(r), t)]
    maxnz = max(len(a) for a in adj)
    rng = np.random.default_rng(3)
    ell = np.full((maxnz, nv), -1, np.int32)
    A = np.zeros((maxnz, 9, nv))
    dense = np.zeros((3 * nv, 3 * nv))
    for i in range(nv):          # a sum of B B^T over the edges, plus the identity
        dense[3 * i:3 * i + 3, 3 * i:3 * i + 3] += np.eye(3)
        for j in adj[i]:
            if j > i:
                e = np.r_[3 * i:3 * i + 3, 3 * j:3 * j + 3]
                B = rng.standard_normal((6, 3))
                dense[np.ix_(e, e)] += B @ B.T
    for i in range(nv):
        order = rng.permutation(sorted(adj[i]))
        for k, j in enumerate(order):
            ell[k, i] = j
            A[k, :, i] = dense[3 * i:3 * i + 3, 3 * j:3 * j + 3].ravel()
    b = rng.standard_normal((3, nv))
    x = np.zeros((3, nv))
    rest = np.ascontiguousarray(np.concatenate([r for r, _ in sheets]), np.float64)
    size = np.diff(voff).astype(np.int32)
    counts = np.zeros(4, np.int32)
    P = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    rc = lib.direct_check(nv, maxnz, P(ell), len(sheets), P(voff), P(size), P(rest), P(A), P(b),
                          P(x), P(counts))
    assert rc == 0
    assert counts[2] <= 96 and counts[3] <= 4096
    ref = np.linalg.solve(dense, b.T.ravel())
    cond = np.linalg.cond(dense)
    # backward-stable elimination: eps times the condition number, with room for the
    # explicit pivot inverses
    assert np.abs(x.T.ravel() - ref).max() <= 64 * np.finfo(float).eps * cond * np.abs(ref).max()
