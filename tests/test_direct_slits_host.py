"""The direct solver's elimination plan on sheets with slits, whose tree has fronts of three
and more children, and the hand-over of its workgroups' waits; both compiled for the CPU."""

import ctypes
import os
import subprocess

import numpy as np
import pytest

import test_direct_host as D


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("slits") / "libdirect_check.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I" + D.CSRC,
                    *(os.path.join(D.HERE, "host", f)
                      for f in ("direct_check.cpp", "wait_check.cpp", "plan_check.cpp")),
                    os.path.join(D.CSRC, "direct_prep.cpp"), "-o", out], check=True)
    return ctypes.CDLL(out)


def comb(teeth, width, length, spine):
    """A grid of `spine` rows below `teeth` strips of `width` vertices and `length` rows."""
    cols, rows = teeth * width, spine + length
    rest = np.array([(i, j, 0.0) for j in range(rows) for i in range(cols)])
    tris = []
    for j in range(rows - 1):
        for i in range(cols - 1):
            if j < spine - 1 or (i + 1) % width:
                a, c = j * cols + i, (j + 1) * cols + i
                tris += [(a, a + 1, c + 1), (a, c + 1, c)]
    return rest, np.array(tris)


@pytest.mark.parametrize("shapes", [[(4, 6, 16, 4)], [(7, 6, 18, 4), (3, 4, 9, 3)]])
def test_plan_with_slits_solves_the_system(lib, shapes, monkeypatch):
    monkeypatch.setitem(D.MESHES, "slits", lambda: [comb(*s) for s in shapes])
    D.test_plan_solves_the_system(lib, "slits")


@pytest.mark.parametrize("shape", [(4, 6, 16, 4), (7, 6, 18, 4), (4, 8, 24, 6)])
def test_slits_give_fronts_of_more_than_two_children(lib, shape):
    rest, tris = comb(*shape)
    adj = D.neighbours(len(rest), tris)
    ell = np.full((max(map(len, adj)), len(rest)), -1, np.int32)
    for i, a in enumerate(adj):
        ell[:len(a), i] = sorted(a)
    P = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    more = ctypes.c_int()
    rest = np.ascontiguousarray(rest, np.float64)
    assert lib.plan_children(len(rest), len(ell), P(ell), P(rest), ctypes.byref(more)) >= 3
    assert more.value > 0


def test_waits_hand_over_their_own_outcome(lib):
    """A wavefront may read a wait's outcome late, when wavefront 0 is already through with
    the next wait: with one word it then reads that one's; with the words the solver uses
    in turn, never."""
    assert lib.wait_check(1) > 0
    assert lib.wait_check(0) == 0
