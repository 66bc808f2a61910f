"""Host side of the C ABI, compiled for the CPU over a device of settable memory whose
kernels are stood for by one number each (host/fake_gpu.cpp): what a handle allocates and
when, where it falls back, and which factors and coarse operators its solves are given."""

import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2203_11938_amd import sim as S, workloads as W

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2203_11938_amd", "csrc")
COUNTS = ("mallocs", "factorised", "passes", "stale_factors", "coarse", "iterated", "stale_coarse")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("api") / "libfake_sim.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", "-I" + CSRC, "-I" + os.path.join(ROOT, "include"),
                    os.path.join(HERE, "host", "fake_gpu.cpp"),
                    *(os.path.join(CSRC, f) for f in ("sim_api.cpp", "mesh_prep.cpp", "direct_prep.cpp")),
                    "-Wl,-Bsymbolic", "-o", out], check=True)
    lib = ctypes.CDLL(out)
    lib.fake_memory.argtypes = [ctypes.c_size_t]
    lib.fake_used.restype = ctypes.c_size_t
    lib.sim_destroy.argtypes = [ctypes.c_void_p]
    return lib


class Handle:
    """A handle over one n x n sheet, its calls on host arrays of the right sizes."""

    def __init__(self, lib, n, memory=1 << 34, fail=0, iterations=1000, **options):
        self.lib = lib
        lib.fake_memory(memory)
        lib.fake_fail(fail)
        lib.fake_iterations(iterations)
        opt = S._Options()
        lib.sim_default_options(ctypes.byref(opt))
        opt.precision = S.SIM_FP64
        for k, v in options.items():
            setattr(opt, k, v)
        rest, tris = W.grid_sheet(n)
        tris = np.ascontiguousarray(tris, np.int32)
        rest = np.ascontiguousarray(rest, np.float64)
        mesh = S._Mesh(len(rest), len(tris), tris.ctypes.data_as(ctypes.POINTER(ctypes.c_int32)))
        mat = S._Material(1e3, 1e-4, 0.1)
        self.h = ctypes.c_void_p()
        self.status = lib.sim_create(ctypes.byref(mesh), rest.ctypes.data_as(ctypes.c_void_p), None, 0,
                                     ctypes.byref(mat), ctypes.c_double(0.01), ctypes.byref(opt),
                                     ctypes.byref(self.h))
        lib.fake_fail(0)
        self.x0 = np.zeros((3, len(rest)))
        self.created = self.counts()

    def counts(self):
        c = (ctypes.c_int * 8)()
        self.lib.fake_counts(c, 1)
        return dict(zip(COUNTS, c))

    def rollout(self, steps, start, stream=None):
        self.x0[0, 0] = start
        st = self.lib.sim_rollout(self.h, steps, self.x0.ctypes.data_as(ctypes.c_void_p), None, None,
                                  None, None, None, 0, None, stream)
        assert st == S.SIM_OK
        return self.counts()

    def adjoint(self, stream=None):
        assert self.lib.sim_adjoint(self.h, None, None, None, None, None, None, stream) == S.SIM_OK
        return self.counts()

    def stats(self):
        s = S._Stats()
        assert self.lib.sim_sync_status(self.h) == S.SIM_OK
        assert self.lib.sim_get_stats(self.h, ctypes.byref(s)) == S.SIM_OK
        return s

    def close(self):
        if self.h:
            self.lib.sim_destroy(self.h)
        self.h = None


@pytest.fixture
def make(lib):
    made = []

    def make(*a, **kw):
        made.append(Handle(lib, *a, **kw))
        return made[-1]

    yield make
    for h in made:
        h.close()
    assert lib.fake_used() == 0


ITERATIVE = dict(cg_tol=1e-13)   # below what the direct solver is given; all else the same


def iterative_bytes(make, n, **options):
    h = make(n, **ITERATIVE, **options)
    assert h.status == S.SIM_OK
    b = h.stats().device_bytes
    h.close()
    return b


def test_solves_are_direct_and_the_adjoint_reuses_the_factors(make):
    h = make(24, max_steps=6)
    assert h.rollout(6, 10.0)["factorised"] == 6
    assert h.adjoint()["factorised"] == 6       # the first shows that factors are worth keeping
    for k in range(2):
        assert h.rollout(6, 20.0 + 100 * k)["factorised"] == 6
        c = h.adjoint()
        assert (c["factorised"], c["passes"], c["stale_factors"], c["iterated"]) == (0, 6, 0, 0)


def test_a_handle_without_room_for_the_direct_solver_is_iterative(make):
    """The direct solver's memory is optional: where an allocation of its set-up fails, the
    handle is created all the same, gives back what that set-up took, and solves
    iteratively."""
    need = iterative_bytes(make, 48, max_steps=4)
    for spare in (0, 1 << 18, 1 << 20, 4 << 20):
        h = make(48, memory=need + spare, max_steps=4)
        assert h.status == S.SIM_OK, spare
        assert h.stats().device_bytes == need and h.lib.fake_used() == need
        c = h.rollout(4, 1.0)
        assert (c["factorised"], c["iterated"]) == (0, 4)
        h.close()
    # one allocation after the other of those an iterative handle does not make
    h = make(48, max_steps=4, **ITERATIVE)
    first = h.created["mallocs"] + 1
    h.close()
    h = make(48, max_steps=4)
    last = h.created["mallocs"]
    h.close()
    assert last > first
    for nth in range(first, last + 1):
        h = make(48, fail=nth, max_steps=4)
        assert h.status == S.SIM_OK, nth
        assert h.stats().device_bytes == need and h.lib.fake_used() == need
        assert h.rollout(4, 1.0)["iterated"] == 4
        h.close()


def test_kept_factors_stay_within_a_fifth_of_the_memory_free_at_the_first_adjoint(make):
    """The bound holds over the handle's life, and calls in the steady state allocate
    nothing: a handle that does not get a slot per step does not ask again."""
    h = make(24, max_steps=60)
    room = h.lib.fake_used() + 5 * 20 * 330000   # a fifth: some 20 factors of this sheet
    h.lib.fake_memory(room)
    held = h.stats().device_bytes
    fifth = (room - h.lib.fake_used()) / 5
    h.rollout(60, 1.0)
    first = h.adjoint()
    got = h.stats().device_bytes - held
    assert 0 < got <= fifth
    for k in range(6):
        a, b = h.rollout(60, 100.0 * k), h.adjoint()
        assert h.stats().device_bytes - held == got
        assert a["mallocs"] == 0 and b["mallocs"] == 0
        assert b["stale_factors"] == 0 and b["iterated"] == 0
        assert 0 < b["passes"] < 60


def test_kept_factors_follow_growing_windows(make):
    """A program that lengthens its rollouts gets a slot per step as long as they fit."""
    h = make(24, max_steps=64)
    for n in range(1, 65):
        h.rollout(n, 1000.0 * n)
        h.adjoint()
    assert h.rollout(64, 5.0)["factorised"] == 64
    c = h.adjoint()
    assert (c["factorised"], c["passes"], c["mallocs"]) == (0, 64, 0)


@pytest.mark.parametrize("keep_all", [0, 1])
def test_checkpointed_adjoint_reuses_what_the_option_keeps(make, keep_all):
    """By default the factors of one segment are kept: the recompute factorises the other
    segments' steps again, the adjoint reuses those. With coarse_keep_all every step's are:
    nothing after the forward pass factorises, from the first adjoint on."""
    h = make(24, max_steps=20, checkpoint_every=5, coarse_keep_all=keep_all)
    for k in range(3):
        assert h.rollout(20, 100.0 * k)["factorised"] == 20
        c = h.adjoint()
        assert c["stale_factors"] == 0 and c["iterated"] == 0
        if keep_all:
            assert (c["factorised"], c["passes"]) == (0, 36)
        elif k > 0:
            # the last segment's are all kept; of the others the ends are not recomputed
            assert (c["factorised"], c["passes"]) == (15, 21)


def test_keep_all_keeps_what_fits(make):
    """Where not every step's factor fits, the recompute still reuses the last ones'."""
    h = make(24, max_steps=20, checkpoint_every=5)
    few = h.stats().device_bytes
    h.rollout(20, 1.0)
    h.adjoint()
    factor = (h.stats().device_bytes - few) // 4
    h.close()
    h = make(24, max_steps=20, checkpoint_every=5, coarse_keep_all=1)
    rest = h.stats().device_bytes - 19 * factor
    h.close()
    # a fifth of what is free holds 11 more
    h = make(24, memory=rest + 5 * 11 * factor + 64, max_steps=20, checkpoint_every=5, coarse_keep_all=1)
    assert h.stats().device_bytes == rest + 11 * factor
    h.rollout(20, 1.0)
    c = h.adjoint()
    # steps 9 to 20 are kept: 1 to 4 and 6 to 8 are recomputed, with 5 and the adjoint's own
    # reuse of those left
    assert 0 < c["factorised"] < 15 and c["factorised"] + c["passes"] == 36
    assert c["stale_factors"] == 0 and c["iterated"] == 0 and c["mallocs"] == 0


@pytest.mark.parametrize("checkpoint", [0, 10])
def test_direct_handles_hold_no_coarse_operators_of_steps(make, checkpoint):
    """The kept coarse operators belong to the iterative solver: a handle solved directly
    takes no memory for them, and its capacity costs a state and statistics a step; one
    left to the iterative solver for want of memory keeps them."""
    V = 48 * 48
    held = {}
    for steps in (100, 200):
        h = make(48, max_steps=steps, checkpoint_every=checkpoint)
        held[steps] = h.stats().device_bytes
        assert h.stats().coarse_store_slots == (checkpoint or steps)
        h.close()
    states = 10 if checkpoint else 100
    assert held[200] - held[100] <= states * 48 * V + 100 * 36
    need = iterative_bytes(make, 48, max_steps=100, checkpoint_every=checkpoint)
    h = make(48, memory=need, max_steps=100, checkpoint_every=checkpoint)
    assert h.stats().coarse_store_slots == (checkpoint or 100)
    h.rollout(100, 1.0)
    c = h.adjoint()
    assert c["iterated"] > 0 and c["stale_coarse"] == 0
    assert c["coarse"] == (90 if checkpoint else 0)   # the rest is kept


@pytest.mark.parametrize("options", [dict(), ITERATIVE])
def test_a_replayed_adjoint_uses_operators_of_its_own_steps(make, options):
    """A captured adjoint holds, per step, whether it forms the step's factor (or coarse
    operator) or takes the one kept. With checkpointing it leaves others behind than it
    found, so a second call after the same rollout is another sequence, not a replay."""
    h = make(24, max_steps=20, checkpoint_every=5, graph=1, **options)
    for k in range(4):
        h.rollout(20, 100.0 * k)
        for call in range(3):
            c = h.adjoint()
            assert (c["stale_factors"], c["stale_coarse"]) == (0, 0), (k, call)
            assert options or c["iterated"] == 0
    # each kind of call is replayed when it comes again
    assert h.stats().graph_replays >= 3


@pytest.mark.parametrize("checkpoint", [0, 5])
def test_captures_of_the_caller(lib, make, checkpoint):
    """Rollout and adjoint in a graph of the caller's, together and each alone beside direct
    calls: no solve is given another state's factor."""
    def captured(h, *calls):
        st = ctypes.c_void_p(id(h) & 0xfffffff0)
        g, e = ctypes.c_void_p(), ctypes.c_void_p()
        lib.hipStreamBeginCapture(st, 0)
        for f in calls:
            f(st)
        lib.hipStreamEndCapture(st, ctypes.byref(g))
        lib.hipGraphInstantiate(ctypes.byref(e), g, None, None, ctypes.c_size_t(0))

        def replay():
            lib.hipGraphLaunch(e, None)
            return h.counts()
        return replay

    def sound(c):
        assert c["stale_factors"] == 0 and c["iterated"] == 0
        return c

    h = make(24, max_steps=20, checkpoint_every=checkpoint)
    h.rollout(20, 1.0)
    sound(h.adjoint())
    both = captured(h, lambda st: h.rollout(20, 0.0, st), lambda st: h.adjoint(st))
    for k in range(3):
        h.x0[0, 0] = 10.0 + 50 * k
        c = sound(both())
        assert c["passes"] > 0        # the adjoint reuses what the rollout formed
    # a captured rollout, direct adjoints
    roll = captured(h, lambda st: h.rollout(20, 0.0, st))
    for k in range(3):
        h.x0[0, 0] = 1000.0 + 50 * k
        sound(roll())
        sound(h.adjoint())
        sound(h.adjoint())
    # direct rollouts, a captured adjoint
    h.rollout(20, 2000.0)
    adj = captured(h, lambda st: h.adjoint(st))
    for k in range(3):
        h.rollout(20, 3000.0 + 50 * k)
        sound(adj())
        sound(adj())
    # back to direct calls
    h.rollout(20, 4000.0)
    sound(h.adjoint())


@pytest.mark.parametrize("tol,corrections", [(1e-8, 0), (5e-10, 0), (5e-12, 6)])
def test_corrections_run_where_a_sheet_is_left(make, tol, corrections):
    """Below 1e-9 an unaccepted solve is corrected, below 1e-11 every one is; the launches
    that follow an accepted solve find no sheet left and do nothing."""
    h = make(24, max_steps=6, cg_tol=tol)
    c = h.rollout(6, 1.0)
    assert (c["factorised"], c["passes"], c["coarse"], c["iterated"]) == (6, corrections, 0, 0)


@pytest.mark.parametrize("n,few,many", [(17, 6, 20), (32, 16, 30), (64, 34, 60), (111, 55, 100)])
def test_solver_follows_the_iterations_it_would_take(make, n, few, many):
    """A handle whose solves the iterative solver would end within a few iterations (loose
    tolerances, short steps) is left to it: a factorisation would take longer. The counts
    stand on either side of the measured break-even."""
    for iterations, direct in ((few, False), (many, True)):
        h = make(n, iterations=iterations, max_steps=2)
        assert h.stats().cg_iters_max == 0 and h.stats().device_status == 0   # nothing left behind
        c = h.rollout(2, 1.0)
        assert (c["factorised"], c["iterated"]) == ((2, 0) if direct else (0, 2)), iterations
        h.close()
    h = make(4, iterations=4, max_steps=2)      # a single front
    assert h.rollout(2, 1.0)["factorised"] == 2
