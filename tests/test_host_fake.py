"""The host side of plans and single solves (paper_1305_3625_amd/csrc/
fftcg_host.cpp and fused.hip, unmodified) on a simulated device, on the CPU
(tests/fake_hip/fake_host.cpp): which route a solve takes when others are in
flight or a meeting gives up.  A solve is held in flight by blocking inside
its launch.

A resident kernel keeps its CUs for a whole solve, and every launch of
another solve's passes whose workgroups do not fit beside it waits for its
end: no resident solve starts beside passes above M = 1024, and at M = 1024
those in FP64 or with the preconditioner start alone."""

import ctypes
import os
import subprocess
import threading

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BUILD = os.path.join(ROOT, "_build", "fake")
P, I, D, S = ctypes.c_void_p, ctypes.c_int, ctypes.c_double, ctypes.c_size_t
FP64, MIXED = 0, 1
APPLY, RESIDENT, CHUNK, SEPARATE, FUSED, CAPTURED_RECORD = range(6)
ROUTES = ("fused", "resident", "turn", "folded", "separate")
HOOK = ctypes.CFUNCTYPE(None, I, I, I)


class Info(ctypes.Structure):
    _fields_ = [("status", I), ("iterations", I), ("iterations_literal", I), ("checks", I),
                ("true_relres", D), ("error_bound", D), ("lambda_lb", D), ("device_ms", D)]


class Fake:
    def __init__(self):
        os.makedirs(BUILD, exist_ok=True)
        out = os.path.join(BUILD, "libfftcg_host_fake.so")
        csrc = os.path.join(ROOT, "paper_1305_3625_amd", "csrc")
        subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fPIC", "-shared", "-Wall", "-Wno-unused-function",
                        "-I" + os.path.join(ROOT, "tests", "fake_hip"), "-I" + os.path.join(ROOT, "include"),
                        "-I" + csrc, os.path.join(csrc, "fftcg_host.cpp"),
                        os.path.join(ROOT, "tests", "fake_hip", "fake_host.cpp"), "-x", "c++",
                        os.path.join(csrc, "fused.hip"), "-o", out, "-lpthread"], check=True)
        self.lib = lib = ctypes.CDLL(out)
        lib.fftcg_plan.argtypes = [I, I, P, ctypes.POINTER(P)]
        lib.fftcg_plan_destroy.argtypes = [P]
        for n in ("fftcg_plan_set_engine", "fftcg_plan_set_precond", "fftcg_plan_set_grid_sync"):
            getattr(lib, n).argtypes = [P, I]
        lib.fftcg_plan_get_grid_sync.argtypes = [P, I, ctypes.POINTER(I)]
        lib.fftcg_plan_get_solve_routes.argtypes = [P, P]
        lib.fftcg_plan_info.argtypes = [P, P, P, P, ctypes.POINTER(S)]
        lib.fftcg_apply.argtypes = [P, I, P, P, P, P]
        lib.fftcg_solve.argtypes = [P, I, P, P, P, D, I, P, ctypes.POINTER(Info), P]
        lib.fake_fail_memset.argtypes = [S]
        lib.fake_meet_bytes.restype = S
        lib.fake_set_hook.argtypes = [P]
        self.gates = {}  # thread -> (kind, entered, go on)
        self.hook = HOOK(self._hook)
        lib.fake_set_hook(ctypes.cast(self.hook, P))

    def _hook(self, kind, M, precision):
        g = self.gates.get(threading.get_ident())
        if g is not None and (g[0] is None or g[0] == kind) and not g[1].is_set():
            g[1].set()
            assert g[2].wait(20)

    def plan(self, L, padded, precond=0):
        M = 2 * L if padded else L
        h = P()
        g = np.ones((M, M))
        assert self.lib.fftcg_plan(L, padded, g.ctypes.data_as(P), ctypes.byref(h)) == 0
        assert self.lib.fftcg_plan_set_precond(h, precond) == 0
        return Plan(self, h, L)


class Plan:
    def __init__(self, fake, h, L):
        self.f, self.lib, self.h, self.L = fake, fake.lib, h, L

    def routes(self):
        r = (ctypes.c_ulonglong * 5)()
        assert self.lib.fftcg_plan_get_solve_routes(self.h, r) == 0
        return dict(zip(ROUTES, r))

    def solve(self, precision=MIXED, in_place=False, stream=None):
        """Solves with a right-hand side of ones; returns the route taken
        (and those of the plan's solves that ended meanwhile)."""
        n = self.L * self.L
        d, b = np.ones(n), np.ones(n)
        x = np.full(n, 7.0) if in_place else np.zeros(n)
        info = Info()
        p = lambda a: a.ctypes.data_as(P)  # noqa: E731
        before = self.routes()
        st = self.lib.fftcg_solve(self.h, precision, p(d), p(b), p(x) if in_place else None, 1e-8, 100, p(x),
                                  ctypes.byref(info), stream)
        assert st == 0 and info.status == 0 and (x == 0.5).all()
        after = self.routes()
        return [k for k in ROUTES if after[k] > before[k]]

    def close(self):
        assert self.lib.fftcg_plan_destroy(self.h) == 0


class InFlight:
    """A call in a thread of its own, held inside its first launch of `kind`
    (None: of any)."""

    def __init__(self, fake, call, kind=None):
        self.fake, self.call, self.kind = fake, call, kind
        self.entered, self.go, self.out = threading.Event(), threading.Event(), None

    def _run(self):
        self.fake.gates[threading.get_ident()] = (self.kind, self.entered, self.go)
        try:
            self.out = self.call()
        finally:
            self.fake.gates.pop(threading.get_ident())
            self.entered.set()

    def __enter__(self):
        self.t = threading.Thread(target=self._run)
        self.t.start()
        assert self.entered.wait(20)
        return self

    def __exit__(self, *a):
        self.go.set()
        self.t.join()


@pytest.fixture(scope="module")
def fake():
    return Fake()


@pytest.mark.parametrize("L,padded,precond,want", [(64, 0, 0, "resident"), (16, 0, 0, "fused"), (128, 1, 0, "resident"),
                                                   (512, 1, 1, "resident"), (1024, 1, 0, "turn"),
                                                   (2048, 1, 1, "turn"), (8, 1, 1, "separate")])
def test_alone(fake, L, padded, precond, want):
    p = fake.plan(L, padded, precond)
    assert p.solve() == [want]
    p.close()


def test_small_solve_without_room_is_fused(fake):
    """AUTO at M <= 64: nine solves at once, and one beside a solve that has
    the whole device, leave no XCD; the fused engine needs none."""
    p = fake.plan(64, 0)
    held = [InFlight(fake, p.solve, RESIDENT).__enter__() for _ in range(8)]
    try:
        assert p.solve(FP64) == ["fused"]
    finally:
        for h in held:
            h.__exit__()
    assert p.routes()["resident"] == 8
    q = fake.plan(512, 1)
    with InFlight(fake, q.solve, RESIDENT):
        assert p.solve() == ["fused"]
    assert p.solve() == ["resident"]
    p.close()
    q.close()


@pytest.mark.parametrize("in_place", [False, True])
def test_small_solve_that_gave_up_is_fused(fake, in_place):
    """A meeting that gave up: the repeat is the fused engine's, and so are
    the plan's later solves."""
    p = fake.plan(32, 1)
    fake.lib.fake_give_up(1)
    try:
        assert p.solve(in_place=in_place) == ["fused"]
    finally:
        fake.lib.fake_give_up(0)
    assert p.solve() == ["fused"]
    st = I()
    assert fake.lib.fftcg_plan_get_grid_sync(p.h, MIXED, ctypes.byref(st)) == 0 and st.value == 3
    assert fake.lib.fftcg_plan_set_grid_sync(p.h, 1) == 0
    assert p.solve() == ["resident"]
    p.close()


def _hold(fake, p, kind=None, **kw):
    return InFlight(fake, lambda: p.solve(**kw), kind)


@pytest.mark.parametrize("big,precond", [((2048, 1), 0), ((2048, 1), 1), ((1024, 1), 0), ((4096, 0), 1)])
def test_no_resident_solve_beside_large_passes(fake, big, precond):
    p, small, mid, tiny = fake.plan(*big, precond), fake.plan(128, 1), fake.plan(512, 1), fake.plan(64, 0)
    with _hold(fake, p):
        for q in (small, mid):
            # a grid that fills the device leaves no room for their barriers either
            assert q.solve() == ["turn" if big[0] == 1024 else "separate"]
        assert tiny.solve() == ["fused"]
    for q in (small, mid, tiny):
        assert q.solve() == ["resident"]
    for q in (p, small, mid, tiny):
        q.close()


def test_resident_solves_beside_each_other(fake):
    """On one XCD each: eight, and the ninth by passes; while that runs, an XCD
    that becomes free is taken again.  On the whole device: one, alone."""
    p, q = fake.plan(128, 1), fake.plan(512, 1, 1)
    held = [_hold(fake, p, RESIDENT).__enter__() for _ in range(8)]
    with _hold(fake, p, CHUNK) as ninth:
        held.pop().__exit__()
        assert p.solve() == ["resident"]
        assert q.solve() == ["separate"]  # (preconditioned at M = 1024: no turns)
    assert "turn" in ninth.out
    for h in held:
        h.__exit__()
    with _hold(fake, q, RESIDENT):
        with _hold(fake, q, SEPARATE) as other:
            assert p.solve() == ["turn"]
    assert other.out == ["separate"]
    with _hold(fake, q, SEPARATE, precision=FP64) as first:  # alone: not the passes
        pass
    assert first.out == ["resident"] and q.solve() == ["resident"]
    p.close()
    q.close()


@pytest.mark.parametrize("precision,precond", [(FP64, 0), (MIXED, 0), (FP64, 1)])
def test_resident_beside_small_passes(fake, precision, precond):
    """Up to M = 512 beside any number of solves with M <= 1024 that run the
    passes; the plain FP32 solve of M = 1024 beside two, FP64 and the
    preconditioned alone."""
    bg, p, q, h = fake.plan(512, 1, precond), fake.plan(256, 1), fake.plan(512, 1), fake.plan(512, 1, 1)
    assert fake.lib.fftcg_plan_set_grid_sync(bg.h, 3) == 0  # its solves run the passes
    held = []
    for n in range(1, 6):
        held.append(_hold(fake, bg, precision=precision).__enter__())
        assert p.solve() == ["resident"] and p.solve(FP64) == ["resident"]
        assert q.solve() == ["resident" if n <= 2 else "turn"]
        assert q.solve(FP64) == ["turn"] and h.solve() == ["separate"]
    for x in held:
        x.__exit__()
    assert q.solve(FP64) == ["resident"] and h.solve() == ["resident"]
    for x in (bg, p, q, h):
        x.close()


def test_barriers_share_the_device(fake):
    """Barriers of grids that do not fit the device together are not tried:
    the later solve runs the separate update, and its plan does not fall
    back."""
    p, q, r = fake.plan(2048, 1), fake.plan(1024, 1), fake.plan(128, 1)
    with _hold(fake, p, CHUNK) as first:
        assert p.solve() == ["separate"] and q.solve() == ["separate"]
    assert "turn" in first.out and p.solve() == ["turn"]
    held = [_hold(fake, q, CHUNK).__enter__() for _ in range(4)]  # four fit
    assert q.solve() == ["separate"]
    for h in held:
        h.__exit__()
        assert "turn" in h.out
    with _hold(fake, r, RESIDENT):
        assert p.solve() == ["separate"] and q.solve() == ["separate"]
    assert p.solve() == ["turn"] and q.solve() == ["turn"]
    st = I()
    for x in (p, q):
        assert fake.lib.fftcg_plan_get_grid_sync(x.h, MIXED, ctypes.byref(st)) == 0 and st.value == 4
        x.close()
    r.close()


def test_products_in_flight(fake):
    """A product returns before its passes have run; on the solve's own
    stream they come before it, on another they run beside it."""
    p, q = fake.plan(2048, 1), fake.plan(128, 1)
    a = [np.zeros(2048 * 2048) for _ in range(3)]
    ptr = [v.ctypes.data_as(P) for v in a]
    fake.lib.fake_hold_events(1)
    try:
        assert fake.lib.fftcg_apply(p.h, FP64, *ptr, P(16)) == 0
        assert q.solve(stream=P(32)) == ["turn"]
        assert q.solve(stream=P(16)) == ["resident"]
    finally:
        fake.lib.fake_hold_events(0)
    assert q.solve(stream=P(32)) == ["resident"]
    p.close()
    assert q.solve(stream=P(32)) == ["resident"]
    # products of M <= 1024: as small passes
    p, r = fake.plan(512, 1), fake.plan(512, 1)
    fake.lib.fake_hold_events(1)
    try:
        assert fake.lib.fftcg_apply(p.h, FP64, *ptr, P(16)) == 0
        assert q.solve(stream=P(32)) == ["resident"] and r.solve(stream=P(32)) == ["resident"]
        assert r.solve(FP64, stream=P(32)) == ["turn"] and r.solve(FP64, stream=P(16)) == ["resident"]
    finally:
        fake.lib.fake_hold_events(0)
    for x in (p, q, r):
        x.close()


def test_captured_products_are_not_queried(fake):
    """The event of a product that is being captured must not be queried (the
    query can end the capture): not after it, and not while it is recorded
    over that of an earlier product still in flight."""
    p, q = fake.plan(2048, 1), fake.plan(128, 1)
    a = [np.zeros(2048 * 2048) for _ in range(3)]
    ptr = [v.ctypes.data_as(P) for v in a]
    fake.lib.fake_hold_events(1)
    try:
        assert fake.lib.fftcg_apply(p.h, FP64, *ptr, P(16)) == 0
        assert q.solve(stream=P(32)) == ["turn"]
        n = fake.lib.fake_captured_queries()
        fake.lib.fake_capture(1)
        with InFlight(fake, lambda: fake.lib.fftcg_apply(p.h, FP64, *ptr, P(16)), CAPTURED_RECORD) as c:
            fake.lib.fake_capture(0)
            q.solve(stream=P(32))
        assert c.out == 0
        q.solve(stream=P(32))
        assert fake.lib.fake_captured_queries() == n
    finally:
        fake.lib.fake_capture(0)
        fake.lib.fake_hold_events(0)
    p.close()
    q.close()


def test_resident_words_cleared_or_not_used(fake):
    """Meetings take any word at or above their token for an arrival, so the
    words must be clear: a workspace whose clearing failed does not keep them
    as cleared ones."""
    p = fake.plan(128, 1)
    fake.lib.fake_fail_memset(fake.lib.fake_meet_bytes())
    assert p.solve() == ["turn"]
    for _ in range(2):
        assert p.solve() == ["resident"] and fake.lib.fake_words_clear() == 1
    p.close()


@pytest.mark.parametrize("L,padded", [(64, 0), (256, 1), (2048, 0)])
def test_device_bytes_counts_the_product_buffer(fake, L, padded):
    """device_bytes of a plan includes the half spectrum of its products, with
    the 128 bytes behind every column that the buffer holds."""
    M = 2 * L if padded else L
    p = fake.plan(L, padded)
    n = S()
    assert fake.lib.fftcg_plan_info(p.h, None, None, None, ctypes.byref(n)) == 0
    quarter = (M // 2 + 1) ** 2
    tables = 2 * M * 12 + (M // 2) * (M // 2 + 1) * 12 + (M // 2 + 1) * 12
    fused = 2 * M * 12 + quarter * 12 if M <= 256 else 0
    assert n.value == tables + fused + (M // 2) * (L * 16 + 128)
    p.close()


@pytest.mark.parametrize("in_place", [False, True])
def test_resident_launch_that_left_no_state(fake, in_place):
    """The state belongs to the launch whose mark it carries: one that an
    earlier solve left (done, solved) is not taken for this one's."""
    p = fake.plan(128, 1)
    assert p.solve() == ["resident"]
    fake.lib.fake_give_up(4)
    try:
        assert p.solve(in_place=in_place) == ["separate"]
    finally:
        fake.lib.fake_give_up(0)
    p.close()
