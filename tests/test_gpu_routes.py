"""What a solve runs (fftcg_plan_get_solve_routes), by grid, precision and
preconditioner, on the device the library is built for: the tests that
compare the resident kernel and the turn passes with the passes whose
arithmetic they repeat compare nothing where both sides take one route.

* every grid the resident kernel is built for, and its neighbours;
* the folded update, the turn pass and the preconditioned turns above;
* giving up (mode 2) on the preconditioned paths too, also for a warm start
  in place: the repeat is the separate passes', bitwise;
* r.r falling at once where the turn pass runs: its second barrier.
"""

import numpy as np
import pytest

from paper_1305_3625_amd import binding
from workloads import spectrum, padded_instance, periodic_instance
from gpu_util import dev, host, relerr, banner

pytestmark = pytest.mark.gpu


def _route(plan, inst, precision, x0=None, tol=1e-8, maxit=10000):
    """Solves, and returns (x, info, the route taken)."""
    import torch
    before = plan.solve_routes()
    L = inst["L"]
    x = torch.zeros((L, L), dtype=torch.float64, device="cuda") if x0 is None else x0
    info = plan.solve(dev(inst["d"]), dev(inst["b"]), x, x0=x0, tol=tol, maxit=maxit, precision=precision,
                      raise_on_error=False)
    after = plan.solve_routes()
    got = [k for k in after for _ in range(after[k] - before[k])]
    assert len(got) == 1, (before, after)
    return host(x), info, got[0]


RESIDENT = [(16, 1), (32, 1), (64, 1), (128, 1), (256, 1), (512, 1), (32, 0), (64, 0), (128, 0), (256, 0), (512, 0),
            (1024, 0)]


@pytest.mark.parametrize("precision", [binding.FP64, binding.MIXED])
@pytest.mark.parametrize("precond", [binding.PRECOND_NONE, binding.PRECOND_CIRCULANT])
@pytest.mark.parametrize("L,padded", RESIDENT)
def test_resident_route(L, padded, precond, precision):
    inst = (padded_instance if padded else periodic_instance)(L, [31, L, padded], eps=1e-2)
    plan = binding.Plan(L, padded, inst["ghat"])
    plan.set_precond(precond)
    banner("route-resident", L, padded, precond, precision)
    for mode, want in ((1, ("resident",)), (3, ("folded", "separate", "fused")), (0, ("separate", "fused"))):
        plan.set_grid_sync(mode)
        x, info, got = _route(plan, inst, precision, maxit=4)
        assert got in want, (mode, got)
        if mode == 3:
            small = plan.M <= 64 and precond == binding.PRECOND_NONE  # (AUTO)
            assert got == ("fused" if small else ("separate" if precond else "folded"))
    plan.close()


@pytest.mark.parametrize("L,padded,precision,precond,want", [
    (8, 1, binding.FP64, 0, "fused"), (8, 1, binding.MIXED, 1, "separate"), (16, 0, binding.MIXED, 0, "fused"),
    (1024, 1, binding.MIXED, 0, "turn"), (1024, 1, binding.FP64, 0, "turn"),
    (1024, 1, binding.MIXED, 1, "turn"), (1024, 1, binding.FP64, 1, "separate"),
    (2048, 1, binding.MIXED, 0, "turn"), (2048, 1, binding.MIXED, 1, "turn"), (2048, 1, binding.FP64, 1, "separate"),
    (2048, 0, binding.MIXED, 0, "turn"), (2048, 0, binding.MIXED, 1, "turn"),
])
def test_passes_route(L, padded, precision, precond, want):
    inst = (padded_instance if padded else periodic_instance)(L, [32, L, padded], eps=1e-2)
    plan = binding.Plan(L, padded, inst["ghat"])
    plan.set_precond(precond)
    banner("route-passes", L, padded, precision, precond)
    x, info, got = _route(plan, inst, precision, maxit=4)
    assert got == want and plan.grid_sync(precision) != binding.GRID_FELL_BACK
    plan.set_grid_sync(0)
    x, info, got = _route(plan, inst, precision, maxit=4)
    assert got == ("fused" if want == "fused" else "separate")
    plan.close()


@pytest.mark.parametrize("L,precision,precond", [(128, binding.FP64, 0), (128, binding.MIXED, 1),
                                                 (512, binding.FP64, 1), (1024, binding.MIXED, 1),
                                                 (2048, binding.MIXED, 1)])
def test_gives_up_and_repeats(L, precision, precond):
    inst = padded_instance(L, [33, L], eps=1e-3)
    plan = binding.Plan(L, 1, inst["ghat"])
    plan.set_precond(precond)
    banner("route-gives-up", L, precision, precond)
    w = np.random.default_rng([33, 1, L]).standard_normal((L, L))
    out = {}
    for mode in (0, 2):
        for kind in ("zero", "in place"):
            plan.set_grid_sync(mode)
            x, info, got = _route(plan, inst, precision, x0=dev(w) if kind == "in place" else None)
            assert got == "separate" and info["status"] == binding.OK
            assert (plan.grid_sync(precision) == binding.GRID_FELL_BACK) == (mode == 2)
            out[mode, kind] = (x, info["iterations"], info["error_bound"])
    for kind in ("zero", "in place"):
        a, b = out[0, kind], out[2, kind]
        assert a[1:] == b[1:] and np.array_equal(a[0], b[0])
    plan.close()


def test_residual_falls_at_once_in_turn_pass():
    """Uniform d and b = 1 plus a thousandth of noise: the first iteration
    takes r.r down to 1e-6 of itself, the difference of the sums cancels, and
    the pass sums r.r anew behind a second barrier.  Mode 3 has the same
    arithmetic in separate launches; the answer is diagonal in Fourier space."""
    L = 2048
    rng = np.random.default_rng([34, L])
    g = spectrum(L, 1e-2)
    b = 1.0 + 1e-3 * rng.standard_normal((L, L))
    inst = dict(L=L, d=np.ones((L, L)), b=b)
    plan = binding.Plan(L, 0, g)
    banner("route-turn-fall", L)
    out = {}
    for mode, want in ((1, "turn"), (3, "folded")):
        plan.set_grid_sync(mode)
        out[mode] = _route(plan, inst, binding.MIXED, tol=1e-8)
        assert out[mode][1]["status"] == binding.OK and out[mode][2] == want
    assert out[1][1]["iterations"] == out[3][1]["iterations"]
    assert np.array_equal(out[1][0], out[3][0])
    ref = np.real(np.fft.ifft2(np.fft.fft2(b) / (1.0 + g)))
    assert relerr(out[1][0], ref) <= 1e-8
    plan.close()


@pytest.mark.parametrize("precision", [binding.FP64, binding.MIXED])
@pytest.mark.parametrize("L,padded", [(128, 1), (256, 1), (512, 1), (256, 0), (512, 0)])
def test_refused_solve_runs_turn_pass(L, padded, precision):
    """Beside a large solve's passes the resident kernel does not start; such
    a solve has the turn pass, with bitwise the result of mode 3."""
    import threading
    import torch
    inst = (padded_instance if padded else periodic_instance)(L, [35, L, padded], eps=1e-3)
    big = padded_instance(2048, [35, 1], eps=1e-4)
    plan, other = binding.Plan(L, padded, inst["ghat"]), binding.Plan(2048, 1, big["ghat"])
    other.set_grid_sync(0)  # no barrier: it leaves the device's share to the others
    banner("route-refused", L, padded, precision)
    assert plan.grid_sync(precision) == binding.GRID_ON_TURN
    plan.set_grid_sync(3)
    want, winfo, got = _route(plan, inst, precision)
    assert got == "folded"
    plan.set_grid_sync(1)
    D, B = dev(big["d"]), dev(big["b"])
    X = torch.zeros((2048, 2048), dtype=torch.float64, device="cuda")
    d, b = dev(inst["d"]), dev(inst["b"])
    torch.cuda.synchronize()
    before = plan.solve_routes()
    th = threading.Thread(target=lambda: other.solve(D, B, X, tol=1e-12, maxit=200, precision=binding.FP64,
                                                     stream=torch.cuda.Stream(), raise_on_error=False))
    th.start()
    s, n = torch.cuda.Stream(), 0
    while th.is_alive() or n == 0:
        x = torch.zeros((L, L), dtype=torch.float64, device="cuda")
        torch.cuda.current_stream().synchronize()
        info = plan.solve(d, b, x, tol=1e-8, precision=precision, stream=s)
        assert np.array_equal(host(x), want) and info["iterations"] == winfo["iterations"]
        n += 1
    th.join()
    after = plan.solve_routes()
    print(n, after)
    assert plan.grid_sync(precision) == binding.GRID_ON_TURN
    assert after["turn"] > before["turn"] and after["folded"] == before["folded"]
    assert after["separate"] == before["separate"]
    plan.close()
    other.close()


@pytest.mark.parametrize("L,padded,precision,precond", [(128, 1, binding.FP64, 1), (256, 0, binding.FP64, 1),
                                                        (128, 1, binding.FP64, 0), (128, 1, binding.MIXED, 1),
                                                        (64, 0, binding.FP64, 0)])
def test_eight_resident_solves_on_eight_xcds(L, padded, precision, precond):
    """Eight threads solve at once, each on a stream of its own: every solve
    finds an XCD that no other holds, whatever XCD the stream's queue begins
    with (where two shared one, workgroups of both kept each other out, and the
    meetings gave up)."""
    import threading
    import torch
    inst = (padded_instance if padded else periodic_instance)(L, [36, L, padded], eps=1e-3)
    plan = binding.Plan(L, padded, inst["ghat"])
    plan.set_precond(precond)
    banner("route-eight", L, padded, precision, precond)
    want, winfo, got = _route(plan, inst, precision)
    assert got == "resident"
    D, B = [dev(inst["d"]) for _ in range(8)], [dev(inst["b"]) for _ in range(8)]
    X = [torch.zeros((L, L), dtype=torch.float64, device="cuda") for _ in range(8)]
    streams = [torch.cuda.Stream() for _ in range(8)]
    torch.cuda.synchronize()
    before = plan.solve_routes()

    def work(k):
        for _ in range(15):
            plan.solve(D[k], B[k], X[k], tol=1e-8, precision=precision, stream=streams[k])

    th = [threading.Thread(target=work, args=(k,)) for k in range(8)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    torch.cuda.synchronize()
    after = plan.solve_routes()
    print(after)
    assert plan.grid_sync(precision) != binding.GRID_FELL_BACK
    assert after["resident"] - before["resident"] == 8 * 15
    assert all(np.array_equal(host(x), want) for x in X)
    plan.close()
