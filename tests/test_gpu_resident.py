"""The resident kernel (whole CG iterations of a single solve in one launch,
Sec. 3, Listing 2) against the passes whose arithmetic it repeats.

* every grid and precision it is built for, and the grids at its edges, plain
  and preconditioned: the iterates and counts are bitwise those of the passes
  (mode 3);
* solves longer than a launch, iteration limits, b = 0 and refused data;
* an iteration that reduces r.r so far that the difference of the sums
  cancels (a right-hand side close to an eigenvector): r.r is summed anew;
* the masked operator (fracture driver), more solves at once than XCDs, and
  the fallback when a meeting gives up.

The results are compared for equality, so there is no tolerance to choose,
except against the dense solution: the solves' certified 1e-10.
"""

import threading

import numpy as np
import pytest

from paper_1305_3625_amd import binding
from workloads import spectrum, padded_instance, periodic_instance, fracture_instance
from oracle import kernel_table, solve_dense
from gpu_util import dev, host, relerr, banner

pytestmark = pytest.mark.gpu


def _run(plan, inst, mode, precision, tol=1e-10, maxit=10000, x0=None):
    import torch
    plan.set_grid_sync(mode)
    x = torch.zeros((inst["L"], inst["L"]), dtype=torch.float64, device="cuda")
    info = plan.solve(dev(inst["d"]), dev(inst["b"]), x, x0=x0, tol=tol, maxit=maxit, precision=precision,
                      raise_on_error=False)
    return host(x), info


@pytest.mark.parametrize("precision", [binding.FP64, binding.MIXED])
@pytest.mark.parametrize("L,padded", [(16, 1), (32, 1), (64, 1), (128, 1), (256, 1), (512, 1), (1024, 1),
                                      (32, 0), (64, 0), (128, 0), (256, 0), (512, 0), (1024, 0)])
def test_resident_bitwise_as_passes(L, padded, precision):
    inst = (padded_instance if padded else periodic_instance)(L, [7, L, padded], eps=1e-3)
    plan = binding.Plan(L, padded, inst["ghat"])
    plan.set_engine(binding.ENGINE_MULTIPASS)
    banner("resident", L, padded, precision)
    w = dev(np.random.default_rng([7, 1, L]).standard_normal((L, L)))
    for kw in (dict(), dict(maxit=3), dict(x0=w)):
        out = {m: _run(plan, inst, m, precision, **kw) for m in (3, 1)}
        print(kw.keys(), [o[1]["iterations"] for o in out.values()], out[1][1]["error_bound"])
        assert out[1][1]["status"] == out[3][1]["status"]
        assert out[1][1]["iterations"] == out[3][1]["iterations"]
        assert out[1][1]["error_bound"] == out[3][1]["error_bound"]
        assert np.array_equal(out[1][0], out[3][0])
    assert plan.grid_sync(precision) != binding.GRID_FELL_BACK
    plan.close()


@pytest.mark.parametrize("precision", [binding.FP64, binding.MIXED])
@pytest.mark.parametrize("L,padded", [(16, 1), (64, 1), (128, 1), (256, 1), (512, 1), (1024, 1), (2048, 1),
                                      (64, 0), (256, 0), (1024, 0), (2048, 0)])
def test_resident_precond_bitwise_as_passes(L, padded, precision):
    """The preconditioned iteration: modes without the resident kernel (0 and
    3) run its passes."""
    inst = (padded_instance if padded else periodic_instance)(L, [7, 6, L, padded], eps=1e-3)
    plan = binding.Plan(L, padded, inst["ghat"])
    plan.set_precond(binding.PRECOND_CIRCULANT)
    banner("resident-precond", L, padded, precision)
    w = dev(np.random.default_rng([7, 7, L]).standard_normal((L, L)))
    for kw in (dict(), dict(maxit=3), dict(x0=w)):
        out = {m: _run(plan, inst, m, precision, **kw) for m in (3, 1)}
        print(kw.keys(), [o[1]["iterations"] for o in out.values()], out[1][1]["error_bound"])
        assert out[1][1]["status"] == out[3][1]["status"]
        assert out[1][1]["iterations"] == out[3][1]["iterations"]
        assert out[1][1]["error_bound"] == out[3][1]["error_bound"]
        assert np.array_equal(out[1][0], out[3][0])
    assert plan.grid_sync(precision) != binding.GRID_FELL_BACK
    plan.close()


def test_resident_many_iterations_and_limits():
    """More iterations than one launch runs (256), maxit inside a launch, b =
    0, invalid data, and a start vector with a NaN."""
    L = 32
    inst = padded_instance(L, [7, 8], eps=1e-3)
    plan = binding.Plan(L, 1, inst["ghat"] ** 3 + 1e-4)  # ill-conditioned: hundreds of iterations
    plan.set_engine(binding.ENGINE_MULTIPASS)
    banner("resident-many", L)
    for precision in (binding.FP64, binding.MIXED):
        out = {m: _run(plan, inst, m, precision, maxit=700) for m in (3, 1)}
        print([o[1] for o in out.values()])
        assert out[1][1]["iterations"] == out[3][1]["iterations"] > 256
        assert out[1][1]["status"] == out[3][1]["status"]
        assert np.array_equal(out[1][0], out[3][0])
    zero = dict(inst, b=np.zeros((L, L)))
    x, info = _run(plan, zero, 1, binding.MIXED)
    assert info["status"] == binding.OK and info["iterations"] == 0 and not x.any()
    bad = dict(inst, d=inst["d"].copy())
    bad["d"][3, 5] = -1.0
    import torch
    for x0, i, want in ((None, bad, binding.EINVAL), (np.full((L, L), np.nan), inst, binding.EBREAKDOWN)):
        x = torch.zeros((L, L), dtype=torch.float64, device="cuda")
        with pytest.raises(binding.FftcgError) as e:
            plan.solve(dev(i["d"]), dev(i["b"]), x, x0=None if x0 is None else dev(x0), precision=binding.MIXED)
        assert e.value.status == want
    plan.close()


@pytest.mark.parametrize("precision", [binding.FP64, binding.MIXED])
def test_resident_residual_falls_at_once(precision):
    """Uniform d and b = 1 plus a thousandth of noise on a periodic grid: the
    first iteration removes the constant, and r.r with it to 1e-6."""
    L = 16
    rng = np.random.default_rng([7, 2])
    g = spectrum(64, 1e-2)
    b = 1.0 + 1e-3 * rng.standard_normal((64, 64))
    inst = dict(L=64, d=np.ones((64, 64)), b=b)
    plan = binding.Plan(64, 0, g)
    plan.set_engine(binding.ENGINE_MULTIPASS)
    banner("resident-fall", 64, precision)
    x, info = _run(plan, inst, 1, precision)
    y, info3 = _run(plan, inst, 3, precision)
    assert info["status"] == binding.OK and info["iterations"] == info3["iterations"]
    assert np.array_equal(x, y)
    # diagonal in Fourier space
    ref = np.real(np.fft.ifft2(np.fft.fft2(b) / (1.0 + g)))
    assert relerr(x, ref) <= 1e-10
    plan.close()
    inst = dict(periodic_instance(L, [7, 3]), padded=0)
    ref = solve_dense(kernel_table(inst["ghat"]), inst["d"], inst["b"], 0)
    plan = binding.Plan(L, 0, inst["ghat"])
    x, info = _run(plan, inst, 1, precision)
    assert relerr(x, ref) <= 1e-10
    plan.close()


def test_resident_masked():
    import torch
    L, steps = 128, 4
    inst = fracture_instance(1, L=L)
    plan = binding.Plan(L, 1, spectrum(2 * L, 1e-3))
    banner("resident-masked", L)
    out = {}
    for mode in (3, 1):
        plan.set_grid_sync(mode)
        f = torch.zeros((L, L), dtype=torch.float64, device="cuda")
        st, broken, dbreak, iters = plan.fracture(inst["k"], dev(inst["t"]), f, steps, tol=1e-9)
        assert st == binding.OK
        out[mode] = (host(f), broken, dbreak, iters)
    assert all(np.array_equal(a, b) for a, b in zip(out[1], out[3]))
    plan.close()


@pytest.mark.parametrize("L,count", [(128, 10), (512, 3)])
def test_resident_solves_at_once(L, count):
    """More solves at once than XCDs (or than one, where a solve takes the
    device): those without room run the passes; every result is the same as
    alone.  A fresh plan each time: its workspaces are made while other
    solves run, and nothing of that may reach into a solve (the clearing of
    the partial sums once did)."""
    import torch
    insts = [padded_instance(L, [7, 4, k], eps=1e-3) for k in range(count)]
    plan = binding.Plan(L, 1, insts[0]["ghat"])
    banner("resident-at-once", L, count)
    ref = [_run(plan, i, 3, binding.MIXED)[0] for i in insts]
    D, B = [dev(i["d"]) for i in insts], [dev(i["b"]) for i in insts]
    for _ in range(6):
        plan.close()
        plan = binding.Plan(L, 1, insts[0]["ghat"])
        X = [torch.zeros((L, L), dtype=torch.float64, device="cuda") for _ in insts]
        streams = [torch.cuda.Stream() for _ in insts]
        infos = [None] * count
        torch.cuda.synchronize()

        def work(k):
            infos[k] = plan.solve(D[k], B[k], X[k], tol=1e-10, precision=binding.MIXED, stream=streams[k],
                                  raise_on_error=False)

        th = [threading.Thread(target=work, args=(k,)) for k in range(count)]
        for t in th:
            t.start()
        for t in th:
            t.join()
        torch.cuda.synchronize()
        fell = plan.grid_sync(binding.MIXED) == binding.GRID_FELL_BACK
        print("fell back:", fell)
        for k in range(count):
            assert infos[k]["status"] == binding.OK
            if fell:
                assert relerr(host(X[k]), ref[k]) <= 2e-10
            else:
                assert np.array_equal(host(X[k]), ref[k])
    plan.close()


@pytest.mark.parametrize("L,padded", [(64, 0), (512, 1)])
def test_resident_gives_up(L, padded):
    """A wait limit of zero: the meetings give up and the solve is repeated
    with the separate update kernel, bitwise that kernel's result."""
    inst = (padded_instance if padded else periodic_instance)(L, [7, 5, L], eps=1e-3)
    plan = binding.Plan(L, padded, inst["ghat"])
    plan.set_engine(binding.ENGINE_MULTIPASS)
    banner("resident-gives-up", L)
    x0, info0 = _run(plan, inst, 0, binding.FP64)
    x2, info2 = _run(plan, inst, 2, binding.FP64)
    assert info2["status"] == binding.OK
    assert plan.grid_sync(binding.FP64) == binding.GRID_FELL_BACK
    assert np.array_equal(x0, x2) and info0["iterations"] == info2["iterations"]
    plan.close()
