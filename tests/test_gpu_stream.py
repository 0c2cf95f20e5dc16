"""Grids whose vectors pass through the last-level cache (L >= 4096), at the
periodic one whose W has no padding behind its tiles (L = M = 4096); the other
two are in test_gpu_large.

* one operator product against the oracle's direct O(L^2) sum at sampled
  outputs, FP64 within 1e-13 and FP32 within 1e-6 of max|x| sum|g| (the bounds
  the other largest grids are held to);
* short solves, plain and preconditioned, with the separate passes (mode 0)
  and as AUTO runs them: the residual that the solve reports against the
  oracle's FP64 residual of its x, to 1e-9 of |b| (FP64 products on both
  sides).
"""

import numpy as np
import pytest

from paper_1305_3625_amd import binding
from workloads import spectrum
from oracle import kernel_table, apply_direct_at, apply_fft
from gpu_util import dev, host, banner

pytestmark = pytest.mark.gpu


def test_periodic_L4096():
    L = 4096
    gh = spectrum(L, 1e-3)
    g = kernel_table(gh)
    rng = np.random.default_rng([97, L])
    d = rng.uniform(0.5, 1.5, (L, L))
    b = rng.standard_normal((L, L))
    plan = binding.Plan(L, 0, gh)
    rows = list(rng.integers(0, L, 12)) + [0, L - 1, L // 2, 1]
    cols = list(rng.integers(0, L, 12)) + [0, L - 1, L // 2, L - 2]
    ref = apply_direct_at(g, d, b, 0, rows, cols)
    scale = np.abs(b).max() * np.abs(g).sum()
    for prec, tol in ((binding.FP64, 1e-13), (binding.MIXED, 1e-6)):
        banner("stream-apply", L, prec)
        y = dev(np.zeros((L, L)))
        plan.apply(dev(d), dev(b), y, precision=prec)
        assert np.max(np.abs(host(y)[rows, cols] - ref)) / scale <= tol
    nb = np.linalg.norm(b)
    for precond in (binding.PRECOND_NONE, binding.PRECOND_CIRCULANT):
        plan.set_precond(precond)
        for prec in (binding.MIXED, binding.FP64):
            for mode in (1, 0):
                banner("stream-solve", L, precond, prec, mode)
                plan.set_grid_sync(mode)
                x = dev(np.zeros((L, L)))
                info = plan.solve(dev(d), dev(b), x, tol=1e-8, maxit=4, precision=prec, raise_on_error=False)
                assert info["iterations"] <= 4
                r = np.linalg.norm(b - apply_fft(gh, d, host(x), 0)) / nb
                print(prec, precond, mode, info["iterations"], info["true_relres"], r)
                assert abs(r - info["true_relres"]) <= 1e-9
    plan.close()
