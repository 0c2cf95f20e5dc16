"""Load-step argmax at the edges of its partition, and the checks inside a
server's chunk.

* fftcg_loadstep takes four entries a thread per round, over at most 1,024
  blocks of 256: grids below one block, of exactly one, of several, of
  exactly one round of all blocks and beyond, with equal ratios placed in one
  thread's entries, at block edges and in the last entry (the lowest index
  wins; the result is exact, so no tolerance);
* a chunk of the multi-pass engine holds checks of its own: when a check runs
  decides nothing about the result, so every chunk length gives bitwise the
  same solution, iteration and check counts.
"""

import numpy as np
import pytest
import torch

from paper_1305_3625_amd import binding
from workloads import spectrum, c4_request
from oracle import loadstep_argmax
from gpu_util import banner
from test_gpu_serve import _wait

pytestmark = pytest.mark.gpu


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("L", [2, 16, 32, 64, 1024, 2048])
def test_loadstep_partition_edges(L):
    n = L * L
    blocks = max(1, min(1024, (n + 1023) // 1024))
    step = 256 * blocks
    plan = binding.Plan(L, 1, spectrum(2 * L, 1e-3))
    rng = np.random.default_rng([91, L])
    places = [[n - 1], [0], [n - 1, n - 2], [step - 1, step, 2 * step], [3 + 3 * step, 3 + step],
              [3 * step, 4 * step], [255, 256]]
    for k, idx in enumerate(places):
        idx = [i for i in idx if i < n]
        if not idx:
            continue
        banner("loadstep-edges", L, k)
        x, t, d = rng.standard_normal(n), rng.uniform(0.05, 1.0, n), rng.uniform(0.5, 1.5, n)
        dead = rng.random(n) < 0.3
        x[dead], d[dead] = 5.0e3, 0.0           # broken entries with larger ratios
        for q, i in enumerate(idx):
            s = 2.0 ** (-(q % 3))
            x[i], t[i], d[i] = 1.0e3 * s, s, 1.0
        want = loadstep_argmax(x.reshape(L, L), t.reshape(L, L), d.reshape(L, L))
        assert want == min(idx)
        assert plan.loadstep(_dev(x.reshape(L, L)), _dev(t.reshape(L, L)), _dev(d.reshape(L, L))) == want
    plan.close()


@pytest.mark.parametrize("precond", [0, 1])
def test_chunk_length_changes_nothing(precond):
    plan = binding.Plan(256, 1, spectrum(512, 1e-3))
    if precond:
        plan.set_precond(binding.PRECOND_CIRCULANT)
    reqs = [c4_request(700 + k, 512) for k in range(5)]
    want = None
    for chunk in (1, 5, 6, 10, 11):
        banner("serve-chunk", precond, chunk)
        srv = binding.Server(memory_budget=1 << 30, chunk_iters=chunk, graphs=chunk != 6)
        tks = [srv.submit(plan, r["d"], r["b"], tol=1e-8)[1] for r in reqs]
        got = _wait(srv, tks, 256)
        srv.close()
        res = [(got[tk].x, got[tk].info["iterations"], got[tk].info["checks"]) for tk in tks]
        assert all(got[tk].status == binding.OK for tk in tks)
        if want is None:
            want = res
        for (xa, ia, ca), (xb, ib, cb) in zip(want, res):
            assert ia == ib and ca == cb and np.array_equal(xa, xb), chunk
    plan.close()
