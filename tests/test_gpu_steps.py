"""Load-step argmax at the edges of its partition.

* fftcg_loadstep takes four entries a thread per round, over at most 1,024
  blocks of 256: grids below one block, of exactly one, of several, of
  exactly one round of all blocks and beyond, with equal ratios placed in one
  thread's entries, at block edges and in the last entry (the lowest index
  wins; the result is exact, so no tolerance).
"""

import numpy as np
import pytest
import torch

from paper_1305_3625_amd import binding
from workloads import spectrum
from oracle import loadstep_argmax
from gpu_util import banner

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
