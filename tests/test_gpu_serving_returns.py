"""Returns of requests that finish on one tick, where they do not fit the server's
page-locked memory (2^17 doubles) at once: a request across its end, a request
larger than it, one that ends on it, an empty one.  Rewards are counts times
constants and actions do not depend on the batch, so the returns equal, bitwise,
those of a server that runs the requests one after the other.
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu
flock = pytest.importorskip("paper_2207_03945_amd")

HALF = 1 << 16


@pytest.mark.parametrize("sizes", [(HALF, HALF, 300), (100_000, 0, 50_000), (1, 2 * HALF + 77)])
def test_returns_over_several_pieces(sizes):
    v = 8
    w, b = workloads.xavier_weights([v, 64, 64, 2], seed=3)
    pol = flock.Policy(w, b)
    reqs = []
    for k, n in enumerate(sizes):
        box = float(np.float32(4.0 * np.sqrt(max(n, 100))))
        reqs.append((flock.Params(n_agents=n, box=box, sectors=v),
                     workloads.uniform_state(n, box, seed=70, env=k)))
    together = flock.Server(pol, 1 << 30, max_slots=8)
    ids = [together.submit(p, st, 2)[0] for p, st in reqs]
    for _ in range(2):
        together.tick()
    for i, (p, st) in zip(ids, reqs):
        alone = flock.Server(pol, 1 << 30, max_slots=8)
        j = alone.submit(p, st, 2)[0]
        while alone.poll(j)[0] != alone.FINISHED:
            alone.tick()
        got, want = together.result(i), alone.result(j)
        assert got.shape == (p.n_agents,) and np.array_equal(got, want)
        if p.n_agents > 1000:
            assert np.count_nonzero(want) > p.n_agents // 2
    torch.cuda.synchronize()
