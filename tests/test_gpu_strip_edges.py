"""The strip sort where it can go wrong: agents crossing the box's periodic edge in
both directions in numbers, every strip count from one up, strips that hold more
records than their block keeps in registers, plans below and above one block per CU.

A twin whose state is set again before every step sorts by the general path (its
records are not in cell order), so views, rewards and states must equal it bitwise.
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu
flock = pytest.importorskip("paper_2207_03945_amd")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def state(n, box, kind, seed):
    g = np.random.default_rng(seed)
    x, y, th, sp = workloads.uniform_state(n, box, seed=seed)
    if kind == "edge":       # most agents within a step of x = 0, heading either way
        k = n - n // 8
        x[:k] = np.where(g.random(k) < 0.7, g.random(k) * 0.8, box - g.random(k) * 0.8)
        th[:k] = np.where(g.random(k) < 0.3, 0.1, np.pi + 0.1)
    elif kind == "dense":    # a few columns hold most of them
        k = n - n // 4
        x[:k] = 0.4 * box + g.random(k) * 0.1 * box
    x = np.clip(x, 0.0, np.nextafter(np.float32(box), np.float32(0)))
    return x.astype(np.float32), y, th.astype(np.float32), sp


CASES = [
    ([(256, 64.0)], "uniform"), ([(600, 64.0)], "edge"), ([(1100, 64.0)], "edge"),
    ([(5000, 316.0)], "edge"), ([(20000, 316.0)], "dense"), ([(9000, 300.0)], "edge"),
    ([(20000, 600.0), (3000, 60.0), (700, 300.0)], "edge"),
    ([(6000, 300.0)] * 40, "dense"), ([(6000, 300.0)] * 40, "edge"),
]


@pytest.mark.parametrize("sizes,kind", CASES)
def test_strip_sort_equals_general_path(sizes, kind):
    states = [state(n, b, kind, seed=60 + k) for k, (n, b) in enumerate(sizes)]
    pair = []
    for _ in range(2):
        envs = [flock.Env(flock.Params(n_agents=n, box=b, sectors=16, flags=1)) for n, b in sizes]
        for e, st in zip(envs, states):
            e.set_state(*[dev(a) for a in st])
            e.reset()
        pair.append((envs, flock.Batch(envs)))
    (ea, ba), (eb, bb) = pair
    n = ba.n
    obs = [torch.empty(n, 16, device="cuda") for _ in range(2)]
    rew = [torch.empty(n, device="cuda") for _ in range(2)]
    for t in range(4):
        act = dev(np.concatenate([workloads.random_actions(m, seed=61, step=t, env=k)
                                  for k, (m, _) in enumerate(sizes)]))
        for e in eb:
            e.set_state(*e.get_state())
        ba.step(act, obs[0], rew[0])
        bb.step(act, obs[1], rew[1])
        torch.cuda.synchronize()
        assert torch.equal(obs[0], obs[1]) and torch.equal(rew[0], rew[1]), t
        for x, y in zip(ea, eb):
            for u, v in zip(x.get_state(), y.get_state()):
                assert torch.equal(u, v), t
