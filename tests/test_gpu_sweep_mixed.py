"""Lane-group sweeps whose waves hold agents of several envs that differ in everything
an env may: box, vision and collision ranges, field of view, columns' reach (single
cells among grids), chasers.  Such a wave takes each agent's values from its own env;
equal bits with the same envs stepped alone with one lane per agent.
"""
from __future__ import annotations

import math

import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu

flock = pytest.importorskip("paper_2207_03945_amd")

# n, box, radius, collide, reach, degrees: at four lanes a wave holds sixteen agents
ENVS = [(5, 20.0, 8.0, 2.0, 0, 250.0), (6, 40.0, 8.0, 1.0, 2, 0.0), (3, 30.0, 3.0, 0.5, 1, 90.0),
        (1, 64.0, 8.0, 2.0, 1, 250.0), (70, 20.0, 6.0, 1.5, 0, 300.0), (9, 16.0, 5.0, 1.0, 1, 0.0),
        (70, 28.0, 8.0, 2.0, 2, 120.0), (2, 100.0, 8.0, 4.0, 2, 250.0), (40, 17.0, 8.0, 0.1, 0, 200.0),
        (4, 25.0, 2.0, 2.0, 1, 250.0), (33, 40.0, 13.0, 6.0, 2, 359.0), (130, 30.0, 7.5, 2.5, 1, 10.0)]


def make(form, k, chase):
    n, box, radius, collide, reach, fov = ENVS[k]
    kw = dict(sectors=form["sectors"], fov=math.radians(fov) if form["fov"] else 0.0)
    flags = flock.ENV_FLAG_COUNTS
    if form["tag"]:
        flags |= flock.ENV_FLAG_TAG
        kw["n_chasers"] = chase
    env = flock.Env(flock.Params(n_agents=n, box=box, radius=radius, collide=collide,
                                 cell_reach=reach, flags=flags, **kw))
    env.set_state(*[torch.from_numpy(a).cuda() for a in workloads.uniform_state(n, box, seed=9, env=k)])
    env.reset()
    return env


@pytest.mark.parametrize("lanes", [4, 16])
@pytest.mark.parametrize("sectors,fov,tag", [(16, False, False), (20, False, False), (8, True, False),
                                             (30, True, False), (9, False, True), (16, True, True)])
def test_mixed_waves(sectors, fov, tag, lanes):
    form = dict(sectors=sectors, fov=fov, tag=tag)
    ks = list(range(len(ENVS))) * 2
    alone = [make(form, k, ENVS[k][0] // (2 + k % 3)) for k in ks]
    batch = flock.Batch([make(form, k, ENVS[k][0] // (2 + k % 3)) for k in ks])
    for e in alone:
        e.set_sweep_lanes(1)
    batch.set_sweep_lanes(lanes)
    off = batch.offsets
    obs, rew = torch.empty(batch.n, batch.d, device="cuda"), torch.empty(batch.n, device="cuda")
    for t in range(3):
        acts = [workloads.random_actions(e.n, seed=4, step=t, env=i) for i, e in enumerate(alone)]
        batch.step(torch.from_numpy(np.concatenate(acts)).cuda(), obs, rew)
        for i, e in enumerate(alone):
            o, r = e.step(torch.from_numpy(acts[i]).cuda())
            assert torch.equal(o, obs[off[i]:off[i + 1]]), f"view, env {i} {ENVS[ks[i]]}, step {t}"
            assert torch.equal(r, rew[off[i]:off[i + 1]]), f"reward, env {i} {ENVS[ks[i]]}, step {t}"
            for u, w in zip(e.counts(), batch.envs[i].counts()):
                assert torch.equal(u, w), f"counts, env {i} {ENVS[ks[i]]}, step {t}"
