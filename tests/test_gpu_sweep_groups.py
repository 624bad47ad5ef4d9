"""Lane-group view sweeps at the edges of their waves and neighbour queue.

A wave holds 64 / lanes agents, of several envs where envs are small, and its
neighbours pass through a queue of 64 and more entries.  Each case batches
envs whose sizes and densities put the edges there (one agent, a wave's
agents +- 1, exactly 64 neighbours, hundreds; a single cell, three columns,
two columns' reach) and compares with the same envs stepped alone with one
lane per agent: equal bits, whatever the lanes; one env also with the oracle.
"""
from __future__ import annotations

import math

import numpy as np
import pytest
import torch

import oracle
import workloads
from parity import EPS_D, EPS_PHI, check_sense

pytestmark = pytest.mark.gpu

flock = pytest.importorskip("paper_2207_03945_amd")

# n, box, reach: tiny envs first, so that one wave holds agents of many
ENVS = [(1, 40.0, 0), (2, 40.0, 0), (3, 24.5, 0), (4, 40.0, 1), (5, 40.0, 2), (15, 33.0, 0),
        (17, 40.0, 0), (63, 17.0, 0), (64, 17.0, 0), (65, 16.5, 0), (66, 40.0, 2), (129, 30.0, 1),
        (500, 40.0, 0), (700, 64.0, 2), (1500, 64.0, 0)]

FORMS = {
    "full16": dict(sectors=16),                       # sectors by octant
    "full20": dict(sectors=20),                       # sectors by arctangent
    "fov30": dict(sectors=30, fov=math.radians(250.0), flags=flock.ENV_FLAG_SPEED_OBS),
    "tag": dict(sectors=16, fov=math.radians(250.0), flags=flock.ENV_FLAG_TAG, collide=1.0),
    "tag_full": dict(sectors=9, flags=flock.ENV_FLAG_TAG, collide=1.0),
}


def make(form, n, box, reach, seed, chasers):
    kw = dict(FORMS[form])
    flags = kw.pop("flags", 0) | flock.ENV_FLAG_COUNTS
    if flags & flock.ENV_FLAG_TAG:
        kw["n_chasers"] = chasers
    env = flock.Env(flock.Params(n_agents=n, box=box, cell_reach=reach, flags=flags, **kw))
    env.set_state(*[torch.from_numpy(a).cuda() for a in workloads.uniform_state(n, box, seed=seed)])
    return env, env.reset()


@pytest.mark.parametrize("form", sorted(FORMS))
@pytest.mark.parametrize("lanes", [4, 16, 64])
def test_groups_equal_one_lane(form, lanes):
    alone, grouped = [], []
    for k, (n, box, reach) in enumerate(ENVS):
        e, _ = make(form, n, box, reach, k, n // 3)
        e.set_sweep_lanes(1)
        alone.append(e)
        grouped.append(make(form, n, box, reach, k, n // 3)[0])
    batch = flock.Batch(grouped)
    batch.set_sweep_lanes(lanes)
    off, G = batch.offsets, batch.n
    obs, rew = torch.empty(G, batch.d, device="cuda"), torch.empty(G, device="cuda")
    for t in range(3):
        acts = [workloads.random_actions(n, seed=3, step=t, env=k)
                for k, (n, _, _) in enumerate(ENVS)]
        batch.step(torch.from_numpy(np.concatenate(acts)).cuda(), obs, rew)
        for k, e in enumerate(alone):
            o, r = e.step(torch.from_numpy(acts[k]).cuda())
            assert torch.equal(o, obs[off[k]:off[k + 1]]), f"view, env {k} {ENVS[k]}, step {t}"
            assert torch.equal(r, rew[off[k]:off[k + 1]]), f"reward, env {k} {ENVS[k]}, step {t}"
            for u, w in zip(e.counts(), grouped[k].counts()):
                assert torch.equal(u, w), f"counts, env {k} {ENVS[k]}, step {t}"
    for u, w in zip(alone, grouped):
        assert torch.equal(u.returns(), w.returns())
    if not FORMS[form].get("flags", 0) & flock.ENV_FLAG_TAG:
        k = len(ENVS) - 1
        p = grouped[k].params
        st = [t.cpu().numpy() for t in grouped[k].get_state()]
        ref = oracle.oracle_sense(st[0], st[1], st[2], p.box, sectors=p.sectors, eps_d=EPS_D,
                                  eps_phi=EPS_PHI, fov=p.fov if p.fov > 0 else oracle.TWO_PI)
        nb, col = (t.cpu().numpy() for t in grouped[k].counts())
        check_sense(ref, obs[off[k]:off[k + 1], :p.sectors].cpu().numpy(),
                    rew[off[k]:off[k + 1]].cpu().numpy(), nb, col, label=f"{form} {lanes}")
