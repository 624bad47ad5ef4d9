"""Lane-group sweeps over the whole range of sectors and in plans of single cells.

Views of many sectors take most of a block's LDS (more than 64 KiB from 218 sectors
on at four lanes; entries of the neighbour queue narrow where that leaves a compute
unit one more block), and plans whose boxes are all narrower than three columns have
no queue at four lanes.  Equal bits with one lane per agent, which needs neither.
"""
from __future__ import annotations

import math

import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu

flock = pytest.importorskip("paper_2207_03945_amd")

FULL, FOV, TAG, TAG_FOV = "full", "fov", "tag", "tag_fov"


def make(n, box, sectors, form, k):
    kw = dict(sectors=sectors)
    flags = flock.ENV_FLAG_COUNTS
    if form in (FOV, TAG_FOV):
        kw["fov"] = math.radians(250.0)
    if form in (TAG, TAG_FOV):
        flags |= flock.ENV_FLAG_TAG
        kw.update(n_chasers=n // 3, collide=1.0)
    env = flock.Env(flock.Params(n_agents=n, box=box, flags=flags, **kw))
    env.set_state(*[torch.from_numpy(a).cuda() for a in workloads.uniform_state(n, box, seed=5, env=k)])
    env.reset()
    return env


def check_lanes(envs, lanes):
    """envs: (n, box, sectors, form); three steps at `lanes` and at one lane per agent."""
    one, many = [flock.Batch([make(*e, k) for k, e in enumerate(envs)]) for _ in range(2)]
    one.set_sweep_lanes(1)
    many.set_sweep_lanes(lanes)
    out = [(torch.empty(b.n, b.d, device="cuda"), torch.empty(b.n, device="cuda")) for b in (one, many)]
    for t in range(3):
        act = torch.from_numpy(workloads.random_actions(one.n, seed=6, step=t)).cuda()
        for b, o in zip((one, many), out):
            b.step(act, *o)
        assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1]), t
        for e, f in zip(one.envs, many.envs):
            for u, w in zip(e.counts(), f.counts()):
                assert torch.equal(u, w), t


@pytest.mark.parametrize("lanes", [4, 16, 64])
@pytest.mark.parametrize("sectors,form", [
    (51, FULL), (121, FULL), (128, FULL), (128, FOV), (129, FOV), (130, FULL), (171, FOV),
    (217, FULL), (218, FULL), (256, FULL), (256, FOV), (64, TAG), (128, TAG), (128, TAG_FOV)])
def test_many_sectors(sectors, form, lanes):
    check_lanes([(700, 48.0, sectors, form), (300, 40.0, sectors, form)], lanes)


@pytest.mark.parametrize("lanes", [4, 16, 64])
@pytest.mark.parametrize("sectors,form", [(16, FULL), (20, FULL), (128, FULL), (20, FOV), (9, TAG),
                                          (64, TAG_FOV)])
def test_single_cells(sectors, form, lanes):
    check_lanes([(n, box, sectors, form) for n, box in
                 [(1, 20.0), (3, 17.0), (15, 20.0), (64, 23.0), (0, 20.0), (65, 20.0), (300, 18.0)]], lanes)


@pytest.mark.parametrize("sectors", [128, 256])
def test_fused_policy_many_sectors(sectors):
    """At four lanes with the policy in the sweep, whose weights and tiles lie behind the queues."""
    pol = flock.Policy(*workloads.xavier_weights([sectors, 64, 64, 2], seed=2))
    acts = []
    for fused in (False, True):
        b = flock.Batch([make(500, 48.0, sectors, FULL, 0)])
        b.set_sweep_lanes(4)
        b.set_policy_fusion(fused)
        s = torch.cuda.Stream()
        obs, act = torch.zeros(5, b.n, b.d, device="cuda"), torch.empty(4, b.n, 2, device="cuda")
        torch.cuda.synchronize()
        b.rollout(pol, 4, obs, act, torch.empty(4, b.n, device="cuda"), stream=s)
        torch.cuda.synchronize()
        acts.append(act)
    assert torch.equal(*acts) and np.isfinite(acts[0].cpu().numpy()).all()
