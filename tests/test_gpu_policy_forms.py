"""The policy kernel's two forms (launches of more than 65,536 rows of up to 32 inputs
keep the weights in LDS), for sampled actions, the critic and tag's two networks: every
row of a launch equals the same row in a launch of a few (bitwise).
"""
from __future__ import annotations

import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu

flock = pytest.importorskip("paper_2207_03945_amd")

ROWS = [65_536, 65_537, 65_553, 131_075]


def views(n, d, seed):
    return torch.rand(n, d, device="cuda", generator=torch.Generator("cuda").manual_seed(seed))


def windows(n):
    return {0, n // 2 + 5, n - 33}


@pytest.mark.parametrize("n", ROWS)
@pytest.mark.parametrize("d", [8, 16, 17, 32, 33])
def test_sample_and_value(d, n):
    pol = flock.Policy(*workloads.xavier_weights([d, 64, 64, 2], seed=d))
    critic = flock.Critic(*workloads.xavier_weights([d, 64, 64, 1], seed=d + 1))
    obs, eps = views(n, d, d), views(n, 2, 3) * 4 - 2
    act, logp = pol.sample(obs, eps, (-1.6, -2.3))
    val = critic.value(obs)
    for lo in windows(n):
        part, noise = obs[lo:lo + 33].contiguous(), eps[lo:lo + 33].contiguous()
        a, p = pol.sample(part, noise, (-1.6, -2.3))
        assert torch.equal(a, act[lo:lo + 33]) and torch.equal(p, logp[lo:lo + 33]), lo
        assert torch.equal(critic.value(part), val[lo:lo + 33]), lo


@pytest.mark.parametrize("sampled", [False, True])
@pytest.mark.parametrize("n", [65_536, 65_553])
def test_tag_rollout(n, sampled):
    """Each type's rows by its own network, in one launch."""
    split, v = n // 3, 8
    p = flock.Params(n_agents=n, box=1100.0, sectors=v, collide=1.0, flags=flock.ENV_FLAG_TAG,
                     n_chasers=split)
    env = flock.Env(p)
    env.set_state(*[torch.from_numpy(a).cuda() for a in workloads.uniform_state(n, 1100.0, seed=8)])
    obs = torch.empty(2, n, p.obs_dim, device="cuda")
    obs[0] = env.reset()
    batch = flock.Batch([env])
    pols = [flock.Policy(*workloads.xavier_weights([p.obs_dim, 64, 64, 2], seed=s)) for s in (1, 2)]
    act, rew, logp = (torch.empty(1, n, *s, device="cuda") for s in ((2,), (), ()))
    eps = (views(n, 2, 4) * 4 - 2)[None] if sampled else None
    ls = (-1.6, -0.7, -1.1, -0.4)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    batch.rollout_tag(*pols, 1, obs, act, rew, logp=logp if sampled else None, eps=eps,
                      log_std=ls if sampled else None, stream=s)
    torch.cuda.synchronize()
    for lo, hi in ((0, 40), (split - 40, split), (split, split + 40), (n - 40, n)):
        pol, sig = (pols[1], ls[2:]) if lo < split else (pols[0], ls[:2])
        part = obs[0, lo:hi].contiguous()
        if sampled:
            a, q = pol.sample(part, eps[0, lo:hi].contiguous(), sig)
            assert torch.equal(q, logp[0, lo:hi])
        else:
            a = pol.forward(part)
        assert torch.equal(a, act[0, lo:hi]), (lo, hi)


@pytest.mark.parametrize("d", [1, 7, 8, 9, 17, 33, 128, 129, 250, 256, 257])
def test_rows_of_any_alignment(d):
    """Rows that start on any four bytes, the last of them at the end of its buffer."""
    pol = flock.Policy(*workloads.xavier_weights([d, 64, 64, 2], seed=d))
    n = 333
    want = pol.forward(views(n, d, d))
    for off in (1, 2, 3):
        flat = torch.empty(off + n * d, device="cuda")
        rows = flat[off:].view(n, d)
        rows.copy_(views(n, d, d))
        assert torch.equal(pol.forward(rows), want), off
