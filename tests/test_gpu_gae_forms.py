"""Advantages on either side of 2 M agent-steps, from which the next chunk's loads go
ahead of the recurrence: equal bits with the FP64 recurrence, rounded once, for agents
at the start, the end and the middle, and the same whatever else the launch holds.
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

from oracle import rl

pytestmark = pytest.mark.gpu

flock = pytest.importorskip("paper_2207_03945_amd")


@pytest.mark.parametrize("T,n", [(15, 133_333), (15, 133_334), (16, 124_999), (16, 125_000),
                                 (33, 60_606), (33, 60_607), (128, 15_624), (128, 15_625),
                                 (1, 1_999_999), (1, 2_000_000)])
def test_forms(T, n):
    g = torch.Generator("cuda").manual_seed(T)
    rew = torch.randn(T, n, device="cuda", generator=g)
    val = torch.randn(T + 1, n, device="cuda", generator=g)
    gamma, lam = np.float32(0.99), np.float32(0.95)
    adv, ret = flock.gae(rew, val, gamma, lam)
    pick = torch.cat([torch.arange(65), torch.arange(n // 2, n // 2 + 65), torch.arange(n - 65, n)])
    rows = [t.cpu()[:, pick].numpy() for t in (rew, val)]
    for got, want in zip((adv, ret), rl.gae(*rows, float(gamma), float(lam))):
        assert np.array_equal(got.cpu()[:, pick].numpy(), want.astype(np.float32))
    part = flock.gae(rew[:, :1000].contiguous(), val[:, :1000].contiguous(), gamma, lam)
    assert torch.equal(part[0], adv[:, :1000]) and torch.equal(part[1], ret[:, :1000])
