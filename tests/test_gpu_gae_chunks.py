"""Advantages at the edges of the kernel's chunks (16 steps, two in flight) and
of its one-wave blocks: equal bits with the oracle's FP64 recurrence, rounded once."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from oracle import rl

pytestmark = pytest.mark.gpu

flock = pytest.importorskip("paper_2207_03945_amd")


@pytest.mark.parametrize("n", [1, 63, 64, 65, 200])
@pytest.mark.parametrize("T", [1, 15, 16, 17, 31, 32, 33, 47, 48, 49, 64, 80])
def test_chunk_edges(T, n):
    g = np.random.default_rng([T, n])
    rew = g.standard_normal((T, n)).astype(np.float32)
    val = g.standard_normal((T + 1, n)).astype(np.float32)
    gamma, lam = np.float32(0.99), np.float32(0.95)
    adv, ret = flock.gae(torch.from_numpy(rew).cuda(), torch.from_numpy(val).cuda(), gamma, lam)
    ref_adv, ref_ret = rl.gae(rew, val, float(gamma), float(lam))
    assert np.array_equal(adv.cpu().numpy(), ref_adv.astype(np.float32))
    assert np.array_equal(ret.cpu().numpy(), ref_ret.astype(np.float32))
