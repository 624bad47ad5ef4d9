"""Policy launches at the edges of their row loads and of the launch choice.

A lane takes eight inputs of its row in two 16-byte loads, and the last few
one by one; launches of more than 65,536 short rows keep the weights in LDS,
others in registers.  Every row of a launch equals the same row in a launch
of a few rows (bitwise), and the FP64 oracle within the BF16 bound.
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from test_gpu_policy import error_bound, make_policy

pytestmark = pytest.mark.gpu

flock = pytest.importorskip("paper_2207_03945_amd")


@pytest.mark.parametrize("n", [1, 15, 17, 65, 65536, 65553])
@pytest.mark.parametrize("in_dim", [1, 4, 7, 8, 9, 16, 17, 31, 32, 33, 39, 65, 129, 255, 257])
def test_rows(in_dim, n):
    if n > 1000 and in_dim > 65:
        n //= 8                     # (long rows do not switch)
    pol, ws, bs = make_policy(in_dim, seed=in_dim)
    obs = torch.rand(n, in_dim, device="cuda", generator=torch.Generator("cuda").manual_seed(in_dim))
    act = pol.forward(obs)
    for lo in {0, max(0, n - 33), n // 2}:
        part = obs[lo:lo + 33].contiguous()
        assert torch.equal(pol.forward(part), act[lo:lo + 33]), f"rows from {lo}"
    pick = np.unique(np.linspace(0, n - 1, 200).astype(np.int64))
    sub = obs.cpu().numpy()[pick]
    err = np.abs(act.cpu().numpy()[pick].astype(np.float64) - oracle.policy_forward(sub, ws, bs))
    assert (err <= error_bound(sub, ws, bs)).all()
