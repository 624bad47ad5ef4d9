"""A server may be released while a stream of the process is captured, as when the
interpreter drops it there: the page-locked memory it returns leaves the capture valid.
"""
from __future__ import annotations

import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu

flock = pytest.importorskip("paper_2207_03945_amd")


def server_with_results():
    pol = flock.Policy(*workloads.xavier_weights([8, 64, 64, 2], seed=3))
    srv = flock.Server(pol, 64 << 20)
    p = flock.Params(n_agents=300, box=70.0, sectors=8)
    i, _ = srv.submit(p, workloads.uniform_state(300, 70.0, seed=1), 2)
    while srv.poll(i)[0] != srv.FINISHED:
        srv.tick()
    assert srv.result(i).shape == (300,)
    return srv


def test_release_during_capture():
    x = torch.arange(64, device="cuda", dtype=torch.float32)
    y = torch.zeros_like(x)
    srv = server_with_results()
    torch.cuda.synchronize()
    handle, srv.handle = srv.handle, None       # released below, by hand
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        y.add_(x)
        flock.flockenv.lib().srv_destroy(handle)
        y.mul_(2.0)
    for k in range(3):
        y.fill_(float(k))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, 2.0 * (x + k))
