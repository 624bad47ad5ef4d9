"""The strip sort of large envs: the ends of a strip's range searched in several
rounds (an end of more than 512 records after the first), strips of more agents
than fit the block's registers and its list in LDS, or that exceed the list too.
As the general path, bitwise.
"""
from __future__ import annotations

import pytest
import torch

import workloads
from test_gpu_strip_edges import dev, state
from test_gpu_strip_edges import test_strip_sort_equals_general_path as strip_equals_general

pytestmark = pytest.mark.gpu
flock = pytest.importorskip("paper_2207_03945_amd")


@pytest.mark.parametrize("kind", ["uniform", "edge", "dense"])
@pytest.mark.parametrize("sizes", [
    [(300_000, 2191.0)],                                    # one column a strip, three ends open
    [(140_000, 900.0), (300, 300.0), (170_000, 1700.0)],    # a list beside small envs
    [(1_100_000, 4196.0)],
])
def test_large_envs(sizes, kind):
    strip_equals_general(sizes, kind)


@pytest.mark.parametrize("kind", ["edge", "dense", "uniform"])
@pytest.mark.parametrize("sizes", [
    [(5000, 316.0), (9000, 300.0)],                         # blocks of 1,024 threads
    [(140_000, 900.0), (300, 300.0), (170_000, 1700.0)],    # lists, short runs
    [(3000, 8192.0)] * 3,                                   # first strips ahead
    [(6000, 300.0)] * 40,
])
def test_wait_that_runs_out(sizes, kind):
    """Strips that do not wait for the edge crossings count the agents before them
    themselves: bitwise as those that wait."""
    states = [state(n, b, kind, seed=80 + k) for k, (n, b) in enumerate(sizes)]
    batches = []
    for wait in (0, 1 << 14):
        envs = [flock.Env(flock.Params(n_agents=n, box=b, sectors=16)) for n, b in sizes]
        for e, st in zip(envs, states):
            e.set_state(*[dev(a) for a in st])
            e.reset()
        batches.append(flock.Batch(envs))
        batches[-1].set_strip_wait(wait)
    n = batches[0].n
    out = [(torch.empty(n, 16, device="cuda"), torch.empty(n, device="cuda")) for _ in batches]
    for t in range(3):
        act = dev(workloads.random_actions(n, seed=62, step=t))
        for b, o in zip(batches, out):
            b.step(act, *o)
        assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1]), t
    for e, f in zip(batches[0].envs, batches[1].envs):
        for u, v in zip(e.get_state(), f.get_state()):
            assert torch.equal(u, v)
