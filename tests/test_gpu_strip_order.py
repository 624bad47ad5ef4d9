"""The strip sort of plans with more strips than can be resident at once (four
blocks on each of 256 compute units), whose strips of every env but its first and
last wait for the count that its first strip publishes.  As the general path, bitwise.
"""
from __future__ import annotations

import pytest

from test_gpu_strip_edges import test_strip_sort_equals_general_path as strip_equals_general

pytestmark = pytest.mark.gpu

# 1,024 columns of 4,096 rows: two columns to a strip whatever the agents
WIDE = 8192.0


@pytest.mark.parametrize("sizes", [
    [(3000, WIDE)] * 3,                                     # 1,536 strips
    [(300, 64.0), (5000, WIDE), (1, 300.0), (9000, WIDE), (2000, 60.0), (700, WIDE)],
])
@pytest.mark.parametrize("kind", ["edge", "uniform"])
def test_more_strips_than_are_resident(sizes, kind):
    strip_equals_general(sizes, kind)


@pytest.mark.parametrize("kind", ["edge", "dense"])
def test_short_runs(kind):
    """Envs that span several XCDs, whose strips are dealt out in runs of eight: alone, and
    beside a small one with more strips than are resident."""
    strip_equals_general([(150_000, 1549.0)], kind)
    strip_equals_general([(9000, 2 * WIDE), (500, 300.0)], kind)
