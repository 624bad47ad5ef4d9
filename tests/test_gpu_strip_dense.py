"""The strip sort of large envs: the ends of a strip's range searched in several
rounds (an end of more than 512 records after the first), strips of more agents
than fit the block's registers and its list in LDS, or that exceed the list too.
As the general path, bitwise.
"""
from __future__ import annotations

import pytest

from test_gpu_strip_edges import test_strip_sort_equals_general_path as strip_equals_general

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["uniform", "edge", "dense"])
@pytest.mark.parametrize("sizes", [
    [(300_000, 2191.0)],                                    # one column a strip, three ends open
    [(140_000, 900.0), (300, 300.0), (170_000, 1700.0)],    # a list beside small envs
    [(1_100_000, 4196.0)],
])
def test_large_envs(sizes, kind):
    strip_equals_general(sizes, kind)
