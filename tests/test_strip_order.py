"""Launch order of the strip sort's blocks (csrc/strip_order.h), on the CPU.

Every strip is taken by one block, whatever the device; where a launch's blocks
are not all resident at once, each env's first strip is taken by a block below
all that wait for its word; an env of more strips than two XCDs' share is spread
evenly over the XCDs, stretch by stretch, and fewer than 64 blocks are idle.
The header is plain C++: a small program prints what each block takes.
"""
from __future__ import annotations

import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2207_03945_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "strip_order.h"
int main(int argc, char **argv) {
    static_assert(flock::strips_wide(256, 256) && !flock::strips_wide(257, 256), "");
    static_assert(flock::strips_wide(32, 32) && !flock::strips_wide(200, 32), "a partition's CUs");
    std::vector<int> ns, base, env;   // strips, strips before each env; env of each place
    int resident = 0, cus = 0, S = 0, most = 0;
    if (std::scanf("%d %d", &resident, &cus) != 2) return 1;
    for (int n; std::scanf("%d", &n) == 1; S += n) ns.push_back(n), base.push_back(S), most = n > most ? n : most;
    const int E = (int)ns.size(), ahead = flock::strips_ahead(S, E, resident);
    for (int e = 0; e < ahead; ++e) env.push_back(e);
    for (int e = 0; e < E; ++e) env.insert(env.end(), ns[e] - (ahead ? 1 : 0), e);
    const int run = flock::strip_run_log(S, most, cus);
    for (unsigned b = 0; b < flock::strip_blocks(S, ahead, run); ++b) {
        const int p = flock::strip_place(b, ahead, flock::strip_run(S, ahead), run);
        if (p >= S) std::printf("-1 -1\n");
        else std::printf("%d %d\n", env[p], flock::strip_in_env(p, ahead, env[p], base[env[p]]));
    }
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("strip_order")
    (d / "main.cpp").write_text(PROGRAM)
    exe = str(d / "main")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", f"-I{CSRC}", str(d / "main.cpp"), "-o", exe],
                   check=True)
    return exe


CASES = {
    "one strip": [1], "one env": [707], "ones": [1] * 300, "four large": [999] * 4,
    "twenty": [106] * 20, "first alone": [1, 2000], "last alone": [2000, 1],
    "uneven": [int(k) for k in np.random.default_rng(1).integers(1, 60, 256)],
}


@pytest.mark.parametrize("resident", [64, 128, 512, 1024])
@pytest.mark.parametrize("name", sorted(CASES))
def test_first_strips_come_before_their_waiters(program, name, resident):
    ns = CASES[name]
    out = subprocess.run([program], input=" ".join(map(str, [resident, resident // 4] + ns)), text=True, check=True,
                         capture_output=True).stdout
    taken = [tuple(map(int, line.split())) for line in out.splitlines()]
    block = {t: b for b, t in enumerate(taken) if t != (-1, -1)}
    assert len(taken) - len(block) < 64
    assert sorted(block) == [(e, k) for e, n in enumerate(ns) for k in range(n)]
    if len(taken) > resident:
        for (e, k), b in block.items():
            assert k == 0 or b > block[e, 0], f"strip {k} of env {e} starts before its first"
    for e, n in enumerate(ns):      # the n / 8 strips of any stretch not on one XCD
        if sum(ns) > resident // 4 and n > 2 * ((sum(ns) + 7) // 8) and n >= 256:
            xcd = np.array([block[e, k] % 8 for k in range(1, n)])
            for lo in range(0, n - n // 8, 16):
                assert np.bincount(xcd[lo:lo + n // 8], minlength=8).max() <= n // 8 // 8 + 16
