// strip_order.h -- the order in which the strip sort's blocks take the strips.
//
// Blocks go to the XCDs round robin, and each XCD takes a run of consecutive
// strips, so that an env's strips share one or two XCDs' L2.
//
// A strip waits for a word that its env's first strip publishes.  Where all of
// the launch's blocks are resident at once they all start at once, and any
// order serves.  Where they are not, a first strip at the end of one XCD's run
// would start long after the strips of its env at the head of the next run,
// which would hold their places and wait (four envs of 4 million agents, 3,996
// strips: 131 ms instead of 3.8).  There the launch's first blocks take
// the envs' first strips, which wait for nothing, and the runs hold the others.
// (Always doing so costs the runs' locality: 40 envs of 50,000 agents, 1,000
// strips, sorted in 66 us instead of 62.)
#pragma once

namespace flock {

constexpr int kXcds = 8;  // MI355X: accelerator dies (XCDs), each with its own L2

// Whether a launch takes blocks of 1,024 threads: while a CU of the device has at
// most one block, its latency counts (10,000 agents in 9 strips: 3 us less than
// with 512 threads), and fewer CUs would take several rounds of such blocks.
constexpr bool strips_wide(int S, int cus) { return S <= cus; }

// First strips at the launch's head: all n_envs of them, or none where all
// blocks are among the `resident` ones that the device holds at once.
constexpr int strips_ahead(int S, int n_envs, int resident) {
    return n_envs > 1 && S + kXcds > resident ? n_envs : 0;
}

// Strips of one XCD's run.
constexpr unsigned strip_run(int S, int ahead) { return (unsigned)(S - ahead + kXcds - 1) / kXcds; }

// Blocks of a launch of S strips (the last few may have none).
constexpr unsigned strip_blocks(int S, int ahead) { return ahead + strip_run(S, ahead) * kXcds; }

// The place of block b's strip among the S strips in launch order (S and more:
// none): [0, ahead) the envs' first strips, then the others, env by env; run =
// strip_run(S, ahead).
constexpr int strip_place(unsigned b, int ahead, unsigned run) {
    if (b < (unsigned)ahead) return (int)b;
    const unsigned r = b - ahead;
    return (int)(ahead + r % kXcds * run + r / kXcds);
}

// Which of its env's strips the one at `place` is; strip_base: strips of the
// envs before env.
constexpr int strip_in_env(int place, int ahead, int env, int strip_base) {
    if (place < ahead) return 0;
    return ahead ? place - ahead - (strip_base - env) + 1 : place - strip_base;
}

}  // namespace flock
