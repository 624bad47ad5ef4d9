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

// log2 of the strips in a run, or -1 for one run per XCD, which gathers an env's
// actions in one or two L2s (four envs of 200,000 agents 44 us per sort, in runs
// of 8 strips 57).  An env of more strips than two XCDs' share spans several of
// them anyway, and where its agents crowd into some of its columns one XCD would
// have them all: such plans deal out short runs (one env of 2 million agents in
// an eighth of its box 1,240 us with one run per XCD, 262 with runs of 8, 264 to 266
// of 1, 4 and 16; all over its box 139 and 138).
constexpr int kShortRun = 3;
constexpr int strip_run_log(int S, int most_of_one_env, int cus) {
    return S > cus && most_of_one_env > 2 * ((S + kXcds - 1) / kXcds) ? kShortRun : -1;
}

// Strips of one XCD's only run.
constexpr unsigned strip_run(int S, int ahead) { return (unsigned)(S - ahead + kXcds - 1) / kXcds; }

// Blocks of a launch of S strips (the last few may have none).
constexpr unsigned strip_blocks(int S, int ahead, int run_log) {
    const unsigned round = kXcds << (run_log < 0 ? 0 : run_log);
    return ahead + ((unsigned)(S - ahead) + round - 1) / round * round;
}

// The place of block b's strip among the S strips in launch order (S and more:
// none): [0, ahead) the envs' first strips, then the others, env by env; run =
// strip_run(S, ahead).
constexpr int strip_place(unsigned b, int ahead, unsigned run, int run_log) {
    if (b < (unsigned)ahead) return (int)b;
    const unsigned r = b - ahead, x = r % kXcds, k = r / kXcds;
    if (run_log < 0) return (int)(ahead + x * run + k);
    return (int)(ahead + ((((k >> run_log) * kXcds) + x) << run_log) + (k & ((1u << run_log) - 1)));
}

// Which of its env's strips the one at `place` is; strip_base: strips of the
// envs before env.
constexpr int strip_in_env(int place, int ahead, int env, int strip_base) {
    if (place < ahead) return 0;
    return ahead ? place - ahead - (strip_base - env) + 1 : place - strip_base;
}

}  // namespace flock
