// rl_kernels.hip -- trajectory processing over an on-device rollout buffer.
//
// Sec. 4.3 and Fig. 5 of arXiv:2207.03945: every agent is an independent PPO
// learner and the simulation's views and rewards feed the learner's
// experience buffer; Sec. 5: t = 128 simulation updates per training step.
// The advantage of each agent is PPO's truncated estimator over the segment,
// bootstrapped with the value of the state after the last step:
//     delta_t = r_t + gamma V_{t+1} - V_t,   A_t = delta_t + gamma lambda A_{t+1},
//     A_T = 0,   R_t = A_t + V_t.
// One thread per agent walks t backwards; rows t of the [T][n] buffers are
// contiguous over agents, so every load and store is coalesced.  The
// recurrence runs in FP64 and each output is rounded once to FP32.  Bound: HBM
// (16 bytes per agent-step) for many agents, the instructions of a wave's T
// steps for few.  So blocks are single waves, one agent a lane, to spread over
// the CUs (4,000 agents, 128 steps: 63 blocks instead of 16, 9.6 -> 8.4 us), and
// the loads of a chunk of steps are issued before its recurrence.  Where the
// inputs exceed what the L2s hold (kAhead, from 2 M agent-steps, 16 MB), the
// next chunk's are issued too: 16,000 agents, 128 steps 12.3 -> 11.7 us; 16,000,
// 500 41 -> 35; 200,000, 16 10.0 -> 9.2; but with 1,000 agents, 128 steps, 9.9
// instead of 8.0.
#include <math.h>

#include "flock_internal.h"

namespace flock {

namespace {

constexpr int kGaeBlock = 64;
constexpr int kChunk = 16;
constexpr int64_t kAheadFrom = 2000000;  // agent-steps

template <bool kAhead>
__global__ __launch_bounds__(kGaeBlock) void k_gae(int T, int64_t n, double gamma, double gl,
                                                   const float *__restrict__ rew,
                                                   const float *__restrict__ val,
                                                   float *__restrict__ adv,
                                                   float *__restrict__ ret) {
    const int64_t i = (int64_t)blockIdx.x * kGaeBlock + threadIdx.x;
    if (i >= n) return;
    double a = 0.0, v_next = (double)val[(size_t)T * n + i];
    auto step = [&](size_t at, float r, float v) {
        const double vt = (double)v;
        a = ((double)r + gamma * v_next - vt) + gl * a;
        adv[at] = (float)a;
        ret[at] = (float)(a + vt);
        v_next = vt;
    };
    // steps t1 - 1 .. t1 - kChunk of both inputs
    auto load = [&](int t1, float (&r)[kChunk], float (&v)[kChunk]) {
#pragma unroll
        for (int u = 0; u < kChunk; ++u) {
            const size_t at = (size_t)(t1 - 1 - u) * n + i;
            r[u] = rew[at];
            v[u] = val[at];
        }
    };
    auto run = [&](int t1, const float (&r)[kChunk], const float (&v)[kChunk]) {
#pragma unroll
        for (int u = 0; u < kChunk; ++u) step((size_t)(t1 - 1 - u) * n + i, r[u], v[u]);
    };
    int t1 = T;  // steps below t1 are left
    if constexpr (kAhead) {
        float r0[kChunk], v0[kChunk], r1[kChunk], v1[kChunk];
        if (t1 >= kChunk) load(t1, r0, v0);  // a whole chunk of them is in (r0, v0)
        while (t1 >= kChunk) {
            if (t1 >= 2 * kChunk) load(t1 - kChunk, r1, v1);
            run(t1, r0, v0);
            t1 -= kChunk;
            if (t1 < kChunk) break;
            if (t1 >= 2 * kChunk) load(t1 - kChunk, r0, v0);
            run(t1, r1, v1);
            t1 -= kChunk;
        }
    } else {
        for (; t1 >= kChunk; t1 -= kChunk) {
            float r[kChunk], v[kChunk];
            load(t1, r, v);
            run(t1, r, v);
        }
    }
    for (int t = t1 - 1; t >= 0; --t) {
        const size_t at = (size_t)t * n + i;
        step(at, rew[at], val[at]);
    }
}

}  // namespace

}  // namespace flock

using namespace flock;

extern "C" {

int rl_gae(int steps, int64_t n, float gamma, float lambda, const float *reward,
           const float *value, float *adv, float *ret, void *stream) {
    if (steps < 1 || n < 0) return set_error(ENV_EINVAL, "need steps >= 1 and n >= 0");
    if (!(gamma >= 0.0f && gamma <= 1.0f) || !(lambda >= 0.0f && lambda <= 1.0f))
        return set_error(ENV_EINVAL, "gamma and lambda must lie in [0, 1]");
    if (n == 0) return ENV_OK;
    if (!reward || !value || !adv || !ret) return set_error(ENV_EINVAL, "NULL buffer");
    const double g = gamma, gl = (double)gamma * (double)lambda;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)((n + kGaeBlock - 1) / kGaeBlock)), dim3(kGaeBlock),
                           0, reinterpret_cast<hipStream_t>(stream), steps, n, g, gl, reward, value,
                           adv, ret);
    };
    if (steps * n < kAheadFrom) go(k_gae<false>);
    else go(k_gae<true>);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return set_error(ENV_EHIP, "rl_gae: %s", hipGetErrorString(e));
    return ENV_OK;
}

}  // extern "C"
