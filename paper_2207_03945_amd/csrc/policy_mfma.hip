// policy_mfma.hip -- the shared policy network on gfx950 matrix cores.
//
// Sec. 4.3 of arXiv:2207.03945: one policy shared by every agent, each agent
// an independent learner, so the batch axis is the agent axis; Sec. 5: two
// hidden layers of 64 units.  Here: in -> 64 -> 64 -> 2, tanh after every
// layer, the two outputs scaled to the turn / speed-change ranges of Sec. 4.1.
//
// Precision: inputs and weights rounded once to BF16 (round to nearest even),
// products accumulated in FP32 by v_mfma_f32_16x16x32_bf16 from the FP32 biases
// on; each hidden layer's tanh in FP32, rounded to BF16 as the next layer's input.
//
// Layout: see policy_tile.h (one wave per 16-agent tile, hidden units as MFMA
// rows, layer 1 -> layer 2 through a per-wave LDS tile).  Small tiles keep the
// tanh work per lane low (16 values per layer) and give a batch many tiles to
// spread over the CUs.

#include <math.h>
#include <string.h>

#include <algorithm>
#include <string>
#include <vector>

#include "flock_internal.h"
#include "policy_tile.h"

namespace flock {

namespace {

constexpr int kMaxIn = 257;                    // 256 sectors + speed

// kc: chunks of 32 inputs.
PolLayout carve_pol(char *base, int kc) {
    PolLayout l;
    Carver cv{base, 0};
    l.w1 = cv.take<bf16x8>((size_t)kc * 4 * 64);
    l.w2 = cv.take<bf16x8>(2 * 4 * 64);
    l.w3 = cv.take<bf16x8>(2 * 64);
    l.b1 = cv.take<float>(64);
    l.b2 = cv.take<float>(64);
    l.b3 = cv.take<float>(4);
    l.bytes = align_up(cv.off, 256);
    return l;
}

// What the output layer produces.
enum PolOut {
    kMean = 0,    // actor: the mean action, tanh-squashed and scaled
    kSample = 1,  // actor: mean + sigma * eps and the Gaussian log density of the sample
    kValue = 2,   // critic: the linear first output
};

// One network of a launch and its output scales.
struct NetArgs {
    PolLayout P;
    float max_turn, max_dspeed;
    float sig0, sig1;  // exp(log_std) per action dimension (kSample)
    float logp_c;      // -(log_std0 + log_std1) - log(2 pi)
};

struct PolArgs {
    NetArgs net[2];     // tag launches: [0] runners', [1] chasers' (blockIdx.y picks)
    int in_dim, kc;     // kc: chunks of 32 inputs
    int64_t n;
    const float *obs;   // [n][in_dim]; null: each row's env-owned rows (envs)
    float2 *act;        // [n], as obs
    const float2 *eps;  // [n] standard-normal draws (kSample)
    float *logp;        // [n] log density of the sample (kSample, may be null)
    float *val;         // [n] critic value (kValue)
    // batch tables: rows' envs, for env-owned rows and for tag types
    const DevEnv *envs;
    const int32_t *base;
    int n_envs, typed;
};

typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

// Rows are agents: one wave per 16-row tile, tiles strided over the grid's
// waves.  Lane (g, col) takes inputs 32 c + 8 g .. + 7 of the tile's row col
// straight from its row, in two 16-byte loads (rows of any length, so 4-byte
// aligned); the four lane groups read 128 consecutive bytes of each row.
// Copying tiles through LDS first took some ten vector instructions per input
// (1M rows of 16: 62.1 -> 38.4 us; critic over 129 x 16,000 rows of 129 and
// advantages: 300 -> 257 us, the critic's 241 us reading its views at 4.4 TB/s;
// a large copy moves 5.2).  Issuing a chunk's loads before the products of the
// chunk before it, across tiles, was slower (500,000 rows of 129 52.6 us, now
// 50.2; 65,536 of 32 7.1, now 6.1), two chunks ahead slower still (54.2): the
// waves of a CU cover each other's loads.
// Bound: tanh on the vector ALUs for short rows (128
// per row, whose exp and reciprocal issue at a quarter of the rate of an FMA:
// about 27 us of issue per 1M rows), reading the rows for long ones, one tile's
// latency for few (so nothing but the layer-1 copy waits before the first tile:
// the other weights and the draws are loaded beside the rows, 2,000 rows of 256
// sampled 7.4 -> 6.0 us).
// Layer 1's A operand lives in LDS, loaded once per block; kReg: the other
// layers' in registers, else in LDS too.  Layer 1's results reach layer 2's B
// operand (eight consecutive hidden units per lane group) through a per-wave
// LDS tile.
template <int NT, bool kReg, int kOut>
__global__ __launch_bounds__(NT) void k_policy(PolArgs A) {
    __shared__ PolConsts s_pc;
    extern __shared__ bf16x8 s_dyn[];
    const int wid = threadIdx.x / 64, lane = threadIdx.x & 63, g = lane >> 4, col = lane & 15;
    const int type = (int)blockIdx.y;
    const NetArgs N = type ? A.net[1] : A.net[0];
    const int kc = A.kc, in_dim = A.in_dim, rem = in_dim & 7;
    bf16x8 *s_w1 = s_dyn, *s_w2 = s_w1 + kc * 256, *s_w3 = s_w2 + (kReg ? 0 : 512);
    __bf16 *s_hid = reinterpret_cast<__bf16 *>(s_w3 + (kReg ? 0 : 128)) + (size_t)wid * 16 * kHidLd;
    const int64_t waves = (int64_t)gridDim.x * (NT / 64);
    const int64_t tiles = (A.n + 15) / 16;

    // the lane's row of a tile: its env-owned rows, whether it is computed
    struct Row {
        const float *x;
        float2 *act;
        bool valid;
    };
    auto row_of = [&](int64_t tile) {
        const int64_t agent = tile * 16 + col;
        const int64_t at = agent < A.n ? agent : A.n - 1;  // rows past the end repeat the last
        Row r{A.obs + at * in_dim, A.act + at, agent < A.n};
        if (A.envs) {
            int e = 0;
            if (A.n_envs > 1) {
                e = wave_env_search(A.base, A.n_envs, (int)(tile * 16));
                while (A.base[e + 1] <= at) ++e;
            }
            const DevEnv &E = A.envs[e];
            const int64_t i = at - E.agent_base;
            if (A.typed) {
                r.valid = r.valid && (i < E.n_chasers ? 1 : 0) == type;
            } else {
                r.x = E.obs + i * in_dim;
                r.act = reinterpret_cast<float2 *>(E.act) + i;
            }
        }
        return r;
    };
    // the wave's first tile from `tile` on that has a row to compute
    auto find = [&](int64_t tile, Row &r) {
        for (; tile < tiles; tile += waves) {
            r = row_of(tile);
            if (!A.typed || __any(r.valid)) break;
        }
        return tile;
    };
    auto load = [&](const Row &r, int c, float (&f)[8]) {
        const int k0 = 32 * c + 8 * g;
        if (k0 + 8 <= in_dim) {
            const f32x4u u = *reinterpret_cast<const f32x4u *>(r.x + k0);
            const f32x4u w = *reinterpret_cast<const f32x4u *>(r.x + k0 + 4);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                f[j] = u[j];
                f[4 + j] = w[j];
            }
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) f[j] = 0.0f;
            if (k0 < in_dim) {
#pragma unroll
                for (int j = 0; j < 7; ++j)
                    if (j < rem) f[j] = r.x[k0 + j];
            }
        }
    };

    Row row{};
    int64_t tile = find((int64_t)blockIdx.x * (NT / 64) + wid, row);
    for (int i = threadIdx.x; i < kc * 256; i += NT) s_w1[i] = N.P.w1[i];
    if constexpr (!kReg) {
        for (int i = threadIdx.x; i < 512; i += NT) s_w2[i] = N.P.w2[i];
        if (threadIdx.x < 128) s_w3[threadIdx.x] = N.P.w3[threadIdx.x];
    }
    load_pol_consts(N.P, &s_pc, threadIdx.x, NT);
    __syncthreads();
    bf16x8 w2[kReg ? 8 : 1], w3[kReg ? 2 : 1];
    if constexpr (kReg) {
#pragma unroll
        for (int k = 0; k < 8; ++k) w2[k] = N.P.w2[k * 64 + lane];
#pragma unroll
        for (int k = 0; k < 2; ++k) w3[k] = N.P.w3[k * 64 + lane];
    }

    while (tile < tiles) {
        const int64_t agent = tile * 16 + col;
        float2 e = make_float2(0.0f, 0.0f);
        if (kOut == kSample && g == 0 && row.valid) e = A.eps[agent];
        Row next{};  // found meanwhile
        const int64_t tnext = find(tile + waves, next);
        // the tile's inputs as BF16
        auto xb = [&](int c) {
            bf16x8 x;
            float f[8];
            load(row, c, f);
#pragma unroll
            for (int j = 0; j < 8; ++j) x[j] = (__bf16)f[j];
            return x;
        };
        auto w1a = [&](int c, int t) { return s_w1[(c * 4 + t) * 64 + lane]; };
        auto w2a = [&](int c, int t) {
            if constexpr (kReg) return w2[c * 4 + t];
            else return s_w2[(c * 4 + t) * 64 + lane];
        };
        auto w3a = [&](int c) {
            if constexpr (kReg) return w3[c];
            else return s_w3[c * 64 + lane];
        };
        auto hrow = [&](int r) { return s_hid + r * kHidLd; };
        const float2 z = mlp_tile(kc, xb, w1a, w2a, w3a, s_pc, hrow, lane);
        if (g == 0 && row.valid) {
            if constexpr (kOut == kValue) {
                A.val[agent] = z.x;
            } else {
                *row.act = pol_output<kOut == kSample>(z, N.max_turn, N.max_dspeed, e, N.sig0,
                                                       N.sig1, N.logp_c,
                                                       A.logp ? A.logp + agent : nullptr);
            }
        }
        tile = tnext;
        row = next;
    }
}

uint16_t bf16_bits_rne(float f) {
    uint32_t u;
    memcpy(&u, &f, 4);
    if ((u & 0x7f800000u) == 0x7f800000u && (u & 0x007fffffu)) return (uint16_t)((u >> 16) | 0x40);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

}  // namespace

}  // namespace flock

using namespace flock;

struct flock_policy {
    int in_dim, kc;  // kc: chunks of 32 inputs
    int critic;      // 0 actor (two scaled tanh outputs), 1 critic (one linear output)
    float max_turn, max_dspeed;
    PolLayout lay;
    std::vector<char> host;  // staged device image, kept until pol_destroy
};

namespace flock {

namespace {
NetArgs net_args(const pol_t *p, const float *log_std) {
    NetArgs n{};
    n.P = p->lay;
    n.max_turn = p->max_turn;
    n.max_dspeed = p->max_dspeed;
    if (log_std) {
        n.sig0 = (float)exp((double)log_std[0]);
        n.sig1 = (float)exp((double)log_std[1]);
        n.logp_c = (float)(-((double)log_std[0] + (double)log_std[1]) - log(2.0 * M_PI));
    }
    return n;
}

PolArgs pol_args(const pol_t *p, const float *log_std, const float *obs, int64_t n, float *act) {
    PolArgs a{};
    a.net[0] = net_args(p, log_std);
    a.in_dim = p->in_dim;
    a.kc = p->kc;
    a.n = n;
    a.obs = obs;
    a.act = reinterpret_cast<float2 *>(act);
    return a;
}

template <int kOut>
hipError_t launch_pol(const PolArgs &a, hipStream_t s) {
    if (a.n <= 0) return hipSuccess;
    const int64_t tiles = (a.n + 15) / 16;
    auto go = [&](auto kernel, int nt, bool reg, int64_t most) {
        const int64_t blocks = std::min<int64_t>((tiles + nt / 64 - 1) / (nt / 64), most);
        const size_t lds = ((size_t)a.kc * 256 + (reg ? 0 : 640)) * sizeof(bf16x8) +
                           (size_t)(nt / 64) * 16 * kHidLd * sizeof(__bf16);
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks, a.typed ? 2 : 1), dim3(nt), lds, s, a);
    };
    // Short rows (one chunk) of large launches: the weights in LDS leave 70
    // registers, seven waves a SIMD (1M rows: 39.7 us; with the weights in 56
    // registers, four waves, 49.3; two tiles side by side to a wave, 53), in
    // more blocks than are resident, so that the last round is even (1,024
    // blocks 44.2 us, 1,536 41.3, 2,048 39.7, 4,096 40.1).  Long rows are
    // bound by their reads, and the LDS by layer 1's operands (four waves and
    // registers 261 us, all in LDS 309); small launches by one tile's latency.
    // The line: 40,000 rows of 16 take 5.5 us in LDS and 5.4 in registers, 65,536
    // 5.6 and 6.0, 98,304 6.7 and 7.2, 262,144 12.7 and 15.0.
    // As many blocks of the other form as are resident: four to a CU, three where
    // layer 1 has eight or nine chunks of 4 KiB (500,000 rows of 256: 1,024 blocks
    // 131 us, 768 102).
    if (a.kc == 1 && tiles > 4096) go(k_policy<512, false, kOut>, 512, false, 2048);
    else go(k_policy<256, true, kOut>, 256, true, a.kc < 8 ? 1024 : 768);
    return hipGetLastError();
}

}  // namespace

hipError_t policy_launch(const pol_t *p, const float *obs, int64_t n, float *act, hipStream_t s) {
    return launch_pol<kMean>(pol_args(p, nullptr, obs, n, act), s);
}

hipError_t policy_launch_sample(const pol_t *p, const float *obs, int64_t n, const float *eps,
                                const float log_std[2], float *act, float *logp, hipStream_t s) {
    PolArgs a = pol_args(p, log_std, obs, n, act);
    a.eps = reinterpret_cast<const float2 *>(eps);
    a.logp = logp;
    return launch_pol<kSample>(a, s);
}

hipError_t policy_launch_value(const pol_t *p, const float *obs, int64_t n, float *val,
                               hipStream_t s) {
    PolArgs a = pol_args(p, nullptr, obs, n, nullptr);
    a.val = val;
    return launch_pol<kValue>(a, s);
}

hipError_t policy_launch_types(const pol_t *runner, const pol_t *chaser, const StepPlan &plan,
                               int table, const float *obs, const float *eps, const float *log_std,
                               float *act, float *logp, hipStream_t s) {
    PolArgs a = pol_args(runner, log_std, obs, plan.G, act);
    a.net[1] = net_args(chaser, log_std ? log_std + 2 : nullptr);
    a.typed = 1;
    a.envs = plan.a.envs[table & 1];
    a.base = plan.a.base;
    a.n_envs = plan.n_envs;
    if (!eps) return launch_pol<kMean>(a, s);
    a.eps = reinterpret_cast<const float2 *>(eps);
    a.logp = logp;
    return launch_pol<kSample>(a, s);
}

hipError_t policy_launch_envs(const pol_t *p, const StepPlan &plan, int table, hipStream_t s) {
    PolArgs a = pol_args(p, nullptr, nullptr, plan.G, nullptr);
    a.envs = plan.a.envs[table & 1];
    a.base = plan.a.base;
    a.n_envs = plan.n_envs;
    return launch_pol<kMean>(a, s);
}

int policy_is_critic(const pol_t *p) { return p->critic; }

const void *policy_weights(const pol_t *p) { return p->lay.w1; }

int policy_in_dim(const pol_t *p) { return p->in_dim; }

PolFuse policy_fuse_args(const pol_t *p) {
    PolFuse f{};
    f.P = p->lay;
    f.in_dim = p->in_dim;
    f.kc = p->kc;
    f.mode = 1;
    f.max_turn = p->max_turn;
    f.max_dspeed = p->max_dspeed;
    return f;
}

void policy_fuse_sampling(PolFuse *f, const float log_std[2], const float *eps, float *logp) {
    f->mode = 2;
    f->eps = reinterpret_cast<const float2 *>(eps);
    f->sig0 = (float)exp((double)log_std[0]);
    f->sig1 = (float)exp((double)log_std[1]);
    f->logp_c = (float)(-((double)log_std[0] + (double)log_std[1]) - log(2.0 * M_PI));
    f->logp = logp;
}

}  // namespace flock

extern "C" {

size_t pol_workspace_bytes(int in_dim, int hidden) {
    if (in_dim < 1 || in_dim > kMaxIn || hidden != kHidden) {
        set_error(ENV_EINVAL, "policy needs 1 <= in_dim <= %d and hidden == 64", kMaxIn);
        return 0;
    }
    return carve_pol(nullptr, (in_dim + 31) / 32).bytes;
}

}  // extern "C"

namespace {

// Shared by the actor (n_out = 2) and the critic (n_out = 1).
int create_net(const float *w, int in_dim, int hidden, int n_out, float max_turn, float max_dspeed,
               void *ws, size_t bytes, void *stream, pol_t **out) {
    if (!w || !ws || !out) return set_error(ENV_EINVAL, "NULL argument to pol_create");
    if (in_dim < 1 || in_dim > kMaxIn || hidden != kHidden)
        return set_error(ENV_EINVAL, "policy needs 1 <= in_dim <= %d and hidden == 64", kMaxIn);
    if (!(max_turn >= 0.0f) || !(max_dspeed >= 0.0f) || !isfinite(max_turn) || !isfinite(max_dspeed))
        return set_error(ENV_EINVAL, "action scales must be finite and >= 0");
    if (reinterpret_cast<uintptr_t>(ws) % 256 != 0)
        return set_error(ENV_EINVAL, "workspace must be 256-byte aligned");
    const int H = kHidden;
    const int kc = (in_dim + 31) / 32;
    const size_t need = carve_pol(nullptr, kc).bytes;
    if (bytes < need)
        return set_error(ENV_ENOMEM, "policy workspace has %zu bytes, needs %zu", bytes, need);
    pol_t *p = new pol_t;
    p->in_dim = in_dim;
    p->kc = kc;
    p->critic = n_out == 1 ? 1 : 0;
    p->max_turn = max_turn;
    p->max_dspeed = max_dspeed;
    p->lay = carve_pol(static_cast<char *>(ws), kc);
    const PolLayout &off = p->lay;
    p->host.assign(need, 0);
    char *hb = p->host.data();
    // host image of the workspace: same offsets from the base as the device arrays
    auto at = [&](const void *dev) {
        return hb + (static_cast<const char *>(dev) - static_cast<const char *>(ws));
    };
    const float *W1 = w;
    const float *b1 = W1 + in_dim * H;
    const float *W2 = b1 + H;
    const float *b2 = W2 + H * H;
    const float *W3 = b2 + H;
    const float *b3 = W3 + H * n_out;
    float *b3d = reinterpret_cast<float *>(at(off.b3));
    for (int o = 0; o < 4; ++o) b3d[o] = o < n_out ? b3[o] : 0.0f;
    // A operands in lane order: lane (g, col) of chunk c, tile t holds
    // W[32 c + 8 g + j][16 t + col] in element j (zero beyond in_dim)
    uint16_t *w1p = reinterpret_cast<uint16_t *>(at(off.w1));
    for (int c = 0; c < kc; ++c)
        for (int t = 0; t < 4; ++t)
            for (int lane = 0; lane < 64; ++lane)
                for (int j = 0; j < 8; ++j) {
                    const int k = 32 * c + 8 * (lane / 16) + j, m = 16 * t + lane % 16;
                    const float v = k < in_dim ? W1[k * H + m] : 0.0f;
                    w1p[((c * 4 + t) * 64 + lane) * 8 + j] = bf16_bits_rne(v);
                }
    uint16_t *w2p = reinterpret_cast<uint16_t *>(at(off.w2));
    for (int c = 0; c < 2; ++c)
        for (int t = 0; t < 4; ++t)
            for (int lane = 0; lane < 64; ++lane)
                for (int j = 0; j < 8; ++j) {
                    const int k = 32 * c + 8 * (lane / 16) + j, m = 16 * t + lane % 16;
                    w2p[((c * 4 + t) * 64 + lane) * 8 + j] = bf16_bits_rne(W2[k * H + m]);
                }
    // output layer: A[m][k] = W3[k][m] for the n_out real rows m, zero rows after
    uint16_t *w3p = reinterpret_cast<uint16_t *>(at(off.w3));
    for (int c = 0; c < 2; ++c)
        for (int lane = 0; lane < 64; ++lane)
            for (int j = 0; j < 8; ++j) {
                const int k = 32 * c + 8 * (lane / 16) + j, m = lane % 16;
                w3p[(c * 64 + lane) * 8 + j] = bf16_bits_rne(m < n_out ? W3[k * n_out + m] : 0.0f);
            }
    float *b1d = reinterpret_cast<float *>(at(off.b1));
    float *b2d = reinterpret_cast<float *>(at(off.b2));
    for (int h = 0; h < H; ++h) {
        b1d[h] = b1[h];
        b2d[h] = b2[h];
    }
    hipError_t e = hipMemcpyAsync(ws, hb, need, hipMemcpyHostToDevice,
                                  reinterpret_cast<hipStream_t>(stream));
    if (e != hipSuccess) {
        delete p;
        return set_error(ENV_EHIP, "pol_create upload: %s", hipGetErrorString(e));
    }
    *out = p;
    return ENV_OK;
}

}  // namespace

extern "C" {

int pol_create(const float *w, int in_dim, int hidden, float max_turn, float max_dspeed, void *ws,
               size_t bytes, void *stream, pol_t **out) {
    return create_net(w, in_dim, hidden, 2, max_turn, max_dspeed, ws, bytes, stream, out);
}

int pol_create_value(const float *w, int in_dim, int hidden, void *ws, size_t bytes, void *stream,
                     pol_t **out) {
    return create_net(w, in_dim, hidden, 1, 1.0f, 1.0f, ws, bytes, stream, out);
}

void pol_destroy(pol_t *p) { delete p; }

int pol_forward(pol_t *p, const float *obs, int64_t n, float *act, void *stream) {
    if (!p) return set_error(ENV_EINVAL, "policy is NULL");
    if (p->critic) return set_error(ENV_EINVAL, "pol_forward needs an actor (this is a critic)");
    if (n < 0) return set_error(ENV_EINVAL, "n < 0");
    if (n > 0 && (!obs || !act)) return set_error(ENV_EINVAL, "obs/act is NULL");
    hipError_t e = policy_launch(p, obs, n, act, reinterpret_cast<hipStream_t>(stream));
    if (e != hipSuccess) return set_error(ENV_EHIP, "pol_forward: %s", hipGetErrorString(e));
    return ENV_OK;
}

int pol_sample(pol_t *p, const float *obs, int64_t n, const float *log_std, const float *eps,
               float *act, float *logp, void *stream) {
    if (!p || !log_std) return set_error(ENV_EINVAL, "policy or log_std is NULL");
    if (p->critic) return set_error(ENV_EINVAL, "pol_sample needs an actor (this is a critic)");
    if (n < 0) return set_error(ENV_EINVAL, "n < 0");
    if (!isfinite(log_std[0]) || !isfinite(log_std[1]))
        return set_error(ENV_EINVAL, "log_std must be finite");
    if (n > 0 && (!obs || !eps || !act)) return set_error(ENV_EINVAL, "obs/eps/act is NULL");
    hipError_t e = policy_launch_sample(p, obs, n, eps, log_std, act, logp,
                                        reinterpret_cast<hipStream_t>(stream));
    if (e != hipSuccess) return set_error(ENV_EHIP, "pol_sample: %s", hipGetErrorString(e));
    return ENV_OK;
}

int pol_value(pol_t *p, const float *obs, int64_t n, float *value, void *stream) {
    if (!p) return set_error(ENV_EINVAL, "critic is NULL");
    if (!p->critic) return set_error(ENV_EINVAL, "pol_value needs a critic (pol_create_value)");
    if (n < 0) return set_error(ENV_EINVAL, "n < 0");
    if (n > 0 && (!obs || !value)) return set_error(ENV_EINVAL, "obs/value is NULL");
    hipError_t e = policy_launch_value(p, obs, n, value, reinterpret_cast<hipStream_t>(stream));
    if (e != hipSuccess) return set_error(ENV_EHIP, "pol_value: %s", hipGetErrorString(e));
    return ENV_OK;
}

}  // extern "C"
