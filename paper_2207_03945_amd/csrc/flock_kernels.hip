// flock_kernels.hip -- gfx950 kernels of one flock-environment step.
//
// One step (Sec. 4.1 of arXiv:2207.03945: apply the actions, then update
// view and reward over every pair in spatial proximity; Sec. 2.1: all agents
// update simultaneously) is four dependent phases over a whole batch of
// environments at once.  Agents are kept in cell order between steps (see
// DevEnv), so every phase streams its per-agent data sequentially:
//
//   k_move_count  record p: rotate/accelerate/move/wrap (FP32), new cell key,
//                 rank within the cell.  Records of a block were sorted by
//                 their previous cell, so their new keys span a narrow range:
//                 ranks come from an LDS histogram and one global atomic per
//                 distinct key (global atomics per record as a fallback)
//   k_scan_*      exclusive prefix of the per-cell counts (and re-zero them)
//   k_scatter     record p -> its new cell-order position (ping-pong buffer),
//                 with its agent id and FP64 return; positions for the sweep
//   k_sweep       one lane per agent in the new cell order walks the cells of
//                 its (2r+1)^2 block (runs of consecutive cells, read from
//                 L2-resident sorted positions); per candidate: periodic
//                 image, d^2, radius tests, sector of the bearing, per-sector
//                 minimum in LDS; then view, reward and the FP64 return
//
// Envs of a batch live in one global cell space (env k's cells start at
// cell_base), so one counting sort serves every env and the cell-order range
// of env k equals its row range [agent_base, agent_base + n).
//
// Arithmetic contract (compiled with -ffp-contract=off):
//   * the move is IEEE FP32 operation by operation; cos/sin of the FP32
//     heading come from an FP32 evaluation within 1 ulp of the correctly
//     rounded values (heading_cs), so a new position is within one rounding
//     of the correctly rounded result of the stated operations;
//   * pair displacement: the periodic shift is applied to whichever operand
//     lies in the far half of the box, where the shift is exact, so dx and
//     dy carry a single rounding; d^2 = fma(dx, dx, dy*dy); the radius tests
//     are strict;
//   * the bearing comes from rotating (dx, dy) into the heading frame,
//     folding into the first octant and an odd polynomial for atan fitted
//     here (max error 3.4e-7 rad); with the FP32 roundings the sector
//     position is within about 1.5e-6 rad of the exact bearing;
//   * view: 1 - sqrt(d^2_min) * (1/R), within a few ulp of 1 - d_min/R.
#include <limits.h>

#include <algorithm>
#include <atomic>
#include <cmath>

#include <type_traits>

#include "flock_internal.h"
#include "strip_order.h"

namespace flock {

namespace {

constexpr uint32_t kInfBits = 0x7f800000u;

// Positions lie in [0, L), so truncation is floor; the clamp keeps any
// out-of-range or NaN coordinate inside the grid (memory safety only).
__device__ __forceinline__ int cell_of(float v, float inv, int ncell) {
    int c = (int)(v * inv);
    c = c < ncell ? c : ncell - 1;
    return c > 0 ? c : 0;
}

// Env of the block's first row into s_env (wave 0 searches).
__device__ __forceinline__ void block_env(int *s_env, const int32_t *base, int n_envs, int row) {
    if (threadIdx.x < 64) {
        const int e = wave_env_search(base, n_envs, row);
        if (threadIdx.x == 0) *s_env = e;
    }
}

__device__ __forceinline__ int wave_min(int x) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) x = min(x, __shfl_xor(x, d, 64));
    return x;
}

__device__ __forceinline__ int wave_max(int x) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) x = max(x, __shfl_xor(x, d, 64));
    return x;
}

// Arrays reached through a DevEnv are device global memory, but a pointer
// read from memory is generic to the compiler, and it waits on generic
// accesses conservatively (they count as both vector-memory and LDS
// operations).  These access such arrays through the global address space.
// The sorts use them, and the sweep where lane groups share an agent (its
// per-agent loads and stores then overlap better: 245 -> 230 us for 50k-agent
// blobs at four lanes); with one lane per agent the generic form measured faster.
#define FLOCK_GLOBAL __attribute__((address_space(1)))
typedef float gfloat4 __attribute__((ext_vector_type(4)));
typedef float gfloat2 __attribute__((ext_vector_type(2)));

template <class T>
__device__ __forceinline__ T gload(const T *p, int64_t i) {
    return ((const FLOCK_GLOBAL T *)p)[i];
}

__device__ __forceinline__ float4 gload(const float4 *p, int64_t i) {
    const gfloat4 v = ((const FLOCK_GLOBAL gfloat4 *)p)[i];
    return make_float4(v.x, v.y, v.z, v.w);
}

__device__ __forceinline__ float2 gload(const float2 *p, int64_t i) {
    const gfloat2 v = ((const FLOCK_GLOBAL gfloat2 *)p)[i];
    return make_float2(v.x, v.y);
}

template <class T>
__device__ __forceinline__ void gstore(T *p, int64_t i, T v) {
    ((FLOCK_GLOBAL T *)p)[i] = v;
}

// Either form, chosen at compile time.
template <bool kGlobal, class T>
__device__ __forceinline__ T load_as(const T *p, int64_t i) {
    if constexpr (kGlobal) return gload(p, i);
    else return p[i];
}

template <bool kGlobal, class T>
__device__ __forceinline__ void store_as(T *p, int64_t i, T v) {
    if constexpr (kGlobal) gstore(p, i, v);
    else p[i] = v;
}

// --------------------------------------------------------------------- move

constexpr int kHistBins = 2048;

// (cos h, sin h) of a heading in FP32 arithmetic.  Cody and Waite's
// additive range reduction (Software Manual for the Elementary Functions,
// 1980): k = nearest integer to h 2/pi, r = h - k pi/2 with pi/2 split into
// three FP32 parts and each product taken exactly inside an FMA, so r carries
// one rounding for |h| < 2^12; then odd / even polynomials in r^2 on
// [-pi/4, pi/4] (minimax fits made for this kernel: relative error 3.8e-9 for
// sin, absolute 9.6e-11 for cos) and the quadrant's swap and signs.  Checked
// on every FP32 heading in [0, 2pi_f]: within 1 ulp of the correctly rounded
// value, and correctly rounded for 99.4 % (cos) and 99.6 % (sin) of them
// (most FP32 values lie near 0); of headings drawn uniformly in value, 84 %
// and 94 %, the final rounding of r costing up to 0.35 ulp near pi/4.
__device__ __forceinline__ float2 heading_cs(float h) {
    const float k = __builtin_rintf(h * 0.636619772f);
    float r = __builtin_fmaf(-k, 1.57079637050628662109375f, h);
    r = __builtin_fmaf(-k, -4.37113882867379e-08f, r);
    r = __builtin_fmaf(-k, -1.7151245e-15f, r);
    const float z = r * r;
    float ps = __builtin_fmaf(z, -0.00019515264f, 0.008332161f);
    ps = __builtin_fmaf(z, ps, -0.16666655f);
    const float sn = __builtin_fmaf(r * z, ps, r);
    float pc = __builtin_fmaf(z, 2.4438208e-05f, -0.0013887365f);
    pc = __builtin_fmaf(z, pc, 0.041666646f);
    const float cs = __builtin_fmaf(z, __builtin_fmaf(z, pc, -0.5f), 1.0f);
    const int q = (int)k & 3;
    float c = (q & 1) ? sn : cs, s = (q & 1) ? cs : sn;
    c = (q == 1 || q == 2) ? -c : c;
    s = (q >= 2) ? -s : s;
    return make_float2(c, s);
}

// One agent's move (Sec. 4.1): turn, speed update (tag: the action is the
// speed), integrate with the new heading and speed, wrap into [0, L).
__device__ __forceinline__ float4 move_record(const DevEnv &E, float4 r, float2 av) {
    float x = r.x, y = r.y, h = r.z, sp = r.w;
    const float turn = fminf(fmaxf(av.x, -E.max_turn), E.max_turn);
    h = h + turn;
    if (h < 0.0f) h = h + kTwoPiF;
    if (h >= kTwoPiF) h = h - kTwoPiF;
    if (E.tag) {
        sp = fminf(fmaxf(av.y, 0.0f), E.s_max);
    } else {
        const float ds = fminf(fmaxf(av.y, -E.max_dspeed), E.max_dspeed);
        sp = fminf(fmaxf(sp + ds, E.s_min), E.s_max);
    }
    const float2 cs = heading_cs(h);
    const float c = cs.x, sn = cs.y;
    const float L = E.box;
    float nx = x + sp * c;
    if (nx < 0.0f) nx = nx + L;
    if (nx >= L) nx = nx - L;
    float ny = y + sp * sn;
    if (ny < 0.0f) ny = ny + L;
    if (ny >= L) ny = ny - L;
    return make_float4(nx, ny, h, sp);
}

// Cell of a position within its env's grid: column-major, rows within a column.
__device__ __forceinline__ int local_cell(const DevEnv &E, float x, float y) {
    return cell_of(x, E.inv_cx, E.ncx) * E.ncy + cell_of(y, E.inv_cy, E.ncy);
}

// Records per thread of the move kernel: a block covers kMoveRecs * kBlock
// consecutive records, all of whose loads are issued before any compute.
constexpr int kMoveRecs = 1;

__global__ __launch_bounds__(kBlock) void k_move_count(SortArrays a, const DevEnv *__restrict__ envs,
                                                       int n_envs, int G, int do_move,
                                                       const float2 *__restrict__ act,
                                                       float2 *__restrict__ act_copy) {
    constexpr int R = kMoveRecs;
    __shared__ int s_env;
    __shared__ int s_kmin[kBlock / 64], s_kmax[kBlock / 64];
    __shared__ int s_hist[kHistBins];
    const int p0 = blockIdx.x * (kBlock * R);
    block_env(&s_env, a.base, n_envs, p0);
    __syncthreads();
    // loads first: records, ids, then the actions they index
    int env[R], key[R];
    bool live[R];
    float4 rec[R];
    int id[R];
    float2 av[R];
    int e = s_env;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int p = p0 + r * kBlock + threadIdx.x;
        live[r] = p < G;
        key[r] = 0;
        env[r] = e;
        if (live[r]) {
            while (a.base[e + 1] <= p) ++e;
            env[r] = e;
            const DevEnv &E = envs[e];
            const int i = p - E.agent_base;
            rec[r] = E.rec_cur[i];
            id[r] = do_move ? E.id_cur[i] : 0;
        }
    }
    if (do_move) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (!live[r]) continue;
            const DevEnv &E = envs[env[r]];
            if ((unsigned)id[r] >= (unsigned)E.n) continue;  // ids are agent indices (a guard)
            av[r] = act ? act[E.agent_base + id[r]] : reinterpret_cast<const float2 *>(E.act)[id[r]];
            if (act_copy) act_copy[E.agent_base + id[r]] = av[r];
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (!live[r]) continue;
        const int p = p0 + r * kBlock + threadIdx.x;
        const DevEnv &E = envs[env[r]];
        const float4 m = do_move ? move_record(E, rec[r], av[r]) : rec[r];
        a.tmp[p] = m;
        key[r] = E.cell_base + local_cell(E, m.x, m.y);
        a.key[p] = key[r];
    }
    // key range of the block
    int kmin = INT_MAX, kmax = INT_MIN;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        kmin = min(kmin, live[r] ? key[r] : INT_MAX);
        kmax = max(kmax, live[r] ? key[r] : INT_MIN);
    }
    kmin = wave_min(kmin);
    kmax = wave_max(kmax);
    const int wid = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        s_kmin[wid] = kmin;
        s_kmax[wid] = kmax;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kBlock / 64; ++w) {
        kmin = min(kmin, s_kmin[w]);
        kmax = max(kmax, s_kmax[w]);
    }
    const int range = kmax - kmin;  // >= 0: every block holds at least one record
    int slot[R];
    if (range < kHistBins) {
        for (int b = threadIdx.x; b <= range; b += kBlock) s_hist[b] = 0;
        __syncthreads();
        int lrank[R];
#pragma unroll
        for (int r = 0; r < R; ++r) lrank[r] = live[r] ? atomicAdd(&s_hist[key[r] - kmin], 1) : 0;
        __syncthreads();
        for (int b = threadIdx.x; b <= range; b += kBlock) {
            const int c = s_hist[b];
            if (c) s_hist[b] = atomicAdd(&a.count[kmin + b], c);
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r) slot[r] = live[r] ? s_hist[key[r] - kmin] + lrank[r] : 0;
    } else {
#pragma unroll
        for (int r = 0; r < R; ++r) slot[r] = live[r] ? atomicAdd(&a.count[key[r]], 1) : 0;
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (live[r]) a.slot[p0 + r * kBlock + threadIdx.x] = slot[r];
}

// --------------------------------------------------------------------- scan

// Exclusive block scan of one int per thread; also returns the block total.
template <int NT>
__device__ __forceinline__ int block_exclusive_scan(int v, int *s_wave, int *total) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    int incl = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        int t = __shfl_up(incl, d, 64);
        if (lane >= d) incl += t;
    }
    if (lane == 63) s_wave[wid] = incl;
    __syncthreads();
    if (wid == 0) {
        int w = lane < NT / 64 ? s_wave[lane] : 0;
        int wi = w;
#pragma unroll
        for (int d = 1; d < NT / 64; d <<= 1) {
            int t = __shfl_up(wi, d, 64);
            if (lane >= d) wi += t;
        }
        if (lane < NT / 64) s_wave[lane] = wi - w;
        if (lane == NT / 64 - 1) s_wave[NT / 64] = wi;
    }
    __syncthreads();
    const int r = s_wave[wid] + incl - v;
    *total = s_wave[NT / 64];
    return r;
}

constexpr int kScanNT = 1024;
constexpr int kScanItems = 16;
constexpr int kScanTile = kScanNT * kScanItems;  // cells of the single-block scan

// Every env has at most kScanTile cells: block e scans env e's cells on its
// own.  An env's agents occupy cell-order positions [agent_base, agent_base
// + n), so its cell starts are agent_base plus the prefix within the env;
// no block waits for another.  Re-zeroes the counts; the last env's block
// also writes start[C] (= the batch's agent total).
// NT threads of ITEMS cells each cover the largest env of the launch.
template <int NT, int ITEMS>
__global__ __launch_bounds__(NT) void k_scan_env(int32_t *__restrict__ count,
                                                 int32_t *__restrict__ start,
                                                 const DevEnv *__restrict__ envs, int n_envs, int C) {
    __shared__ int s_wave[NT / 64 + 1];
    __shared__ int s_tile[NT * ITEMS];
    const int t = threadIdx.x;
    const DevEnv &E = envs[blockIdx.x];
    const int cb = E.cell_base, Ce = E.ncx * E.ncy, base = E.agent_base;
    count += cb;
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int idx = k * NT + t;  // coalesced: item-major
        s_tile[idx] = idx < Ce ? count[idx] : 0;
    }
    __syncthreads();
    int vals[ITEMS];
    int sum = 0;
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        vals[k] = s_tile[t * ITEMS + k];
        sum += vals[k];
    }
    int total;
    int run = block_exclusive_scan<NT>(sum, s_wave, &total) + base;
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        s_tile[t * ITEMS + k] = run;
        run += vals[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int idx = k * NT + t;
        if (idx < Ce) {
            start[cb + idx] = s_tile[idx];
            count[idx] = 0;
        }
    }
    if (t == 0 && blockIdx.x == n_envs - 1) start[C] = base + total;
}

// Large C: tiles of kTile2 cells, one 256-thread block each.
constexpr int kScan2NT = 256;
constexpr int kScan2Items = 8;
constexpr int kTile2 = kScan2NT * kScan2Items;

// Phase 1: per-tile totals.  The phases are separate launches, whose
// boundaries order them; no block waits on another (a device-wide fence per
// block writes back an XCD's L2 and costs far more than a launch).
__global__ __launch_bounds__(kScan2NT) void k_tile_sums(const int32_t *__restrict__ count,
                                                        int32_t *__restrict__ part, int C) {
    __shared__ int s_wave[kScan2NT / 64 + 1];
    const int t = threadIdx.x;
    const int64_t base = (int64_t)blockIdx.x * kTile2;
    int sum = 0;
#pragma unroll
    for (int k = 0; k < kScan2Items; ++k) {
        const int64_t idx = base + k * kScan2NT + t;
        sum += idx < C ? count[idx] : 0;
    }
    int total;
    (void)block_exclusive_scan<kScan2NT>(sum, s_wave, &total);
    if (t == 0) part[blockIdx.x] = total;
}

// Up to this many tiles, each tile of phase 2 sums the totals before it
// itself; beyond, one block first turns them into exclusive offsets.
constexpr int kDirectTiles = 4096;

// Phase 1b (more than kDirectTiles tiles): one block, exclusive offsets of
// the nb tile totals in place, in chunks of kTile2 with a running carry.
__global__ __launch_bounds__(kScan2NT) void k_scan_parts(int32_t *__restrict__ part, int nb) {
    __shared__ int s_wave[kScan2NT / 64 + 1];
    const int t = threadIdx.x;
    int carry = 0;
    for (int c0 = 0; c0 < nb; c0 += kTile2) {
        int vals[kScan2Items];
        int psum = 0;
#pragma unroll
        for (int k = 0; k < kScan2Items; ++k) {
            const int idx = c0 + t * kScan2Items + k;
            vals[k] = idx < nb ? part[idx] : 0;
            psum += vals[k];
        }
        int chunk;
        int run = block_exclusive_scan<kScan2NT>(psum, s_wave, &chunk) + carry;
#pragma unroll
        for (int k = 0; k < kScan2Items; ++k) {
            const int idx = c0 + t * kScan2Items + k;
            if (idx < nb) part[idx] = run;
            run += vals[k];
        }
        carry += chunk;
        __syncthreads();  // s_wave is reused by the next chunk
    }
}

// Phase 2: scan each tile from its offset; re-zero the counts.  kSum: the
// offset is the sum of the totals of the tiles before (at most kDirectTiles
// of them), else part holds the offsets.  The last tile writes start[C].
template <bool kSum>
__global__ __launch_bounds__(kScan2NT) void k_scan_down(int32_t *__restrict__ count,
                                                        const int32_t *__restrict__ part,
                                                        int32_t *__restrict__ start, int C) {
    __shared__ int s_wave[kScan2NT / 64 + 1];
    __shared__ int s_tile[kTile2];
    __shared__ int s_off;
    const int t = threadIdx.x;
    const int64_t base = (int64_t)blockIdx.x * kTile2;
    if constexpr (kSum) {
        int before = 0;
        for (int b = t; b < (int)blockIdx.x; b += kScan2NT) before += part[b];
        int sum_before;
        (void)block_exclusive_scan<kScan2NT>(before, s_wave, &sum_before);
        if (t == 0) s_off = sum_before;
    } else {
        if (t == 0) s_off = part[blockIdx.x];
    }
#pragma unroll
    for (int k = 0; k < kScan2Items; ++k) {
        const int64_t idx = base + k * kScan2NT + t;
        s_tile[k * kScan2NT + t] = idx < C ? count[idx] : 0;
    }
    __syncthreads();
    int vals[kScan2Items];
    int sum = 0;
#pragma unroll
    for (int k = 0; k < kScan2Items; ++k) {
        vals[k] = s_tile[t * kScan2Items + k];
        sum += vals[k];
    }
    int total;
    const int off = s_off;  // published before the scan's barriers
    int run = block_exclusive_scan<kScan2NT>(sum, s_wave, &total) + off;
#pragma unroll
    for (int k = 0; k < kScan2Items; ++k) {
        s_tile[t * kScan2Items + k] = run;
        run += vals[k];
    }
    if (t == 0 && blockIdx.x == gridDim.x - 1) start[C] = off + total;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kScan2Items; ++k) {
        const int64_t idx = base + k * kScan2NT + t;
        if (idx < C) {
            start[idx] = s_tile[k * kScan2NT + t];
            count[idx] = 0;
        }
    }
}

// --------------------------------------------------- per-env fused sort

// Batches of many envs that each fit one block: block e moves env e's
// agents, counts them per cell in LDS, scans its own cells and scatters the
// records into the new cell order -- the move, count, scan and scatter of
// the separate kernels in one launch, with no global atomics.  Ranks within
// a cell come from LDS atomics, so the order inside a cell varies from run
// to run; every output is independent of that order.  Up to R records per
// thread; the env's cell counts, then starts, live in dynamic LDS.  Up to
// kEnvRegR records per thread the moved records and ids wait in registers
// for the scatter; above that they are staged in `tmp`.
// What bounds it: the addresses of the scattered stores and of the action
// gather (the texture addresser is busy 22,000 of 37,000 cycles per CU at
// 200 envs of 5,000), with one block per CU.  Measured there, us per step, 68.0
// as it stands: records staged in LDS and stored in order 73 to 75; all loads of
// a thread's records issued first 68.0; two blocks of 512 threads per CU 71.4;
// the strip sort 74 to 75; generic instead of global loads and stores 68.8.
constexpr int kEnvNT = 1024;
constexpr int kEnvRegR = 8;

template <int R>
__global__ __launch_bounds__(kEnvNT) void k_env_sort(SortArrays a, const DevEnv *__restrict__ envs,
                                                     int n_envs, int C, int do_move,
                                                     const float2 *__restrict__ act, int tag,
                                                     float2 *__restrict__ act_copy) {
    extern __shared__ int s_cells[];  // [Ce] counts, then starts within the env
    __shared__ int s_wave[kEnvNT / 64 + 1];
    const int tid = threadIdx.x;
    const DevEnv &E = envs[blockIdx.x];
    const int n = E.n, base = E.agent_base, cb = E.cell_base, Ce = E.ncx * E.ncy;
    for (int c = tid; c < Ce; c += kEnvNT) s_cells[c] = 0;
    __syncthreads();
    constexpr bool kRegs = R <= kEnvRegR;
    constexpr int RR = kRegs ? R : 1;
    int key[R], rank[R];
    float4 mr[RR];
    int idr[RR];
    double retr[RR];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = r * kEnvNT + tid;
        key[r] = 0;
        rank[r] = 0;
        if (i < n) {
            float4 m = gload(E.rec_cur, i);
            const int id = gload(E.id_cur, i);
            if (do_move) {
                float2 av = make_float2(0.0f, 0.0f);
                if ((unsigned)id < (unsigned)n) {  // ids are agent indices (a guard)
                    av = act ? act[base + id] : gload(reinterpret_cast<const float2 *>(E.act), id);
                    if (act_copy) act_copy[base + id] = av;
                }
                m = move_record(E, m, av);
            }
            if constexpr (kRegs) {
                mr[r] = m;
                idr[r] = id;
                retr[r] = gload(E.ret_cur, i);  // loaded now, stored after the scan
            } else {
                a.tmp[base + i] = m;
            }
            key[r] = local_cell(E, m.x, m.y);
            rank[r] = atomicAdd(&s_cells[key[r]], 1);
        }
    }
    __syncthreads();
    // exclusive scan of the counts: thread t owns cells [t k, t k + k)
    const int per = (Ce + kEnvNT - 1) / kEnvNT;
    const int c0 = tid * per;
    int sum = 0;
    for (int c = c0; c < c0 + per && c < Ce; ++c) sum += s_cells[c];
    int total;
    int run = block_exclusive_scan<kEnvNT>(sum, s_wave, &total);
    for (int c = c0; c < c0 + per && c < Ce; ++c) {
        const int cnt = s_cells[c];
        s_cells[c] = run;
        run += cnt;
    }
    if (tid == 0 && blockIdx.x == n_envs - 1) a.start[C] = base + n;
    __syncthreads();
    for (int c = tid; c < Ce; c += kEnvNT) a.start[cb + c] = base + s_cells[c];  // coalesced
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = r * kEnvNT + tid;
        if (i < n) {
            const int j = s_cells[key[r]] + rank[r];
            float4 m;
            int id;
            double ret;
            if constexpr (kRegs) {
                m = mr[r];
                id = idr[r];
                ret = retr[r];
            } else {
                m = a.tmp[base + i];
                id = gload(E.id_cur, i);
                ret = gload(E.ret_cur, i);
            }
            ((FLOCK_GLOBAL gfloat4 *)E.rec_nxt)[j] = gfloat4{m.x, m.y, m.z, m.w};
            gstore(E.id_nxt, j, id);
            gstore(E.ret_nxt, j, ret);
            a.sxy[base + j] = make_float2(m.x, m.y);
            if (tag) a.stype[base + j] = id < E.n_chasers ? 1 : 0;
        }
    }
}

// ------------------------------------------------------------- strip sort

// One block per strip of columns of one env (see carve_sort and the plan's
// strips in flock_internal.h).  The records are in cell order (column
// major), so the records of a range of columns are one range of records; an
// agent moves at most one column per step, so the agents now in the strip
// were, before the move, in its columns or in the one on either side.  The
// block loads and moves those, ranks its agents by cell in LDS, and writes
// them in cell order with the strip's cell starts.  The first NT * R records
// stay in registers between counting and placing; of the rest, the strip's
// agents wait in a list in LDS (kList, whose registers take the own columns
// first; the list sized for uniform agents), and a strip that exceeds it reads
// the rest twice, actions included.
//
// Where the strip's agents go: the agents now in columns below c0 are the
// records before the block's range, plus those in its range that are now
// below c0 -- all known to the block -- but for the agents that crossed the
// box's periodic edge outside the range, either way.  The env's first strip
// has both edge columns in its range and publishes the net count of those
// crossings, one word, as soon as it has moved them; the last strip needs
// only the env's size.  So no strip waits for any but the first, and none
// where an env has at most two.
//
// What bounds it: a chain of dependent memory accesses (descriptor, ends of
// the range, records, actions by id, stores), and for large plans the traffic
// of about 80 bytes per agent with the records of the strips' neighbouring
// columns on top.  So as few rounds as the registers allow: up to one block
// per CU, 1024 threads of 4 records (10,000 agents in 9 strips: 3 us less than
// with 512 threads); else 512 threads of 3, which four blocks per CU hold without
// spilling (4 records, 3 blocks per CU: the same on uniform agents, steps 3 %
// slower on clustered ones; 8 records or 256 threads: steps 3 to 25 % slower).
// MI355X, against look-back over all strips of the env, tickets, and a list in
// LDS instead of registers: 256 uneven envs of 0.96 M agents 38.6 -> 25.5 us, 20
// clustered envs of 50,000 57.8 -> 42.2 (the densest strip: 5,800 of its 7,000
// records), 16,000 agents in 20 strips 13.2 -> 11.0, 5,000 in 10 strips
// 9.6 -> 7.7.
// In envs of millions a strip is one column of thousands of agents.  One round of
// probes leaves each end of its range open by n / 256 records, and reading the
// rest twice gathers every action up to six times: one env of 2 million 297 us,
// with ends searched to 512 records 212 (to 128 or 1,024 the same), with the
// list 138 (look-back, tickets and a list of all: 160); four of 4 million 3,800,
// 1,930 and 1,220 (2,050); one of 300,000 34, 28 and 26 (27).
constexpr int kStripNear = 512;          // records to which an end of the range is searched
constexpr int kStripRegs = 512 * 3;      // records in the registers of a block of 512 threads
constexpr int kStripLds = 156 * 1024;    // LDS of a CU's blocks (160 KiB, less the static part)
constexpr uint32_t kStripSet = 1u << 31;  // status word: the env's edge crossings are set
// The wait for that word is bounded (the plan's strip_wait polls).  The first
// strips run at once with the strips that wait for them or come before them in
// the launch (strip_order.h), so the word comes where blocks start in order, but
// nothing guarantees that.  A strip whose wait runs out counts the agents before
// it itself (strip_base_by_count), so the sort stays exact and every block ends.

// The env's agents that the step moves into columns below c0: every old
// record of env E moved as in the strip sort (one wave, all of its lanes
// calling).  The fallback for a wait that ran out, O(n) per call.
__device__ int strip_base_by_count(const DevEnv &E, int c0, int do_move,
                                   const float2 *__restrict__ act) {
    const int lane = threadIdx.x & 63;
    int cnt = 0;
    for (int i = lane; i < E.n; i += 64) {
        float4 m = E.rec_cur[i];
        if (do_move) {
            const int id = E.id_cur[i];
            float2 av = make_float2(0.0f, 0.0f);
            if ((unsigned)id < (unsigned)E.n)
                av = act ? act[E.agent_base + id] : reinterpret_cast<const float2 *>(E.act)[id];
            m = move_record(E, m, av);
        }
        cnt += cell_of(m.x, E.inv_cx, E.ncx) < c0 ? 1 : 0;
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) cnt += __shfl_xor(cnt, d, 64);
    return cnt;
}

template <int NT, int R, int kWaves, bool kOrdered, bool kList>
__global__ __launch_bounds__(NT, kWaves) void k_strip_sort(
    SortArrays a, const DevEnv *__restrict__ envs, int n_envs, int C, int G, int S, int do_move,
    const float2 *__restrict__ act, int tag, float2 *__restrict__ act_copy, int n_ahead,
    int run_len, int run_log, int wait, int cap) {
    // the strip's cells: counts, then each cell's first row; then the list
    extern __shared__ int s_cells[];
    __shared__ int s_wave[NT / 64 + 1], s_probe[NT / 64];
    __shared__ int s_base, s_side, s_listed;
    const int tid = threadIdx.x, lane = tid & 63;
    const int ahead = kOrdered ? n_ahead : 0;
    const int place = strip_place(blockIdx.x, ahead, run_len, kOrdered ? run_log : -1);
    if (place >= S) return;  // a block past the last strip
    const int e = n_envs == 1 ? 0 : a.strip_env[place];
    const DevEnv &E = envs[e];
    const int ls = strip_in_env(place, ahead, e, E.strip_base);
    const int nst = E.n_strips, ncx = E.ncx, ncy = E.ncy, n = E.n;
    const int c0 = ls * E.strip_cols, c1 = ls == nst - 1 ? ncx : c0 + E.strip_cols;
    const int cbase = c0 * ncy, ncell = (c1 - c0) * ncy;
    for (int c = tid; c < ncell; c += NT) s_cells[c] = 0;
    if (tid == 0) s_side = s_listed = 0;
    int *const s_li = s_cells + ((ncell + 3) & ~3), *const s_lc = s_li + cap;
    float2 *const s_la = reinterpret_cast<float2 *>(s_lc + cap);
    // A range of old records that holds those of columns c0 - 1 .. c1
    // (periodic; two ranges where they wrap; all records when they cover the
    // box).  Half the block's waves look for either end, one probe per lane
    // at equal distances: columns are nondecreasing, so the probes below a
    // column are the first ones, and the end lies between the last of them and
    // the next.  More rounds probe between the two while they are more than
    // kStripNear records apart.  The few records too many fall to the column
    // test below.
    int r0 = 0, r1 = n, r2 = 0;  // [r0, r1) and then [0, r2)
    const bool part = nst > 1 && c1 - c0 + 2 < ncx;
    if (part) {
        constexpr int P = NT / 2;
        const int half = tid / P, q = tid - half * P;
        // first column of the range, first column past it
        const int col = half == 0 ? (c0 == 0 ? ncx : c0) - 1 : (c1 == ncx ? 0 : c1) + 1;
        // the probes below an end, `step` records apart from lo0 / lo1 on
        int k0, k1;
        auto probe = [&](int at) {
            const bool lower = at < n && cell_of(gload(E.rec_cur, at).x, E.inv_cx, ncx) < col;
            const uint64_t m = __ballot(lower);
            if (lane == 0) s_probe[tid >> 6] = __popcll(m);
            __syncthreads();
            k0 = k1 = 0;
#pragma unroll
            for (int w = 0; w < NT / 128; ++w) {
                k0 += s_probe[w];
                k1 += s_probe[NT / 128 + w];
            }
            k0 = __builtin_amdgcn_readfirstlane(k0);
            k1 = __builtin_amdgcn_readfirstlane(k1);
        };
        int step = (n + P - 1) / P;
        probe(q * step);
        int lo = k0 > 0 ? (k0 - 1) * step + 1 : 0, hi = min(k1 * step, n);
        int lo1 = k1 > 0 ? (k1 - 1) * step + 1 : 0;
        while (__builtin_expect(step > kStripNear, 0)) {
            const int width = step;
            step = (width + P - 1) / P;
            __syncthreads();  // the last counts are read before the next
            probe(q * step < width ? (half == 0 ? lo : lo1) + q * step : n);
            lo += k0 > 0 ? (k0 - 1) * step + 1 : 0;
            hi = min(lo1 + k1 * step, n);
            lo1 += k1 > 0 ? (k1 - 1) * step + 1 : 0;
        }
        if (c0 == 0 || c1 == ncx) {
            if (lo > hi) r0 = lo, r2 = hi;  // else they meet: all records
        } else {
            r0 = lo;
            r1 = max(hi, lo);
        }
    } else {
        __syncthreads();
    }
    const int len = r1 - r0, total_old = len + r2;
    // the own columns' records first (about: the range's columns counted as equal)
    const int turn = kList && part ? total_old / (c1 - c0 + 2) : 0;
    auto index = [&](int v) {
        const int w = !kList ? v : v + turn < total_old ? v + turn : v + turn - total_old;
        return w < len ? r0 + w : w - len;
    };
    // the wave's count of records now below c0, edge crossings taken back; of
    // the crossings, in minus out, in the first strip
    int side = 0;
    // NT * R old records from v0 on, all loads issued before any is used
    // (each record's action is a gather by its id), each record moved as in
    // k_env_sort; cell[u] < 0: not an agent of this strip
    auto load_move = [&](int v0, int (&id)[R], float4 (&m)[R], float2 (&av)[R], int (&cell)[R],
                         auto count) {
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const int v = v0 + u * NT;
            id[u] = 0;
            m[u] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (v < total_old) {
                const int i = index(v);
                id[u] = gload(E.id_cur, i);
                m[u] = gload(E.rec_cur, i);
            }
        }
#pragma unroll
        for (int u = 0; u < R; ++u) {
            av[u] = make_float2(0.0f, 0.0f);
            if (do_move && v0 + u * NT < total_old && (unsigned)id[u] < (unsigned)n) {
                av[u] = act ? gload(act, E.agent_base + id[u])
                            : gload(reinterpret_cast<const float2 *>(E.act), id[u]);
            }
        }
#pragma unroll
        for (int u = 0; u < R; ++u) {
            cell[u] = -1;
            bool before = false, in = false, out = false;
            if (v0 + u * NT < total_old) {
                const int ox = cell_of(m[u].x, E.inv_cx, ncx);
                if (do_move) m[u] = move_record(E, m[u], av[u]);
                const int cx = cell_of(m[u].x, E.inv_cx, ncx);
                if (cx >= c0 && cx < c1) cell[u] = cx * ncy + cell_of(m[u].y, E.inv_cy, ncy) - cbase;
                in = part && ox == ncx - 1 && cx == 0;
                out = part && ox == 0 && cx == ncx - 1;
                before = out || (cx < c0 && !in);
            }
            if (count) {
                if (ls == 0) side += __popcll(__ballot(in)) - __popcll(__ballot(out));
                else side += __popcll(__ballot(before));
            }
        }
    };
    int id[R], cell[R], rank[R];
    float4 m[R];
    double ret[R];
    {
        float2 av[R];
        load_move(tid, id, m, av, cell, std::true_type{});
#pragma unroll
        for (int u = 0; u < R; ++u) {
            rank[u] = 0;
            ret[u] = 0.0;
            if (cell[u] >= 0) {
                ret[u] = gload(E.ret_cur, index(tid + u * NT));
                rank[u] = atomicAdd(&s_cells[cell[u]], 1);
                if (do_move && act_copy && (unsigned)id[u] < (unsigned)n)
                    act_copy[E.agent_base + id[u]] = av[u];
            }
        }
    }
    // a denser strip's further records: counted now, placed by a second pass
    const bool more = total_old > NT * R;
    for (int v0 = NT * R + tid; v0 < total_old; v0 += NT * R) {
        int id2[R], cell2[R];
        float4 m2[R];
        float2 av[R];
        load_move(v0, id2, m2, av, cell2, std::true_type{});
#pragma unroll
        for (int u = 0; u < R; ++u) {
            int at = 0;
            if constexpr (kList) {
                const uint64_t own = __ballot(cell2[u] >= 0);
                if (own == 0) continue;
                if (lane == 0) at = atomicAdd(&s_listed, __popcll(own));
                at = __builtin_amdgcn_readfirstlane(at) + __popcll(own & ((1ull << lane) - 1ull));
            }
            if (cell2[u] >= 0) {
                atomicAdd(&s_cells[cell2[u]], 1);
                if (kList && at < cap) {
                    s_li[at] = index(v0 + u * NT);
                    s_lc[at] = cell2[u];
                    s_la[at] = av[u];
                }
                if (do_move && act_copy && (unsigned)id2[u] < (unsigned)n)
                    act_copy[E.agent_base + id2[u]] = av[u];
            }
        }
    }
    if (lane == 0 && side != 0) atomicAdd(&s_side, side);
    __syncthreads();
    uint32_t *const word = &a.status[E.strip_base];
    if (ls == 0 && nst > 2 && tid == 0)
        __hip_atomic_store(word, kStripSet | ((uint32_t)s_side & ~kStripSet), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    // exclusive scan of the counts: thread t owns cells [t k, t k + k)
    const int per = (ncell + NT - 1) / NT;
    const int q0 = tid * per;
    int sum = 0;
    for (int c = q0; c < q0 + per && c < ncell; ++c) sum += s_cells[c];
    int total;
    int run = block_exclusive_scan<NT>(sum, s_wave, &total);
    for (int c = q0; c < q0 + per && c < ncell; ++c) {
        const int cnt = s_cells[c];
        s_cells[c] = run;
        run += cnt;
    }
    if (tid < 64) {
        // the env's agents before this strip
        int base = 0;
        if (ls == nst - 1) {
            base = n - total;
        } else if (ls > 0) {
            base = s_side;
            if (part) {
                uint32_t w = 0;
                int polls = 0;
                while (polls < wait && !(w & kStripSet)) {
                    w = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    ++polls;
                }
                if (w & kStripSet) base += r0 + ((int)(w << 1) >> 1);
                else base = strip_base_by_count(E, c0, do_move, act);
                base = max(0, min(base, n - total));  // whatever the records hold
            }
        }
        if (lane == 0) {
            s_base = base;
            if (blockIdx.x == 0) a.start[C] = G;
        }
    }
    __syncthreads();
    const int base = s_base;
    for (int c = tid; c < ncell; c += NT) a.start[E.cell_base + cbase + c] = E.agent_base + base + s_cells[c];
    auto put = [&](int j, const float4 &r, int who, double sum_ret) {
        ((FLOCK_GLOBAL gfloat4 *)E.rec_nxt)[j] = gfloat4{r.x, r.y, r.z, r.w};
        gstore(E.id_nxt, j, who);
        gstore(E.ret_nxt, j, sum_ret);
        a.sxy[E.agent_base + j] = make_float2(r.x, r.y);
        if (tag) a.stype[E.agent_base + j] = who < E.n_chasers ? 1 : 0;
    };
    if (!more) {
#pragma unroll
        for (int u = 0; u < R; ++u)
            if (cell[u] >= 0) put(base + s_cells[cell[u]] + rank[u], m[u], id[u], ret[u]);
        return;
    }
    __syncthreads();  // the starts are read before they become row cursors
#pragma unroll
    for (int u = 0; u < R; ++u)
        if (cell[u] >= 0) put(base + atomicAdd(&s_cells[cell[u]], 1), m[u], id[u], ret[u]);
    const int listed = s_listed;
    if (kList && listed <= cap) {
        for (int k0 = tid; k0 < listed; k0 += NT * R) {
            int at[R];
#pragma unroll
            for (int u = 0; u < R; ++u) {
                const int k = min(k0 + u * NT, listed - 1);
                at[u] = s_li[k];
                id[u] = gload(E.id_cur, at[u]);
                m[u] = gload(E.rec_cur, at[u]);
                ret[u] = gload(E.ret_cur, at[u]);
            }
#pragma unroll
            for (int u = 0; u < R; ++u) {
                const int k = k0 + u * NT;
                if (k >= listed) continue;
                const float4 r = do_move ? move_record(E, m[u], s_la[k]) : m[u];
                put(base + atomicAdd(&s_cells[s_lc[k]], 1), r, id[u], ret[u]);
            }
        }
        return;
    }
    for (int v0 = NT * R + tid; v0 < total_old; v0 += NT * R) {
        float2 av[R];
        load_move(v0, id, m, av, cell, std::false_type{});
#pragma unroll
        for (int u = 0; u < R; ++u)
            if (cell[u] >= 0) ret[u] = gload(E.ret_cur, index(v0 + u * NT));
#pragma unroll
        for (int u = 0; u < R; ++u)
            if (cell[u] >= 0) put(base + atomicAdd(&s_cells[cell[u]], 1), m[u], id[u], ret[u]);
    }
}

// ------------------------------------------------------------------ scatter

__global__ __launch_bounds__(kBlock) void k_scatter(SortArrays a, const DevEnv *__restrict__ envs,
                                                    int n_envs, int G, int tag) {
    __shared__ int s_env;
    const int p0 = blockIdx.x * kBlock;
    block_env(&s_env, a.base, n_envs, p0);
    __syncthreads();
    const int p = p0 + threadIdx.x;
    if (p >= G) return;
    int e = s_env;
    while (a.base[e + 1] <= p) ++e;
    const DevEnv &E = envs[e];
    const int i = p - E.agent_base;
    const int pos = a.start[a.key[p]] + a.slot[p];
    const int j = pos - E.agent_base;
    const float4 r = a.tmp[p];
    const int id = E.id_cur[i];
    E.rec_nxt[j] = r;
    E.id_nxt[j] = id;
    E.ret_nxt[j] = E.ret_cur[i];
    a.sxy[pos] = make_float2(r.x, r.y);
    if (tag) a.stype[pos] = id < E.n_chasers ? 1 : 0;
}

// -------------------------------------------------------------------- sweep

// atan(t) / (2 pi) for t in [0, 1] as t * P(t^2); least-squares fit with
// minimax reweighting on Chebyshev nodes, max error 5.4e-8 turns.
__device__ __forceinline__ float atan_turns01(float t) {
    const float t2 = t * t;
    float p = 0.0010841276962310076f;
    p = __builtin_fmaf(t2, p, -0.005348269362002611f);
    p = __builtin_fmaf(t2, p, 0.012672491371631622f);
    p = __builtin_fmaf(t2, p, -0.02106151357293129f);
    p = __builtin_fmaf(t2, p, 0.03152511641383171f);
    p = __builtin_fmaf(t2, p, -0.0530262365937233f);
    p = __builtin_fmaf(t2, p, 0.15915432572364807f);
    return p * t;
}

// Sector of the bearing of (dx, dy) relative to the heading (c, s): sector 0
// starts at the heading, sectors run counter-clockwise; (0, 0) -> sector 0.
__device__ __forceinline__ int sector_of(float dx, float dy, float c, float s, float vf, int v) {
    const float u = __builtin_fmaf(dx, c, dy * s);      // along the heading
    const float w = __builtin_fmaf(dy, c, -(dx * s));   // to its left
    const float au = fabsf(u), aw = fabsf(w);
    const float mx = fmaxf(au, aw), mn = fminf(au, aw);
    const float t = mx > 0.0f ? mn * __builtin_amdgcn_rcpf(mx) : 0.0f;
    float a = atan_turns01(t);
    a = aw > au ? 0.25f - a : a;
    a = u < 0.0f ? 0.5f - a : a;
    a = w < 0.0f ? 1.0f - a : a;
    const int k = (int)(a * vf);
    return k < v - 1 ? k : v - 1;
}

// As sector_of for a full view with v = 8 M sectors (M sectors per octant),
// without the arctangent: the octant comes from the signs and the larger of
// |u| and |w|, the sector within it from comparing min/max with the
// tangents of the octant's interior sector edges, and mirrored octants
// count their sectors backwards.  A bearing exactly on an octant edge may
// land in either neighbouring sector (both are within the ambiguity band).
//
// Comparisons, selections and minima issue at half the rate of FP32 additions,
// multiplications and bitwise operations on gfx950 (0.9 against 1.7 wave
// instructions per clock per CU, measured), so the conditions are the sign
// bits of differences (exact in sign; + 0 turns a -0 into +0).
template <int M>
__device__ __forceinline__ int sector_oct(float dx, float dy, float c, float s) {
    const float u = __builtin_fmaf(dx, c, dy * s) + 0.0f;
    const float w = __builtin_fmaf(dy, c, -(dx * s)) + 0.0f;
    // mirroring within [0, 2^b) is an XOR with 2^b - 1, so the three mirrors
    // (past 45 degrees, past 90, past 180) flip whole bit groups: the top bit
    // is w < 0, the next (u < 0) ^ (w < 0), the lower ones that ^ (|w| > |u|),
    // and the sector within the octant flips with those
    const uint32_t x3 = __float_as_uint(w);
    const uint32_t x2 = x3 ^ __float_as_uint(u);
    const uint32_t x1 = x2 ^ __float_as_uint(fabsf(u) - fabsf(w));
    const uint32_t oct =
        __builtin_amdgcn_alignbit(__builtin_amdgcn_alignbit(x3 >> 31, x2, 31), x1, 31);
    // min(|u|, |w|) > t max(|u|, |w|) for t < 1, as a sign: both |u| > t |w| and
    // |w| > t |u| (no division; a coincident pair stays in sector 0)
    auto past = [&](float t) {
        return __float_as_uint(fabsf(t * w) - fabsf(u)) & __float_as_uint(fabsf(t * u) - fabsf(w));
    };
    if constexpr (M == 1) return (int)oct;
    else if constexpr (M == 2)
        return (int)__builtin_amdgcn_alignbit(oct, x1 ^ past(0.41421356237309503f), 31);  // tan(pi/8)
    else {
        static_assert(M == 4, "sector_oct takes M = 1, 2 or 4");
        // edges passed, 0 .. 3: tan(pi/16), tan(pi/8), tan(3 pi/16)
        const uint32_t e1 = past(0.19891236737965800f), e2 = past(0.41421356237309503f),
                       e3 = past(0.66817863791929891f);
        return (int)__builtin_amdgcn_alignbit(__builtin_amdgcn_alignbit(oct, x1 ^ e2, 31),
                                              x1 ^ e1 ^ e2 ^ e3, 31);
    }
}

// View sector of the bearing of (dx, dy) for a limited field of view: the
// bearing in turns from the heading (as in sector_of), shifted by half the
// arc and wrapped, is seen iff it lies in the arc; -1 when not seen.  A
// coincident agent counts as straight ahead: the middle sector v/2.
__device__ __forceinline__ int view_sector(float dx, float dy, float c, float s, float fov_half,
                                           float fov_t, float sec_scale, int v) {
    const float u = __builtin_fmaf(dx, c, dy * s);
    const float w = __builtin_fmaf(dy, c, -(dx * s));
    const float au = fabsf(u), aw = fabsf(w);
    const float mx = fmaxf(au, aw), mn = fminf(au, aw);
    const float t = mx > 0.0f ? mn * __builtin_amdgcn_rcpf(mx) : 0.0f;
    float a = atan_turns01(t);
    a = aw > au ? 0.25f - a : a;
    a = u < 0.0f ? 0.5f - a : a;
    a = w < 0.0f ? 1.0f - a : a;
    float p = a + fov_half;
    p = p >= 1.0f ? p - 1.0f : p;
    int k = (int)(p * sec_scale);
    k = p < fov_t ? (k < v - 1 ? k : v - 1) : -1;
    return mx > 0.0f ? k : (v >> 1);
}

// Periodic displacement for single-cell (all-pairs) envs: the shift by L is
// applied to whichever operand lies in the far half, where it is exact.
__device__ __forceinline__ float min_image_delta(float xj, float xi, float L) {
    const float d = xj - xi;
    if (d > 0.5f * L) return (xj - L) - xi;
    if (d < -0.5f * L) return xj - (xi - L);
    return d;
}

// View constants of the lane's agent (see DevEnv).
struct ViewK {
    float c, s;                       // cos / sin of the heading
    float fov_half, fov_t, sec_scale;
    float vf;
    int v;
};

// Test candidate qq against the lane's agent (ok: the slot holds a candidate
// other than the agent itself): distance test, and for a
// neighbour the count, the collision count and the per-sector minimum (an
// LDS atomic min on the agent's own minima, S words apart).  The sector is
// computed for every candidate (branch-free); only the LDS update is
// predicated.  (offx, xi), (offy, yi): candidate shift (0 or -L) and
// centre (x or x - L) per axis; minimg selects the per-candidate minimum
// image (single-cell envs).  kFov selects the limited-view sector
// (candidates outside the arc are counted but update no sector).
//
// kTag (tag environment): candidate q's type stype[q] picks the view channel
// (minima at smin_own[(tj v + k) S]); nb counts runners in range and col
// touches with the other type (the lane's own type is ti).
// kShiftX / kShiftY: the candidate-side shift offx / offy may be nonzero (a
// zero shift is left out: x + 0 = x for the nonnegative coordinates here).
template <int S, bool kFov, bool kTag, int kM, bool kShiftX, bool kShiftY>
__device__ __forceinline__ void test_pair(uint32_t *smin_own, const uint8_t *__restrict__ stype,
                                          int ti, const float2 pj, int qq, bool ok, float offx,
                                          float xi, float offy, float yi, bool minimg, float L,
                                          float r2, float c2, const ViewK &K, int &nb, int &col) {
    float dx, dy;
    if (minimg) {
        dx = min_image_delta(pj.x, xi, L);
        dy = min_image_delta(pj.y, yi, L);
    } else {
        dx = (kShiftX ? pj.x + offx : pj.x) - xi;
        dy = (kShiftY ? pj.y + offy : pj.y) - yi;
    }
    const float d2 = __builtin_fmaf(dx, dx, dy * dy);
    const bool nbr = ok && d2 < r2;
    int ch = 0;  // view channel offset (sectors)
    if constexpr (kTag) {
        const int tj = stype[qq];
        nb += (nbr && tj == 0) ? 1 : 0;
        col += (nbr && tj != ti && d2 < c2) ? 1 : 0;
        ch = tj * K.v;
    } else if constexpr (kFov) {
        nb += nbr ? 1 : 0;
        col += (nbr && d2 < c2) ? 1 : 0;
    }
    if (kFov) {
        const int k = view_sector(dx, dy, K.c, K.s, K.fov_half, K.fov_t, K.sec_scale, K.v);
        if (nbr && k >= 0) atomicMin(&smin_own[(ch + k) * S], __float_as_uint(d2));
    } else {
        int k;
        if constexpr (kM > 0) k = sector_oct<kM>(dx, dy, K.c, K.s);
        else k = sector_of(dx, dy, K.c, K.s, K.vf, K.v);
        if (nbr) {
            // full view: the counts go with the neighbour's branch, which some
            // lane of the wave takes on nearly every slot anyway
            if constexpr (!kTag) {
                ++nb;
                if (d2 < c2) ++col;
            }
            atomicMin(&smin_own[(ch + k) * S], __float_as_uint(d2));
        }
    }
}

// Candidates per step of a run walked on its own (one lane per agent, stencil
// half-width 2 or a single cell).
constexpr int kRunUnroll = 4;

template <int S, bool kFov, bool kTag, int kM, bool kShiftX, bool kShiftY>
__device__ __forceinline__ void sweep_run(uint32_t *smin_own, const float2 *__restrict__ sxy,
                                          const uint8_t *__restrict__ stype, int ti,
                                          int q, int q1, int self, float offx, float xi,
                                          float offy, float yi, bool minimg, float L, float r2,
                                          float c2, const ViewK &K, int &nb, int &col) {
    // kRunUnroll candidates per step, those past the run's end masked (the
    // position arrays are padded for the reads)
    for (; q < q1; q += kRunUnroll) {
        float2 pj[kRunUnroll];
#pragma unroll
        for (int u = 0; u < kRunUnroll; ++u) pj[u] = sxy[q + u];
#pragma unroll
        for (int u = 0; u < kRunUnroll; ++u)
            test_pair<S, kFov, kTag, kM, kShiftX, kShiftY>(smin_own, stype, ti, pj[u], q + u,
                                                           q + u < q1 && q + u != self, offx, xi,
                                                           offy, yi, minimg, L, r2, c2, K, nb, col);
    }
}

// Rows [lo, hi] of the column ox columns from the agent's own that can hold
// a point within the vision radius: the column's nearest x lies dmin from
// the agent, so only |dy| < sqrt(R^2 - dmin^2) matters.  fx is the agent's
// offset within its own column.  Both bounds widen by E.marg, which covers
// the FP32 rounding of the row assignment, of these bounds and of the pair
// test.  hi - lo < ncy; lo < 0 or hi >= ncy wrap through the column's ends.
// False when no point of the column is within the radius.
struct RowGeom {
    float cw, marg, r2, inv_cy;
    int ncy;
};

__device__ __forceinline__ bool column_rows(const RowGeom &E, float fx, int ox, float y, int &lo,
                                            int &hi) {
    float dmin = 0.0f;
    if (ox < 0) dmin = fx + (float)(-ox - 1) * E.cw;
    else if (ox > 0) dmin = (E.cw - fx) + (float)(ox - 1) * E.cw;
    dmin = fmaxf(dmin - E.marg, 0.0f);
    const float e2 = E.r2 - dmin * dmin;
    if (!(e2 > 0.0f)) return false;
    const float ext = __builtin_amdgcn_sqrtf(e2) + E.marg;  // within 1 ulp
    const int n = E.ncy;
    int l = (int)floorf((y - ext) * E.inv_cy);
    int h = (int)floorf((y + ext) * E.inv_cy);
    // in range for finite positions in [0, L); the clamps keep any other
    // input inside the column (memory safety only)
    l = max(min(l, n - 1), -n);
    h = max(min(h, l + n - 1), l);
    lo = l;
    hi = h;
    return true;
}

// One lane per agent, stencil half-width 1: walk the agent's runs as one
// sequence (a lane moves to its next run as soon as its current one ends)
// instead of run by run, so a wave waits for its longest total rather than
// for the longest lane of every run.  The runs are found once per agent and
// queued in registers: lanes switch runs at different steps, so whatever a
// switch costs is paid by the whole wave on nearly every step.
constexpr bool kFlatRuns = true;
// Candidates per step of the flat walk; step of 200 x 5,000 agents, 16 sectors:
// 4 -> 70.1 us, 5 -> 71.0, 6 -> 70.6, 8 -> 73.2.
constexpr int kFlatUnroll = 4;
// Candidates per lane and step of a lane group's run (four lanes without the
// queue: 4).
constexpr int kGroupUnroll = 2;
// Entries past the end of the cell-order position and type arrays, so that a
// step's reads past the last run stay inside the allocation: a lane reads at
// most kGroupUnroll * G - 1 entries (lane groups of G <= 64) or kFlatUnroll - 1
// entries past its run's end.
constexpr int kSortPad = 256;
static_assert(kFlatUnroll <= kSortPad + 1 && kRunUnroll <= kSortPad + 1 && 4 * 4 <= kSortPad + 1 &&
                  kGroupUnroll * 64 <= kSortPad + 1,
              "pad the cell-order arrays for the unrolled reads");

// The runs of one agent's flat walk (one lane per agent, one column either
// side), for an agent at (fx into its column cx, y): slot c (c < 3) holds
// column cx + c - 1's first segment, slot 3 + c its second (empty unless the
// rows wrap), each as [rq, rq1) in cell order, with 4 bits of shift flags per
// slot in fl (1 candidate x - L, 2 centre x - L, 4 candidate y - L, 8 centre
// y - L).  nr: the slots up to the last nonempty one, which the walk takes in
// order.
struct FlatRuns {
    int rq[6], rq1[6];
    uint32_t fl;
    int nr;
};

__device__ __forceinline__ void flat_runs(const RowGeom &RG, const int32_t *__restrict__ start,
                                          int cb, int ncx, int cx, float fx, float y,
                                          FlatRuns &F) {
    const int ncy = RG.ncy;
    F.fl = 0u;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        int lo = 0, hi = -1;
        const bool any = column_rows(RG, fx, c - 1, y, lo, hi);
        int ccx = cx + c - 1;
        uint32_t fxs = 0;
        if (ccx < 0) {
            ccx += ncx;
            fxs = 1;
        } else if (ccx >= ncx) {
            ccx -= ncx;
            fxs = 2;
        }
        const int colb = cb + ccx * ncy;
        const bool wlo = lo < 0, whi = hi >= ncy;
        // first segment [ia, ib), second [colb, id)
        int ia = colb + (wlo ? lo + ncy : lo);
        int ib = colb + ((wlo || whi) ? ncy : hi + 1);
        int id = colb + (wlo ? hi + 1 : (whi ? hi - ncy + 1 : 0));
        if (!any) ia = ib = id = colb;
        F.rq[c] = start[ia];
        F.rq1[c] = start[ib];
        F.rq[3 + c] = start[colb];
        F.rq1[3 + c] = start[id];
        F.fl |= (fxs | (wlo ? 4u : 0u)) << (4 * c);
        F.fl |= (fxs | (whi ? 8u : 0u)) << (4 * (3 + c));
    }
    int nr = 0;
#pragma unroll
    for (int k = 0; k < 6; ++k) nr = F.rq1[k] > F.rq[k] ? k + 1 : nr;
    F.nr = nr;
}

// ---- lane groups: G lanes share an agent, 64 / G agents to a wave
//
// A wave's neighbours pass through a queue in LDS.  Distance tests (some ten
// vector instructions per candidate) push the displacement of each candidate
// in range, and its agent's place in the wave; whenever 64 are queued, each
// lane takes one and evaluates its bearing, sector and minimum (30 to 50
// instructions), for whichever agent it belongs to.  Testing and seeing in
// one pass paid the bearing for every candidate slot, since some lane of a
// wave has a neighbour on nearly each of them.  Bound by vector-ALU issue
// (10,000 agents, 128 sectors, 250 degrees, 64 lanes: 998 -> 671 wave
// instructions per agent; the launch 22.8 -> 17.7 us, 16,000 agents at reach
// two 36.6 -> 28.9 us).
constexpr int kQueue = 63 + 64 * kGroupUnroll + 1;  // entries: a rest below 64, one step's pushes

// Whether a lane group's sweep queues its neighbours (meta: bytes per entry
// beside its displacement, 0 for plans of single cells): views whose sector takes the
// arctangent, and steps of 64 lanes.  Sectors by octant (kM > 0) cost
// about what a push and a pop do, so where most candidates are neighbours they
// are evaluated in place (20 x 50,000 clustered agents at four lanes: 266 us
// per step against 309 queued, 282 before); with 64 lanes few lanes of a slot
// have one (one 5,000-agent env: 16.7 us per step against 17.7 in place).
// Single cells, whose boxes are hardly wider than a view, are evaluated in
// place at four lanes, and at 16 if the view is full (1,000 agents in a box of
// 20, 20 sectors, four lanes: 79 us per step, 95 queued, with a view of 250
// degrees 88 and 101; 200 envs of 600 at 16 lanes 98 and 102); plans of nothing
// else have no queue there.
__host__ __device__ constexpr bool queued(int G, int kM, int meta) {
    return meta > 0 && (kM == 0 || G == 64);
}

// 32-bit words of LDS per wave.
__host__ __device__ constexpr int queue_words(int G, int kM, int meta) {
    return queued(G, kM, meta) ? (2 * kQueue + meta * kQueue / 4 + 3 * (64 / G) + 3) & ~3 : 0;
}

template <int kMeta>
struct WaveQueue {
    using Meta = std::conditional_t<kMeta == 1, uint8_t, uint32_t>;
    float *x, *y;        // [kQueue] displacement of a neighbour from its agent
    float2 *cs;          // [64 / G] cos / sin of the agents' headings
    int *col;            // [64 / G] collisions (tag: touches)
    Meta *meta;          // [kQueue] agent of the entry; tag: + 64 type, + 128 types differ
};

template <int G, int kMeta>
__device__ __forceinline__ WaveQueue<kMeta> wave_queue(uint32_t *words) {
    WaveQueue<kMeta> Q;
    Q.x = reinterpret_cast<float *>(words);
    Q.y = Q.x + kQueue;
    Q.cs = reinterpret_cast<float2 *>(words + 2 * kQueue);
    Q.col = reinterpret_cast<int *>(Q.cs + 64 / G);
    Q.meta = reinterpret_cast<typename WaveQueue<kMeta>::Meta *>(Q.col + 64 / G);
    return Q;
}

// n + (the lane's bit of mask b) in one vector instruction.
__device__ __forceinline__ int add_bit(int n, uint64_t b) {
    uint64_t carry;
    int r;
    asm("v_addc_co_u32_e64 %0, %1, 0, %2, %3" : "=v"(r), "=s"(carry) : "v"(n), "s"(b));
    return r;
}

// The candidates of the wave's agents: neighbours per lane into nb (tag:
// runners), minima and collision counts in LDS.  mine: the lane's agent exists;
// every lane of the wave takes part.  smin_w: minima of the wave's first agent
// (agent i's i words on).  E is the env of all of them, or, with kMixed, that of
// the lane's own agent: then every value of it differs from lane to lane.
template <int A, int G, bool kFov, bool kTag, int kM, bool kMixed, int kMeta>
__device__ __forceinline__ void sweep_group(const SortArrays &a, const DevEnv &E, uint32_t *smin_w,
                                            const WaveQueue<kMeta> &Q, bool mine, float4 me, int pos,
                                            int ti, const ViewK &K, int &nb, int &col) {
    const int lane = threadIdx.x & 63, li = lane % G, own = lane / G;
    const float L = E.box, r2 = E.r2, c2 = E.c2;
    const int ncx = E.ncx, ncy = E.ncy, cb = E.cell_base, reach = E.reach;
    constexpr bool kQueued = queued(G, kM, kMeta);
    using Meta = typename WaveQueue<kMeta>::Meta;
    int cnt = 0;  // queued entries (wave-uniform)

    // the last n (at most 64) entries, one per lane
    auto drain = [&](int n) {
        cnt -= n;
        wave_lds_fence();
        int o = 0, meta = 0;
        if constexpr (G < 64 || kTag) {
            if (lane < n) meta = (int)Q.meta[cnt + lane];
            o = kTag ? meta & 63 : meta;
        }
        // what the entry's agent's env says of it
        float oc2 = c2, ohalf = K.fov_half, ot = K.fov_t, oscale = K.sec_scale;
        if constexpr (kMixed) {
            oc2 = __shfl(c2, o * G, 64);
            if constexpr (kFov) {
                ohalf = __shfl(K.fov_half, o * G, 64);
                ot = __shfl(K.fov_t, o * G, 64);
                oscale = __shfl(K.sec_scale, o * G, 64);
            }
        }
        if (lane < n) {
            const float2 d = make_float2(Q.x[cnt + lane], Q.y[cnt + lane]);
            const float2 cs = G < 64 ? Q.cs[o] : make_float2(K.c, K.s);
            const float d2 = __builtin_fmaf(d.x, d.x, d.y * d.y);
            int ch = 0;
            if constexpr (kTag) ch = (meta & 64) ? K.v : 0;
            int k;
            if constexpr (kFov)
                k = view_sector(d.x, d.y, cs.x, cs.y, ohalf, ot, oscale, K.v);
            else if constexpr (kM > 0) k = sector_oct<kM>(d.x, d.y, cs.x, cs.y);
            else k = sector_of(d.x, d.y, cs.x, cs.y, K.vf, K.v);
            if (!kFov || k >= 0) atomicMin(&smin_w[(ch + k) * A + o], __float_as_uint(d2));
            if (d2 < oc2 && (!kTag || (meta & 128))) atomicAdd(&Q.col[o], 1);
        }
        wave_lds_fence();
    };
    // candidates [q, q + len) of the lane's group (lane li takes every G-th);
    // kMode 1: candidate shifts (offx, offy), centres (xi, yi); 2: minimum
    // image; kSelf: the agent itself may be among them
    auto run = [&](auto kmode, auto kself, int q, int len, float offx, float xi, float offy,
                   float yi) {
        constexpr int kMode = decltype(kmode)::value;
        if constexpr (!kQueued || (kMode == 2 && G <= 16 && !kFov && !kTag)) {
            constexpr int U = G == 4 ? 4 : kGroupUnroll;
            for (int t = li; t < len; t += U * G) {
                float2 p[U];
#pragma unroll
                for (int u = 0; u < U; ++u) p[u] = a.sxy[q + t + u * G];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    bool ok = t + u * G < len;
                    if constexpr (decltype(kself)::value) ok = ok && q + t + u * G != pos;
                    test_pair<A, kFov, kTag, kM, kMode == 1, kMode == 1>(
                        smin_w + own, a.stype, ti, p[u], q + t + u * G, ok, offx,
                        kMode == 1 ? xi : me.x, offy, kMode == 1 ? yi : me.y, kMode == 2, L, r2,
                        c2, K, nb, col);
                }
            }
            if (kQueued && col > 0) {
                atomicAdd(&Q.col[own], col);
                col = 0;
            }
            return;
        }
        for (int t = li; __any(t < len); t += kGroupUnroll * G) {
            const int at = G < 64 && t >= len ? q : q + t;
            float2 p[kGroupUnroll];
            int tj[kGroupUnroll];
#pragma unroll
            for (int u = 0; u < kGroupUnroll; ++u) {
                p[u] = a.sxy[at + u * G];
                if constexpr (kTag) tj[u] = a.stype[at + u * G];
            }
#pragma unroll
            for (int u = 0; u < kGroupUnroll; ++u) {
                float dx, dy;
                if constexpr (kMode == 0) {
                    dx = p[u].x - me.x;
                    dy = p[u].y - me.y;
                } else if constexpr (kMode == 1) {
                    dx = (p[u].x + offx) - xi;
                    dy = (p[u].y + offy) - yi;
                } else {
                    dx = min_image_delta(p[u].x, me.x, L);
                    dy = min_image_delta(p[u].y, me.y, L);
                }
                // lane masks (combined by scalar instructions)
                uint64_t b = __ballot(__builtin_fmaf(dx, dx, dy * dy) < r2) &
                             __ballot(t + u * G < len);
                if constexpr (decltype(kself)::value) b &= ~__ballot(q + t + u * G == pos);
                if (b == 0) continue;
                const int n = __popcll(b);
                if constexpr (kTag) nb = add_bit(nb, b & __ballot(tj[u] == 0));
                else if constexpr (G < 64) nb = add_bit(nb, b);
                else nb += n;
                const uint32_t k = __builtin_amdgcn_mbcnt_hi(
                    (uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
                if (__builtin_amdgcn_inverse_ballot_w64(b)) {
                    (Q.x + cnt)[k] = dx;
                    (Q.y + cnt)[k] = dy;
                    if constexpr (kTag)
                        (Q.meta + cnt)[k] = (Meta)(own | (tj[u] ? 64 : 0) | (tj[u] != ti ? 128 : 0));
                    else if constexpr (G < 64) (Q.meta + cnt)[k] = (Meta)own;
                }
                cnt += n;
            }
            while (cnt >= 64) drain(64);
        }
    };
    using Yes = std::true_type;
    using No = std::false_type;
    using Plain = std::integral_constant<int, 0>;
    using Shift = std::integral_constant<int, 1>;
    using Image = std::integral_constant<int, 2>;

    const bool single = mine && ncx == 1;
    if (kMixed ? __any(single) : ncx == 1)
        run(Image{}, Yes{}, a.start[cb], single ? a.start[cb + 1] - a.start[cb] : 0, 0.0f, 0.0f, 0.0f, 0.0f);
    if (kMeta > 0 && (kMixed ? __any(mine && ncx > 1) : ncx > 1)) {
        const int cx = cell_of(me.x, E.inv_cx, ncx);
        const float fx = me.x - (float)cx * E.cw;  // offset within the own column
        const RowGeom RG{E.cw, E.marg, r2, E.inv_cy, ncy};
        const int nc = kMixed && __any(mine && reach == 2) ? 5 : 2 * (kMixed ? 1 : reach) + 1;
        // lane li plans column li (four lanes: and column 4 + li): run A, its
        // rows inside the column, and run B, those that wrap through the
        // column's ends (as [q, q + l) in cell order)
        constexpr int kSets = G < 5 ? 2 : 1;
        int qa[kSets], la[kSets], qb[kSets], lb[kSets];
#pragma unroll
        for (int r = 0; r < kSets; ++r) {
            const int c = min(li + r * G, 2 * reach), ox = c - reach;
            int lo = 0, hi = -1;
            const bool any = column_rows(RG, fx, ox, me.y, lo, hi);
            int ccx = cx + ox;
            ccx = ccx < 0 ? ccx + ncx : (ccx >= ncx ? ccx - ncx : ccx);
            const int colb = cb + ccx * ncy;
            const int i0 = min(max(lo, 0), ncy), i1 = min(max(hi + 1, i0), ncy);
            const int j0 = lo < 0 ? lo + ncy : 0, j1 = lo < 0 ? ncy : max(hi + 1 - ncy, 0);
            qa[r] = a.start[colb + i0];
            la[r] = a.start[colb + i1] - qa[r];
            qb[r] = lb[r] = 0;
            if (j1 > j0) {
                qb[r] = a.start[colb + j0];
                lb[r] = a.start[colb + j1] - qb[r];
            }
            if (!mine || !any || (kMixed && (ncx == 1 || c < li + r * G))) la[r] = lb[r] = 0;
        }
        const bool wraps = __any(lb[0] > 0 || lb[kSets - 1] > 0);
        // a column left of column 0 wraps to the right edge with its candidates
        // shifted by -L, one right of the last to the left edge with the centre
        // shifted instead; rows wrap likewise (only near one end: 2 R < L)
        const bool low = me.y < 0.5f * L;
        const float oyb = low ? -L : 0.0f, yb = low ? me.y : me.y - L;
        for (int c = 0; c < nc; ++c) {
            const int r = kSets > 1 && c >= G ? 1 : 0;
            auto of = [&](const int (&x)[kSets]) {
                const int v = kSets > 1 && r ? x[kSets - 1] : x[0];
                if constexpr (G == 64) return __builtin_amdgcn_readlane(v, c);
                else return __shfl(v, (lane & ~(G - 1)) + c - r * G, 64);
            };
            const int ccx = cx + c - reach;
            const float offx = ccx < 0 ? -L : 0.0f, xi = ccx >= ncx ? me.x - L : me.x;
            const int q = of(qa), l = of(la);
            if (kMixed || __any(ccx < 0 || ccx >= ncx)) run(Shift{}, Yes{}, q, l, offx, xi, 0.0f, me.y);
            else if (c == reach) run(Plain{}, Yes{}, q, l, 0.0f, 0.0f, 0.0f, 0.0f);
            else run(Plain{}, No{}, q, l, 0.0f, 0.0f, 0.0f, 0.0f);
            if (wraps) {
                const int w = of(lb);
                if (__any(w > 0)) run(Shift{}, Yes{}, of(qb), w, offx, xi, oyb, yb);
            }
        }
    }
    if (kQueued && cnt > 0) drain(cnt);
}

// NT threads per block, G lanes per agent (in the new cell order): A = NT/G
// agents per block, their sector minima v * A * 4 bytes of dynamic LDS.  G = 1
// suits sparse neighbourhoods (a few dozen candidates); dense ones (hundreds
// to thousands of candidates per agent) share each agent's candidate runs
// among a lane group, which keeps the lanes busy and the LDS per agent small.
// kFov: some env of the launch has a limited field of view.  obs rows hold
// obs_dim floats: the v sectors, then the speed when obs_dim > v.
// kM > 0: full view with v = 8 kM sectors (sector_oct); 0: any v.
//
// kPol (1 mean action, 2 Gaussian sample; not with kTag): the shared policy
// runs on the views the block has just produced, still in LDS, and writes each
// agent's next action (PolFuse).  The views replace the minima in LDS, the
// block's agents are cut into 16-agent tiles spread over its waves, and each
// tile goes through mlp_tile as in the policy kernels.  LDS after the minima:
// the network constants, per-agent speed / env / id, one hidden tile per wave.
// With one lane per agent a wave's agents are its own lanes: each wave runs
// its tiles as soon as its views are written, reading the inputs of its four
// tiles into registers first when they fit one chunk (kc == 1), after which
// its own stretch of the minima (16 rows of 64 words, v >= 16) serves as its
// hidden tile; otherwise (and with four lanes per agent, which needs a block
// barrier) the hidden tiles have a region of their own.  Smaller blocks (lane
// groups of 16 or 64) would read the weights once per tile and are not fused.
struct SweepPolLds {
    int pc, speed, env, id, hid, words;  // offsets in 32-bit words from the minima's start
};
__host__ __device__ constexpr bool sweep_pol_alias(int G, int kc, int vs) {
    return G == 1 && kc == 1 && vs >= 16;
}
__host__ __device__ constexpr SweepPolLds sweep_pol_lds(int min_words, int A, int NT, int G,
                                                        bool alias) {
    const int pc = (min_words + 3) & ~3;
    const int speed = pc + (int)((sizeof(PolConsts) + 15) / 16) * 4;
    const int per_agent = G == 1 ? 0 : A;  // one lane per agent: shuffled from the owner lane
    const int env = speed + per_agent, id = env + per_agent;
    const int hid = (id + per_agent + 3) & ~3;
    return SweepPolLds{pc, speed, env, id, hid, hid + (alias ? 0 : (NT / 64) * 16 * kHidLd / 2)};
}

// Blocks go to the XCDs round robin, and each XCD has an L2 of its own.  The
// sweep hands each XCD runs of 2^log_run consecutive blocks, so that the
// agent-order rows and rewards an env's agents write merge into whole lines in
// one L2, and candidates are read into one, instead of into all eight.  Of the
// blocks left over after the whole rounds, each XCD takes one eighth, and the
// last few stay in place.  With one lane per agent, whose sweep is half bound
// by those lines, runs hold 8,192 agents (200 x 5,000 agents: 72.1 us per step
// without runs, 71.3 with 1,024 agents each, 69.5 with 2,048, 68.9 with 4,096,
// 69.2 with 8,192; 256 uneven envs 82.0, 82.0, 81.0, 79.6, 78.7).  Lane groups
// sweep dense neighbourhoods, whose agents differ in cost and lie together in
// cell order: 256 agents keep the XCDs' shares even (20 x 50,000 clustered,
// four lanes: 257 -> 252 us; 16,000 agents drawn together by their policy, 64
// lanes: 4.7 ms per 128 steps, 5.1 with runs of 1,024, 5.3 of 4,096).
constexpr int kSweepRunOne = 13, kSweepRunGroup = 8;  // log2 agents

__device__ __forceinline__ int sweep_block(int b, int nb, int log_run) {
    const int round = nb >> (log_run + 3) << (log_run + 3);
    if (b < round) {
        const int k = b >> 3;
        return ((((k >> log_run) << 3) + (b & 7)) << log_run) + (k & ((1 << log_run) - 1));
    }
    const int per = (nb - round) >> 3, r = b - round;
    return r < per << 3 ? round + (r & 7) * per + (r >> 3) : b;
}

// 32-bit words of LDS of a sweep block before the policy's: the minima, then
// (lane groups) each wave's queue.
__host__ __device__ constexpr int sweep_words(int vs, int NT, int G, int kM, int meta) {
    const int minima = vs * (NT / G);
    return G == 1 ? minima : ((minima + 3) & ~3) + NT / 64 * queue_words(G, kM, meta);
}

template <int NT, int G, bool kFov, bool kTag, int kM, int kPol, int kMeta>
__global__ __launch_bounds__(NT) void k_sweep(SortArrays a, const DevEnv *__restrict__ envs,
                                              int n_envs, int Gtot, int v, int obs_dim,
                                              float *__restrict__ obs, float *__restrict__ reward,
                                              int add_ret, PolFuse pf) {
    static_assert(kPol == 0 || !kTag, "the fused policy serves flock envs");
    constexpr int A = NT / G;
    extern __shared__ uint32_t s_min[];  // [channels * v][A], the queues, the policy's (kPol)
    const int vs = kTag ? 2 * v : v;     // minima per agent
    __shared__ int s_env;
    __shared__ float *s_orow[G == 1 && kPol == 0 ? NT : 1];  // view rows (one lane per agent)
    const int tid = threadIdx.x, slot = tid / G, li = tid % G;
    constexpr int kLogRun = (G == 1 ? kSweepRunOne : kSweepRunGroup) - __builtin_ctz(A);
    const int p0 = sweep_block((int)blockIdx.x, (int)gridDim.x, kLogRun) * A;
    if constexpr (G == 1) block_env(&s_env, a.base, n_envs, p0);
    uint32_t *smin = s_min + slot;
    if constexpr (G > 1)
        for (int k = li; k < vs; k += G) smin[k * A] = kInfBits;
    static_assert(kPol == 0 || G <= 4, "the fused policy needs blocks of at least 64 agents");
    const SweepPolLds PL =
        sweep_pol_lds(sweep_words(vs, NT, G, kM, kMeta), A, NT, G, sweep_pol_alias(G, pf.kc, vs));
    PolConsts *s_pc = reinterpret_cast<PolConsts *>(s_min + PL.pc);
    float *s_speed = reinterpret_cast<float *>(s_min + PL.speed);
    int *s_pe = reinterpret_cast<int *>(s_min + PL.env);
    int *s_pid = reinterpret_cast<int *>(s_min + PL.id);
    if constexpr (kPol != 0) load_pol_consts(pf.P, s_pc, tid, NT);
    // the strip sort's words, zero again for the next step
    if (blockIdx.x == 0)
        for (int i = tid; i < a.n_status; i += NT) a.status[i] = 0u;
    if constexpr (G == 1 || kPol != 0) __syncthreads();
    const int pos = p0 + slot;
    if constexpr (G == 1 && kPol == 0) {
        if (pos >= Gtot) return;
    }
    // a group is active or not as a whole
    const bool active = pos < Gtot;
    int e = 0;
    if constexpr (G == 1) {
        e = s_env;
    } else if (n_envs > 1) {
        // lane groups: each wave finds the env of its first agent itself
        e = wave_env_search(a.base, n_envs, min(p0 + (tid >> 6) * (64 / G), Gtot - 1));
    }
    if (active && (G == 1 || n_envs > 1))
        while (a.base[e + 1] <= pos) ++e;
    const DevEnv &E = envs[e];
    const int j = pos - E.agent_base;
    float4 me = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    int nb = 0, col = 0, ti = 0, my_id = 0;
    double ret0 = 0.0;
    if (G > 1 && active) {
        // everything the agent needs from its env, loaded at once
        me = gload(E.rec_nxt, j);
        my_id = gload(E.id_nxt, j);
        if (add_ret) ret0 = gload(E.ret_nxt, j);
    }
    if constexpr (G > 1) {
        const int lane = tid & 63;
        const WaveQueue<kMeta> Q = wave_queue<G, kMeta>(
            s_min + ((vs * A + 3) & ~3) + (tid >> 6) * queue_words(G, kM, kMeta));
        const float2 cs = heading_cs(me.z);
        constexpr bool kQueued = queued(G, kM, kMeta);
        if (kQueued && li == 0) {
            Q.cs[lane / G] = cs;
            Q.col[lane / G] = 0;
        }
        const ViewK K{cs.x, cs.y, E.fov_half, E.fov_t, E.sec_scale, (float)v, v};
        if (kTag && active) ti = my_id < E.n_chasers ? 1 : 0;
        uint32_t *const smin_w = s_min + (tid >> 6) * (64 / G);
        const int e0 = __builtin_amdgcn_readfirstlane(e);
        if (G == 64 || !__any(active && e != e0)) {
            // one env, as in nearly every wave: its descriptor in scalar registers
            int eu = e0;
            asm("" : "+s"(eu));  // (else the compiler takes the lane's own equal e)
            const DevEnv &U = envs[eu];
            const ViewK KU{cs.x, cs.y, U.fov_half, U.fov_t, U.sec_scale, (float)v, v};
            sweep_group<A, G, kFov, kTag, kM, false>(a, U, smin_w, Q, active, me, pos, ti, KU, nb, col);
        } else if constexpr (G < 64) {
            sweep_group<A, G, kFov, kTag, kM, true>(a, E, smin_w, Q, active, me, pos, ti, K, nb, col);
        }
        if constexpr (kQueued) {
            col = Q.col[lane / G];
#pragma unroll  // (64 lanes: nb is the whole group's already)
            for (int m = (G < 64 || kTag) ? G / 2 : 0; m >= 1; m >>= 1) nb += __shfl_xor(nb, m, 64);
        } else {
            wave_lds_fence();  // the group's minima are complete
#pragma unroll
            for (int m = G / 2; m >= 1; m >>= 1) {
                nb += __shfl_xor(nb, m, 64);
                col += __shfl_xor(col, m, 64);
            }
        }
    } else if (active) {
        me = E.rec_nxt[j];
        const float2 cs = heading_cs(me.z);
        const float c = cs.x, s = cs.y;
        for (int k = 0; k < vs; ++k) smin[k * A] = kInfBits;

        const ViewK K{c, s, E.fov_half, E.fov_t, E.sec_scale, (float)v, v};
        ti = kTag ? (E.id_nxt[j] < E.n_chasers ? 1 : 0) : 0;
        const float L = E.box, r2 = E.r2, c2 = E.c2;
        const int ncx = E.ncx, ncy = E.ncy, cb = E.cell_base;
        // one run of candidates [q, q1): template flags say which shifts are nonzero
        auto run = [&](auto sx, auto sy, int q, int q1, float offx, float xi, float offy, float yi,
                       bool minimg) {
            sweep_run<A, kFov, kTag, kM, decltype(sx)::value, decltype(sy)::value>(
                smin, a.sxy, a.stype, ti, q, q1, pos, offx, xi, offy, yi, minimg, L, r2, c2, K, nb,
                col);
        };
        using No = std::false_type;
        using Yes = std::true_type;
        if (ncx == 1) {
            run(No{}, No{}, a.start[cb], a.start[cb + 1], 0.0f, me.x, 0.0f, me.y, true);
        } else {
            const int reach = E.reach;
            const int cx = cell_of(me.x, E.inv_cx, ncx);
            const float fx = me.x - (float)cx * E.cw;  // offset within the own column
            const RowGeom RG{E.cw, E.marg, r2, E.inv_cy, ncy};  // held in registers
            // the column's runs over rows [lo, hi]; a column left of column 0
            // wraps to the right edge with its candidates shifted by -L (sx),
            // one right of the last wraps to the left edge with the centre
            // shifted instead; rows wrap likewise
            auto column_at = [&](auto sx, int colb, float offx, float xi, int lo, int hi) {
                if (lo < 0) {
                    run(sx, Yes{}, a.start[colb + lo + ncy], a.start[colb + ncy], offx, xi, -L,
                        me.y, false);
                    run(sx, No{}, a.start[colb], a.start[colb + hi + 1], offx, xi, 0.0f, me.y, false);
                } else if (hi >= ncy) {
                    run(sx, No{}, a.start[colb + lo], a.start[colb + ncy], offx, xi, 0.0f, me.y,
                        false);
                    run(sx, No{}, a.start[colb], a.start[colb + hi - ncy + 1], offx, xi, 0.0f,
                        me.y - L, false);
                } else {
                    run(sx, No{}, a.start[colb + lo], a.start[colb + hi + 1], offx, xi, 0.0f, me.y,
                        false);
                }
            };
            if (kFlatRuns && reach == 1) {
                FlatRuns F;
                flat_runs(RG, a.start, cb, ncx, cx, fx, me.y, F);
                // the current run [q, q1) and its shifts; the rest queue in F
                int q = F.rq[0], q1 = F.rq1[0], left = F.nr;
                uint32_t fl = F.fl;
                float offx, xi, offy, yi;
                auto shifts = [&]() {
                    offx = (fl & 1u) ? -L : 0.0f;
                    xi = (fl & 2u) ? me.x - L : me.x;
                    offy = (fl & 4u) ? -L : 0.0f;
                    yi = (fl & 8u) ? me.y - L : me.y;
                };
                shifts();
                // kFlatUnroll candidates per step, those past the run's end
                // masked (the position arrays are padded for the reads); each
                // step loads the next one's before its tests: the rest of this
                // run, else the next queued run's start (a stale but in-range
                // start once none is left)
                float2 pj[kFlatUnroll];
#pragma unroll
                for (int u = 0; u < kFlatUnroll; ++u) pj[u] = a.sxy[q + u];
                while (true) {
                    const int qn = q + kFlatUnroll < q1 ? q + kFlatUnroll : F.rq[1];
                    float2 pn[kFlatUnroll];
#pragma unroll
                    for (int u = 0; u < kFlatUnroll; ++u) pn[u] = a.sxy[qn + u];
                    const int rem = q1 - q, so = pos - q;  // slots in the run; the agent's own
                    // most runs have no candidate-side shift: a step in which no
                    // lane of the wave has one leaves out the two additions
                    if (__any((fl & 5u) != 0u)) {
#pragma unroll
                        for (int u = 0; u < kFlatUnroll; ++u)
                            test_pair<A, kFov, kTag, kM, true, true>(
                                smin, a.stype, ti, pj[u], q + u, u < rem && u != so, offx, xi,
                                offy, yi, false, L, r2, c2, K, nb, col);
                    } else {
#pragma unroll
                        for (int u = 0; u < kFlatUnroll; ++u)
                            test_pair<A, kFov, kTag, kM, false, false>(
                                smin, a.stype, ti, pj[u], q + u, u < rem && u != so, offx, xi,
                                offy, yi, false, L, r2, c2, K, nb, col);
                    }
                    q += kFlatUnroll;
                    if (q >= q1) {
                        // next slot (an empty one costs a step of masked tests)
                        if (--left <= 0) break;
#pragma unroll
                        for (int k = 0; k < 5; ++k) {
                            F.rq[k] = F.rq[k + 1];
                            F.rq1[k] = F.rq1[k + 1];
                        }
                        fl >>= 4;
                        q = F.rq[0];
                        q1 = F.rq1[0];
                        shifts();
                    }
#pragma unroll
                    for (int u = 0; u < kFlatUnroll; ++u) pj[u] = pn[u];
                }
            } else {
                for (int ox = -reach; ox <= reach; ++ox) {
                    int lo, hi;
                    if (!column_rows(RG, fx, ox, me.y, lo, hi)) continue;
                    const int ccx = cx + ox;
                    if (ccx < 0) column_at(Yes{}, cb + (ccx + ncx) * ncy, -L, me.x, lo, hi);
                    else if (ccx >= ncx) column_at(No{}, cb + (ccx - ncx) * ncy, 0.0f, me.x - L, lo, hi);
                    else column_at(No{}, cb + ccx * ncy, 0.0f, me.x, lo, hi);
                }
            }
        }
    }  // active

    if constexpr (G > 1) {
        if (kPol == 0 && !active) return;
    }
    constexpr bool kGl = G > 1;
    // A view value from a sector minimum; with kPol it also replaces the minimum in LDS.
    auto view = [&](int k, float inv_r) {
        const uint32_t m = smin[k * A];
        const float o = m == kInfBits ? 0.0f : 1.0f - __builtin_amdgcn_sqrtf(__uint_as_float(m)) * inv_r;
        if constexpr (kPol != 0) smin[k * A] = __float_as_uint(o);
        return o;
    };
    // One lane per agent: rows of 4, 8, 16, 32 or 64 views (no speed column)
    // leave the wave whole, vs / 4 lanes to a row, so that each store instruction writes
    // 64 / (vs / 4) whole rows rather than 16 bytes of each of 64 rows.
    const bool rows_whole =
        G == 1 && kPol == 0 && obs_dim == vs && vs >= 4 && vs <= 64 && (vs & (vs - 1)) == 0;
    if (active) {
        // agent-order rows are addressed by id: an id out of range (a sort
        // that went wrong) writes agent 0's rows instead of outside them
        const int id0 = G > 1 ? my_id : E.id_nxt[j];
        const int id = (unsigned)id0 < (unsigned)E.n ? id0 : 0;
        my_id = id;
        const float inv_r = E.inv_radius;
        float *orow = obs ? obs + ((size_t)E.agent_base + id) * obs_dim : E.obs + (size_t)id * obs_dim;
        if (li == 0 && obs_dim > vs) store_as<kGl>(orow, vs, me.w);  // speed after the move (Sec. 4.1)
        if constexpr (G > 1) {
            for (int k = li; k < vs; k += G) store_as<kGl>(orow, k, view(k, inv_r));
        } else if (rows_whole) {
            // the views in place of the minima, the row's address beside them
            for (int k = 0; k < vs; ++k) smin[k * A] = __float_as_uint(view(k, inv_r));
            if constexpr (kPol == 0) s_orow[slot] = orow;
        } else if ((obs_dim & 3) == 0 && (vs & 3) == 0) {
            for (int k = 0; k < vs; k += 4) {
                float o[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) o[u] = view(k + u, inv_r);
                *reinterpret_cast<float4 *>(orow + k) = make_float4(o[0], o[1], o[2], o[3]);
            }
        } else {
            for (int k = 0; k < vs; ++k) orow[k] = view(k, inv_r);
        }
        if (li == 0) {
            const float r =
                (kTag && ti) ? E.r_catch * (float)col : E.r_nb * (float)nb + E.r_col * (float)col;
            if (reward) reward[E.agent_base + id] = r;
            else if (E.rew) store_as<kGl>(E.rew, id, r);
            if (add_ret) store_as<kGl>(E.ret_nxt, j, (G > 1 ? ret0 : E.ret_nxt[j]) + (double)r);
            if (E.nb) {
                store_as<kGl>(E.nb, id, nb);
                store_as<kGl>(E.col, id, col);
            }
            if constexpr (kPol != 0 && G > 1) {
                s_speed[slot] = me.w;
                s_pe[slot] = e;
                s_pid[slot] = id;
            }
        }
    } else if constexpr (kPol != 0 && G > 1) {
        if (li == 0) s_pe[slot] = -1;
    }
    if constexpr (G == 1 && kPol == 0) {
        if (rows_whole) {
            // The lanes left here are the wave's active ones, a prefix of it
            // (in the last wave of a launch the others have returned): they
            // share out the n_act rows' vs / 4 pieces, piece t = row t / lpr,
            // columns 4 (t % lpr) on.
            wave_lds_fence();
            const int lane = tid & 63, w0 = tid - lane;
            const int n_act = __popcll(__ballot(1));
            const int lpr = vs >> 2, lg = __builtin_ctz(lpr);
            for (int t = lane; t < n_act * lpr; t += n_act) {
                const int r = t >> lg, c4 = 4 * (t & (lpr - 1));
                const uint32_t *col4 = s_min + c4 * A + w0 + r;
                *reinterpret_cast<float4 *>(s_orow[w0 + r] + c4) =
                    make_float4(__uint_as_float(col4[0]), __uint_as_float(col4[A]),
                                __uint_as_float(col4[2 * A]), __uint_as_float(col4[3 * A]));
            }
        }
    }
    // The policy's action of a tile's agent from its output pre-activations
    // (lanes g == 0 of a valid column write).
    auto write_act = [&](float2 z, int pe, int idj, bool wr) {
        if (!wr) return;
        const DevEnv &Ej = envs[pe];
        const int64_t row = (int64_t)Ej.agent_base + idj;
        const float2 ev = kPol == 2 ? pf.eps[row] : make_float2(0.0f, 0.0f);
        const float2 av = pol_output<kPol == 2>(z, pf.max_turn, pf.max_dspeed, ev, pf.sig0, pf.sig1,
                                                pf.logp_c,
                                                (kPol == 2 && pf.logp) ? pf.logp + row : nullptr);
        if (pf.act) pf.act[row] = av;
        else reinterpret_cast<float2 *>(Ej.act)[idj] = av;
    };
    // weight fragments read at use from global memory (cached): held in
    // registers they would lower the whole kernel's occupancy, staged in LDS
    // they made the policy phase LDS-bound (measured slower)
    const int lane = tid & 63, g = lane >> 4, colx = lane & 15;
    auto w1a = [&](int c, int t) { return pf.P.w1[(c * 4 + t) * 64 + lane]; };
    auto w2a = [&](int c, int t) { return pf.P.w2[(c * 4 + t) * 64 + lane]; };
    auto w3a = [&](int c) { return pf.P.w3[c * 64 + lane]; };
    if constexpr (kPol != 0 && G == 1) {
        const int w0 = tid - lane;  // the wave's first slot
        const int my_e = active ? e : -1;
        const float my_sp = me.w;
        wave_lds_fence();           // the wave's views in LDS before its reads
        // inputs of tile t (agents w0 + 16 t + col, owned by lane 16 t + col):
        // the view, then the speed when the row carries it, zero beyond
        auto input = [&](int t, int k, int pe, float sp) {
            float o = 0.0f;
            if (pe >= 0) {
                if (k < vs) o = __uint_as_float(s_min[k * A + w0 + 16 * t + colx]);
                else if (k == vs && obs_dim > vs) o = sp;
            }
            return (__bf16)o;
        };
        if (sweep_pol_alias(G, pf.kc, vs)) {
            bf16x8 xr[4];
            int te[4], ti4[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int src = 16 * t + colx;
                te[t] = __shfl(my_e, src, 64);
                ti4[t] = __shfl(my_id, src, 64);
                const float sp = __shfl(my_sp, src, 64);
#pragma unroll
                for (int jj = 0; jj < 8; ++jj) xr[t][jj] = input(t, 8 * g + jj, te[t], sp);
            }
            wave_lds_fence();  // every lane's reads before the stretch becomes the hidden tile
            // row r: minima row r of the wave's stretch, skewed by (r % 8) * 4 words
            auto hrow = [&](int r) {
                return reinterpret_cast<__bf16 *>(s_min + r * A + w0 + (r & 7) * 4);
            };
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float2 z =
                    mlp_tile(1, [&](int) { return xr[t]; }, w1a, w2a, w3a, *s_pc, hrow, lane);
                write_act(z, te[t], ti4[t], g == 0 && te[t] >= 0);
            }
        } else {
            __bf16 *s_hid = reinterpret_cast<__bf16 *>(s_min + PL.hid) + (size_t)(tid >> 6) * 16 * kHidLd;
            auto hrow = [&](int r) { return s_hid + r * kHidLd; };
            for (int t = 0; t < 4; ++t) {
                const int src = 16 * t + colx;
                const int pe = __shfl(my_e, src, 64), idj = __shfl(my_id, src, 64);
                const float sp = __shfl(my_sp, src, 64);
                auto xb = [&](int c) {
                    bf16x8 x;
#pragma unroll
                    for (int jj = 0; jj < 8; ++jj) x[jj] = input(t, 32 * c + 8 * g + jj, pe, sp);
                    return x;
                };
                const float2 z = mlp_tile(pf.kc, xb, w1a, w2a, w3a, *s_pc, hrow, lane);
                write_act(z, pe, idj, g == 0 && pe >= 0);
            }
        }
        return;
    }
    if constexpr (kPol != 0) {
        __syncthreads();  // every agent's view, speed and row are in LDS
        constexpr int kTiles = (A + 15) / 16;
        const int wid = tid >> 6;
        __bf16 *s_hid = reinterpret_cast<__bf16 *>(s_min + PL.hid) + (size_t)wid * 16 * kHidLd;
        auto hrow = [&](int r) { return s_hid + r * kHidLd; };
        if (wid >= kTiles) return;
        for (int tile = wid; tile < kTiles; tile += NT / 64) {
            const int sl = tile * 16 + colx;
            const int pe = sl < A ? s_pe[sl] : -1;
            const bool valid = pe >= 0;
            // inputs 32 c + 8 g .. + 7 of agent sl: the view, then the speed when
            // the row carries it, zero beyond
            auto xb = [&](int c) {
                bf16x8 x;
#pragma unroll
                for (int jj = 0; jj < 8; ++jj) {
                    const int k = 32 * c + 8 * g + jj;
                    float o = 0.0f;
                    if (valid) {
                        if (k < vs) o = __uint_as_float(s_min[k * A + sl]);
                        else if (k == vs && obs_dim > vs) o = s_speed[sl];
                    }
                    x[jj] = (__bf16)o;
                }
                return x;
            };
            const float2 z = mlp_tile(pf.kc, xb, w1a, w2a, w3a, *s_pc, hrow, lane);
            write_act(z, pe, valid ? s_pid[sl] : 0, g == 0 && valid);
        }
    }
}

// ------------------------------------------------------------------ helpers

__global__ void k_clear(int32_t *count, int64_t C) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < C) count[i] = 0;
}

__global__ void k_load_state(const float *x, const float *y, const float *th, const float *sp,
                             float4 *rec, int32_t *id, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    rec[i] = make_float4(x[i], y[i], th[i], sp[i]);
    id[i] = i;
}

__global__ void k_store_state(const float4 *rec, const int32_t *id, float *x, float *y, float *th,
                              float *sp, int n) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const float4 r = rec[p];
    const int i = id[p];
    x[i] = r.x;
    y[i] = r.y;
    th[i] = r.z;
    sp[i] = r.w;
}

__global__ void k_store_returns(const double *ret, const int32_t *id, double *out, int n) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p < n) out[id[p]] = ret[p];
}

__global__ void k_load_returns(const double *in, const int32_t *id, double *ret, int n) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p < n) ret[p] = in[id[p]];
}

__global__ void k_zero_f64(double *p, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0.0;
}

__global__ void k_copy_i32(const int32_t *src, int32_t *dst, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

inline unsigned blocks_for(int64_t n, int nt) { return (unsigned)((n + nt - 1) / nt); }

}  // namespace

int env_sort_recs_for(int n_envs, int64_t max_env_agents, int64_t max_env_cells) {
    if (n_envs < 64 || max_env_cells > 16384) return 0;
    // (envs up to 16,384 agents: a 20,000-agent env in a batch of smaller
    // ones keeps its block busy long after the rest are done)
    for (int r = 2; r <= 16; r *= 2)
        if (max_env_agents <= (int64_t)r * kEnvNT) return r;
    return 0;
}

int scan_blocks_for(int64_t C, int64_t max_env_cells) {
    return max_env_cells <= kScanTile ? 0 : (int)((C + kTile2 - 1) / kTile2);
}

void carve_sort(Carver &cv, int64_t G, int64_t C, int E, SortArrays *a, int64_t S) {
    const int64_t nb = (C + kTile2 - 1) / kTile2;  // partials of the two-level scan
    a->key = cv.take<int32_t>(G);
    a->slot = cv.take<int32_t>(G);
    a->tmp = cv.take<float4>(G);
    a->sxy = cv.take<float2>(G + kSortPad);
    a->stype = cv.take<uint8_t>(G + kSortPad);
    a->count = cv.take<int32_t>(C);
    a->start = cv.take<int32_t>(C + 1);
    a->part = cv.take<int32_t>(nb + 1);
    a->envs[0] = cv.take<DevEnv>(E);
    a->envs[1] = cv.take<DevEnv>(E);
    a->base = cv.take<int32_t>(E + 1);
    a->strip_env = S > 0 ? cv.take<int32_t>(S) : nullptr;
    a->status = S > 0 ? cv.take<uint32_t>(S) : nullptr;
    a->n_status = S > 0 ? (int32_t)S : 0;
}

bool strips_allowed(const DevEnv &d) {
    // at most one column per step (half a column leaves room for the rounding
    // of the column boundaries), and one column's cells fit the block
    return d.ncy <= kStripCells && d.s_max <= 0.5f * d.cw;
}

int strip_cols_for(const DevEnv &d, int64_t G) {
    // about G / 512 agents per strip (at least 512, at most 4,096), so a
    // large batch gives hundreds of blocks and a small one still several
    const double target = std::min(4096.0, std::max(512.0, (double)G / 512.0));
    const double per_col = (double)std::max(d.n, 1) / d.ncx;
    int cols = (int)std::lround(target / per_col);
    cols = std::max(1, std::min(cols, kStripCells / d.ncy));
    return std::min(cols, d.ncx);
}

// CUs of the current device (asked for once per device).
static int device_cus() {
    static std::atomic<int> known[64];
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    cus = known[dev].load(std::memory_order_relaxed);
    if (cus > 0) return cus;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
        return 256;
    known[dev].store(cus, std::memory_order_relaxed);
    return cus;
}

void plan_strip_device(StepPlan *p) {
    const int cus = device_cus();
    p->strips_wide = strips_wide(p->strips, cus);
    p->strips_ahead = strips_ahead(p->strips, p->n_envs, p->strips_per_cu * cus);
    p->strip_run_log = strip_run_log(p->strips, p->strips_most, cus);
}

std::vector<int32_t> strip_launch_order(StepPlan *p, const std::vector<int32_t> &strips_of) {
    plan_strip_device(p);
    const int first = p->strips_ahead ? 1 : 0;
    std::vector<int32_t> env;
    for (int e = 0; e < p->strips_ahead; ++e) env.push_back(e);
    for (int e = 0; e < p->n_envs; ++e) env.insert(env.end(), strips_of[e] - first, e);
    return env;
}

void plan_strip_launch(StepPlan *p, const DevEnv *envs, int n_envs) {
    int cells = 1, most = 1;
    for (int e = 0; e < n_envs; ++e) {
        cells = std::max(cells, envs[e].strip_cols * envs[e].ncy);
        most = std::max(most, envs[e].n_strips);
    }
    p->strip_cells = cells;
    p->strips_most = most;
    // Strips whose neighbouring columns alone exceed the registers list their
    // agents beyond them (uniform agents' and four deviations), in the LDS that
    // leaves a CU four, three or two blocks.  Where less is read again, reading it
    // again is as fast (256 uneven envs, half the own agents' number: steps 2 %
    // slower with a list).
    p->strip_cap = 0;
    double list = 0.0;
    for (int e = 0; e < n_envs; ++e) {
        const DevEnv &d = envs[e];
        const double per_col = (double)d.n / d.ncx, own = per_col * d.strip_cols;
        if (2.0 * per_col <= kStripRegs) continue;
        const double in = 0.64 * d.s_max / d.cw * per_col;  // come in over either border
        list = std::max(list, std::max(own - kStripRegs, 0.0) + in + 4.0 * std::sqrt(own));
    }
    p->strips_per_cu = 4;
    for (int k = 4; k >= 2 && list > 0.0 && p->strip_cap == 0; --k) {
        const int cap = (kStripLds / k / (int)sizeof(int) - ((cells + 3) & ~3)) / 4;
        if (list <= cap) {
            p->strip_cap = cap;
            p->strips_per_cu = k;
        }
    }
}

int64_t assign_strips(DevEnv *const *tabs, int n_tabs, int n_envs, int64_t G,
                      std::vector<int32_t> *strips_of) {
    int64_t S = 0;
    if (strips_of) strips_of->clear();
    for (int e = 0; e < n_envs; ++e) {
        const int cols = strip_cols_for(tabs[0][e], G);
        const int ns = (tabs[0][e].ncx + cols - 1) / cols;
        for (int k = 0; k < n_tabs; ++k) {
            tabs[k][e].strip_base = (int32_t)S;
            tabs[k][e].strip_cols = cols;
            tabs[k][e].n_strips = ns;
        }
        if (strips_of) strips_of->push_back(ns);
        S += ns;
    }
    return S;
}

// Descriptor tables and agent offsets of a one-env plan, written from the
// kernel's by-value arguments (no copy from host memory), and the plan's cell
// counts zeroed: what a step needs in its sort scratch before it starts.
__global__ void k_bind_one(SortArrays a, DevEnv d0, DevEnv d1, int32_t n, int64_t C) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < C) a.count[i] = 0;
    if (i < a.n_status) a.status[i] = 0u;
    if (i == 0) {
        a.envs[0][0] = d0;
        a.envs[1][0] = d1;
        a.base[0] = 0;
        a.base[1] = n;
    }
}

hipError_t launch_bind_one(const StepPlan &p, const DevEnv &d0, const DevEnv &d1, int32_t n,
                           hipStream_t s) {
    const int64_t c = std::max<int64_t>(std::max<int64_t>(p.C, p.a.n_status), 1);
    hipLaunchKernelGGL(k_bind_one, dim3(blocks_for(c, 256)), dim3(256), 0, s, p.a, d0, d1, n, p.C);
    return hipGetLastError();
}

bool plan_fuses_policy(const StepPlan &p) { return !p.tag && (p.lanes == 1 || p.lanes == 4); }

hipError_t launch_clear(const StepPlan &p, hipStream_t s) {
    const int64_t n = p.C > 0 ? p.C : 1;
    hipLaunchKernelGGL(k_clear, dim3(blocks_for(n, 256)), dim3(256), 0, s, p.a.count, p.C);
    if (p.a.n_status > 0)
        hipLaunchKernelGGL(k_clear, dim3(blocks_for(p.a.n_status, 256)), dim3(256), 0, s,
                           reinterpret_cast<int32_t *>(p.a.status), (int64_t)p.a.n_status);
    return hipGetLastError();
}

namespace {
template <int NT, int G, bool kFov, bool kTag, int kM = 0, int kPol = 0, int kMeta = 4>
void launch_sweep_v(const StepPlan &p, const DevEnv *envs, int Gtot, float *obs, float *reward,
                    int add_return, hipStream_t s, const PolFuse *pf) {
    constexpr int A = NT / G;
    const int vs = (kTag ? 2 : 1) * p.v, min_words = sweep_words(vs, NT, G, kM, kMeta);
    if constexpr (G == 4 && kM == 0 && kPol == 0 && kMeta == 4) {
        // blocks in a CU's 160 KiB (1,280 bytes at a time, 64 of them static) and registers
        auto blocks = [](int words) {
            return std::min(8, 163840 / ((4 * words + 64 + 1279) / 1280 * 1280));
        };
        auto go = [&](auto launch) { launch(p, envs, Gtot, obs, reward, add_return, s, pf); };
        if (p.max_env_cells == 1) return go(launch_sweep_v<NT, G, kFov, kTag, kM, kPol, 0>);
        if (blocks(sweep_words(vs, NT, G, kM, 1)) > blocks(min_words))
            return go(launch_sweep_v<NT, G, kFov, kTag, kM, kPol, 1>);
    }
    const size_t lds =
        (size_t)(kPol ? sweep_pol_lds(min_words, A, NT, G, sweep_pol_alias(G, pf->kc, vs)).words
                      : min_words) *
        sizeof(uint32_t);
    hipLaunchKernelGGL((k_sweep<NT, G, kFov, kTag, kM, kPol, kMeta>), dim3(blocks_for(Gtot, A)), dim3(NT),
                       lds, s, p.a, envs, p.n_envs, Gtot, p.v, p.obs_dim, obs, reward, add_return,
                       pf ? *pf : PolFuse{});
}

// Flock plans: the view variant (limited view, or 8 / 16 / 32 sectors without
// the arctangent) and, with pf, the fused policy's output mode.
template <int NT, int G, int kPol>
void launch_sweep_flock(const StepPlan &p, const DevEnv *envs, int Gtot, float *obs, float *reward,
                        int add_return, hipStream_t s, const PolFuse *pf) {
    if (p.fov) launch_sweep_v<NT, G, true, false, 0, kPol>(p, envs, Gtot, obs, reward, add_return, s, pf);
    else if (p.v == 8) launch_sweep_v<NT, G, false, false, 1, kPol>(p, envs, Gtot, obs, reward, add_return, s, pf);
    else if (p.v == 16) launch_sweep_v<NT, G, false, false, 2, kPol>(p, envs, Gtot, obs, reward, add_return, s, pf);
    else if (p.v == 32) launch_sweep_v<NT, G, false, false, 4, kPol>(p, envs, Gtot, obs, reward, add_return, s, pf);
    else launch_sweep_v<NT, G, false, false, 0, kPol>(p, envs, Gtot, obs, reward, add_return, s, pf);
}

template <int NT, int G>
void launch_sweep(const StepPlan &p, const DevEnv *envs, int Gtot, float *obs, float *reward,
                  int add_return, hipStream_t s, const PolFuse *pf) {
    if (p.tag) {
        if (p.fov) launch_sweep_v<NT, G, true, true>(p, envs, Gtot, obs, reward, add_return, s, nullptr);
        else launch_sweep_v<NT, G, false, true>(p, envs, Gtot, obs, reward, add_return, s, nullptr);
    } else if (!pf) {
        launch_sweep_flock<NT, G, 0>(p, envs, Gtot, obs, reward, add_return, s, nullptr);
    } else if constexpr (G <= 4) {
        if (pf->mode == 2) launch_sweep_flock<NT, G, 2>(p, envs, Gtot, obs, reward, add_return, s, pf);
        else launch_sweep_flock<NT, G, 1>(p, envs, Gtot, obs, reward, add_return, s, pf);
    }
}
}  // namespace

hipError_t launch_phase(const StepPlan &p, int table, StepPhase phase, int do_move,
                        const float *act, float *obs, float *reward, int add_return,
                        hipStream_t s, const PolFuse *pf, float *act_copy) {
    if (pf && !plan_fuses_policy(p)) return hipErrorInvalidValue;
    if (p.G == 0) return hipSuccess;
    const int G = (int)p.G, C = (int)p.C;
    const DevEnv *envs = p.a.envs[table & 1];
    const unsigned nb = blocks_for(G, kBlock);
    switch (phase) {
        case kPhaseMove:
            if (p.env_sort_recs == 0 && p.strips > 0 && p.strip_now) {
                auto go = [&](auto kernel, int nt, int cap) {
                    const size_t lds = (((p.strip_cells + 3) & ~3) + 4 * (size_t)cap) * sizeof(int);
                    hipLaunchKernelGGL(kernel, dim3(strip_blocks(p.strips, p.strips_ahead, p.strip_run_log)), dim3(nt),
                                       lds, s, p.a, envs, p.n_envs, C, G, (int)p.strips, do_move,
                                       reinterpret_cast<const float2 *>(act), p.tag,
                                       reinterpret_cast<float2 *>(act_copy),
                                       p.strips_ahead, (int)strip_run(p.strips, p.strips_ahead), p.strip_run_log,
                                       p.strip_wait, cap);
                };
                // one block per CU: latency; more: see the kernel
                const bool ordered = p.strips_ahead > 0 || p.strip_run_log >= 0;
                const int cap = p.strip_cap;
                if (p.strips_wide && !ordered) go(k_strip_sort<1024, 4, 4, false, false>, 1024, 0);
                else if (ordered && cap) go(k_strip_sort<512, 3, 8, true, true>, 512, cap);
                else if (ordered) go(k_strip_sort<512, 3, 8, true, false>, 512, 0);
                else if (cap) go(k_strip_sort<512, 3, 8, false, true>, 512, cap);
                else go(k_strip_sort<512, 3, 8, false, false>, 512, 0);
                break;
            }
            if (p.env_sort_recs > 0) {
                const size_t lds = (size_t)p.max_env_cells * sizeof(int);
                const float2 *a2 = reinterpret_cast<const float2 *>(act);
                float2 *ac2 = reinterpret_cast<float2 *>(act_copy);
                const dim3 grid(p.n_envs), block(kEnvNT);
                switch (p.env_sort_recs) {
                    case 2: hipLaunchKernelGGL(k_env_sort<2>, grid, block, lds, s, p.a, envs, p.n_envs, C, do_move, a2, p.tag, ac2); break;
                    case 4: hipLaunchKernelGGL(k_env_sort<4>, grid, block, lds, s, p.a, envs, p.n_envs, C, do_move, a2, p.tag, ac2); break;
                    case 8: hipLaunchKernelGGL(k_env_sort<8>, grid, block, lds, s, p.a, envs, p.n_envs, C, do_move, a2, p.tag, ac2); break;
                    default: hipLaunchKernelGGL(k_env_sort<16>, grid, block, lds, s, p.a, envs, p.n_envs, C, do_move, a2, p.tag, ac2); break;
                }
                break;
            }
            hipLaunchKernelGGL(k_move_count, dim3(blocks_for(G, kBlock * kMoveRecs)), dim3(kBlock),
                               0, s, p.a, envs, p.n_envs, G, do_move,
                               reinterpret_cast<const float2 *>(act),
                               reinterpret_cast<float2 *>(act_copy));
            break;
        case kPhaseScan:
            if (p.env_sort_recs > 0 || (p.strips > 0 && p.strip_now)) break;  // one-kernel sorts
            if (p.scan_blocks == 0) {
                if (p.max_env_cells <= 2048)
                    hipLaunchKernelGGL((k_scan_env<256, 8>), dim3(p.n_envs), dim3(256), 0, s,
                                       p.a.count, p.a.start, envs, p.n_envs, C);
                else
                    hipLaunchKernelGGL((k_scan_env<kScanNT, kScanItems>), dim3(p.n_envs),
                                       dim3(kScanNT), 0, s, p.a.count, p.a.start, envs, p.n_envs, C);
            } else {
                hipLaunchKernelGGL(k_tile_sums, dim3(p.scan_blocks), dim3(kScan2NT), 0, s,
                                   p.a.count, p.a.part, C);
                if (p.scan_blocks <= kDirectTiles) {
                    hipLaunchKernelGGL(k_scan_down<true>, dim3(p.scan_blocks), dim3(kScan2NT), 0,
                                       s, p.a.count, p.a.part, p.a.start, C);
                } else {
                    hipLaunchKernelGGL(k_scan_parts, dim3(1), dim3(kScan2NT), 0, s, p.a.part,
                                       p.scan_blocks);
                    hipLaunchKernelGGL(k_scan_down<false>, dim3(p.scan_blocks), dim3(kScan2NT), 0,
                                       s, p.a.count, p.a.part, p.a.start, C);
                }
            }
            break;
        case kPhaseScatter:
            if (p.env_sort_recs > 0 || (p.strips > 0 && p.strip_now)) break;  // one-kernel sorts
            hipLaunchKernelGGL(k_scatter, dim3(nb), dim3(kBlock), 0, s, p.a, envs, p.n_envs, G,
                               p.tag);
            break;
        case kPhaseSweep: {
            const int lanes = p.lanes;
            if (lanes == 4) launch_sweep<256, 4>(p, envs, G, obs, reward, add_return, s, pf);
            else if (lanes == 16) launch_sweep<256, 16>(p, envs, G, obs, reward, add_return, s, pf);
            else if (lanes == 64) launch_sweep<256, 64>(p, envs, G, obs, reward, add_return, s, pf);
            else if ((p.tag ? 2 * p.v : p.v) <= 32)
                launch_sweep<256, 1>(p, envs, G, obs, reward, add_return, s, pf);
            else launch_sweep<64, 1>(p, envs, G, obs, reward, add_return, s, pf);
            break;
        }
    }
    return hipGetLastError();
}

hipError_t launch_step(const StepPlan &p, int table, int do_move, const float *act, float *obs,
                       float *reward, int add_return, hipStream_t s, hipEvent_t *ev,
                       const PolFuse *pf, float *act_copy) {
    if (p.G == 0) return hipSuccess;
    const StepPhase order[4] = {kPhaseMove, kPhaseScan, kPhaseScatter, kPhaseSweep};
    hipError_t e = hipSuccess;
    for (int k = 0; k < 4 && e == hipSuccess; ++k) {
        if (ev) (void)hipEventRecord(ev[k], s);
        e = launch_phase(p, table, order[k], do_move, act, obs, reward, add_return, s, pf,
                         act_copy);
    }
    if (ev) (void)hipEventRecord(ev[4], s);
    return e;
}

hipError_t launch_load_state(const float *x, const float *y, const float *th, const float *sp,
                             float4 *rec, int32_t *id, int n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_load_state, dim3(blocks_for(n, 256)), dim3(256), 0, s, x, y, th, sp, rec,
                       id, n);
    return hipGetLastError();
}

hipError_t launch_store_state(const float4 *rec, const int32_t *id, float *x, float *y, float *th,
                              float *sp, int n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_store_state, dim3(blocks_for(n, 256)), dim3(256), 0, s, rec, id, x, y, th,
                       sp, n);
    return hipGetLastError();
}

hipError_t launch_store_returns(const double *ret, const int32_t *id, double *out, int n,
                                hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_store_returns, dim3(blocks_for(n, 256)), dim3(256), 0, s, ret, id, out, n);
    return hipGetLastError();
}

hipError_t launch_load_returns(const double *in, const int32_t *id, double *ret, int n,
                               hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_load_returns, dim3(blocks_for(n, 256)), dim3(256), 0, s, in, id, ret, n);
    return hipGetLastError();
}

hipError_t launch_zero_f64(double *p, int64_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_zero_f64, dim3(blocks_for(n, 256)), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_copy_i32(const int32_t *src, int32_t *dst, int64_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_copy_i32, dim3(blocks_for(n, 256)), dim3(256), 0, s, src, dst, n);
    return hipGetLastError();
}

}  // namespace flock
