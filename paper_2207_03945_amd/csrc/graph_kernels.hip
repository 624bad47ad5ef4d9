// graph_kernels.hip -- the graph interaction: opinion dynamics over CSR edges.
//
// Sec. 2.1 of arXiv:2207.03945 gives interactions over the edges of a graph
// as the engine's second base pattern, with an opinion model as example:
// for each edge (me, you) of weight w_e, when |op_me - op_you| < threshold,
// me's new opinion moves toward you's current opinion,
//     new <- (1 - s w_e) new + s w_e op_you        (s = strength),
// starting from new = op_me; a self interaction then commits the new
// opinions.  A step reads op_in and writes op_out (the caller ping-pongs).
//
// Each node applies its incoming edges in CSR order, so its new opinion is
// the composition of per-edge affine maps x -> (1 - w) x + w y.  G lanes share
// a node: lane l applies the edges of the l-th contiguous chunk of the row to
// an affine map (a, b), the G maps are composed in chunk order by a shuffle
// butterfly, and lane 0 applies the result to op_me.  With G = 1 the lane
// runs the recurrence itself, in exactly the order the model states.
// Arithmetic: the threshold test in FP32 on the FP32 opinions, the updates
// in FP64, one rounding to FP32 at the end.
//
// Memory safety: row ranges are clamped to [0, n_edges] and edges whose
// `you` lies outside [0, n) are skipped, whatever the arrays hold.
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "flock_internal.h"

namespace flock {

namespace {

constexpr int kGraphBlock = 256;
// Edges a lane loads at once: their targets, weights and then the targets'
// opinions are each one round of loads in flight, instead of two dependent
// loads per edge (rows of power-law graphs reach thousands of edges, and a
// lane's chain of loads over its chunk sets the step's critical path).
// MI355X, 1M nodes, mean degree 14, 16 lanes: 0.208 ms per step one edge at
// a time, 0.139 with 4, 0.148 with 8, 0.217 with 16 (short chunks then load
// mostly padding).
constexpr int kEdgeBatch = 4;

// Loads of edges e .. e + kEdgeBatch - 1 of [e, c1) (e < c1): slots past c1
// read edge c1 - 1 and targets outside [0, n) read node 0; ok[u] says which
// slots hold an edge to apply.
__device__ __forceinline__ void load_edges(int64_t e, int64_t c1, int64_t n,
                                           const int32_t *__restrict__ col,
                                           const float *__restrict__ weight,
                                           const float *__restrict__ op_in, bool (&ok)[kEdgeBatch],
                                           float (&wt)[kEdgeBatch], float (&you)[kEdgeBatch]) {
    int32_t j[kEdgeBatch];
#pragma unroll
    for (int u = 0; u < kEdgeBatch; ++u) {
        const int64_t k = e + u < c1 ? e + u : c1 - 1;
        j[u] = col[k];
        wt[u] = weight[k];
        ok[u] = e + u < c1 && j[u] >= 0 && (int64_t)j[u] < n;
    }
#pragma unroll
    for (int u = 0; u < kEdgeBatch; ++u) you[u] = op_in[ok[u] ? j[u] : 0];
}

template <int G>
__global__ __launch_bounds__(kGraphBlock) void k_opinion(int64_t n, int64_t n_edges,
                                                         const int64_t *__restrict__ row_ptr,
                                                         const int32_t *__restrict__ col,
                                                         const float *__restrict__ weight,
                                                         float thr, double strength,
                                                         const float *__restrict__ op_in,
                                                         float *__restrict__ op_out) {
    constexpr int A = kGraphBlock / G;  // nodes per block
    const int tid = threadIdx.x, slot = tid / G, li = tid % G;
    const int64_t i = (int64_t)blockIdx.x * A + slot;
    const bool active = i < n;
    float me = 0.0f;
    int64_t e0 = 0, e1 = 0;
    if (active) {
        me = op_in[i];
        e0 = row_ptr[i];
        e1 = row_ptr[i + 1];
        e0 = e0 < 0 ? 0 : (e0 > n_edges ? n_edges : e0);
        e1 = e1 < e0 ? e0 : (e1 > n_edges ? n_edges : e1);
    }
    if constexpr (G == 1) {
        if (!active) return;
        double x = (double)me;
        for (int64_t e = e0; e < e1; e += kEdgeBatch) {
            bool ok[kEdgeBatch];
            float wt[kEdgeBatch], you[kEdgeBatch];
            load_edges(e, e1, n, col, weight, op_in, ok, wt, you);
#pragma unroll
            for (int u = 0; u < kEdgeBatch; ++u) {  // in edge order
                if (ok[u] && fabsf(me - you[u]) < thr) {
                    const double w = strength * (double)wt[u];
                    x = (1.0 - w) * x + w * (double)you[u];
                }
            }
        }
        op_out[i] = (float)x;
    } else {
        const int64_t len = e1 - e0;
        const int64_t chunk = (len + G - 1) / G;
        int64_t c0 = e0 + (int64_t)li * chunk;
        c0 = c0 < e1 ? c0 : e1;
        const int64_t c1 = c0 + chunk < e1 ? c0 + chunk : e1;
        double a = 1.0, b = 0.0;  // x -> a x + b over this lane's chunk
        for (int64_t e = c0; e < c1; e += kEdgeBatch) {
            bool ok[kEdgeBatch];
            float wt[kEdgeBatch], you[kEdgeBatch];
            load_edges(e, c1, n, col, weight, op_in, ok, wt, you);
#pragma unroll
            for (int u = 0; u < kEdgeBatch; ++u) {  // in edge order
                if (ok[u] && fabsf(me - you[u]) < thr) {
                    const double w = strength * (double)wt[u];
                    a = (1.0 - w) * a;
                    b = (1.0 - w) * b + w * (double)you[u];
                }
            }
        }
        // butterfly: after level `off`, each lane holds the composition of
        // the 2 off consecutive chunks round it, later chunks applied last
#pragma unroll
        for (int off = 1; off < G; off <<= 1) {
            const double pa = __shfl_xor(a, off, 64);
            const double pb = __shfl_xor(b, off, 64);
            if (li & off) {  // mine is the later range
                b = a * pb + b;
                a = a * pa;
            } else {
                b = pa * b + pb;
                a = pa * a;
            }
        }
        if (active && li == 0) op_out[i] = (float)(a * (double)me + b);
    }
}

template <int G>
void launch_opinion(int64_t n, int64_t n_edges, const int64_t *row_ptr, const int32_t *col,
                    const float *weight, float thr, double strength, const float *op_in,
                    float *op_out, hipStream_t s) {
    constexpr int A = kGraphBlock / G;
    const int64_t blocks = (n + A - 1) / A;
    hipLaunchKernelGGL(k_opinion<G>, dim3((unsigned)blocks), dim3(kGraphBlock), 0, s, n, n_edges,
                       row_ptr, col, weight, thr, strength, op_in, op_out);
}

// A few lanes to a short row, a wave to a long one.  A row of thousands of edges
// is a long chain of loads in a few lanes, and the step waits for the longest:
// rows of kLongRow edges and more are left to the whole wave, one after the
// other, lane l composing the l-th part.  Offsets are 32 bits (fewer than 2^30
// edges and nodes).  Bound: three dependent loads (row, target, opinion), then
// the reads of the L2.
// MI355X, per step, four lanes alone / tiles / this: 10,000 power-law rows of 7
// (longest 2000) 20.6 / 13.7 / 7.0 us, 200,000 60 / 22 / 15.3; even rows of 7
// 3.0 / 3.8 / 2.9 and 9.7 / 10.0 / 9.0, with near targets 2.8 / 3.7 / 2.8 and
// 7.3 / 5.0 / 5.1.  Sixteen lanes / this: 60,000 power-law rows of 14 21.9 / 12.7,
// even 6.9 / 6.0.  kLongRow 32 or 128: within 6 %.  As many lanes as a mean row
// fills one batch of: two up to 8 edges (four take 5.5 and 13.7 us for the power-law
// rows of 7, but 2.9 and 9.5 for the even ones and 2.8 and 7.0 for the near ones),
// four up to 16, else eight (3,000 even rows of 20 2.9 us, with four 3.4, with 16 3.0).
constexpr int kLongRow = 64;

template <class T>
__device__ __forceinline__ T load32(const T *p, int i) {
    return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(p) +
                                        (uint32_t)i * (uint32_t)sizeof(T));
}

template <int G>
__global__ __launch_bounds__(kGraphBlock) void k_opinion_rows(int n, int n_edges,
                                                              const int64_t *__restrict__ row_ptr,
                                                              const int32_t *__restrict__ col,
                                                              const float *__restrict__ weight,
                                                              float thr, double strength,
                                                              const float *__restrict__ op_in,
                                                              float *__restrict__ op_out) {
    constexpr int A = kGraphBlock / G;
    const int tid = threadIdx.x, li = tid % G, lane = tid & 63;
    const int i = (int)blockIdx.x * A + tid / G;
    const bool active = i < n;
    float me = 0.0f;
    int e0 = 0, e1 = 0;
    if (active) {
        me = load32(op_in, i);
        const int64_t r0 = row_ptr[i], r1 = row_ptr[i + 1];
        e0 = (int)(r0 < 0 ? 0 : (r0 > n_edges ? n_edges : r0));
        e1 = (int)(r1 < e0 ? e0 : (r1 > n_edges ? n_edges : r1));
    }
    // part `who` of `of` of the edges [f0, f1) of a node at `own`: x -> a x + b,
    // then the parts' composition, later ones applied last
    auto part = [&](int f0, int f1, int who, auto of, float own, double &a, double &b) {
        constexpr int P = decltype(of)::value;
        const int chunk = (f1 - f0 + P - 1) / P;
        const int c0 = min(f0 + who * chunk, f1), c1 = min(c0 + chunk, f1);
        a = 1.0;
        b = 0.0;
        for (int e = c0; e < c1; e += kEdgeBatch) {
            int32_t j[kEdgeBatch];
            float wt[kEdgeBatch], you[kEdgeBatch];
            bool ok[kEdgeBatch];
#pragma unroll
            for (int u = 0; u < kEdgeBatch; ++u) {
                const int k = min(e + u, c1 - 1);
                j[u] = load32(col, k);
                wt[u] = load32(weight, k);
                ok[u] = e + u < c1 && j[u] >= 0 && j[u] < n;
            }
#pragma unroll
            for (int u = 0; u < kEdgeBatch; ++u) you[u] = load32(op_in, ok[u] ? j[u] : 0);
#pragma unroll
            for (int u = 0; u < kEdgeBatch; ++u) {  // in edge order
                if (ok[u] && fabsf(own - you[u]) < thr) {
                    const double w = strength * (double)wt[u];
                    a = (1.0 - w) * a;
                    b = (1.0 - w) * b + w * (double)you[u];
                }
            }
        }
#pragma unroll
        for (int off = 1; off < P; off <<= 1) {
            const double pa = __shfl_xor(a, off, 64), pb = __shfl_xor(b, off, 64);
            b = (who & off) ? a * pb + b : pa * b + pb;
            a = a * pa;
        }
    };
    const bool big = e1 - e0 >= kLongRow;
    double a, b;
    part(e0, big ? e0 : e1, li, std::integral_constant<int, G>{}, me, a, b);
    for (uint64_t todo = __ballot(big && li == 0); todo != 0; todo &= todo - 1) {
        const int o = __builtin_ctzll(todo);
        double wa, wb;
        part(__shfl(e0, o, 64), __shfl(e1, o, 64), lane, std::integral_constant<int, 64>{},
             __shfl(me, o, 64), wa, wb);
        if (lane == o) {
            a = wa;
            b = wb;
        }
    }
    if (active && li == 0) op_out[i] = (float)(a * (double)me + b);
}

// The tile kernel, for many short rows.  With lanes sharing a node, a row of 14
// edges gives 16 lanes one edge each in slots for kEdgeBatch of them, so most
// loads and FP64 maps are padding.  Here a block takes kTileNodes consecutive
// nodes, whose edges are one range, and brings it into LDS tile by tile with
// all its threads: consecutive loads, kTileLoads targets and then as many
// opinions in flight per thread, the opinion and the weight of an edge kept as a
// pair.  Then each lane applies its node's edges one by one in the stated order;
// a node with kTileRow or more edges in the tile is applied by its wave, lane l
// composing the l-th part of them, the parts composed in order.  What is left
// is the scattered read of the opinions: 64 lanes ask for 64 lines, about
// 15 M requests of the L2 per step of the first graph below, 5 in 6 of which hit.
//
// MI355X, per step, power-law rows (longest 2000), lanes per node / tiles:
// 1M nodes of mean degree 14, 136 / 104 us; of 8, 112 / 66.
// 128 nodes and 1024 edges: 256 and 2048 take 104, 512 and 4096 123, 64 and 768
// 110, 128 and 2304 106.  4 loads: 106.  kTileRow 24 or 32 gives up the order at
// rows where one lane is as fast, and then takes 45 us for 10,000 rows of 30
// edges that 64 does in 16.
constexpr int kTileNodes = 128, kTileEdges = 1024, kTileRow = 64, kTileLoads = 8;

__global__ __launch_bounds__(kTileNodes) void k_opinion_tile(int64_t n, int64_t n_edges,
                                                          const int64_t *__restrict__ row_ptr,
                                                          const int32_t *__restrict__ col,
                                                          const float *__restrict__ weight,
                                                          float thr, double strength,
                                                          const float *__restrict__ op_in,
                                                          float *__restrict__ op_out) {
    __shared__ float2 s_edge[kTileEdges];  // (opinion, weight); NaN opinion: no such node
    __shared__ int64_t s_lo, s_hi;
    const int tid = threadIdx.x, lane = tid & 63;
    const int64_t first = (int64_t)blockIdx.x * kTileNodes, i = first + tid;
    const bool active = i < n;
    const int64_t r0 = active ? row_ptr[i] : 0, r1 = active ? row_ptr[i + 1] : 0;
    const float me = active ? op_in[i] : 0.0f;
    double x = (double)me;
    // rows that ascend within [0, n_edges] lie end to end
    const bool csr = !active || (r0 >= 0 && r0 <= r1 && r1 <= n_edges);
    if (tid == 0) s_lo = r0;
    if (active && (tid == kTileNodes - 1 || i == n - 1)) s_hi = r1;
    if (!__syncthreads_and(csr ? 1 : 0)) {
        // anything else: the clamped ranges, node by node from memory
        if (!active) return;
        const int64_t e0 = r0 < 0 ? 0 : (r0 > n_edges ? n_edges : r0);
        const int64_t e1 = r1 < e0 ? e0 : (r1 > n_edges ? n_edges : r1);
        for (int64_t e = e0; e < e1; ++e) {
            const int32_t j = col[e];
            if (j < 0 || (int64_t)j >= n) continue;
            const float you = op_in[j];
            if (fabsf(me - you) < thr) {
                const double w = strength * (double)weight[e];
                x = (1.0 - w) * x + w * (double)you;
            }
        }
        op_out[i] = (float)x;
        return;
    }
    const int64_t lo = s_lo, hi = s_hi;
    for (int64_t t0 = lo; t0 < hi; t0 += kTileEdges) {
        const int len = hi - t0 < kTileEdges ? (int)(hi - t0) : kTileEdges;
        for (int k0 = tid; k0 < len; k0 += kTileNodes * kTileLoads) {
            int32_t j[kTileLoads];
            float wt[kTileLoads], you[kTileLoads];
#pragma unroll
            for (int u = 0; u < kTileLoads; ++u) {
                const int k = k0 + u * kTileNodes;
                const int64_t e = t0 + (k < len ? k : k0);
                j[u] = col[e];
                wt[u] = weight[e];
            }
#pragma unroll
            for (int u = 0; u < kTileLoads; ++u) {
                const bool ok = j[u] >= 0 && (int64_t)j[u] < n;
                const float y = op_in[ok ? j[u] : 0];
                you[u] = ok ? y : __builtin_nanf("");
            }
#pragma unroll
            for (int u = 0; u < kTileLoads; ++u) {
                const int k = k0 + u * kTileNodes;
                if (k < len) s_edge[k] = make_float2(you[u], wt[u]);
            }
        }
        __syncthreads();
        // the node's edges in the tile
        const int64_t f0 = r0 > t0 ? r0 - t0 : 0, f1 = r1 - t0 < len ? r1 - t0 : len;
        const int b0 = (int)f0, b1 = f1 > f0 ? (int)f1 : (int)f0;
        const bool big = b1 - b0 >= kTileRow;
        for (int b = b0; b < (big ? b0 : b1); ++b) {
            const float2 ed = s_edge[b];
            if (fabsf(me - ed.x) < thr) {
                const double w = strength * (double)ed.y;
                x = (1.0 - w) * x + w * (double)ed.x;
            }
        }
        for (uint64_t todo = __ballot(big); todo != 0; todo &= todo - 1) {
            const int o = __builtin_ctzll(todo);
            const int q0 = __builtin_amdgcn_readlane(b0, o), q1 = __builtin_amdgcn_readlane(b1, o);
            const float own = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(me), o));
            const int part = (q1 - q0 + 63) >> 6;
            const int c0 = min(q0 + lane * part, q1), c1 = min(c0 + part, q1);
            double a = 1.0, s = 0.0;  // x -> a x + s over this lane's part
            for (int b = c0; b < c1; ++b) {
                const float2 ed = s_edge[b];
                if (fabsf(own - ed.x) < thr) {
                    const double w = strength * (double)ed.y;
                    a = (1.0 - w) * a;
                    s = (1.0 - w) * s + w * (double)ed.x;
                }
            }
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {  // later parts applied last
                const double pa = __shfl_xor(a, off, 64), ps = __shfl_xor(s, off, 64);
                s = (lane & off) ? a * ps + s : pa * s + ps;
                a = a * pa;
            }
            if (lane == o) x = a * x + s;
        }
        __syncthreads();
    }
    if (active) op_out[i] = (float)x;
}

// What takes the step where the caller leaves the choice.  Below 3 edges a
// node, one lane per node reads little that it does not need (1M rows of 1 to 3:
// 17 us, tiles 20).  From 24 a share of a row fills the slots of 16 lanes (300,000 rows of
// 30: 50 us, tiles 53).  Between, rows by a few lanes and by waves: even rows take no
// longer than with lanes alone at any size (3,000 to 2M nodes), power-law
// rows a half to a seventh.  In large graphs tiles, whose loads of the edges are
// consecutive: power-law / even rows of 5 at 1M nodes (5.2 and 5.0 M edges) 52 / 35 us by
// rows and 47 / 38 in tiles, of 7 68 / 46 and 63 / 47; longer rows from 8 M edges: 500,000 of
// 14 (7 M) 50 / 36 and 59 / 39, 1M of 8 70 / 55 and 66 / 49, of 14 108 / 87 and 104 / 85.
enum class GraphForm { kLanes, kRows, kTiles };
GraphForm graph_form(int64_t n_edges, double mean_degree) {
    if (mean_degree < 3.0 || mean_degree >= 24.0) return GraphForm::kLanes;
    return n_edges < (mean_degree <= 8.0 ? 5000000 : 8000000) ? GraphForm::kRows : GraphForm::kTiles;
}

// Lanes per node for the rest, from the mean degree: power-law rows are uneven,
// so wide groups pay off early.
int graph_auto_lanes(double mean_degree) {
    if (mean_degree < 3.0) return 1;
    if (mean_degree < 256.0) return 16;
    return 64;
}

}  // namespace

}  // namespace flock

using namespace flock;

extern "C" {

int gr_opinion_step(int64_t n, int64_t n_edges, const int64_t *row_ptr, const int32_t *col,
                    const float *weight, float threshold, float strength, const float *op_in,
                    float *op_out, int lanes, void *stream) {
    if (n < 0 || n > INT32_MAX || n_edges < 0)
        return set_error(ENV_EINVAL, "need 0 <= n <= 2^31 - 1 and n_edges >= 0");
    if (!isfinite(threshold) || !isfinite(strength))
        return set_error(ENV_EINVAL, "threshold and strength must be finite");
    if (lanes != 0 && lanes != 1 && lanes != 4 && lanes != 16 && lanes != 64)
        return set_error(ENV_EINVAL, "lanes must be 0, 1, 4, 16 or 64");
    if (n == 0) return ENV_OK;
    if (!row_ptr || !op_in || !op_out || (n_edges > 0 && (!col || !weight)))
        return set_error(ENV_EINVAL, "NULL array");
    if (op_in == op_out) return set_error(ENV_EINVAL, "op_in and op_out must differ");
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const double st = (double)strength;
    const double mean = (double)n_edges / (double)n;
    const GraphForm form = lanes ? GraphForm::kLanes : graph_form(n_edges, mean);
    if (form != GraphForm::kLanes) {
        auto rows = [&](auto kernel, int per_block) {
            hipLaunchKernelGGL(kernel, dim3((unsigned)((n + per_block - 1) / per_block)),
                               dim3(kGraphBlock), 0, s, (int)n, (int)n_edges, row_ptr, col, weight,
                               threshold, st, op_in, op_out);
        };
        if (form == GraphForm::kTiles)
            hipLaunchKernelGGL(k_opinion_tile, dim3((unsigned)((n + kTileNodes - 1) / kTileNodes)),
                               dim3(kTileNodes), 0, s, n, n_edges, row_ptr, col, weight, threshold,
                               st, op_in, op_out);
        else if (mean <= 2.0 * kEdgeBatch) rows(k_opinion_rows<2>, kGraphBlock / 2);
        else if (mean < 4.0 * kEdgeBatch) rows(k_opinion_rows<4>, kGraphBlock / 4);
        else rows(k_opinion_rows<8>, kGraphBlock / 8);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return set_error(ENV_EHIP, "gr_opinion_step: %s", hipGetErrorString(e));
        return ENV_OK;
    }
    const int g = lanes ? lanes : graph_auto_lanes(mean);
    auto run = [&](auto tag) {
        constexpr int G = decltype(tag)::value;
        launch_opinion<G>(n, n_edges, row_ptr, col, weight, threshold, st, op_in, op_out, s);
    };
    if (g == 1) run(std::integral_constant<int, 1>{});
    else if (g == 4) run(std::integral_constant<int, 4>{});
    else if (g == 16) run(std::integral_constant<int, 16>{});
    else run(std::integral_constant<int, 64>{});
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return set_error(ENV_EHIP, "gr_opinion_step: %s", hipGetErrorString(e));
    return ENV_OK;
}

}  // extern "C"
