// Edge-weight derivatives that serve the constrained-SGD edge scaling of
// Sec. 3.3.4 (Alg. 1): the undirected edge list of a CSR graph, FP64
// Rayleigh quotients R_i = u_i^T L(w) u_i / u_i^T B u_i with their
// edge-weight gradients (first-order eigenvalue perturbation, Sec. 3.3.3),
// and the reverse pass through the Gauss-Seidel smoothing.
#include "gr_internal.hpp"
#include "gr_device.hpp"

#include <algorithm>
#include <mutex>

namespace gr {

constexpr int kA = 256;

// lanes per row for the row-walking kernels below: one below a mean degree
// of 8 (extra lanes only add waves there), else a power of two up to a
// wave, about half the mean degree (hub rows loop)
inline int lanes_per_row(int64_t n, int64_t nnz) {
    if (n <= 0 || nnz < 8 * n) return 1;
    int G = 4;
    while (G < kWave && G * 2 <= nnz / n) G *= 2;
    return G;
}

// ------------------------------------------------------------- edge list
// Undirected edge e = (p, q), p < q, is numbered by the position of the upper
// entry (p, q) among all upper entries in CSR order; both stored entries map
// to it.
// G lanes per row for both kernels (one thread would serialise a hub row)
__global__ void k_upper_counts(const int32_t* __restrict__ rp, const int32_t* __restrict__ col,
                               int64_t n, int G, int32_t* __restrict__ flag) {
    const int64_t t = (int64_t)blockIdx.x * kA + threadIdx.x;
    const int64_t v = t / G;
    const int lane = (int)(t % G);
    if (v >= n) return;
    for (int32_t e = rp[v] + lane; e < rp[v + 1]; e += G) flag[e] = col[e] > v ? 1 : 0;
}

__global__ void k_edge_fill(const int32_t* __restrict__ rp, const int32_t* __restrict__ col,
                            const int32_t* __restrict__ pos, int64_t n, int G,
                            int32_t* __restrict__ eu, int32_t* __restrict__ ev,
                            int32_t* __restrict__ eoe) {
    const int64_t t = (int64_t)blockIdx.x * kA + threadIdx.x;
    const int64_t v = t / G;
    const int lane = (int)(t % G);
    if (v >= n) return;
    for (int32_t e = rp[v] + lane; e < rp[v + 1]; e += G) {
        int32_t j = col[e];
        if (j > v) {
            int32_t k = pos[e];
            eu[k] = (int32_t)v;
            ev[k] = j;
            if (eoe) eoe[e] = k;
        } else if (eoe) {
            // the partner entry (j, v) lies in row j; columns ascend there
            int32_t lo = rp[j], hi = rp[j + 1] - 1, f = -1;
            while (lo <= hi) {
                int32_t mid = lo + ((hi - lo) >> 1);
                int32_t c = col[mid];
                if (c == (int32_t)v) { f = mid; break; }
                if (c < (int32_t)v) lo = mid + 1; else hi = mid - 1;
            }
            eoe[e] = f >= 0 ? pos[f] : -1;
        }
    }
}

int edge_list(const gr_graph* g, int32_t* eu, int32_t* ev, int32_t* eoe, int64_t* n_edges, Arena& ws,
              hipStream_t st) {
    *n_edges = 0;
    if (g->nnz == 0) return GR_OK;
    size_t mark = ws.used;
    int32_t* flag = ws.take<int32_t>(g->nnz);
    int32_t* pos = ws.take<int32_t>(g->nnz + 1);
    if (ws.overflow) return set_error(GR_ENOMEM, "workspace too small (edge list)");
    const int G = lanes_per_row(g->n, g->nnz);
    const unsigned nb = blocks_for(g->n * G, kA);
    hipLaunchKernelGGL(k_upper_counts, dim3(nb), dim3(kA), 0, st, g->row_ptr, g->col, g->n, G, flag);
    GR_LAUNCHED("upper counts");
    GR_TRY(scan_exclusive_i32(flag, pos, g->nnz, pos + g->nnz, ws, st));
    hipLaunchKernelGGL(k_edge_fill, dim3(nb), dim3(kA), 0, st, g->row_ptr, g->col, pos, g->n, G, eu,
                       ev, eoe);
    GR_LAUNCHED("edge fill");
    int32_t E = 0;
    GR_TRY(fetch({{pos + g->nnz, sizeof(int32_t)}}, &E, st));
    *n_edges = E;
    ws.used = mark;
    return GR_OK;
}

// set when a caller-supplied edge id lies outside [0, E); the offending
// entry is never dereferenced
__device__ int32_t g_bad_edge_id;

__global__ void k_expand_weights(const int32_t* __restrict__ eoe, int64_t nnz, int64_t E,
                                 const float* __restrict__ wE, float* __restrict__ w) {
    int64_t e = (int64_t)blockIdx.x * kA + threadIdx.x;
    if (e >= nnz) return;
    int32_t k = eoe[e];
    if (k >= 0 && k < E) {
        w[e] = wE[k];
    } else {
        w[e] = 0.0f;
        g_bad_edge_id = 1;
    }
}

static int reset_bad_edge_flag(hipStream_t st) {
    int32_t zero = 0;
    GR_HIP(hipMemcpyToSymbolAsync(HIP_SYMBOL(g_bad_edge_id), &zero, sizeof(int32_t), 0,
                                  hipMemcpyHostToDevice, st));
    GR_HIP(hipStreamSynchronize(st));
    return GR_OK;
}

static int check_bad_edge_flag(hipStream_t st) {
    int32_t bad = 0;
    GR_HIP(hipMemcpyFromSymbolAsync(&bad, HIP_SYMBOL(g_bad_edge_id), sizeof(int32_t), 0,
                                    hipMemcpyDeviceToHost, st));
    GR_HIP(hipStreamSynchronize(st));
    if (bad) return set_error(GR_EINVAL, "edge_of_entry holds ids outside [0, n_edges)");
    return GR_OK;
}

int expand_weights(const int32_t* eoe, int64_t nnz, int64_t E, const float* wE, float* w,
                   hipStream_t st) {
    if (nnz == 0) return GR_OK;
    GR_TRY(reset_bad_edge_flag(st));
    hipLaunchKernelGGL(k_expand_weights, dim3(blocks_for(nnz, kA)), dim3(kA), 0, st, eoe, nnz, E, wE,
                       w);
    GR_LAUNCHED("expand weights");
    return check_bad_edge_flag(st);
}

// ------------------------------------------------------- Rayleigh quotients
constexpr int kRqBlocks = 512;

// Bound by the gathers of the edges' end rows (16 m bytes per edge, out of
// L2 on reduced graphs).  cw lanes hold one edge's columns, two each as one
// 16-byte load where m and U's alignment allow it, so that a wave's load
// covers 64 / cw edges' whole rows; kRqU edges are in flight per lane.
// (The column as a grid dimension read the edge list m times over, and a
// thread per edge in the gradient touched a line per lane and column: 65 and
// 57 us at 1.28M edges and m = 10; here 22 and 26 us, 10 and 9 TB/s with the
// edge list.)
constexpr int kRqThreads = 512;
constexpr int kRqWaves = kRqThreads / kWave;
constexpr int kRqU = 4;

// columns cl C .. of row v
template <int C>
__device__ inline void rq_row(const double* __restrict__ U, int64_t v, int m, int cl, double* x) {
    const double* at = U + v * m + cl * C;
    if constexpr (C == 2) {
        const double2 t = *reinterpret_cast<const double2*>(at);
        x[0] = t.x;
        x[1] = t.y;
    } else {
        x[0] = *at;
    }
}

// per block (grid-stride): partial sums over edges of
//   num_i = sum_e w_e (u_pi - u_qi)^2   and, for B = D(w),
//   den_i = sum_e w_e (u_pi^2 + u_qi^2)  (= u_i^T D u_i),
// for B = I the partial sums over nodes of den_i = u_i^T u_i
template <int C>
__global__ void __launch_bounds__(kRqThreads) k_rq_sums(int64_t n, int64_t E,
                                                        const int32_t* __restrict__ eu,
                                                        const int32_t* __restrict__ ev,
                                                        const double* __restrict__ w,
                                                        const double* __restrict__ U, int32_t m,
                                                        int cw, int mode,
                                                        double* __restrict__ part_num,
                                                        double* __restrict__ part_den) {
    __shared__ double red[2][kRqWaves][kWave * C];
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    const int slots = kWave / cw, slot = lane / cw, cl = lane - slot * cw;
    const bool active = slot < slots;
    const int64_t wave = (int64_t)blockIdx.x * kRqWaves + wid;
    const int64_t step = (int64_t)gridDim.x * kRqWaves * slots * kRqU;
    double num[C], den[C];
#pragma unroll
    for (int q = 0; q < C; ++q) num[q] = den[q] = 0.0;
    if (active)
        for (int64_t b = wave * slots * kRqU + slot; b < E; b += step) {
            int32_t p[kRqU], q[kRqU];
            double we[kRqU], xp[kRqU][C], xq[kRqU][C];
#pragma unroll
            for (int u = 0; u < kRqU; ++u) {
                const int64_t e = b + u * slots < E ? b + u * slots : b;
                p[u] = eu[e];
                q[u] = ev[e];
                we[u] = w[e];
            }
#pragma unroll
            for (int u = 0; u < kRqU; ++u) {
                rq_row<C>(U, p[u], m, cl, xp[u]);
                rq_row<C>(U, q[u], m, cl, xq[u]);
            }
#pragma unroll
            for (int u = 0; u < kRqU; ++u)
                if (b + u * slots < E) {
#pragma unroll
                    for (int k = 0; k < C; ++k) {
                        const double df = xp[u][k] - xq[u][k];
                        num[k] = fma(we[u] * df, df, num[k]);
                        if (mode == GR_RQ_DEGREE)
                            den[k] = fma(we[u], xp[u][k] * xp[u][k] + xq[u][k] * xq[u][k], den[k]);
                    }
                }
        }
    if (active && mode == GR_RQ_IDENTITY)
        for (int64_t v = wave * slots + slot; v < n; v += (int64_t)gridDim.x * kRqWaves * slots) {
            double x[C];
            rq_row<C>(U, v, m, cl, x);
#pragma unroll
            for (int k = 0; k < C; ++k) den[k] = fma(x[k], x[k], den[k]);
        }
#pragma unroll
    for (int k = 0; k < C; ++k) {
        red[0][wid][lane * C + k] = num[k];
        red[1][wid][lane * C + k] = den[k];
    }
    __syncthreads();
    // column t % m of the sums t / m (num, den): slots in order, then waves
    const int t = threadIdx.x;
    if (t < 2 * m) {
        const int c = t % m;
        double s = 0.0;
        for (int k = 0; k < kRqWaves; ++k) {
            double x = 0.0;
            for (int l = 0; l < slots; ++l) x += red[t / m][k][l * cw * C + c];
            s += x;
        }
        (t < m ? part_num : part_den)[(int64_t)c * gridDim.x + blockIdx.x] = s;
    }
}

// a block per column: its nb partial sums in a fixed tree
__global__ void __launch_bounds__(kA) k_rq_final(const double* __restrict__ part_num,
                                                 const double* __restrict__ part_den, int nb,
                                                 double* __restrict__ R,
                                                 double* __restrict__ den_out) {
    __shared__ double sh[2][kA / kWave];
    const int i = blockIdx.x;
    double num = 0.0, den = 0.0;
    for (int b = threadIdx.x; b < nb; b += kA) {
        num += part_num[(int64_t)i * nb + b];
        den += part_den[(int64_t)i * nb + b];
    }
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        num += __shfl_xor(num, off, kWave);
        den += __shfl_xor(den, off, kWave);
    }
    if ((threadIdx.x & (kWave - 1)) == 0) {
        sh[0][threadIdx.x / kWave] = num;
        sh[1][threadIdx.x / kWave] = den;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int k = 1; k < kA / kWave; ++k) {
        num += sh[0][k];
        den += sh[1][k];
    }
    R[i] = den != 0.0 ? num / den : 0.0;
    if (den_out) den_out[i] = den;
}

// gw_e = sum_i gR_i [ (u_pi - u_qi)^2 - (B = D: R_i (u_pi^2 + u_qi^2)) ] / den_i
template <int C>
__global__ void __launch_bounds__(kRqThreads) k_rq_backward(
    int64_t E, const int32_t* __restrict__ eu, const int32_t* __restrict__ ev,
    const double* __restrict__ U, int32_t m, int cw, int mode, const double* __restrict__ R,
    const double* __restrict__ den, const double* __restrict__ gR, double* __restrict__ gw) {
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    const int slots = kWave / cw, slot = lane / cw, cl = lane - slot * cw;
    const int64_t b = ((int64_t)blockIdx.x * kRqWaves + wid) * slots * kRqU + slot;
    double f[C], r[C];
    bool use[C];
#pragma unroll
    for (int k = 0; k < C; ++k) {
        const double d = den[cl * C + k];
        use[k] = d != 0.0;
        f[k] = use[k] ? gR[cl * C + k] / d : 0.0;
        r[k] = R[cl * C + k];
    }
    int32_t p[kRqU], q[kRqU];
    double xp[kRqU][C], xq[kRqU][C];
#pragma unroll
    for (int u = 0; u < kRqU; ++u) {
        const int64_t e = min(b + u * slots, E - 1);
        p[u] = eu[e];
        q[u] = ev[e];
    }
#pragma unroll
    for (int u = 0; u < kRqU; ++u) {
        rq_row<C>(U, p[u], m, cl, xp[u]);
        rq_row<C>(U, q[u], m, cl, xq[u]);
    }
#pragma unroll
    for (int u = 0; u < kRqU; ++u) {
        double g = 0.0;
#pragma unroll
        for (int k = 0; k < C; ++k) {
            const double df = xp[u][k] - xq[u][k];
            double t = df * df;
            if (mode == GR_RQ_DEGREE) t -= r[k] * (xp[u][k] * xp[u][k] + xq[u][k] * xq[u][k]);
            if (use[k]) g = fma(f[k], t, g);
        }
        // the edge's lanes, in order (every lane of the wave takes part)
        double s = g;
        for (int l = 1; l < cw; ++l) s += __shfl(g, min(lane + l, kWave - 1), kWave);
        if (slot < slots && cl == 0 && b + u * slots < E) gw[b + u * slots] = s;
    }
}

// whether a lane may take two columns per load
static bool rq_pairs(const double* U, int32_t m) {
    return m % 2 == 0 && (reinterpret_cast<uintptr_t>(U) & 15) == 0;
}

int rq_forward(int64_t n, int64_t E, const int32_t* eu, const int32_t* ev, const double* w,
               const double* U, int32_t m, int32_t mode, double* R, double* den, Arena& ws,
               hipStream_t st) {
    size_t mark = ws.used;
    double* pn = ws.take<double>((size_t)kRqBlocks * m);
    double* pd = ws.take<double>((size_t)kRqBlocks * m);
    if (ws.overflow) return set_error(GR_ENOMEM, "workspace too small (rq)");
    // no more blocks than the edges and nodes fill
    const bool pair = rq_pairs(U, m);
    const int cw = pair ? m / 2 : m;
    const int64_t per = (int64_t)kRqWaves * (kWave / cw);
    const int nb = (int)std::min<int64_t>(
        kRqBlocks, std::max<int64_t>(1, std::max((E + per * kRqU - 1) / (per * kRqU),
                                                 mode == GR_RQ_IDENTITY ? (n + per - 1) / per : 0)));
    if (pair)
        hipLaunchKernelGGL(k_rq_sums<2>, dim3(nb), dim3(kRqThreads), 0, st, n, E, eu, ev, w, U, m, cw,
                           mode, pn, pd);
    else
        hipLaunchKernelGGL(k_rq_sums<1>, dim3(nb), dim3(kRqThreads), 0, st, n, E, eu, ev, w, U, m, cw,
                           mode, pn, pd);
    GR_LAUNCHED("rq sums");
    hipLaunchKernelGGL(k_rq_final, dim3(m), dim3(kA), 0, st, (const double*)pn, (const double*)pd, nb,
                       R, den);
    GR_LAUNCHED("rq final");
    ws.used = mark;
    return GR_OK;
}

// ------------------------------------- Rayleigh quotients, no allocation
// The scratch of rq_forward (three per-block partial-sum arrays) for the
// widest block, m = 64, in a file-scope device array: one copy per GPU,
// held until the process ends.  Host code never passes the array's name to
// a kernel (in host code it is a stand-in, not a device address); it looks
// up the array's address on each device once, with that device current,
// and passes that pointer instead.
constexpr size_t kRqScratchPart = ((size_t)kRqBlocks * 64 * sizeof(double) + 255) & ~size_t(255);
constexpr size_t kRqScratchBytes = 3 * kRqScratchPart;
static __device__ __align__(256) unsigned char scratch[kRqScratchBytes];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void* g_scratch_ptr[kMaxDevices] = {};

static int scratch_on_current_device(void** out) {
    int dev = 0;
    GR_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices)
        return set_error(GR_EINVAL, "device %d: at most %d devices are supported", dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        GR_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return set_error(GR_EHIP, "no device address for the static scratch array");
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return GR_OK;
}

size_t rq_forward_scratch_bytes(int32_t m) {
    Arena sizing(nullptr, ~size_t(0));
    for (int i = 0; i < 3; ++i) sizing.take<double>((size_t)kRqBlocks * (size_t)(m > 0 ? m : 0));
    return sizing.used;
}

size_t rq_forward_scratch_capacity() { return kRqScratchBytes; }

int rq_forward_noalloc(int64_t n, int64_t E, const int32_t* eu, const int32_t* ev, const double* w,
                       const double* U, int32_t m, int32_t mode, double* R, double* den,
                       hipStream_t st) {
    const size_t need = rq_forward_scratch_bytes(m);
    if (need > kRqScratchBytes)
        return set_error(GR_EINVAL, "m = %d needs %zu scratch bytes; the static scratch holds %zu",
                         m, need, kRqScratchBytes);
    void* p = nullptr;
    GR_TRY(scratch_on_current_device(&p));
    Arena A(p, kRqScratchBytes);
    return rq_forward(n, E, eu, ev, w, U, m, mode, R, den, A, st);
}

int rq_backward(int64_t E, const int32_t* eu, const int32_t* ev, const double* U, int32_t m,
                int32_t mode, const double* R, const double* den, const double* gR, double* gw,
                hipStream_t st) {
    if (E == 0) return GR_OK;
    const bool pair = rq_pairs(U, m);
    const int cw = pair ? m / 2 : m;
    const unsigned nb = blocks_for(E, kRqWaves * (kWave / cw) * kRqU);
    if (pair)
        hipLaunchKernelGGL(k_rq_backward<2>, dim3(nb), dim3(kRqThreads), 0, st, E, eu, ev, U, m, cw,
                           mode, R, den, gR, gw);
    else
        hipLaunchKernelGGL(k_rq_backward<1>, dim3(nb), dim3(kRqThreads), 0, st, E, eu, ev, U, m, cw,
                           mode, R, den, gR, gw);
    GR_LAUNCHED("rq backward");
    return GR_OK;
}

}  // namespace gr

// ------------------------------------------- reverse pass of the smoothing
// A colour step maps row i of colour c (d_i > 0) to x_i' = sum_j w_ij x_j / d_i
// and leaves the other rows.  Its partial derivatives are
// dx_i'/dw_ij = (x_j - x_i') / d_i and dx_i'/dx_j = w_ij / d_i, and x_i' does
// not depend on the old x_i.  The steps are undone in reverse order (sweeps
// S..1, colours C-1..0) in pull form.  Let g_i be the adjoint of the value
// x_i^s that step (s, c) gives row i, and h_i = g_i / d_i.  That value is
// read by the steps of sweep s with a larger colour and by the steps of
// sweep s+1 with a smaller one, so
//   g_i = [s = S] G_i + sum_{j in N(i)} w_ij h_j,
// with h_j from sweep s when colour(j) > c and from sweep s+1 when
// colour(j) < c.  One array H holds exactly that: in reverse order, step
// (s, c) runs after the larger colours of sweep s have rewritten their rows
// and before the smaller colours of sweep s replace their sweep-(s+1)
// values (H starts at zero: there is no sweep S+1).  Then
//   wbar_ij += h_i . (x_j - x_i')   for j in N(i),
// and, once sweep 1 is undone, x_j^0 has been read only by the sweep-1 steps
// of smaller colours:  gX0_j = sum_{i in N(j), colour(i) < colour(j)} w_ij h_i
// (a row without neighbours keeps G_j).  The state seen by step (s, c) is, in
// the colour-major order, rows of colour < c from X_s and rows of colour
// >= c from X_{s-1}; so the sweep-boundary states X_0..X_S (stored, or
// recomputed from X_0) suffice.  No value is accumulated by atomics and no
// array is written by two steps of one launch (a colour class has no inner
// edges).
namespace gr {

template <int E>
__device__ inline void load_f32(const float* __restrict__ A, int64_t row, int K, int q, float* v) {
#pragma unroll
    for (int i = 0; i < E; i += 4) {
        float4 t = *reinterpret_cast<const float4*>(A + row * K + q * E + i);
        v[i] = t.x; v[i + 1] = t.y; v[i + 2] = t.z; v[i + 3] = t.w;
    }
}
template <int E>
__device__ inline void store_f32(float* __restrict__ A, int64_t row, int K, int q, const float* v) {
#pragma unroll
    for (int i = 0; i < E; i += 4)
        *reinterpret_cast<float4*>(A + row * K + q * E + i) = make_float4(v[i], v[i + 1], v[i + 2], v[i + 3]);
}

// d_i = sum_j w_ij, G lanes per row; constant over the sweeps
__global__ void k_row_weight(const int32_t* __restrict__ rp, const float* __restrict__ w, int64_t n,
                             int G, float* __restrict__ dw) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t r = t / G;
    const int lane = (int)(t % G);
    if (r >= n) return;  // G divides the wave: a row's lanes leave together
    float d = 0.0f;
    for (int32_t e = rp[r] + lane; e < rp[r + 1]; e += G) d += w[e];
    for (int off = 1; off < G; off <<= 1) d += __shfl_xor(d, off, kWave);
    if (lane == 0) dw[r] = d;
}

// trips (entries per lane) up to which a reverse step keeps the gathered
// state rows in registers instead of a second pass over the row: 32 values
// per lane (8 float32 or 4 bfloat16 chunks)
template <int DT>
constexpr int vjp_keep() { return 32 / Chunk<DT>::E; }

// Rows [lo, hi) of colour c with degree <= kLongRow, L = Q*P lanes per row.
// FINAL = 0: the reverse step (G = the cotangent in the last sweep, else
// null; the last sweep is undone first and stores its gradients, the others
// add to them).  FINAL = 1: gX0 of those rows into out.
template <int Q, int P, int DT, int FINAL>
__global__ void __launch_bounds__(256) k_vjp_rows(
    const int32_t* __restrict__ rp, const int32_t* __restrict__ col, const float* __restrict__ w,
    const void* __restrict__ Xs, const void* __restrict__ Xp, int32_t K, int64_t clo, int64_t lo,
    int64_t hi, const float* __restrict__ dw, const float* __restrict__ G, float* __restrict__ H,
    float* __restrict__ ge, int first, float* __restrict__ out) {
    constexpr int L = Q * P;
    constexpr int RPW = kWave / L;
    constexpr int E = Chunk<DT>::E;
    const int lane = threadIdx.x & (kWave - 1);
    const int l = lane % L;
    const int p = l / Q, q = l % Q;
    const int64_t wave = ((int64_t)blockIdx.x * 256 + threadIdx.x) / kWave;
    const int64_t r = lo + wave * RPW + lane / L;
    if (r >= hi) return;
    const int32_t e0 = rp[r], e1 = rp[r + 1];
    const float d = dw[r];
    if (!(d > 0.0f)) {  // no neighbours, or no weight: no step changes this row
        if (FINAL && p == 0) {
            float gi[E];
            load_f32<E>(G, r, K, q, gi);
            store_f32<E>(out, r, K, q, gi);
        }
        if (!FINAL && first && q == 0)
            for (int32_t e = e0 + p; e < e1; e += P) ge[e] = 0.0f;
        return;
    }
    float acc[E];
#pragma unroll
    for (int i = 0; i < E; ++i) acc[i] = 0.0f;
    const int32_t trips = (e1 - e0 + P - 1) / P;  // the same for every lane of the row
    if constexpr (!FINAL) {
        constexpr int kKeep = vjp_keep<DT>();
        if (trips <= kKeep) {
            // one pass: the state rows x_j are gathered with h_j and kept for
            // the gradient
            float xj[kKeep][E];
#pragma unroll
            for (int t = 0; t < kKeep; ++t) {
                if (t < trips) {
                    const int32_t e = e0 + p + t * P;
                    const bool ok = e < e1;
                    const int32_t j = ok ? col[e] : (int32_t)r;
                    Chunk<DT>::load(j < clo ? Xs : Xp, j, K, q, xj[t]);
                    if (ok) {
                        float hj[E];
                        load_f32<E>(H, j, K, q, hj);
                        const float wt = w[e];
#pragma unroll
                        for (int i = 0; i < E; ++i) acc[i] = __fmaf_rn(wt, hj[i], acc[i]);
                    }
                }
            }
#pragma unroll
            for (int off = Q; off < L; off <<= 1)
#pragma unroll
                for (int i = 0; i < E; ++i) acc[i] += __shfl_xor(acc[i], off, kWave);
            if (G) {
                float gi[E];
                load_f32<E>(G, r, K, q, gi);
#pragma unroll
                for (int i = 0; i < E; ++i) acc[i] += gi[i];
            }
            float h[E], xi[E];
#pragma unroll
            for (int i = 0; i < E; ++i) h[i] = acc[i] / d;
            if (p == 0) store_f32<E>(H, r, K, q, h);
            Chunk<DT>::load(Xs, r, K, q, xi);
#pragma unroll
            for (int t = 0; t < kKeep; ++t) {
                if (t < trips) {
                    const int32_t e = e0 + p + t * P;
                    float sdot = 0.0f;
#pragma unroll
                    for (int i = 0; i < E; ++i) sdot = __fmaf_rn(h[i], xj[t][i] - xi[i], sdot);
                    sdot = qsum<Q>(sdot);
                    if (e < e1 && q == 0) ge[e] = first ? sdot : ge[e] + sdot;
                }
            }
            return;
        }
    }
    for (int32_t e = e0 + p; e < e1; e += P) {
        const int32_t j = col[e];
        if (FINAL && j >= clo) continue;
        float hj[E];
        load_f32<E>(H, j, K, q, hj);
        const float wt = w[e];
#pragma unroll
        for (int i = 0; i < E; ++i) acc[i] = __fmaf_rn(wt, hj[i], acc[i]);
    }
#pragma unroll
    for (int off = Q; off < L; off <<= 1)
#pragma unroll
        for (int i = 0; i < E; ++i) acc[i] += __shfl_xor(acc[i], off, kWave);
    if constexpr (FINAL) {
        if (p == 0) store_f32<E>(out, r, K, q, acc);
    } else {
        if (G) {
            float gi[E];
            load_f32<E>(G, r, K, q, gi);
#pragma unroll
            for (int i = 0; i < E; ++i) acc[i] += gi[i];
        }
        float h[E], xi[E];
#pragma unroll
        for (int i = 0; i < E; ++i) h[i] = acc[i] / d;
        if (p == 0) store_f32<E>(H, r, K, q, h);
        Chunk<DT>::load(Xs, r, K, q, xi);
        for (int32_t t = 0; t < trips; ++t) {
            const int32_t e = e0 + p + t * P;
            const bool ok = e < e1;
            const int32_t j = ok ? col[e] : (int32_t)r;
            float xj[E];
            Chunk<DT>::load(j < clo ? Xs : Xp, j, K, q, xj);
            float s = 0.0f;
#pragma unroll
            for (int i = 0; i < E; ++i) s = __fmaf_rn(h[i], xj[i] - xi[i], s);
            s = qsum<Q>(s);
            if (ok && q == 0) ge[e] = first ? s : ge[e] + s;
        }
    }
}

// The rows of degree above kLongRow (the colour's first rows: its degree
// tiers come in decreasing order) are cut into pieces of kPiece entries, so
// that a hub row is spread over many workgroups.  Two launches: the partial
// sums of w_ij h_j of every piece, then a workgroup per piece that forms
// h_i = g_i / d_i and applies it to the piece's entries.  Weights are
// positive, so d_i > 0 on these rows.
constexpr int kPiece = 256;

__global__ void k_piece_counts(const int32_t* __restrict__ rp, int64_t n, int32_t* __restrict__ cnt) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n) return;
    const int32_t deg = rp[r + 1] - rp[r];
    cnt[r] = deg > kLongRow ? (deg + kPiece - 1) / kPiece : 0;
}

__global__ void k_gather_i32(const int32_t* __restrict__ src, const int64_t* __restrict__ idx,
                             int64_t m, int32_t* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < m) out[i] = src[idx[i]];
}

// the row of piece k among the long rows [lo, hi): last r with ppos[r] <= k
__device__ inline int64_t piece_row(const int32_t* __restrict__ ppos, int64_t lo, int64_t hi,
                                    int64_t k) {
    int64_t a = lo, b = hi - 1;
    while (a < b) {
        const int64_t m = (a + b + 1) >> 1;
        if (ppos[m] <= k) a = m; else b = m - 1;
    }
    return a;
}

// pieces [pbeg, pbeg + gridDim.x) of the long rows [lo, hi); FINAL: only
// neighbours j < clo count
template <int Q, int DT, int FINAL>
__global__ void __launch_bounds__(256) k_vjp_pieces(
    const int32_t* __restrict__ rp, const int32_t* __restrict__ col, const float* __restrict__ w,
    const float* __restrict__ H, int32_t K, const int32_t* __restrict__ ppos, int64_t lo,
    int64_t hi, int64_t pbeg, int64_t clo, float* __restrict__ part) {
    constexpr int P = 256 / Q;
    constexpr int NW = 256 / kWave;
    constexpr int E = Chunk<DT>::E;
    __shared__ float red[NW * Q * E];
    const int tid = threadIdx.x;
    const int p = tid / Q, q = tid % Q;
    const int64_t k = pbeg + blockIdx.x;
    const int64_t r = piece_row(ppos, lo, hi, k);
    const int32_t e0 = rp[r] + (int32_t)(k - ppos[r]) * kPiece;
    const int32_t e1 = min(e0 + kPiece, rp[r + 1]);
    float acc[E];
#pragma unroll
    for (int i = 0; i < E; ++i) acc[i] = 0.0f;
    for (int32_t e = e0 + p; e < e1; e += P) {
        const int32_t j = col[e];
        if (FINAL && j >= clo) continue;
        float hj[E];
        load_f32<E>(H, j, K, q, hj);
        const float wt = w[e];
#pragma unroll
        for (int i = 0; i < E; ++i) acc[i] = __fmaf_rn(wt, hj[i], acc[i]);
    }
#pragma unroll
    for (int off = Q; off < kWave; off <<= 1)
#pragma unroll
        for (int i = 0; i < E; ++i) acc[i] += __shfl_xor(acc[i], off, kWave);
    if ((tid & (kWave - 1)) < Q)
#pragma unroll
        for (int i = 0; i < E; ++i) red[(tid / kWave) * Q * E + q * E + i] = acc[i];
    __syncthreads();
    if (tid < Q) {
#pragma unroll
        for (int i = 0; i < E; ++i) acc[i] = red[q * E + i];
#pragma unroll
        for (int ww = 1; ww < NW; ++ww)
#pragma unroll
            for (int i = 0; i < E; ++i) acc[i] += red[ww * Q * E + q * E + i];
        store_f32<E>(part, k, K, q, acc);
    }
}

// a workgroup per piece: h_i of its row from the row's pieces in order (plus
// G_i in the last sweep) over d_i, stored into H by the row's first piece;
// then every entry of the piece, Q lanes each, adds h_i . (x_j - x_i) to its
// gradient
template <int Q, int DT>
__global__ void __launch_bounds__(256) k_vjp_long_apply(
    const int32_t* __restrict__ rp, const int32_t* __restrict__ col, const void* __restrict__ Xs,
    const void* __restrict__ Xp, int32_t K, int64_t clo, const int32_t* __restrict__ ppos,
    int64_t lo, int64_t hi, int64_t pbeg, const float* __restrict__ dw,
    const float* __restrict__ G, const float* __restrict__ part, float* __restrict__ H,
    float* __restrict__ ge, int first) {
    constexpr int P = 256 / Q;
    constexpr int E = Chunk<DT>::E;
    const int tid = threadIdx.x;
    const int p = tid / Q, q = tid % Q;
    const int64_t k = pbeg + blockIdx.x;
    const int64_t r = piece_row(ppos, lo, hi, k);
    const int32_t k0 = ppos[r], k1 = ppos[r + 1];
    float h[E];
#pragma unroll
    for (int i = 0; i < E; ++i) h[i] = 0.0f;
    for (int32_t kk = k0; kk < k1; ++kk) {
        float v[E];
        load_f32<E>(part, kk, K, q, v);
#pragma unroll
        for (int i = 0; i < E; ++i) h[i] += v[i];
    }
    if (G) {
        float gi[E];
        load_f32<E>(G, r, K, q, gi);
#pragma unroll
        for (int i = 0; i < E; ++i) h[i] += gi[i];
    }
    const float d = dw[r];
#pragma unroll
    for (int i = 0; i < E; ++i) h[i] = h[i] / d;
    if (k == k0 && p == 0) store_f32<E>(H, r, K, q, h);
    float xi[E];
    Chunk<DT>::load(Xs, r, K, q, xi);
    const int32_t e0 = rp[r] + (int32_t)(k - k0) * kPiece;
    const int32_t e1 = min(e0 + kPiece, rp[r + 1]);
#pragma unroll
    for (int t = 0; t < kPiece / P; ++t) {
        const int32_t e = e0 + p + t * P;
        const bool ok = e < e1;
        const int32_t j = ok ? col[e] : (int32_t)r;
        float xj[E];
        Chunk<DT>::load(j < clo ? Xs : Xp, j, K, q, xj);
        float s = 0.0f;
#pragma unroll
        for (int i = 0; i < E; ++i) s = __fmaf_rn(h[i], xj[i] - xi[i], s);
        s = qsum<Q>(s);
        if (ok && q == 0) ge[e] = first ? s : ge[e] + s;
    }
}

// after the last reverse step: gX0_i of the long rows [lo, hi) from their
// pieces in order, a thread per (row, chunk)
template <int Q, int DT>
__global__ void k_vjp_long_final(const int32_t* __restrict__ ppos, const float* __restrict__ part,
                                 int32_t K, int64_t lo, int64_t hi, float* __restrict__ out) {
    constexpr int E = Chunk<DT>::E;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t r = lo + t / Q;
    const int q = (int)(t % Q);
    if (r >= hi) return;
    float g[E];
#pragma unroll
    for (int i = 0; i < E; ++i) g[i] = 0.0f;
    for (int32_t k = ppos[r]; k < ppos[r + 1]; ++k) {
        float v[E];
        load_f32<E>(part, k, K, q, v);
#pragma unroll
        for (int i = 0; i < E; ++i) g[i] += v[i];
    }
    store_f32<E>(out, r, K, q, g);
}

// gw_e = the gradient of e's upper entry (row = the smaller endpoint) plus
// that of the lower one: the lower entries' gradients go to gw (upper = 0),
// then the upper entries, whose ids ascend, add theirs in front.  The rows
// are walked in the caller's order, G lanes each; relabelled row iperm[v]
// holds row v's entries in the same order.  (Listing both relabelled
// entries of every edge first and gathering through the list took 1.2 ms on
// the 434,000-node power-law graph, this takes 0.68 ms.)
__global__ void k_edge_grad(const int32_t* __restrict__ rp, const int32_t* __restrict__ col,
                            const int32_t* __restrict__ eoe, const int32_t* __restrict__ iperm,
                            const int32_t* __restrict__ nrp, const float* __restrict__ ge,
                            int64_t n, int64_t E, int G, int upper, float* __restrict__ gw) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t v = t / G;
    if (v >= n) return;
    const int32_t e0 = rp[v], e1 = rp[v + 1];
    const int64_t o = (int64_t)nrp[iperm[v]] - e0;
    for (int32_t e = e0 + (int32_t)(t % G); e < e1; e += G) {
        if ((col[e] > v) != (upper != 0)) continue;
        const int32_t k = eoe[e];
        if (k < 0 || k >= E) g_bad_edge_id = 1;
        else gw[k] = upper ? ge[o + e] + gw[k] : ge[o + e];
    }
}

__global__ void k_zero_f32(float* p, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0.0f;
}

// entry slots per row (a power of two, about a quarter of the mean degree):
// each lane then has a few gathers to overlap and a wave holds more rows
// (on the 256^3 grid, mean degree 6: one slot per row 34.0 ms, 2 slots
// 33.7, 4 slots 40.4, 8 slots 47.8 per backward call)
static int pick_p_vjp(int Q, double mean_deg) {
    int P = 1;
    while (P * 4 <= mean_deg && Q * P * 2 <= kWave) P *= 2;
    return P;
}

// What the launches of one colour need, fixed for the whole call.
struct VjpPlan {
    const OrderedGraph* og;
    const float* dw;
    const int32_t* ppos;
    std::vector<int64_t> pbeg, pend;  // the pieces of each colour's long rows
    std::vector<int> P;               // lanes per row (x Q) for its short rows
    float* part;
};

template <int Q, int DT, int FINAL>
static int vjp_colour(const VjpPlan& pl, int c, const void* Xs, const void* Xp, int K,
                      const float* G, float* H, float* ge, float* out, hipStream_t st) {
    const OrderedGraph* og = pl.og;
    const gr_graph* g = &og->g;
    const int64_t clo = og->class_ptr_h[c], chi = og->class_ptr_h[c + 1];
    const int64_t mid = og->long_end_h[c];
    if (mid > clo && pl.pend[c] > pl.pbeg[c]) {
        hipLaunchKernelGGL((k_vjp_pieces<Q, DT, FINAL>), dim3((unsigned)(pl.pend[c] - pl.pbeg[c])),
                           dim3(256), 0, st, g->row_ptr, g->col, g->w, (const float*)H, K, pl.ppos,
                           clo, mid, pl.pbeg[c], clo, pl.part);
        GR_LAUNCHED("vjp pieces");
        if constexpr (FINAL) {
            hipLaunchKernelGGL((k_vjp_long_final<Q, DT>), dim3(blocks_for((mid - clo) * Q, 256)),
                               dim3(256), 0, st, pl.ppos, (const float*)pl.part, K, clo, mid, out);
            GR_LAUNCHED("vjp long final");
        } else {
            hipLaunchKernelGGL((k_vjp_long_apply<Q, DT>), dim3((unsigned)(pl.pend[c] - pl.pbeg[c])),
                               dim3(256), 0, st, g->row_ptr, g->col, Xs, Xp, K, clo, pl.ppos, clo,
                               mid, pl.pbeg[c], pl.dw, G, (const float*)pl.part, H, ge, G ? 1 : 0);
            GR_LAUNCHED("vjp long apply");
        }
    }
    if (chi <= mid) return GR_OK;
    const int64_t waves = ((chi - mid) * Q * pl.P[c] + kWave - 1) / kWave;
    dim3 grid(blocks_for(waves * kWave, 256));
#define GR_VR(PP)                                                                                   \
    case PP:                                                                                       \
        if constexpr (Q * PP <= kWave)                                                             \
            hipLaunchKernelGGL((k_vjp_rows<Q, PP, DT, FINAL>), grid, dim3(256), 0, st, g->row_ptr,  \
                               g->col, g->w, Xs, Xp, K, clo, mid, chi, pl.dw, G, H, ge, G ? 1 : 0, out);  \
        break;
    switch (pl.P[c]) {
        GR_VR(1) GR_VR(2) GR_VR(4) GR_VR(8) GR_VR(16) GR_VR(32) GR_VR(64)
        default: return set_error(GR_EINVAL, "bad lane split");
    }
#undef GR_VR
    GR_LAUNCHED("vjp rows");
    return GR_OK;
}

size_t vjp_workspace(int64_t n, int64_t nnz, int32_t K, int32_t dtype, int32_t S, int32_t store) {
    const size_t N = (size_t)n + 1, M = (size_t)nnz + 1;
    const size_t xb = N * (size_t)K * (dtype == GR_BF16 ? 2 : 4) + 256;
    const size_t fb = N * (size_t)K * 4 + 256;
    const size_t pieces = M / kPiece + M / kLongRow + 1;
    size_t b = 4 * N * 4 + 8 * M          // relabelled graph
               + 4 * M                    // per-entry gradients
               + (size_t)(store ? S + 1 : 3) * xb + 3 * fb  // states, G, H, gX0
               + 12 * N                   // weighted degrees, piece offsets and counts
               + pieces * (size_t)K * 4   // piece sums
               + 48 * M + 64 * N;         // sort / relabel temporaries
    return b + b / 16 + (16u << 20);
}

// The sweep-boundary states X_{s-1} and X_s for s = S .. 1.  With all of
// them stored they are there.  Otherwise slot 0 keeps X_0, two slots hold
// the states in use, and `spare` slots (room that the pass needs only at its
// end) keep states on the way: a run of sweeps from state a to state b
// leaves one half-way for each spare slot that is free, so that the next
// states are rebuilt from there and not from X_0.  Sweeps for S = 5: 7 with
// one spare slot, 6 with two, where rebuilding every pair from X_0 takes 15
// (434,000-node power law, float32: 12.4 of the backward's 24.3 ms).
template <int DT>
struct VjpStates {
    const OrderedGraph* og;
    int K;
    std::vector<char*> slot;  // store: S + 1 of them; else X_0, two, spares
    std::vector<int> holds;   // the state in each slot, -1 for none
    Arena& ws;
    hipStream_t st;

    int find(int s) const {
        for (size_t i = 0; i < slot.size(); ++i)
            if (holds[i] == s) return (int)i;
        return -1;
    }
    // `sweeps` sweeps on from slot `from`, into slot `to` (the same one or not)
    int sweep(int from, int to, int sweeps) {
        GR_TRY(smooth_ordered(og, K, sweeps, DT, slot[to], ws, st, from == to ? nullptr : slot[from]));
        holds[to] = holds[from] + sweeps;
        return GR_OK;
    }
    // state s into a slot other than `keep`, from the nearest earlier one
    int build(int s, int keep, int* at) {
        if ((*at = find(s)) >= 0) return GR_OK;
        int from = 0;
        for (size_t i = 0; i < slot.size(); ++i)
            if (holds[i] >= 0 && holds[i] < s && holds[i] > holds[from]) from = (int)i;
        const int to = keep == 1 ? 2 : 1;  // of the two slots in use
        for (size_t i = 3; i < slot.size() && holds[from] + 1 < s; ++i) {
            const bool free = holds[i] < 0 || holds[i] > s;
            if (!free || (int)i == keep) continue;
            const int left = (int)(slot.size() - i);  // spare slots from here on
            GR_TRY(sweep(from, (int)i, (s - holds[from] + left) / (left + 1)));
            from = (int)i;
        }
        GR_TRY(sweep(from, to, s - holds[from]));
        *at = to;
        return GR_OK;
    }
    // X_{s-1} and X_s
    int pair(int s, const void** Xp, const void** Xs) {
        int p = -1, q = find(s);
        if (q < 0) {  // the first pair: X_s is one sweep from X_{s-1}
            GR_TRY(build(s - 1, -1, &p));
            q = p == 1 ? 2 : 1;
            GR_TRY(sweep(p, q, 1));
        } else {
            GR_TRY(build(s - 1, q, &p));
        }
        *Xp = slot[p];
        *Xs = slot[q];
        return GR_OK;
    }
};

template <int Q, int DT>
static int vjp_impl(const VjpPlan& pl, int K, int S, int store, void* states, size_t xstride,
                    const float* Gp, float* H, float* ge, float* gx, Arena& ws, hipStream_t st) {
    const OrderedGraph* og = pl.og;
    const int C = og->n_colours;
    const size_t xbytes = (size_t)og->g.n * K * (DT == GR_BF16 ? 2 : 4);
    VjpStates<DT> X{og, K, {}, {}, ws, st};
    for (int s = 0; s < (store ? S + 1 : 3); ++s) X.slot.push_back((char*)states + (size_t)s * xstride);
    if (!store)  // gx, float32, is written after the last reverse step
        for (int s = 0; s < (DT == GR_BF16 ? 2 : 1); ++s) X.slot.push_back((char*)gx + s * xbytes);
    X.holds.assign(X.slot.size(), -1);
    X.holds[0] = 0;
    if (store)
        for (int s = 1; s <= S; ++s) GR_TRY(X.sweep(s - 1, s, 1));
    for (int s = S; s >= 1; --s) {
        const void *Xs, *Xp;
        GR_TRY(X.pair(s, &Xp, &Xs));
        const float* G = s == S ? Gp : nullptr;
        for (int c = C - 1; c >= 0; --c)
            GR_TRY((vjp_colour<Q, DT, 0>(pl, c, Xs, Xp, K, G, H, ge, nullptr, st)));
    }
    if (S >= 1)
        for (int c = 0; c < C; ++c)
            GR_TRY((vjp_colour<Q, DT, 1>(pl, c, nullptr, nullptr, K, Gp, H, nullptr, gx, st)));
    return GR_OK;
}

int smooth_vjp(const gr_graph* g, const int32_t* eoe, int64_t E, const int32_t* colours, int32_t C,
               int32_t K, int32_t S, int32_t dtype, const void* X0, const float* Gc, float* gw,
               float* gX0, int32_t store, Arena& ws, hipStream_t st) {
    const int64_t n = g->n, nnz = g->nnz;
    OrderedGraph og;
    GR_TRY(order_by_colour(g, colours, C, true, &og, ws, st));
    // weighted degrees, long-row pieces
    const int G = lanes_per_row(n, nnz);
    float* dw = ws.take<float>(n + 1);
    int32_t* ppos = ws.take<int32_t>(n + 1);
    int32_t* pbounds = ws.take<int32_t>(2 * (size_t)C + 1);
    int64_t* pidx = ws.take<int64_t>(2 * (size_t)C + 1);
    if (ws.overflow) return set_error(GR_ENOMEM, "workspace too small (vjp)");
    hipLaunchKernelGGL(k_row_weight, dim3(blocks_for(n * G, 256)), dim3(256), 0, st, og.g.row_ptr,
                       og.g.w, n, G, dw);
    GR_LAUNCHED("row weights");
    {
        size_t mark = ws.used;
        int32_t* cnt = ws.take<int32_t>(n);
        if (ws.overflow) return set_error(GR_ENOMEM, "workspace too small (vjp pieces)");
        hipLaunchKernelGGL(k_piece_counts, dim3(blocks_for(n, 256)), dim3(256), 0, st, og.g.row_ptr,
                           n, cnt);
        GR_LAUNCHED("piece counts");
        GR_TRY(scan_exclusive_i32(cnt, ppos, n, ppos + n, ws, st));
        ws.used = mark;
    }
    // piece ranges of every colour's long rows [class start, long end), and the total
    std::vector<int64_t> hidx(2 * (size_t)C + 1);
    for (int c = 0; c < C; ++c) {
        hidx[2 * c] = og.class_ptr_h[c];
        hidx[2 * c + 1] = og.long_end_h[c];
    }
    hidx[2 * C] = n;
    std::vector<int32_t> hpb(2 * (size_t)C + 1);
    GR_HIP(hipMemcpyAsync(pidx, hidx.data(), sizeof(int64_t) * hidx.size(), hipMemcpyHostToDevice, st));
    hipLaunchKernelGGL(k_gather_i32, dim3(blocks_for(2 * C + 1, 256)), dim3(256), 0, st,
                       (const int32_t*)ppos, (const int64_t*)pidx, (int64_t)(2 * C + 1), pbounds);
    GR_LAUNCHED("piece bounds");
    GR_TRY(fetch({{pbounds, sizeof(int32_t) * hpb.size()}}, hpb.data(), st));
    const int64_t n_pieces = hpb[2 * C];
    VjpPlan pl;
    pl.og = &og;
    pl.dw = dw;
    pl.ppos = ppos;
    pl.pbeg.resize(C);
    pl.pend.resize(C);
    pl.P.resize(C);
    const int Q = K * (dtype == GR_BF16 ? 2 : 4) / 16;
    for (int c = 0; c < C; ++c) {
        pl.pbeg[c] = hpb[2 * c];
        pl.pend[c] = hpb[2 * c + 1];
        const int64_t rows = og.class_ptr_h[c + 1] - og.long_end_h[c];
        const int64_t nz = og.class_nnz_h[c] - og.long_nnz_h[c];
        pl.P[c] = pick_p_vjp(Q, rows > 0 ? (double)nz / (double)rows : 1.0);
    }
    pl.part = ws.take<float>((size_t)(n_pieces + 1) * K);
    // states, cotangent, H, gX0 (relabelled), per-entry gradients
    const size_t xbytes = (size_t)n * K * (dtype == GR_BF16 ? 2 : 4);
    const size_t xstride = (xbytes + 255) & ~size_t(255);
    void* states = ws.take<char>((size_t)(store ? S + 1 : 3) * xstride);
    float* Gp = ws.take<float>((size_t)n * K + 4);
    float* H = ws.take<float>((size_t)n * K + 4);
    float* gx = ws.take<float>((size_t)n * K + 4);
    float* ge = ws.take<float>(nnz + 1);
    if (ws.overflow) return set_error(GR_ENOMEM, "workspace too small (vjp states)");
    GR_TRY(permute_rows(X0, states, og.perm, n, (size_t)K * (dtype == GR_BF16 ? 2 : 4), 0, st));
    GR_TRY(permute_rows(Gc, Gp, og.perm, n, (size_t)K * 4, 0, st));
    hipLaunchKernelGGL(k_zero_f32, dim3(blocks_for(n * K, 256)), dim3(256), 0, st, H, (int64_t)n * K);
    GR_LAUNCHED("zero");
    if (S == 0) {  // no sweep stores the entries' gradients
        hipLaunchKernelGGL(k_zero_f32, dim3(blocks_for(nnz + 1, 256)), dim3(256), 0, st, ge, nnz + 1);
        GR_LAUNCHED("zero");
    }
#define GR_VJ(QQ, DD) \
    case QQ: GR_TRY((vjp_impl<QQ, DD>(pl, K, S, store, states, xstride, Gp, H, ge, gx, ws, st))); break;
    if (dtype == GR_BF16) {
        switch (Q) {
            GR_VJ(1, GR_BF16) GR_VJ(2, GR_BF16) GR_VJ(4, GR_BF16) GR_VJ(8, GR_BF16)
            default: return set_error(GR_EUNSUP, "unsupported K");
        }
    } else {
        switch (Q) {
            GR_VJ(1, GR_F32) GR_VJ(2, GR_F32) GR_VJ(4, GR_F32) GR_VJ(8, GR_F32) GR_VJ(16, GR_F32)
            default: return set_error(GR_EUNSUP, "unsupported K");
        }
    }
#undef GR_VJ
    // no sweep: X_S = X0 and the cotangent passes through
    GR_TRY(permute_rows(S >= 1 ? gx : Gp, gX0, og.perm, n, (size_t)K * 4, 1, st));
    if (E > 0) {
        hipLaunchKernelGGL(k_zero_f32, dim3(blocks_for(E, 256)), dim3(256), 0, st, gw, E);
        GR_LAUNCHED("zero");
        GR_TRY(reset_bad_edge_flag(st));
        for (int upper = 0; upper < 2; ++upper) {
            hipLaunchKernelGGL(k_edge_grad, dim3(blocks_for(n * G, 256)), dim3(256), 0, st,
                               g->row_ptr, g->col, eoe, (const int32_t*)og.iperm, og.g.row_ptr,
                               (const float*)ge, n, E, G, upper, gw);
            GR_LAUNCHED("edge grad");
        }
        GR_TRY(check_bad_edge_flag(st));
    }
    GR_HIP(hipStreamSynchronize(st));  // host vectors above end here
    return GR_OK;
}

}  // namespace gr
