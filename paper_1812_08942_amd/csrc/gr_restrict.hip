// The reduced data set of the multilevel data visualisation (Alg. 6):
// F_R = H_G^R F, with H_G^R read as the averaging restriction for data, so
// that row I of F_R is the mean of the rows of F over the nodes of aggregate
// I.  The nodes are sorted by aggregate (stable, so members stay in node
// order); every aggregate is cut into pieces of kRPiece members whose FP64
// partial sums are added in order, so hub aggregates spread over many
// threads and the result does not depend on scheduling.
#include "gr_internal.hpp"
#include "gr_device.hpp"

namespace gr {

constexpr int kRT = 256;
constexpr int kRPiece = 256;  // members per piece
constexpr int kRRows = 8;     // rows in flight per thread

// flag bits: 1 = an aggregate id outside [0, n_coarse), 2 = an empty aggregate
__global__ void k_restrict_keys(const int32_t* __restrict__ agg, int64_t n, int64_t nc,
                                uint32_t* __restrict__ key, uint32_t* __restrict__ val,
                                int32_t* bad) {
    const int64_t v = (int64_t)blockIdx.x * kRT + threadIdx.x;
    if (v >= n) return;
    int32_t a = agg[v];
    if (a < 0 || a >= nc) {
        atomicOr(bad, 1);
        a = 0;
    }
    key[v] = (uint32_t)a;
    val[v] = (uint32_t)v;
}

// mstart[c] = the first sorted position whose aggregate is >= c; k over [0, n]
__global__ void k_member_bounds(const uint32_t* __restrict__ skey, int64_t n, int64_t nc,
                                int32_t* __restrict__ mstart) {
    const int64_t k = (int64_t)blockIdx.x * kRT + threadIdx.x;
    if (k > n) return;
    const int64_t lo = k == 0 ? -1 : (int64_t)skey[k - 1];
    const int64_t hi = k == n ? nc : (int64_t)skey[k];
    for (int64_t c = lo + 1; c <= hi; ++c) mstart[c] = (int32_t)k;
}

__global__ void k_restrict_piece_counts(const int32_t* __restrict__ mstart, int64_t nc,
                                        int32_t* __restrict__ cnt, int32_t* bad) {
    const int64_t c = (int64_t)blockIdx.x * kRT + threadIdx.x;
    if (c >= nc) return;
    const int32_t m = mstart[c + 1] - mstart[c];
    if (m == 0) atomicOr(bad, 2);
    cnt[c] = (m + kRPiece - 1) / kRPiece;
}

__global__ void k_restrict_piece_rows(const int32_t* __restrict__ ppos, int64_t nc,
                                      int32_t* __restrict__ prow) {
    const int64_t c = (int64_t)blockIdx.x * kRT + threadIdx.x;
    if (c >= nc) return;
    for (int32_t k = ppos[c]; k < ppos[c + 1]; ++k) prow[k] = (int32_t)c;
}

// V neighbouring columns of a row
template <int V, class T>
struct alignas(V * sizeof(T)) RCols {
    T x[V];
};

// A thread per (piece, V columns): the FP64 sums of the piece's members in
// order.  Bound by one read of F.  An aggregate of one piece is finished here
// (FR: the mean), so that only the others pass through `part`: writing every
// piece's sums and reading them back took a second launch and, at 70,000 x
// 784 and 4,375 aggregates, 55 of 290 MB (52 + 13 -> 43 + 5 us, 5.4 TB/s).
// V = 2 where d and the arrays allow 8-byte loads, kRRows rows in flight: 4
// or 8 rows take 50 or 46 us at V = 1, 55 or 43 at V = 2, 66 or 46 at V = 4
// (wider loads leave fewer threads to hide the members' latency).
template <int V, class T>
__global__ void k_restrict_pieces(const uint32_t* __restrict__ members,
                                  const int32_t* __restrict__ mstart,
                                  const int32_t* __restrict__ ppos,
                                  const int32_t* __restrict__ prow, int64_t npieces, int32_t d,
                                  const T* __restrict__ F, double* __restrict__ part,
                                  float* __restrict__ FR) {
    const int64_t t = (int64_t)blockIdx.x * kRT + threadIdx.x;
    const int32_t dv = d / V;
    int64_t k;
    if (npieces * dv <= 0xffffffffll) k = (int64_t)((uint32_t)t / (uint32_t)dv);
    else k = t / dv;
    if (k >= npieces) return;
    const int32_t col = (int32_t)(t - k * dv) * V;
    const int32_t c = prow[k];
    const int32_t first = mstart[c], end = mstart[c + 1];
    const int32_t m0 = first + (int32_t)(k - ppos[c]) * kRPiece;
    const int32_t m1 = min(m0 + kRPiece, end);
    auto cols = [&](int32_t m) {
        return *reinterpret_cast<const RCols<V, T>*>(F + (int64_t)members[m] * d + col);
    };
    double s[V];
#pragma unroll
    for (int v = 0; v < V; ++v) s[v] = 0.0;
    int32_t m = m0;
    for (; m + kRRows <= m1; m += kRRows) {  // added in member order
        RCols<V, T> r[kRRows];
#pragma unroll
        for (int u = 0; u < kRRows; ++u) r[u] = cols(m + u);
#pragma unroll
        for (int u = 0; u < kRRows; ++u)
#pragma unroll
            for (int v = 0; v < V; ++v) s[v] += (double)r[u].x[v];
    }
    for (; m < m1; ++m) {
        const RCols<V, T> r = cols(m);
#pragma unroll
        for (int v = 0; v < V; ++v) s[v] += (double)r.x[v];
    }
    if (FR && end - first <= kRPiece) {
        RCols<V, float> o;
#pragma unroll
        for (int v = 0; v < V; ++v) o.x[v] = (float)(s[v] / (double)(end - first));
        *reinterpret_cast<RCols<V, float>*>(FR + (int64_t)c * d + col) = o;
    } else {
#pragma unroll
        for (int v = 0; v < V; ++v) part[k * d + col + v] = s[v];
    }
}

// a thread per (aggregate, column): its pieces in order, over the member
// count (the mean, float32; aggregates of several pieces only) or not (the
// sum, FP64)
__global__ void k_restrict_final(const int32_t* __restrict__ mstart,
                                 const int32_t* __restrict__ ppos, int64_t nc, int32_t d,
                                 const double* __restrict__ part, float* __restrict__ FR) {
    const int64_t t = (int64_t)blockIdx.x * kRT + threadIdx.x;
    const int64_t c = t / d;
    const int32_t col = (int32_t)(t % d);
    if (c >= nc || ppos[c + 1] - ppos[c] < 2) return;
    double s = 0.0;
    for (int32_t k = ppos[c]; k < ppos[c + 1]; ++k) s += part[(int64_t)k * d + col];
    FR[c * d + col] = (float)(s / (double)(mstart[c + 1] - mstart[c]));
}

__global__ void k_restrict_final_sum(const int32_t* __restrict__ ppos, int64_t nc, int32_t d,
                                     const double* __restrict__ part, double* __restrict__ FR) {
    const int64_t t = (int64_t)blockIdx.x * kRT + threadIdx.x;
    const int64_t c = t / d;
    const int32_t col = (int32_t)(t % d);
    if (c >= nc) return;
    double s = 0.0;
    for (int32_t k = ppos[c]; k < ppos[c + 1]; ++k) s += part[(int64_t)k * d + col];
    FR[c * d + col] = s;
}

size_t restrict_workspace(int64_t n, int64_t nc, int32_t d) {
    const size_t N = (size_t)n + 1, C = (size_t)nc + 1;
    const size_t pieces = N / kRPiece + C;
    size_t b = 24 * N                          // keys and values, twice
               + 16 * C                        // member bounds, piece counts and offsets
               + 4 * pieces                    // piece aggregates
               + 8 * pieces * (size_t)d        // partial sums
               + 4 * N;                        // sort histograms and scans
    return b + b / 8 + (1u << 20);
}

// mean (FR32 != NULL) or FP64 sum (FR64 != NULL) of F's rows per aggregate
template <class T>
static int restrict_rows(const int32_t* agg, int64_t n, int64_t nc, int32_t d, const T* F,
                         float* FR32, double* FR64, Arena& ws, hipStream_t st) {
    const size_t mark = ws.used;
    uint32_t* k0 = ws.take<uint32_t>(n);
    uint32_t* v0 = ws.take<uint32_t>(n);
    uint32_t* k1 = ws.take<uint32_t>(n);
    uint32_t* v1 = ws.take<uint32_t>(n);
    int32_t* mstart = ws.take<int32_t>(nc + 1);
    int32_t* cnt = ws.take<int32_t>(nc);
    int32_t* ppos = ws.take<int32_t>(nc + 1);
    int32_t* bad = ws.take<int32_t>(4);
    if (ws.overflow) return set_error(GR_ENOMEM, "workspace too small (restriction)");
    GR_TRY(fill_i32(bad, 0, 4, st));
    hipLaunchKernelGGL(k_restrict_keys, dim3(blocks_for(n, kRT)), dim3(kRT), 0, st, agg, n, nc, k0, v0,
                       bad);
    GR_LAUNCHED("restrict keys");
    GR_TRY(radix_sort_pairs32(k0, v0, k1, v1, n, bits_for(nc), ws, st));
    hipLaunchKernelGGL(k_member_bounds, dim3(blocks_for(n + 1, kRT)), dim3(kRT), 0, st,
                       (const uint32_t*)k1, n, nc, mstart);
    GR_LAUNCHED("member bounds");
    hipLaunchKernelGGL(k_restrict_piece_counts, dim3(blocks_for(nc, kRT)), dim3(kRT), 0, st,
                       (const int32_t*)mstart, nc, cnt, bad);
    GR_LAUNCHED("piece counts");
    GR_TRY(scan_exclusive_i32(cnt, ppos, nc, ppos + nc, ws, st));
    int32_t hb[2] = {0, 0};
    GR_TRY(fetch({{bad, sizeof(int32_t)}, {ppos + nc, sizeof(int32_t)}}, hb, st));
    if (hb[0] & 1) return set_error(GR_EINVAL, "an aggregate id lies outside [0, %lld)", (long long)nc);
    if (hb[0] & 2) return set_error(GR_EINVAL, "an aggregate has no member");
    const int64_t np = hb[1];
    int32_t* prow = ws.take<int32_t>(np + 1);
    double* part = ws.take<double>((size_t)np * d + 1);
    if (ws.overflow) return set_error(GR_ENOMEM, "workspace too small (restriction pieces)");
    hipLaunchKernelGGL(k_restrict_piece_rows, dim3(blocks_for(nc, kRT)), dim3(kRT), 0, st,
                       (const int32_t*)ppos, nc, prow);
    GR_LAUNCHED("piece rows");
    const bool wide = d % 2 == 0 && (uintptr_t)F % (2 * sizeof(T)) == 0 && (uintptr_t)FR32 % 8 == 0;
    const int V = wide ? 2 : 1;
    hipLaunchKernelGGL((wide ? k_restrict_pieces<2, T> : k_restrict_pieces<1, T>),
                       dim3(blocks_for(np * (d / V), kRT)), dim3(kRT), 0, st, (const uint32_t*)v1,
                       (const int32_t*)mstart, (const int32_t*)ppos, (const int32_t*)prow, np, d, F, part,
                       FR32);
    GR_LAUNCHED("restrict pieces");
    if (FR32) {
        if (np > nc)
            hipLaunchKernelGGL(k_restrict_final, dim3(blocks_for(nc * d, kRT)), dim3(kRT), 0, st,
                               (const int32_t*)mstart, (const int32_t*)ppos, nc, d,
                               (const double*)part, FR32);
    } else {
        hipLaunchKernelGGL(k_restrict_final_sum, dim3(blocks_for(nc * d, kRT)), dim3(kRT), 0, st,
                           (const int32_t*)ppos, nc, d, (const double*)part, FR64);
    }
    GR_LAUNCHED("restrict final");
    ws.used = mark;
    return GR_OK;
}

int restrict_mean(const int32_t* agg, int64_t n, int64_t nc, int32_t d, const float* F, float* FR,
                  Arena& ws, hipStream_t st) {
    return restrict_rows<float>(agg, n, nc, d, F, FR, nullptr, ws, st);
}

// B^{l+1} = P^T B^l P for a diagonal B: the FP64 sum of b over each
// aggregate's members, in node order (in fixed pieces of kRPiece)
int restrict_sum_f64(const int32_t* agg, int64_t n, int64_t nc, const double* b, double* bc,
                     Arena& ws, hipStream_t st) {
    if (n == 0) return GR_OK;
    return restrict_rows<double>(agg, n, nc, 1, b, nullptr, bc, ws, st);
}

}  // namespace gr
