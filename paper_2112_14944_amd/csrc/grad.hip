// Gradient of a loss on the all-pairs DPPR with respect to the edge weights.
//
// Chain rule through the walk of Section 3.1 and Definition def:pprdist
// (rows = sources, Q = (1-alpha) P = (1-alpha) D^-1 W, pi_hat = alpha sum Q^j):
//   Gb = D G                       G = dLoss/dpi_d, pi_d = D pi_hat
//   A  = sum_{j<T} (Q^T)^j Gb      adjoint of pi = alpha (I - Q)^-1, truncated
//                                  like the T-push forward
//   dQ[u][v] = <A[u,:], pi_hat[v,:]>
//   g(u->v)  = (1-alpha)/d_u (dQ[u][v] - sum_b P_ub dQ[u][b]) + sum_t G[u][t] pi_hat[u][t]
//   dLoss/dw_{u,v} = g(u->v) + g(v->u)   (one weight shared by both arcs)
// Two ways to A, chosen by adjoint_dense:
//  - the sum over j is the transposed forward result, (sum_{j<T} Q^j)^T =
//    pi_hat^T / alpha, and pi_hat is at hand: A = pi_hat^T D G / alpha is one
//    dense product, whose cost does not depend on T;
//  - T - 1 streaming steps with a dense forcing term (the adjoint gathers over
//    the same neighbours with the same coefficients as the forward push).
#include "dense.hpp"
#include "internal.hpp"

namespace pprviz {

// A = pi_hat^T D G / alpha, row-major n x n, one BT x BT tile per block.
// Blocks go to the XCDs round-robin, so block b takes tile (b % 8) of every
// eighth part of the list: each XCD works through one contiguous part, in
// bands of 8 tile rows, whose operand rows its L2 keeps.
// Bound: the matrix cores (2 n^3 FLOP): 132 TFLOP/s at n = 8192, 84% of the
// FP32 matrix peak.
constexpr int kAdjBand = 8;
// 128-wide tiles from this size on, where they fill the 256 CUs twice over
// (two blocks per CU); below it 64-wide ones, which need twice the operand
// traffic but leave four times the blocks.
constexpr int kAdjWideN = 3000;

template <int BT>
__global__ __launch_bounds__(kDenseThreads, 2) void adjoint_dense_kernel(const float* __restrict__ pi,
                                                                       const float* __restrict__ G,
                                                                       const float* __restrict__ deg, int32_t n,
                                                                       float alpha, float* __restrict__ A) {
    __shared__ DenseLds<BT> L;
    const int nt = (n + BT - 1) / BT;
    const int64_t total = (int64_t)nt * nt;
    const int64_t part = (total + kXcds - 1) / kXcds;
    const int64_t item = (blockIdx.x % kXcds) * part + blockIdx.x / kXcds;
    if (blockIdx.x / kXcds >= part || item >= total) return;  // block-uniform
    const int64_t band = item / ((int64_t)kAdjBand * nt);
    const int rows = (int)min((int64_t)kAdjBand, nt - band * kAdjBand);
    const int64_t in = item - band * kAdjBand * nt;
    const int i0 = (int)(band * kAdjBand + in % rows) * BT, j0 = (int)(in / rows) * BT;
    DenseTile<BT> t;
    // the sums are set aside every BT rows: about as many parts as terms of a part,
    // where a tile's width is chosen, which rounds least (error of the weight
    // gradient for a given pi, n = 1000: 1.9e-7 with parts of 256 rows, 1.65e-7 so;
    // n = 3100 1.8e-7 and 1.7e-7; 1% of the time at n = 8192)
    dense_tile<BT, BT / kDenseK>(pi, n, G, n, deg, 1.0f / alpha, n, i0, j0, L, t);
    dense_each<BT>(t, i0, j0, [&](int i, int j, float v) {
        if (i < n && j < n) A[(int64_t)i * n + j] = v;
    });
}

// One wave per arc: dq[e] = <A[u, :], pi[v, :]>, pi row-major n x n; A
// row-major as well (SLAB = false), or in the slab layout of the streaming
// iterate.
template <bool SLAB>
__global__ __launch_bounds__(256) void arc_dot_kernel(const int32_t* __restrict__ row_of_arc,
                                                      const int32_t* __restrict__ col_idx, int64_t nnz,
                                                      const float* __restrict__ A,
                                                      const float* __restrict__ pi, int32_t n,
                                                      double* __restrict__ dq) {
    const int lane = threadIdx.x & 63;
    const int64_t e = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (e >= nnz) return;
    const int64_t u = row_of_arc[e];
    const int64_t v = col_idx[e];
    const float* p = pi + v * (int64_t)n;
    double s = 0.0;
    for (int t = lane; t < n; t += 64) s = fma((double)A[SLAB ? sidx(u, t, n) : u * n + t], (double)p[t], s);
    s = wave_sum(s);
    if (lane == 0) dq[e] = s;
}

// The same for row-major A, kArcDotArcs consecutive arcs per block: the arcs of
// one row u share A's row through LDS, so that pi's rows are all that is read
// per arc.  Bound: those reads (nnz n 4 bytes, pi mostly from the last-level
// cache): n = 8192, 1.97e5 arcs 1340 us with both rows read per arc, 876 us
// (7.4 TB/s) now.
constexpr int kArcDotArcs = 32;
constexpr int kArcDotMaxN = 16384;  // A's row in 64 KB of LDS

__global__ __launch_bounds__(256) void arc_dot_rows_kernel(const int32_t* __restrict__ row_ptr,
                                                           const int32_t* __restrict__ row_of_arc,
                                                           const int32_t* __restrict__ col_idx, int64_t nnz,
                                                           const float* __restrict__ A,
                                                           const float* __restrict__ pi, int32_t n,
                                                           double* __restrict__ dq) {
    extern __shared__ float arow[];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int64_t e1 = min(nnz, ((int64_t)blockIdx.x + 1) * kArcDotArcs);
    int64_t e = (int64_t)blockIdx.x * kArcDotArcs;
    while (e < e1) {  // block-uniform
        const int u = row_of_arc[e];
        const int64_t end = min(e1, (int64_t)row_ptr[u + 1]);
        __syncthreads();  // the previous row's readers are done
        for (int t = threadIdx.x; t < n; t += 256) arow[t] = A[(int64_t)u * n + t];
        __syncthreads();
        for (int64_t a = e + wave; a < end; a += 4) {
            const float* __restrict__ p = pi + (int64_t)col_idx[a] * n;
            double s = 0.0;
            int t = lane;
            for (; t + 7 * kWave < n; t += 8 * kWave) {
                float x[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) x[j] = p[t + j * kWave];
#pragma unroll
                for (int j = 0; j < 8; ++j) s = fma((double)arow[t + j * kWave], (double)x[j], s);
            }
            for (; t < n; t += kWave) s = fma((double)arow[t], (double)p[t], s);
            s = wave_sum(s);
            if (lane == 0) dq[a] = s;
        }
        e = end;
    }
}

// dd[u] = sum_t G[u][t] pi[u][t]
__global__ __launch_bounds__(256) void row_dot_kernel(const float* __restrict__ G, const float* __restrict__ pi,
                                                      int32_t n, double* __restrict__ dd) {
    const int lane = threadIdx.x & 63;
    const int64_t u = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (u >= n) return;
    double s = 0.0;
    for (int t = lane; t < n; t += 64) s = fma((double)G[u * n + t], (double)pi[u * n + t], s);
    s = wave_sum(s);
    if (lane == 0) dd[u] = s;
}

__global__ void row_of_arc_kernel(const int32_t* __restrict__ row_ptr, int32_t n, int32_t* __restrict__ row_of_arc) {
    const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= n) return;
    for (int e = row_ptr[u]; e < row_ptr[u + 1]; ++e) row_of_arc[e] = (int32_t)u;
}

// g(u->v) per arc; one thread per row.
__global__ void arc_grad_kernel(const int32_t* __restrict__ row_ptr, const float* __restrict__ weight,
                                const float* __restrict__ deg, const double* __restrict__ dq,
                                const double* __restrict__ dd, int32_t n, float alpha, double* __restrict__ g) {
    const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= n) return;
    const int rs = row_ptr[u], re = row_ptr[u + 1];
    if (rs == re) return;
    const double d = deg[u];
    double row = 0.0;
    for (int e = rs; e < re; ++e) row += (weight ? (double)weight[e] : 1.0) / d * dq[e];
    const double f = (1.0 - (double)alpha) / d;
    for (int e = rs; e < re; ++e) g[e] = f * (dq[e] - row) + dd[u];
}

// Edge gradient: the arc's own term plus that of its reverse arc, found by
// binary search in the (sorted) neighbour list of the other endpoint.
__global__ void edge_sum_kernel(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
                                const int32_t* __restrict__ row_of_arc, int64_t nnz, const double* __restrict__ g,
                                float* __restrict__ out) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= nnz) return;
    const int u = row_of_arc[e];
    const int v = col_idx[e];
    int lo = row_ptr[v], hi = row_ptr[v + 1] - 1;
    int rev = -1;
    while (lo <= hi) {
        const int mid = (lo + hi) >> 1;
        const int c = col_idx[mid];
        if (c == u) {
            rev = mid;
            break;
        }
        if (c < u) lo = mid + 1; else hi = mid - 1;
    }
    out[e] = (float)(g[e] + (rev >= 0 ? g[rev] : 0.0));
}

// Whether the adjoint is taken as the dense product: by the time each takes.
// Measured: the product runs at 132 TFLOP/s (n = 8192: 8.4 ms; n = 1000: 32
// us), a streaming step moves nnz n 4-byte values at 11-12 TB/s and takes 6 us
// at least (T - 1 = 99 steps: 53.9 ms for n = 8192 and 1.97e5 arcs, 1.0 ms for
// n = 1000).  For short series of sparse graphs the steps win.
static bool adjoint_dense(int n, int64_t nnz, int T) {
    const double dense = 2.0 * n * n * n / 110e12 + 10e-6;
    const double stream = (double)(T - 1) * (4.0 * nnz * n / 11e12 + 6e-6);
    return dense < stream;
}

static void adjoint_launch(const float* pi, const float* G, const float* deg, int n, float alpha, float* A,
                           hipStream_t s) {
    auto blocks = [&](int bt) {
        const int64_t nt = (n + bt - 1) / bt;
        return dim3((unsigned)((nt * nt + kXcds - 1) / kXcds * kXcds));
    };
    if (n >= kAdjWideN)
        hipLaunchKernelGGL(adjoint_dense_kernel<128>, blocks(128), dim3(kDenseThreads), 0, s, pi, G, deg, n, alpha, A);
    else
        hipLaunchKernelGGL(adjoint_dense_kernel<64>, blocks(64), dim3(kDenseThreads), 0, s, pi, G, deg, n, alpha, A);
}

struct BwdWs {
    PprWs f;  // forward recompute (any kernel) plus the streaming buffers of the adjoint
    float* pi;
    double* dq;
    double* dd;
    double* g;
    int32_t* row_of_arc;
};

template <typename Cursor>
static void bwd_layout(Cursor& c, int n, int64_t nnz, bool weighted, bool recompute, BwdWs* w) {
    BwdWs t;
    ppr_ws_layout(c, n, nnz, weighted, n, &t.f, true);
    t.pi = recompute ? c.template take<float>((size_t)n * n) : nullptr;
    t.dq = c.template take<double>((size_t)std::max<int64_t>(nnz, 1));
    t.dd = c.template take<double>(n);
    t.g = c.template take<double>((size_t)std::max<int64_t>(nnz, 1));
    t.row_of_arc = c.template take<int32_t>((size_t)std::max<int64_t>(nnz, 1));
    if (w) *w = t;
}

}  // namespace pprviz

using namespace pprviz;

extern "C" {

size_t ppr_backward_workspace(const ppr_csr* g, int recompute) {
    if (g == nullptr || g->n < 1 || g->nnz < 0) return 0;
    WsSize c;
    bwd_layout(c, g->n, g->nnz, g->weight != nullptr, recompute != 0, nullptr);
    if (recompute) ppr_extra_layout(c, g->n, g->n, false, nullptr);
    return c.used;
}

ppr_status ppr_matrix_backward(const ppr_csr* g, float alpha, int32_t T, const float* ppr,
                               const float* grad_dppr, float* grad_arc, void* ws, size_t ws_bytes,
                               void* stream) {
    ppr_status st = validate_csr(g);
    if (st != PPR_OK) return st;
    if (!(alpha > 0.0f && alpha < 1.0f) || T < 0 || grad_dppr == nullptr || (g->nnz > 0 && grad_arc == nullptr))
        return PPR_EINVAL;
    if ((int64_t)g->n * g->n > ((int64_t)1 << 36) || g->n > kStreamMaxN) return PPR_EUNSUPPORTED;
    const bool recompute = (ppr == nullptr);
    WsCursor cur{static_cast<char*>(ws), ws_bytes};
    BwdWs w;
    bwd_layout(cur, g->n, g->nnz, g->weight != nullptr, recompute, &w);
    if (ws == nullptr || cur.used > ws_bytes) return PPR_EWORKSPACE;
    // the recomputed forward takes the route ppr_matrix takes with the
    // workspace of ppr_matrix_workspace_fast, so that it gives the same bits
    if (recompute) ppr_extra_take(cur, g->n, g->n, false, &w.f);
    if (pending_error() != PPR_OK) return PPR_EHIP;
    if (g->nnz == 0) return PPR_OK;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int n = g->n;
    const PprWs& f = w.f;
    launch_degree(g->row_ptr, g->weight, n, f.deg, f.invd, s);
    const float* pi = ppr;
    if (recompute) {
        ppr_forward(g, nullptr, n, nullptr, n, alpha, T, w.pi, nullptr, f.deg, f.invd, nullptr, f, s);
        pi = w.pi;
    }
    hipLaunchKernelGGL(row_of_arc_kernel, dim3((n + 255) / 256), dim3(256), 0, s, g->row_ptr, n, w.row_of_arc);
    const dim3 dots((unsigned)((g->nnz + 3) / 4));
    if (adjoint_dense(n, g->nnz, T)) {
        adjoint_launch(pi, grad_dppr, f.deg, n, alpha, f.ya, s);
        if (n <= kArcDotMaxN)
            hipLaunchKernelGGL(arc_dot_rows_kernel, dim3((unsigned)((g->nnz + kArcDotArcs - 1) / kArcDotArcs)),
                               dim3(256), (size_t)n * sizeof(float), s, g->row_ptr, w.row_of_arc, g->col_idx, g->nnz,
                               f.ya, pi, n, w.dq);
        else
            hipLaunchKernelGGL(arc_dot_kernel<false>, dots, dim3(256), 0, s, w.row_of_arc, g->col_idx, g->nnz, f.ya,
                               pi, n, w.dq);
    } else {
        stream_row_order(g->row_ptr, n, f.hist, f.rows, s);
        StreamArgs sa;
        sa.rows = f.rows;
        sa.row_ptr = g->row_ptr;
        sa.col_idx = g->col_idx;
        sa.weight = g->weight;
        sa.invd = f.invd;
        sa.deg = f.deg;
        sa.n = n;
        sa.nnz = g->nnz;
        sa.ncols = n;
        sa.ld = stream_ld(n);
        sa.alpha = alpha;
        sa.forcing = grad_dppr;
        sa.ld_forcing = n;
        const float* A = stream_adjoint(sa, T, f.ya, f.yb, s);
        hipLaunchKernelGGL(arc_dot_kernel<true>, dots, dim3(256), 0, s, w.row_of_arc, g->col_idx, g->nnz, A, pi, n,
                           w.dq);
    }
    hipLaunchKernelGGL(row_dot_kernel, dim3((n + 3) / 4), dim3(256), 0, s, grad_dppr, pi, n, w.dd);
    hipLaunchKernelGGL(arc_grad_kernel, dim3((n + 255) / 256), dim3(256), 0, s, g->row_ptr, g->weight, f.deg, w.dq,
                       w.dd, n, alpha, w.g);
    hipLaunchKernelGGL(edge_sum_kernel, dim3((unsigned)((g->nnz + 255) / 256)), dim3(256), 0, s, g->row_ptr,
                       g->col_idx, w.row_of_arc, g->nnz, w.g, grad_arc);
    return launch_status();
}

}  // extern "C"
