// Multi-source PPR with the iterate in HBM, each push one launch over the
// whole chip: graphs too large for LDS (more than 40831 nodes), and smaller
// ones asked for few sources, whose LDS-resident kernels would occupy a block
// per handful of sources and leave the other CUs idle.
//
// The iterate Y = (1-alpha) X / d is kept node-major in column slabs of W = 32
// sources (16 or 8 when no more are asked for), ping-pong.  A row piece of W
// columns belongs to Q = W / 4 lanes, 16 bytes each; a wave takes 64 / Q rows
// of the degree order side by side, or all of it one row of more than
// kQueryWide arcs, whose 64 / Q lane groups take every (64 / Q)-th 8 arcs and
// add their sums in a fixed tree.  Waves walk the rows with the grid's stride.
//
// Bound: on large graphs the gathers' misses in L2 (10^6 nodes, 3e7 arcs, 64
// sources: 0.87 ms per push, 8.8 TB/s of gathered bytes, of which a quarter hit
// the L2); on small ones a push's latency, which the
// longest row of a lane group sets (8 arcs per half load latency; hence whole
// waves from 65 arcs on).
//
// A query among its own sources (the targets are the source list) needs only
// the block [sources x sources] of the result, and Y is symmetric:
//     Y_{a+b}[S, S] = Y_a[S, S] + (Y_{a+1} - Y_a)[:, S]^T D Y_b[:, S] / (alpha (1-alpha)).
// A push passes from one factor of the product to the other, (Q V)^T D Y = V^T D
// (Q Y), and Q Y_b = Y_{b+1} - E with E the sources' own term (alpha (1-alpha) / d
// at each source), so with a = P = T / 2 + 1
//     Y_T[S, S] = Y_P[S, S] + (Y_P - Y_{P-1})[:, S]^T D (Y_{T-P+1} - E)[:, S] / (alpha (1-alpha)),
// T - P + 1 = P - 1 or P: about T / 2 pushes and one tall product on the matrix
// cores replace T pushes.  The product carries (1-alpha)^(T/2) of the mass (1e-3
// at T = 86).  Without E, an entry of the difference, which holds the rounding of
// two iterates, meets no entry near 1 of the other factor; and X_P is summed anew
// from Y_{P-1} at the sources' rows, so that its rounding to Y's scale does not
// reach the result.  The result is then no further from 64 bits than T pushes
// (block of 250 sources of 12000 nodes, T = 86, norm of the error: 3.0e-8 by the
// LDS kernels and 3.0e-8 so; 4.8e-8 with (Y_{P} - Y_{P-1})^T D Y_{T-P+1} added to
// Y_{P-1}).
#pragma once

#include <type_traits>

#include "dense.hpp"
#include "ppr_dense.hpp"
#include "ppr_mid.hpp"
#include "ppr_stream.hpp"

namespace pprviz {

constexpr int kQueryWide = 64;        // arcs from which on a row takes a whole wave
constexpr int kQueryMaxSrc = 256;     // sources up to which a graph that fits LDS may come here
constexpr int kQueryMinT = 8;         // pushes from which on they may be halved
constexpr int kQueryMaxBlocks = 2048; // blocks of a push: 8 per CU

inline int query_width(int n_src) { return n_src <= 8 ? 8 : (n_src <= 16 ? 16 : kSlab); }
inline int64_t query_ld(int n_src) {
    const int w = query_width(n_src);
    return ((int64_t)n_src + w - 1) / w * w;
}

// Entry (v, col) of the slab layout.
__device__ __forceinline__ int64_t qidx(int64_t v, int64_t col, int64_t n, int W) {
    return ((col / W) * n + v) * W + (col % W);
}

// Sum over the arcs of this lane's row of w_vu Y[u][its 4 columns] (see
// slab_gather, whose passes, order and pipelining this keeps, for Q lanes per
// row).  step: arcs a lane group advances per pass.
template <int Q, bool WEIGHTED>
__device__ __forceinline__ float4 query_gather(__amdgpu_buffer_rsrc_t rin, const int32_t* __restrict__ col_idx,
                                               const float* __restrict__ weight, int rs, int dg, int step, int lane) {
    constexpr int A = 8;          // arcs per pass
    constexpr int LPI = A / Q;    // of which a lane loads this many
    const int q = lane % Q;
    const uint32_t qoff = (uint32_t)q * 16u;
    const int lead = (lane & ~(Q - 1)) * 4;
    int dmax = dg;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) dmax = max(dmax, __shfl_xor(dmax, o, kWave));
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    int cur[LPI], nxt[LPI];
    float wcur[LPI];
    auto arc = [&](int k) { return k < dg ? col_idx[rs + k] : -1; };
    auto wgt = [&](int k) { return WEIGHTED && k < dg ? weight[rs + k] : 0.f; };
#pragma unroll
    for (int i = 0; i < LPI; ++i) {
        cur[i] = arc(q + Q * i);
        nxt[i] = arc(step + q + Q * i);
        wcur[i] = wgt(q + Q * i);
    }
    int k0 = 0;
    auto issue = [&](float4 (&y)[A], float (&wl)[LPI]) {
        int use[LPI];
#pragma unroll
        for (int i = 0; i < LPI; ++i) {
            use[i] = cur[i];
            wl[i] = wcur[i];
            cur[i] = nxt[i];
            nxt[i] = arc(k0 + 2 * step + q + Q * i);
            wcur[i] = wgt(k0 + step + q + Q * i);
        }
        k0 += step;
#pragma unroll
        for (int j = 0; j < A; ++j) {
            const int u = __builtin_amdgcn_ds_bpermute(lead + 4 * (j % Q), use[j / Q]);
            y[j] = slab_load(rin, ((uint32_t)u * (16u * Q)) | qoff);
        }
    };
    auto add = [&](const float4 (&y)[A], const float (&wl)[LPI]) {
#pragma unroll
        for (int j = 0; j < A; ++j) {
            if (WEIGHTED) {
                const float w =
                    __int_as_float(__builtin_amdgcn_ds_bpermute(lead + 4 * (j % Q), __float_as_int(wl[j / Q])));
                f4_fma(acc, w, y[j]);
            } else {
                f4_acc(acc, y[j]);
            }
        }
    };
    float4 ya[A], yb[A];
    float wa[LPI], wb[LPI];
    if (dmax > 0) {
        issue(ya, wa);
        for (;;) {
            const bool more = k0 < dmax;  // wave-uniform
            issue(yb, wb);
            add(ya, wa);
            if (!more) break;
            const bool more2 = k0 < dmax;
            issue(ya, wa);
            add(yb, wb);
            if (!more2) break;
        }
    }
    return acc;
}

// Adds a wave's lane groups of Q lanes, in FP64 like the parts of a split row of
// the mid-size kernel, into every lane.
template <int Q>
__device__ __forceinline__ float4 query_group_sum(const float4& a) {
    double s[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
    for (int o = Q; o < kWave; o <<= 1)
#pragma unroll
        for (int c = 0; c < 4; ++c) s[c] += __shfl_xor(s[c], o, kWave);
    return make_float4((float)s[0], (float)s[1], (float)s[2], (float)s[3]);
}

// One push.  hist: the class ends of the row order (stream_row_order).  FINAL:
// the last push leaves X itself, as no factor follows its sums.
template <int Q, bool WEIGHTED, bool FINAL>
__global__ __launch_bounds__(256) void query_step_kernel(const RowEnt* __restrict__ rows,
                                                         const int32_t* __restrict__ hist,
                                                         const int32_t* __restrict__ col_idx,
                                                         const float* __restrict__ weight,
                                                         const float* __restrict__ invd,
                                                         const int32_t* __restrict__ src, int32_t n, int32_t ncols,
                                                         float alpha, const float* __restrict__ yin,
                                                         float* __restrict__ yout) {
    constexpr int W = 4 * Q;
    constexpr int G = kWave / Q;
    const int lane = threadIdx.x & 63;
    const int q = lane % Q, grp = lane / Q;
    const int slab = blockIdx.y;
    const int64_t slab_off = (int64_t)slab * n * W;
    const __amdgpu_buffer_rsrc_t rin =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(yin + slab_off), 0, (int)((uint32_t)n * (W * 4)),
                                            0x00020000);
    float4* o4 = reinterpret_cast<float4*>(yout + slab_off);
    const int wide = hist[kDegKeys - 2 - kQueryWide];
    const int items = wide + (n - wide + G - 1) / G;
    int sn[4];  // source node of the lane's columns
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int col = slab * W + q * 4 + c;
        sn[c] = col < ncols ? (src ? src[col] : col) : -1;
    }
    const int stride = (int)gridDim.x * 4;
    for (int item = __builtin_amdgcn_readfirstlane((int)blockIdx.x * 4 + (int)(threadIdx.x >> 6)); item < items;
         item += stride) {
        const bool whole = item < wide;  // wave-uniform
        const int ri = whole ? item : wide + (item - wide) * G + grp;
        const bool has = ri < n;
        int rs = 0, dg = 0, v = 0;
        if (has) {
            const RowEnt e = load_row(as_global(rows), ri);
            rs = e.rs;
            dg = e.re - e.rs;
            v = e.v;
        }
        // a whole wave's lane groups start 8 arcs apart and step over each other
        const int skip = whole ? 8 * grp : 0;
        float4 acc = query_gather<Q, WEIGHTED>(rin, col_idx, weight, rs + skip, max(dg - skip, 0), whole ? 8 * G : 8,
                                               lane);
        if (whole) acc = query_group_sum<Q>(acc);
        if (has && dg == 0) acc = slab_load(rin, (uint32_t)v * (16u * Q) | (uint32_t)q * 16u);
        if (has && (!whole || grp == 0)) {
            const float sv = FINAL ? 1.0f : (1.0f - alpha) * invd[v];
            acc.x = (acc.x + (v == sn[0] ? alpha : 0.f)) * sv;
            acc.y = (acc.y + (v == sn[1] ? alpha : 0.f)) * sv;
            acc.z = (acc.z + (v == sn[2] ? alpha : 0.f)) * sv;
            acc.w = (acc.w + (v == sn[3] ? alpha : 0.f)) * sv;
            o4[(int64_t)v * Q + q] = acc;
        }
    }
}

// Y_1 (X_1 when final) at the source rows (the rest is zero).
static __global__ void query_init_kernel(const int32_t* __restrict__ src, const float* __restrict__ invd, int32_t n,
                                         int32_t ncols, float alpha, int W, int final_, float* __restrict__ y) {
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= ncols) return;
    const int v = src ? src[s] : s;
    y[qidx(v, s, n, W)] = final_ ? alpha : alpha * ((1.0f - alpha) * invd[v]);
}

// part[c] = (hi - lo)[:, S]^T D (b - E)[:, S] / (alpha (1-alpha)) over the c-th
// piece of the rows, b = lo or hi; tiles (I, J), I <= J, of 64 x 64 sources.
// The terms are positive, so a chain of FP32 sums rounds the more the longer it
// is: the running sums are set aside in FP64 every kGramChunk rows, whatever the
// length of a piece (few pieces are left when there are many tiles).
// It reads the iterate's columns once per tile and is a small part of a query
// (64 sources, 10^6 nodes: 0.27 ms of 38).
constexpr int kGramChunk = 128;

static __global__ __launch_bounds__(kDenseThreads) void query_gram_kernel(
    const float* __restrict__ lo, const float* __restrict__ hi, int use_hi, const float* __restrict__ deg,
    const float* __restrict__ invd, const int32_t* __restrict__ src, float alpha, int32_t n, int W, int32_t ld,
    int32_t k, int32_t rows, float* __restrict__ part) {
    constexpr int KB = kDenseK;
    constexpr int NP = KB / 4;
    __shared__ DenseLds<64> L;
    int I, J;
    dense_tile_ij(blockIdx.x, (k + 63) / 64, I, J);
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wi = (wave >> 1) * 32, wj = (wave & 1) * 32;
    const int lc = tid & 63, lr = tid >> 6;
    const int half = lane >> 5, l32 = lane & 31;
    const int v0 = (int)min((int64_t)n, (int64_t)blockIdx.y * rows), v1 = (int)min((int64_t)n, (int64_t)v0 + rows);
    const int ci = I * 64 + lc, cj = J * 64 + lc;
    const bool oki = ci < ld, okj = cj < ld;
    const int64_t bi = oki ? qidx(0, ci, n, W) : 0, bj = okj ? qidx(0, cj, n, W) : 0;
    const float* __restrict__ b = use_hi ? hi : lo;
    const float scale = 1.0f / (alpha * (1.0f - alpha));
    // E's one entry in this thread's column of b
    const int sj = cj < k ? src[cj] : -1;
    const float ej = sj >= 0 ? alpha * ((1.0f - alpha) * invd[sj]) : 0.f;
    DenseAcc c;
    double sum[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        c[r] = 0.f;
        sum[r] = 0.0;
    }
    float ra[NP], rb[NP];
    auto fetch = [&](int v) {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int u = v + lr + 4 * p;
            const bool in = u < v1;
            const int64_t o = (int64_t)(in ? u : 0) * W;
            const float d = in ? deg[u] : 0.f;
            ra[p] = in && oki ? hi[bi + o] - lo[bi + o] : 0.f;
            rb[p] = in && okj ? (b[bj + o] - (u == sj ? ej : 0.f)) * (scale * (d > 0.f ? d : 1.0f)) : 0.f;
        }
    };
    fetch(v0);
    static_assert(kGramChunk % KB == 0, "whole steps");
    for (int v = v0; v < v1; v += KB) {
        __syncthreads();
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int row = lr + 4 * p, col = lc ^ (32 * (row & 1));
            L.a[0][row][col] = ra[p];
            L.b[0][row][col] = rb[p];
        }
        __syncthreads();
        fetch(v + KB);
#pragma unroll
        for (int kk = 0; kk < KB; kk += 2)
            c = __builtin_amdgcn_mfma_f32_32x32x2f32(L.a[0][kk + half][(wi ^ (32 * half)) + l32],
                                                     L.b[0][kk + half][(wj ^ (32 * half)) + l32], c, 0, 0, 0);
        if ((v - v0) % kGramChunk == kGramChunk - KB || v + KB >= v1) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                sum[r] += (double)c[r];
                c[r] = 0.f;
            }
        }
    }
    float* out = part + (int64_t)blockIdx.y * k * k;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int i = I * 64 + wi + dense_row(r, lane), j = J * 64 + wj + l32;
        if (i >= k || j >= k) continue;
        out[(int64_t)i * k + j] = (float)sum[r];
        if (I != J) out[(int64_t)j * k + i] = (float)sum[r];
    }
}

// Sum of the product's pieces in FP64: 64 entries per block, wave w takes
// every fourth piece from w on, 8 loads in flight; the waves' sums in order.
static __global__ __launch_bounds__(256) void query_gram_sum_kernel(const float* __restrict__ part, int64_t kk,
                                                                    int32_t pieces, double* __restrict__ prod) {
    __shared__ double red[4][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t e = (int64_t)blockIdx.x * 64 + lane;
    double t = 0.0;
    if (e < kk) {
        int p = w;
        for (; p + 28 < pieces; p += 32) {
            float x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = part[(int64_t)(p + 4 * u) * kk + e];
#pragma unroll
            for (int u = 0; u < 8; ++u) t += (double)x[u];
        }
        for (; p < pieces; p += 4) t += (double)part[(int64_t)p * kk + e];
    }
    red[w][lane] = t;
    __syncthreads();
    if (w == 0 && e < kk) prod[e] = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
}

// Outputs: row i of pi_hat / DPPR over the targets, from X (64 targets x one slab
// through LDS).
static __global__ __launch_bounds__(256) void query_out_kernel(
    const float* __restrict__ x, int32_t n, int W, int32_t ncols, const int32_t* __restrict__ src,
    const int32_t* __restrict__ tgt, int32_t n_tgt, const float* __restrict__ deg,
    const int32_t* __restrict__ refuse, float* __restrict__ ppr_out, float* __restrict__ dppr_out) {
    __shared__ float tile[64][kSlab + 1];
    const int64_t j0 = (int64_t)blockIdx.x * 64;
    const int c0 = blockIdx.y * W;
    const bool none = refuse && *refuse;
    for (int e = threadIdx.x; e < 64 * W; e += 256) {
        const int jj = e / W, c = e % W;
        const int64_t j = j0 + jj;
        tile[jj][c] = none ? __int_as_float(0x7fc00000) : (j < n_tgt ? x[qidx(tgt ? tgt[j] : j, c0 + c, n, W)] : 0.f);
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int64_t j = j0 + lane;
    if (j >= n_tgt) return;
    for (int c = threadIdx.x >> 6; c < W; c += 4) {
        const int i = c0 + c;
        if (i >= ncols) break;
        const float v = tile[lane][c];
        if (ppr_out) ppr_out[(int64_t)i * n_tgt + j] = v;
        if (dppr_out) dppr_out[(int64_t)i * n_tgt + j] = v * deg[src ? src[i] : i];
    }
}

// Outputs of a query among its sources: X_P at each source's row, the push of
// Y_{P-1} over that row by one wave per slab, plus the product; one rounding.
template <int Q, bool WEIGHTED>
__global__ __launch_bounds__(256) void query_block_out_kernel(
    const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx, const float* __restrict__ weight,
    const float* __restrict__ deg, const float* __restrict__ invd, const int32_t* __restrict__ src, int32_t n,
    int32_t k, float alpha, const float* __restrict__ y, const double* __restrict__ prod,
    const int32_t* __restrict__ refuse, float* __restrict__ ppr_out, float* __restrict__ dppr_out) {
    constexpr int W = 4 * Q;
    constexpr int G = kWave / Q;
    const int lane = threadIdx.x & 63;
    const int q = lane % Q, grp = lane / Q;
    const int slab = blockIdx.y;
    const int j = __builtin_amdgcn_readfirstlane((int)blockIdx.x * 4 + (int)(threadIdx.x >> 6));
    if (j >= k) return;
    const __amdgpu_buffer_rsrc_t rin = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(y + (int64_t)slab * n * W), 0, (int)((uint32_t)n * (W * 4)), 0x00020000);
    const int v = src[j];
    const int rs = row_ptr[v], dg = row_ptr[v + 1] - rs;
    const int skip = 8 * grp;
    float4 acc = query_gather<Q, WEIGHTED>(rin, col_idx, weight, rs + skip, max(dg - skip, 0), 8 * G, lane);
    acc = query_group_sum<Q>(acc);
    if (dg == 0) acc = slab_load(rin, (uint32_t)v * (16u * Q) | (uint32_t)q * 16u);
    if (grp != 0) return;
    const double un = dense_unscale(invd[v], alpha);
    const float s[4] = {acc.x, acc.y, acc.z, acc.w};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int i = slab * W + q * 4 + c;
        if (i >= k) continue;
        const int si = src[i];
        double x = (double)s[c] + (si == v ? (double)alpha : 0.0) + prod[(int64_t)i * k + j] * un;
        if (refuse && *refuse) x = (double)__int_as_float(0x7fc00000);
        if (ppr_out) ppr_out[(int64_t)i * k + j] = (float)x;
        if (dppr_out) dppr_out[(int64_t)i * k + j] = (float)(x * (double)deg[si]);
    }
}

// The LDS-resident kernels refuse a graph whose padded arc copy exceeds its
// workspace bound, which takes a row of more than n arcs (repeated
// neighbours): NaN outputs.  Such a graph is refused here as well, whichever
// kernel its sources would have chosen: one block evaluates the same bounds
// from the degrees (res_sort_kernel's groups; mid_split_kernel's parts and
// mid_plan_kernel's slices).  Without such a row, which is the rule, it returns
// after a look at the first rows of the degree order.  Classes from kDegKeys - 1
// arcs on share the first class, whose rows are ranked here as those kernels rank
// them, by degree up to a limit and by id among rows beyond it (kDegKeys - 1 in the
// resident tile, kMidKeys - 1 in the other); deg_sorted (n ints) takes the degrees
// in that order.
static __global__ __launch_bounds__(1024) void query_refuse_kernel(const RowEnt* __restrict__ rows,
                                                                   const int32_t* __restrict__ hist, int32_t n,
                                                                   int64_t nnz, int64_t cap_groups,
                                                                   int32_t* __restrict__ deg_sorted,
                                                                   int32_t* __restrict__ refuse) {
    __shared__ int long_row;
    const int tid = threadIdx.x;
    const bool res = res_cols_for(n) != 0;
    if (tid == 0) long_row = 0;
    __syncthreads();
    const int cap = (res ? kDegKeys : kMidKeys) - 1;
    const int c0 = hist[0];
    for (int i = tid; i < max(c0, 1); i += 1024)
        if (rows[i].re - rows[i].rs > n) long_row = 1;
    __syncthreads();
    if (!long_row) {
        if (tid == 0) *refuse = 0;
        return;
    }
    for (int i = tid; i < n; i += 1024) {
        const int d = rows[i].re - rows[i].rs;
        int at = i;
        if (i < c0) {
            at = 0;
            for (int j = 0; j < c0; ++j) {
                const int o = min(rows[j].re - rows[j].rs, cap), k = min(d, cap);
                at += o > k || (o == k && rows[j].rs < rows[i].rs) ? 1 : 0;
            }
        }
        deg_sorted[at] = d;
    }
    __syncthreads();
    if (tid != 0) return;
    bool over;
    if (res) {
        const int GW = 256 / res_cols_for(n);
        int64_t words = 0;
        for (int g = 0; g < n; g += GW) {
            int64_t dmax = 1;
            for (int p = g; p < min(n, g + GW); ++p) dmax = max(dmax, (int64_t)deg_sorted[p]);
            words += ((dmax + 7) / 8 + 1) / 2 * 16 * GW;
        }
        over = words > res_arc_words(nnz, n);
    } else {
        const int C = mid_cols_for(n);
        int64_t D;
        int H, P;
        mid_split_choose([&](int i) { return (int64_t)deg_sorted[i]; }, n, nnz, C, D, H, P);
        // slices of 64 rows: the parts (full ones, then each row's last), then the rest
        int64_t groups = 0, width = 1;
        int in = 0;
        auto row = [&](int64_t d) {
            width = max(width, d);
            if (++in == 64) {
                groups += (width + 3) / 4;
                width = 1;
                in = 0;
            }
        };
        for (int h = 0; h < H; ++h)
            for (int64_t a = 0; a < deg_sorted[h]; a += D) row(min(D, (int64_t)deg_sorted[h] - a));
        for (int i = H; i < n; ++i) row(deg_sorted[i]);
        if (in > 0) groups += (width + 3) / 4;
        over = groups > cap_groups;
    }
    *refuse = over ? 1 : 0;
}

// Column sums of X over pieces of the rows in FP64 (the residual's first pass).
static __global__ __launch_bounds__(256) void query_colsum_kernel(const float* __restrict__ x, int32_t n, int W,
                                                                  int64_t ld, const int32_t* __restrict__ refuse,
                                                                  double* __restrict__ part) {
    __shared__ double red[256];
    const int c = threadIdx.x % W, g = threadIdx.x / W, ng = 256 / W;
    const int64_t r0 = (int64_t)blockIdx.x * kStreamResidRows;
    const int64_t r1 = min((int64_t)n, r0 + kStreamResidRows);
    const int64_t col = (int64_t)blockIdx.y * W + c;
    double s = 0.0;
    for (int64_t r = r0 + g; r < r1; r += ng) s += (double)x[qidx(r, col, n, W)];
    red[threadIdx.x] = s;
    __syncthreads();
    if (g == 0) {
        double t = 0.0;
        for (int h = 0; h < ng; ++h) t += red[h * W + c];
        if (refuse && *refuse) t = (double)__int_as_float(0x7fc00000);
        part[(int64_t)blockIdx.x * ld + col] = t;
    }
}

// Buffers beyond the row order, degrees and residuals.
struct QueryWs {
    int32_t* hist;
    int32_t* refuse;  // graphs that fit LDS only (query_refuse_kernel), with deg_sorted
    int32_t* deg_sorted;
    float* ya;
    float* yb;
    double* part;  // residual, row pieces x columns
    float* gram;   // product pieces, nullptr: all pushes
    double* prod;  // their sum
    int32_t pieces;
};

// Pieces of the product's rows: about 1024 blocks in all, which the 256 CUs hold at
// once (1088 instead of 952 blocks take half as long again), at least 256 rows each.
inline int query_pieces(int n, int k) {
    const int64_t nt = (k + 63) / 64;
    const int64_t tiles = nt * (nt + 1) / 2;
    const int64_t most = std::max<int64_t>(1, n / 256);
    return (int)std::min(most, std::max<int64_t>(1, 1024 / tiles));
}
inline size_t query_gram_floats(int n, int k) { return (size_t)query_pieces(n, k) * k * k; }

// Whether the product costs less than the pushes it saves, a push at 9 TB/s of
// gathered values (7.2 to 10), the product at 15 TFLOP/s of n k^2 (13 at 64 sources,
// 26 to 30 at 256, 1000 and 4000, 15 to 17 at 2000, whose 528 tiles are two or three
// to a CU).  Measured, n = 200000, all pushes and halved: 8 arcs per node, T = 8, 64
// sources 0.48 and 0.35 ms, 1000 sources 6.3 and 10.5; 24 arcs per node, T = 20, 1000
// sources 36.8 and 26.3 ms, 2000 sources 72 and 85; T = 86, 4000 sources 641 and 432.
inline bool query_halves(int n, int64_t nnz, int n_src, int T) {
    return T >= kQueryMinT &&
           (double)n * n_src / 15e12 < (double)(T - 1 - T / 2) * (double)nnz * 4 / 9e12;
}

// Whether a query on a graph that fits LDS is faster here, by the time of
// either route in microseconds, fitted to both routes' times over 150 to 40000
// nodes, degrees 3 to 50, 1 to 256 sources and 8, 30 and 86 pushes (nine in ten
// within 15 % of the fit).  A push here takes 6 us, 2.3e-6 us per row and column
// held and 2.2e-7 us per arc and column held.  There, the preparation grows with
// nodes and arcs; a push of the resident tile, 16 columns per block in a graph by
// itself, takes 1.1 us, 1.56e-3 us per row and 1.4e-4 us per arc, one of the
// mid-size kernel 3.6 us and 2.6e-5 us per arc (7.9e-5 with 1 column per block).  48
// sources of 20000 nodes, T = 86: 2.97 ms there, 1.25 ms here, 0.71 ms with halved
// pushes; 256 sources of 15000 nodes, T = 86: 1.36 ms there and 1.56 here at 9e4
// arcs, 3.64 and 4.06 at 6e5.
inline bool query_faster(int n, int64_t nnz, int n_src, int T, bool halved) {
    if (n_src > kQueryMaxSrc || n_src >= n) return false;
    const double rows = (double)n, arcs = (double)nnz;
    const double steps = halved ? T / 2 + 1 : T;
    const double here =
        (halved ? 85.0 : 50.0) + steps * (6.0 + (double)query_ld(n_src) * (2.3e-6 * rows + 2.2e-7 * arcs));
    double there;
    if (res_cols_for(n) != 0) {
        there = 44.0 + 0.059 * rows + 2.1e-3 * arcs + T * (1.1 + 1.56e-3 * rows + 1.4e-4 * arcs);
    } else {
        const int C = mid_cols_for(n);
        const int rounds = ((n_src + C - 1) / C + 255) / 256;
        there = 100.0 + 0.025 * rows + 2.6e-3 * arcs + T * rounds * (3.6 + (C == 1 ? 7.9e-5 : 2.6e-5) * arcs);
    }
    return here < there;
}

template <int Q, bool FINAL>
inline void query_step(const ppr_csr* g, const RowEnt* rows, const int32_t* hist, const float* invd,
                       const int32_t* src, int n_src, float alpha, const float* in, float* out, hipStream_t s) {
    constexpr int G = kWave / Q;
    const int64_t upper = std::min<int64_t>(g->n, g->nnz / (kQueryWide + 1)) + (g->n + G - 1) / G;
    const dim3 grid((unsigned)std::min<int64_t>((upper + 3) / 4, kQueryMaxBlocks),
                    (unsigned)(query_ld(n_src) / (4 * Q)));
    if (g->weight)
        hipLaunchKernelGGL((query_step_kernel<Q, true, FINAL>), grid, dim3(256), 0, s, rows, hist, g->col_idx, g->weight,
                           invd, src, g->n, n_src, alpha, in, out);
    else
        hipLaunchKernelGGL((query_step_kernel<Q, false, FINAL>), grid, dim3(256), 0, s, rows, hist, g->col_idx, nullptr,
                           invd, src, g->n, n_src, alpha, in, out);
}

template <int Q>
inline void query_block_out(const ppr_csr* g, const int32_t* src, int n_src, float alpha, const float* y,
                            const float* deg, const float* invd, const QueryWs& w, float* ppr_out, float* dppr_out,
                            hipStream_t s) {
    const dim3 grid((unsigned)((n_src + 3) / 4), (unsigned)(query_ld(n_src) / (4 * Q)));
    if (g->weight)
        hipLaunchKernelGGL((query_block_out_kernel<Q, true>), grid, dim3(256), 0, s, g->row_ptr, g->col_idx, g->weight,
                           deg, invd, src, g->n, n_src, alpha, y, w.prod, w.refuse, ppr_out, dppr_out);
    else
        hipLaunchKernelGGL((query_block_out_kernel<Q, false>), grid, dim3(256), 0, s, g->row_ptr, g->col_idx, nullptr,
                           deg, invd, src, g->n, n_src, alpha, y, w.prod, w.refuse, ppr_out, dppr_out);
}

// T pushes from every source; halved when the targets are the sources and the
// workspace holds the product's pieces (w.gram).
inline void query_forward(const ppr_csr* g, const int32_t* src, int32_t n_src, const int32_t* tgt, int32_t n_tgt,
                          float alpha, int32_t T, float* ppr_out, float* dppr_out, const float* deg,
                          const float* invd, double* resid, RowEnt* rows, const QueryWs& w, hipStream_t s) {
    const int n = g->n;
    const int W = query_width(n_src);
    const int64_t ld = query_ld(n_src);
    stream_row_order(g->row_ptr, n, w.hist, rows, s);
    if (w.refuse)
        hipLaunchKernelGGL(query_refuse_kernel, dim3(1), dim3(1024), 0, s, rows, w.hist, n, g->nnz,
                           mid_stream_groups(n, g->nnz), w.deg_sorted, w.refuse);
    fill<float>(w.ya, 0.0f, (int64_t)n * ld, s);
    float* in = w.ya;
    float* out = w.yb;
    // iterates to reach: X_T, or with P = T / 2 + 1 both Y_{P-1} and Y_P
    const int last = w.gram ? T / 2 + 1 : T;
    if (T >= 1)
        hipLaunchKernelGGL(query_init_kernel, dim3((unsigned)((n_src + 255) / 256)), dim3(256), 0, s, src, invd, n,
                           n_src, alpha, W, last == 1, in);
    auto push = [&](auto final_) {
        constexpr bool F = decltype(final_)::value;
        if (W == 8) query_step<2, F>(g, rows, w.hist, invd, src, n_src, alpha, in, out, s);
        else if (W == 16) query_step<4, F>(g, rows, w.hist, invd, src, n_src, alpha, in, out, s);
        else query_step<8, F>(g, rows, w.hist, invd, src, n_src, alpha, in, out, s);
        std::swap(in, out);
    };
    for (int t = 1; t < last; ++t) {
        if (t == last - 1 && !w.gram) push(std::true_type{});
        else push(std::false_type{});
    }
    if (w.gram) {
        // in = Y_P, out = Y_{P-1}
        const int64_t nt = (n_src + 63) / 64;
        const int rows_per = (n + w.pieces - 1) / w.pieces;
        hipLaunchKernelGGL(query_gram_kernel, dim3((unsigned)(nt * (nt + 1) / 2), (unsigned)w.pieces),
                           dim3(kDenseThreads), 0, s, out, in, T & 1, deg, invd, src, alpha, n, W, (int32_t)ld, n_src,
                           rows_per, w.gram);
        const int64_t kk = (int64_t)n_src * n_src;
        hipLaunchKernelGGL(query_gram_sum_kernel, dim3((unsigned)((kk + 63) / 64)), dim3(256), 0, s, w.gram, kk,
                           w.pieces, w.prod);
        if (W == 8) query_block_out<2>(g, src, n_src, alpha, out, deg, invd, w, ppr_out, dppr_out, s);
        else if (W == 16) query_block_out<4>(g, src, n_src, alpha, out, deg, invd, w, ppr_out, dppr_out, s);
        else query_block_out<8>(g, src, n_src, alpha, out, deg, invd, w, ppr_out, dppr_out, s);
        return;
    }
    if (ppr_out || dppr_out)
        hipLaunchKernelGGL(query_out_kernel, dim3((unsigned)((n_tgt + 63) / 64), (unsigned)(ld / W)), dim3(256), 0, s,
                           in, n, W, n_src, src, tgt, n_tgt, deg, w.refuse, ppr_out, dppr_out);
    if (resid) {
        const int64_t chunks = stream_resid_chunks(n);
        hipLaunchKernelGGL(query_colsum_kernel, dim3((unsigned)chunks, (unsigned)(ld / W)), dim3(256), 0, s, in, n, W,
                           ld, w.refuse, w.part);
        hipLaunchKernelGGL(stream_resid_kernel, dim3((unsigned)((n_src + 255) / 256)), dim3(256), 0, s, w.part,
                           chunks, ld, n_src, resid);
    }
}

}  // namespace pprviz
