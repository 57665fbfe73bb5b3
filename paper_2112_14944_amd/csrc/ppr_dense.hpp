// All-pairs PPR of a graph of the resident range by a short push series and a
// few dense products.
//
// On an undirected graph Y_t(s, v) = (1-alpha) X_t(s, v) / d(v), the form the
// resident tile keeps the iterate in, is symmetric in s and v (reversibility),
// and with X_T = alpha sum_{t<T} Q^t the series can be cut into pieces:
//     Y_{m+b} = Y_m + (Y_{m+1} - Y_m) D Y_b / (alpha (1-alpha)).
// With V = Y_{m+1} - Y_m and T = k m + r (0 < r < m), T pushes from every
// source are m + 1 pushes, which give Y_r, X_m and V, and then k products
//     W_0 = Y_r,   W_{p+1} = Y_m + V D W_p / (alpha (1-alpha)),   W_k = Y_T.
// V, Y_m and W_p are symmetric, so a product takes only the tiles on and above
// the diagonal and stores each twice: n^3 FLOP on the matrix cores, against
// nnz n additions per push.  The products carry the last (1-alpha)^m of the
// mass (3% of it for m = 22).
//
// V is small against the iterates it is the difference of, and 1 / alpha scales
// it.  So that the result is no further from 64 bits than T pushes, the push
// behind V comes after the difference, each column of V is brought to the mass
// it has to hold (res_tile), and the last product adds to X_m, unscaled and
// without the sources' own alpha, in FP64: one rounding.  Norm of the error of X,
// n = 1000, 24 arcs per node, T = 100: 6.4e-8 by pushes, 8.4e-8 by plain
// differences, 6.6e-8 so.
//
// Measured (MI355X): 512 block-model subgraphs of 32 to 2048 nodes (T = 86),
// PPR stage 43.7 ms by pushes alone, 24.2 ms as 14.2 ms of pushes and 10.0 ms
// of products; one graph of 2048 nodes, all pairs, 2.01 ms against 0.50 ms of
// pushes and three products of 0.13.
//
// A 32x32 block on or above the diagonal is stored as computed, one below it
// is the mirror image of its partner, whatever the tile size: the batch and
// the single-graph path give the same bits.
#pragma once

#include "dense.hpp"
#include "ppr_core.hpp"

namespace pprviz {

constexpr int kDenseMinN = 192;   // below it a product's tiles are mostly padding and latency
constexpr int kDenseMinT = 24;    // the pieces have at least 4 pushes
constexpr int kDenseMaxT = 4096;  // keeps the cost comparison below 2^63
constexpr int kDenseMaxK = 3;     // products
// alpha from which on pushes are replaced by products, here and for few sources
// (ppr_query.hpp): the rounding that the difference of two iterates holds reaches
// the result over alpha.  Error against 64 bits over that of all pushes, T for a
// residual of 1e-6, graphs of 300 to 2048 nodes here: 0.95 to 1.1 at alpha = 0.1
// and above, 0.5 to 1.6 at 0.05, up to 2.6 at 0.01; few sources 0.7 to 1.05 from
// 0.05 on, 1.1 to 1.3 at 0.01.  At 0.5 (few pushes matter, an entry's error is that
// of few roundings, and X_m and the sum are one more than pushes have) 1.14 here, at
// 0.3 1.02.
constexpr float kDenseMinAlpha = 0.1f;
constexpr float kDenseMaxAlpha = 0.4f;  // all pairs
__host__ __device__ inline bool dense_alpha(float alpha) { return alpha >= kDenseMinAlpha && alpha <= kDenseMaxAlpha; }
constexpr int kDenseWideN = 512;  // batch: 128-wide tiles from this size on

struct DensePlan {
    int32_t k;  // products (0: all T pushes)
    int32_t m;  // pushes behind Y_m
    int32_t r;  // pushes behind W_0 = Y_r, 0 < r < m
};

// Number of products: the k with the least time, in hundredths of a push of
// one arc from one source.  Measured in the batch: pushes run at 23e12
// additions/s and products at 89 to 100 TFLOP/s, so n^3 FLOP cost what 0.22 to
// 0.26 n^2 / nnz pushes do (0.22 here); writing the three matrices and the extra
// push behind V cost about three pushes.  Integer arithmetic, so that host and
// device agree.
__host__ __device__ inline DensePlan dense_plan(int n, int64_t nnz, int T) {
    DensePlan best{0, T, 0};
    if (n < kDenseMinN || n > Res<16>::NMAX || T < kDenseMinT || T > kDenseMaxT) return best;
    int64_t cost = 90 * (int64_t)T * nnz;  // a tenth less than T pushes
    for (int k = 1; k <= kDenseMaxK; ++k) {
        const int m = (T + k) / (k + 1);
        const int64_t c = 100 * (int64_t)(m + 4) * nnz + 22 * (int64_t)k * n * (n + 64);
        if (c < cost) {
            cost = c;
            best = DensePlan{k, m, T - k * m};
        }
    }
    if (best.r == best.m) {  // W_0 is an iterate of its own
        best.m += 1;
        best.r -= best.k;
    }
    return best;
}

__host__ __device__ inline int dense_bt(int n) { return n < kDenseWideN ? 64 : 128; }
__host__ __device__ inline int64_t dense_tiles(int n, int bt) {
    const int64_t nt = (n + bt - 1) / bt;
    return nt * (nt + 1) / 2;
}

// Tile t of the upper triangle (row by row) -> (I, J), I <= J.
__device__ __forceinline__ void dense_tile_ij(int64_t t, int nt, int& I, int& J) {
    int i = 0;
    while (t >= nt - i) {
        t -= nt - i;
        ++i;
    }
    I = i;
    J = i + (int)t;
}

// X(s, v) from Y(s, v): over the FP32 scale (1-alpha)/d(v) the resident tile
// multiplied by, in FP64, so that neither the scale's rounding nor the way
// back adds to the result's.
__device__ __forceinline__ double dense_unscale(float invd, float alpha) {
    const float sc = (1.0f - alpha) * invd;
    const double r = (double)__builtin_amdgcn_rcpf(sc);
    const double r1 = r * (2.0 - (double)sc * r);  // two steps from 1 ulp of FP32
    return r1 * (2.0 - (double)sc * r1);
}

// What a product leaves: W_{p+1}, or, the last, X_T or DPPR, d(s) X_T(s, v) with
// X rounded to FP32 first, like ppr_matrix's.
enum DenseOut { kDenseNext, kDensePpr, kDenseDppr };

// One tile of a product (all n x n, row-major, ld = n; xm: X_m without the
// sources' own alpha).
template <int BT, DenseOut OUT>
__device__ __forceinline__ void dense_product_tile(const float* V, const float* xm, const float* W,
                                                   const float* deg, const float* invd, float alpha, int n, int64_t t,
                                                   DenseLds<BT>& L, float* out) {
    int I, J;
    dense_tile_ij(t, (n + BT - 1) / BT, I, J);
    const int i0 = I * BT, j0 = J * BT;
    DenseTile<BT> c;
    dense_tile<BT, 0>(V, n, W, n, deg, 1.0f / (alpha * (1.0f - alpha)), n, i0, j0, L, c);
    dense_each<BT>(c, i0, j0, [&](int i, int j, float v) {
        if (i >= n || j >= n || (i >> 5) > (j >> 5)) return;
        const bool twice = (i >> 5) < (j >> 5);
        const float x = as_global(xm)[(int64_t)i * n + j];
        float a, b;
        if (OUT == kDenseNext) {
            a = b = fmaf(x + (i == j ? alpha : 0.f), (1.0f - alpha) * as_global(invd)[j], v);
        } else {
            const double own = i == j ? (double)alpha : 0.0;
            a = (float)((double)x + own + (double)v * dense_unscale(as_global(invd)[j], alpha));
            b = twice ? (float)((double)as_global(xm)[(int64_t)j * n + i] +
                                (double)v * dense_unscale(as_global(invd)[i], alpha))
                      : 0.f;
            if (OUT == kDenseDppr) {
                a *= as_global(deg)[i];
                b *= as_global(deg)[j];
            }
        }
        as_global_w(out)[(int64_t)i * n + j] = a;
        if (twice) as_global_w(out)[(int64_t)j * n + i] = b;
    });
}

}  // namespace pprviz
