// PDist (Eq. eq:pprdist), its backward, and the O(k^2) stress layout kernels
// (Eq. eq:loss; the appendix's stress majorization in Jacobi form).
#include <math.h>

#include "layout_core.hpp"

namespace pprviz {

// Delta from a k x k DPPR block, 64x64 output tiles.  The transposed tile is
// staged through LDS so both reads are coalesced.  z_ij and z_ji are the same
// FP32 sum (addition commutes), so the result is exactly symmetric.
__global__ __launch_bounds__(256) void pdist_kernel(const float* __restrict__ pid, int32_t k, int64_t n_clamp,
                                                    float* __restrict__ delta) {
    const float hi = pdist_hi(n_clamp);
    __shared__ float tt[64][65];
    const int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6;
    const int64_t i0 = (int64_t)blockIdx.y * 64;
    const int64_t j0 = (int64_t)blockIdx.x * 64;
    // tt[jj][ii] = pid[j0+jj][i0+ii]
    for (int jj = w; jj < 64; jj += 4) {
        const int64_t j = j0 + jj, i = i0 + lane;
        tt[jj][lane] = (j < k && i < k) ? pid[j * k + i] : 0.f;
    }
    __syncthreads();
    for (int ii = w; ii < 64; ii += 4) {
        const int64_t i = i0 + ii, j = j0 + lane;
        if (i >= k || j >= k) continue;
        const float z = pid[i * k + j] + tt[lane][ii];
        delta[i * k + j] = (i == j) ? 0.f : pdist_value(z, hi);
    }
}

__global__ __launch_bounds__(256) void pdist_backward_kernel(const float* __restrict__ pid,
                                                             const float* __restrict__ gdelta, int32_t k,
                                                             int64_t n_clamp, float* __restrict__ gpid) {
    const float hi = pdist_hi(n_clamp);
    __shared__ float tt[64][65];
    const int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6;
    const int64_t i0 = (int64_t)blockIdx.y * 64;
    const int64_t j0 = (int64_t)blockIdx.x * 64;
    for (int jj = w; jj < 64; jj += 4) {
        const int64_t j = j0 + jj, i = i0 + lane;
        tt[jj][lane] = (j < k && i < k) ? pid[j * k + i] : 0.f;
    }
    __syncthreads();
    for (int ii = w; ii < 64; ii += 4) {
        const int64_t i = i0 + ii, j = j0 + lane;
        if (i >= k || j >= k) continue;
        const float z = pid[i * k + j] + tt[lane][ii];
        gpid[i * k + j] = (i == j) ? 0.f : gdelta[i * k + j] * pdist_dz(z, hi);
    }
}

// One row sweep; returns the number of stress partials it writes.
template <int MODE>
static int64_t launch_layout(const float* delta, int32_t k, const float* x, float* xout, double* part, float scale,
                             float* gx, float* gd, hipStream_t s) {
    const LayoutSplit p = layout_split(k, MODE == kLayoutStepStress || MODE == kLayoutStress);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)p.blocks), dim3(kSplitThreads), 0, s, delta, k,
                           reinterpret_cast<const float2*>(x), reinterpret_cast<float2*>(xout), part, scale,
                           reinterpret_cast<float2*>(gx), gd, p.sl);
    };
    if (p.units == 4) go(layout_split_kernel<MODE, 4>);
    else if (p.units == 2) go(layout_split_kernel<MODE, 2>);
    else go(layout_split_kernel<MODE, 1>);
    return p.blocks;
}

// Stress partials a workspace holds (one per 16 rows, at least what a sweep
// writes).
static unsigned layout_blocks(int32_t k) {
    return (unsigned)((k + kLayoutRowsPerBlock - 1) / kLayoutRowsPerBlock);
}

// All sweeps of a small layout in one block: 1/Delta stays in registers and the
// positions in LDS, so a sweep is a few hundred instructions and one barrier
// instead of a launch.  Sixteen lanes share a row (columns l, l + 16, ...) and
// each wave holds 4 rows side by side, 64 rows per pass of the block; a row's
// sums take four rotations within its 16 lanes.
// Bound: latency of a sweep's dependent steps.  k = 25, 50 sweeps: 112 us as
// launches, 24 us; k = 180 3.3 us per sweep; beyond 192 nodes one block's arithmetic outlasts a launch.
constexpr int kRunThreads = 1024;
constexpr int kRunPassRows = kRunThreads / 16;
constexpr int kRunMaxPasses = 3;
constexpr int kRunMaxK = kRunPassRows * kRunMaxPasses;

// Sum over the 16 lanes of a DPP row, in every lane.
__device__ __forceinline__ float row_sum16(float v) {
#define PPRVIZ_ROR(N) \
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + N, 0xf, 0xf, true));
    PPRVIZ_ROR(8)
    PPRVIZ_ROR(4)
    PPRVIZ_ROR(2)
    PPRVIZ_ROR(1)
#undef PPRVIZ_ROR
    return v;
}

template <int PASSES>
__global__ __launch_bounds__(kRunThreads) void layout_run_kernel(const float* __restrict__ delta, int32_t k,
                                                               const float2* __restrict__ x0,
                                                               float2* __restrict__ xout, int32_t steps) {
    constexpr int C = PASSES * kRunPassRows / 16;  // columns per lane
    __shared__ float2 xs[2][PASSES * kRunPassRows];
    const int l = threadIdx.x & 15;
    const int row = threadIdx.x >> 4;
    float inv[PASSES][C], sw[PASSES];
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
        const int i = p * kRunPassRows + row;
        float w = 0.f;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int j = c * 16 + l;
            const bool in = i < k && j < k && i != j;
            const float d = in ? delta[(int64_t)i * k + j] : 1.0f;
            inv[p][c] = in ? __builtin_amdgcn_rcpf(d) : 0.f;
            w = fmaf(inv[p][c], inv[p][c], w);
        }
        sw[p] = row_sum16(w);
    }
    for (int i = threadIdx.x; i < PASSES * kRunPassRows; i += kRunThreads) {
        xs[0][i] = i < k ? x0[i] : make_float2(0.f, 0.f);
        xs[1][i] = make_float2(0.f, 0.f);
    }
    __syncthreads();
    for (int s = 0; s < steps; ++s) {
        const float2* in = xs[s & 1];
        float2* out = xs[(s & 1) ^ 1];
        float2 xj[C];
#pragma unroll
        for (int c = 0; c < C; ++c) xj[c] = in[c * 16 + l];
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const int i = p * kRunPassRows + row;
            const float2 xi = in[i];
            float ax = 0.f, ay = 0.f;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const float dx = xi.x - xj[c].x;
                const float dy = xi.y - xj[c].y;
                const float rs = __builtin_amdgcn_rsqf(fmaf(dx, dx, fmaf(dy, dy, kMinSq)));
                const float g = fmaf(inv[p][c], rs, -(inv[p][c] * inv[p][c]));
                ax = fmaf(g, dx, ax);
                ay = fmaf(g, dy, ay);
            }
            ax = row_sum16(ax);
            ay = row_sum16(ay);
            if (l == 0 && i < k)
                out[i] = sw[p] > 0.f ? make_float2(xi.x + ax / sw[p], xi.y + ay / sw[p]) : xi;
        }
        __syncthreads();
    }
    for (int i = threadIdx.x; i < k; i += kRunThreads) xout[i] = xs[steps & 1][i];
}

__global__ void layout_copy_kernel(const float2* __restrict__ a, float2* __restrict__ b, int32_t k) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < k) b[i] = a[i];
}

}  // namespace pprviz

using namespace pprviz;

extern "C" {

ppr_status pdist(const float* dppr, int32_t k, int64_t n_clamp, float* delta, void* stream) {
    if (dppr == nullptr || delta == nullptr || k < 1 || n_clamp < 1 || dppr == delta) return PPR_EINVAL;
    if (pending_error() != PPR_OK) return PPR_EHIP;
    dim3 grid((k + 63) / 64, (k + 63) / 64);
    hipLaunchKernelGGL(pdist_kernel, grid, dim3(256), 0, static_cast<hipStream_t>(stream), dppr, k, n_clamp, delta);
    return launch_status();
}

ppr_status pdist_backward(const float* dppr, const float* grad_delta, int32_t k, int64_t n_clamp,
                          float* grad_dppr, void* stream) {
    if (!dppr || !grad_delta || !grad_dppr || k < 1 || n_clamp < 1) return PPR_EINVAL;
    if (grad_dppr == dppr || grad_dppr == grad_delta) return PPR_EINVAL;
    if (pending_error() != PPR_OK) return PPR_EHIP;
    dim3 grid((k + 63) / 64, (k + 63) / 64);
    hipLaunchKernelGGL(pdist_backward_kernel, grid, dim3(256), 0, static_cast<hipStream_t>(stream), dppr,
                       grad_delta, k, n_clamp, grad_dppr);
    return launch_status();
}

size_t layout_workspace(int32_t k) {
    if (k < 1) return 0;
    return align_up(sizeof(double) * (size_t)layout_blocks(k));
}

ppr_status stress_eval(const float* delta, int32_t k, const float* x, double* stress_out, void* ws,
                       size_t ws_bytes, void* stream) {
    if (!delta || !x || !stress_out || k < 1) return PPR_EINVAL;
    if (ws == nullptr || ws_bytes < layout_workspace(k)) return PPR_EWORKSPACE;
    if (pending_error() != PPR_OK) return PPR_EHIP;
    hipStream_t s = static_cast<hipStream_t>(stream);
    double* part = static_cast<double*>(ws);
    const int64_t m = launch_layout<kLayoutStress>(delta, k, x, nullptr, part, 1.f, nullptr, nullptr, s);
    hipLaunchKernelGGL(sum_partials_kernel, dim3(1), dim3(256), 0, s, part, m, stress_out);
    return launch_status();
}

ppr_status layout_step(const float* delta, int32_t k, const float* x_in, float* x_out, double* stress_out,
                       void* ws, size_t ws_bytes, void* stream) {
    if (!delta || !x_in || !x_out || k < 1 || x_in == x_out) return PPR_EINVAL;
    if (stress_out && (ws == nullptr || ws_bytes < layout_workspace(k))) return PPR_EWORKSPACE;
    if (pending_error() != PPR_OK) return PPR_EHIP;
    hipStream_t s = static_cast<hipStream_t>(stream);
    double* part = static_cast<double*>(ws);
    if (stress_out) {
        const int64_t m = launch_layout<kLayoutStepStress>(delta, k, x_in, x_out, part, 1.f, nullptr, nullptr, s);
        hipLaunchKernelGGL(sum_partials_kernel, dim3(1), dim3(256), 0, s, part, m, stress_out);
    } else {
        launch_layout<kLayoutStep>(delta, k, x_in, x_out, nullptr, 1.f, nullptr, nullptr, s);
    }
    return launch_status();
}

size_t layout_run_workspace(int32_t k) {
    if (k < 1) return 0;
    return align_up(sizeof(float2) * (size_t)k);
}

ppr_status layout_run(const float* delta, int32_t k, const float* x_in, float* x_out, int32_t steps, void* ws,
                      size_t ws_bytes, void* stream) {
    if (!delta || !x_in || !x_out || k < 1 || x_in == x_out || steps < 0) return PPR_EINVAL;
    if (ws == nullptr || ws_bytes < layout_run_workspace(k)) return PPR_EWORKSPACE;
    if (pending_error() != PPR_OK) return PPR_EHIP;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const float2* x = reinterpret_cast<const float2*>(x_in);
    float2* out = reinterpret_cast<float2*>(x_out);
    if (steps == 0) {
        hipLaunchKernelGGL(layout_copy_kernel, dim3((unsigned)((k + 255) / 256)), dim3(256), 0, s, x, out, k);
    } else if (k <= kRunMaxK) {
        const int passes = (k + kRunPassRows - 1) / kRunPassRows;
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(1), dim3(kRunThreads), 0, s, delta, k, x, out, steps);
        };
        if (passes == 1) go(layout_run_kernel<1>);
        else if (passes == 2) go(layout_run_kernel<2>);
        else go(layout_run_kernel<3>);
    } else {
        // ping-pong so that the last sweep lands in x_out
        float* bufs[2] = {x_out, static_cast<float*>(ws)};
        int next = steps % 2 == 1 ? 0 : 1;
        const float* cur = x_in;
        for (int32_t i = 0; i < steps; ++i) {
            launch_layout<kLayoutStep>(delta, k, cur, bufs[next], nullptr, 1.f, nullptr, nullptr, s);
            cur = bufs[next];
            next ^= 1;
        }
    }
    return launch_status();
}

ppr_status stress_backward(const float* delta, int32_t k, const float* x, float grad_scale, float* grad_x,
                           float* grad_delta, void* stream) {
    if (!delta || !x || k < 1 || (!grad_x && !grad_delta)) return PPR_EINVAL;
    if (pending_error() != PPR_OK) return PPR_EHIP;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (grad_delta)
        launch_layout<kLayoutGradBoth>(delta, k, x, nullptr, nullptr, grad_scale, grad_x, grad_delta, s);
    else
        launch_layout<kLayoutGradX>(delta, k, x, nullptr, nullptr, grad_scale, grad_x, nullptr, s);
    return launch_status();
}

}  // extern "C"
