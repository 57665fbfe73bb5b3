// Iterates in HBM in column slabs of 32: the degree row order, the slab gather
// of the Group Forward- and Backward-Push rounds, and the adjoint solve of the
// weight gradient by streaming steps,
//     A_{k+1} = Gb + (1-alpha) P^T A_k      (Gb = D G, forcing term),
// one launch per term.  A wave takes 8 rows side by side, so every gathered
// neighbour row is one contiguous 128-byte read (details at
// stream_step_kernel).
#pragma once

#include "ppr_core.hpp"

namespace pprviz {

inline int64_t stream_ld(int64_t ncols) { return (ncols + 63) / 64 * 64; }
constexpr int kStreamResidRows = 4096;
inline int64_t stream_resid_chunks(int64_t n) { return (n + kStreamResidRows - 1) / kStreamResidRows; }

// Iterate layout: column slabs of 32 columns, each slab stored node-major
// and contiguous (n rows of 128 bytes), slab after slab; ld columns in all
// (ld a multiple of 64), so a buffer holds n * ld floats.
constexpr int kSlab = 32;
constexpr int kSlabVec = kSlab / 4;             // float4 per slab row
constexpr int kArcsPerLoad = kWave / kSlabVec;  // arcs one wave load covers

__host__ __device__ __forceinline__ int64_t sidx(int64_t v, int64_t col, int64_t n) {
    return ((col / kSlab) * n + v) * kSlab + (col % kSlab);
}

struct StreamArgs {
    const RowEnt* rows;   // rows by non-increasing degree (stream_row_order)
    const int32_t* row_ptr;
    const int32_t* col_idx;
    const float* weight;
    const float* invd;
    const float* deg;
    int32_t n;
    int64_t nnz;
    int32_t ncols;        // valid columns (right-hand sides)
    int64_t ld;           // columns held (multiple of 64)
    float alpha;
    const float* forcing; // G [n][ld_forcing] (Gb = deg[v] * G[v][s])
    int64_t ld_forcing;
};

constexpr int kStreamRowsPerWave = kWave / kSlabVec;  // 8 rows side by side
constexpr int kStreamRowsPerBlock = 4 * kStreamRowsPerWave;
constexpr int kXcds = 8;
// A slab of the iterate that fits this budget stays in one XCD's L2 (4 MB)
// next to the arc stream while that XCD sweeps it.
constexpr int64_t kStreamSlabBudget = 3 << 20;
constexpr int kDegKeys = 4096;
// Slab gathers use 32-bit byte offsets: n * 128 must stay below 2^31.
constexpr int32_t kStreamMaxN = 1 << 24;  // degree classes of the row order (exact below 4095)

// Launch shape of one push: `slabs` column slabs, each swept by `row_blocks`
// blocks of 32 rows.
struct StreamGrid {
    int32_t row_blocks;
    int32_t slabs;
    int32_t full_rounds;  // rounds of 8 slabs run one per XCD (0: none)
};

// Block -> (slab, row block).  Workgroups go to the 8 XCDs round-robin by
// linear id, so blocks b, b + 8, b + 16, ... share one XCD.  In each of the
// first full_rounds rounds every XCD sweeps all rows of a slab of its own, so
// the neighbour rows it gathers are served by its own L2.  The remaining
// slabs are taken one after another by all XCDs together (for large n that
// keeps one slab at a time in the shared last-level cache).  The grid has
// exactly slabs * row_blocks blocks and the map is a bijection onto the pairs.
__device__ __forceinline__ void stream_block_map(const StreamGrid& g, int& slab, int& rb) {
    const int b = blockIdx.x;
    const int full_blocks = g.full_rounds * kXcds * g.row_blocks;
    if (b < full_blocks) {
        const int local = b / kXcds;
        slab = (local / g.row_blocks) * kXcds + b % kXcds;
        rb = local % g.row_blocks;
    } else {
        const int local = b - full_blocks;
        slab = g.full_rounds * kXcds + local / g.row_blocks;
        rb = local % g.row_blocks;
    }
}

// Row order by degree, largest first: a counting sort over KEYS degree
// classes (degrees from KEYS - 1 up share the first class), so that the 8
// rows a streaming-step wave takes side by side have (nearly) equal arc
// counts.  The order within a class is whatever the atomics give; it only
// decides which rows share a wave, never a sum.  This histogram with one
// global atomic per row serves the mid-size kernel's 65536 exact classes
// (which do not fit in LDS; it has a stable scatter of its own); the
// streaming row order below counts per block in LDS.
template <int KEYS>
static __global__ void stream_deg_hist_kernel(const int32_t* __restrict__ row_ptr, int32_t n,
                                              int32_t* __restrict__ hist) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    const int d = min(row_ptr[v + 1] - row_ptr[v], KEYS - 1);
    atomicAdd(&hist[KEYS - 1 - d], 1);
}

// Exclusive prefix sum of the KEYS class counts, in place (one block).
template <int KEYS>
static __global__ __launch_bounds__(1024) void stream_deg_scan_kernel(int32_t* __restrict__ hist) {
    constexpr int kPer = KEYS / 1024;
    static_assert(KEYS % 1024 == 0, "keys");
    __shared__ int32_t part[1024];
    const int t0 = threadIdx.x * kPer;
    int32_t t = 0;
    for (int i = 0; i < kPer; ++i) t += hist[t0 + i];
    part[threadIdx.x] = t;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
        const int32_t x = threadIdx.x >= o ? part[threadIdx.x - o] : 0;
        __syncthreads();
        part[threadIdx.x] += x;
        __syncthreads();
    }
    int32_t run = part[threadIdx.x] - t;
    for (int i = 0; i < kPer; ++i) {
        const int32_t h = hist[t0 + i];
        hist[t0 + i] = run;
        run += h;
    }
}

// Streaming row order: the class counts are kept per block in LDS.  A block
// counts its kOrderNodes rows there and adds each nonzero class count to the
// global histogram once, then reserves one range per class with one atomic
// and hands out positions inside it from LDS.  With a few hundred rows per
// degree class in a block, this takes the global atomics on the few classes
// of common degrees down from one per row to one per block and class.
constexpr int kOrderNodes = 2048;

template <int KEYS>
static __global__ __launch_bounds__(1024) void stream_deg_hist_lds_kernel(const int32_t* __restrict__ row_ptr,
                                                                          int32_t n, int32_t* __restrict__ hist) {
    __shared__ int32_t cnt[KEYS];
    for (int i = threadIdx.x; i < KEYS; i += blockDim.x) cnt[i] = 0;
    __syncthreads();
    const int64_t b = (int64_t)blockIdx.x * kOrderNodes;
    const int64_t e = min((int64_t)n, b + kOrderNodes);
    for (int64_t v = b + threadIdx.x; v < e; v += blockDim.x) {
        const int d = min(row_ptr[v + 1] - row_ptr[v], KEYS - 1);
        atomicAdd(&cnt[KEYS - 1 - d], 1);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < KEYS; i += blockDim.x)
        if (cnt[i]) atomicAdd(&hist[i], cnt[i]);
}

template <int KEYS>
static __global__ __launch_bounds__(1024) void stream_deg_scatter_lds_kernel(const int32_t* __restrict__ row_ptr,
                                                                             int32_t n, int32_t* __restrict__ cursor,
                                                                             RowEnt* __restrict__ rows) {
    __shared__ int32_t cnt[KEYS];
    for (int i = threadIdx.x; i < KEYS; i += blockDim.x) cnt[i] = 0;
    __syncthreads();
    const int64_t b = (int64_t)blockIdx.x * kOrderNodes;
    const int64_t e = min((int64_t)n, b + kOrderNodes);
    for (int64_t v = b + threadIdx.x; v < e; v += blockDim.x) {
        const int d = min(row_ptr[v + 1] - row_ptr[v], KEYS - 1);
        atomicAdd(&cnt[KEYS - 1 - d], 1);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < KEYS; i += blockDim.x)
        if (cnt[i]) cnt[i] = atomicAdd(&cursor[i], cnt[i]);
    __syncthreads();
    for (int64_t v = b + threadIdx.x; v < e; v += blockDim.x) {
        const int rs = row_ptr[v], re = row_ptr[v + 1];
        const int d = min(re - rs, KEYS - 1);
        const int pos = atomicAdd(&cnt[KEYS - 1 - d], 1);
        rows[pos] = RowEnt{rs, re, (int32_t)v, 0};
    }
}

template <int KEYS = kDegKeys>
inline void stream_row_order(const int32_t* row_ptr, int32_t n, int32_t* hist, RowEnt* rows, hipStream_t s) {
    static_assert(KEYS * 4 <= 32768, "per-block class counts must fit in LDS");
    fill<int32_t>(hist, 0, KEYS, s);
    const unsigned blocks = (unsigned)((n + kOrderNodes - 1) / kOrderNodes);
    hipLaunchKernelGGL(stream_deg_hist_lds_kernel<KEYS>, dim3(blocks), dim3(1024), 0, s, row_ptr, n, hist);
    hipLaunchKernelGGL(stream_deg_scan_kernel<KEYS>, dim3(1), dim3(1024), 0, s, hist);
    hipLaunchKernelGGL(stream_deg_scatter_lds_kernel<KEYS>, dim3(blocks), dim3(1024), 0, s, row_ptr, n, hist,
                       rows);
}

__device__ __forceinline__ void f4_acc(float4& a, float4 y) {
    a.x += y.x;
    a.y += y.y;
    a.z += y.z;
    a.w += y.w;
}

__device__ __forceinline__ void f4_fma(float4& a, float w, float4 y) {
    a.x = fmaf(w, y.x, a.x);
    a.y = fmaf(w, y.y, a.y);
    a.z = fmaf(w, y.z, a.z);
    a.w = fmaf(w, y.w, a.w);
}

// Gather of one 16-byte piece of a slab row through a buffer resource: an
// offset past the slab (a padded arc slot) reads zeros and touches no memory.
__device__ __forceinline__ float4 slab_load(__amdgpu_buffer_rsrc_t r, uint32_t off) {
    const auto v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0);
    return make_float4(__int_as_float(v[0]), __int_as_float(v[1]), __int_as_float(v[2]), __int_as_float(v[3]));
}

// Sum over the arcs of this lane's row of w_vu * Y[u][4 columns of piece
// qoff] (w = 1 without weights).  The 8 lanes of a row read 8 arc indices at
// once, coalesced, and pass them round with ds_bpermute; each lane then adds
// its row's neighbours in arc order, so a row's sum does not depend on which
// rows share its wave.  Every lane of the wave must call it (dg = 0 for a
// lane without a row).
// FLAGGED: only neighbours u with flags[u] != 0 are read (the others count
// as zero rows), and `got` is set when the row has such a neighbour.
// STEP: arcs a lane group advances per pass; 8 when each group owns a row,
// 64 when the wave's 8 groups share one row (group g then passes its row's
// arcs from 8g on, and the caller adds the groups' sums).
// AHEAD: the gathers of a pass go out before the pass ahead of it is summed,
// so that a row waits for half a load latency per pass; it costs 32 registers
// (streaming step at 10^6 nodes, 3e7 arcs, 64 columns: 1233 us per push
// without, 1040 us with; short rows lose, see stream_launch_step); it also
// shortens the Group Forward-Push rounds of small grids, whose longest row sets
// their time.  The flagged rounds of large grids lose more by the lower occupancy
// than they gain (late rounds 57-135 us without, 100 us and more with), dense ones
// do not change.
template <bool WEIGHTED, bool FLAGGED, int STEP, bool AHEAD>
__device__ __forceinline__ float4 slab_gather(__amdgpu_buffer_rsrc_t rin, const int32_t* __restrict__ col_idx,
                                              const float* __restrict__ weight, int rs, int dg, int lane,
                                              uint32_t qoff, const uint8_t* __restrict__ flags = nullptr,
                                              int* got = nullptr) {
    const int q = lane % kSlabVec;
    int dmax = dg;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) dmax = max(dmax, __shfl_xor(dmax, o, kWave));
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    int any = 0;
    const int lead = (lane & ~(kSlabVec - 1)) * 4;  // ds_bpermute address of the group's first lane
    // Software pipeline over the passes: arc indices are loaded two passes
    // ahead of a pass's gathers, weights and push flags one pass ahead.  A
    // pass past the longest row reads zeros and touches no memory.
    int idx_cur = q < dg ? col_idx[rs + q] : -1;
    int idx_next = STEP + q < dg ? col_idx[rs + STEP + q] : -1;
    float wl_cur = 0.f;
    if (WEIGHTED) wl_cur = q < dg ? weight[rs + q] : 0.f;
    bool on_cur = true;
    if (FLAGGED) on_cur = idx_cur >= 0 && flags[idx_cur] != 0;
    int k0 = 0;  // the pass issued next
    auto issue = [&](float4 (&y)[kSlabVec], float& wl) {
        int idx = idx_cur;
        wl = wl_cur;
        const bool on = on_cur;
        const int idx_after = k0 + 2 * STEP + q < dg ? col_idx[rs + k0 + 2 * STEP + q] : -1;
        if (WEIGHTED) wl_cur = k0 + STEP + q < dg ? weight[rs + k0 + STEP + q] : 0.f;
        if (FLAGGED) {
            on_cur = idx_next >= 0 && flags[idx_next] != 0;
            idx = on ? idx : -1;
            any |= on ? 1 : 0;
        }
        idx_cur = idx_next;
        idx_next = idx_after;
        k0 += STEP;
#pragma unroll
        for (int j = 0; j < kSlabVec; ++j) {
            const int u = __builtin_amdgcn_ds_bpermute(lead + 4 * j, idx);
            y[j] = slab_load(rin, ((uint32_t)u << 7) | qoff);
        }
    };
    auto add = [&](const float4 (&y)[kSlabVec], float wl) {
#pragma unroll
        for (int j = 0; j < kSlabVec; ++j) {
            if (WEIGHTED) {
                const float w = __int_as_float(__builtin_amdgcn_ds_bpermute(lead + 4 * j, __float_as_int(wl)));
                f4_fma(acc, w, y[j]);
            } else {
                f4_acc(acc, y[j]);
            }
        }
    };
    float4 ya[kSlabVec], yb[kSlabVec];
    float wa = 0.f, wb = 0.f;
    if (!AHEAD) {
        while (k0 < dmax) {
            issue(ya, wa);
            add(ya, wa);
        }
    } else if (dmax > 0) {
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
    if (FLAGGED) {
        // OR over the 8 lanes of the row
#pragma unroll
        for (int o = 1; o < kSlabVec; o <<= 1) any |= __shfl_xor(any, o, kWave);
        *got = any;
    }
    return acc;
}

// One adjoint term, forcing deg[v] * G[v][col].  A wave takes 8 rows of the
// degree order side by side within one slab: lane = 8 * g + q, where g picks
// the row and q 4 of the slab's 32 columns (one 16-byte load per arc, summed
// by slab_gather).
template <bool WEIGHTED, bool FINAL, bool AHEAD>
__global__ __launch_bounds__(256) void stream_step_kernel(
    const RowEnt* __restrict__ rows, const int32_t* __restrict__ col_idx,
    const float* __restrict__ weight, const float* __restrict__ invd, const float* __restrict__ deg,
    const float* __restrict__ forcing, int64_t ld_forcing, int32_t n,
    int32_t ncols, float alpha, StreamGrid grid, const float* __restrict__ yin, float* __restrict__ yout) {
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int q = lane % kSlabVec;
    int slab, rb;
    stream_block_map(grid, slab, rb);
    const int64_t slab_off = (int64_t)slab * n * kSlab;
    const uint32_t slab_bytes = (uint32_t)n * (kSlab * 4);
    const __amdgpu_buffer_rsrc_t rin =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(yin + slab_off), 0, (int)slab_bytes, 0x00020000);
    const int ri = rb * kStreamRowsPerBlock + wave * kStreamRowsPerWave + lane / kSlabVec;
    const bool has_row = ri < n;
    int rs = 0, dg = 0, v = 0;
    if (has_row) {
        const RowEnt e = load_row(as_global(rows), ri);
        rs = e.rs;
        dg = e.re - e.rs;
        v = e.v;
    }
    const uint32_t qoff = (uint32_t)q * 16u;
    float4 acc = slab_gather<WEIGHTED, false, kSlabVec, AHEAD>(rin, col_idx, weight, rs, dg, lane, qoff);
    if (has_row && dg == 0) acc = slab_load(rin, ((uint32_t)v << 7) | qoff);
    if (!has_row) return;
    const int col0 = slab * kSlab + q * 4;
    float x[4] = {acc.x, acc.y, acc.z, acc.w};
    const float sv = FINAL ? 1.0f : (1.0f - alpha) * invd[v];
    const float dv = deg[v];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int col = col0 + c;
        x[c] += col < ncols ? dv * forcing[(int64_t)v * ld_forcing + col] : 0.0f;
        x[c] = FINAL ? x[c] : x[c] * sv;
    }
    float4* o4 = reinterpret_cast<float4*>(yout + slab_off);
    o4[(int64_t)v * kSlabVec + q] = make_float4(x[0], x[1], x[2], x[3]);
}

// Y_0 = (1-alpha)/d * Gb for the adjoint (Gb = d * G), or Gb itself when final.
static __global__ void stream_init_adjoint_kernel(const float* __restrict__ forcing, int64_t ld_forcing,
                                           const float* __restrict__ deg, const float* __restrict__ invd,
                                           int32_t n, int32_t ncols, int64_t ld, float alpha, int final_,
                                           float* __restrict__ y) {
    const int64_t col = (int64_t)blockIdx.y * 64 + (threadIdx.x & 63);
    const int64_t v = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (v >= n) return;
    float g = col < ncols ? deg[v] * forcing[v * ld_forcing + col] : 0.0f;
    y[sidx(v, col, n)] = final_ ? g : g * (1.0f - alpha) * invd[v];
}

static __global__ void stream_resid_kernel(const double* __restrict__ part, int64_t chunks, int64_t ld, int32_t ncols,
                                    double* __restrict__ resid) {
    int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= ncols) return;
    double t = 0.0;
    for (int64_t c = 0; c < chunks; ++c) t += part[c * ld + s];
    resid[s] = 1.0 - t;
}

// Gathers go out a pass ahead from a mean of 20 arcs per row on: shorter rows are
// one to three passes and wait less than the lower occupancy costs.  A step with and
// without, weights: 12000 nodes, 4, 12, 20 and 80 arcs 582, 842, 1047 and 2658 us and
// 557, 815, 1055 and 2691; 36000 nodes, 40 arcs 18.1 and 18.8 ms.
template <bool FINAL, bool AHEAD>
inline void stream_launch_step(const StreamArgs& a, const float* yin, float* yout, hipStream_t s) {
    StreamGrid g;
    g.row_blocks = (a.n + kStreamRowsPerBlock - 1) / kStreamRowsPerBlock;
    g.slabs = (int32_t)(a.ld / kSlab);
    g.full_rounds = ((int64_t)a.n * kSlab * 4 <= kStreamSlabBudget) ? g.slabs / kXcds : 0;
    const dim3 grid((unsigned)((int64_t)g.row_blocks * g.slabs));
    if (a.weight)
        hipLaunchKernelGGL((stream_step_kernel<true, FINAL, AHEAD>), grid, dim3(256), 0, s, a.rows, a.col_idx, a.weight,
                           a.invd, a.deg, a.forcing, a.ld_forcing, a.n, a.ncols, a.alpha, g, yin, yout);
    else
        hipLaunchKernelGGL((stream_step_kernel<false, FINAL, AHEAD>), grid, dim3(256), 0, s, a.rows, a.col_idx, a.weight,
                           a.invd, a.deg, a.forcing, a.ld_forcing, a.n, a.ncols, a.alpha, g, yin, yout);
}

// T adjoint terms; returns the buffer that holds the final unscaled iterate.
inline const float* stream_adjoint(const StreamArgs& a, int T, float* ya, float* yb, hipStream_t s) {
    fill<float>(ya, 0.0f, (int64_t)a.n * a.ld, s);
    if (T <= 0) return ya;
    const dim3 grid((unsigned)((a.n + 3) / 4), (unsigned)(a.ld / 64));
    hipLaunchKernelGGL(stream_init_adjoint_kernel, grid, dim3(256), 0, s, a.forcing, a.ld_forcing, a.deg, a.invd, a.n,
                       a.ncols, a.ld, a.alpha, T == 1 ? 1 : 0, ya);
    float* in = ya;
    float* out = yb;
    const bool ahead = a.nnz >= 20 * (int64_t)a.n;
    for (int it = 1; it < T; ++it) {
        if (it == T - 1) {
            if (ahead) stream_launch_step<true, true>(a, in, out, s);
            else stream_launch_step<true, false>(a, in, out, s);
        } else {
            if (ahead) stream_launch_step<false, true>(a, in, out, s);
            else stream_launch_step<false, false>(a, in, out, s);
        }
        float* t = in;
        in = out;
        out = t;
    }
    return in;
}

}  // namespace pprviz
