// Single-graph multi-source PPR / DPPR (ppr_matrix) and shared helpers.
#include <math.h>
#include <string.h>

#include <algorithm>

#include "internal.hpp"
#include "ppr_core.hpp"
#include "ppr_dense.hpp"

namespace pprviz {

__global__ void degree_kernel(const int32_t* __restrict__ row_ptr, const float* __restrict__ weight,
                              int64_t n, float* __restrict__ deg, float* __restrict__ invd) {
    int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    const int rs = row_ptr[v], re = row_ptr[v + 1];
    float d;
    if (weight) {
        float s = 0.f;
        for (int e = rs; e < re; ++e) s += weight[e];
        d = s;
    } else {
        d = (float)(re - rs);
    }
    deg[v] = d;
    invd[v] = (re > rs && d > 0.f) ? 1.0f / d : 1.0f;
}

// Slot table and arc copy of the resident tile (group layout, see
// ppr_core.hpp), in two kernels.
// res_sort_kernel, one block per graph:
//  1. Rows sorted by degree, longest first, ties by row id (bitonic sort of
//     4096 keys in LDS; a graph of the resident tile has at most 2304 rows).
//  2. Group g's length: its longest row (at least 1: a row without arcs gets
//     its self arc) in 8-arc halves; chunk offsets by a prefix sum in sorted
//     order; the slot table.
// res_deal_kernel, one block per four groups:
//  3. Arcs are dealt by LDS bank class.  One LDS cycle of the tile's
//     16-byte reads serves M rows at once (M = 4, 2, 1 for 16, 32, 64
//     columns: 64 bytes of each of 4 rows, 128 of 2, 256 of 1;
//     res_conflict_set names them), and row u starts in bank class u mod M.
//     Four lanes first group the arcs of one row by class.  Then one lane
//     takes such a set of M rows and fills their positions m = 0, 1, ...
//     together: each row takes, among the classes no other row has
//     taken at m, the one it holds most arcs of; a row with no such arc pads
//     with the zero row of a free class (the tile has one zero row per class)
//     as long as it can still fit its arcs, and otherwise takes a
//     conflicting class.  Only the order of each row's arcs changes (and
//     with it the order of the FP32 sum).  The deal notes where an arc is to
//     be found, so that nothing it does waits for memory; all lanes then put
//     the arcs themselves in place.  The copy holds each arc's LDS byte
//     offset in the tile, (u - first node) * 4 COLS, not its node id.
// A graph whose padded groups exceed its reserved region (possible only with
// repeated arcs, when a row is longer than n) gets one half chunk per row
// holding the row's own offset and a NaN scale, so that its outputs are NaN.
//
// Bound: latency.  One block per graph for all of it left a graph's rows to
// 256 threads, each with its own chain of dependent loads (n = 2048, 1.3e5
// arcs: 1190 us, more than its push series); with four groups per block
// 182 us (28 the sort, 154 the deal); with four lanes per row in the grouping
// by class 116 to 131 the deal (of n = 2048, a quarter the grouping before, two
// thirds the serial choice).
// The rows of a group whose LDS reads are served in the same cycles.  A
// 16-byte LDS read by a wave is served 16 lanes at a time, lanes grouped by
// lane bit 5 and the parity of lane bits 2..4 (a probe of the patterns
// across the 16 quads of a wave: quads {0,3,5,6} share cycles, as do
// {1,2,4,7} and the same sets plus 8).  With 16 columns a quad is a row,
// so those quad sets are the row sets; with 32 columns quads 2r and 2r+1
// read the two halves of row r, and the rows whose halves meet in one
// cycle set are {0,3} and {1,2} (and plus 4); with 64 columns one row fills
// a cycle set.
__device__ __forceinline__ void res_conflict_set(int M, int j, int rr[4]) {
    if (M == 4) {
        const int h = (j >> 1) * 8;
        const bool odd = (j & 1) != 0;
        rr[0] = h + (odd ? 1 : 0);
        rr[1] = h + (odd ? 2 : 3);
        rr[2] = h + (odd ? 4 : 5);
        rr[3] = h + (odd ? 7 : 6);
    } else if (M == 2) {
        const int h = (j >> 1) * 4;
        rr[0] = h + ((j & 1) ? 1 : 0);
        rr[1] = h + ((j & 1) ? 2 : 3);
        rr[2] = rr[3] = 0;
    } else {
        rr[0] = j;
        rr[1] = rr[2] = rr[3] = 0;
    }
}

// One set of M rows of a group (res_conflict_set), dealt together.
struct ResDealSet {
    int L;          // positions every row of the set fills (the group's length)
    int words;      // entries per row over all its chunks
    int32_t* ca;    // the group's chunk 0 in the arc copy
    float* wa;      // same for the weights, or nullptr
    int GW, n, stride;
    int64_t base;
    bool over;      // NaN layout: each row holds only its own offset
    const int32_t* row_ptr;
    const int32_t (*cstart)[4];  // per row of the block: where its arcs of each class start in the grouped copy
    int row0;                    // the group's first row in cstart
};

// Fills the set's rows position by position.  At position m the rows choose
// in the order m, m+1, ... (mod M); each takes the free class it holds most
// arcs of (the lowest such class), pads with the zero row of a free class when
// it has none and can still fit its arcs, and otherwise takes its largest
// class (a conflict).  Rows without arcs hold their own offset first; v[i] < 0
// marks a dummy slot.  The choice is arithmetic on keys 4 count + 3 - class,
// without branches: the lanes of a wave hold rows of different lengths, and
// branching cost each of them every path.
template <int M>
__device__ __forceinline__ void res_deal_set(const ResDealSet& d, const int rr[4], const int v[4]) {
    auto at = [&](int m) { return (int64_t)(m >> 4) * 16 * d.GW + (m & 15); };
    int zero[M];  // offset of each class's zero row
#pragma unroll
    for (int c = 0; c < M; ++c) zero[c] = (d.n + (((c - d.n) % M) + M) % M) * d.stride;
    auto put = [&](int i, int m, int off, float w) {
        d.ca[16 * rr[i] + at(m)] = off;
        if (d.wa) d.wa[16 * rr[i] + at(m)] = w;
    };
    int cnt[M][M], end[M][M], rem[M];  // arcs left per class, one past the class's last arc, arcs left
    bool fixed[M];                     // rows written outside the deal (own offset first)
#pragma unroll
    for (int i = 0; i < M; ++i) {
        rem[i] = 0;
        fixed[i] = false;
#pragma unroll
        for (int c = 0; c < M; ++c) cnt[i][c] = end[i][c] = 0;
        if (v[i] < 0) continue;
        const int rs = d.row_ptr[d.base + v[i]];
        const int re = d.row_ptr[d.base + v[i] + 1];
        if (d.over || re == rs) {
            put(i, 0, v[i] * d.stride, 1.f);
            for (int m = 1; m < d.words; ++m) put(i, m, d.n * d.stride, 0.f);
            fixed[i] = true;
            continue;
        }
        rem[i] = re - rs;
#pragma unroll
        for (int c = 0; c < M; ++c) {
            const int c0 = d.cstart[d.row0 + rr[i]][c];
            const int c1 = c + 1 < M ? d.cstart[d.row0 + rr[i]][c + 1] : re - rs;
            cnt[i][c] = c1 - c0;
            end[i][c] = rs + c1;
        }
    }
    constexpr uint32_t kFull = (1u << M) - 1u;
    for (int mb = 0; mb < d.L; mb += M) {
#pragma unroll
        for (int s = 0; s < M; ++s) {
            const int m = mb + s;
            uint32_t taken = 0;
            bool live[M];
#pragma unroll
            for (int i = 0; i < M; ++i) live[i] = rem[i] > 0;
#pragma unroll
            for (int k = 0; k < M; ++k) {
                const int i = (s + k) % M;
                int any = 0, fre = 0;
#pragma unroll
                for (int c = 0; c < M; ++c) {
                    const int key = 4 * cnt[i][c] + 3 - c;
                    any = max(any, key);
                    fre = max(fre, (taken >> c & 1u) ? 0 : key);
                }
                const bool has = fre >= 4;
                const bool pad = !has && rem[i] < d.L - m && taken != kFull;
                const int open = __builtin_ctz(~taken);
                const int c = pad ? open : 3 - ((has ? fre : any) & 3);
                // the arc's place in the grouped copy, as a negative number:
                // the arcs are filled in afterwards
                int off = pad ? zero[0] : cnt[i][0] - 1 - end[i][0];
#pragma unroll
                for (int q = 1; q < M; ++q) off = c == q ? (pad ? zero[q] : cnt[i][q] - 1 - end[i][q]) : off;
                if (live[i]) put(i, m, off, 0.f);
                taken |= live[i] ? 1u << c : 0u;
                const int took = live[i] && !pad ? 1 : 0;
                rem[i] -= took;
#pragma unroll
                for (int q = 0; q < M; ++q) cnt[i][q] -= c == q ? took : 0;
            }
            // rows already done, and dummy slots: zero rows of free classes
#pragma unroll
            for (int i = 0; i < M; ++i) {
                const bool idle = !live[i] && !fixed[i];
                const int c = taken == kFull ? 0 : __builtin_ctz(~taken);
                int off = zero[0];
#pragma unroll
                for (int q = 1; q < M; ++q) off = c == q ? zero[q] : off;
                if (idle) put(i, m, off, 0.f);
                taken |= idle ? 1u << c : 0u;
            }
        }
    }
    // entries past L up to the end of the last chunk (read where wider groups hold the dealt one)
#pragma unroll
    for (int i = 0; i < M; ++i) {
        if (fixed[i]) continue;
        for (int m = d.L; m < d.words; ++m) put(i, m, d.n * d.stride, 0.f);
    }
}

constexpr int kResSortThreads = 512;

// A graph by itself takes 16-column tiles at any size, so that its sources make
// as many blocks as they can (pushes of n = 500, all sources: 8 blocks 275 us,
// 32 blocks 111 us; n = 1000, weighted: 386 and 238 us): its rows then
// stand in groups of 16, with each row's arcs in the order that its own size's
// groups of 4 or 8 would give them, so that its sums are the batch's to the
// bit.  Only repeated arcs can make the wider groups too long for the arc
// copy; such a graph keeps its own size's tile.  The tile width chosen stands
// in the last entry of the slot table.
__device__ __forceinline__ bool res_narrow(const int64_t* node_off, int cols) {
    return node_off == nullptr && cols > 16;
}

__global__ __launch_bounds__(kResSortThreads) void res_sort_kernel(const int32_t* __restrict__ row_ptr,
                                                                  const float* __restrict__ invd,
                                                                  const int64_t* __restrict__ node_off,
                                                                  int32_t n_single, ResSlot* __restrict__ slots) {
    constexpr int kMaxRows = 4096;
    __shared__ uint32_t key[kMaxRows];
    __shared__ int64_t goff[256];  // group offsets; kResMaxGroups + 1 used
    __shared__ int32_t ghalves[kResMaxGroups];
    static_assert(kResMaxGroups < 256, "the prefix sum below covers 256 groups");
    const int g = blockIdx.x;
    const int64_t base = node_off ? node_off[g] : 0;
    const int n = node_off ? (int)(node_off[g + 1] - base) : n_single;
    const int cols = n > 0 ? res_cols_for(n) : 0;
    if (cols == 0) return;  // larger graphs never use the resident tile
    TileTask tb;
    res_graph_bases(base, row_ptr[base], row_ptr[base + n], g, n, tb);

    int P = 1;
    while (P < n) P <<= 1;
    for (int i = threadIdx.x; i < P; i += kResSortThreads) {
        if (i < n) {
            const int d = min(row_ptr[base + i + 1] - row_ptr[base + i], 4095);
            key[i] = ((uint32_t)(4095 - d) << 12) | (uint32_t)i;
        } else {
            key[i] = 0xFFFFFFFFu;
        }
    }
    __syncthreads();
    // bitonic sort, ascending key = descending degree, ties by row id
    for (int k = 2; k <= P; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int h = threadIdx.x; h < P / 2; h += kResSortThreads) {
                const int i = ((h & ~(j - 1)) << 1) | (h & (j - 1));
                const int ixj = i | j;
                const uint32_t x = key[i], y = key[ixj];
                const bool up = (i & k) == 0;
                if ((x > y) == up) {
                    key[i] = y;
                    key[ixj] = x;
                }
            }
            __syncthreads();
        }
    }
    // the groups of GW rows: their lengths and places; returns the arc copy's size
    auto place_groups = [&](int GW) -> int64_t {
        const int ng = (n + GW - 1) / GW;
        __syncthreads();
        if (threadIdx.x < 256) {
            const int gi = threadIdx.x;
            int64_t words = 0;
            if (gi < ng) {
                int dmax = 1;
                for (int r = 0; r < GW; ++r) {
                    const int p = gi * GW + r;
                    if (p < n) {
                        const int64_t gv = base + (int)(key[p] & 4095u);
                        dmax = max(dmax, row_ptr[gv + 1] - row_ptr[gv]);
                    }
                }
                const int h = (int)(((int64_t)dmax + 7) / 8);
                ghalves[gi] = h;
                words = (int64_t)((h + 1) / 2) * 16 * GW;
            }
            goff[gi] = words;
        }
        __syncthreads();
        // exclusive prefix sum of the groups' sizes
        for (int o = 1; o < 256; o <<= 1) {
            int64_t x = 0;
            if (threadIdx.x < 256 && (int)threadIdx.x >= o) x = goff[threadIdx.x - o];
            __syncthreads();
            if (threadIdx.x < 256) goff[threadIdx.x] += x;
            __syncthreads();
        }
        return goff[ng - 1];
    };
    int GW = Res<16>::RPW;
    int64_t words = 0;
    if (cols == 16 || res_narrow(node_off, cols)) words = place_groups(GW);
    if (cols != 16 && (!res_narrow(node_off, cols) || words > (int64_t)tb.cwords)) {
        GW = 256 / cols;  // group size, Res<cols>::RPW
        words = place_groups(GW);
    }
    if (res_narrow(node_off, cols) && threadIdx.x == 0) slots[tb.tbase + n + kResTabPad - 1].off = 256 / GW;
    const int ng = (n + GW - 1) / GW;
    const bool over = words > (int64_t)tb.cwords;
    // slot table
    for (int p = threadIdx.x; p < ng * GW; p += kResSortThreads) {
        const int gi = p / GW;
        const int r = p - gi * GW;
        const int h = over ? 1 : ghalves[gi];
        const int64_t o = (over ? (int64_t)gi * 16 * GW : (gi > 0 ? goff[gi - 1] : 0)) + 16 * r;
        int v = n;
        float iv = 0.f;
        if (p < n) {
            v = (int)(key[p] & 4095u);
            iv = over ? __int_as_float(0x7fc00000) : invd[base + v];
        }
        slots[tb.tbase + p] = ResSlot{(int32_t)o, h, v, iv};
    }
}

constexpr int kResDealThreads = 256;
constexpr int kResDealGroups = 4;                                                      // groups per block
constexpr int kResDealBlocks = (kResMaxGroups + kResDealGroups - 1) / kResDealGroups;  // blocks per graph, at most

__global__ __launch_bounds__(kResDealThreads) void res_deal_kernel(const int32_t* __restrict__ row_ptr,
                                                      const int32_t* __restrict__ col_idx,
                                                      const float* __restrict__ weight,
                                                      const int64_t* __restrict__ node_off, int32_t n_single,
                                                      const ResSlot* __restrict__ slots, int32_t* __restrict__ arcs,
                                                      float* __restrict__ warcs, int32_t* sorted, float* wsorted) {
    __shared__ int32_t cstart[kResDealGroups * Res<16>::RPW][4];
    const int lane = threadIdx.x;
    const int g = blockIdx.x / kResDealBlocks;
    const int g0 = (blockIdx.x % kResDealBlocks) * kResDealGroups;
    const int64_t base = node_off ? node_off[g] : 0;
    const int n = node_off ? (int)(node_off[g + 1] - base) : n_single;
    const int cols = n > 0 ? res_cols_for(n) : 0;
    if (cols == 0) return;
    TileTask tb;
    res_graph_bases(base, row_ptr[base], row_ptr[base + n], g, n, tb);
    const ResSlot* tab = slots + tb.tbase;
    const int width = res_narrow(node_off, cols) ? tab[n + kResTabPad - 1].off : cols;  // of the tile
    const int GW = 256 / width;
    const int ng = (n + GW - 1) / GW;
    if (g0 >= ng) return;
    const int M = cols == 16 ? 4 : (cols == 32 ? 2 : 1);  // bank classes = rows per LDS pass
    const int DW = 256 / cols;                            // rows dealt as one group, in sets of M
    const int stride = width * 4;                         // LDS bytes per row
    const float s0 = tab[0].invd;
    const bool over = s0 != s0;
    const int gn = min(kResDealGroups, ng - g0);
    // each row's arcs as LDS offsets, grouped by bank class (CSR order within
    // a class), and where each class starts
    // (four lanes per row, a quarter of its arcs each)
    const int part = lane & 3;
    for (int q = lane >> 2; q < gn * GW; q += kResDealThreads / 4) {
        const int v = tab[g0 * GW + q].v;
        if (v >= n || over) continue;
        const int rs = row_ptr[base + v], re = row_ptr[base + v + 1];
        const int share = (re - rs + 3) / 4;
        const int e0 = min(re, rs + part * share), e1 = min(re, e0 + share);
        int cn[4] = {0, 0, 0, 0};
#pragma unroll 8
        for (int e = e0; e < e1; ++e) {
            const int c = (int)((col_idx[e] - base) & (M - 1));
#pragma unroll
            for (int k = 0; k < 4; ++k) cn[k] += c == k;
        }
        int pos[4], at = rs;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int a0 = quad_bcast<0>(cn[k]), a1 = quad_bcast<1>(cn[k]), a2 = quad_bcast<2>(cn[k]),
                      a3 = quad_bcast<3>(cn[k]);
            pos[k] = at + (part > 0 ? a0 : 0) + (part > 1 ? a1 : 0) + (part > 2 ? a2 : 0);
            if (part == 0) cstart[q][k] = at - rs;
            at += a0 + a1 + a2 + a3;
        }
#pragma unroll 8
        for (int e = e0; e < e1; ++e) {
            const int u = (int)(col_idx[e] - base);
            const int c = u & (M - 1);
            const int to = c == 0 ? pos[0]++ : (c == 1 ? pos[1]++ : (c == 2 ? pos[2]++ : pos[3]++));
            sorted[to] = u * stride;
            if (wsorted) wsorted[to] = weight[e];
        }
    }
    __syncthreads();
    // one lane per set of M rows of a group of DW whose reads share LDS cycles
    // (4 sets per group)
    const int parts = GW / DW;
    if (lane < gn * parts * 4) {
        const int gl = lane / (4 * parts);
        const int gi = g0 + gl;
        const int sub = (lane >> 2) % parts * DW;  // the dealt group's first row in its group
        const ResSlot e = tab[gi * GW];
        const int first = gi * GW + sub;
        int len = e.halves;  // of the dealt group
        if (parts > 1) {
            int dmax = 1;
            for (int p = first; p < min(first + DW, n); ++p) {
                const int fv = tab[p].v;
                dmax = max(dmax, row_ptr[base + fv + 1] - row_ptr[base + fv]);
            }
            len = (dmax + 7) / 8;
        }
        ResDealSet d;
        d.L = len * 8;
        d.words = (e.halves + 1) / 2 * 16;
        d.ca = arcs + tb.cbase + e.off;
        d.wa = warcs ? warcs + tb.cbase + e.off : nullptr;
        d.GW = GW;
        d.n = n;
        d.stride = stride;
        d.base = base;
        d.over = over;
        d.row_ptr = row_ptr;
        d.cstart = cstart;
        d.row0 = gl * GW;
        int rr[4];
        res_conflict_set(M, lane & 3, rr);
        int v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            rr[i] += sub;
            const int p = gi * GW + rr[i];
            v[i] = (i < M && p < n) ? tab[p].v : -1;
        }
        if (M == 4) res_deal_set<4>(d, rr, v);
        else if (M == 2) res_deal_set<2>(d, rr, v);
        else res_deal_set<1>(d, rr, v);
    }
    __syncthreads();
    // the arcs, where the deal put them
    const int64_t w0 = tb.cbase + tab[g0 * GW].off;
    const ResSlot le = tab[(g0 + gn - 1) * GW];
    const int64_t w1 = tb.cbase + le.off + (int64_t)((le.halves + 1) / 2) * 16 * GW;
    constexpr int kBatch = 8;  // loads in flight per lane
    for (int64_t i0 = w0 + lane; i0 < w1; i0 += kBatch * kResDealThreads) {
        int a[kBatch], x[kBatch];
        float w[kBatch];
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            const int64_t i = i0 + j * kResDealThreads;
            a[j] = i < w1 ? arcs[i] : 0;
        }
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            x[j] = a[j] < 0 ? sorted[-1 - a[j]] : 0;
            w[j] = a[j] < 0 && warcs ? wsorted[-1 - a[j]] : 0.f;
        }
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            if (a[j] >= 0) continue;
            arcs[i0 + j * kResDealThreads] = x[j];
            if (warcs) warcs[i0 + j * kResDealThreads] = w[j];
        }
    }
}

void launch_res_layout(const int32_t* row_ptr, const int32_t* col_idx, const float* weight, const float* invd,
                       const int64_t* node_off, int32_t n_single, int32_t blocks, ResSlot* slots, int32_t* arcs,
                       float* warcs, int32_t* sorted, float* wsorted, hipStream_t s) {
    hipLaunchKernelGGL(res_sort_kernel, dim3(blocks), dim3(kResSortThreads), 0, s, row_ptr, invd, node_off, n_single,
                       slots);
    hipLaunchKernelGGL(res_deal_kernel, dim3(blocks * kResDealBlocks), dim3(kResDealThreads), 0, s, row_ptr, col_idx, weight,
                       node_off, n_single, slots, arcs, warcs, sorted, wsorted);
}

template <int COLS, bool WEIGHTED>
__global__ __launch_bounds__(kResThreads) void ppr_resident_kernel(ResArgs a, int32_t n, int64_t nnz,
                                                                 int32_t n_src, int32_t n_tgt, int32_t T,
                                                                 int32_t m, int32_t r, bool chosen) {
    __shared__ ResLds L;
    if (chosen && a.slots[n + kResTabPad - 1].off != COLS) return;  // the other width's launch does it
    TileTask t;
    t.n = n;
    t.s0 = blockIdx.x * COLS;
    t.ncols = min(COLS, n_src - t.s0);
    t.n_tgt = n_tgt;
    t.base = 0;
    t.out_off = 0;
    t.ld = n_tgt;
    t.T = T;
    t.m = m;
    t.r = r;
    res_graph_bases(0, 0, nnz, 0, n, t);
    res_tile<COLS, WEIGHTED>(t, a, L);
}

void launch_degree(const int32_t* row_ptr, const float* weight, int64_t n, float* deg, float* invd,
                   hipStream_t s) {
    int64_t blocks = (n + 255) / 256;
    hipLaunchKernelGGL(degree_kernel, dim3((unsigned)blocks), dim3(256), 0, s, row_ptr, weight, n, deg, invd);
}

template <int COLS>
static void launch_resident(bool weighted, const ResArgs& a, int n, int64_t nnz, int n_src, int n_tgt, int T, int m,
                            int r, bool chosen, hipStream_t s) {
    dim3 grid((n_src + COLS - 1) / COLS);
    if (weighted)
        hipLaunchKernelGGL((ppr_resident_kernel<COLS, true>), grid, dim3(kResThreads), 0, s, a, n, nnz, n_src, n_tgt,
                           T, m, r, chosen);
    else
        hipLaunchKernelGGL((ppr_resident_kernel<COLS, false>), grid, dim3(kResThreads), 0, s, a, n, nnz, n_src,
                           n_tgt, T, m, r, chosen);
}

static void launch_resident_any(bool weighted, const ResArgs& a, int n, int64_t nnz, int n_src, int n_tgt, int T,
                                int m, int r, hipStream_t s) {
    // up to 1152 nodes the layout's width decides which launch does the work (res_narrow)
    const int cols = res_cols_for(n);
    launch_resident<16>(weighted, a, n, nnz, n_src, n_tgt, T, m, r, cols != 16, s);
    if (cols == 32) launch_resident<32>(weighted, a, n, nnz, n_src, n_tgt, T, m, r, true, s);
    if (cols == 64) launch_resident<64>(weighted, a, n, nnz, n_src, n_tgt, T, m, r, true, s);
}

// One product of the all-pairs series (ppr_dense.hpp), one 64-wide tile per
// block: a single graph has too few 128-wide tiles to fill the chip (n = 2048:
// 136 of them, 204 us a product; 528 64-wide ones, 136 us then, 125 us now).
constexpr int kSingleBT = 64;

template <DenseOut OUT>
__global__ __launch_bounds__(kDenseThreads, 2) void ppr_product_kernel(const float* V, const float* xm,
                                                                     const float* W, const float* deg,
                                                                     const float* invd, float alpha, int32_t n,
                                                                     float* out) {
    __shared__ DenseLds<kSingleBT> L;
    dense_product_tile<kSingleBT, OUT>(V, xm, W, deg, invd, alpha, n, blockIdx.x, L, out);
}

// Outputs from X_T, one block per source: pi_hat(s, t), DPPR, and the FP64
// residual over all nodes.
__global__ __launch_bounds__(256) void ppr_series_out_kernel(const float* __restrict__ X,
                                                             const float* __restrict__ deg, int32_t n,
                                                             const int32_t* __restrict__ src,
                                                             const int32_t* __restrict__ tgt, int32_t n_tgt,
                                                             float* __restrict__ ppr_out,
                                                             float* __restrict__ dppr_out,
                                                             double* __restrict__ resid) {
    __shared__ double red[4];
    const int i = blockIdx.x;
    const int s = src ? src[i] : i;
    const float* row = X + (int64_t)s * n;
    const float ds = deg[s];
    for (int j = threadIdx.x; j < n_tgt; j += 256) {
        const float x = row[tgt ? tgt[j] : j];
        if (ppr_out) ppr_out[(int64_t)i * n_tgt + j] = x;
        if (dppr_out) dppr_out[(int64_t)i * n_tgt + j] = x * ds;
    }
    if (resid == nullptr) return;
    double sum = 0.0;
    for (int v = threadIdx.x; v < n; v += 256) sum += (double)row[v];
    sum = wave_sum(sum);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) resid[i] = 1.0 - ((red[0] + red[1]) + (red[2] + red[3]));
}

// All pairs by the series: a short run of pushes from every node, k products,
// outputs.  buf: 4 n^2 floats (V, X_m, and two that the W_p alternate between).
static void ppr_series(const ppr_csr* g, const DensePlan& p, const int32_t* src, const int32_t* tgt, int32_t n_tgt,
                       ResArgs a, const float* invd, float* ppr_out, float* dppr_out, double* resid, float* buf,
                       hipStream_t s) {
    const int n = g->n;
    const int64_t n2 = (int64_t)n * n;
    float* w[2] = {buf + 2 * n2, buf + 3 * n2};
    a.src = nullptr;
    a.tgt = nullptr;
    a.ppr_out = a.dppr_out = nullptr;
    a.resid = nullptr;
    a.vd = buf;
    a.xm = buf + n2;
    a.yr = w[0];
    launch_resident_any(g->weight != nullptr, a, n, g->nnz, n, n, p.m + 1, p.m, p.r, s);
    const dim3 grid((unsigned)dense_tiles(n, kSingleBT));
    for (int i = 0; i < p.k; ++i) {
        const float* from = w[i & 1];
        float* to = w[(i + 1) & 1];
        if (i + 1 < p.k)
            hipLaunchKernelGGL(ppr_product_kernel<kDenseNext>, grid, dim3(kDenseThreads), 0, s, a.vd, a.xm, from,
                               a.deg, invd, a.alpha, n, to);
        else
            hipLaunchKernelGGL(ppr_product_kernel<kDensePpr>, grid, dim3(kDenseThreads), 0, s, a.vd, a.xm, from,
                               a.deg, invd, a.alpha, n, to);
    }
    hipLaunchKernelGGL(ppr_series_out_kernel, dim3(n), dim3(256), 0, s, w[p.k & 1], a.deg, n, src, tgt, n_tgt,
                       ppr_out, dppr_out, resid);
}

ppr_status validate_csr(const ppr_csr* g) {
    if (g == nullptr || g->n < 1 || g->nnz < 0 || g->nnz >= (int64_t)INT32_MAX) return PPR_EINVAL;
    if (g->row_ptr == nullptr || (g->nnz > 0 && g->col_idx == nullptr)) return PPR_EINVAL;
    return PPR_OK;
}

bool use_resident(int n) { return res_cols_for(n) != 0; }

// T pushes from every source; deg/invd must already hold the degrees.  Three
// kernels by size: the LDS-resident tile (n <= 2304; all pairs by fewer pushes
// and dense products where that is faster and the workspace has room for it),
// the mid-size kernel with the iterate columns in LDS (n <= 40831), and the
// iterate in HBM (larger graphs; smaller ones with few sources where that is
// faster and the workspace has room for it).
void ppr_forward(const ppr_csr* g, const int32_t* src, int32_t n_src, const int32_t* tgt, int32_t n_tgt,
                 float alpha, int32_t T, float* ppr_out, float* dppr_out, const float* deg, const float* invd,
                 double* resid, const PprWs& w, hipStream_t s) {
    const int n = g->n;
    // The iterate in HBM: always for graphs that do not fit LDS, else for few
    // sources where it is faster.  The targets being the sources halves the
    // pushes where that is faster (query_halves); a residual needs every node.
    QueryWs q = w.query;
    const bool halve = q.gram != nullptr && alpha >= kDenseMinAlpha && tgt == src && n_tgt == n_src &&
                       resid == nullptr && query_halves(n, g->nnz, n_src, T);
    if (!halve) q.gram = nullptr;
    const bool lds = use_resident(n) || mid_cols_for(n) != 0;
    if (!lds || (q.ya != nullptr && query_faster(n, g->nnz, n_src, T, halve))) {
        query_forward(g, src, n_src, tgt, n_tgt, alpha, T, ppr_out, dppr_out, deg, invd, resid, w.rows, q, s);
    } else if (use_resident(n)) {
        launch_res_layout(g->row_ptr, g->col_idx, g->weight, invd, nullptr, n, 1, w.slots, w.col_r,
                          g->weight ? w.w_r : nullptr, w.sorted_r, g->weight ? w.sorted_w : nullptr, s);
        ResArgs a;
        a.slots = w.slots;
        a.arcs = w.col_r;
        a.warcs = g->weight ? w.w_r : nullptr;
        a.deg = deg;
        a.src = src;
        a.tgt = tgt;
        a.alpha = alpha;
        a.ppr_out = ppr_out;
        a.dppr_out = dppr_out;
        a.resid = resid;
        a.yr = a.xm = a.vd = nullptr;
        // every node a source (sources are distinct): all pairs
        const bool products = n_src == n && w.series != nullptr && dense_alpha(alpha);
        const DensePlan p = dense_plan(n, g->nnz, products ? T : 0);
        if (p.k > 0)
            ppr_series(g, p, src, tgt, n_tgt, a, invd, ppr_out, dppr_out, resid, w.series, s);
        else
            launch_resident_any(g->weight != nullptr, a, n, g->nnz, n_src, n_tgt, T, 0, 0, s);
    } else {
        mid_forward(g, src, n_src, tgt, n_tgt, alpha, T, ppr_out, dppr_out, deg, invd, resid, w.mid, s);
    }
}


// ppr_matrix with the workspace given (the caller's, or this GPU's scratch).
static ppr_status ppr_matrix_impl(const ppr_csr* g, const int32_t* src, int32_t n_src, const int32_t* tgt,
                                  int32_t n_tgt, float alpha, double tol_l1, int32_t max_iter, float* ppr_out,
                                  float* dppr_out, double* resid_out, int32_t* iters_out, void* ws,
                                  size_t ws_bytes, void* stream, bool scratch_ws) {
    ppr_status st = validate_csr(g);
    if (st != PPR_OK) return st;
    if (n_src < 0 || n_tgt < 0 || (n_src > 0 && src == nullptr)) return PPR_EINVAL;
    if (tgt == nullptr && n_tgt != g->n) return PPR_EINVAL;
    if (!(alpha > 0.0f && alpha < 1.0f) || max_iter < 0) return PPR_EINVAL;
    if ((int64_t)n_src * (int64_t)std::max(n_tgt, 1) > ((int64_t)1 << 40)) return PPR_EUNSUPPORTED;
    if (g->n > kStreamMaxN) return PPR_EUNSUPPORTED;
    int32_t T = 0, conv = 1;
    st = pprviz_pushes_for_tolerance(alpha, tol_l1, max_iter, &T, &conv);
    if (st != PPR_OK) return st;
    if (iters_out) *iters_out = T;
    if (n_src == 0) return conv ? PPR_OK : PPR_ENOCONV;
    WsCursor cur{static_cast<char*>(ws), ws_bytes};
    PprWs w;
    ppr_ws_layout(cur, g->n, g->nnz, g->weight != nullptr, n_src, &w);
    if (ws == nullptr || cur.used > ws_bytes) return scratch_ws ? PPR_EUNSUPPORTED : PPR_EWORKSPACE;
    // a workspace with room for a faster route's buffers takes it
    if (scratch_ws) {
        cur.used = kScratchBytes;
        cur.cap = kScratchBytes + kScratchExtraBytes;
    }
    const bool same = tgt != nullptr && tgt == src && n_tgt == n_src;
    ppr_extra_take(cur, g->n, n_src, same, &w);
    if (pending_error() != PPR_OK) return PPR_EHIP;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int n = g->n;
    launch_degree(g->row_ptr, g->weight, n, w.deg, w.invd, s);

    ppr_forward(g, src, n_src, tgt, n_tgt, alpha, T, ppr_out, dppr_out, w.deg, w.invd,
                resid_out ? w.resid : nullptr, w, s);
    st = launch_status();
    if (st != PPR_OK) return st;
    if (resid_out) {
        PPRVIZ_HIP_TRY(hipMemcpyAsync(resid_out, w.resid, sizeof(double) * n_src, hipMemcpyDeviceToHost, s));
        PPRVIZ_HIP_TRY(hipStreamSynchronize(s));
        for (int i = 0; i < n_src; ++i)
            if (!isfinite(resid_out[i])) return PPR_ENONFINITE;
    }
    return conv ? PPR_OK : PPR_ENOCONV;
}

}  // namespace pprviz

using namespace pprviz;

extern "C" {

const char* pprviz_version(void) { return "pprviz-gfx950 1.0"; }

const char* pprviz_status_string(int status) {
    switch (status) {
        case PPR_OK: return "ok";
        case PPR_EINVAL: return "invalid argument";
        case PPR_ENOCONV: return "iteration cap reached before the residual tolerance";
        case PPR_EWORKSPACE: return "workspace missing or too small";
        case PPR_EHIP: return "HIP runtime error";
        case PPR_ENONFINITE: return "non-finite result";
        case PPR_EUNSUPPORTED: return "size not supported by this build";
        default: return "unknown status";
    }
}

ppr_status pprviz_pushes_for_tolerance(float alpha, double tol, int32_t max_iter, int32_t* pushes,
                                       int32_t* converged) {
    if (!(alpha > 0.0f && alpha < 1.0f) || max_iter < 0 || pushes == nullptr) return PPR_EINVAL;
    const double q = 1.0 - (double)alpha;
    int32_t T;
    int32_t conv = 1;
    if (!(tol > 0.0)) {
        T = max_iter;
    } else if (tol >= 1.0) {
        T = 0;
    } else {
        double t = ceil(log(tol) / log(q));
        if (t < 0) t = 0;
        if (t > 2.0e9) t = 2.0e9;
        int64_t ti = (int64_t)t;
        while (ti > 0 && pow(q, (double)(ti - 1)) <= tol) --ti;
        while (pow(q, (double)ti) > tol) ++ti;
        if (ti > max_iter) {
            T = max_iter;
            conv = 0;
        } else {
            T = (int32_t)ti;
        }
    }
    *pushes = T;
    if (converged) *converged = conv;
    return PPR_OK;
}


size_t ppr_matrix_workspace(const ppr_csr* g, int32_t n_src, int32_t n_tgt) {
    (void)n_tgt;
    if (g == nullptr || g->n < 1 || n_src < 0) return 0;
    WsSize c;
    ppr_ws_layout(c, g->n, g->nnz, g->weight != nullptr, n_src, nullptr);
    return c.used;
}

size_t ppr_matrix_workspace_fast(const ppr_csr* g, int32_t n_src, int32_t n_tgt) {
    if (g == nullptr || g->n < 1 || n_src < 0) return 0;
    WsSize c;
    ppr_ws_layout(c, g->n, g->nnz, g->weight != nullptr, n_src, nullptr);
    ppr_extra_layout(c, g->n, n_src, n_src == n_tgt, nullptr);
    return c.used;
}

ppr_status ppr_matrix(const ppr_csr* g, const int32_t* src, int32_t n_src, const int32_t* tgt,
                      int32_t n_tgt, float alpha, double tol_l1, int32_t max_iter, float* ppr_out,
                      float* dppr_out, double* resid_out, int32_t* iters_out, void* ws, size_t ws_bytes,
                      void* stream) {
    return ppr_matrix_impl(g, src, n_src, tgt, n_tgt, alpha, tol_l1, max_iter, ppr_out, dppr_out, resid_out,
                           iters_out, ws, ws_bytes, stream, false);
}

size_t ppr_matrix_noalloc_max_scratch(void) { return kScratchBytes; }

ppr_status ppr_matrix_noalloc(const ppr_csr* g, const int32_t* src, int32_t n_src, const int32_t* tgt,
                              int32_t n_tgt, float alpha, double tol_l1, int32_t max_iter, float* ppr_out,
                              float* dppr_out, double* resid_out, int32_t* iters_out, void* stream) {
    // The workspace bound is checked before the scratch address is looked up,
    // so an oversized request fails without touching the device.
    ppr_status st = validate_csr(g);
    if (st != PPR_OK) return st;
    if (n_src < 0) return PPR_EINVAL;
    if (ppr_matrix_workspace(g, n_src, n_tgt) > kScratchBytes) return PPR_EUNSUPPORTED;
    void* scr = nullptr;
    st = scratch_address(static_cast<hipStream_t>(stream), &scr);
    if (st != PPR_OK) return st;
    return ppr_matrix_impl(g, src, n_src, tgt, n_tgt, alpha, tol_l1, max_iter, ppr_out, dppr_out, resid_out,
                           iters_out, scr, kScratchBytes, stream, true);
}

}  // extern "C"
