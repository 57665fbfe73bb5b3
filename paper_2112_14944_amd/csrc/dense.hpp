// Dense FP32 products on the matrix cores (v_mfma_f32_32x32x2_f32), one tile
// of C[i][j] = sum_k A[k][i] f_k B[k][j] per block: both operands are read
// row by row along k, so that every load is a contiguous row segment and LDS
// needs no transposition.  Two users: the adjoint of the weight gradient
// (grad.hip) and the products of the all-pairs PPR (ppr_dense.hpp).
//
// FP32 products and FP32 accumulation throughout: an element is summed in
// ascending k, two terms per instruction, whatever the tile size, so a tile
// size never changes a result.
//
// Bound: the matrix cores.  A 32x32x2 instruction takes 64 cycles on its
// SIMD (256 CUs x 4 SIMDs x 4096 FLOP / 64 cycles at 2.4 GHz = 157 TFLOP/s)
// and needs one 4-byte LDS read per operand block, so LDS, loads and address
// arithmetic all fit beside it; what matters is that a SIMD always has a next
// instruction to issue, which two to four waves per SIMD give, with a step's
// loads and LDS writes dealt out between its products.  n = 8192: 117 TFLOP/s
// with 16 rows per step, loads before and LDS writes after the products; 127
// with 32 rows per step; 132 now (matrix units busy 86% of the cycles; waves as
// priorities or two steps of loads ahead changed nothing).  n = 2048, 64-wide
// tiles: 136, 133 and 125 us.
#pragma once

#include "common.hpp"

namespace pprviz {

typedef float DenseAcc __attribute__((ext_vector_type(16)));

// k rows staged per step, so that a step's products outweigh its LDS latency
// and barrier.
constexpr int kDenseK = 32;
constexpr int kDenseThreads = 256;

// Staged k rows, BT columns each.  Odd rows hold column c at c ^ 32, so that
// the two k rows a 32x32x2 operand read touches (lanes 0-31 and 32-63) fall
// into different halves of the 64 LDS banks.
template <int BT>
struct DenseLds {
    float a[2][kDenseK][BT];
    float b[2][kDenseK][BT];
};

// Wave tile: 4 waves as 2 x 2, each (BT/2) x (BT/2) as NB x NB blocks of 32.
template <int BT>
struct DenseTile {
    static constexpr int NB = BT / 64;
    DenseAcc c[NB][NB];
};

// Where lane l holds element r of a 32x32 block: row (r % 4) + 8 (r / 4) +
// 4 (l / 32), column l % 32.
__device__ __forceinline__ int dense_row(int r, int lane) { return (r & 3) + 8 * (r >> 2) + 4 * (lane >> 5); }

// Rows k of an operand from k0 on: the resource ends with the operand's last
// row, so that rows past K read zeros; columns past the row's end read the
// next row (or zeros) and only reach elements of C outside the matrix.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t dense_rows(const float* p, int64_t ld, int K, int k0) {
    const int64_t bytes = k0 < K ? (int64_t)(K - k0) * ld * 4 : 0;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p + (int64_t)k0 * ld), 0,
                                             (int)(bytes < 0x7fffffff ? bytes : 0x7fffffff), 0x00020000);
}

// C tile (i0, j0) over k in [0, K).  A and B row-major with leading
// dimensions lda, ldb (wave-uniform).  f_k = scale * (deg[k] > 0 ? deg[k] : 1)
// multiplies B's rows.  CHUNKS > 0: the running sum is set aside every CHUNKS
// staged steps and the parts added up, so that a long sum's error does not
// grow with all of its K terms one after another.
template <int BT, int CHUNKS>
__device__ __forceinline__ void dense_tile(const float* __restrict__ A, int64_t lda, const float* __restrict__ B,
                                           int64_t ldb, const float* __restrict__ deg, float scale, int K, int i0,
                                           int j0, DenseLds<BT>& L, DenseTile<BT>& out) {
    constexpr int NB = DenseTile<BT>::NB;
    constexpr int RP = kDenseThreads / BT;  // k rows one pass of the block loads
    constexpr int NP = kDenseK / RP;        // passes per staged step
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wi = (wave >> 1) * (BT / 2), wj = (wave & 1) * (BT / 2);
    const int lc = tid % BT;
    const int lr = __builtin_amdgcn_readfirstlane(tid / BT);
    const int half = lane >> 5, l32 = lane & 31;
    const __amdgpu_buffer_rsrc_t dr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(deg), 0, K * 4, 0x00020000);
    DenseAcc c[NB][NB];
#pragma unroll
    for (int p = 0; p < NB; ++p)
#pragma unroll
        for (int q = 0; q < NB; ++q) {
#pragma unroll
            for (int r = 0; r < 16; ++r) c[p][q][r] = 0.f;
            if (CHUNKS > 0) out.c[p][q] = c[p][q];
        }
    // Operand rows travel through registers, PD staged steps ahead of their
    // use: the loads of step s + PD are issued in the first half of step s's
    // arithmetic, and the set of step s + 1 is written to LDS in the second. A
    // 128-wide tile's half step (32 instructions of 64 cycles per wave) covers a
    // load's way to memory and back by itself; a 64-wide tile's (8 of them) does
    // not.
    constexpr int PD = NB == 1 ? 2 : 1;
    // Operand reads ahead of their products, in pairs of k rows: an LDS read
    // takes longer than the one instruction per pair of a 64-wide tile.
    constexpr int OD = NB == 1 ? 4 : 1;
    float ra[PD][NP], rb[PD][NP], rd[PD];  // rd: lane l holds deg of the step's row l % 32
    __amdgpu_buffer_rsrc_t ar, br;
    auto fetch = [&](int s, int set, int p0, int p1) {
        const int k0 = s * kDenseK;
        if (p0 == 0) {
            ar = dense_rows(A, lda, K, k0);
            br = dense_rows(B, ldb, K, k0);
            rd[set] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(dr, (k0 + l32) * 4, 0, 0));
        }
#pragma unroll
        for (int p = p0; p < p1; ++p) {
            const int row = lr + p * RP;
            ra[set][p] =
                __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ar, (int)((row * lda + i0 + lc) * 4), 0, 0));
            rb[set][p] =
                __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(br, (int)((row * ldb + j0 + lc) * 4), 0, 0));
        }
        asm volatile("" ::: "memory");
    };
    static_assert(kDenseK == 32, "rd: one lane per row of a step");
    auto stage = [&](int buf, int set, int p0, int p1) {
        const float f = scale * (rd[set] > 0.f ? rd[set] : 1.0f);
#pragma unroll
        for (int p = p0; p < p1; ++p) {
            const int row = lr + p * RP, col = lc ^ (32 * (row & 1));
            L.a[buf][row][col] = ra[set][p];
            L.b[buf][row][col] =
                rb[set][p] * __int_as_float(__builtin_amdgcn_readlane(__float_as_int(f), row));
        }
    };
    const int steps = (K + kDenseK - 1) / kDenseK;
    auto step = [&](int s, int set) {  // set: s % 2, and s & 1 the LDS buffer
        constexpr int G = kDenseK / 4;
        const int buf = set;
        float av[OD + 1][NB], bv[OD + 1][NB];
        auto operands = [&](int kk, int w) {
#pragma unroll
            for (int p = 0; p < NB; ++p) {
                av[w][p] = L.a[buf][kk + half][((wi + 32 * p) ^ (32 * half)) + l32];
                bv[w][p] = L.b[buf][kk + half][((wj + 32 * p) ^ (32 * half)) + l32];
            }
        };
#pragma unroll
        for (int i = 0; i < OD; ++i) operands(2 * i, i);
#pragma unroll
        for (int kk = 0; kk < kDenseK; kk += 2) {
            const int w = (kk >> 1) % (OD + 1);
            if (kk + 2 * OD < kDenseK) operands(kk + 2 * OD, (w + OD) % (OD + 1));
            const int g = kk >> 1;
            if (g < G)
                fetch(s + PD, set % PD, g * NP / G, (g + 1) * NP / G);  // past the last row: zeros, no memory access
            else
                stage(buf ^ 1, (set + 1) % PD, (g - G) * NP / G, (g - G + 1) * NP / G);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int p = 0; p < NB; ++p)
#pragma unroll
                for (int q = 0; q < NB; ++q)
                    c[p][q] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[w][p], bv[w][q], c[p][q], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (CHUNKS > 0 && ((s + 1) % (CHUNKS > 0 ? CHUNKS : 1) == 0 || s + 1 == steps)) {
#pragma unroll
            for (int p = 0; p < NB; ++p)
#pragma unroll
                for (int q = 0; q < NB; ++q)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        out.c[p][q][r] += c[p][q][r];
                        c[p][q][r] = 0.f;
                    }
        }
        __syncthreads();
    };
#pragma unroll
    for (int i = 0; i < PD; ++i) fetch(i, i, 0, NP);
    __syncthreads();  // the previous tile's readers are done with the buffers
    stage(0, 0, 0, NP);
    __syncthreads();
    int s = 0;
    for (; s + 1 < steps; s += 2) {
        step(s, 0);
        step(s + 1, 1);
    }
    if (s < steps) step(s, 0);
    if (CHUNKS == 0) {
#pragma unroll
        for (int p = 0; p < NB; ++p)
#pragma unroll
            for (int q = 0; q < NB; ++q) out.c[p][q] = c[p][q];
    }
}

// Calls f(i, j, value) for every element of the tile this lane holds.
template <int BT, typename F>
__device__ __forceinline__ void dense_each(const DenseTile<BT>& t, int i0, int j0, F f) {
    constexpr int NB = DenseTile<BT>::NB;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int wi = i0 + (wave >> 1) * (BT / 2), wj = j0 + (wave & 1) * (BT / 2);
#pragma unroll
    for (int p = 0; p < NB; ++p)
#pragma unroll
        for (int q = 0; q < NB; ++q)
#pragma unroll
            for (int r = 0; r < 16; ++r) f(wi + 32 * p + dense_row(r, lane), wj + 32 * q + (lane & 31), t.c[p][q][r]);
}

}  // namespace pprviz
