// Host-side functions and workspace layouts shared between the library's
// translation units.
#pragma once

#include <algorithm>

#include "common.hpp"
#include "ppr_core.hpp"
#include "ppr_dense.hpp"
#include "ppr_mid.hpp"
#include "ppr_query.hpp"
#include "ppr_stream.hpp"

namespace pprviz {

// Workspace of the forward PPR (ppr_matrix, and the recompute inside
// ppr_matrix_backward).  Only the buffers of the kernel that n selects are
// taken, unless the streaming buffers are asked for as well.
struct PprWs {
    RowEnt* rows;
    ResSlot* slots;  // resident tile: slot table
    float* deg;
    float* invd;
    double* resid;
    int32_t* col_r;  // resident tile: arc copy in group layout
    float* w_r;
    int32_t* sorted_r;  // resident tile: arcs grouped by LDS bank class (layout staging)
    float* sorted_w;
    MidWs mid;       // mid-size kernel: plan and arc stream
    float* ya;       // streaming SpMM: iterate ping-pong
    float* yb;
    double* part;
    int32_t* hist;
    float* series;   // all-pairs series (ppr_extra_layout), nullptr: not taken
    QueryWs query;   // iterate in HBM; ya == nullptr: not taken
};

// Bytes a call's fastest route needs beyond ppr_ws_layout (none of them is
// needed: without them the call takes its general route):
//  - all pairs of 192 to 2304 nodes: 4 n^2 floats of the series;
//  - a few sources of a graph that fits LDS: the iterate in HBM;
//  - targets that may be the sources (same): the pieces of the product that
//    halves the pushes.
constexpr int kQueryMaxSame = 8192;
template <typename Cursor>
void ppr_extra_layout(Cursor& c, int n, int n_src, bool same, PprWs* w) {
    float* series = nullptr;
    QueryWs q{};
    const bool lds = res_cols_for(n) != 0 || mid_cols_for(n) != 0;
    if (res_cols_for(n) != 0 && n >= kDenseMinN && n_src == n) {
        series = c.template take<float>((size_t)4 * n * n);
    } else if (lds && n_src > 0 && n_src <= kQueryMaxSrc && n_src < n) {
        const size_t ld = (size_t)query_ld(n_src);
        q.hist = c.template take<int32_t>(kDegKeys);
        q.refuse = c.template take<int32_t>(1);
        q.deg_sorted = c.template take<int32_t>((size_t)n);
        q.ya = c.template take<float>((size_t)n * ld);
        q.yb = c.template take<float>((size_t)n * ld);
        q.part = c.template take<double>((size_t)stream_resid_chunks(n) * ld);
    }
    if (same && n_src > 0 && (lds ? n_src <= kQueryMaxSrc && n_src < n : n_src <= kQueryMaxSame)) {
        q.pieces = query_pieces(n, n_src);
        q.gram = c.template take<float>(query_gram_floats(n, n_src));
        q.prod = c.template take<double>((size_t)n_src * n_src);
    }
    if (w) {
        w->series = series;
        if (!lds) {
            q.hist = w->hist;
            q.ya = w->ya;
            q.yb = w->yb;
            q.part = w->part;
        }
        w->query = q;
    }
}
// The extra buffers where the workspace has room for them: all, those without the
// product that halves the pushes, or none.
inline void ppr_extra_take(WsCursor& c, int n, int n_src, bool same, PprWs* w) {
    for (const bool product : {same, false}) {
        WsCursor t = c;
        ppr_extra_layout(t, n, n_src, product, w);
        if (t.used <= t.cap) {
            c = t;
            return;
        }
    }
    ppr_extra_layout(c, n, 0, false, w);
}

template <typename Cursor>
void ppr_ws_layout(Cursor& c, int n, int64_t nnz, bool weighted, int n_src, PprWs* w, bool with_stream = false) {
    PprWs t{};
    t.rows = c.template take<RowEnt>(n);
    t.deg = c.template take<float>(n);
    t.invd = c.template take<float>(n);
    t.resid = c.template take<double>(std::max(n_src, 1));
    const bool res = res_cols_for(n) != 0;
    const bool mid = mid_cols_for(n) != 0;
    if (res) {
        t.slots = c.template take<ResSlot>((size_t)n + kResTabPad);
        t.col_r = c.template take<int32_t>((size_t)res_arc_words(nnz, n));
        t.w_r = weighted ? c.template take<float>((size_t)res_arc_words(nnz, n)) : nullptr;
        t.sorted_r = c.template take<int32_t>((size_t)std::max<int64_t>(nnz, 1));
        t.sorted_w = weighted ? c.template take<float>((size_t)std::max<int64_t>(nnz, 1)) : nullptr;
    }
    if (mid) {
        const int64_t groups = mid_stream_groups(n, nnz);
        t.mid.rows = t.rows;
        t.mid.hist = c.template take<int32_t>(kMidKeys);
        t.mid.plan = c.template take<int32_t>(kPlanInts);
        t.mid.slice_goff = c.template take<int32_t>((size_t)mid_slices(n + kMidMaxParts));
        t.mid.slice_slot = c.template take<int32_t>((size_t)mid_slices(n + kMidMaxParts));
        t.mid.vrows = c.template take<RowEnt>((size_t)n + kMidMaxParts);
        t.mid.comb = c.template take<int4>(kMidMaxParts);
        t.mid.part_dst = c.template take<int32_t>(kMidWaves * kWave);
        t.mid.rowpos = c.template take<int32_t>(n);
        t.mid.vtab = c.template take<int2>((size_t)kMidWaves * kMidSlotCap * 64);
        t.mid.sell = c.template take<uint16_t>((size_t)(groups * kMidGroup));
        t.mid.sellw = weighted ? c.template take<float>((size_t)(groups * kMidGroup)) : nullptr;
        t.mid.tmp_u = c.template take<int32_t>((size_t)std::max<int64_t>(nnz, 1));
        t.mid.tmp_w = weighted ? c.template take<float>((size_t)std::max<int64_t>(nnz, 1)) : nullptr;
    }
    if ((!res && !mid) || with_stream) {
        const int64_t ldy = stream_ld(with_stream ? n : n_src);
        t.ya = c.template take<float>((size_t)n * ldy);
        t.yb = c.template take<float>((size_t)n * ldy);
        t.part = c.template take<double>((size_t)stream_resid_chunks(n) * ldy);
        t.hist = c.template take<int32_t>(kDegKeys);
    }
    if (w) *w = t;
}

// Scratch memory of ppr_matrix_noalloc (noalloc.hip): kScratchBytes for the
// workspace proper, then room for the buffers of the faster routes.  It fits the
// all-pairs series of the resident range's largest size; a query that needs more
// (a few sources of a nearly edgeless graph of 30000 nodes and up) goes without
// the product, or takes a general route.
constexpr size_t kScratchBytes = size_t(8) << 20;
constexpr size_t kScratchExtraBytes = size_t(4) * Res<16>::NMAX * Res<16>::NMAX * sizeof(float);
ppr_status scratch_address(hipStream_t s, void** out);

ppr_status validate_csr(const ppr_csr* g);
bool use_resident(int n);
void launch_degree(const int32_t* row_ptr, const float* weight, int64_t n, float* deg, float* invd,
                   hipStream_t s);
void ppr_forward(const ppr_csr* g, const int32_t* src, int32_t n_src, const int32_t* tgt, int32_t n_tgt,
                 float alpha, int32_t T, float* ppr_out, float* dppr_out, const float* deg, const float* invd,
                 double* resid, const PprWs& w, hipStream_t s);
void launch_res_layout(const int32_t* row_ptr, const int32_t* col_idx, const float* weight, const float* invd,
                       const int64_t* node_off, int32_t n_single, int32_t blocks, ResSlot* slots, int32_t* arcs,
                       float* warcs, int32_t* sorted, float* wsorted, hipStream_t s);

}  // namespace pprviz
