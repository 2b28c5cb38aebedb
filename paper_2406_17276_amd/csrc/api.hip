// C ABI of libopttree: argument validation, workspace carving and kernel sequencing.
// No arithmetic of the method lives here.
#include <string.h>

#include <algorithm>

#include "common.hpp"
#include "internal.h"

namespace ot {

static thread_local int g_last_hip_error = 0;
void set_last_hip_error(int e) { g_last_hip_error = e; }

Frontier make_frontier(int k, int n, int depth) {
    Frontier f;
    memset(&f, 0, sizeof(f));
    f.F[0] = 1;
    f.row_start[0] = 0;
    long long rows = 0, pool = 0;
    for (int t = 0; t < depth; ++t) {
        rows += f.F[t];
        f.row_start[t + 1] = (int)rows;
        const long long next = (long long)k * f.F[t];
        f.F[t + 1] = (int)(next < n ? next : n);
        pool += f.F[t + 1];
    }
    f.rows = (int)rows;
    f.pool = (int)pool;
    return f;
}

static size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

static int validate_build(const ot_build_params* p, bool check_strides) {
    if (!p) return OT_ERR_INVALID_ARG;
    if (p->batch < 1 || p->vocab < 1 || p->depth < 1 || p->k < 1 || p->n < 1) return OT_ERR_INVALID_ARG;
    if (p->k > p->vocab) return OT_ERR_INVALID_ARG;
    if (p->logits_dtype != OT_F32 && p->logits_dtype != OT_BF16) return OT_ERR_INVALID_ARG;
    if (p->k > OT_MAX_TOPK || p->n > OT_MAX_NODES || p->depth > OT_MAX_DEPTH) return OT_ERR_UNSUPPORTED;
    if (p->vocab > kMaxVocab) return OT_ERR_UNSUPPORTED;
    if (check_strides) {
        if (p->stride_row < p->vocab || p->stride_depth < 0 || p->stride_seq < 0) return OT_ERR_INVALID_ARG;
    }
    return OT_OK;
}

BuildWorkspace carve_build_workspace(const ot_build_params& p, void* base) {
    const Frontier f = make_frontier(p.k, p.n, p.depth);
    const size_t rows = (size_t)p.batch * (size_t)(f.rows > p.n ? f.rows : p.n);
    const size_t parts = (size_t)max_scan_parts(p.vocab);
    const size_t k = (size_t)p.k;
    const size_t pool = (size_t)p.batch * p.depth * p.n;
    BuildWorkspace w;
    memset(&w, 0, sizeof(w));
    size_t off = 0;
    char* b = (char*)base;
    // (a null base is the sizing pass: offsets only)
    auto take = [&](size_t bytes) { char* q = b ? b + off : nullptr; off = align_up(off + bytes, 256); return (void*)q; };
    w.row_lse = (double*)take(rows * 8);
    w.row_topv = (float*)take(rows * k * 4);
    w.row_topi = (int32_t*)take(rows * k * 4);
    if (parts > 1) {
        w.part_m = (float*)take(rows * parts * 4);
        w.part_s = (double*)take(rows * parts * 8);
        w.part_topv = (float*)take(rows * parts * k * 4);
        w.part_topi = (int32_t*)take(rows * parts * k * 4);
    }
    w.pool_key = (double*)take(pool * 8);
    w.step_tau = (double*)take((size_t)p.batch * p.depth * 8);
    w.pool_tok = (int32_t*)take(pool * 4);
    w.pool_par = (int32_t*)take(pool * 4);
    w.pool_p = (double*)take(pool * 8);
    w.seq_E = (double*)take((size_t)p.batch * 8);
    w.seq_steps = (int32_t*)take((size_t)p.batch * 4);
    w.seq_active = (int32_t*)take((size_t)p.batch * 4);
    w.front_anc = (unsigned short*)take((size_t)2 * p.batch * p.n * OT_MAX_DEPTH * sizeof(unsigned short));
    w.bytes = off;
    return w;
}

static int check_tree_out(const ot_tree_out* o) {
    if (!o || !o->token || !o->parent || !o->depth || !o->score || !o->mask || !o->n_out || !o->expect)
        return OT_ERR_INVALID_ARG;
    if (((uintptr_t)o->mask % 8) || ((uintptr_t)o->expect % 8)) return OT_ERR_INVALID_ARG;
    return OT_OK;
}

static SelectGeometry select_geometry(const ot_build_params& p, const Frontier& f) {
    SelectGeometry g;
    g.batch = p.batch; g.k = p.k; g.n = p.n; g.depth = p.depth;
    g.rows_per_seq = f.rows;
    for (int i = 0; i < OT_MAX_DEPTH + 2; ++i) { g.F[i] = f.F[i]; g.row_start[i] = f.row_start[i]; }
    return g;
}

}  // namespace ot

using namespace ot;

extern "C" {

int ot_version(void) { return 100; }

const char* ot_status_string(int status) {
    switch (status) {
        case OT_OK: return "ok";
        case OT_ERR_INVALID_ARG: return "invalid argument";
        case OT_ERR_UNSUPPORTED: return "unsupported size or type";
        case OT_ERR_WORKSPACE_TOO_SMALL: return "workspace too small";
        case OT_ERR_HIP: return "HIP runtime error";
        case OT_ERR_SCRATCH_LIMIT: return "needs more scratch memory than the no-allocation entry point owns";
        default: return "unknown status";
    }
}

int ot_last_hip_error(void) { return g_last_hip_error; }

size_t ot_build_workspace_bytes(const ot_build_params* p) {
    if (validate_build(p, false) != OT_OK) return 0;
    return carve_build_workspace(*p, nullptr).bytes;
}

// One-shot build: the rows of all steps are scanned, then the tree is drafted from their statistics.  A tree is usually
// complete long before the last step (tree_draft.hpp), so big inputs go in chunks of steps: scan a chunk, draft it, and
// leave the rows of finished sequences unread from then on.  A chunk costs two more launches and another pass over the
// pool, 8 to 14 us on the stream, which is all that it brings where no tree is complete before the last step (rows in which
// one token has nearly all of the probability).  So a chunk has at least 192 MB of rows, some 35 us of reading, and later
// ones half of what was read before, up to 1 GB, and a sixth of it.  Measured, us, trees that stay open / trees complete
// after half of the steps: one launch, chunks of 96 MB and a sixth, this rule (n = 60, k = 8, 10 steps, 32000 tokens):
// 8 sequences 63 / 54, 76 / 40, 63 / 54; 16: 102 / 94, 146 / 76, 115 / 60; 32: 180 / 174, 255 / 148, 206 / 126;
// 64: 332 / 326, 408 / 214, 374 / 219; n = 256, k = 16, 20 steps, 8 sequences of 128256 tokens: 1496 / 1439, 1739 / 515,
// 1619 / 523.
static long long chunk_bytes(long long before) {
    const long long mb = 1ll << 20;
    return std::max({192 * mb, std::min(before / 2, 1024 * mb), before / 6});
}

// Polls of a drafting workgroup for a row, some 30 ms: longer than any launch that has the chip to itself takes
constexpr int kArrivalPolls = 30000;

static int build_steps(const ot_build_params* p, bool adapt, double delta, const void* logits, void* workspace,
                       size_t workspace_bytes, const ot_tree_out* out, int32_t* steps_used, double* e_sub, void* hip_stream,
                       void* ev0, void* ev1, int polls = kArrivalPolls, int32_t* one_launch = nullptr) {
    int st = validate_build(p, true);
    if (st != OT_OK) return st;
    if (!logits || !workspace) return OT_ERR_INVALID_ARG;
    if ((uintptr_t)workspace % 16) return OT_ERR_INVALID_ARG;
    const int esize = p->logits_dtype == OT_BF16 ? 2 : 4;
    if ((uintptr_t)logits % esize) return OT_ERR_INVALID_ARG;
    st = check_tree_out(out);
    if (st != OT_OK) return st;
    const BuildWorkspace ws = carve_build_workspace(*p, workspace);
    if (workspace_bytes < ws.bytes) return OT_ERR_WORKSPACE_TOO_SMALL;
    const Frontier f = make_frontier(p->k, p->n, p->depth);
    const SelectGeometry g = select_geometry(*p, f);
    hipStream_t s = (hipStream_t)hip_stream;

    ScanGeometry sg;
    sg.batch = p->batch; sg.vocab = p->vocab; sg.k = p->k; sg.dtype = p->logits_dtype;
    sg.nsteps = p->depth; sg.rows_per_seq = f.rows;
    sg.grow_k = p->k; sg.grow_n = p->n;
    sg.stride_seq = p->stride_seq; sg.stride_depth = p->stride_depth; sg.stride_row = p->stride_row;
    const long long row_bytes = (long long)p->batch * p->vocab * esize;
    for (int t0 = 0; t0 < p->depth;) {
        int t1 = t0 + 1;
        const long long least = chunk_bytes(f.row_start[t0] * row_bytes);
        while (t1 < p->depth && (f.row_start[t1] - f.row_start[t0]) * row_bytes < least) ++t1;
        if ((f.rows - f.row_start[t1]) * row_bytes < least) t1 = p->depth;
        if (ev0 || ev1) t1 = p->depth;                         // the timed form brackets one scan of everything
        sg.row0 = f.row_start[t0]; sg.rows = f.row_start[t1] - f.row_start[t0];
        const bool fused = t0 == 0 && t1 == p->depth && !ev0 && !ev1 && fuse_build(sg, g, logits);
        if (one_launch) *one_launch = fused;
        if (fused)
            return launch_fused_build(sg, g, logits, adapt, delta, ws, *out, steps_used, e_sub, polls, s);
        st = launch_row_scan(sg, logits, ws, s, (hipEvent_t)ev0, (hipEvent_t)ev1, t0 > 0);
        if (st != OT_OK) return st;
        st = launch_tree_build(g, t0, t1, adapt, delta, ws, *out, steps_used, e_sub, s);
        if (st != OT_OK) return st;
        t0 = t1;
    }
    return OT_OK;
}

int ot_build_tree(const ot_build_params* p, const void* logits, void* workspace, size_t workspace_bytes,
                  const ot_tree_out* out, void* hip_stream) {
    return build_steps(p, false, 0.0, logits, workspace, workspace_bytes, out, nullptr, nullptr, hip_stream, nullptr, nullptr);
}

int ot_internal_build_tree(const ot_build_params* p, int32_t adapt, double delta, const void* logits, void* workspace,
                           size_t workspace_bytes, const ot_tree_out* out, int32_t* steps_used, double* e_sub, int32_t polls,
                           int32_t* one_launch, void* hip_stream) {
    if (adapt && (!(delta == delta) || !steps_used || !e_sub)) return OT_ERR_INVALID_ARG;
    return build_steps(p, adapt != 0, delta, logits, workspace, workspace_bytes, out, steps_used, e_sub, hip_stream, nullptr, nullptr,
                       polls, one_launch);
}

int ot_build_tree_timed(const ot_build_params* p, const void* logits, void* workspace, size_t workspace_bytes,
                        const ot_tree_out* out, void* hip_stream, void* scan_begin_event, void* scan_end_event) {
    return build_steps(p, false, 0.0, logits, workspace, workspace_bytes, out, nullptr, nullptr, hip_stream, scan_begin_event,
                       scan_end_event);
}

int ot_build_tree_adaptive(const ot_build_params* p, double delta, const void* logits, void* workspace,
                           size_t workspace_bytes, const ot_tree_out* out, int32_t* steps_used, double* e_sub,
                           void* hip_stream) {
    int st = validate_build(p, true);
    if (st != OT_OK) return st;
    if (!(delta == delta)) return OT_ERR_INVALID_ARG;
    if (!steps_used || !e_sub || (uintptr_t)steps_used % 4 || (uintptr_t)e_sub % 8) return OT_ERR_INVALID_ARG;
    return build_steps(p, true, delta, logits, workspace, workspace_bytes, out, steps_used, e_sub, hip_stream, nullptr, nullptr);
}

static int begin_entry(const ot_build_params* p, void* workspace, size_t workspace_bytes, int32_t* frontier_token,
                       int32_t* frontier_parent, int32_t* frontier_count, void* hip_stream) {
    int st = validate_build(p, false);
    if (st != OT_OK) return st;
    if (!workspace || (uintptr_t)workspace % 16) return OT_ERR_INVALID_ARG;
    const BuildWorkspace ws = carve_build_workspace(*p, workspace);
    if (workspace_bytes < ws.bytes) return OT_ERR_WORKSPACE_TOO_SMALL;
    // every step overwrites the pool state it owns; only the per-sequence loop state (E = 0, no layer, not
    // stopped) has to be set
    return launch_tree_begin(select_geometry(*p, make_frontier(p->k, p->n, p->depth)), ws, (hipStream_t)hip_stream, frontier_token,
                             frontier_parent, frontier_count);
}

int ot_tree_begin(const ot_build_params* p, void* workspace, size_t workspace_bytes, void* hip_stream) {
    return begin_entry(p, workspace, workspace_bytes, nullptr, nullptr, nullptr, hip_stream);
}

int ot_internal_tree_begin(const ot_build_params* p, void* workspace, size_t workspace_bytes, int32_t* frontier_token,
                           int32_t* frontier_parent_slot, int32_t* frontier_count, void* hip_stream) {
    if (!frontier_token || !frontier_parent_slot || !frontier_count) return OT_ERR_INVALID_ARG;
    return begin_entry(p, workspace, workspace_bytes, frontier_token, frontier_parent_slot, frontier_count, hip_stream);
}

int ot_tree_expand(const ot_build_params* p, int32_t step, const void* rows, int64_t stride_seq, int64_t stride_row,
                   void* workspace, size_t workspace_bytes, int32_t* frontier_token, int32_t* frontier_parent_slot,
                   int32_t* frontier_count, void* hip_stream) {
    int st = validate_build(p, false);
    if (st != OT_OK) return st;
    if (step < 0 || step >= p->depth) return OT_ERR_INVALID_ARG;
    if (!rows || !workspace || !frontier_token || !frontier_parent_slot) return OT_ERR_INVALID_ARG;
    if ((uintptr_t)workspace % 16) return OT_ERR_INVALID_ARG;
    if (((uintptr_t)frontier_token % 4) || ((uintptr_t)frontier_parent_slot % 4) || ((uintptr_t)frontier_count % 4))
        return OT_ERR_INVALID_ARG;
    const int esize = p->logits_dtype == OT_BF16 ? 2 : 4;
    if ((uintptr_t)rows % esize) return OT_ERR_INVALID_ARG;
    if (stride_row < p->vocab || stride_seq < 0) return OT_ERR_INVALID_ARG;
    const BuildWorkspace ws = carve_build_workspace(*p, workspace);
    if (workspace_bytes < ws.bytes) return OT_ERR_WORKSPACE_TOO_SMALL;
    const Frontier f = make_frontier(p->k, p->n, p->depth);
    hipStream_t s = (hipStream_t)hip_stream;

    ScanGeometry sg;
    sg.batch = p->batch; sg.vocab = p->vocab; sg.k = p->k; sg.dtype = p->logits_dtype;
    sg.nsteps = 1; sg.rows_per_seq = f.F[step]; sg.row0 = 0; sg.rows = f.F[step];
    sg.grow_k = 1; sg.grow_n = 1;
    sg.stride_seq = stride_seq; sg.stride_depth = 0; sg.stride_row = stride_row;
    SelectGeometry g = select_geometry(*p, f);
    g.rows_per_seq = f.F[step];
    if (fuse_expand(sg, p->n, rows))
        return launch_fused_expand(sg, g, rows, step, ws, frontier_token, frontier_parent_slot, frontier_count, s);
    st = launch_row_scan(sg, rows, ws, s, nullptr, nullptr, true);      // rows of frozen sequences are not read
    if (st != OT_OK) return st;
    return launch_tree_step(g, step, ws, frontier_token, frontier_parent_slot, frontier_count, s);
}

int ot_tree_finalize(const ot_build_params* p, int32_t steps_done, void* workspace, size_t workspace_bytes,
                     const ot_tree_out* out, void* hip_stream) {
    int st = validate_build(p, false);
    if (st != OT_OK) return st;
    if (steps_done < 1 || steps_done > p->depth) return OT_ERR_INVALID_ARG;
    if (!workspace || (uintptr_t)workspace % 16) return OT_ERR_INVALID_ARG;
    st = check_tree_out(out);
    if (st != OT_OK) return st;
    const BuildWorkspace ws = carve_build_workspace(*p, workspace);
    if (workspace_bytes < ws.bytes) return OT_ERR_WORKSPACE_TOO_SMALL;
    const Frontier f = make_frontier(p->k, p->n, p->depth);
    return launch_tree_finalize(select_geometry(*p, f), steps_done, ws, *out, (hipStream_t)hip_stream);
}

int ot_tree_frontier_mask(const ot_build_params* p, int32_t steps_done, void* workspace, size_t workspace_bytes,
                          uint64_t* mask, void* hip_stream) {
    int st = validate_build(p, false);
    if (st != OT_OK) return st;
    if (steps_done < 1 || steps_done > p->depth) return OT_ERR_INVALID_ARG;
    if (!workspace || (uintptr_t)workspace % 16 || !mask || (uintptr_t)mask % 8) return OT_ERR_INVALID_ARG;
    const BuildWorkspace ws = carve_build_workspace(*p, workspace);
    if (workspace_bytes < ws.bytes) return OT_ERR_WORKSPACE_TOO_SMALL;
    const Frontier f = make_frontier(p->k, p->n, p->depth);
    return launch_tree_front_mask(select_geometry(*p, f), steps_done, ws, mask, OT_MASK_WORDS(p->depth * p->n),
                                  (hipStream_t)hip_stream);
}

int ot_tree_esub(const ot_build_params* p, int32_t steps_done, double delta, void* workspace, size_t workspace_bytes,
                 double* e_sub, int32_t* go_on, void* hip_stream) {
    int st = validate_build(p, false);
    if (st != OT_OK) return st;
    if (steps_done < 1 || steps_done > p->depth) return OT_ERR_INVALID_ARG;
    if (!(delta == delta)) return OT_ERR_INVALID_ARG;
    if (!workspace || (uintptr_t)workspace % 16 || !e_sub || !go_on) return OT_ERR_INVALID_ARG;
    if ((uintptr_t)e_sub % 8 || (uintptr_t)go_on % 4) return OT_ERR_INVALID_ARG;
    const BuildWorkspace ws = carve_build_workspace(*p, workspace);
    if (workspace_bytes < ws.bytes) return OT_ERR_WORKSPACE_TOO_SMALL;
    const Frontier f = make_frontier(p->k, p->n, p->depth);
    return launch_tree_esub(select_geometry(*p, f), steps_done, delta, ws, e_sub, go_on, (hipStream_t)hip_stream);
}

}  // extern "C"
