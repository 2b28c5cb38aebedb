// Launches of the one-shot tree construction (tree_draft.hpp).
#include <algorithm>

#include "tree_draft.hpp"

namespace ot {
namespace {

template <int NT, int KPT, bool STAGE, bool ADAPT>
__global__ __launch_bounds__(NT) void tree_build_kernel(const float* topv, const double* row_lse, const int k, const int rows,
                                                        const int n, const int depth, const int t0, const int t1,
                                                        const TreeBuildArgs a) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ Shared<NT> s;
    const int b = blockIdx.x;
    if (t0 > 0 && a.seq_active[b] == 0) return;
    draft_tree<NT, KPT, STAGE ? kStaged : kStep, ADAPT>(s, smem, NT, b, topv, row_lse, k, rows, n, depth, t0, t1, a, Arrivals{});
}


template <int NT, int KPT, bool STAGE, bool ADAPT>
int launch_t(const TreeBuildArgs& a, const SelectGeometry& g, const BuildWorkspace& ws, int t0, int t1, size_t lds, hipStream_t s) {
    if (lds + sizeof(Shared<NT>) > 64 * 1024)
        OT_HIP_CHECK(hipFuncSetAttribute((const void*)tree_build_kernel<NT, KPT, STAGE, ADAPT>,
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    const int per = sequences_per_launch(g.batch, NT);
    for (size_t b = 0; b < (size_t)g.batch; b += per) {
        const size_t rows = b * g.rows_per_seq, pool = b * a.batch_pool, nodes = b * g.n, words = nodes * OT_MASK_WORDS(g.n);
        TreeBuildArgs c = a;
        c.topi += rows * g.k;
        c.pool_key += pool; c.pool_meta += pool; c.pool_par += pool;
        if (c.seq_active) c.seq_active += b;
        c.seq_E += b;
        if (ADAPT) { c.steps_used += b; c.e_sub += b; }
        c.out.token += nodes; c.out.parent += nodes; c.out.depth += nodes; c.out.score += nodes; c.out.mask += words;
        c.out.n_out += b; c.out.expect += b;
        hipLaunchKernelGGL((tree_build_kernel<NT, KPT, STAGE, ADAPT>), dim3(std::min<size_t>(per, g.batch - b)), dim3(NT), lds, s,
                           ws.row_topv + rows * g.k, ws.row_lse + rows, g.k, g.rows_per_seq, g.n, g.depth, t0, t1, c);
        OT_HIP_CHECK(hipGetLastError());
    }
    return OT_OK;
}

template <int NT, int KPT>
int launch_n(TreeBuildArgs& a, const SelectGeometry& g, const BuildWorkspace& ws, int t0, int t1, bool adapt, hipStream_t s) {
    const int rows = g.row_start[t1] - g.row_start[t0];
    const size_t base = pool_bytes(a.batch_pool) + 16;
    const size_t tv = ((size_t)rows * g.k * 4 + 15) / 16 * 16, stage = tv + (size_t)rows * 8;
    a.stage_off_lse = (int)tv;
    if (base + sizeof(Shared<NT>) > kLdsLimit) return OT_ERR_UNSUPPORTED;
    // a single step has nothing to overlap with: its candidates go straight to registers
    if (t1 - t0 > 1 && base + stage + sizeof(Shared<NT>) <= kLdsLimit) {
        return adapt ? launch_t<NT, KPT, true, true>(a, g, ws, t0, t1, base + stage, s)
                     : launch_t<NT, KPT, true, false>(a, g, ws, t0, t1, base + stage, s);
    }
    return adapt ? launch_t<NT, KPT, false, true>(a, g, ws, t0, t1, base, s)
                 : launch_t<NT, KPT, false, false>(a, g, ws, t0, t1, base, s);
}

}  // namespace

// Threads: one candidate each while that takes at most 512 of them (more wavefronts only lengthen the barriers), then
// two and four each; and eight pool nodes per thread at most in the final selection.
int launch_tree_build(const SelectGeometry& g, int t0, int t1, bool adapt, double delta, const BuildWorkspace& ws,
                      const ot_tree_out& out, int32_t* steps_used, double* e_sub, hipStream_t s) {
    TreeBuildArgs a;
    a.topi = ws.row_topi;
    a.batch_pool = g.row_start[g.depth] + g.F[g.depth] - 1;   // sum of F_1 .. F_depth
    a.delta = delta; a.steps_used = steps_used; a.e_sub = e_sub;
    a.pool_key = ws.pool_key; a.pool_meta = ws.pool_tok; a.pool_par = ws.pool_par;
    a.seq_active = (t0 == 0 && t1 == g.depth) ? nullptr : ws.seq_active;
    a.seq_E = ws.seq_E;
    a.out = out;
    int wide = 0;                                             // largest number of candidates of a step
    for (int t = t0; t < t1; ++t) wide = g.k * g.F[t] > wide ? g.k * g.F[t] : wide;
    const int need = (a.batch_pool + kPoolPerThread - 1) / kPoolPerThread;
    if (wide <= 256 && need <= 256) return launch_n<256, 1>(a, g, ws, t0, t1, adapt, s);
    if (wide <= 512 && need <= 512) return launch_n<512, 1>(a, g, ws, t0, t1, adapt, s);
    if (wide <= 1024 && need <= 512) return launch_n<512, 2>(a, g, ws, t0, t1, adapt, s);
    if (wide <= 2048) return launch_n<1024, 2>(a, g, ws, t0, t1, adapt, s);
    return launch_n<1024, 4>(a, g, ws, t0, t1, adapt, s);
}

}  // namespace ot
