// Streaming tree selection (one drafting step per call): everything of Algorithm 1 that follows the row scan.
//   per drafting step t: candidate score = score(parent) + (x - lse)            (Eq. 2 in log space)
//                        keep the F_{t+1} = min(n, k F_t) best candidates       (Algorithm 1, "topk")
//                        number them by (parent slot, rank)
//   finally:             the n best nodes of the whole pool                     (Algorithm 1, last line)
//                        output order (depth, slot); parents, depths (= position offsets, Fig. 1),
//                        ancestor bitmask (Algorithm 2), E = sum of p^           (Eq. 3)
//
// One workgroup per sequence; lane j owns frontier slot j.  Scores are fp64 and compared
// through an order-preserving 64-bit integer key.  "Keep the best m of the workgroup's keys"
// never sorts: it finds the m-th largest key tau by pivoting (each round a lane proposes one
// of its keys still inside the open interval (lo, hi), the workgroup counts keys >= pivot and
// narrows the interval), then every lane keeps its keys > tau and ties at tau are handed out
// in index order.  Because each lane's candidates are already sorted by rank, the kept ones
// are a prefix per lane and the new slot numbering is an exclusive prefix sum of the counts.
#include "tree_select.hpp"

namespace ot {
namespace {

// LDS carve-up shared by the kernels below.  DK = rows of the key region (>= depth, and >= DMAX so
// that the final selection can reuse the region as its key table once the keys sit in registers).
struct Pool {
    double* key;            // [DK][NT]  log p^ of pool node (layer t+1, slot)
    double* kt;             // [KMAX][NT] per-lane key table of the per-step selection
    int* tok;               // [D][NT]
    unsigned char* par;     // [D][NT]   parent slot in the previous layer (< 256)
    unsigned char* oidx;    // [D][NT]   output index of a selected node (< 256)
    u64* mrow;              // [NT][4]   ancestor bitmask rows by output index
};
__device__ __forceinline__ Pool carve_pool(void* smem, int D, int NT, int DK, int KM) {
    Pool p;
    p.key = (double*)smem;
    p.kt = p.key + (size_t)DK * NT;
    p.mrow = (u64*)(p.kt + (size_t)KM * NT);
    p.tok = (int*)(p.mrow + (size_t)NT * 4);
    p.par = (unsigned char*)(p.tok + (size_t)D * NT);
    p.oidx = p.par + (size_t)D * NT;
    return p;
}
inline size_t pool_lds_bytes(int D, int NT, int DK, int KM) {
    return (size_t)DK * NT * 8 + (size_t)KM * NT * 8 + (size_t)NT * 4 * 8 + (size_t)D * NT * (4 + 1 + 1);
}

// The n best nodes of a pool of `steps` layers (last line of Algorithm 1; also the set whose p^ sum is
// E_sub(T, n)).  pk[t] = log p^ of pool node (layer t+1, slot tid), NaN = absent; lo0 (or NaN) is a value that
// at least n pool nodes reach.  Returns bit t set for the selected nodes of this thread.  Ties at the cut:
// shallower first, then smaller slot.  The pool's key region in LDS becomes the selection's table.
template <int DMAX, bool SINGLE>
__device__ unsigned int pool_select(const SelKArgs& a, const Pool& P, const double (&pk)[DMAX], int steps, int pool_nodes,
                                    double lo0, Group<SINGLE>& g, int* s_hist) {
    const int n = a.n;
    unsigned int sel = 0;           // bit t: pool node (layer t+1, slot tid) is in the tree
    if (pool_nodes <= n) {
#pragma unroll
        for (int t = 0; t < DMAX; ++t) sel |= (pk[t] == pk[t] ? 1u : 0u) << t;
    } else {
        lds_sync<SINGLE>();         // every lane has its pool keys in registers: the key region becomes the table
        const Cut cut = select_keys<DMAX, SINGLE, false>(pk, P.key, s_hist, n, lo0 == lo0, lo0, g);
        sel = cut.keep;
        int need = cut.need;
        if (need > 0 && cut.total_eq == need) {
#pragma unroll
            for (int t = 0; t < DMAX; ++t) sel |= (pk[t] == cut.tau ? 1u : 0u) << t;
        } else if (need > 0) {       // ties at the cut: shallower first, then smaller slot
            for (int t = 0; t < steps; ++t) {
                double kt = nan_d();
#pragma unroll
                for (int tt = 0; tt < DMAX; ++tt) kt = (tt == t) ? pk[tt] : kt;
                const int eq = kt == cut.tau ? 1 : 0;
                const int before = g.excl_scan(eq);
                const int layer_eq = g.sum_i(eq);
                if (eq && before < need) sel |= 1u << t;
                need -= layer_eq < need ? layer_eq : need;
            }
        }
    }
    return sel;
}

// Last line of Algorithm 1 and the outputs.  `steps` layers are in the pool; lo0 (or NaN) is a
// value that at least n pool nodes reach (the largest cut value of the steps that cut to n).
template <int DMAX, bool SINGLE>
__device__ void finalize_tree(const SelKArgs& a, const Pool& P, int steps, int b, double lo0, Group<SINGLE>& g,
                              int* s_cntw /*[OT_MAX_DEPTH][4]*/, int* s_hist) {
    const int NT = blockDim.x, tid = threadIdx.x, n = a.n;
    const int W = OT_MASK_WORDS(n);
    int pool_nodes = 0;
    for (int t = 0; t < steps; ++t) pool_nodes += a.F[t + 1];
    const int n_out = pool_nodes < n ? pool_nodes : n;

    double pk[DMAX];
#pragma unroll
    for (int t = 0; t < DMAX; ++t) pk[t] = (t < steps && tid < a.F[t + 1]) ? P.key[t * NT + tid] : nan_d();

    const unsigned int sel = pool_select<DMAX, SINGLE>(a, P, pk, steps, pool_nodes, lo0, g, s_hist);

    // output index = rank in (depth, slot) order among the selected nodes
    const int lane = tid & 63;
    if (SINGLE) {
        int base = 0;               // wave-uniform: nodes selected in shallower layers
#pragma unroll
        for (int t = 0; t < DMAX; ++t) {
            const u64 bal = __ballot((sel >> t) & 1u);
            if ((sel >> t) & 1u) P.oidx[t * NT + tid] = (unsigned char)(base + __popcll(bal & ((1ull << lane) - 1ull)));
            base += __popcll(bal);
        }
    } else {
        int my_prefix[DMAX];
#pragma unroll
        for (int t = 0; t < DMAX; ++t) {
            const u64 bal = __ballot((sel >> t) & 1u);
            my_prefix[t] = __popcll(bal & ((1ull << lane) - 1ull));
            if (lane == 0 && t < steps) s_cntw[t * 4 + g.wave] = __popcll(bal);
        }
        lds_sync<SINGLE>();
        int base = 0;
#pragma unroll
        for (int t = 0; t < DMAX; ++t) {
            if (t < steps) {
                int mine = base;
                for (int w = 0; w < g.nw; ++w) {
                    const int c = s_cntw[t * 4 + w];
                    if (w < g.wave) mine += c;
                    base += c;
                }
                if ((sel >> t) & 1u) P.oidx[t * NT + tid] = (unsigned char)(mine + my_prefix[t]);
            }
        }
    }
    lds_sync<SINGLE>();

    // output index of every selected node of this lane and of its parent (independent LDS reads)
    int my_i[DMAX], my_pi[DMAX];
#pragma unroll
    for (int t = 0; t < DMAX; ++t) {
        my_i[t] = 0; my_pi[t] = -1;
        if (t < steps && ((sel >> t) & 1u)) {
            my_i[t] = P.oidx[t * NT + tid];
            if (t > 0) my_pi[t] = P.oidx[(t - 1) * NT + P.par[t * NT + tid]];
        }
    }
    if (SINGLE) {
        // n <= 64: node i becomes lane i (tables by output index in place of the mask rows and the keys).  Every round doubles
        // the stretch of a root path that a mask holds: the mask of the node at its end is added, and that node's end is the
        // new one.  (Layer by layer, with a trip to LDS each, and two trips to memory for the layers above: 9.6 us for ten
        // layers of 50 nodes, now 8.5.)
        int* const r_tok = (int*)P.mrow;
        int* const r_par = r_tok + NT;
        int* const r_dep = r_par + NT;
        double* const r_key = P.key;
#pragma unroll
        for (int t = 0; t < DMAX; ++t)
            if (t < steps && ((sel >> t) & 1u)) {
                const int i = my_i[t];
                r_key[i] = pk[t]; r_tok[i] = P.tok[t * NT + tid]; r_par[i] = my_pi[t]; r_dep[i] = t + 1;
            }
        lds_sync<SINGLE>();
        const bool node = tid < n_out;
        const double key = node ? r_key[tid] : -INFINITY;
        const int par = node ? r_par[tid] : -1;
        u64 row = node ? 1ull << tid : 0ull;
        int up = par;
        for (int stretch = 1; stretch < OT_MAX_DEPTH; stretch *= 2) {
            if (!__any(up >= 0)) break;
            const int at = max(up, 0);
            const u64 above = (u64)(unsigned)__shfl((int)(row >> 32), at) << 32 | (unsigned)__shfl((int)row, at);
            const int next = __shfl(up, at);
            if (up >= 0) { row |= above; up = next; }
        }
        if (tid < n) {
            const size_t o = (size_t)b * n + tid;
            a.out.token[o] = node ? r_tok[tid] : -1;
            a.out.parent[o] = par;
            a.out.depth[o] = node ? r_dep[tid] : 0;
            a.out.score[o] = (float)key;
            a.out.mask[o] = row;
        }
        const double e = wave_sum_d(node ? exp(key) : 0.0);            // E = sum of p^ (Eq. 3)
        if (tid == 0) {
            a.out.expect[b] = e;
            a.out.n_out[b] = n_out;
        }
        return;
    }
    // ancestor masks, layer by layer (a parent's row is complete before its children read it), and
    // the per-node outputs.  The key region is free again: it collects log p^ by output index.
    const size_t ob = (size_t)b * n;
    double* sc_by_index = P.key;
#pragma unroll
    for (int t = 0; t < DMAX; ++t) {
        if (t < steps) {
            if ((sel >> t) & 1u) {
                const int i = my_i[t], pi = my_pi[t];
                u64 row[4] = {0ull, 0ull, 0ull, 0ull};
                if (t > 0) {
#pragma unroll
                    for (int w = 0; w < 4; ++w) row[w] = P.mrow[pi * 4 + w];
                }
#pragma unroll
                for (int w = 0; w < 4; ++w) row[w] |= (w == (i >> 6)) ? (1ull << (i & 63)) : 0ull;
#pragma unroll
                for (int w = 0; w < 4; ++w) P.mrow[i * 4 + w] = row[w];
                sc_by_index[i] = pk[t];
                a.out.token[ob + i] = P.tok[t * NT + tid];
                a.out.parent[ob + i] = pi;
                a.out.depth[ob + i] = t + 1;
                a.out.score[ob + i] = (float)pk[t];
#pragma unroll
                for (int w = 0; w < 4; ++w)
                    if (w < W) a.out.mask[(ob + i) * W + w] = row[w];
            }
            lds_sync<SINGLE>();
        }
    }
    for (int i = n_out + tid; i < n; i += NT) {
        a.out.token[ob + i] = -1;
        a.out.parent[ob + i] = -1;
        a.out.depth[ob + i] = 0;
        a.out.score[ob + i] = -INFINITY;
        for (int w = 0; w < W; ++w) a.out.mask[(ob + i) * W + w] = 0ull;
    }
    // E = sum of p^ (Eq. 3): one exp per lane, node i on lane i
    double e_sum = tid < n_out ? exp(sc_by_index[tid]) : 0.0;
    e_sum = g.sum_d(e_sum);
    if (tid == 0) {
        a.out.expect[b] = e_sum;
        a.out.n_out[b] = n_out;
    }
}

template <int KMAX, bool SINGLE>
__global__ __launch_bounds__(256) void tree_step_kernel(const SelKArgs a) {
    extern __shared__ u64 smem[];
    draft_step<KMAX, SINGLE, false>(a, blockIdx.x, blockDim.x, (double*)smem);
}

template <int DMAX, bool SINGLE>
__global__ __launch_bounds__(256) void tree_finalize_kernel(const SelKArgs a) {
    extern __shared__ u64 smem[];
    OT_SELECT_SHARED((int)blockDim.x)
    const int NT = blockDim.x, tid = threadIdx.x, b = blockIdx.x, n = a.n;
    const int steps = a.step < a.seq_steps[b] ? a.step : a.seq_steps[b];     // a frozen sequence has fewer layers
    const Pool P = carve_pool(smem, a.depth, NT, DMAX, 0);
    const size_t pb = (size_t)b * a.depth * n;
    double lo0 = nan_d();
    constexpr int BATCH = DMAX < 16 ? DMAX : 16;   // layers requested at once
#pragma unroll
    for (int t0 = 0; t0 < DMAX; t0 += BATCH) {
        if (t0 >= a.step) break;
        double key[BATCH], tau[BATCH];
        int tok[BATCH], par[BATCH];
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            const int t = min(t0 + u, a.depth - 1);
            const size_t o = pb + (size_t)t * n + min(tid, n - 1);
            key[u] = a.pool_key[o]; tok[u] = a.pool_tok[o]; par[u] = a.pool_par[o];
            tau[u] = a.step_tau[(size_t)b * a.depth + t];
        }
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            const int t = t0 + u;
            if (t < steps) {
                if (tid < a.F[t + 1]) {
                    P.key[t * NT + tid] = key[u];
                    P.tok[t * NT + tid] = tok[u];
                    P.par[t * NT + tid] = (unsigned char)par[u];
                }
                if (tau[u] == tau[u]) lo0 = (lo0 == lo0) ? fmax(lo0, tau[u]) : tau[u];
            }
        }
    }
    __syncthreads();
    finalize_tree<DMAX, SINGLE>(a, P, steps, b, lo0, g, s_cntw, s_hist);
}

// E_sub(T, n) of the tree drafted so far = the sum of the n largest p^ of the pool (Sec. 3, text ahead of
// Algorithm 1), and the loop condition of Algorithm 1: go on while E_sub - E > delta, with E <- E_sub.
// A sequence that stops is frozen (tree_step_kernel skips it, tree_finalize_kernel uses its layer count).
template <int DMAX, bool SINGLE>
__global__ __launch_bounds__(256) void tree_esub_kernel(const SelKArgs a) {
    extern __shared__ u64 smem[];
    OT_SELECT_SHARED((int)blockDim.x)
    (void)s_cntw;
    const int NT = blockDim.x, tid = threadIdx.x, b = blockIdx.x, n = a.n;
    const int steps = a.step < a.seq_steps[b] ? a.step : a.seq_steps[b];
    const Pool P = carve_pool(smem, a.depth, NT, DMAX, 0);
    const size_t pb = (size_t)b * a.depth * n;
    double lo0 = nan_d();
    int pool_nodes = 0;
    double pk[DMAX], pp[DMAX], tau[DMAX];
#pragma unroll
    for (int t = 0; t < DMAX; ++t) {
        const int tc = min(t, a.depth - 1);
        const size_t o = pb + (size_t)tc * n + min(tid, n - 1);
        pk[t] = a.pool_key[o];
        pp[t] = a.pool_p[o];
        tau[t] = a.step_tau[(size_t)b * a.depth + tc];
    }
    const int live = a.seq_active[b];
    const double E = a.seq_E[b];
    asm volatile("" ::: "memory");              // (all requested by now)
#pragma unroll
    for (int t = 0; t < DMAX; ++t) {
        const bool have = t < steps && tid < a.F[t + 1];
        pk[t] = have ? pk[t] : nan_d();
        pp[t] = have ? pp[t] : 0.0;
        if (t < steps) {
            pool_nodes += a.F[t + 1];
            if (tau[t] == tau[t]) lo0 = (lo0 == lo0) ? fmax(lo0, tau[t]) : tau[t];
        }
    }
    __syncthreads();
    const unsigned int sel = pool_select<DMAX, SINGLE>(a, P, pk, steps, pool_nodes, lo0, g, s_hist);
    double e = 0.0;
#pragma unroll
    for (int t = 0; t < DMAX; ++t) e += ((sel >> t) & 1u) ? pp[t] : 0.0;
    e = g.sum_d(e);
    if (tid == 0) {
        a.e_sub[b] = e;
        int go = 0;
        if (live) {
            go = (e - E > a.delta) ? 1 : 0;
            if (go) a.seq_E[b] = e; else a.seq_active[b] = 0;
        }
        a.go_on[b] = go;
    }
}

// The frontier's ancestor masks, from the root paths the step kernel keeps: mask_out [batch][n][mask_words].
// A thread per word (one workgroup per sequence took 64 rounds at the largest shapes).
__global__ __launch_bounds__(256) void tree_front_mask_kernel(const SelKArgs a) {
    const int b = blockIdx.x, n = a.n, i = blockIdx.y * 256 + threadIdx.x;
    if (i >= n * a.mask_words) return;
    const int s = i / a.mask_words, w = i - s * a.mask_words;
    const int steps = min(a.step, a.seq_steps[b]);
    const int F = steps > 0 ? a.F[steps] : 0;
    const size_t fa = (size_t)a.gridDim_batch * n * OT_MAX_DEPTH;
    const u32x4* const src = (const u32x4*)(a.front_anc + (size_t)((steps - 1) & 1) * fa + ((size_t)b * n + s) * OT_MAX_DEPTH);
    u64 bits = 0ull;
    if (s < F) {
        u32x4 path[kPathVecs];
#pragma unroll
        for (int q = 0; q < kPathVecs; ++q) path[q] = src[q];
#pragma unroll
        for (int q = 0; q < kPathVecs; ++q) {
            if (8 * q >= steps) break;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int idx = (int)((path[q][e >> 1] >> (16 * (e & 1))) & 0xffffu);
                bits |= 8 * q + e < steps && (idx >> 6) == w ? 1ull << (idx & 63) : 0ull;
            }
        }
    }
    a.mask_out[(size_t)b * n * a.mask_words + i] = bits;
}

// Loop state of every sequence; with frontier arrays given, these too (tokens and parents -1, counts 0).
__global__ __launch_bounds__(256) void tree_begin_kernel(double* seq_E, int32_t* seq_steps, int32_t* seq_active, int batch, int n,
                                                         int32_t* frontier_token, int32_t* frontier_parent, int32_t* frontier_count) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < batch) {
        seq_E[i] = 0.0; seq_steps[i] = 0; seq_active[i] = 1;
        if (frontier_count) frontier_count[i] = 0;
    }
    if (frontier_token && i < batch * n) { frontier_token[i] = -1; frontier_parent[i] = -1; }
}

template <typename K>
int set_lds(K kernel, size_t bytes) {
    if (bytes > 64 * 1024) {
        if (bytes > 160 * 1024) return OT_ERR_UNSUPPORTED;
        OT_HIP_CHECK(hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
    }
    return OT_OK;
}

template <int KMAX, bool SINGLE>
int launch_step_t(const SelKArgs& a, int batch, int NT, hipStream_t s) {
    const size_t lds = (size_t)KMAX * NT * 8;
    hipLaunchKernelGGL((tree_step_kernel<KMAX, SINGLE>), dim3(batch), dim3(NT), lds, s, a);
    OT_HIP_CHECK(hipGetLastError());
    return OT_OK;
}
template <bool SINGLE>
int launch_step_s(const SelKArgs& a, int batch, int NT, hipStream_t s) {
    if (a.k <= 4) return launch_step_t<4, SINGLE>(a, batch, NT, s);
    if (a.k <= 8) return launch_step_t<8, SINGLE>(a, batch, NT, s);
    if (a.k <= 10) return launch_step_t<10, SINGLE>(a, batch, NT, s);
    return launch_step_t<16, SINGLE>(a, batch, NT, s);
}

template <int DMAX, bool SINGLE>
int launch_finalize_t(const SelKArgs& a, int batch, int NT, hipStream_t s) {
    const size_t lds = pool_lds_bytes(a.depth, NT, DMAX, 0);
    int st = set_lds(tree_finalize_kernel<DMAX, SINGLE>, lds);
    if (st != OT_OK) return st;
    hipLaunchKernelGGL((tree_finalize_kernel<DMAX, SINGLE>), dim3(batch), dim3(NT), lds, s, a);
    OT_HIP_CHECK(hipGetLastError());
    return OT_OK;
}

}  // namespace

int launch_tree_step(const SelectGeometry& g, int step, const BuildWorkspace& ws, int32_t* frontier_token,
                     int32_t* frontier_parent, int32_t* frontier_count, hipStream_t s) {
    SelKArgs a = make_args(g, ws);
    a.step = step;
    a.frontier_token = frontier_token; a.frontier_parent = frontier_parent; a.frontier_count = frontier_count;
    const int NT = threads_for(g.n);
    return NT == 64 ? launch_step_s<true>(a, g.batch, NT, s) : launch_step_s<false>(a, g.batch, NT, s);
}

template <int DMAX, bool SINGLE>
int launch_esub_t(const SelKArgs& a, int batch, int NT, hipStream_t s) {
    const size_t lds = pool_lds_bytes(a.depth, NT, DMAX, 0);
    int st = set_lds(tree_esub_kernel<DMAX, SINGLE>, lds);
    if (st != OT_OK) return st;
    hipLaunchKernelGGL((tree_esub_kernel<DMAX, SINGLE>), dim3(batch), dim3(NT), lds, s, a);
    OT_HIP_CHECK(hipGetLastError());
    return OT_OK;
}

int launch_tree_begin(const SelectGeometry& g, const BuildWorkspace& ws, hipStream_t s, int32_t* frontier_token,
                      int32_t* frontier_parent, int32_t* frontier_count) {
    const long long items = frontier_token ? (long long)g.batch * g.n : g.batch;
    if (items > 0x7fffffffLL - 256) return OT_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(tree_begin_kernel, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, s, ws.seq_E, ws.seq_steps,
                       ws.seq_active, g.batch, g.n, frontier_token, frontier_parent, frontier_count);
    OT_HIP_CHECK(hipGetLastError());
    return OT_OK;
}

int launch_tree_esub(const SelectGeometry& g, int steps_done, double delta, const BuildWorkspace& ws, double* e_sub,
                     int32_t* go_on, hipStream_t s) {
    SelKArgs a = make_args(g, ws);
    a.step = steps_done; a.delta = delta; a.e_sub = e_sub; a.go_on = go_on;
    const int NT = threads_for(g.n);
    if (NT == 64) {
        if (steps_done <= 4) return launch_esub_t<4, true>(a, g.batch, NT, s);
        if (steps_done <= 8) return launch_esub_t<8, true>(a, g.batch, NT, s);
        if (steps_done <= 12) return launch_esub_t<12, true>(a, g.batch, NT, s);
        if (steps_done <= 16) return launch_esub_t<16, true>(a, g.batch, NT, s);
        return launch_esub_t<32, true>(a, g.batch, NT, s);
    }
    if (steps_done <= 8) return launch_esub_t<8, false>(a, g.batch, NT, s);
    if (steps_done <= 16) return launch_esub_t<16, false>(a, g.batch, NT, s);
    return launch_esub_t<32, false>(a, g.batch, NT, s);
}

int launch_tree_front_mask(const SelectGeometry& g, int steps_done, const BuildWorkspace& ws, uint64_t* mask_out,
                           int mask_words, hipStream_t s) {
    SelKArgs a = make_args(g, ws);
    a.step = steps_done; a.mask_out = (u64*)mask_out; a.mask_words = mask_words;
    hipLaunchKernelGGL(tree_front_mask_kernel, dim3(g.batch, (g.n * mask_words + 255) / 256), dim3(256), 0, s, a);
    OT_HIP_CHECK(hipGetLastError());
    return OT_OK;
}

int launch_tree_finalize(const SelectGeometry& g, int steps_done, const BuildWorkspace& ws, const ot_tree_out& out,
                         hipStream_t s) {
    SelKArgs a = make_args(g, ws);
    a.out = out;
    a.step = steps_done;
    const int NT = threads_for(g.n);
    if (NT == 64) {
        if (steps_done <= 8) return launch_finalize_t<8, true>(a, g.batch, NT, s);
        if (steps_done <= 16) return launch_finalize_t<16, true>(a, g.batch, NT, s);
        return launch_finalize_t<32, true>(a, g.batch, NT, s);
    }
    if (steps_done <= 8) return launch_finalize_t<8, false>(a, g.batch, NT, s);
    if (steps_done <= 16) return launch_finalize_t<16, false>(a, g.batch, NT, s);
    return launch_finalize_t<32, false>(a, g.batch, NT, s);
}

}  // namespace ot
