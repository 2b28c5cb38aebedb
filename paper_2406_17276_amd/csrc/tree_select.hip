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
#include "common.hpp"

namespace ot {
namespace {

typedef unsigned long long u64;

struct SelKArgs {
    const double* row_lse; const float* row_topv; const int32_t* row_topi;
    int k, n, depth, rows_per_seq;
    int F[OT_MAX_DEPTH + 2];
    int r0[OT_MAX_DEPTH + 2];      // rank whose per-lane minimum is a lower bound of step t's cut
    double* pool_key; int32_t* pool_tok; int32_t* pool_par;   // [batch][depth][n]  (streaming state)
    double* step_tau;                                         // [batch][depth]     (streaming state)
    double* pool_p;                                           // [batch][depth][n]  (streaming state) p^ of every pool node
    double* seq_E; int32_t* seq_steps; int32_t* seq_active;   // [batch]            (streaming state) adaptive depth
    double* e_sub; int32_t* go_on; double delta;              // outputs / threshold of the E_sub query
    unsigned short* front_anc;                                // [2][batch][n][OT_MAX_DEPTH] (streaming state): the pool
                                                              // indices of every node of the last two frontiers' root
                                                              // paths, the node itself last
    u64* mask_out; int mask_words;                            // output of the frontier-mask query
    int gridDim_batch;                                        // batch size (the grid of these kernels)
    ot_tree_out out;
    int32_t* frontier_token; int32_t* frontier_parent;        // [batch][n]         (streaming step)
    int32_t* frontier_count;                                  // [batch] or null    (streaming step)
    int step;
};

__device__ __forceinline__ double nan_d() { return __longlong_as_double(0x7ff8000000000000ll); }   // "absent"

// ---- integer wavefront reductions that end in a scalar ----
__device__ __forceinline__ int wave_max_u(int v) {
    v = max(v, dpp_i<DPP_QUAD_XOR1>(v, v));
    v = max(v, dpp_i<DPP_QUAD_XOR2>(v, v));
    v = max(v, dpp_i<DPP_ROW_HALF_MIRROR>(v, v));
    v = max(v, dpp_i<DPP_ROW_MIRROR>(v, v));
    return max(max(rl(v, 0), rl(v, 16)), max(rl(v, 32), rl(v, 48)));
}
__device__ __forceinline__ int wave_sum_u(int v) {
    v += dpp_i<DPP_QUAD_XOR1>(v, v);
    v += dpp_i<DPP_QUAD_XOR2>(v, v);
    v += dpp_i<DPP_ROW_HALF_MIRROR>(v, v);
    v += dpp_i<DPP_ROW_MIRROR>(v, v);
    return (rl(v, 0) + rl(v, 16)) + (rl(v, 32) + rl(v, 48));
}
// fmin/fmax ignore NaN operands, NaN marks "absent"
__device__ __forceinline__ double wave_min_d(double v) {
    v = fmin(v, dpp_d<DPP_QUAD_XOR1>(v));
    v = fmin(v, dpp_d<DPP_QUAD_XOR2>(v));
    v = fmin(v, dpp_d<DPP_ROW_HALF_MIRROR>(v));
    v = fmin(v, dpp_d<DPP_ROW_MIRROR>(v));
    return fmin(fmin(rl_d(v, 0), rl_d(v, 16)), fmin(rl_d(v, 32), rl_d(v, 48)));
}
// Barrier that orders LDS traffic only: nothing here communicates through global memory, so loads and stores that are still
// under way need not end first.
template <bool SINGLE>
__device__ __forceinline__ void lds_sync() {
    if (SINGLE) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    else        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Workgroup collectives.  SINGLE: the workgroup is one wavefront, no LDS and no barrier needed.
template <bool SINGLE>
struct Group {
    int* red;        // LDS int[2][4]
    double* bc;      // LDS double[2]
    double* redd;    // LDS double[2][4]
    int phase, bphase, dphase;
    int tid, lane, wave, nw;
    int nt;          // threads of the group = stride of its LDS key tables

    __device__ __forceinline__ int combine(int v, bool is_max) {
        if (SINGLE) return v;
        if (lane == 0) red[phase * 4 + wave] = v;
        lds_sync<false>();
        int r = red[phase * 4];
        for (int w = 1; w < nw; ++w) r = is_max ? max(r, red[phase * 4 + w]) : r + red[phase * 4 + w];
        phase ^= 1;
        return r;
    }
    __device__ __forceinline__ int max_i(int v) { return combine(wave_max_u(v), true); }
    __device__ __forceinline__ int sum_i(int v) { return combine(wave_sum_u(v), false); }
    __device__ __forceinline__ double min_d(double v) {
        v = wave_min_d(v);
        if (SINGLE) return v;
        if (lane == 0) redd[dphase * 4 + wave] = v;
        lds_sync<false>();
        double r = redd[dphase * 4];
        for (int w = 1; w < nw; ++w) r = fmin(r, redd[dphase * 4 + w]);
        dphase ^= 1;
        return r;
    }
    __device__ __forceinline__ double sum_d(double v) {
        v = wave_sum_d(v);
        if (SINGLE) return v;
        if (lane == 0) redd[dphase * 4 + wave] = v;
        lds_sync<false>();
        double r = redd[dphase * 4];
        for (int w = 1; w < nw; ++w) r += redd[dphase * 4 + w];
        dphase ^= 1;
        return r;
    }
    // value of thread `src` (uniform) for everybody
    __device__ __forceinline__ double bcast(double v, int src) {
        if (SINGLE) return rl_d(v, src);
        if (tid == src) bc[bphase] = v;
        lds_sync<false>();
        const double r = bc[bphase];
        bphase ^= 1;
        return r;
    }
    // exclusive prefix sum over the workgroup in thread order
    __device__ __forceinline__ int excl_scan(int v) {
        const int inc = wave_incl_scan(v, lane);
        if (SINGLE) return inc - v;
        if (lane == 63) red[phase * 4 + wave] = inc;
        lds_sync<false>();
        int off = 0;
        for (int w = 0; w < wave; ++w) off += red[phase * 4 + w];
        phase ^= 1;
        return inc - v + off;
    }
};

constexpr int kBuckets = 256;

// next double above v (v finite)
__device__ __forceinline__ double next_up(double v) {
    if (v == 0.0) return __longlong_as_double(1ll);
    const long long bits = __double_as_longlong(v);
    return __longlong_as_double(v > 0.0 ? bits + 1 : bits - 1);
}

// Sort M doubles in registers, descending, NaN last (Batcher's odd-even merge network).
template <int M>
__device__ __forceinline__ void sort_desc(double (&x)[M]) {
#pragma unroll
    for (int p = 1; p < M; p *= 2)
#pragma unroll
        for (int k = p; k >= 1; k /= 2)
#pragma unroll
            for (int j = k % p; j <= M - 1 - k; j += 2 * k)
#pragma unroll
                for (int i = 0; i < k; ++i)
                    if (i + j + k <= M - 1 && (i + j) / (2 * p) == (i + j + k) / (2 * p)) {
                        const double u = x[i + j], w = x[i + j + k];
                        const bool swap = !(u >= w) && (w == w);
                        x[i + j] = swap ? w : u;
                        x[i + j + k] = swap ? u : w;
                    }
}

// Exact end game of a selection, on keys sorted per lane (descending, NaN last): ks[a..b) are this lane's
// keys still inside the range, f_hi keys of the workgroup lie above the range, f_lo lie above or inside it,
// every key inside is >= lo and f_lo >= want > f_hi.  Pivots are keys strictly above lo, proposed by the lane
// with most keys in range; the workgroup counts the keys >= pivot and narrows the range.  Ends when no key
// lies strictly above lo inside the range: then every key left inside equals lo, the cut value.
// kt is an LDS table [M][threads of the group].
struct Range {
    int a, b;          // this lane's keys inside the range: ks[a..b)
    int f_hi, f_lo;    // keys of the workgroup above the range / above or inside it
    double lo;         // every key inside is >= lo
};
template <int M, bool SINGLE>
__device__ __forceinline__ Range pivot_rounds(const double (&ks)[M], double* kt, int want, Range rg, Group<SINGLE>& g) {
    int a = rg.a, b = rg.b, f_hi = rg.f_hi, f_lo = rg.f_lo;
    double lo = rg.lo;
    const int NT = g.nt, tid = g.tid;
#pragma unroll
    for (int r = 0; r < M; ++r) kt[r * NT + tid] = ks[r];
    // every round moves lo up or the upper end down to a key strictly inside, so M * blockDim rounds
    // always suffice; the bound makes termination unconditional
    for (int round = 0; round < M * 256 + 2; ++round) {
        const int cnt = b - a;
        double prop = nan_d();
        if (cnt > 0) {
            const int T = want - f_hi, R = f_lo - f_hi;
            int q = (int)((float)cnt * (float)(2 * T - 1) * __frcp_rn((float)(2 * R)));
            q = q > cnt - 1 ? cnt - 1 : (q < 0 ? 0 : q);
            const double top = kt[a * NT + tid];
            prop = kt[(a + q) * NT + tid];
            if (!(prop > lo)) prop = top;
        }
        const bool valid = prop > lo;
        const int win = g.max_i(valid ? ((cnt << 16) | (0xffff - tid)) : 0);
        if (win == 0) break;
        const double p = g.bcast(prop, 0xffff - (win & 0xffff));
        int ge = 0;
#pragma unroll
        for (int r = 0; r < M; ++r) ge += ks[r] >= p ? 1 : 0;
        const int f_p = g.sum_i(ge);
        if (f_p >= want) { lo = p; b = ge; f_lo = f_p; }
        else             { a = ge; f_hi = f_p; }
    }
    Range out;
    out.a = a; out.b = b; out.f_hi = f_hi; out.f_lo = f_lo; out.lo = lo;
    return out;
}

// Result of "keep the `want` largest keys of the workgroup".
struct Cut {
    unsigned keep;     // bit r: this lane's key[r] is kept for certain
    double tau;        // every kept key is >= tau, at least `want` keys are >= tau
    int need;          // > 0: besides `keep`, `need` of the `total_eq` keys == tau are kept, in the caller's tie order
    int total_eq;
};

// Every lane holds M keys (NaN = absent); SORTED: in descending order with NaN last.
// kt is an LDS table [M][blockDim] (used only by phase 2), hist an LDS scratch of kBuckets + 4 ints.
//   phase 1  [lo, hi) = [caller's lower bound (or the smallest key), just above the largest key).
//            The keys inside are binned into 256 equal-width buckets (LDS atomics); a suffix scan of
//            the histogram finds the bucket that holds the cut; the same is repeated once inside
//            that bucket (65536 cells overall).  If the cut falls between two cells the kept set is
//            known exactly and the search is over.  Needs no order inside a lane.
//   phase 2  (ties or near-ties at the cut) on sorted keys: pivots are keys strictly inside the
//            remaining range, proposed by the lane with most keys in range; per lane a = #keys
//            above the range, b = #keys above or in it.  Ends when no key lies strictly inside, so
//            that every key left in range equals tau.
template <int M, bool SINGLE, bool SORTED>
__device__ Cut select_keys(const double (&key)[M], double* kt, int* hist, int want, bool have_first,
                           double first_pivot, Group<SINGLE>& g) {
    (void)kt;
    Cut cut;
    cut.keep = 0u; cut.need = 0; cut.total_eq = 0;
    double lmin = nan_d(), lmax = nan_d();
#pragma unroll
    for (int r = 0; r < M; ++r) { lmin = fmin(lmin, key[r]); lmax = fmax(lmax, key[r]); }
    double lo = have_first ? first_pivot : g.min_d(lmin);
    const double gmax = -g.min_d(-lmax);
    unsigned in = 0u;                              // keys inside [lo, hi)
#pragma unroll
    for (int r = 0; r < M; ++r) in |= (key[r] >= lo ? 1u : 0u) << r;
    int f_hi = 0, f_lo = 0;
    bool exact = false;
    if (gmax > lo) {
        const double hi = next_up(gmax);
        double u[M];
        const double scale = (double)kBuckets / (hi - lo);
#pragma unroll
        for (int r = 0; r < M; ++r) u[r] = (key[r] - lo) * scale;
        for (int level = 0; level < 2; ++level) {
            int bk[M];
#pragma unroll
            for (int r = 0; r < M; ++r) {
                int q = (int)u[r];
                bk[r] = q < 0 ? 0 : (q > kBuckets - 1 ? kBuckets - 1 : q);
            }
            // hist is all zero here (cleared once per kernel, and re-cleared by the scan below)
#pragma unroll
            for (int r = 0; r < M; ++r)
                if ((in >> r) & 1u) atomicAdd(&hist[bk[r]], 1);
            lds_sync<SINGLE>();
            const int T = want - f_hi;            // rank of the cut among the keys in range
            int B = -1, above = 0, inb = 0, total = 0;
            if (g.wave == 0) {
                constexpr int BPL = kBuckets / 64;                 // buckets per lane of the scanning wavefront
                const int L = g.lane;
                int c[BPL];
                int sum = 0;
#pragma unroll
                for (int i = 0; i < BPL; ++i) { c[i] = hist[BPL * L + i]; sum += c[i]; }
#pragma unroll
                for (int i = 0; i < BPL; ++i) hist[BPL * L + i] = 0;
                const int P = wave_incl_scan(sum, L);
                total = rl(P, 63);
                const int above_lane = total - P;                 // keys in higher lanes' buckets
                const bool has = above_lane < T && above_lane + sum >= T;
                int Bl = BPL * L, abl = above_lane, inl = 0;
                bool found = false;
#pragma unroll
                for (int i = BPL - 1; i >= 0; --i) {              // highest bucket first
                    if (!found) {
                        if (abl + c[i] >= T) { found = true; Bl = BPL * L + i; inl = c[i]; }
                        else abl += c[i];
                    }
                }
                const u64 bal = __ballot(has);
                if (bal != 0ull) {
                    const int src = __ffsll((long long)bal) - 1;
                    B = rl(Bl, src); above = rl(abl, src); inb = rl(inl, src);
                }
                if (!SINGLE && L == 0) {
                    hist[kBuckets] = B; hist[kBuckets + 1] = above; hist[kBuckets + 2] = inb; hist[kBuckets + 3] = total;
                }
            }
            if (!SINGLE) {
                lds_sync<SINGLE>();
                B = hist[kBuckets]; above = hist[kBuckets + 1]; inb = hist[kBuckets + 2]; total = hist[kBuckets + 3];
            }
            if (level == 0) f_lo = f_hi + total;
            if (B < 0) break;                     // cannot happen while count(key >= lo) >= want; be safe
            unsigned gt = 0u, eq = 0u;
#pragma unroll
            for (int r = 0; r < M; ++r) {
                gt |= (bk[r] > B ? 1u : 0u) << r;
                eq |= (bk[r] == B ? 1u : 0u) << r;
            }
            cut.keep |= in & gt;
            if (above + inb == T) { exact = true; cut.keep |= in & eq; break; }
            in &= eq;
            f_hi += above; f_lo = f_hi + inb;
#pragma unroll
            for (int r = 0; r < M; ++r) u[r] = (u[r] - (double)B) * (double)kBuckets;
        }
    } else {
        f_lo = g.sum_i(__popc(in));
    }
    if (exact) {
        double kmin = nan_d();
#pragma unroll
        for (int r = 0; r < M; ++r) kmin = fmin(kmin, ((cut.keep >> r) & 1u) ? key[r] : nan_d());
        cut.tau = g.min_d(kmin);
        return cut;
    }

    // ---- phase 2 -----------------------------------------------------------------------------
    double ks[M];
#pragma unroll
    for (int r = 0; r < M; ++r) ks[r] = key[r];
    if (!SORTED) sort_desc<M>(ks);
    Range rg;
    rg.a = __popc(cut.keep); rg.b = rg.a + __popc(in); rg.f_hi = f_hi; rg.f_lo = f_lo; rg.lo = lo;
    rg = pivot_rounds<M, SINGLE>(ks, kt, want, rg, g);
    cut.tau = rg.lo;
    cut.keep = 0u;
#pragma unroll
    for (int r = 0; r < M; ++r) cut.keep |= (key[r] > rg.lo ? 1u : 0u) << r;
    cut.need = want - rg.f_hi;
    cut.total_eq = rg.f_lo - rg.f_hi;
    return cut;
}

// One drafting step's cut: how many of this lane's (rank-sorted) candidates survive, and the
// first slot they occupy in the next layer.  tau_out: a value reached by at least `want`
// candidates (NaN when nothing was cut).
template <int KMAX, bool SINGLE>
__device__ void layer_cut(const double (&ck)[KMAX], double* kt, int* hist, bool active, int k, int F, int want,
                          int r0, Group<SINGLE>& g, int& cnt, int& off, double& tau_out) {
    tau_out = nan_d();
    if (k * F <= want) {
        cnt = active ? k : 0;
    } else {
        // every lane holds at least r0+1 candidates and (r0+1) F >= want, so the smallest rank-r0
        // candidate is a lower bound of the cut: it discards most candidates at once
        double c0 = nan_d();
#pragma unroll
        for (int r = 0; r < KMAX; ++r) c0 = (r == r0) ? ck[r] : c0;
        const double m0 = g.min_d(c0);
        const Cut cut = select_keys<KMAX, SINGLE, true>(ck, kt, hist, want, true, m0, g);
        cnt = __popc(cut.keep);               // sorted candidates: the kept ones are a prefix
        if (cut.need > 0) {                   // ties at the cut: smaller parent slot first, then smaller rank
            int lane_eq = 0;
#pragma unroll
            for (int r = 0; r < KMAX; ++r) lane_eq += ck[r] == cut.tau ? 1 : 0;
            int take = lane_eq;
            if (cut.total_eq != cut.need) {
                const int before = g.excl_scan(lane_eq);
                take = cut.need - before;
                take = take < 0 ? 0 : (take > lane_eq ? lane_eq : take);
            }
            cnt += take;
        }
        tau_out = cut.tau;
    }
    off = g.excl_scan(cnt);
}

// candidate scores of one frontier slot: log p^(child) = log p^(parent) + (x - lse)   (Eq. 2)
template <int KMAX>
__device__ __forceinline__ void candidate_scores(double S, double lse, const float (&v)[KMAX], bool active, int k,
                                                 double (&ck)[KMAX]) {
#pragma unroll
    for (int r = 0; r < KMAX; ++r)
        ck[r] = (active && r < k) ? S + ((double)v[r] - lse) : __longlong_as_double(0x7ff8000000000000ll);
}

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

#define OT_SELECT_SHARED                                   \
    extern __shared__ u64 smem[];                          \
    __shared__ int s_red[8];                               \
    __shared__ double s_bc[2];                             \
    __shared__ double s_redd[8];                           \
    __shared__ int s_cntw[OT_MAX_DEPTH * 4];               \
    __shared__ int s_hist[kBuckets + 4];                   \
    Group<SINGLE> g;                                       \
    g.red = s_red; g.bc = s_bc; g.redd = s_redd;           \
    g.phase = g.bphase = g.dphase = 0;                     \
    g.tid = threadIdx.x; g.lane = threadIdx.x & 63;        \
    g.wave = threadIdx.x >> 6; g.nw = blockDim.x >> 6;     \
    g.nt = blockDim.x;                                     \
    for (int i_ = threadIdx.x; i_ < kBuckets + 4; i_ += blockDim.x) s_hist[i_] = 0; \
    __syncthreads();

// The streaming kernels are short, and what bounds them is trips to memory (0.6 to 0.8 us each): every load whose address
// does not depend on another is requested ahead of the first use, from clamped addresses instead of under a condition, and
// a root path is four 16-byte vectors.  Measured (MI355X, 7B-shaped drafting loop of ten steps): step kernel 7.8 -> 4.0 us,
// E_sub 4.5..6.8 -> 4.0..5.3 us, mask 2.3 us; the whole loop replayed from a graph 156 -> 148 us, through the binding 181 ->
// 154 us; eight sequences of n = 256, k = 16, 12 steps: 816 -> 465 us.
constexpr int kPathVecs = OT_MAX_DEPTH / 8;      // u16 entries

// Streaming: one drafting step; the pool lives in the caller's workspace between launches.
template <int KMAX, bool SINGLE>
__global__ __launch_bounds__(256) void tree_step_kernel(const SelKArgs a) {
    const int tid = threadIdx.x, b = blockIdx.x, t = a.step, n = a.n;
    const int live = a.seq_active[b];
    const int F = a.F[t], Fn = a.F[t + 1];
    const bool active = tid < F;
    const size_t pb = (size_t)b * a.depth * n, fa = (size_t)a.gridDim_batch * n * OT_MAX_DEPTH;
    const int slot = active ? tid : 0;
    const long long rid = (long long)b * a.rows_per_seq + slot;
    const double lse = a.row_lse[rid];
    float v[KMAX];
    int id[KMAX];
#pragma unroll
    for (int r = 0; r < KMAX; ++r) {
        v[r] = a.row_topv[rid * a.k + min(r, a.k - 1)];
        id[r] = a.row_topi[rid * a.k + min(r, a.k - 1)];
    }
    const double S0 = a.pool_key[pb + (size_t)max(t - 1, 0) * n + slot];
    u32x4 path[kPathVecs];                      // of this lane's frontier node
    const u32x4* const prev = (const u32x4*)(a.front_anc + (size_t)((t & 1) ^ 1) * fa + ((size_t)b * n + slot) * OT_MAX_DEPTH);
#pragma unroll
    for (int q = 0; q < kPathVecs; ++q) path[q] = prev[q];
    asm volatile("" ::: "memory");              // (the loads stay ahead of the branch)
    if (!live) {                                // frozen by the adaptive-depth rule: its tree stays as it is
        if (a.frontier_count && threadIdx.x == 0) a.frontier_count[blockIdx.x] = 0;
        return;
    }
    OT_SELECT_SHARED
    (void)s_cntw;
    const double S = (t == 0 || !active) ? 0.0 : S0;
    double ck[KMAX];
    candidate_scores<KMAX>(S, lse, v, active, a.k, ck);
    int cnt, off;
    double tau;
    layer_cut<KMAX, SINGLE>(ck, (double*)smem, s_hist, active, a.k, F, Fn, a.r0[t], g, cnt, off, tau);
    if (tid == 0) {
        a.step_tau[(size_t)b * a.depth + t] = tau;
        a.seq_steps[b] = t + 1;
        if (a.frontier_count) a.frontier_count[b] = Fn;
    }
#pragma unroll
    for (int r = 0; r < KMAX; ++r) {
        if (r < cnt) {
            const size_t o = pb + (size_t)t * n + off + r;
            a.pool_key[o] = ck[r];
            a.pool_p[o] = exp(ck[r]);             // p^ (Eq. 2), kept for E_sub
            a.pool_tok[o] = id[r];
            a.pool_par[o] = tid;
            a.frontier_token[(size_t)b * n + off + r] = id[r];
            a.frontier_parent[(size_t)b * n + off + r] = tid;
        }
    }
    // Root paths of the new frontier over pool indices ((layer t+1, slot s) -> t n + s): the parent's path plus the
    // node itself -- the incremental form of Algorithm 2's mask for the drafting phase.  A path has at most `depth`
    // entries however many nodes the pool holds, so the state stays small; ot_tree_frontier_mask turns it into bits.
    u32x4* const cur = (u32x4*)(a.front_anc + (size_t)(t & 1) * fa + (size_t)b * n * OT_MAX_DEPTH);
    for (int r = 0; r < cnt; ++r) {
        const unsigned node = (unsigned)(t * n + off + r);
#pragma unroll
        for (int q = 0; q < kPathVecs; ++q) {
            if (q > (t >> 3)) continue;
            u32x4 x = path[q];
            if (q == (t >> 3)) {
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (c == ((t >> 1) & 3)) x[c] = (t & 1) ? (x[c] & 0xffffu) | (node << 16) : node;
            }
            cur[(size_t)(off + r) * kPathVecs + q] = x;
        }
    }
}

template <int DMAX, bool SINGLE>
__global__ __launch_bounds__(256) void tree_finalize_kernel(const SelKArgs a) {
    OT_SELECT_SHARED
    const int NT = blockDim.x, tid = threadIdx.x, b = blockIdx.x, n = a.n;
    const int steps = a.step < a.seq_steps[b] ? a.step : a.seq_steps[b];     // a frozen sequence has fewer layers
    const Pool P = carve_pool(smem, a.depth, NT, DMAX, 0);
    const size_t pb = (size_t)b * a.depth * n;
    double lo0 = nan_d();
    constexpr int BATCH = 8;                    // layers requested at once
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
    OT_SELECT_SHARED
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

SelKArgs make_args(const SelectGeometry& g, const BuildWorkspace& ws) {
    SelKArgs a;
    a.row_lse = ws.row_lse; a.row_topv = ws.row_topv; a.row_topi = ws.row_topi;
    a.k = g.k; a.n = g.n; a.depth = g.depth; a.rows_per_seq = g.rows_per_seq;
    for (int i = 0; i < OT_MAX_DEPTH + 2; ++i) {
        a.F[i] = g.F[i];
        a.r0[i] = 0;
    }
    for (int t = 0; t < g.depth; ++t) {
        const int want = g.F[t + 1], F = g.F[t];
        a.r0[t] = F > 0 ? (want + F - 1) / F - 1 : 0;
    }
    a.pool_key = ws.pool_key; a.pool_tok = ws.pool_tok; a.pool_par = ws.pool_par; a.step_tau = ws.step_tau;
    a.pool_p = ws.pool_p; a.seq_E = ws.seq_E; a.seq_steps = ws.seq_steps; a.seq_active = ws.seq_active;
    a.e_sub = nullptr; a.go_on = nullptr; a.delta = 0.0;
    a.front_anc = ws.front_anc; a.mask_out = nullptr; a.mask_words = 0; a.gridDim_batch = g.batch;
    a.out = ot_tree_out{nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr};
    a.frontier_token = nullptr; a.frontier_parent = nullptr; a.frontier_count = nullptr;
    a.step = 0;
    return a;
}

int threads_for(int n) { return ((n + 63) / 64) * 64; }

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
        if (steps_done <= 8) return launch_esub_t<8, true>(a, g.batch, NT, s);
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
