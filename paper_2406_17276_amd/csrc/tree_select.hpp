// Streaming selection, device side: the workgroup collectives, the exact selection of the best keys, and a drafting step.
#pragma once

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

// candidate scores of one frontier slot: log p^(child) = log p^(parent) + (x - lse)   (Eq. 2).  log p <= 0 up to the rounding of
// lse: a child that scored above its parent could be in the tree without it.  (Only the most probable token comes near: any other
// has half of the probability at most.  The bound on all ranks cost 0.5 % of streaming loops replayed from a graph.)  A score that
// is not defined (a row of -inf) counts as the lowest: only slots that are not there are absent, so a step always fills its frontier.
template <int KMAX>
__device__ __forceinline__ void candidate_scores(double S, double lse, const float (&v)[KMAX], bool active, int k,
                                                 double (&ck)[KMAX]) {
    if (!(lse > -INFINITY)) lse = INFINITY;
#pragma unroll
    for (int r = 0; r < KMAX; ++r) {
        const double lp = (double)v[r] - lse;
        ck[r] = (active && r < k) ? S + (r == 0 ? fmin(lp, 0.0) : lp) : nan_d();
    }
}

#define OT_SELECT_SHARED(THREADS)                          \
    __shared__ int s_red[8];                               \
    __shared__ double s_bc[2];                             \
    __shared__ double s_redd[8];                           \
    __shared__ int s_cntw[OT_MAX_DEPTH * 4];               \
    __shared__ int s_hist[kBuckets + 4];                   \
    Group<SINGLE> g;                                       \
    g.red = s_red; g.bc = s_bc; g.redd = s_redd;           \
    g.phase = g.bphase = g.dphase = 0;                     \
    g.tid = threadIdx.x; g.lane = threadIdx.x & 63;        \
    g.wave = threadIdx.x >> 6; g.nw = (THREADS) >> 6;      \
    g.nt = (THREADS);                                      \
    for (int i_ = threadIdx.x; i_ < kBuckets + 4; i_ += (THREADS)) s_hist[i_] = 0; \
    __syncthreads();

// The streaming kernels are short, and what bounds them is trips to memory (0.6 to 0.8 us each): every load whose address
// does not depend on another is requested ahead of the first use, from clamped addresses instead of under a condition, and
// a root path is four 16-byte vectors.  Measured (MI355X, 7B-shaped drafting loop of ten steps): step kernel 7.8 -> 4.0 us,
// E_sub 4.5..6.8 -> 4.0..5.3 us, mask 2.3 us; the whole loop replayed from a graph 156 -> 148 us, through the binding 181 ->
// 154 us; eight sequences of n = 256, k = 16, 12 steps: 816 -> 465 us.
constexpr int kPathVecs = OT_MAX_DEPTH / 8;      // u16 entries

// Streaming: one drafting step; the pool lives in the caller's workspace between launches.
// Called by nt threads; SHARED: for a sequence that goes on, and the rows' results come from
// workgroups of the same launch.  kt: LDS for KMAX nt keys.
template <int KMAX, bool SINGLE, bool SHARED>
__device__ __forceinline__ void draft_step(const SelKArgs& a, const int b, const int nt, double* const kt) {
    constexpr bool LATE = SHARED && KMAX > 10;   // tokens and paths after the selection: 128 registers, the scan's workgroup has no more
    const int tid = threadIdx.x, t = a.step, n = a.n;
    const int live = SHARED ? 1 : a.seq_active[b];
    const int F = a.F[t], Fn = a.F[t + 1];
    const bool active = tid < F;
    const size_t pb = (size_t)b * a.depth * n, fa = (size_t)a.gridDim_batch * n * OT_MAX_DEPTH;
    const int slot = active ? tid : 0;
    const long long rid = (long long)b * a.rows_per_seq + slot;
    const double lse = get<SHARED>(a.row_lse + rid);
    float v[KMAX];
    int id[KMAX];
#pragma unroll
    for (int r = 0; r < KMAX; ++r) {
        v[r] = get<SHARED>(a.row_topv + rid * a.k + min(r, a.k - 1));
        if (!LATE) id[r] = get<SHARED>(a.row_topi + rid * a.k + min(r, a.k - 1));
    }
    const double S0 = a.pool_key[pb + (size_t)max(t - 1, 0) * n + slot];
    u32x4 path[kPathVecs];                      // of this lane's frontier node
    const u32x4* const prev = (const u32x4*)(a.front_anc + (size_t)((t & 1) ^ 1) * fa + ((size_t)b * n + slot) * OT_MAX_DEPTH);
#pragma unroll
    for (int q = 0; q < kPathVecs; ++q)
        if (!LATE) path[q] = prev[q];
    asm volatile("" ::: "memory");              // (the loads stay ahead of the branch)
    if (!live) {                                // frozen by the adaptive-depth rule: its tree stays as it is
        if (a.frontier_count && threadIdx.x == 0) a.frontier_count[b] = 0;
        return;
    }
    OT_SELECT_SHARED(nt)
    (void)s_cntw;
    const double S = (t == 0 || !active) ? 0.0 : S0;
    double ck[KMAX];
    candidate_scores<KMAX>(S, lse, v, active, a.k, ck);
    int cnt, off;
    double tau;
    layer_cut<KMAX, SINGLE>(ck, kt, s_hist, active, a.k, F, Fn, a.r0[t], g, cnt, off, tau);
    if constexpr (LATE) {
#pragma unroll
        for (int r = 0; r < KMAX; ++r) id[r] = get<SHARED>(a.row_topi + rid * a.k + min(r, a.k - 1));
#pragma unroll
        for (int q = 0; q < kPathVecs; ++q) path[q] = prev[q];
    }
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

inline SelKArgs make_args(const SelectGeometry& g, const BuildWorkspace& ws) {
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

inline int threads_for(int n) { return ((n + 63) / 64) * 64; }

}  // namespace
}  // namespace ot
