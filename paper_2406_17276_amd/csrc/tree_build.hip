// One-shot tree construction: everything of Algorithm 1 that follows the row scan, for a launch whose rows are all in
// memory (ot_build_tree, ot_build_tree_adaptive).
//   per drafting step t: candidate score = score(parent) + (x - lse)            (Eq. 2 in log space)
//                        keep the F_{t+1} = min(n, k F_t) best candidates       (Algorithm 1, "topk")
//                        number them by (parent slot, rank)
//   finally:             the n best nodes of the whole pool                     (Algorithm 1, last line)
//                        output order (depth, slot); parents, depths (= position offsets, Fig. 1),
//                        ancestor bitmask (Algorithm 2), E = sum of p^           (Eq. 3)
//
// What bounds it: a chain of selections in which every step waits for the one before; nothing but the latency of that
// chain counts.  One workgroup per sequence; a thread owns one candidate (two or four in wide shapes), candidate
// c = parent slot * k + rank, so thread order is the order of every tie rule and of the slot numbering.
//
// "Keep the `want` best" = one pass over a fixed-grid histogram: the bin of a score is the exponent and the leading
// mantissa bits of -log p^ (512 bins per octave, and 64 times coarser ones above them).  The grid needs no minimum or
// maximum of the keys first, and it is the same for every step, so a second histogram of the same grid accumulates the
// pool: it locates the n-th best pool node at any time.  Every wavefront finds the cut by itself, one coarse and one fine
// bin per lane (a scan by one wavefront and a broadcast took 1600 cycles of a step, this takes 450).  Keys better than the
// bin of the cut are kept; where the cut falls inside a bin its keys are ranked exactly by counting; crowded bins
// (near-uniform rows, ties) are split again on a linear grid between their smallest and largest key until few are left or
// all are equal, and equal keys go in index order.  Loops over pool nodes stay rolled: the workgroup lands on a compute
// unit whose instruction cache is cold, and every line of straight code is a trip to the L2.
//
// Drafting ends early when the result is known: a child's score never exceeds its parent's, so once n pool nodes score
// above every candidate of a step, neither that step nor any later one has a node in the tree.  (7B-shaped rows: the
// tree is complete after 4 to 7 of 10 steps.)
//
// Measured, MI355X, whole kernel under rocprofv3 (one wavefront per selection before): 7B-shaped build 22 to 24 ->
// 9.9 us, 13B-shaped 9.3.
#include <algorithm>

#include "common.hpp"

namespace ot {
namespace {

typedef unsigned long long u64;

constexpr int kCoarse = 64, kFine = 64, kBins = kCoarse * kFine;
constexpr int kList = 64;              // keys of the cut's bin that are ranked by counting
constexpr int kPoolPerThread = 8;
constexpr double kFloor = -1e300;      // what -inf (or an undefined score) counts as in the selections

struct TreeBuildArgs {
    const int32_t* topi;               // [rows][k]
    int batch_pool;                    // pool nodes a sequence may have = stride of the carried pool arrays
    int stage_off_lse;                 // STAGE: byte offset of the lse table behind the logits table
    double delta; int32_t* steps_used; double* e_sub;                                     // ADAPT
    double* pool_key; int32_t* pool_meta; int32_t* pool_par; int32_t* seq_active; double* seq_E;   // carried between launches
    ot_tree_out out;
};

// Barrier that orders LDS traffic only: loads from global memory stay in flight across it.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

__device__ __forceinline__ int grid_bin(double ks) {
    constexpr int MB = 23 - 9, OFF = (127 - 2) << 9;                           // [2^-2, 2^6): 8 octaves of 8 coarse bins
    const int q = (__float_as_int((float)-ks) >> MB) - OFF;                    // ks > 0 by rounding: negative -> bin 0
    return min(max(q, 0), kBins - 1);
}

struct Hist { int coarse[kCoarse], fine[kBins]; };
__device__ __forceinline__ void hist_add(Hist& h, int bin) {
    atomicAdd(&h.coarse[bin >> 6], 1);
    atomicAdd(&h.fine[bin], 1);
}

// Bin of the `want`-th best key: B, keys in better bins, keys in bin B.  Fewer than `want` keys in all: B = kBins,
// above = all keys, inb = 0.  first: best occupied coarse bin.  Every wavefront for itself.
struct HistCut { int B, above, inb, first; };
__device__ __forceinline__ HistCut hist_cut(const Hist& h, int want, int lane) {
    const int c = h.coarse[lane];
    const int ci = wave_incl_scan(c, lane);
    const u64 any = __ballot(c > 0), hit = __ballot(ci >= want);
    const int C = hit ? __ffsll((long long)hit) - 1 : kCoarse - 1;
    const int f = h.fine[C * kFine + lane];
    const int fi = wave_incl_scan(f, lane) + rl(ci - c, C);
    const u64 fhit = __ballot(fi >= want);
    HistCut r;
    r.first = any ? __ffsll((long long)any) - 1 : kCoarse;
    const int L = fhit ? __ffsll((long long)fhit) - 1 : 63;
    r.B = fhit ? C * kFine + L : kBins;
    r.inb = fhit ? rl(f, L) : 0;
    r.above = rl(fi, L) - r.inb;
    return r;
}

template <int NT>
struct Shared {
    static constexpr int NW = NT / 64;
    Hist cand;                         // candidates of a step; all zero between steps
    Hist pool;                         // pool nodes
    struct { double key; int idx, pad; } list[kList + 4];
    int lcnt;
    u64 mn, mx;
    int wc[NW * kPoolPerThread];
    double red[NW];
    // tree nodes by output index
    double rec_key[OT_MAX_NODES];
    int rec_tok[OT_MAX_NODES];
    unsigned short rec_pool[OT_MAX_NODES];
    unsigned short rec_par[OT_MAX_NODES];
};

// Of the keys flagged in `in` (m of them in the workgroup, `need` to be kept, 0 < need < m), which of this thread's are
// among the `need` best; equal keys: smaller index first, index = i NT + tid, i < iters.  key(i): this thread's key i.
// lcnt and the histogram s.cand are zero on entry.  Called by the whole workgroup.
template <int NT, int UNROLL, typename KEY>
__device__ __forceinline__ unsigned resolve_bin(KEY key, int iters, unsigned in, int m, int need, Shared<NT>& s, int tid, int lane,
                                                int wave) {
    constexpr int NW = NT / 64;
    unsigned keep = 0u;
    while (m > kList) {
        if (tid == 0) { s.mn = ~0ull; s.mx = 0ull; }
        lds_barrier();
#pragma unroll UNROLL
        for (int i = 0; i < iters; ++i)
            if ((in >> i) & 1u) {
                const u64 q = f64_key(key(i));
                atomicMin(&s.mn, q); atomicMax(&s.mx, q);
            }
        lds_barrier();
        const u64 mn = s.mn, mx = s.mx;
        if (mn == mx) {                                       // all equal: the first `need` in index order
#pragma unroll UNROLL
            for (int i = 0; i < iters; ++i) {
                const u64 bal = __ballot((in >> i) & 1u);
                if (lane == 0) s.wc[i * NW + wave] = __popcll(bal);
            }
            lds_barrier();
            int before = 0;
#pragma unroll UNROLL
            for (int i = 0; i < iters; ++i) {
                const u64 bal = __ballot((in >> i) & 1u);
#pragma unroll 1
                for (int w = 0; w < NW; ++w) {
                    const int c = s.wc[i * NW + w];
                    if (w == wave) {
                        const int r = before + __popcll(bal & ((1ull << lane) - 1ull));
                        if (((in >> i) & 1u) && r < need) keep |= 1u << i;
                    }
                    before += c;
                }
            }
            lds_barrier();                                    // wc is free again
            return keep;
        }
        const double lo = key_f64(mn), hi = key_f64(mx);
        // smallest key -> last bin, largest key -> bin 0: at least two bins are occupied, so every round splits
        const double scale = (double)(kBins - 1) / (hi - lo);
        auto bin_of = [&](double q) { return q == lo ? kBins - 1 : min((int)((hi - q) * scale), kBins - 2); };
#pragma unroll UNROLL
        for (int i = 0; i < iters; ++i)
            if ((in >> i) & 1u) hist_add(s.cand, bin_of(key(i)));
        lds_barrier();
        const HistCut c = hist_cut(s.cand, need, lane);
        lds_barrier();
        unsigned left = 0u;
#pragma unroll UNROLL
        for (int i = 0; i < iters; ++i)
            if ((in >> i) & 1u) {
                const int bin = bin_of(key(i));
                s.cand.fine[bin] = 0; s.cand.coarse[bin >> 6] = 0;
                keep |= (bin < c.B ? 1u : 0u) << i;
                left |= (bin == c.B ? 1u : 0u) << i;
            }
        need -= c.above; m = c.inb; in = left;
        if (need == m) return keep | in;
    }
#pragma unroll UNROLL
    for (int i = 0; i < iters; ++i)
        if ((in >> i) & 1u) {
            const int q = atomicAdd(&s.lcnt, 1);
            s.list[q].key = key(i); s.list[q].idx = i * NT + tid;
        }
    lds_barrier();
#pragma unroll UNROLL
    for (int i = 0; i < iters; ++i)
        if ((in >> i) & 1u) {
            const double mine = key(i);
            const int id = i * NT + tid;
            int rank = 0;
#pragma unroll 1
            for (int q = 0; q < m; q += 4) {                  // four rivals per trip to LDS
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const double u = s.list[q + e].key;
                    const int ui = s.list[q + e].idx;
                    rank += (q + e < m && (u > mine || (u == mine && ui < id))) ? 1 : 0;
                }
            }
            keep |= (rank < need ? 1u : 0u) << i;
        }
    return keep;
}

// The n best pool nodes: flags of this thread's pool nodes (node i NT + tid, bit i).
template <int NT>
__device__ __forceinline__ unsigned pool_best(const double* pkey, int pool, int n, Shared<NT>& s, int tid, int lane, int wave) {
    const HistCut cut = hist_cut(s.pool, n, lane);
    unsigned keep = 0u, in = 0u;
    const int iters = (pool + NT - 1) / NT;
    auto key = [&](int i) { return fmax(pkey[i * NT + tid], kFloor); };
#pragma unroll 1
    for (int i = 0; i < iters; ++i)
        if (i * NT + tid < pool) {
            const int bin = grid_bin(key(i));
            keep |= (bin < cut.B ? 1u : 0u) << i;
            in |= (bin == cut.B ? 1u : 0u) << i;
        }
    const int need = n - cut.above;
    if (cut.inb == need) keep |= in;
    else if (cut.inb > need) keep |= resolve_bin<NT, 1>(key, iters, in, cut.inb, need, s, tid, lane, wave);
    return keep;
}

// KPT candidates per thread.  STAGE: the launch's logits and normalisers are copied to LDS first (all trips to memory
// overlap, once); otherwise every step's are fetched one step ahead.  ADAPT: Algorithm 1 with its stopping rule -- after
// every step E_sub(T, n) = sum of p^ over the n best pool nodes, and drafting stops when E_sub - E <= delta.
// Steps t0 .. t1-1 are drafted; a sequence that is not finished then leaves its pool in memory for the next launch.
template <int NT, int KPT, bool STAGE, bool ADAPT>
__global__ __launch_bounds__(NT) void tree_build_kernel(const float* topv, const double* row_lse, const int k, const int rows,
                                                        const int n, const int depth, const int t0, const int t1,
                                                        const TreeBuildArgs a) {
    constexpr int NW = NT / 64;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ Shared<NT> s;
    const int tid = threadIdx.x, b = blockIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (t0 > 0 && a.seq_active[b] == 0) return;

    // frontier sizes ahead of step t0 (Algorithm 1: F_0 = 1, F_{t+1} = min(n, k F_t)); rs = rows before step t0, and
    // pool node (layer t+1, slot j) has index row_start(t+1) + j - 1: layer after layer without gaps
    int F = 1, rs = 0;
    for (int t = 0; t < t0; ++t) { rs += F; F = min(n, k * F); }
    int rows_here = rows - rs;                                // rows of steps t0 .. t1-1
    if (t1 < depth) {
        rows_here = 0;
        int f = F;
        for (int t = t0; t < t1; ++t) { rows_here += f; f = min(n, k * f); }
    }
    double* const pkey = (double*)smem;
    unsigned* const pmeta = (unsigned*)(pkey + a.batch_pool);                 // index into topv / topi | depth << 20
    unsigned short* const ppar = (unsigned short*)(pmeta + a.batch_pool);     // pool index of the parent, 0xffff: root
    unsigned char* const oidx = (unsigned char*)(ppar + a.batch_pool);        // output index of a selected node
    float* const sv = (float*)(((uintptr_t)(oidx + a.batch_pool) + 15) & ~(uintptr_t)15);
    double* const sl = (double*)((char*)sv + a.stage_off_lse);
    const size_t rbase = (size_t)b * rows;
    const float* const gv = topv + (rbase + rs) * k;
    const double* const gl = row_lse + rbase + rs;
    const int rs0 = rs;

    // ---- prologue: the loads first, the histograms are cleared under them ----
    float v[KPT];
    double l[KPT];
    int cj[KPT];                                              // parent slot of this thread's candidates
    if (STAGE) {
        constexpr int VB = 8, LB = 2;
        const int nv = rows_here * k;
        for (int base = 0; base < nv; base += VB * NT) {      // a batch of loads per trip to memory
            float x[VB];
            double y[LB];
            const int lb = (base / (VB * NT)) * (LB * NT);
#pragma unroll
            for (int u = 0; u < VB; ++u) x[u] = gv[min(base + u * NT + tid, nv - 1)];
#pragma unroll
            for (int u = 0; u < LB; ++u) y[u] = gl[min(lb + u * NT + tid, rows_here - 1)];
            if (base == 0) {
                for (int i = tid; i < (int)(sizeof(Hist) * 2 / 16); i += NT) ((int4*)&s.cand)[i] = int4{0, 0, 0, 0};
            }
#pragma unroll
            for (int u = 0; u < VB; ++u) { const int i = base + u * NT + tid; if (i < nv) sv[i] = x[u]; }
#pragma unroll
            for (int u = 0; u < LB; ++u) { const int i = lb + u * NT + tid; if (i < rows_here) sl[i] = y[u]; }
        }
        for (int i = (nv + VB * NT - 1) / (VB * NT) * (LB * NT) + tid; i < rows_here; i += NT) sl[i] = gl[i];
#pragma unroll
        for (int i = 0; i < KPT; ++i) cj[i] = (i * NT + tid) / k;
    } else {
#pragma unroll
        for (int i = 0; i < KPT; ++i) {
            const int c = min(i * NT + tid, k * F - 1);
            v[i] = gv[c];
            cj[i] = (i * NT + tid) / k;
            l[i] = gl[min(cj[i], F - 1)];
        }
        for (int i = tid; i < (int)(sizeof(Hist) * 2 / 16); i += NT) ((int4*)&s.cand)[i] = int4{0, 0, 0, 0};
    }
    __syncthreads();
    int pool = t0 > 0 ? rs - 1 + F : 0;                       // nodes drafted so far
    if (t0 > 0) {
        for (int i = tid; i < pool; i += NT) {
            const size_t o = (size_t)b * a.batch_pool + i;
            const double q = a.pool_key[o];
            pkey[i] = q;
            pmeta[i] = (unsigned)a.pool_meta[o];
            ppar[i] = (unsigned short)a.pool_par[o];
            hist_add(s.pool, grid_bin(fmax(q, kFloor)));
        }
        lds_barrier();
    }

    double E_prev = (ADAPT && t0 > 0) ? a.seq_E[b] : 0.0, E_sub = 0.0;
    unsigned pkeep = 0u;                                      // ADAPT: the n best pool nodes after the last step
    int steps = t1;
    bool done = t1 == depth, complete = false;
    for (int t = t0; t < t1; ++t) {
        const int Fn = min(n, k * F), C = k * F;
        float vn[KPT];
        double ln[KPT];
        if (!STAGE && t + 1 < t1) {                           // the next step's rows: their place does not depend on the tree
            const float* nv = gv + (size_t)(rs + F - rs0) * k;
            const double* nl = gl + (rs + F - rs0);
#pragma unroll
            for (int i = 0; i < KPT; ++i) {
                vn[i] = nv[min(i * NT + tid, k * Fn - 1)];
                ln[i] = nl[min(cj[i], Fn - 1)];
            }
        }
        double raw[KPT];
        int bin[KPT], idx[KPT];
        unsigned keep = 0u;
#pragma unroll
        for (int i = 0; i < KPT; ++i) {
            const int c = i * NT + tid;
            raw[i] = 0.0; bin[i] = 0; idx[i] = c;
            if (c < C) {
                keep |= 1u << i;
                if (STAGE) { v[i] = sv[(rs - rs0) * k + c]; l[i] = sl[rs - rs0 + cj[i]]; }
                const double S = t == 0 ? 0.0 : pkey[rs - 1 + cj[i]];
                // log p^(child) = log p^(parent) + log p (Eq. 2); log p <= 0 up to the rounding of lse
                const double lp = (double)v[i] - l[i];
                raw[i] = S + (lp > 0.0 ? 0.0 : lp);
                bin[i] = grid_bin(fmax(raw[i], kFloor));
                if (C > Fn) hist_add(s.cand, bin[i]);
            }
        }
        if (C > Fn) {
            if (tid == 0) s.lcnt = 0;
            lds_barrier();
            const HistCut cut = hist_cut(s.cand, Fn, lane);
            // complete when n pool nodes are better than every candidate; a look at the coarse bins settles most steps
            const int pc = s.pool.coarse[lane];
            const int pi = wave_incl_scan(pc, lane);
            const u64 ph = __ballot(pi >= n);
            const int PC = ph ? __ffsll((long long)ph) - 1 : kCoarse;
            complete = cut.first > PC;
            if (cut.first == PC) {
                const u64 cf = __ballot(s.cand.fine[PC * kFine + lane] > 0);
                const int pf = wave_incl_scan(s.pool.fine[PC * kFine + lane], lane) + rl(pi - pc, PC);
                complete = __ffsll((long long)cf) > __ffsll((long long)__ballot(pf >= n));
            }
            if (complete) {
                done = true;
                steps = t;
                lds_barrier();
#pragma unroll
                for (int i = 0; i < KPT; ++i)
                    if ((keep >> i) & 1u) { s.cand.fine[bin[i]] = 0; s.cand.coarse[bin[i] >> 6] = 0; }
                if (ADAPT) { steps = (a.delta >= 0.0) ? t + 1 : depth; E_sub = E_prev; }
                break;
            }
            unsigned in = 0u, better = 0u;
#pragma unroll
            for (int i = 0; i < KPT; ++i) {
                better |= (bin[i] < cut.B ? 1u : 0u) << i;
                in |= (bin[i] == cut.B ? 1u : 0u) << i;
            }
            const unsigned act = keep;
            in &= act;
            keep &= better;
            const int need = Fn - cut.above;
            if (cut.inb == need) keep |= in;
            const bool crowded = cut.inb > need && cut.inb > kList;
            auto clear = [&]() {
#pragma unroll
                for (int i = 0; i < KPT; ++i)
                    if ((act >> i) & 1u) { s.cand.fine[bin[i]] = 0; s.cand.coarse[bin[i] >> 6] = 0; }
            };
            if (cut.inb > need) {
                if (crowded) { lds_barrier(); clear(); }      // the histogram is used again
                auto key = [&](int i) {
                    return fmax(raw[i], kFloor);
                };
                keep |= resolve_bin<NT, KPT>(key, KPT, in, cut.inb, need, s, tid, lane, wave);
            }
            // slot of a kept candidate = its rank among the kept ones in index order
            u64 bal[KPT];
#pragma unroll
            for (int i = 0; i < KPT; ++i) {
                bal[i] = __ballot((keep >> i) & 1u);
                if (lane == 0) s.wc[i * NW + wave] = __popcll(bal[i]);
            }
            lds_barrier();
            if (!crowded) clear();                            // everybody has read the histogram
            const int c0 = lane < KPT * NW ? s.wc[lane] : 0;
            const int e0 = wave_incl_scan(c0, lane) - c0;
#pragma unroll
            for (int i = 0; i < KPT; ++i) idx[i] = rl(e0, i * NW + wave) + __popcll(bal[i] & ((1ull << lane) - 1ull));
        }
        pool = rs + F - 1 + Fn;
#pragma unroll
        for (int i = 0; i < KPT; ++i) {
            if ((keep >> i) & 1u) {
                const int p = rs + F - 1 + idx[i];
                pkey[p] = raw[i];
                pmeta[p] = (unsigned)(rs * k + i * NT + tid) | (unsigned)(t + 1) << 20;
                ppar[p] = t == 0 ? (unsigned short)0xffff : (unsigned short)(rs - 1 + cj[i]);
                hist_add(s.pool, bin[i]);
            }
        }
        if (ADAPT && tid == 0) s.lcnt = 0;
        lds_barrier();
        rs += F; F = Fn;
        if (!STAGE) {
#pragma unroll
            for (int i = 0; i < KPT; ++i) { v[i] = vn[i]; l[i] = ln[i]; }
        }
        if (ADAPT) {
            pkeep = pool_best<NT>(pkey, pool, n, s, tid, lane, wave);
            double e = 0.0;                                   // fp64 exp, as in the streaming form: both stop at the same step
#pragma unroll 1
            for (int i = 0; i * NT < pool; ++i)
                if ((pkeep >> i) & 1u) e += exp(pkey[i * NT + tid]);
            e = wave_sum_d(e);
            if (lane == 0) s.red[wave] = e;
            lds_barrier();
            E_sub = 0.0;
#pragma unroll
            for (int w = 0; w < NW; ++w) E_sub += s.red[w];
            if (t + 1 < depth) {                              // the loop condition of Algorithm 1
                if (!(E_sub - E_prev > a.delta)) { done = true; steps = t + 1; break; }
                E_prev = E_sub;
            }
        }
    }
    if (!done) {                                              // more steps in a later launch
        for (int i = tid; i < pool; i += NT) {
            const size_t o = (size_t)b * a.batch_pool + i;
            a.pool_key[o] = pkey[i];
            a.pool_meta[o] = (int32_t)pmeta[i];
            a.pool_par[o] = (int32_t)ppar[i];
        }
        if (tid == 0) {
            a.seq_active[b] = 1;
            if (ADAPT) a.seq_E[b] = E_prev;
        }
        return;
    }

    // ---- last line of Algorithm 1: the n best nodes of the pool ----
    const int n_out = min(pool, n), iters = (pool + NT - 1) / NT;
    const int32_t* const ti = a.topi + rbase * k;
    // token id of the first node of this thread (all of them, mostly): in flight during the selection
    const int tok0 = ti[pmeta[min(tid, pool - 1)] & 0xfffffu];
    unsigned keep = pkeep;                                    // ADAPT: the set behind the last E_sub
    if (!ADAPT || complete) {
        if (!complete) {
            if (tid == 0) s.lcnt = 0;
            lds_barrier();
        }
        keep = pool_best<NT>(pkey, pool, n, s, tid, lane, wave);
    }
    // output index = rank in (depth, slot) order among the selected nodes
#pragma unroll 1
    for (int i = 0; i < iters; ++i) {
        const u64 bal = __ballot((keep >> i) & 1u);
        if (lane == 0) s.wc[i * NW + wave] = __popcll(bal);
    }
    lds_barrier();
    int carry = 0;
#pragma unroll 1
    for (int i = 0; i < iters; ++i) {
        const int c = lane < NW ? s.wc[i * NW + lane] : 0;
        const int inc = wave_incl_scan(c, lane);
        const u64 bal = __ballot((keep >> i) & 1u);
        const int base = carry + rl(inc - c, wave);           // (outside the branch: all lanes take part)
        if ((keep >> i) & 1u) {
            const int p = i * NT + tid, o = base + __popcll(bal & ((1ull << lane) - 1ull));
            oidx[p] = (unsigned char)o;
            s.rec_key[o] = pkey[p];
            s.rec_tok[o] = i == 0 ? tok0 : ti[pmeta[p] & 0xfffffu];
            s.rec_pool[o] = (unsigned short)p;
        }
        carry += rl(inc, 63);
    }
    lds_barrier();
    const bool node = tid < n_out;
    int p = 0, par = -1;
    if (node) {
        p = s.rec_pool[tid];
        const int pp = ppar[p];
        if (pp != 0xffff) par = (int)oidx[pp];
        s.rec_par[tid] = (unsigned short)par;
    }
    if (n > 64) lds_barrier();
    else asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // node i = thread i: wavefront 0 alone
    if (n <= 64 && wave > 0) return;
    const int W = OT_MASK_WORDS(n);
    const size_t ob = (size_t)b * n + tid;
    const double key = node ? s.rec_key[tid] : -INFINITY;
    if (tid < n) {
        a.out.token[ob] = node ? s.rec_tok[tid] : -1;
        a.out.parent[ob] = par;
        a.out.depth[ob] = node ? (int)(pmeta[p] >> 20) : 0;
        a.out.score[ob] = (float)key;
    }
    // ancestors (Algorithm 2): the parents' output indices up to the root
    int o = node ? tid : -1;
    if (W == 1) {
        u64 row = 0ull;
        for (int guard = 0; guard < OT_MAX_DEPTH && o >= 0; ++guard) {
            row |= 1ull << (o & 63);
            o = guard == 0 ? par : (int)(short)s.rec_par[o];
        }
        if (tid < n) a.out.mask[ob] = row;
    } else {
        u64 row[4] = {0ull, 0ull, 0ull, 0ull};
        for (int guard = 0; guard < OT_MAX_DEPTH && o >= 0; ++guard) {
            const u64 bit = 1ull << (o & 63);
#pragma unroll
            for (int w = 0; w < 4; ++w) row[w] |= (w == (o >> 6)) ? bit : 0ull;
            o = guard == 0 ? par : (int)(short)s.rec_par[o];
        }
        if (tid < n) {
#pragma unroll
            for (int w = 0; w < 4; ++w)
                if (w < W) a.out.mask[ob * W + w] = row[w];
        }
    }
    // E = sum of p^ (Eq. 3)
    double e = wave_sum_d(node ? exp(key) : 0.0);
    if (n > 64) {
        if (lane == 0) s.red[wave] = e;
        lds_barrier();
        e = s.red[0];
        for (int w = 1; w * 64 < n; ++w) e += s.red[w];
    }
    if (tid == 0) {
        a.out.expect[b] = e;
        a.out.n_out[b] = n_out;
        if (a.seq_active) a.seq_active[b] = 0;
        if (ADAPT) { a.steps_used[b] = steps; a.e_sub[b] = E_sub; }
    }
}

// LDS a workgroup may use in all (of the 160 KB of a compute unit)
constexpr size_t kLdsLimit = 160 * 1024;
size_t pool_bytes(int pool) { return ((size_t)pool * (8 + 4 + 2 + 1) + 15) / 16 * 16; }

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
