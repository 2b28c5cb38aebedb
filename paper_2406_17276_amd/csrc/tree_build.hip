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
// mantissa bits of -log p^ (64 or 128 bins per octave).  The grid needs no minimum or maximum of the keys first, and it
// is the same for every step, so a second histogram of the same grid accumulates the pool: it locates the n-th best
// pool node at any time.  Keys better than the bin of the cut are kept, the few keys inside it are ranked exactly by
// counting; crowded bins (near-uniform rows, ties) are split again on a linear grid between their smallest and largest
// key until few are left or all are equal, and equal keys go in index order.
//
// Drafting ends early when the result is known: a child's score never exceeds its parent's, so once n pool nodes score
// above every candidate of a step, neither that step nor any later one has a node in the tree.  (7B-shaped rows: the
// tree is complete after 4 to 7 of 10 steps.)
//
// Measured, MI355X, whole kernel: see the dispatch rule at the end of the file.
#include "common.hpp"

namespace ot {
namespace {

typedef unsigned long long u64;

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

template <int NB>
__device__ __forceinline__ int grid_bin(double ks) {
    constexpr int MB = NB == 512 ? 17 : 16, OFF = (127 - 2) << (23 - MB);      // [2^-2, 2^6) in 8 octaves
    const int q = (__float_as_int((float)-ks) >> MB) - OFF;                    // ks > 0 by rounding: negative -> bin 0
    return min(max(q, 0), NB - 1);
}

// Bin of the `want`-th best key: B, keys in better bins, keys in bin B, best occupied bin (NB: none).  Fewer than
// `want` keys in all: B = NB, above = all keys, inb = 0.  One wavefront; clears what it read if CLEAR.
struct HistCut { int B, above, inb, first; };
template <int NB, bool CLEAR>
__device__ __forceinline__ HistCut hist_scan(int* hist, int want, int lane) {
    constexpr int BPL = NB / 64;
    int c[BPL];
    int4* h4 = (int4*)(hist + BPL * lane);
#pragma unroll
    for (int i = 0; i < BPL / 4; ++i) {
        const int4 q = h4[i];
        c[4 * i] = q.x; c[4 * i + 1] = q.y; c[4 * i + 2] = q.z; c[4 * i + 3] = q.w;
    }
    if (CLEAR) {
#pragma unroll
        for (int i = 0; i < BPL / 4; ++i) h4[i] = int4{0, 0, 0, 0};
    }
    int sum = 0;
#pragma unroll
    for (int i = 0; i < BPL; ++i) sum += c[i];
    const int incl = wave_incl_scan(sum, lane);
    const int before = incl - sum;
    int Bl = 0, abl = before, inl = 0, fl = 0;
    bool found = false, some = false;
#pragma unroll
    for (int i = 0; i < BPL; ++i) {
        if (!some && c[i] > 0) { some = true; fl = i; }
        if (!found) {
            if (abl + c[i] >= want) { found = true; Bl = i; inl = c[i]; }
            else abl += c[i];
        }
    }
    HistCut r;
    const u64 any = __ballot(some);
    const u64 hit = __ballot(before < want && incl >= want);
    const int f = any ? __ffsll((long long)any) - 1 : 0;
    r.first = any ? BPL * f + rl(fl, f) : NB;
    const int src = hit ? __ffsll((long long)hit) - 1 : 0;
    r.B = hit ? BPL * src + rl(Bl, src) : NB;
    r.above = hit ? rl(abl, src) : rl(incl, 63);
    r.inb = hit ? rl(inl, src) : 0;
    return r;
}

template <int NT, int NB>
struct Shared {
    static constexpr int NW = NT / 64;
    int hist[NB];                      // all zero between uses
    int phist[NB];                     // pool nodes by bin
    int4 cut, pcut;
    double lkey[kList];
    int lidx[kList];
    int lcnt;
    u64 mn, mx;
    int wc[NW * kPoolPerThread];
    double red[NW];
    // tree nodes by output index
    double rec_key[OT_MAX_NODES];
    int rec_tok[OT_MAX_NODES];
    unsigned short rec_pool[OT_MAX_NODES];
};

// Of the keys flagged in `in` (m of them in the workgroup, `need` to be kept, 0 < need < m), which of this thread's are
// among the `need` best; equal keys: smaller index first, index = i NT + tid.  lcnt is zero on entry.  Called by the
// whole workgroup.
template <int K, int NT, int NB>
__device__ unsigned resolve_bin(const double (&key)[K], unsigned in, int m, int need, Shared<NT, NB>& s, int tid, int lane, int wave) {
    constexpr int NW = NT / 64;
    unsigned keep = 0u;
    while (m > kList) {
        if (tid == 0) { s.mn = ~0ull; s.mx = 0ull; }
        lds_barrier();
#pragma unroll
        for (int i = 0; i < K; ++i)
            if ((in >> i) & 1u) {
                const u64 q = f64_key(key[i]);
                atomicMin(&s.mn, q); atomicMax(&s.mx, q);
            }
        lds_barrier();
        const u64 mn = s.mn, mx = s.mx;
        if (mn == mx) {                                       // all equal: the first `need` in index order
#pragma unroll
            for (int i = 0; i < K; ++i) {
                const u64 bal = __ballot((in >> i) & 1u);
                if (lane == 0) s.wc[i * NW + wave] = __popcll(bal);
            }
            lds_barrier();
            int before = 0;
            for (int i = 0; i < K; ++i) {
                const u64 bal = __ballot((in >> i) & 1u);
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
        const double scale = (double)(NB - 1) / (hi - lo);
        int bin[K];
#pragma unroll
        for (int i = 0; i < K; ++i) {
            bin[i] = -1;
            if ((in >> i) & 1u) {
                bin[i] = key[i] == lo ? NB - 1 : min((int)((hi - key[i]) * scale), NB - 2);
                atomicAdd(&s.hist[bin[i]], 1);
            }
        }
        lds_barrier();
        if (wave == 0) {
            const HistCut c = hist_scan<NB, true>(s.hist, need, lane);
            if (lane == 0) s.cut = int4{c.B, c.above, c.inb, c.first};
        }
        lds_barrier();
        const int4 c = s.cut;
        unsigned left = 0u;
#pragma unroll
        for (int i = 0; i < K; ++i) {
            if (bin[i] >= 0 && bin[i] < c.x) keep |= 1u << i;
            if (bin[i] == c.x) left |= 1u << i;
        }
        need -= c.y; m = c.z; in = left;
        if (need == m) return keep | in;
    }
#pragma unroll
    for (int i = 0; i < K; ++i)
        if ((in >> i) & 1u) {
            const int p = atomicAdd(&s.lcnt, 1);
            s.lkey[p] = key[i]; s.lidx[p] = i * NT + tid;
        }
    lds_barrier();
#pragma unroll
    for (int i = 0; i < K; ++i)
        if ((in >> i) & 1u) {
            int rank = 0;
            for (int q = 0; q < m; ++q) {
                const double u = s.lkey[q];
                rank += (u > key[i] || (u == key[i] && s.lidx[q] < i * NT + tid)) ? 1 : 0;
            }
            if (rank < need) keep |= 1u << i;
        }
    return keep;
}

// Rank of every kept key among the kept keys in index order (i NT + tid).
template <int K, int NT, int NB>
__device__ __forceinline__ void rank_kept(unsigned keep, int (&idx)[K], Shared<NT, NB>& s, int lane, int wave) {
    constexpr int NW = NT / 64, E = K * NW;
    u64 bal[K];
#pragma unroll
    for (int i = 0; i < K; ++i) {
        bal[i] = __ballot((keep >> i) & 1u);
        if (lane == 0) s.wc[i * NW + wave] = __popcll(bal[i]);
    }
    lds_barrier();
    const int c0 = lane < E ? s.wc[lane] : 0;
    const int e0 = wave_incl_scan(c0, lane) - c0;
    int e1 = 0;
    if (E > 64) {
        const int c1 = 64 + lane < E ? s.wc[64 + lane] : 0;
        e1 = wave_incl_scan(c1, lane) - c1 + rl(e0 + c0, 63);
    }
#pragma unroll
    for (int i = 0; i < K; ++i) {
        const int e = i * NW + wave;
        const int base = e < 64 ? rl(e0, e) : rl(e1, e - 64);
        idx[i] = base + __popcll(bal[i] & ((1ull << lane) - 1ull));
    }
}

// The n best pool nodes: flags of this thread's pool nodes (node i NT + tid).  pcut = cut of the pool histogram.
template <int NT, int NB>
__device__ __forceinline__ unsigned pool_best(const double (&pk)[kPoolPerThread], int pool, int n, int4 pcut, Shared<NT, NB>& s,
                                              int tid, int lane, int wave) {
    unsigned keep = 0u, in = 0u;
#pragma unroll
    for (int i = 0; i < kPoolPerThread; ++i) {
        if (i * NT >= pool) break;
        if (i * NT + tid < pool) {
            const int bin = grid_bin<NB>(pk[i]);
            keep |= (bin < pcut.x ? 1u : 0u) << i;
            in |= (bin == pcut.x ? 1u : 0u) << i;
        }
    }
    const int need = n - pcut.y;
    if (pcut.z == need) keep |= in;
    else if (pcut.z > need) keep |= resolve_bin<kPoolPerThread, NT, NB>(pk, in, pcut.z, need, s, tid, lane, wave);
    return keep;
}

// KPT candidates per thread.  STAGE: the launch's logits and normalisers are copied to LDS first (all trips to memory
// overlap, once); otherwise every step's are fetched one step ahead.  ADAPT: Algorithm 1 with its stopping rule -- after
// every step E_sub(T, n) = sum of p^ over the n best pool nodes, and drafting stops when E_sub - E <= delta.
// Steps t0 .. t1-1 are drafted; a sequence that is not finished then leaves its pool in memory for the next launch.
template <int NT, int KPT, int NB, bool STAGE, bool ADAPT>
__global__ __launch_bounds__(NT) void tree_build_kernel(const float* topv, const double* row_lse, const int k, const int rows,
                                                        const int n, const int depth, const int t0, const int t1,
                                                        const TreeBuildArgs a) {
    constexpr int NW = NT / 64;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ Shared<NT, NB> s;
    const int tid = threadIdx.x, b = blockIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (t0 > 0 && a.seq_active[b] == 0) return;

    // frontier sizes ahead of step t0 (Algorithm 1: F_0 = 1, F_{t+1} = min(n, k F_t)); rs = rows before step t0, and
    // pool node (layer t+1, slot j) has index row_start(t+1) + j - 1: layer after layer without gaps
    int F = 1, rs = 0;
    for (int t = 0; t < t0; ++t) { rs += F; F = min(n, k * F); }
    int rows_here = 0;                                        // rows of steps t0 .. t1-1
    {
        int f = F;
        for (int t = t0; t < t1; ++t) { rows_here += f; f = min(n, k * f); }
    }
    double* const pkey = (double*)smem;
    unsigned* const pmeta = (unsigned*)(pkey + a.batch_pool);                 // index into topv / topi | depth << 20
    unsigned short* const ppar = (unsigned short*)(pmeta + a.batch_pool);     // pool index of the parent, 0xffff: root
    unsigned short* const oidx = ppar + a.batch_pool;                         // output index of a selected node
    float* const sv = (float*)(((uintptr_t)(oidx + a.batch_pool) + 15) & ~(uintptr_t)15);
    double* const sl = (double*)((char*)sv + a.stage_off_lse);
    const size_t rbase = (size_t)b * rows;
    const float* const gv = topv + (rbase + rs) * k;
    const double* const gl = row_lse + rbase + rs;
    const int rs0 = rs;

    // this thread's candidates: parent slots
    int cj[KPT];
#pragma unroll
    for (int i = 0; i < KPT; ++i) cj[i] = (i * NT + tid) / k;

    float v[KPT];
    double l[KPT];
    if (STAGE) {
        for (int i = tid; i < rows_here * k; i += NT) sv[i] = gv[i];
        for (int i = tid; i < rows_here; i += NT) sl[i] = gl[i];
    } else {
#pragma unroll
        for (int i = 0; i < KPT; ++i) {
            const bool act = i * NT + tid < k * F;
            v[i] = act ? gv[i * NT + tid] : 0.f;
            l[i] = act ? gl[cj[i]] : 0.0;
        }
    }
    for (int i = tid; i < NB; i += NT) { s.hist[i] = 0; s.phist[i] = 0; }
    __syncthreads();
    int pool = t0 > 0 ? rs - 1 + F : 0;                       // nodes drafted so far
    if (t0 > 0) {
        for (int i = tid; i < pool; i += NT) {
            const size_t o = (size_t)b * a.batch_pool + i;
            const double q = a.pool_key[o];
            pkey[i] = q;
            pmeta[i] = (unsigned)a.pool_meta[o];
            ppar[i] = (unsigned short)a.pool_par[o];
            atomicAdd(&s.phist[grid_bin<NB>(fmax(q, kFloor))], 1);
        }
        lds_barrier();
    }

    double E_prev = (ADAPT && t0 > 0) ? a.seq_E[b] : 0.0, E_sub = 0.0;
    unsigned pkeep = 0u;                                      // ADAPT: the n best pool nodes after the last step
    int steps = t1;
    bool done = t1 == depth, have_pcut = false;
    for (int t = t0; t < t1; ++t) {
        const int Fn = min(n, k * F), C = k * F;
        float vn[KPT];
        double ln[KPT];
        if (!STAGE && t + 1 < t1) {                           // the next step's rows: their place does not depend on the tree
            const float* nv = gv + (size_t)(rs + F - rs0) * k;
            const double* nl = gl + (rs + F - rs0);
#pragma unroll
            for (int i = 0; i < KPT; ++i) {
                const bool act = i * NT + tid < k * Fn;
                vn[i] = act ? nv[i * NT + tid] : 0.f;
                ln[i] = act ? nl[cj[i]] : 0.0;
            }
        }
        double raw[KPT], ks[KPT];
        int bin[KPT];
        unsigned keep = 0u;
#pragma unroll
        for (int i = 0; i < KPT; ++i) {
            const int c = i * NT + tid;
            raw[i] = 0.0; ks[i] = 0.0; bin[i] = 0;
            if (c < C) {
                keep |= 1u << i;
                if (STAGE) { v[i] = sv[(rs - rs0) * k + c]; l[i] = sl[rs - rs0 + cj[i]]; }
                const double S = t == 0 ? 0.0 : pkey[rs - 1 + cj[i]];
                // log p^(child) = log p^(parent) + log p (Eq. 2); log p <= 0 up to the rounding of lse
                const double lp = (double)v[i] - l[i];
                raw[i] = S + (lp > 0.0 ? 0.0 : lp);
                ks[i] = fmax(raw[i], kFloor);
                bin[i] = grid_bin<NB>(ks[i]);
                if (C > Fn) atomicAdd(&s.hist[bin[i]], 1);
            }
        }
        int idx[KPT];
        if (C > Fn) {
            if (tid == 0) s.lcnt = 0;
            lds_barrier();
            if (wave == 0) {
                const HistCut c = hist_scan<NB, true>(s.hist, Fn, lane);
                if (lane == 0) s.cut = int4{c.B, c.above, c.inb, c.first};
            } else if (wave == 1) {
                const HistCut c = hist_scan<NB, false>(s.phist, n, lane);
                if (lane == 0) s.pcut = int4{c.B, c.above, c.inb, c.first};
            }
            lds_barrier();
            const int4 cut = s.cut;
            if (cut.w > s.pcut.x) {                           // n pool nodes are better than every candidate: complete
                done = true; have_pcut = true;
                steps = t;
                if (ADAPT) { steps = (a.delta >= 0.0) ? t + 1 : depth; E_sub = E_prev; }
                break;
            }
            unsigned in = 0u, better = 0u;
#pragma unroll
            for (int i = 0; i < KPT; ++i) {
                better |= (bin[i] < cut.x ? 1u : 0u) << i;
                in |= (bin[i] == cut.x ? 1u : 0u) << i;
            }
            in &= keep;
            keep &= better;
            const int need = Fn - cut.y;
            if (cut.z == need) keep |= in;
            else if (cut.z > need) keep |= resolve_bin<KPT, NT, NB>(ks, in, cut.z, need, s, tid, lane, wave);
            rank_kept<KPT, NT, NB>(keep, idx, s, lane, wave);
        } else {
#pragma unroll
            for (int i = 0; i < KPT; ++i) idx[i] = i * NT + tid;
        }
        pool = rs + F - 1 + Fn;
#pragma unroll
        for (int i = 0; i < KPT; ++i) {
            if ((keep >> i) & 1u) {
                const int p = rs + F - 1 + idx[i];
                pkey[p] = raw[i];
                pmeta[p] = (unsigned)(rs * k + i * NT + tid) | (unsigned)(t + 1) << 20;
                ppar[p] = t == 0 ? (unsigned short)0xffff : (unsigned short)(rs - 1 + cj[i]);
                atomicAdd(&s.phist[bin[i]], 1);
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
            if (wave == 0) {
                const HistCut c = hist_scan<NB, false>(s.phist, n, lane);
                if (lane == 0) s.pcut = int4{c.B, c.above, c.inb, c.first};
            }
            lds_barrier();
            double pk[kPoolPerThread];
#pragma unroll
            for (int i = 0; i < kPoolPerThread; ++i) pk[i] = i * NT + tid < pool ? fmax(pkey[i * NT + tid], kFloor) : 0.0;
            pkeep = pool_best<NT, NB>(pk, pool, n, s.pcut, s, tid, lane, wave);
            double e = 0.0;
#pragma unroll
            for (int i = 0; i < kPoolPerThread; ++i) {
                if (i * NT >= pool) break;
                if ((pkeep >> i) & 1u) e += NT > 512 ? exp(pk[i]) : exp_of_logp(pk[i]);
            }
            e = wave_sum_d(e);
            if (lane == 0) s.red[wave] = e;
            lds_barrier();
            E_sub = 0.0;
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
    const int n_out = min(pool, n);
    double pk[kPoolPerThread];
    int tok[kPoolPerThread];
    const int32_t* const ti = a.topi + rbase * k;
#pragma unroll
    for (int i = 0; i < kPoolPerThread; ++i) {                // token ids: in flight during the selection
        pk[i] = 0.0; tok[i] = 0;
        if (i * NT + tid < pool) {
            tok[i] = ti[pmeta[i * NT + tid] & 0xfffffu];
            pk[i] = fmax(pkey[i * NT + tid], kFloor);
        }
    }
    unsigned keep = 0u;
    if (ADAPT && !have_pcut) {
        keep = pkeep;                                         // the set behind the last E_sub
    } else {
        if (!have_pcut) {
            if (wave == 0) {
                const HistCut c = hist_scan<NB, false>(s.phist, n, lane);
                if (lane == 0) s.pcut = int4{c.B, c.above, c.inb, c.first};
            }
            if (tid == 0) s.lcnt = 0;
            lds_barrier();
        }
        keep = pool_best<NT, NB>(pk, pool, n, s.pcut, s, tid, lane, wave);
    }
    int idx[kPoolPerThread];
    rank_kept<kPoolPerThread, NT, NB>(keep, idx, s, lane, wave);
#pragma unroll
    for (int i = 0; i < kPoolPerThread; ++i) {
        if (i * NT >= pool) break;
        if ((keep >> i) & 1u) {
            const int p = i * NT + tid;
            oidx[p] = (unsigned short)idx[i];
            s.rec_key[idx[i]] = pkey[p];
            s.rec_tok[idx[i]] = tok[i];
            s.rec_pool[idx[i]] = (unsigned short)p;
        }
    }
    lds_barrier();
    if (wave * 64 < n) {                                      // node i = thread i (n <= 256 <= NT)
        const int W = OT_MASK_WORDS(n), i = tid;
        double p_hat = 0.0;
        if (i < n) {
            const bool node = i < n_out;
            u64 row[4] = {0ull, 0ull, 0ull, 0ull};
            int par = -1, dep = 0, token = -1;
            double key = -INFINITY;
            if (node) {
                const int p = s.rec_pool[i];
                key = s.rec_key[i];
                token = s.rec_tok[i];
                dep = (int)(pmeta[p] >> 20);
                p_hat += NT > 512 ? exp(key) : exp_of_logp(key);
                // ancestors (Algorithm 2): the parents' output indices up to the root
                int anc = ppar[p];
                if (anc != 0xffff) par = (int)oidx[anc];
                int o = i;
                for (int guard = 0; guard < OT_MAX_DEPTH; ++guard) {
#pragma unroll
                    for (int w = 0; w < 4; ++w) row[w] |= (w == (o >> 6)) ? (1ull << (o & 63)) : 0ull;
                    if (anc == 0xffff) break;
                    o = (int)oidx[anc];
                    anc = ppar[anc];
                }
            }
            const size_t ob = (size_t)b * n + i;
            a.out.token[ob] = token;
            a.out.parent[ob] = par;
            a.out.depth[ob] = dep;
            a.out.score[ob] = (float)key;
#pragma unroll
            for (int w = 0; w < 4; ++w)
                if (w < W) a.out.mask[ob * W + w] = row[w];
        }
        p_hat = wave_sum_d(p_hat);                            // E = sum of p^ (Eq. 3)
        if (lane == 0) s.red[wave] = p_hat;
    }
    if (n > 64) lds_barrier();
    if (tid == 0) {
        double e = s.red[0];
        for (int w = 1; w * 64 < n; ++w) e += s.red[w];
        a.out.expect[b] = e;
        a.out.n_out[b] = n_out;
        if (a.seq_active) a.seq_active[b] = 0;
        if (ADAPT) { a.steps_used[b] = steps; a.e_sub[b] = E_sub; }
    }
}

// LDS a workgroup may use in all (of the 160 KB of a compute unit)
constexpr size_t kLdsLimit = 160 * 1024;
size_t pool_bytes(int pool) { return ((size_t)pool * (8 + 4 + 2 + 2) + 15) / 16 * 16; }

template <int NT, int KPT, int NB, bool STAGE, bool ADAPT>
int launch_t(const TreeBuildArgs& a, const SelectGeometry& g, const BuildWorkspace& ws, int t0, int t1, size_t lds, hipStream_t s) {
    if (lds > 64 * 1024 - sizeof(Shared<NT, NB>))
        OT_HIP_CHECK(hipFuncSetAttribute((const void*)tree_build_kernel<NT, KPT, NB, STAGE, ADAPT>,
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL((tree_build_kernel<NT, KPT, NB, STAGE, ADAPT>), dim3(g.batch), dim3(NT), lds, s, ws.row_topv, ws.row_lse, g.k,
                       g.rows_per_seq, g.n, g.depth, t0, t1, a);
    OT_HIP_CHECK(hipGetLastError());
    return OT_OK;
}

template <int NT, int KPT, int NB>
int launch_n(TreeBuildArgs& a, const SelectGeometry& g, const BuildWorkspace& ws, int t0, int t1, bool adapt, hipStream_t s) {
    const int rows = g.row_start[t1] - g.row_start[t0];
    const size_t base = pool_bytes(a.batch_pool) + 16;
    const size_t tv = ((size_t)rows * g.k * 4 + 15) / 16 * 16, stage = tv + (size_t)rows * 8;
    a.stage_off_lse = (int)tv;
    if (base + sizeof(Shared<NT, NB>) > kLdsLimit) return OT_ERR_UNSUPPORTED;
    // a single step has nothing to overlap with: its candidates go straight to registers
    if (t1 - t0 > 1 && base + stage + sizeof(Shared<NT, NB>) <= kLdsLimit) {
        return adapt ? launch_t<NT, KPT, NB, true, true>(a, g, ws, t0, t1, base + stage, s)
                     : launch_t<NT, KPT, NB, true, false>(a, g, ws, t0, t1, base + stage, s);
    }
    return adapt ? launch_t<NT, KPT, NB, false, true>(a, g, ws, t0, t1, base, s)
                 : launch_t<NT, KPT, NB, false, false>(a, g, ws, t0, t1, base, s);
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
    if (g.n <= 256 && wide <= 256 && need <= 256) return launch_n<256, 1, 512>(a, g, ws, t0, t1, adapt, s);
    if (wide <= 512 && need <= 512) return launch_n<512, 1, 512>(a, g, ws, t0, t1, adapt, s);
    if (wide <= 1024 && need <= 512) return launch_n<512, 2, 512>(a, g, ws, t0, t1, adapt, s);
    if (wide <= 2048) return launch_n<1024, 2, 1024>(a, g, ws, t0, t1, adapt, s);
    return launch_n<1024, 4, 1024>(a, g, ws, t0, t1, adapt, s);
}

}  // namespace ot
