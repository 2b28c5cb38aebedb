// One-shot tree construction (ot_build_tree, ot_build_tree_adaptive): everything of Algorithm 1 that follows the row scan, for rows
// that are all in memory or that workgroups of the same launch scan meanwhile.
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
// 9.9 us, 13B-shaped 9.3; in one launch with the scan see build_fused.hip.  A step takes 2500 cycles with its rows in LDS: loads, scores
// and counting 720, cut 440, slots 540, writing 350, the rest barriers and, where the cut falls inside a bin, ranking (600).
#pragma once

#include "common.hpp"
#include "arrivals.hpp"

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

// LDS a workgroup may use in all (of the 160 KB of a compute unit)
constexpr size_t kLdsLimit = 160 * 1024;
// LDS that draft_tree needs at `smem` for a pool
inline size_t pool_bytes(int pool) { return ((size_t)pool * (8 + 4 + 2 + 1) + 15) / 16 * 16; }

// Barrier that orders LDS traffic only: loads from global memory stay in flight across it.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

__device__ __forceinline__ int grid_bin(double ks) {
    constexpr int MB = 23 - 9, OFF = (127 - 2) << 9;                           // [2^-2, 2^6): 8 octaves of 8 coarse bins
    const int q = (__float_as_int((float)-ks) >> MB) - OFF;                    // ks > 0 by rounding: negative -> bin 0
    return min(max(q, 0), kBins - 1);
}

// A coarse bin is counted in eight words, by the lane's last three bits: most keys of a wavefront share one or two coarse bins,
// and lanes that add to the same word wait for each other.
constexpr int kCopies = 8;
struct Hist { int coarse[kCoarse * kCopies], fine[kBins]; };
__device__ __forceinline__ int* coarse_of(Hist& h, int bin) { return &h.coarse[(bin >> 6) * kCopies + (threadIdx.x & (kCopies - 1))]; }
__device__ __forceinline__ void hist_add(Hist& h, int bin) {
    atomicAdd(coarse_of(h, bin), 1);
    atomicAdd(&h.fine[bin], 1);
}
// by the lane that has added to it
__device__ __forceinline__ void hist_clear(Hist& h, int bin) { *coarse_of(h, bin) = 0; h.fine[bin] = 0; }
__device__ __forceinline__ int coarse_count(const Hist& h, int lane) {
    typedef int i32x4 __attribute__((ext_vector_type(4)));
    const i32x4 x = *(const i32x4*)&h.coarse[lane * kCopies], y = *(const i32x4*)&h.coarse[lane * kCopies + 4];
    return ((x[0] + x[1]) + (x[2] + x[3])) + ((y[0] + y[1]) + (y[2] + y[3]));
}

// Bin of the `want`-th best key: B, keys in better bins, keys in bin B.  Fewer than `want` keys in all: B = kBins,
// above = all keys, inb = 0.  first: best occupied coarse bin.  Every wavefront for itself.
struct HistCut { int B, above, inb, first; };
__device__ __forceinline__ HistCut hist_cut(const Hist& h, int want, int lane) {
    const int c = coarse_count(h, lane);
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
struct alignas(16) Shared {
    static constexpr int NW = NT / 64;
    Hist cand;                         // candidates of a step; all zero between steps
    Hist pool;                         // pool nodes
    struct { double key; int idx, pad; } list[kList + 4];
    int lcnt;
    Quit quit;                         // kArrive
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
// among the `need` best; equal keys: smaller index first, index = i nt + tid, i < iters.  key(i): this thread's key i.
// lcnt and the histogram s.cand are zero on entry.  Called by the whole workgroup.
template <int NT, int UNROLL, typename KEY>
__device__ __forceinline__ unsigned resolve_bin(KEY key, int iters, unsigned in, int m, int need, Shared<NT>& s, int nt, int tid,
                                                int lane, int wave) {
    const int nw = nt >> 6;
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
                if (lane == 0) s.wc[i * nw + wave] = __popcll(bal);
            }
            lds_barrier();
            int before = 0;
#pragma unroll UNROLL
            for (int i = 0; i < iters; ++i) {
                const u64 bal = __ballot((in >> i) & 1u);
#pragma unroll 1
                for (int w = 0; w < nw; ++w) {
                    const int c = s.wc[i * nw + w];
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
                hist_clear(s.cand, bin);
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
            s.list[q].key = key(i); s.list[q].idx = i * nt + tid;
        }
    lds_barrier();
#pragma unroll UNROLL
    for (int i = 0; i < iters; ++i)
        if ((in >> i) & 1u) {
            const double mine = key(i);
            const int id = i * nt + tid;
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

// The n best pool nodes: flags of this thread's pool nodes (node i nt + tid, bit i).
template <int NT>
__device__ __forceinline__ unsigned pool_best(const double* pkey, int pool, int n, Shared<NT>& s, int nt, int tid, int lane, int wave) {
    const HistCut cut = hist_cut(s.pool, n, lane);
    unsigned keep = 0u, in = 0u;
    int iters = 0;
    while (iters * nt < pool) ++iters;
    auto key = [&](int i) { return fmax(pkey[i * nt + tid], kFloor); };
#pragma unroll 1
    for (int i = 0; i < iters; ++i)
        if (i * nt + tid < pool) {
            const int bin = grid_bin(key(i));
            keep |= (bin < cut.B ? 1u : 0u) << i;
            in |= (bin == cut.B ? 1u : 0u) << i;
        }
    const int need = n - cut.above;
    if (cut.inb == need) keep |= in;
    else if (cut.inb > need) keep |= resolve_bin<NT, 1>(key, iters, in, cut.inb, need, s, nt, tid, lane, wave);
    return keep;
}

// Where a step's rows come from.
//   kStep     memory, one step ahead
//   kStaged   memory, all of the launch's copied to LDS first (all trips to memory overlap, once)
//   kArrive   workgroups of the same launch, which publish them one by one (build_fused.hip)
enum Source { kStep, kStaged, kArrive };

// A wavefront of the GPU (arrivals.hpp)
struct ChipWave {
    static constexpr int kLanes = 64;
    int lane;
    bool first;                        // of its workgroup
    __device__ __forceinline__ u64 load(const u64* p) const { return ot::get<true>(p); }
    __device__ __forceinline__ void store(u64* p, u64 v) const { ot::put<true>(p, v); }
    __device__ __forceinline__ bool swap_if(u64* p, u64& v, u64 x) const {
        return __hip_atomic_compare_exchange_strong(p, &v, x, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ void stores_done() const { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
    __device__ __forceinline__ bool all(bool ok) const { return __all(ok); }
    __device__ __forceinline__ void pause() const { __builtin_amdgcn_s_sleep(1); }
    __device__ __forceinline__ void set(short& flag, int v) const { flag = (short)v; }
    __device__ __forceinline__ int get(const short& flag) const { return flag; }
    __device__ __forceinline__ void barrier() const { lds_barrier(); }
};

// KPT candidates per thread.  ADAPT: Algorithm 1 with its stopping rule -- after every step E_sub(T, n) = sum of p^ over the n
// best pool nodes, and drafting stops when E_sub - E <= delta.
// Steps t0 .. t1-1 of sequence b are drafted (kArrive: all steps); a sequence that is not finished then leaves its pool in
// memory for the next launch.  Called by nt <= NT threads; the histograms of s and what follows it at `smem` are scratch.
template <int NT, int KPT, Source SRC, bool ADAPT>
__device__ __forceinline__ void draft_tree(Shared<NT>& s, char* const smem, const int nt, const int b, const float* topv, const double* row_lse,
                                           const int k, const int rows, const int n, const int depth, const int t0, const int t1,
                                           const TreeBuildArgs& a, Arrivals ar) {
    const int nw = nt >> 6;
    constexpr bool STAGE = SRC == kStaged, ARRIVE = SRC == kArrive;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

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
        for (int base = 0; base < nv; base += VB * nt) {      // a batch of loads per trip to memory
            float x[VB];
            double y[LB];
            const int lb = (base / (VB * nt)) * (LB * nt);
#pragma unroll
            for (int u = 0; u < VB; ++u) x[u] = gv[min(base + u * nt + tid, nv - 1)];
#pragma unroll
            for (int u = 0; u < LB; ++u) y[u] = gl[min(lb + u * nt + tid, rows_here - 1)];
            if (base == 0) {
                for (int i = tid; i < (int)(sizeof(Hist) * 2 / 16); i += nt) ((int4*)&s.cand)[i] = int4{0, 0, 0, 0};
            }
#pragma unroll
            for (int u = 0; u < VB; ++u) { const int i = base + u * nt + tid; if (i < nv) sv[i] = x[u]; }
#pragma unroll
            for (int u = 0; u < LB; ++u) { const int i = lb + u * nt + tid; if (i < rows_here) sl[i] = y[u]; }
        }
        for (int i = (nv + VB * nt - 1) / (VB * nt) * (LB * nt) + tid; i < rows_here; i += nt) sl[i] = gl[i];
#pragma unroll
        for (int i = 0; i < KPT; ++i) cj[i] = (i * nt + tid) / k;
    } else {
        for (int i = tid; i < (int)(sizeof(Hist) * 2 / 16); i += nt) ((int4*)&s.cand)[i] = int4{0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < KPT; ++i) cj[i] = (i * nt + tid) / k;
    }
    // kArrive: rows of the next step that this wavefront's candidates need; are they there (the same for the wavefront)
    const ChipWave chip{lane, wave == 0};
    bool next_there = false;
    u64 word[KPT], word2[KPT];                                // words of the next step's rows, of those of the step after
    auto request = [&](u64 (&w)[KPT], int first, int count) {
#pragma unroll
        for (int i = 0; i < KPT; ++i) w[i] = get<true>(ar.there + first + min(cj[i], count - 1));
    };
    auto here = [&](const u64 (&w)[KPT]) {
        bool ok = true;
#pragma unroll
        for (int i = 0; i < KPT; ++i) ok = ok && w[i] == kRowThere;
        return (bool)__all(ok);
    };
    // Rows of a step, whose words are requested: wait for them; too many polls: quit
    auto poll = [&](int step, int first, int count) {
        int polls = 0;
        while (!here(word)) {
            if (++polls > ar.spin) { quit_waiting(chip, s.quit, step); return; }
            __builtin_amdgcn_s_sleep(1);
            request(word, first, count);
        }
    };
    if (ARRIVE) {
        if (tid == 0) quit_none(chip, s.quit);
        lds_barrier();
        if (ar.wait) {
            request(word, 0, 1);
            if (t1 > 1) request(word2, 1, min(n, k));
            poll(0, 0, 1);
            next_there = t1 > 1 && here(word2);
        }
        lds_barrier();
        if (__builtin_expect(has_quit(chip, s.quit, 0), 0) && !go_alone(chip, s.quit, ar)) return;
    }
    if (!STAGE) {
#pragma unroll
        for (int i = 0; i < KPT; ++i) {
            v[i] = get<ARRIVE>(gv + min(i * nt + tid, k * F - 1));
            l[i] = get<ARRIVE>(gl + min(cj[i], F - 1));
        }
    }
    // kArrive: nothing is under way at a step's top, where the compiler, which cannot count the loads of several branches, would
    // otherwise wait for the next step's as well (1000 cycles a step)
    auto arrived = [&]() { if (ARRIVE) __builtin_amdgcn_s_waitcnt(0x0f70); };      // vmcnt(0)
    if (!ARRIVE) __syncthreads();
    arrived();
    int pool = t0 > 0 ? rs - 1 + F : 0;                       // nodes drafted so far
    if (t0 > 0) {
        for (int i = tid; i < pool; i += nt) {
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
    int seen = 0;                                             // rows of the steps so far
    for (int t = t0; t < t1; ++t) {
        const int Fn = min(n, k * F), C = k * F;
        float vn[KPT];
        double ln[KPT];
        auto fetch = [&]() {                                  // the next step's rows: their place does not depend on the tree
            const float* nv = gv + (size_t)(rs + F - rs0) * k;
            const double* nl = gl + (rs + F - rs0);
#pragma unroll
            for (int i = 0; i < KPT; ++i) {
                vn[i] = get<ARRIVE>(nv + min(i * nt + tid, k * Fn - 1));
                ln[i] = get<ARRIVE>(nl + min(cj[i], Fn - 1));
            }
        };
        const bool fetched = !ARRIVE || !ar.wait || next_there;    // kArrive: at the end of the step otherwise
        if (!STAGE && t + 1 < t1) {
            if (fetched) fetch();
            else request(word, rs + F, Fn);
            if (ARRIVE && ar.wait && t + 2 < t1) request(word2, rs + F + Fn, min(n, k * Fn));
        }
        seen = rs + F;
        double raw[KPT];
        int bin[KPT], idx[KPT];
        unsigned keep = 0u;
#pragma unroll
        for (int i = 0; i < KPT; ++i) {
            const int c = i * nt + tid;
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
            // the coarse bin of the n-th best pool node, while the candidates are counted
            const int pc = coarse_count(s.pool, lane);
            const int pi = wave_incl_scan(pc, lane);
            const u64 ph = __ballot(pi >= n);
            const int PC = ph ? __ffsll((long long)ph) - 1 : kCoarse;
            lds_barrier();
            const HistCut cut = hist_cut(s.cand, Fn, lane);
            // complete when n pool nodes are better than every candidate; a look at the coarse bins settles most steps
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
                    if ((keep >> i) & 1u) hist_clear(s.cand, bin[i]);
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
                    if ((act >> i) & 1u) hist_clear(s.cand, bin[i]);
            };
            if (cut.inb > need) {
                if (crowded) { lds_barrier(); clear(); }      // the histogram is used again
                auto key = [&](int i) {
                    return fmax(raw[i], kFloor);
                };
                keep |= resolve_bin<NT, KPT>(key, KPT, in, cut.inb, need, s, nt, tid, lane, wave);
            }
            // slot of a kept candidate = its rank among the kept ones in index order
            u64 bal[KPT];
#pragma unroll
            for (int i = 0; i < KPT; ++i) {
                bal[i] = __ballot((keep >> i) & 1u);
                if (lane == 0) s.wc[i * nw + wave] = __popcll(bal[i]);
            }
            lds_barrier();
            if (!crowded) clear();                            // everybody has read the histogram
            const int c0 = lane < KPT * nw ? s.wc[lane] : 0;
            const int e0 = wave_incl_scan(c0, lane) - c0;
#pragma unroll
            for (int i = 0; i < KPT; ++i) idx[i] = rl(e0, i * nw + wave) + __popcll(bal[i] & ((1ull << lane) - 1ull));
        }
        pool = rs + F - 1 + Fn;
#pragma unroll
        for (int i = 0; i < KPT; ++i) {
            if ((keep >> i) & 1u) {
                const int p = rs + F - 1 + idx[i];
                pkey[p] = raw[i];
                pmeta[p] = (unsigned)(rs * k + i * nt + tid) | (unsigned)(t + 1) << 20;
                ppar[p] = t == 0 ? (unsigned short)0xffff : (unsigned short)(rs - 1 + cj[i]);
                hist_add(s.pool, bin[i]);
            }
        }
        if (ADAPT && tid == 0) s.lcnt = 0;
        if (ARRIVE && t + 1 < t1) {
            if (!fetched) {
                poll(t + 1, rs + F, Fn);
                fetch();
            }
            next_there = ar.wait && t + 2 < t1 && here(word2);
        }
        lds_barrier();
        if (ARRIVE && __builtin_expect(has_quit(chip, s.quit, t + 1), 0)) {
            if (!go_alone(chip, s.quit, ar)) return;
            if (t + 1 < t1) fetch();
        }
        arrived();
        rs += F; F = Fn;
        if (!STAGE) {
#pragma unroll
            for (int i = 0; i < KPT; ++i) { v[i] = vn[i]; l[i] = ln[i]; }
        }
        if (ADAPT) {
            pkeep = pool_best<NT>(pkey, pool, n, s, nt, tid, lane, wave);
            double e = 0.0;                                   // fp64 exp, as in the streaming form: both stop at the same step
#pragma unroll 1
            for (int i = 0; i * nt < pool; ++i)
                if ((pkeep >> i) & 1u) e += exp(pkey[i * nt + tid]);
            e = wave_sum_d(e);
            if (lane == 0) s.red[wave] = e;
            lds_barrier();
            E_sub = 0.0;
            for (int w = 0; w < nw; ++w) E_sub += s.red[w];
            if (t + 1 < depth) {                              // the loop condition of Algorithm 1
                if (!(E_sub - E_prev > a.delta)) { done = true; steps = t + 1; break; }
                E_prev = E_sub;
            }
        }
    }
    if (!done) {                                              // more steps in a later launch
        for (int i = tid; i < pool; i += nt) {
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
    const int32_t* const ti = a.topi + rbase * k;
    // token id of the first node of this thread (all of them, mostly): in flight during the selection
    const int tok0 = get<ARRIVE>(ti + (pmeta[min(tid, pool - 1)] & 0xfffffu));
    unsigned keep = pkeep;                                    // ADAPT: the set behind the last E_sub
    if (!ADAPT || complete) {
        if (!complete) {
            if (tid == 0) s.lcnt = 0;
            lds_barrier();
        }
        keep = pool_best<NT>(pkey, pool, n, s, nt, tid, lane, wave);
    }
    // output index = rank in (depth, slot) order among the selected nodes
#pragma unroll 1
    for (int i = 0; i * nt < pool; ++i) {
        const u64 bal = __ballot((keep >> i) & 1u);
        if (lane == 0) s.wc[i * nw + wave] = __popcll(bal);
    }
    lds_barrier();
    int carry = 0;
#pragma unroll 1
    for (int i = 0; i * nt < pool; ++i) {
        const int c = lane < nw ? s.wc[i * nw + lane] : 0;
        const int inc = wave_incl_scan(c, lane);
        const u64 bal = __ballot((keep >> i) & 1u);
        const int base = carry + rl(inc - c, wave);           // (outside the branch: all lanes take part)
        if ((keep >> i) & 1u) {
            const int p = i * nt + tid, o = base + __popcll(bal & ((1ull << lane) - 1ull));
            oidx[p] = (unsigned char)o;
            s.rec_key[o] = pkey[p];
            s.rec_tok[o] = i == 0 ? tok0 : get<ARRIVE>(ti + (pmeta[p] & 0xfffffu));
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
    }
    const int W = OT_MASK_WORDS(n);
    const size_t ob = (size_t)b * n + (n > 64 ? tid : lane);
    if (W == 1) {
        // wavefront 0: parents, depths and ancestors (Algorithm 2).  Every round doubles the stretch of a root path that a mask
        // holds: the mask of the node at its end is added, and that node's end is the new one.
        if (wave == 0) {
            u64 row = node ? 1ull << lane : 0ull;
            int up = par;
            for (int stretch = 1; stretch < OT_MAX_DEPTH; stretch *= 2) {
                if (!__any(up >= 0)) break;
                const int at = max(up, 0);
                const u64 above = (u64)(unsigned)__shfl((int)(row >> 32), at) << 32 | (unsigned)__shfl((int)row, at);
                const int next = __shfl(up, at);
                if (up >= 0) { row |= above; up = next; }
            }
            if (tid < n) {
                a.out.parent[ob] = par;
                a.out.depth[ob] = node ? (int)(pmeta[p] >> 20) : 0;
                a.out.mask[ob] = row;
            }
            return;
        }
        if (wave > 1) {
            if (ARRIVE && wave == 2) clear_arrivals(chip, ar, seen);
            return;
        }
    }
    const int i = n > 64 ? tid : lane;                        // wavefront 1 (all of them): the rest
    const bool have = i < n_out;
    const double key = have ? s.rec_key[i] : -INFINITY;
    if (i < n) {
        a.out.token[ob] = have ? s.rec_tok[i] : -1;
        a.out.score[ob] = (float)key;
    }
    if (W > 1) {
        if (node) s.rec_par[tid] = (unsigned short)par;
        lds_barrier();
        // ancestors (Algorithm 2): the parents' output indices up to the root
        int o = node ? tid : -1;
        u64 row[4] = {0ull, 0ull, 0ull, 0ull};
        for (int guard = 0; guard < OT_MAX_DEPTH && o >= 0; ++guard) {
            const u64 bit = 1ull << (o & 63);
#pragma unroll
            for (int w = 0; w < 4; ++w) row[w] |= (w == (o >> 6)) ? bit : 0ull;
            o = guard == 0 ? par : (int)(short)s.rec_par[o];
        }
        if (tid < n) {
            a.out.parent[ob] = par;
            a.out.depth[ob] = node ? (int)(pmeta[p] >> 20) : 0;
#pragma unroll
            for (int w = 0; w < 4; ++w)
                if (w < W) a.out.mask[ob * W + w] = row[w];
        }
    }
    // E = sum of p^ (Eq. 3)
    double e = wave_sum_d(have ? exp(key) : 0.0);
    if (n > 64) {
        if (lane == 0) s.red[wave] = e;
        lds_barrier();
        e = s.red[0];
        for (int w = 1; w * 64 < n; ++w) e += s.red[w];
    }
    if (i == 0) {
        a.out.expect[b] = e;
        a.out.n_out[b] = n_out;
        if (a.seq_active) a.seq_active[b] = 0;
        if (ADAPT) { a.steps_used[b] = steps; a.e_sub[b] = E_sub; }
    }
    if (ARRIVE && n > 64 && wave == nw - 1) clear_arrivals(chip, ar, seen);
}

}  // namespace
}  // namespace ot
