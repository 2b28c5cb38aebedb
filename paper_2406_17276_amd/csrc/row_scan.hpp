// Row scan: for every logits row of the draft model, one pass over the row yields
//   lse  = log sum_v exp(x_v)            (normaliser of p_d = softmax(row), Sec. 2 "Inference")
//   top-k tokens by logit, equal logits -> smaller token id   (children of a node, Sec. 3 after Eq. 2)
// This is the HBM-bound part of tree construction: every element is read once, 16 bytes per lane per load, from
// addresses aligned to 16 bytes whatever the row's own alignment is (the elements of the first and the last vector that
// do not belong to the row count as -inf).
//
// One workgroup handles one row, or one part of a row longer than the workgroup's capacity.
//   1. every wavefront, on its own, vector by vector: the vector's maximum, and sum of exp(x - ref) over its elements.
//      ref is the wavefront's maximum so far; when it moves up, the sum so far is scaled once, so exponentials need no
//      second pass over the row, and the terms that matter have exponents near 0, which fp32 rounds least.
//   2. barrier; tau = a lower bound of the k-th largest element: the k-th largest (or a little less) of the maxima of 64
//      groups of lanes -- each group holds an element >= its maximum, so at least k elements are >= tau,
//   3. elements >= tau (about k + 3) of the vectors whose own maximum reaches tau become candidates,
//   4. the k best candidates are ranked by counting (value desc, token asc); the wave partials are combined in fp64:
//      M = max ref_w, s = sum s_w exp(ref_w - M), lse = M + log s,
//   5. part results are written; rows split over several parts are merged by merge_parts_kernel.
// If the candidate list overflows (massive ties), a slow exact path extracts the k best by k rounds of a workgroup-wide
// arg-max over the part, re-read from memory.
//
// Two forms of step 1.  KEEP: few rows (the launch does not fill the chip): many threads per row, all loads in flight at
// once, the vectors stay in registers and step 3 takes the candidates from there.  Rolling: many rows: 16 vectors per
// lane pass through a ring of six in flight, which leaves a fourth of the fixed work per element, and the dozen vectors
// that hold candidates are read again.  Short rows in great numbers take one wavefront each.
#pragma once

#include "common.hpp"

namespace ot {
namespace {

typedef unsigned long long u64;

constexpr int kVecCap = 512;           // rolling form: pairs of vectors that hold candidates
constexpr float kLog2e = 1.4426950408889634f;
constexpr int kRollVpl = 16;

struct ScanKArgs {
    int k, parts;
    int rows_per_seq;                 // stride of the per-row results
    // parts == 1: final row results; parts > 1: per-part results
    double* row_lse; float* row_topv; int32_t* row_topi;
    float* part_m; double* part_s; float* part_topv; int32_t* part_topi;
    const int32_t* seq_active;        // SKIP kernels: rows of sequence b are left unread when seq_active[b] == 0
};

// The order of candidates as one integer: value desc, token asc (-0 counts as +0: equal logits)
__device__ __forceinline__ u64 cand_key(float v, int e) {
    const unsigned bits = __float_as_uint(v), u = bits == 0x80000000u ? 0u : bits;
    const unsigned f = (u >> 31) ? ~u : (u | 0x80000000u);
    return ((u64)f << 32) | (u64)(0xffffffffu - (unsigned)e);
}
__device__ __forceinline__ float cand_val(u64 key) {
    const unsigned f = (unsigned)(key >> 32);
    return __uint_as_float((f >> 31) ? (f & 0x7fffffffu) : ~f);
}
__device__ __forceinline__ int cand_tok(u64 key) { return (int)(0xffffffffu - (unsigned)key); }
// order-preserving map from float to int
__device__ __forceinline__ int ordered(float v) {
    const int i = __float_as_int(v);
    return i ^ ((i >> 31) & 0x7fffffff);
}

// order-preserving map from int to float, the inverse
__device__ __forceinline__ float unordered(int o) { return __int_as_float(o ^ ((o >> 31) & 0x7fffffff)); }

// max over groups of G consecutive lanes (1, 4, 8 or 16), result in every lane of the group
template <int G>
__device__ __forceinline__ int group_max(int v) {
    if (G >= 4) {
        v = max(v, dpp_i<DPP_QUAD_XOR1>(v, v));
        v = max(v, dpp_i<DPP_QUAD_XOR2>(v, v));
    }
    if (G >= 8) v = max(v, dpp_i<DPP_ROW_HALF_MIRROR>(v, v));
    if (G >= 16) v = max(v, dpp_i<DPP_ROW_MIRROR>(v, v));
    return v;
}
// max over each row of 16 lanes, result in every lane of the row, and over the wavefront, as a scalar.  Written out because of the
// quieting instructions (max2), which would also keep the lane exchange out of the maximum.  A lane exchange may read what the
// instruction before the last one or earlier wrote.  (row_scan.hip alone used to be compiled without NaNs instead; in the kernels
// that share the scan with a selection, which counts on NaNs, the quieting took 190 of 4900 instructions of the rolling form:
// streaming loops replayed from a graph, 11 steps of 5 nodes of 70016 bf16 246.6 -> 241.9 us, 10 of 24 of 40000 192.8 -> 189.4, 1 %
// over 49; row_scan.hip as before, 32 sequences of 128256 2130 -> 2123)
#define OT_MAX_DPP(CTRL) "s_nop 1\n\tv_max_f32_dpp %0, %0, %0 " CTRL "\n\t"
#define OT_MAX_ROW16 OT_MAX_DPP("quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf") OT_MAX_DPP("quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf") \
                     OT_MAX_DPP("row_half_mirror row_mask:0xf bank_mask:0xf") OT_MAX_DPP("row_mirror row_mask:0xf bank_mask:0xf")
__device__ __forceinline__ float row_max(float v) {
    asm volatile(OT_MAX_ROW16 : "+v"(v));
    return v;
}
__device__ __forceinline__ float wavefront_max(float v) {
    asm volatile(OT_MAX_ROW16 OT_MAX_DPP("row_bcast:15 row_mask:0xa bank_mask:0xf") OT_MAX_DPP("row_bcast:31 row_mask:0xc bank_mask:0xf") : "+v"(v));
    return rl_f(v, 63);
}
#undef OT_MAX_ROW16
#undef OT_MAX_DPP

// 2^x in fp64 for the factor between two references, to 1e-8 (Taylor series of e^t on |t| <= ln 2 / 2, seven terms): the
// exponential instruction's 2^-24 would be an error of everything summed so far
__device__ __forceinline__ double exp2_factor(double x) {
    const double n = rint(x), t = (x - n) * 0.6931471805599453;
    double p = 1.0 / 5040;
    p = fma(p, t, 1.0 / 720);
    p = fma(p, t, 1.0 / 120);
    p = fma(p, t, 1.0 / 24);
    p = fma(p, t, 1.0 / 6);
    p = fma(p, t, 0.5);
    p = fma(p, t, 1.0);
    p = fma(p, t, 1.0);
    return ldexp(p, (int)n);
}

template <int NT, bool KEEP>
struct ScanShared {
    static constexpr int NW = NT / 64;
    // groups for the threshold (ranked one ballot per group and wavefront in the KEEP form: fewer for small workgroups)
    static constexpr int G = KEEP && NT < 512 ? NT / 8 : 64, GL = NT / G;
    static_assert(GL == 1 || GL == 4 || GL == 8 || GL == 16, "group_max");
    // candidates of one part (one wavefront: 5 KB of LDS, so that 29 rows share a compute unit)
    static constexpr int kCandCap = NT == 64 ? 512 : 1024;
    u64 key[kCandCap];
    unsigned short vec[KEEP ? 1 : kVecCap];
    int g[G];
    float wm[NW];                      // reference exponent and sum of every wavefront
    double ws[NW];
    int count, nvec;                   // candidates; rolling form: pairs of vectors that hold some
    int tau;
    u64 best[NW];
};

// Where a work item's elements are (the same for the whole workgroup): vector v of the item holds its elements
// v VEC - shift .. v VEC - shift + VEC - 1, base is aligned to 16 bytes.
struct Item {
    const char* base;
    int shift, len, nvec;
    int e_begin;                      // token id of the item's first element
    int rid, part;                    // row of the results, part of it
};
// Part `part` of row r of sequence b.
//   part_geom  parts | part_elems << 4
//   grow       nsteps | k << 8 | n << 16: step t covers F_t rows, F_0 = 1, F_{t+1} = min(n, k F_t)
template <int DT>
__device__ __forceinline__ Item locate(const void* logits, const long long stride_seq, const long long stride_depth,
                                       const long long stride_row, const int vocab, const int part_geom, const int grow,
                                       const int rows_per_seq, const int b, const int r, const int part) {
    constexpr int VEC = VecOf<DT>::N, ESIZE = 16 / VEC;
    const int part_elems = part_geom >> 4;
    // row r of a sequence is slot j of step t (Algorithm 1: the frontier grows k-fold per step up to n)
    const int nsteps = grow & 255, grow_k = (grow >> 8) & 255, grow_n = grow >> 16;
    int t = 0, start = 0, F = 1;
    while (t + 1 < nsteps && r >= start + F) {
        start += F;
        F = min(grow_n, grow_k * F);
        ++t;
    }
    const int j = r - start;
    const long long row_off = (long long)b * stride_seq + (long long)t * stride_depth + (long long)j * stride_row;
    const int e_begin = part * part_elems;
    const int len = min(vocab, e_begin + part_elems) - e_begin;

    const char* const first = (const char*)logits + (row_off + e_begin) * ESIZE;
    Item it;
    it.shift = (int)((uintptr_t)first & 15) / ESIZE;
    it.base = first - it.shift * ESIZE;
    it.len = len;
    it.nvec = (it.shift + len + VEC - 1) / VEC;
    it.e_begin = e_begin;
    it.rid = b * rows_per_seq + r;
    it.part = part;
    return it;
}

// PUB: other workgroups of the launch read the results.
template <int DT, int NT, int VPL, bool KEEP, bool PUB = false>
struct Scan {
    static constexpr int VEC = VecOf<DT>::N, ESIZE = 16 / VEC;
    static constexpr int NW = NT / 64, G = ScanShared<NT, KEEP>::G, GL = ScanShared<NT, KEEP>::GL;
    static constexpr int R = KEEP ? VPL : 6;                  // vectors in flight per lane (64 registers in all)
    static constexpr int kCandCap = ScanShared<NT, KEEP>::kCandCap;
    ScanShared<NT, KEEP>& sh;
    const ScanKArgs& a;
    const int wave;

    __device__ __forceinline__ static u32x4 load(const Item& it, int i, int tid) {
        const unsigned v = (unsigned)min(i * NT + tid, it.nvec - 1);
        return __builtin_nontemporal_load((const u32x4*)(it.base + v * 16u));
    }
    // the elements >= tau of vector v
    __device__ __forceinline__ void take(const Item& it, const float (&x)[VEC], int v, float tau) {
#pragma unroll
        for (int c = 0; c < VEC; ++c) {
            const int e = v * VEC + c - it.shift;
            if (x[c] >= tau && (unsigned)e < (unsigned)it.len) {
                const int p = atomicAdd(&sh.count, 1);
                if (p < kCandCap) sh.key[p] = cand_key(x[c], it.e_begin + e);
            }
        }
    }
    __device__ __forceinline__ void take_again(const Item& it, int v, float tau) {
        const int v2 = v + NT;
        const u32x4 w0 = *(const u32x4*)(it.base + (unsigned)v * 16u), w1 = *(const u32x4*)(it.base + (unsigned)min(v2, it.nvec - 1) * 16u);
        float x[VEC];
        VecOf<DT>::unpack(w0, x);
        take(it, x, v, tau);
        VecOf<DT>::unpack(w1, x);
        take(it, x, v2, tau);                          // (past the end: no element in range)
    }

    // Steps 1 to 3 on an item whose first R vectors are requested; returns tau.
    __device__ __forceinline__ float stream(const Item& it, u32x4 (&w)[R]) {
        const int tid = threadIdx.x, lane = tid & 63, nvec = it.nvec;
        // ---- 1. the vectors ---------------------------------------------------
        auto mask_edges = [&](float (&x)[VEC], int v) {
#pragma unroll
            for (int c = 0; c < VEC; ++c) x[c] = (unsigned)(v * VEC + c - it.shift) < (unsigned)it.len ? x[c] : -INFINITY;
        };
        auto edge = [&](int i) { return (i == 0 && it.shift > 0) || (i + 1) * NT * VEC > it.shift + it.len; };
        // maximum of every vector; rolling form: of every pair of vectors, which are read again together (registers)
        constexpr int PER = KEEP ? 1 : 2;
        float vmax[VPL / PER];
        float xk[KEEP ? VPL : 1][VEC];                            // KEEP: all elements of this lane
        float m, mc;                                              // this lane's maximum; reference exponent (log2 units)
        double s_w;                                               // sum over the wavefront
        if constexpr (KEEP) {
            float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < VPL; ++i) {
                VecOf<DT>::unpack(w[i], xk[i]);
                if (edge(i)) {
                    asm volatile("");      // keeps this a branch: full vectors skip the selects
                    mask_edges(xk[i], i * NT + tid);
                }
                vmax[i] = max_of(xk[i]);
            }
            m = vmax[0];
#pragma unroll
            for (int i = 1; i < VPL; ++i) m = max2(m, vmax[i]);
            const float mw = wavefront_max(m);
            mc = mw * kLog2e;
            if (mw > -INFINITY) {
#pragma unroll
                for (int i = 0; i < VPL; ++i)
#pragma unroll
                    for (int c = 0; c < VEC; ++c) acc[c & 3] += __builtin_amdgcn_exp2f(fmaf(xk[i][c], kLog2e, -mc));
            }
            s_w = wave_sum_rows_d((acc[0] + acc[1]) + (acc[2] + acc[3]));
        } else {
            // a lane adds up 16 vectors: fp32 inside a vector, fp64 above
            float ref = -INFINITY;                                // the wavefront's maximum so far
            double acc = 0.0;
            mc = 0.f;
#pragma unroll
            for (int i = 0; i < VPL; ++i) {
                const u32x4 cur = w[i % R];
                if (i + R < VPL) w[i % R] = load(it, i + R, tid);
                if (i % 2 == 0) vmax[i / 2] = -INFINITY;
                if (i * NT < nvec) {
                    float x[VEC];
                    VecOf<DT>::unpack(cur, x);
                    if (edge(i)) {
                        asm volatile("");      // keeps this a branch: full vectors skip the selects
                        mask_edges(x, i * NT + tid);
                    }
                    const float v = max_of(x);
                    vmax[i / 2] = i % 2 == 0 ? v : max2(vmax[i / 2], v);
                    // e^(x - m) = 2^(x log2e - mc) with mc = fl(m log2e): one fma per element.  mc is carried along as the
                    // wave's reference exponent, so its rounding cancels when the partial sums are combined.
                    if (__any(v > ref)) {
                        ref = wavefront_max(v);
                        const float mn = max2(ref, -1e38f) * kLog2e;                     // (finite for the lowest masks too)
                        if (i > 0) acc = acc > 0.0 ? acc * exp2_factor((double)mc - (double)mn) : 0.0;
                        mc = mn;
                    }
                    float e[VEC];
#pragma unroll
                    for (int c = 0; c < VEC; ++c) e[c] = __builtin_amdgcn_exp2f(fmaf(x[c], kLog2e, -mc));
#pragma unroll
                    for (int h = VEC / 2; h >= 1; h /= 2)
#pragma unroll
                        for (int c = 0; c < h; ++c) e[c] += e[c + h];
                    acc += (double)e[0];
                }
            }
            m = vmax[0];
#pragma unroll
            for (int i = 1; i < VPL / 2; ++i) m = max2(m, vmax[i]);
            s_w = wave_sum_d(acc);
        }
        if (lane == 0) { sh.wm[wave] = s_w > 0.0 ? mc : -INFINITY; sh.ws[wave] = s_w; }
        const int gm = group_max<GL>(ordered(m));
        if ((lane & (GL - 1)) == 0) sh.g[tid / GL] = gm;
        __syncthreads();

        // ---- 2. tau -----------------------------------------------------------
        const int kk = min(a.k, G);
        const int mine = G == 64 || lane < G ? sh.g[lane] : (int)0x80000000;
        float tau;
        if (KEEP) {
            // latency counts: wavefront w ranks maxima w, w + NW, ...: one ballot per maximum, all wavefronts at once
#pragma unroll
            for (int q = 0; q < G / NW; ++q) {
                const int v = rl(mine, q * NW + wave);
                const u64 before = __ballot(mine > v || (mine == v && lane < q * NW + wave));
                if (__popcll(before) == kk - 1 && lane == 0) sh.tau = v;
            }
            __syncthreads();
            tau = unordered(sh.tau);
        } else {
            // issue slots count: every wavefront bisects for a value that k to k + 2 of the maxima reach, one vector
            // instruction per round
            int lo = ordered(-INFINITY), hi = ordered(INFINITY) + 1;      // count(>= lo) >= k > count(>= hi)
            for (int round = 0; round < 32; ++round) {
                const int mid = (int)(((long long)lo + (long long)hi) >> 1);
                if (mid == lo) break;
                const int cnt = __popcll(__ballot(mine >= mid));
                if (cnt >= kk) { lo = mid; if (cnt <= kk + 2) break; }
                else hi = mid;
            }
            tau = unordered(lo);
        }

        // ---- 3. candidates ----------------------------------------------------
        if constexpr (KEEP) {
#pragma unroll
            for (int i = 0; i < VPL; ++i)
                if (vmax[i] >= tau && i * NT + tid < nvec) take(it, xk[i], i * NT + tid, tau);
        } else if (m >= tau) {
#pragma unroll
            for (int i = 0; i < VPL; i += 2)
                if (vmax[i / 2] >= tau && i * NT + tid < nvec) {
                    const int p = atomicAdd(&sh.nvec, 1);
                    if (p < kVecCap) sh.vec[p] = (unsigned short)(i * NT + tid);
                }
        }
        __syncthreads();
        return tau;
    }

    // Step 4 of an item.  Rolling form: wavefronts 0 and 1 (or the only one) alone, unless an unusual number of vectors holds
    // candidates.
    __device__ __forceinline__ void finish(const Item& it, float tau) {
        const int tid = threadIdx.x, lane = tid & 63;
        bool slow = false;
        int nv = 0;                                               // rolling form: pairs of vectors that hold candidates
        if constexpr (!KEEP) {
            nv = sh.nvec;
            slow = nv > kVecCap;
            if (nv <= 64) {
                if (wave > 1) return;
                if (tid < nv) take_again(it, sh.vec[tid], tau);
            } else {
                for (int q = tid; q < min(nv, kVecCap); q += NT) take_again(it, sh.vec[q], tau);
                __syncthreads();
            }
        }

        const int rid = it.rid;
        // where the k winners of this part go
        float* outv; int32_t* outi;
        if (a.parts == 1) {
            outv = a.row_topv + (size_t)rid * a.k;
            outi = a.row_topi + (size_t)rid * a.k;
        } else {
            outv = a.part_topv + ((size_t)rid * a.parts + it.part) * a.k;
            outi = a.part_topi + ((size_t)rid * a.parts + it.part) * a.k;
        }
        // ---- 4a. combine the wave partials in fp64 (one wavefront, 16 lanes) ----
        if (wave == (KEEP || NW == 1 ? NW - 1 : 1) && lane < 16) {
            const bool have = lane < NW;
            const float mw = have ? sh.wm[lane] : -INFINITY;
            const float M = row_max(mw);
            double part_sum = (have && mw > -INFINITY) ? sh.ws[lane] * (double)__builtin_amdgcn_exp2f(mw - M) : 0.0;
            part_sum += dpp_d<DPP_QUAD_XOR1>(part_sum);
            part_sum += dpp_d<DPP_QUAD_XOR2>(part_sum);
            part_sum += dpp_d<DPP_ROW_HALF_MIRROR>(part_sum);
            part_sum += dpp_d<DPP_ROW_MIRROR>(part_sum);
            if (lane == 0) {
                if (a.parts == 1) {
                    // the terms are 2^(x c - M) with c = the fp32 constant, i.e. e^((x - M / c) c / log2e): dividing
                    // M by the same c puts the reference back into natural-log units without a bias in the constant
                    put<PUB>(a.row_lse + rid, (double)M / (double)kLog2e + log(part_sum));
                } else {
                    a.part_m[(size_t)rid * a.parts + it.part] = M;
                    a.part_s[(size_t)rid * a.parts + it.part] = part_sum;
                }
            }
        }

        // ---- 4b. rank the candidates -------------------------------------------
        if (!KEEP && nv <= 64) {
            if (wave != 0) return;
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");    // (the list is this wavefront's own work)
        }
        const int ncand = sh.count;
        if (!slow && ncand <= kCandCap) {
            if (KEEP && ncand <= 32 && NT >= 1024) {
                // one (candidate i, rival j) pair per thread: rank of i = rivals that precede it, counted with a ballot
                const int i = tid >> 5, q = tid & 31;
                const u64 key = sh.key[i < ncand ? i : 0], u = sh.key[q < ncand ? q : 0];
                const u64 bal = __ballot(q < ncand && u > key);
                const int rank = __popcll((lane & 32) ? (bal >> 32) : (bal & 0xffffffffull));
                if (q == 0 && i < ncand && rank < a.k) { put<PUB>(outv + rank, cand_val(key)); put<PUB>(outi + rank, cand_tok(key)); }
                return;
            }
            if (ncand <= 64) {
                if (wave == 0) {          // candidate i sits in lane i; the others are broadcast by v_readlane
                    const u64 key = lane < ncand ? sh.key[lane] : 0ull;
                    const int hi = (int)(key >> 32), lo = (int)(unsigned)key;
                    int rank = 0;
                    for (int q = 0; q < ncand; ++q) {
                        const u64 u = ((u64)(unsigned)rl(hi, q) << 32) | (u64)(unsigned)rl(lo, q);
                        rank += u > key ? 1 : 0;
                    }
                    if (lane < ncand && rank < a.k) { put<PUB>(outv + rank, cand_val(key)); put<PUB>(outi + rank, cand_tok(key)); }
                }
                return;
            }
            if (!KEEP && nv <= 64) {                          // wavefront 0 alone, up to 64 VEC candidates
                for (int i = lane; i < ncand; i += 64) {
                    const u64 key = sh.key[i];
                    int rank = 0;
                    for (int q = 0; q < ncand; ++q) rank += sh.key[q] > key ? 1 : 0;
                    if (rank < a.k) { put<PUB>(outv + rank, cand_val(key)); put<PUB>(outi + rank, cand_tok(key)); }
                }
                return;
            }
            for (int i = tid; i < ncand; i += NT) {
                const u64 key = sh.key[i];
                int rank = 0;
                for (int q = 0; q < ncand; ++q) rank += sh.key[q] > key ? 1 : 0;
                if (rank < a.k) { put<PUB>(outv + rank, cand_val(key)); put<PUB>(outi + rank, cand_tok(key)); }
            }
            return;
        }

        // ---- slow exact path: k rounds of arg-max, re-reading the part from memory ----
        u64 prev = ~0ull;
        for (int round = 0; round < a.k; ++round) {
            u64 best = 0ull;
            const char* const first = it.base + it.shift * ESIZE;
            for (int e = tid; e < it.len; e += NT) {
                float v;
                if (DT == OT_BF16) v = __uint_as_float((unsigned)((const unsigned short*)first)[e] << 16);
                else v = ((const float*)first)[e];
                const u64 key = cand_key(v, it.e_begin + e);
                if (key < prev) best = key > best ? key : best;
            }
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const u64 other = __shfl_xor(best, o);
                best = other > best ? other : best;
            }
            __syncthreads();
            if (lane == 0) sh.best[wave] = best;
            __syncthreads();
            best = sh.best[0];
            for (int q = 1; q < NW; ++q) best = sh.best[q] > best ? sh.best[q] : best;
            if (best == 0ull) break;      // fewer than k valid elements in this part
            prev = best;
            if (tid == 0) { put<PUB>(outv + round, cand_val(best)); put<PUB>(outi + round, cand_tok(best)); }
        }
    }
};

// Which form: KEEP while a workgroup's registers hold the row and the rows do not fill the chip a few times over.
// Rolling, a wavefront per row: short rows in great numbers, where what a workgroup does once per row -- a barrier and the
// threshold per wavefront -- is all that counts.  Up to half of the wavefront's 128 elements a lane it pays from 2000 to
// 4000 rows on, beyond from some 10000: KEEP / rolling, us, 2048, 4096, 16384 and 32000 rows: 1000 bf16 13.7 / 12.0,
// 20.4 / 14.2, 54.6 / 31.2, 100.6 / 52.4; 4096 bf16 13.3 / 15.4, 21.3 / 18.0, 58.1 / 41.3, 107 / 69; 2048 fp32 14.6 / 13.0,
// 21.0 / 16.2, 57.7 / 36.9, 105.8 / 62.0; 7743 bf16 15.4 / 17.2, 22.4 / 24.2, 61.4 / 56.7, 113 / 100.  (Four rows to a
// workgroup of four wavefronts, one row each or several in turn, gave 58 to 67 us instead of 52 for 32000 rows of 1000.)
// Rolling, 256 threads per row: rows of all that a workgroup's registers hold (32000 bf16, 16000 fp32) break even at
// some 1536 rows, shorter ones -- their 1024 threads have less than a register set each -- in proportion to their length,
// from some 700 rows on: KEEP / rolling 32000 bf16 1024 rows 19.5 / 21.1, 1536 24.7 / 25.4, 2048 31.0 / 31.5, 4096
// 53.5 / 52.1, 8192 96.5 / 90.0; 24000 bf16 1024 18.3 / 18.9, 2048 31.2 / 26.9, 4096 52.4 / 42.1; 16384 bf16 512
// 11.1 / 13.0, 1024 18.0 / 16.4, 4096 50.6 / 32.7; 9000 bf16 512 11.7 / 12.1, 1024 17.9 / 14.8, 4096 51.0 / 27.4; 12000
// fp32 512 11.8 / 13.0, 1024 19.6 / 16.6, 4096 54.4 / 39.2.
// Longer rows would need parts and a merge launch (4 us and more) in the KEEP form, so they roll at any number of rows:
// 128256 bf16, 256 rows 20.2 / 17.3 us, 2048 rows 97 / 83.
struct ScanForm {
    int threads; bool keep;           // per row or part
    int parts, part_elems;            // parts of a row, elements of each
};
inline ScanForm scan_form(const ScanGeometry& g, const void* logits) {
    const int vec = g.dtype == OT_BF16 ? VecOf<OT_BF16>::N : VecOf<OT_F32>::N;
    const long long rows = (long long)g.batch * g.rows;
    // elements a workgroup can take: where a row may start inside a vector, one vector less
    const bool aligned = (uintptr_t)logits % 16 == 0 && g.stride_seq % vec == 0 && g.stride_depth % vec == 0 && g.stride_row % vec == 0;
    auto capacity = [&](int NT, int VPL) { return (NT * VPL - (aligned ? 0 : 1)) * vec; };
    const int KV = 32 / vec;                                  // KEEP: 32 elements per lane
    const int wave_cap = capacity(64, kRollVpl), roll_cap = capacity(256, kRollVpl);
    if (g.vocab <= wave_cap && rows >= (g.vocab <= wave_cap / 2 ? 2560 : 12288)) return {64, false, 1, g.vocab};
    if (g.vocab <= capacity(256, KV)) return {256, true, 1, g.vocab};
    if (g.vocab <= roll_cap && rows >= (1536LL * g.vocab / roll_cap > 768 ? 1536LL * g.vocab / roll_cap : 768))
        return {256, false, 1, g.vocab};
    if (g.vocab <= capacity(1024, KV)) return {1024, true, 1, g.vocab};
    if (g.vocab <= capacity(512, kRollVpl)) return {512, false, 1, g.vocab};
    const int cap = capacity(1024, kRollVpl), parts = (g.vocab + cap - 1) / cap;
    return {1024, false, parts, ((g.vocab + parts - 1) / parts + vec - 1) / vec * vec};
}

}  // namespace
}  // namespace ot
