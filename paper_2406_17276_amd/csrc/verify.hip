// Verification of a draft tree (Preliminaries, "Speculative Decoding"; Algorithm 2, "Verify"):
//   ground truth after a position = the target model's most probable token there;
//   the longest root branch of the tree that agrees with the ground truth is accepted, and the target's token
//   after the last accepted node is produced as well (A tokens for A - 1 accepted nodes);
//   the accepted nodes' K/V rows are appended to the cache.
// Random sampling (Sec. 4, non-greedy settings): the paper changes only which tokens are acceptable and gives no
// rule; here the ground truth after a position is DRAWN from softmax(target logits / temperature) by the inverse
// CDF in token order of a caller-supplied uniform number, the walk is the same.
//
// One launch: a workgroup per target row finds the row's ground truth and publishes it; the workgroup that completes a
// sequence's set walks down the tree.  A second launch copies K/V rows.
//
// What bounds it: one sequence's rows are 3 MB, so launches and trips to memory count; for batches, reading the rows.
// The greedy form needs no exponentials and, since the threshold of the builder's scan would be the maximum itself, no
// candidate lists.  Measured (MI355X, verification and append together; before: scan with statistics + walk + append,
// segment sums + pick + walk + append): one sequence of 51 rows of 32000, greedy 14.3 -> 10.5 us; 16 x 61 rows, sampled 28.0 ->
// 20.7 us (its rows end 7 to 13.5 us after the start, 62 MB; the draw takes 3 us behind the last, word and walk 1.5).
#include <string.h>

#include <algorithm>

#include "common.hpp"

namespace ot {
namespace {

typedef unsigned long long u64;

struct VerifyKArgs {
    const void* logits;
    long long stride_seq, stride_row;
    int vocab, n;
    float c;                     // sampling: log2(e) / temperature
    const float* u;              // sampling: [batch][n + 1]
    const int32_t *token, *parent, *n_out;
    u64* truth;                  // [batch][word_stride(n)]  kPublished | token
    int32_t *accept_len, *accept_node, *accept_token;
};

// A row's result as one 64-bit word, so that the words of a sequence tell both whether all its rows are there and what
// they are.  The workspace needs no preparation: a word counts only with these upper 46 bits (the lower 18 hold any
// token), and the workgroup that walks the tree clears the words again.
constexpr int kTokenBits = 18;
constexpr u64 kPublished = 0x1fd2a470cb5dull << kTokenBits;
static_assert(kMaxVocab <= 1 << kTokenBits, "a token fits the word");
// Words of a sequence start a cache line of their own (side by side: greedy 62 us instead of 50 in the case below).
__host__ __device__ inline int word_stride(int n) { return (n + 16) & ~15; }
constexpr int kBatch = 4;        // vectors per lane requested at once; the next batch is in flight while one is processed

// One wavefront: publish the row's ground truth, and walk the tree if that completes the sequence.  Words travel through
// device-scope stores and loads (rows of a sequence are on different XCDs).  Every workgroup's word has reached memory
// before it looks at the others', so at least the last one sees them all; should two see them all, both write the same.
// The walk is a serial chain, so what a step needs is prepared for all positions at once -- which node follows a position is
// known as soon as all ground truths are -- and a step is one v_readlane.  (A ballot over all nodes per step: 24.8 us
// for two sequences of 65 rows of 300 bf16 with a branch of 64 nodes, against 15.8.)
__device__ __forceinline__ void publish_and_walk(const VerifyKArgs& a, int b, int j, int truth, int lane) {
    constexpr int Q = (OT_MAX_NODES + 1 + 63) / 64, QN = OT_MAX_NODES / 64;
    const int n = a.n;
    u64* const words = a.truth + (size_t)b * word_stride(n);
    if (lane == 0) __hip_atomic_store(words + j, kPublished | (u64)(unsigned)truth, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // the tree: lane owns nodes lane, lane + 64, ...; few rows ask for it ahead of knowing whether it is needed
    int n_out = 0, tok[QN], par[QN];
    auto load_tree = [&]() {
        n_out = min(a.n_out[b], n);
#pragma unroll
        for (int q = 0; q < QN; ++q) {
            const int i = min(lane + 64 * q, n - 1);
            tok[q] = a.token[(size_t)b * n + i];
            par[q] = a.parent[(size_t)b * n + i];
        }
    };
    const bool early = gridDim.x <= 1024;
    if (early) load_tree();
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    auto word = [&](int i) -> u64 {
        return i <= n ? __hip_atomic_load(words + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : kPublished;
    };
    auto there = [](u64 v) { return (v >> kTokenBits) == (kPublished >> kTokenBits); };
    // many rows: most workgroups see from the 64 words around their own that rows are missing (32 sequences of 257 rows of
    // 8192 fp32, greedy / sampled, all words read past the caches by every row, words of sequences side by side 67 / 66 us; now
    // 52 / 54.  A look at the 16 words of the own cache line first gains 1 us at 62 rows a sequence and loses 2 at 257.)
    if (!early && n >= 64 && !__all(there(word((j & ~63) + lane)))) return;
    u64 w[Q];
    bool all = true;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        w[q] = word(lane + 64 * q);
        all = all && there(w[q]);
    }
    if (!__all(all)) return;
    if (!early) load_tree();
    int32_t* const out_tok = a.accept_token + (size_t)b * (n + 1);
    int32_t* const out_node = a.accept_node + (size_t)b * n;
    // Position 0 is the root, position i + 1 node i.  next[p] = ground truth after position p | the child that carries it
    // << kTokenBits (kNoChild: none; children of one node carry distinct tokens, among equal ones the smaller index counts).
    constexpr int kNoChild = 511, kTokenMask = (1 << kTokenBits) - 1;
    static_assert(OT_MAX_NODES <= kNoChild && kTokenBits + 9 < 31, "a child fits the word");
    __shared__ int s_truth[64 * Q], s_child[64 * Q];
    int next[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        s_truth[lane + 64 * q] = (int)w[q] & kTokenMask;
        s_child[lane + 64 * q] = kNoChild;
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");        // (one wavefront: its own LDS traffic only)
#pragma unroll
    for (int q = 0; q < QN; ++q) {
        const int p = par[q] + 1;
        if ((unsigned)p <= (unsigned)n && lane + 64 * q < n_out && s_truth[p] == tok[q]) atomicMin(&s_child[p], lane + 64 * q);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int q = 0; q < Q; ++q) next[q] = s_truth[lane + 64 * q] | s_child[lane + 64 * q] << kTokenBits;
    // the results of 64 steps wait in the lanes
    int p = 0, A = 0, my_tok = -1, my_node = -1;
    auto store = [&](int i) {
        if (i <= n) out_tok[i] = my_tok;
        if (i < n) out_node[i] = my_node;
    };
    for (int step = 0; step <= n_out; ++step) {               // a branch has at most n_out nodes
        int v = rl(next[0], p & 63);
        if (n >= 64) {
#pragma unroll
            for (int q = 1; q < Q; ++q)
                if ((p >> 6) == q) v = rl(next[q], p & 63);
        }
        const int nx = v >> kTokenBits;
        if (lane == (A & 63)) { my_tok = v & kTokenMask; my_node = nx != kNoChild && step < n_out ? nx : -1; }
        if ((A & 63) == 63) {
            store(A - 63 + lane);
            my_tok = my_node = -1;
        }
        ++A;
        if (nx == kNoChild) break;
        p = nx + 1;
    }
    // A tokens produced, A - 1 nodes accepted; the rest of the output rows is padding
    for (int i = (A & ~63) + lane; i <= n; i += 64) {
        store(i);
        my_tok = my_node = -1;
    }
    if (lane == 0) a.accept_len[b] = A;
#pragma unroll
    for (int q = 0; q < Q; ++q)
        if (lane + 64 * q <= n) __hip_atomic_store(words + lane + 64 * q, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A row's vectors: vector v holds elements v VEC - shift .. v VEC - shift + VEC - 1; loads are aligned whatever the row's
// alignment is.
template <int DT>
struct Row {
    static constexpr int VEC = VecOf<DT>::N, ESIZE = 16 / VEC;
    const char* base;
    int shift, len, nvec;
    __device__ __forceinline__ Row(const VerifyKArgs& a, int b, int j) {
        const char* const first = (const char*)a.logits + ((long long)b * a.stride_seq + (long long)j * a.stride_row) * ESIZE;
        shift = (int)((uintptr_t)first & 15) / ESIZE;
        base = first - shift * ESIZE;
        len = a.vocab;
        nvec = (shift + len + VEC - 1) / VEC;
    }
    __device__ __forceinline__ u32x4 load(int v) const { return *(const u32x4*)(base + (unsigned)min(v, nvec - 1) * 16u); }
    __device__ __forceinline__ u32x4 stream(int v) const {
        return __builtin_nontemporal_load((const u32x4*)(base + (unsigned)min(v, nvec - 1) * 16u));
    }
    // vectors v0 .. v0 + count - 1 may hold elements that are not the row's (uniform)
    __device__ __forceinline__ bool edge(int v0, int count) const { return (v0 == 0 && shift > 0) || (v0 + count) * VEC > shift + len; }
    __device__ __forceinline__ void mask(float (&x)[VEC], int v) const {
#pragma unroll
        for (int c = 0; c < VEC; ++c) x[c] = (unsigned)(v * VEC + c - shift) < (unsigned)len ? x[c] : -INFINITY;
    }
};

// Greedy: the most probable token of a row (equal logits: the smaller token id)
template <int DT, int NT>
__global__ __launch_bounds__(NT) void verify_greedy_kernel(const VerifyKArgs a) {
    constexpr int NW = NT / 64, VEC = Row<DT>::VEC;
    __shared__ float s_m[NW];
    __shared__ int s_tok;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = blockIdx.x / (a.n + 1), j = blockIdx.x - b * (a.n + 1);
    const Row<DT> row(a, b, j);
    if (tid == 0) s_tok = 0x7fffffff;
    u32x4 w[kBatch], nw[kBatch];
#pragma unroll
    for (int i = 0; i < kBatch; ++i) w[i] = row.stream(i * NT + tid);
    float m = -INFINITY;                                      // this lane's maximum and the first of its vectors that has it
    int at = tid;
    for (int v0 = 0; v0 < row.nvec; v0 += kBatch * NT) {
#pragma unroll
        for (int i = 0; i < kBatch; ++i) nw[i] = w[i];
        if (v0 + kBatch * NT < row.nvec) {
#pragma unroll
            for (int i = 0; i < kBatch; ++i) nw[i] = row.stream(v0 + (kBatch + i) * NT + tid);
        }
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            const int v = v0 + i * NT;
            if (v < row.nvec) {
                float x[VEC];
                VecOf<DT>::unpack(w[i], x);
                if (row.edge(v, NT)) row.mask(x, v + tid);
                float q = x[0];
#pragma unroll
                for (int c = 1; c < VEC; ++c) q = fmaxf(q, x[c]);
                at = q > m ? v + tid : at;
                m = fmaxf(q, m);
            }
        }
#pragma unroll
        for (int i = 0; i < kBatch; ++i) w[i] = nw[i];
    }
    const float mw = wave_max_f(m);
    if (lane == 0) s_m[wave] = mw;
    __syncthreads();
    float M = s_m[lane & (NW - 1)];
    M = wave_max_f(M);
    if (m == M) {                                             // (few lanes: their vectors again)
        float x[VEC];
        VecOf<DT>::unpack(row.load(at), x);
        int e = 0x7fffffff;
#pragma unroll
        for (int c = VEC - 1; c >= 0; --c) {
            const int t = at * VEC + c - row.shift;
            e = (x[c] == M && (unsigned)t < (unsigned)row.len) ? t : e;
        }
        atomicMin(&s_tok, e);
    }
    __syncthreads();
    if (wave == 0) publish_and_walk(a, b, j, s_tok < row.len ? s_tok : 0, lane);     // (a row of NaNs only: token 0)
}

// inclusive prefix sum over the lanes of a wavefront, as wave_incl_scan (lane exchanges by __shfl are trips
// to LDS: 31 x 156 rows of 1792 bf16 with the append 19.1 -> 18.3 us, 2 x 55 of 70400 fp32 17.3 -> 16.5.  Not kept: terms as one
// multiply-add with the rounded product of reference and factor as exponent, and asking for the whole segment's vectors while the drawn
// one is looked for: 4 % slower than before at short rows)
template <int CTRL, int ROW_MASK> __device__ __forceinline__ double dpp_zero_d(double v) {
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROW_MASK, 0xf, false),
                            __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROW_MASK, 0xf, false));
}
__device__ __forceinline__ double wave_scan_f64(double v) {
    v += dpp_zero_d<0x111, 0xf>(v);                           // row_shr 1, 2, 4, 8
    v += dpp_zero_d<0x112, 0xf>(v);
    v += dpp_zero_d<0x114, 0xf>(v);
    v += dpp_zero_d<0x118, 0xf>(v);
    v += dpp_zero_d<DPP_ROW_BCAST15, 0xa>(v);
    v += dpp_zero_d<DPP_ROW_BCAST31, 0xc>(v);
    return v;
}

// Sampling: the token at which the cumulative sum of exp(x / T), in token order, passes u x total.  The sums of all
// 16-byte vectors stay in LDS (fp32 inside a vector, fp64 above); 64 consecutive vectors are a segment, which one
// wavefront reads in one go with one reference exponent.  The segment that holds the draw, then the vector, are found by
// prefix sums over lanes; only that vector is read again.
// The reference of a segment is the wavefront's maximum so far: no term exceeds 1, whatever the temperature, and the terms
// that matter have exponents near 0, which fp32 rounds least.
constexpr int kMaxSeg = 512;
__device__ __forceinline__ float sample_term(float x, float ref, float c) { return __builtin_amdgcn_exp2f((x - ref) * c); }
template <int DT, int NT>
__global__ __launch_bounds__(NT) void verify_sample_kernel(const VerifyKArgs a) {
    constexpr int VEC = Row<DT>::VEC, PER_MAX = kMaxSeg / 64 + 1;    // (the longest row may start inside a vector)
    extern __shared__ __attribute__((aligned(16))) float s_e[];      // [segments x 64]  sum of exp2((x - ref) c) per vector
    __shared__ float s_ref[kMaxSeg + 1];                             // reference of a segment
    __shared__ double s_seg[kMaxSeg + 1];                              // sum over a segment
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = blockIdx.x / (a.n + 1), j = blockIdx.x - b * (a.n + 1);
    const Row<DT> row(a, b, j);
    const int nseg = (row.nvec + 63) / 64;
    float u = 0.f;
    u32x4 w[kBatch], nw[kBatch];
#pragma unroll
    for (int i = 0; i < kBatch; ++i) w[i] = row.stream(i * NT + tid);
    if (wave == 0) u = a.u[blockIdx.x];
    float ref = -INFINITY;
    for (int v0 = 0; v0 < row.nvec; v0 += kBatch * NT) {
#pragma unroll
        for (int i = 0; i < kBatch; ++i) nw[i] = w[i];
        if (v0 + kBatch * NT < row.nvec) {
#pragma unroll
            for (int i = 0; i < kBatch; ++i) nw[i] = row.stream(v0 + (kBatch + i) * NT + tid);
        }
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            const int v = v0 + i * NT, seg = v / 64 + wave;
            if (v < row.nvec && seg < nseg) {
                float x[VEC];
                VecOf<DT>::unpack(w[i], x);
                if (row.edge(v, NT)) row.mask(x, v + tid);
                float q = x[0];
#pragma unroll
                for (int c = 1; c < VEC; ++c) q = fmaxf(q, x[c]);
                if (__any(q > ref)) ref = wave_max_f(q);
                const float r = ref == -INFINITY ? 0.f : ref;        // (no logit yet: every term is 0)
                float e = 0.f;
#pragma unroll
                for (int c = 0; c < VEC; ++c) e += sample_term(x[c], r, a.c);
                s_e[v + tid] = fmaxf(e, 0.f);                        // (a vector with a NaN weighs nothing)
                if (lane == 0) s_ref[seg] = ref;
            }
        }
#pragma unroll
        for (int i = 0; i < kBatch; ++i) w[i] = nw[i];
    }
    __syncthreads();
    // segment sums, four threads each
    for (int q = tid; q < nseg * 4; q += NT) {
        double sum = 0.0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const f32x4 x = *(const f32x4*)(s_e + 16 * q + 4 * i);
#pragma unroll
            for (int c = 0; c < 4; ++c) sum += (double)x[c];
        }
        sum += dpp_d<DPP_QUAD_XOR1>(sum);
        sum += dpp_d<DPP_QUAD_XOR2>(sum);
        if ((q & 3) == 0) s_seg[q >> 2] = sum;
    }
    __syncthreads();
    if (wave > 0) return;
    // lane L owns the segments [L per, (L + 1) per)
    const int per = (nseg + 63) / 64;                                // <= PER_MAX, checked by the host
    float ms[PER_MAX], M = -INFINITY;
#pragma unroll
    for (int i = 0; i < PER_MAX; ++i) {
        const int s = lane * per + i;
        ms[i] = i < per && s < nseg ? s_ref[s] : -INFINITY;
        M = fmaxf(M, ms[i]);
    }
    M = wave_max_f(M);
    int truth = 0;                                                   // no finite logit in the row: nothing to draw from
    if (M != -INFINITY) {
        double sc[PER_MAX], wt[PER_MAX], lane_sum = 0.0;
#pragma unroll
        for (int i = 0; i < PER_MAX; ++i) {
            sc[i] = wt[i] = 0.0;
            if (i < per) {
                // weight of the segment relative to the largest reference (double exp2: relative error 1e-16)
                sc[i] = ms[i] == -INFINITY ? 0.0 : exp2(((double)ms[i] - (double)M) * (double)a.c);
                wt[i] = ms[i] == -INFINITY ? 0.0 : s_seg[lane * per + i] * sc[i];
                lane_sum += wt[i];
            }
        }
        const double incl = wave_scan_f64(lane_sum);
        const double target = (double)u * rl_d(incl, 63);
        // first lane whose segments reach past the target; by rounding there may be none: the last lane with weight
        const u64 past = __ballot(incl > target), any = __ballot(lane_sum > 0.0);
        if (past || any) {
            const int Ls = past ? __ffsll((long long)past) - 1 : 63 - __clzll((long long)any);
            // inside that lane: the first segment that passes the target, else (rounding) the end of its last one with weight
            bool found = false;
            int seg = 0;
            float mseg = 0.f;
            double before = incl - lane_sum, rs = 0.0;               // rs: residual in the segment's own units
#pragma unroll
            for (int i = 0; i < PER_MAX; ++i) {
                if (i < per && wt[i] > 0.0 && !found) {
                    seg = lane * per + i;
                    mseg = ms[i];
                    if (before + wt[i] > target) { found = true; rs = (target - before) / sc[i]; }
                    else rs = wt[i] / sc[i];
                }
                if (!found) before += wt[i];
            }
            seg = rl(seg, Ls);
            mseg = rl_f(mseg, Ls);
            rs = rl_d(rs, Ls);
            // inside the segment: the vector
            const int v = seg * 64 + lane;
            const double e = v < row.nvec ? (double)s_e[v] : 0.0;
            const double incl_e = wave_scan_f64(e);
            const u64 past_e = __ballot(incl_e > rs), any_e = __ballot(e > 0.0);
            const int Le = past_e ? __ffsll((long long)past_e) - 1 : max(63 - __clzll((long long)any_e), 0);
            // inside the vector: the element (every lane does the same)
            const double start = rl_d(incl_e - e, Le);
            float x[VEC];
            VecOf<DT>::unpack(row.load(seg * 64 + Le), x);
            row.mask(x, seg * 64 + Le);
            double acc = start;
            int k = -1, lastk = 0;
#pragma unroll
            for (int i = 0; i < VEC; ++i) {
                const float p = sample_term(x[i], mseg, a.c);
                acc += (double)p;
                if (p > 0.f) { lastk = i; if (k < 0 && acc > rs) k = i; }
            }
            truth = min(max((seg * 64 + Le) * VEC + (k < 0 ? lastk : k) - row.shift, 0), row.len - 1);
        }
    }
    publish_and_walk(a, b, j, truth, lane);
}

// Threads per row.  Few rows: more wavefronts per row shorten its latency; many: fewer leave less fixed work per element.
// Sampled rows keep 4 bytes of LDS per vector, so long ones leave room for few workgroups on a compute unit, which then need
// more threads each.  Measured, greedy / sampled us at 64, 256, 512, 1024 threads: 1000 bf16, 8100 rows 12.8 / 21.0,
// 19.5 / 27.7, 31.6 / 40.1, 60.7 / 57.2; 32000 bf16, 51 rows 13.4 / 20.0, 7.5 / 10.4, 7.5 / 9.5, 7.8 / 9.6; 976 rows
// 17.6 / 22.4, 15.5 / 19.4, 16.8 / 19.0, 18.3 / 22.8; 128256 bf16, 51 rows 39 / 60, 14.5 / 21.4, 10.6 / 16.8, 10.5 / 16.0;
// 2040 rows 79 / 259, 81 / 102, 81 / 90, 81 / 96; 128256 fp32, 2040 rows 154 / 722, 157 / 244, 158 / 188, 154 / 181.
template <int DT>
int launch_rows(VerifyKArgs a, int batch, bool sample, hipStream_t s) {
    const long long rows = (long long)batch * (a.n + 1), bytes = (long long)a.vocab * Row<DT>::ESIZE;
    int nt = bytes <= 16384 || rows > 256 ? 256 : (rows > 128 ? 512 : 1024);
    if (bytes <= 8192 && rows > 512) nt = 64;
    if (sample && bytes > 65536 && rows > 256) nt = bytes > 262144 ? 1024 : 512;
    const int nseg = (a.vocab + Row<DT>::VEC - 1 + 64 * Row<DT>::VEC - 1) / (64 * Row<DT>::VEC);
    const size_t lds = sample ? (size_t)nseg * 64 * 4 : 0;
#define OT_ROWS(KERNEL, NT)                                                                                                  \
    do {                                                                                                                     \
        if (lds > 48 * 1024)                                                                                                 \
            OT_HIP_CHECK(hipFuncSetAttribute((const void*)KERNEL<DT, NT>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)); \
        hipLaunchKernelGGL((KERNEL<DT, NT>), dim3(grid), dim3(NT), lds, s, a);                                               \
    } while (0)
#define OT_ROWS_NT(KERNEL)                                                          \
    do {                                                                            \
        if (nt == 64) OT_ROWS(KERNEL, 64);                                          \
        else if (nt == 256) OT_ROWS(KERNEL, 256);                                        \
        else if (nt == 512) OT_ROWS(KERNEL, 512);                                   \
        else OT_ROWS(KERNEL, 1024);                                                 \
    } while (0)
    const int per = sequences_per_launch(batch, (long long)nt * (a.n + 1));
    for (long long b = 0; b < batch; b += per) {
        const unsigned grid = (unsigned)((batch - b < per ? batch - b : per) * (a.n + 1));
        if (sample) OT_ROWS_NT(verify_sample_kernel);
        else OT_ROWS_NT(verify_greedy_kernel);
        OT_HIP_CHECK(hipGetLastError());
        const size_t nodes = (size_t)per * a.n, words = nodes + per;
        a.logits = (const char*)a.logits + per * a.stride_seq * Row<DT>::ESIZE;
        if (sample) a.u += words;
        a.token += nodes; a.parent += nodes; a.n_out += per;
        a.truth += (size_t)per * word_stride(a.n);
        a.accept_len += per; a.accept_node += nodes; a.accept_token += words;
    }
#undef OT_ROWS_NT
#undef OT_ROWS
    return OT_OK;
}

int launch_verify(const ot_verify_params& p, bool sample, float c, const void* logits, const float* u, const int32_t* token,
                  const int32_t* parent, const int32_t* n_out, void* workspace, int32_t* accept_len, int32_t* accept_node,
                  int32_t* accept_token, hipStream_t s) {
    VerifyKArgs a;
    a.logits = logits; a.stride_seq = p.stride_seq; a.stride_row = p.stride_row; a.vocab = p.vocab; a.n = p.n;
    a.c = c; a.u = u;
    a.token = token; a.parent = parent; a.n_out = n_out;
    a.truth = (u64*)workspace;
    a.accept_len = accept_len; a.accept_node = accept_node; a.accept_token = accept_token;
    return p.logits_dtype == OT_BF16 ? launch_rows<OT_BF16>(a, p.batch, sample, s) : launch_rows<OT_F32>(a, p.batch, sample, s);
}

size_t verify_bytes(const ot_verify_params& p) { return ((size_t)p.batch * (size_t)word_stride(p.n) * 8 + 255) / 256 * 256; }

struct AppendKArgs {
    void *Kp, *Vp;
    const void *Kt, *Vt;
    const int32_t *prefix_len, *accept_len, *accept_node;
    int32_t* new_prefix_len;
    int kv_heads, n, D, max_prefix, esize;
    long long kps[3], vps[3], kts[3], vts[3];
};

// A workgroup per (sequence, KV head) and kAppendRounds x 256 vectors that could be accepted: K and V rows of the accepted
// nodes accept_node[j] go to prefix rows L + j, 16 bytes per lane, all of a branch's usual few rows at once.  Three trips to
// memory bound it (lengths and node, rows, writes).  (A wavefront for every row that could be accepted had n times as many
// workgroups, nearly all without work; one workgroup whatever n and head_dim are took 235 us for 256 accepted rows of 1024
// fp32 of four heads, 7 as now.)
constexpr int kAppendRounds = 8;
__global__ __launch_bounds__(256) void kv_append_kernel(const AppendKArgs a) {
    const int b = blockIdx.x / a.kv_heads, h = blockIdx.x - b * a.kv_heads;
    const int chunks = a.D * a.esize / 16;                    // 16-byte chunks per row
    // the first round's node, asked for together with the lengths
    const int first = blockIdx.y * 256 + threadIdx.x, step = gridDim.y * 256;
    int node = a.accept_node[(size_t)b * a.n + min(first / (2 * chunks), a.n - 1)];
    int L = a.prefix_len[b];
    L = L < 0 ? 0 : (L > a.max_prefix ? a.max_prefix : L);
    const int cnt = a.accept_len[b] - 1;                      // accepted nodes
    if (h == 0 && first == 0) a.new_prefix_len[b] = L + cnt < a.max_prefix ? L + cnt : a.max_prefix;
    const int rows = min(min(cnt, a.n), a.max_prefix - L);
    for (int i = first; i < rows * 2 * chunks; i += step) {
        const int r = i / chunks, c = i - r * chunks, j = r >> 1;
        if (i != first) node = a.accept_node[(size_t)b * a.n + j];
        if (node < 0 || node >= a.n) continue;
        const bool v = r & 1;
        const long long* const ts = v ? a.vts : a.kts;
        const long long* const ps = v ? a.vps : a.kps;
        const char* const src = (const char*)(v ? a.Vt : a.Kt) + ((long long)b * ts[0] + (long long)h * ts[1] + (long long)node * ts[2]) * a.esize;
        char* const dst = (char*)(v ? a.Vp : a.Kp) + ((long long)b * ps[0] + (long long)h * ps[1] + (long long)(L + j) * ps[2]) * a.esize;
        *(u32x4*)(dst + 16 * c) = *(const u32x4*)(src + 16 * c);
    }
}

int validate_verify(const ot_verify_params* p) {
    if (!p) return OT_ERR_INVALID_ARG;
    if (p->batch < 1 || p->vocab < 1 || p->n < 1) return OT_ERR_INVALID_ARG;
    if (p->logits_dtype != OT_F32 && p->logits_dtype != OT_BF16) return OT_ERR_INVALID_ARG;
    if (p->stride_row < p->vocab || p->stride_seq < 0) return OT_ERR_INVALID_ARG;
    if (p->n > OT_MAX_NODES || p->vocab > kMaxVocab) return OT_ERR_UNSUPPORTED;
    return OT_OK;
}

// segments of 64 vectors that the picking wavefront has room for
bool sample_supported(const ot_verify_params& p) { return p.vocab <= kMaxSeg * 64 * (p.logits_dtype == OT_BF16 ? 8 : 4); }

}  // namespace
}  // namespace ot

using namespace ot;

extern "C" {

size_t ot_verify_workspace_bytes(const ot_verify_params* p) {
    if (validate_verify(p) != OT_OK) return 0;
    return verify_bytes(*p);
}

int ot_verify_greedy(const ot_verify_params* p, const void* target_logits, const int32_t* token, const int32_t* parent,
                     const int32_t* n_out, void* workspace, size_t workspace_bytes, int32_t* accept_len,
                     int32_t* accept_node, int32_t* accept_token, void* hip_stream) {
    int st = validate_verify(p);
    if (st != OT_OK) return st;
    if (!target_logits || !token || !parent || !n_out || !workspace || !accept_len || !accept_node || !accept_token)
        return OT_ERR_INVALID_ARG;
    if ((uintptr_t)workspace % 16) return OT_ERR_INVALID_ARG;
    const int esize = p->logits_dtype == OT_BF16 ? 2 : 4;
    if ((uintptr_t)target_logits % esize) return OT_ERR_INVALID_ARG;
    const void* ip[6] = {token, parent, n_out, accept_len, accept_node, accept_token};
    for (int i = 0; i < 6; ++i)
        if ((uintptr_t)ip[i] % 4) return OT_ERR_INVALID_ARG;
    if (workspace_bytes < verify_bytes(*p)) return OT_ERR_WORKSPACE_TOO_SMALL;
    return launch_verify(*p, false, 0.f, target_logits, nullptr, token, parent, n_out, workspace, accept_len, accept_node,
                         accept_token, (hipStream_t)hip_stream);
}

size_t ot_verify_sample_workspace_bytes(const ot_verify_params* p) {
    if (validate_verify(p) != OT_OK) return 0;
    return sample_supported(*p) ? verify_bytes(*p) : 0;
}

int ot_verify_sample(const ot_verify_params* p, float temperature, const void* target_logits, const float* u,
                     const int32_t* token, const int32_t* parent, const int32_t* n_out, void* workspace,
                     size_t workspace_bytes, int32_t* accept_len, int32_t* accept_node, int32_t* accept_token,
                     void* hip_stream) {
    int st = validate_verify(p);
    if (st != OT_OK) return st;
    if (!(temperature > 0.f) || !(temperature <= 3.0e38f)) return OT_ERR_INVALID_ARG;
    if (!target_logits || !u || !token || !parent || !n_out || !workspace || !accept_len || !accept_node || !accept_token)
        return OT_ERR_INVALID_ARG;
    if ((uintptr_t)workspace % 16) return OT_ERR_INVALID_ARG;
    const int esize = p->logits_dtype == OT_BF16 ? 2 : 4;
    if ((uintptr_t)target_logits % esize) return OT_ERR_INVALID_ARG;
    const void* ip[7] = {u, token, parent, n_out, accept_len, accept_node, accept_token};
    for (int i = 0; i < 7; ++i)
        if ((uintptr_t)ip[i] % 4) return OT_ERR_INVALID_ARG;
    if (!sample_supported(*p)) return OT_ERR_UNSUPPORTED;
    if ((long long)p->batch * (p->n + 1) > 65535) return OT_ERR_UNSUPPORTED;
    if (workspace_bytes < verify_bytes(*p)) return OT_ERR_WORKSPACE_TOO_SMALL;
    const float c = fminf((float)(1.4426950408889634 / (double)temperature), 3.4028234e38f);      // (finite for any temperature)
    return launch_verify(*p, true, c, target_logits, u, token, parent, n_out,
                         workspace, accept_len, accept_node, accept_token, (hipStream_t)hip_stream);
}

int ot_kv_append(const ot_attn_params* p, void* K_prefix, void* V_prefix, const void* K_tree, const void* V_tree,
                 const int32_t* prefix_len, const int32_t* accept_len, const int32_t* accept_node,
                 int32_t* new_prefix_len, void* hip_stream) {
    if (!p) return OT_ERR_INVALID_ARG;
    if (p->batch < 1 || p->kv_heads < 1 || p->n < 1 || p->max_prefix < 1 || p->head_dim < 1) return OT_ERR_INVALID_ARG;
    if (p->dtype != OT_F32 && p->dtype != OT_BF16) return OT_ERR_INVALID_ARG;
    if (p->n > OT_MAX_NODES) return OT_ERR_UNSUPPORTED;
    if ((long long)p->batch * p->kv_heads > 65535) return OT_ERR_UNSUPPORTED;
    const int esize = p->dtype == OT_BF16 ? 2 : 4;
    if ((p->head_dim * esize) % 16) return OT_ERR_UNSUPPORTED;
    if (!K_prefix || !V_prefix || !K_tree || !V_tree || !prefix_len || !accept_len || !accept_node || !new_prefix_len)
        return OT_ERR_INVALID_ARG;
    const void* vp[4] = {K_prefix, V_prefix, K_tree, V_tree};
    for (int i = 0; i < 4; ++i)
        if ((uintptr_t)vp[i] % 16) return OT_ERR_INVALID_ARG;
    if (((uintptr_t)prefix_len % 4) || ((uintptr_t)accept_len % 4) || ((uintptr_t)accept_node % 4) ||
        ((uintptr_t)new_prefix_len % 4))
        return OT_ERR_INVALID_ARG;
    {   // the copying workgroups read prefix_len[b] while new_prefix_len[b] is written: the arrays must be disjoint
        const uintptr_t a0 = (uintptr_t)prefix_len, b0 = (uintptr_t)new_prefix_len, len = (uintptr_t)p->batch * 4;
        if (a0 < b0 + len && b0 < a0 + len) return OT_ERR_INVALID_ARG;
    }
    const int vec = 16 / esize;
    const int64_t* strides[4] = {p->kp_strides, p->vp_strides, p->kt_strides, p->vt_strides};
    for (int t = 0; t < 4; ++t) {
        for (int i = 0; i < 3; ++i)
            if (strides[t][i] < 0 || strides[t][i] % vec) return OT_ERR_INVALID_ARG;
        if (strides[t][2] < p->head_dim) return OT_ERR_INVALID_ARG;
    }
    AppendKArgs a;
    a.Kp = K_prefix; a.Vp = V_prefix; a.Kt = K_tree; a.Vt = V_tree;
    a.prefix_len = prefix_len; a.accept_len = accept_len; a.accept_node = accept_node; a.new_prefix_len = new_prefix_len;
    a.kv_heads = p->kv_heads; a.n = p->n; a.D = p->head_dim; a.max_prefix = p->max_prefix; a.esize = esize;
    for (int i = 0; i < 3; ++i) {
        a.kps[i] = p->kp_strides[i]; a.vps[i] = p->vp_strides[i]; a.kts[i] = p->kt_strides[i]; a.vts[i] = p->vt_strides[i];
    }
    const long long vectors = 2LL * p->n * (p->head_dim / vec);
    const unsigned groups = (unsigned)std::min((vectors + kAppendRounds * 256 - 1) / (kAppendRounds * 256), 65535LL);
    hipLaunchKernelGGL(kv_append_kernel, dim3(p->batch * p->kv_heads, groups), dim3(256), 0, (hipStream_t)hip_stream, a);
    OT_HIP_CHECK(hipGetLastError());
    return OT_OK;
}

}  // extern "C"
