// Kernels and launches of the row scan (row_scan.hpp).
#include <algorithm>

#include "row_scan.hpp"

namespace ot {
namespace {

// The kernel's leading scalar arguments are what a work item needs to find its logits; the hardware hands them over in
// registers at wavefront start (kernel-argument preload), so the loads go out without a read of the argument block.
//   rows       rows of a sequence in this launch | first row << 16
// SKIP: rows of sequences that are finished (stopped by the rule of Algorithm 1, or their tree complete) are not read;
// the flags are on the device.  (A fixed set of workgroups that walks the rows of the live sequences makes launches over
// finished ones cheaper, 4.9 against 12 us at 8192 rows, but reads 5 to 8 % slower: 335 against 309 us for 2.1 GB.)
template <int DT, int NT, int VPL, bool KEEP, bool SKIP>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(8, 8))) void row_scan_kernel(
    const void* logits, const long long stride_seq, const long long stride_depth, const long long stride_row,
    const int vocab, const int part_geom, const int rows, const int grow, const ScanKArgs a) {
    __shared__ ScanShared<NT, KEEP> sh;
    const int parts = part_geom & 15, rows_here = rows & 0xffff, row0 = rows >> 16;
    if (threadIdx.x == 0) { sh.count = 0; sh.nvec = 0; }
    typedef Scan<DT, NT, VPL, KEEP> S;
    const int tid = threadIdx.x;
    const int lrow = blockIdx.x / parts, b = lrow / rows_here;
    if (SKIP && a.seq_active[b] == 0) return;
    const Item it = locate<DT>(logits, stride_seq, stride_depth, stride_row, vocab, part_geom, grow, a.rows_per_seq, b,
                               row0 + lrow - b * rows_here, blockIdx.x - lrow * parts);
    u32x4 w[S::R];
#pragma unroll
    for (int i = 0; i < S::R; ++i) w[i] = S::load(it, i, tid);
    S scan{sh, a, __builtin_amdgcn_readfirstlane(tid >> 6)};
    const float tau = scan.stream(it, w);
    scan.finish(it, tau);
}

// Rows that span several parts: combine the per-part (max, sum) pairs and merge the per-part top-k lists.
// One wavefront per row: the parts' statistics sit in the first lanes, the parts * k <= 128 candidates go through
// LDS and every lane ranks its (at most two) candidates by counting those that precede them (value desc, token
// asc: tokens of different parts differ, so the order is total); ranks below k are the row's list.
__global__ __launch_bounds__(256) void merge_parts_kernel(int items, int rows, int row0, int rows_per_seq, const int32_t* seq_active,
                                                          int parts, int k, const float* part_m,
                                                          const double* part_s, const float* part_topv,
                                                          const int32_t* part_topi, double* row_lse, float* row_topv,
                                                          int32_t* row_topi) {
    __shared__ float s_v[4][128];
    __shared__ int s_i[4][128];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int lrow = blockIdx.x * 4 + w;              // row of this launch; sequence b, row row0 + j of it
    const int b = min(lrow, items - 1) / rows, j = min(lrow, items - 1) - b * rows;
    const int rid = b * rows_per_seq + row0 + j;
    const bool live = lrow < items && !(seq_active && seq_active[b] == 0);
    const size_t base = (size_t)(live ? rid : 0) * parts;
    const int total = parts * k;
    // part_m is the part's reference exponent in log2 units (fp32 max times the fp32 log2e of the scan kernel)
    const float pm = lane < parts ? part_m[base + lane] : -INFINITY;
    const float M = wave_max(pm);
    const double s = wave_sum(lane < parts ? part_s[base + lane] * exp2((double)pm - (double)M) : 0.0);
    if (live && lane == 0) row_lse[rid] = (double)M / (double)kLog2e + log(s);
    for (int c = lane; c < total; c += 64) {               // the row's lists are contiguous: part p, rank r at p k + r
        s_v[w][c] = part_topv[base * k + c];
        s_i[w][c] = part_topi[base * k + c];
    }
    __syncthreads();
    float v[2]; int id[2], rank[2] = {0, 0};
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int c = lane + 64 * q;
        v[q] = c < total ? s_v[w][c] : -INFINITY;
        id[q] = c < total ? s_i[w][c] : 0x7fffffff;
    }
    for (int j = 0; j < total; ++j) {
        const float u = s_v[w][j];
        const int ui = s_i[w][j];
#pragma unroll
        for (int q = 0; q < 2; ++q) rank[q] += (u > v[q] || (u == v[q] && ui < id[q])) ? 1 : 0;
    }
#pragma unroll
    for (int q = 0; q < 2; ++q)
        if (live && lane + 64 * q < total && rank[q] < k) {
            row_topv[(size_t)rid * k + rank[q]] = v[q];
            row_topi[(size_t)rid * k + rank[q]] = id[q];
        }
}

}  // namespace

namespace {

template <int DT, int NT, int VPL, bool KEEP>
int launch_scan_t(const ScanGeometry& g, const void* logits, const ScanKArgs& a, int part_elems, hipStream_t s, hipEvent_t ev0,
                  hipEvent_t ev1) {
    const int part_geom = a.parts | (part_elems << 4);
    const int grow = g.nsteps | (g.grow_k << 8) | (g.grow_n << 16);
    const int rows = g.rows | (g.row0 << 16);
    const dim3 gd((unsigned)((long long)g.batch * g.rows * a.parts));
#define OT_SCAN_ARGS logits, g.stride_seq, g.stride_depth, g.stride_row, g.vocab, part_geom, rows, grow, a
    if (a.seq_active) hipLaunchKernelGGL((row_scan_kernel<DT, NT, VPL, KEEP, true>), gd, dim3(NT), 0, s, OT_SCAN_ARGS);
    else if (ev0 || ev1) hipExtLaunchKernelGGL((row_scan_kernel<DT, NT, VPL, KEEP, false>), gd, dim3(NT), 0, s, ev0, ev1, 0, OT_SCAN_ARGS);
    else hipLaunchKernelGGL((row_scan_kernel<DT, NT, VPL, KEEP, false>), gd, dim3(NT), 0, s, OT_SCAN_ARGS);
#undef OT_SCAN_ARGS
    OT_HIP_CHECK(hipGetLastError());
    return OT_OK;
}

template <int DT>
int launch_scan_dt(const ScanGeometry& g, const void* logits, ScanKArgs& a, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    constexpr int KV = 32 / VecOf<DT>::N;                     // KEEP: 32 elements per lane
    const ScanForm f = scan_form(g, logits);
    a.parts = f.parts;
    if (f.keep) {
        return f.threads == 256 ? launch_scan_t<DT, 256, KV, true>(g, logits, a, f.part_elems, s, ev0, ev1)
                                : launch_scan_t<DT, 1024, KV, true>(g, logits, a, f.part_elems, s, ev0, ev1);
    }
    if (f.threads == 64) return launch_scan_t<DT, 64, kRollVpl, false>(g, logits, a, f.part_elems, s, ev0, ev1);
    if (f.threads == 256) return launch_scan_t<DT, 256, kRollVpl, false>(g, logits, a, f.part_elems, s, ev0, ev1);
    if (f.threads == 512) return launch_scan_t<DT, 512, kRollVpl, false>(g, logits, a, f.part_elems, s, ev0, ev1);
    const int st = launch_scan_t<DT, 1024, kRollVpl, false>(g, logits, a, f.part_elems, s, ev0, ev1);
    if (st != OT_OK || a.parts == 1) return st;
    const long long rows = (long long)g.batch * g.rows;
    hipLaunchKernelGGL(merge_parts_kernel, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, s,
                       (int)rows, g.rows, g.row0, g.rows_per_seq, a.seq_active, a.parts, g.k, a.part_m, a.part_s, a.part_topv,
                       a.part_topi, a.row_lse, a.row_topv, a.row_topi);
    OT_HIP_CHECK(hipGetLastError());
    return OT_OK;
}

}  // namespace

int launch_row_scan(const ScanGeometry& g, const void* logits, const BuildWorkspace& ws, hipStream_t s, hipEvent_t ev0,
                    hipEvent_t ev1, bool skip_frozen) {
    if (g.vocab > kMaxVocab) return OT_ERR_UNSUPPORTED;
    if (g.nsteps < 1 || g.nsteps > 255 || g.grow_k < 1 || g.grow_k > 255 || g.grow_n < 1 || g.grow_n > 32767)
        return OT_ERR_INVALID_ARG;
    if (g.rows < 1 || g.row0 < 0 || g.row0 + g.rows > g.rows_per_seq || g.rows_per_seq > 0x7fff) return OT_ERR_INVALID_ARG;
    // the results of all rows of all sequences are indexed with 32 bits, however few of them this launch covers
    if ((long long)g.batch * g.rows_per_seq * max_scan_parts(g.vocab) > 0x7fffffffLL) return OT_ERR_UNSUPPORTED;
    ScanKArgs a;
    a.k = g.k;
    a.rows_per_seq = g.rows_per_seq;
    a.row_lse = ws.row_lse; a.row_topv = ws.row_topv; a.row_topi = ws.row_topi;
    a.part_m = ws.part_m; a.part_s = ws.part_s; a.part_topv = ws.part_topv; a.part_topi = ws.part_topi;
    a.seq_active = skip_frozen ? ws.seq_active : nullptr;
    auto launch = [&](const ScanGeometry& q, const void* x, hipEvent_t e0, hipEvent_t e1) {
        return q.dtype == OT_BF16 ? launch_scan_dt<OT_BF16>(q, x, a, s, e0, e1) : launch_scan_dt<OT_F32>(q, x, a, s, e0, e1);
    };
    const int per = sequences_per_launch(g.batch, 1024LL * g.rows * max_scan_parts(g.vocab));
    if (per == g.batch) return launch(g, logits, ev0, ev1);
    const size_t rows = (size_t)g.rows_per_seq, parts = (size_t)max_scan_parts(g.vocab);
    for (long long b = 0; b < g.batch; b += per) {
        ScanGeometry q = g;
        q.batch = g.batch - b < per ? (int)(g.batch - b) : per;
        const int st = launch(q, (const char*)logits + b * g.stride_seq * (g.dtype == OT_BF16 ? 2 : 4),
                              b == 0 ? ev0 : nullptr, b + per >= g.batch ? ev1 : nullptr);
        if (st != OT_OK) return st;
        a.row_lse += per * rows; a.row_topv += per * rows * g.k; a.row_topi += per * rows * g.k;
        if (parts > 1) {
            a.part_m += per * rows * parts; a.part_s += per * rows * parts;
            a.part_topv += per * rows * parts * g.k; a.part_topi += per * rows * parts * g.k;
        }
        if (a.seq_active) a.seq_active += per;
    }
    return OT_OK;
}

}  // namespace ot
