// A drafting step of the streaming builder as one launch: workgroups scan a row each (row_scan.hpp), and the one that completes a
// sequence's rows goes on with the step (tree_select.hpp).
//
// What bounds a decoder that calls the builder between its draft model's forwards is launches: 3.5 us of host time each.
#include <algorithm>
#include <type_traits>

#include "row_scan.hpp"
#include "tree_select.hpp"

namespace ot {
namespace {

struct ExpandArgs {
    ScanKArgs scan;
    SelKArgs step;
};

// Rows of a sequence are counted in its flag of the adaptive depth, by twos: 0 is a stopped sequence, 1 + 2 m one that goes on, m
// of whose rows are done.  The workgroup that finds all others done sets it to 1 again and takes the step.
template <int DT, int NT, int VPL, bool KEEP, int KMAX>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4, 4))) void tree_expand_kernel(
    const void* logits, const long long stride_seq, const long long stride_row, const int vocab, const int part_geom, const int F,
    const ExpandArgs a) {
    typedef Scan<DT, NT, VPL, KEEP, true> S;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    ScanShared<NT, KEEP>& sh = *(ScanShared<NT, KEEP>*)smem;
    __shared__ int s_last;
    const int tid = threadIdx.x, b = blockIdx.x / F, r = blockIdx.x - b * F;
    if (tid == 0) { sh.count = 0; sh.nvec = 0; }
    if (a.step.seq_active[b] == 0) {                          // stopped by the rule of Algorithm 1: its tree stays as it is
        if (r == 0 && tid == 0 && a.step.frontier_count) a.step.frontier_count[b] = 0;
        return;
    }
    const Item it = locate<DT>(logits, stride_seq, 0, stride_row, vocab, part_geom, 1 | 1 << 8 | 1 << 16, F, b, r, 0);
    u32x4 w[S::R];
#pragma unroll
    for (int i = 0; i < S::R; ++i) w[i] = S::load(it, i, tid);
    S scan{sh, a.scan, __builtin_amdgcn_readfirstlane(tid >> 6)};
    const float tau = scan.stream(it, w);
    scan.finish(it, tau);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");          // the results have reached memory before they count
    __syncthreads();
    if (tid == 0) {
        int32_t* const flag = a.step.seq_active + b;
        s_last = __hip_atomic_fetch_add(flag, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 1 + 2 * (F - 1);
        if (s_last) put<true>(flag, 1);
    }
    __syncthreads();
    if (!s_last || tid >= 64) return;
    draft_step<KMAX, true, true>(a.step, b, 64, (double*)smem);
}

template <int DT, int NT, int VPL, bool KEEP, int KMAX>
int launch_t(const ScanGeometry& g, const void* rows, const ExpandArgs& a, hipStream_t s) {
    const size_t lds = std::max(sizeof(ScanShared<NT, KEEP>), (size_t)KMAX * 64 * 8);
    hipLaunchKernelGGL((tree_expand_kernel<DT, NT, VPL, KEEP, KMAX>), dim3((unsigned)(g.batch * g.rows)), dim3(NT), lds, s, rows,
                       g.stride_seq, g.stride_row, g.vocab, 1 | (g.vocab << 4), g.rows, a);
    OT_HIP_CHECK(hipGetLastError());
    return OT_OK;
}
template <int DT, int NT, int VPL, bool KEEP>
int launch_n(const ScanGeometry& g, const void* rows, const ExpandArgs& a, hipStream_t s) {
    if (a.step.k <= 4) return launch_t<DT, NT, VPL, KEEP, 4>(g, rows, a, s);
    if (a.step.k <= 8) return launch_t<DT, NT, VPL, KEEP, 8>(g, rows, a, s);
    if (a.step.k <= 10) return launch_t<DT, NT, VPL, KEEP, 10>(g, rows, a, s);
    return launch_t<DT, NT, VPL, KEEP, 16>(g, rows, a, s);
}

}  // namespace

// Where one launch is faster: steps of one wavefront (n <= 64), with a row per compute unit at most.  Called one by one, ten steps of 50
// rows of 32000 with masks and E_sub 193 -> 156 us (the host's launches), seven other loops 1.02 to 1.2 times as fast; five loops of
// 74 to 239 nodes 0.4 to 1 % slower.  Replayed from a graph, the same ten steps 149 -> 141 us, 8 sequences of 7 nodes 185 -> 171,
// 15 of 6 168 -> 158, 0.93 to 1.02 over 40 loops, 0.97 in the mean; with more rows the step's registers leave the scan too few wavefronts (375 rows of 4736
// 155 -> 166, 966 of 3392 fp32 92 -> 98).
bool fuse_expand(const ScanGeometry& sg, int n, const void* rows) {
    const ScanForm f = scan_form(sg, rows);
    if (f.parts > 1 || f.threads == 64 || (f.threads == 256 && !f.keep)) return false;
    return n <= 64 && (long long)sg.batch * sg.rows <= 256;
}

int launch_fused_expand(const ScanGeometry& sg, const SelectGeometry& g, const void* rows, int step, const BuildWorkspace& ws,
                        int32_t* frontier_token, int32_t* frontier_parent, int32_t* frontier_count, hipStream_t s) {
    ExpandArgs a;
    a.scan = ScanKArgs{};
    a.scan.k = g.k; a.scan.parts = 1; a.scan.rows_per_seq = sg.rows_per_seq;
    a.scan.row_lse = ws.row_lse; a.scan.row_topv = ws.row_topv; a.scan.row_topi = ws.row_topi;
    a.step = make_args(g, ws);
    a.step.step = step;
    a.step.frontier_token = frontier_token; a.step.frontier_parent = frontier_parent; a.step.frontier_count = frontier_count;
    const ScanForm f = scan_form(sg, rows);
    auto launch = [&](auto dt) {
        constexpr int DT = decltype(dt)::value, KV = 32 / VecOf<DT>::N;
        if (f.threads == 256) return launch_n<DT, 256, KV, true>(sg, rows, a, s);
        if (f.threads == 512) return launch_n<DT, 512, kRollVpl, false>(sg, rows, a, s);
        return f.keep ? launch_n<DT, 1024, KV, true>(sg, rows, a, s) : launch_n<DT, 1024, kRollVpl, false>(sg, rows, a, s);
    };
    return sg.dtype == OT_BF16 ? launch(std::integral_constant<int, OT_BF16>{}) : launch(std::integral_constant<int, OT_F32>{});
}

}  // namespace ot
