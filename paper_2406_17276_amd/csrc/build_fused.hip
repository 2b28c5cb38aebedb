// One-shot tree construction as one launch: workgroups that scan rows (row_scan.hpp) and, per sequence, one that drafts the
// tree (tree_draft.hpp) while they do.
//
// What bounds a small build is a chain: launch, rows, launch, selections step by step.  The rows of the first steps are
// few and come first, so the drafting workgroup, on the chip from the start, has most of its steps behind it when the last rows
// arrive.
#include <algorithm>
#include <type_traits>

#include "row_scan.hpp"
#include "tree_draft.hpp"

namespace ot {
namespace {

struct FusedArgs {
    ScanKArgs scan;
    TreeBuildArgs tree;
    u64* there;                        // [batch][rows]
    u64* marks;                        // [batch]
    int n, depth, spin;
    int draft_threads;                 // wavefronts that draft: as many as a step has candidates for
};

// Workgroups 0 .. batch - 1 draft, the others scan a row each, rows of a step before those of the next.  SNT threads draft.
template <int DT, int NT, int VPL, bool KEEP, int SNT, int KPT, bool ADAPT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(NT >= 1024 ? 8 : 4, NT >= 1024 ? 8 : 4))) void build_fused_kernel(
    const void* logits, const long long stride_seq, const long long stride_depth, const long long stride_row, const int vocab,
    const int part_geom, const int batch, const int grow, const FusedArgs a) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int tid = threadIdx.x, rows = a.scan.rows_per_seq;
    int b = blockIdx.x;
    Arrivals ar;
    ar.rows = rows; ar.spin = a.spin; ar.wait = true;
    if (b >= batch) {
        typedef Scan<DT, NT, VPL, KEEP, true> S;
        ScanShared<NT, KEEP>& sh = *(ScanShared<NT, KEEP>*)smem;
        if (tid == 0) { sh.count = 0; sh.nvec = 0; }
        const int r = b / batch - 1;
        b -= (r + 1) * batch;
        const Item it = locate<DT>(logits, stride_seq, stride_depth, stride_row, vocab, part_geom, grow, rows, b, r, 0);
        u32x4 w[S::R];
#pragma unroll
        for (int i = 0; i < S::R; ++i) w[i] = S::load(it, i, tid);
        S scan{sh, a.scan, __builtin_amdgcn_readfirstlane(tid >> 6)};
        const float tau = scan.stream(it, w);
        scan.finish(it, tau);
        // the row's results have reached memory before its word is set
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        int* const over = (int*)smem;
        if (tid == 0)
            *over = __hip_atomic_exchange(a.there + it.rid, kRowThere, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == kRowLate;
        __syncthreads();
        if (!*over) return;
        // the drafting workgroup has marked this row
        ar.wait = false;
        ar.there = a.there + (size_t)b * rows; ar.marks = a.marks + b;
        __syncthreads();                                      // (everybody has looked)
        if (tid < 64) *over = take_over(ChipWave{tid, true}, ar);
        __syncthreads();
        if (!*over) return;
        __syncthreads();
    }
    if (tid >= a.draft_threads) return;
    ar.there = a.there + (size_t)b * rows; ar.marks = a.marks + b;
    Shared<SNT>& s = *(Shared<SNT>*)smem;
    draft_tree<SNT, KPT, kArrive, ADAPT>(s, smem + sizeof(Shared<SNT>), a.draft_threads, b, a.scan.row_topv, a.scan.row_lse, a.scan.k, rows, a.n, a.depth, 0,
                                         a.depth, a.tree, ar);
}

template <int DT, int NT, int VPL, bool KEEP, int SNT, int KPT>
int launch_t(const ScanGeometry& g, const void* logits, FusedArgs a, int wide, bool adapt, hipStream_t s) {
    auto waves = [](int n) { return (n + 63) / 64 * 64; };
    a.draft_threads = KPT > 1 ? SNT : std::max({256, waves(wide), waves((a.tree.batch_pool + kPoolPerThread - 1) / kPoolPerThread)});
    const size_t lds = std::max(sizeof(ScanShared<NT, KEEP>), sizeof(Shared<SNT>) + pool_bytes(a.tree.batch_pool) + 16);
    const int part_geom = 1 | (g.vocab << 4), grow = g.nsteps | (g.grow_k << 8) | (g.grow_n << 16);
    const dim3 gd((unsigned)(g.batch * (g.rows + 1)));
#define OT_FUSED(ADAPT)                                                                                                             \
    do {                                                                                                                            \
        if (lds > 64 * 1024)                                                                                                        \
            OT_HIP_CHECK(hipFuncSetAttribute((const void*)build_fused_kernel<DT, NT, VPL, KEEP, SNT, KPT, ADAPT>,                    \
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));                                \
        hipLaunchKernelGGL((build_fused_kernel<DT, NT, VPL, KEEP, SNT, KPT, ADAPT>), gd, dim3(NT), lds, s, logits, g.stride_seq,      \
                           g.stride_depth, g.stride_row, g.vocab, part_geom, g.batch, grow, a);                                     \
    } while (0)
    if (adapt) OT_FUSED(true);
    else OT_FUSED(false);
#undef OT_FUSED
    OT_HIP_CHECK(hipGetLastError());
    return OT_OK;
}

// Threads that draft, as in tree_build.hip: a candidate each while that takes at most 512 of them.
template <int DT, int NT, int VPL, bool KEEP>
int launch_n(const ScanGeometry& g, const void* logits, const FusedArgs& a, int wide, bool adapt, hipStream_t s) {
    if constexpr (NT == 256) {
        if (wide <= 256) return launch_t<DT, NT, VPL, KEEP, 256, 1>(g, logits, a, wide, adapt, s);
        return launch_t<DT, NT, VPL, KEEP, 256, 2>(g, logits, a, wide, adapt, s);
    } else {
        if (wide <= 512) return launch_t<DT, NT, VPL, KEEP, 512, 1>(g, logits, a, wide, adapt, s);
        return launch_t<DT, NT, VPL, KEEP, NT, 1024 / NT>(g, logits, a, wide, adapt, s);
    }
}

int widest(const SelectGeometry& g) { return g.k * *std::max_element(g.F, g.F + g.depth); }

}  // namespace

// Where one launch is faster: the drafting workgroup needs steps to do while rows are scanned, a candidate or two per thread,
// and its LDS, 45 KB and more, must not take the place of the scan's workgroups.  Two launches / one, us:
// 412 rows of 32000 bf16 (n = 50, k = 10) 19.7 / 16.1, 823 26.3 / 18.2, 1235 30.7 / 23.9; 612 rows, n = 64, stopping rule 23.3 / 17.1;
// 516 rows of 32003 20.8 / 15.6; 800 rows of 4000 16.6 / 14.2, 1600 19.8 / 16.6, 3200 24.1 / 27.3; 800 rows of 50000 30.4 / 28.1,
// 1600 42.1 / 47.6; 37 rows of 1000 fp32 10.4 / 9.9; 258 rows of 66040 25.6 / 20.7.  One step or two: 6 groups of 47268 fp32 15.5 /
// 16.0, 35 of 39956 13.9 / 14.2; k = 1: 50 rows of 960 12.1 / 13.5; 928 candidates by 256 threads 21.9 / 24.2.
bool fuse_build(const ScanGeometry& sg, const SelectGeometry& g, const void* logits) {
    const ScanForm f = scan_form(sg, logits);
    if (f.parts > 1 || f.threads == 64 || (f.threads == 256 && !f.keep)) return false;
    if (g.batch > 32 || g.k == 1 || g.depth <= 2) return false;
    const int pool = g.row_start[g.depth] + g.F[g.depth] - 1;
    if (widest(g) > (f.threads == 256 ? 512 : 1024) || pool > kPoolPerThread * (f.threads == 256 ? 256 : 512)) return false;
    if (sizeof(Shared<1024>) + pool_bytes(pool) + 16 > 80 * 1024) return false;       // two workgroups a compute unit
    const long long groups = (long long)g.batch * (sg.rows + 1);
    return f.threads == 1024 || groups <= (f.threads == 256 ? 1536 : 1024);
}

int launch_fused_build(const ScanGeometry& sg, const SelectGeometry& g, const void* logits, bool adapt, double delta,
                       const BuildWorkspace& ws, const ot_tree_out& out, int32_t* steps_used, double* e_sub, int spin, hipStream_t s) {
    FusedArgs a;
    a.scan = ScanKArgs{};
    a.scan.k = g.k; a.scan.parts = 1; a.scan.rows_per_seq = sg.rows_per_seq;
    a.scan.row_lse = ws.row_lse; a.scan.row_topv = ws.row_topv; a.scan.row_topi = ws.row_topi;
    a.tree = TreeBuildArgs{};
    a.tree.topi = ws.row_topi;
    a.tree.batch_pool = g.row_start[g.depth] + g.F[g.depth] - 1;
    a.tree.delta = delta; a.tree.steps_used = steps_used; a.tree.e_sub = e_sub;
    a.tree.out = out;
    // state of a streaming build, which a one-shot build has no use for
    a.there = (u64*)ws.pool_p;
    a.marks = (u64*)ws.step_tau;
    a.n = g.n; a.depth = g.depth; a.spin = spin;
    const ScanForm f = scan_form(sg, logits);
    const int wide = widest(g);
    auto launch = [&](auto dt) {
        constexpr int DT = decltype(dt)::value, KV = 32 / VecOf<DT>::N;
        if (f.threads == 256) return launch_n<DT, 256, KV, true>(sg, logits, a, wide, adapt, s);
        if (f.threads == 512) return launch_n<DT, 512, kRollVpl, false>(sg, logits, a, wide, adapt, s);
        return f.keep ? launch_n<DT, 1024, KV, true>(sg, logits, a, wide, adapt, s)
                      : launch_n<DT, 1024, kRollVpl, false>(sg, logits, a, wide, adapt, s);
    };
    return sg.dtype == OT_BF16 ? launch(std::integral_constant<int, OT_BF16>{}) : launch(std::integral_constant<int, OT_F32>{});
}

}  // namespace ot
