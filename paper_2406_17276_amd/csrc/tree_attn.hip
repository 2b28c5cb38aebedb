// Tree-masked attention (Algorithm 2: the target model's forward over the drafted nodes with the tree
// attention mask; with n_keys > n also the draft model's attention of a drafting step, Sec. 4).
// For query row i of sequence b and query head h:
//   O[i] = sum_j softmax_j(scale q_i.k_j) v_j,  j over the cached prefix and the tree rows
//   whose bit is set in mask[b][i] (the node itself and its ancestors).
//
// The keys of one (sequence, KV head) are cut into 64-key tiles: ceil(L_b/64) prefix tiles,
// then ceil(n_keys/64) tree tiles.  Contiguous tile ranges ("splits") go to different workgroups so
// that a single small sequence still fills the chip; every split leaves an un-normalised
// partial (softmax reference, sum l, O); the last workgroup of a row block to finish merges them.
//
// bf16 path (attn_mfma_kernel): one workgroup = 64, 128 or 256 packed query rows of one KV head (GQA: the
// g = q_heads/kv_heads query heads that share the KV head are stacked, row = head*n + node), four
// wavefronts, eight for 256 rows.  Each wavefront
//   S^T = K Q^T   v_mfma_f32_32x32x16_bf16, A = K rows from LDS, B = Q held in registers;
//                 the accumulator leaves every lane with 16 scores of ONE query, so the
//                 online-softmax statistics and the rescale factor are per-lane scalars;
//   O^T += V^T P^T  same instruction, B = P straight from the S^T accumulators (the key order
//                 inside a 16-key slab is whatever the accumulator layout gives; V is read in
//                 the same order), A = V gathered from LDS.
// K/V tiles go from global memory straight into LDS (global_load_lds_dwordx4: 16 bytes per lane, no
// register staging), one to three tiles ahead of the computation, into a ring of two to four buffers; a tree
// tile's mask words (one 64-bit word per query row) travel the same way, just ahead of the tile.  A
// wavefront's 64 lanes land on 1 KB of consecutive LDS, so rows are unpadded and bank conflicts are
// avoided by an XOR swizzle instead: lane -> global chunk is chosen such that 16-byte chunk c of key
// row r sits at chunk position c ^ (r mod 16) (K), and 32-byte segment g of row r at g ^ v_swizzle(r) (V; see the kernel).
// Tiles that reach past the end of the keys re-read the last valid row for the missing rows (their scores
// are masked).  V is the transposed operand (a lane needs 8 keys of ONE column): it is read with the gfx950
// LDS transpose load ds_read_b64_tr_b16, which lets 16 lanes read four 32-byte row segments and hands
// lane i the i-th column of that 4x16 block -- two such loads per MFMA operand.
// The ancestor mask is applied bit by bit on tree tiles only (any number of tree keys: a tile needs one word per
// row); prefix tiles only mask the tail.  The kernel's first memory requests decide its length at the small
// shapes, so the prologue is kept short: divisions are multiplications by constants prepared on the host, the
// prefix length is fetched first, Q is requested before and the first tiles right after it is known.
//
// f32 path (attn_f32_kernel): fp32 matrix instructions, operands straight from memory; see there.
#include <math.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "common.hpp"
#include "internal.h"

namespace ot {
namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr int kMaxSplits = 32;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

struct AttnKArgs {
    const void *Q, *Kp, *Vp, *Kt, *Vt;
    const int32_t* prefix_len;
    const uint64_t* mask;
    void* O;
    unsigned int* counters;   // one ticket counter per (sequence, KV head, row block), zero between launches
    float* part_o;      // per-split partial O   (layout: see the kernel that writes it)
    float* part_ml;     // per-split (ref, l)
    int batch, kv_heads, g, n, nk, max_prefix, splits, W, row_blocks;   // n query rows, nk tree keys
    int splits_share_xcd;   // workgroup numbering of the bf16 kernel, see there
    unsigned int inv_splits, inv_kv_heads, inv_n;   // division by multiplication (fast_div): ceil(2^32 / d), unused for d = 1
    float scale_log2;   // softmax scale * log2(e)
    const float *k_scale, *v_scale;   // 8-bit K/V cache: one factor per (sequence, KV head) each; null otherwise
    long long qs[3], kps[3], vps[3], kts[3], vts[3], os[3];
};

// max over lanes l and l ^ 32 (v_permlane32_swap: no LDS round trip)
__device__ __forceinline__ float xhalf_max(float v) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float xhalf_sum(float v) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ int clamp_len(int L, int maxp) { return L < 0 ? 0 : (L > maxp ? maxp : L); }

// A prefix length outside [0, max_prefix] is clamped and reported in the workspace's status word.
__device__ __forceinline__ void report_clamp(unsigned int* sync_words, int raw, int maxp) {
    if (raw < 0 || raw > maxp)
        __hip_atomic_fetch_or(sync_words + OT_ATTN_STATUS_OFFSET / 4, OT_ATTN_STATUS_PREFIX_CLAMPED, __ATOMIC_RELAXED,
                              __HIP_MEMORY_SCOPE_AGENT);
}

// Wait until all but the N youngest memory requests of this lane have landed.  The Q fragments were requested
// with assembly the compiler does not track; they are in/out operands here, which places whatever reads them
// after this wait.  Executed once, ahead of the tile loop (straight-line code: the operands stay where they are).
template <int N, int SLABS>
__device__ __forceinline__ void wait_q(u32x4 (&q)[SLABS]) {
    static_assert(SLABS == 4 || SLABS == 8, "head_dim 64 or 128");
    if constexpr (SLABS == 8)
        asm volatile("s_waitcnt vmcnt(%8)"
                     : "+v"(q[0]), "+v"(q[1]), "+v"(q[2]), "+v"(q[3]), "+v"(q[4]), "+v"(q[5]), "+v"(q[6]), "+v"(q[7])
                     : "n"(N) : "memory");
    else
        asm volatile("s_waitcnt vmcnt(%4)" : "+v"(q[0]), "+v"(q[1]), "+v"(q[2]), "+v"(q[3]) : "n"(N) : "memory");
}

// x / d for x d < 2^32 as one multiplication by M = ceil(2^32 / d), prepared on the host (an integer division
// costs some forty instructions here, and the kernel's first memory requests wait for several of them).
__device__ __forceinline__ int fast_div(int x, int d, unsigned int M) {
    return d == 1 ? x : (int)__umulhi((unsigned int)x, M);
}

// Tile range of split s out of S over T tiles (T s < 2^32 / S).
__device__ __forceinline__ void split_range(int T, int S, unsigned int inv_S, int s, int& t0, int& t1) {
    t0 = fast_div(T * s, S, inv_S);
    t1 = fast_div(T * (s + 1), S, inv_S);
}

// Key splits that the merge of the bf16 kernel takes in one trip to memory (64 registers of partials, 96 in the narrow
// variant; 128, or none for splits that are not there, were 0.5 to 2 us slower)
constexpr int merge_chunk(int head_dim, bool wide) { return (wide ? 256 : 768) / head_dim; }

// Tile buffers of a variant (0: 64 rows, 1: 128, 2: 256, 3: 64 rows of 128, 16-bit cache, more workgroups than compute units).
// 64 rows: two buffers let two workgroups share a compute unit, one of which computes or widens while the other waits; with no
// more workgroups than units that gains nothing and the third buffer's second tile in flight does (four are 3 to 7 % slower
// than three).  An 8-bit tile is half the bytes in flight and has the widening in front of it: two buffers throughout.  us with
// three / two, one key range a KV head: 9 x 32 heads of 50 rows, 1000 keys 49.5 / 38.5 (8-bit 52.5 / 37.5), 4000 keys 161 / 115
// (165 / 113); 16 x 32 of 64 rows, 2000 keys 114 / 111 (101 / 81); 32 x 40 of 30 rows, 1000 keys 133 / 132 (127 / 93);
// 32 x 8 = 256 of 60 rows, 3000 keys 77 / 81 (70 / 66); one sequence of 32 heads, 1024 keys 12.0 / 12.1 (13.3 / 12.8).
constexpr int tile_buffers(int var, bool kv8) { return var == 2 ? (kv8 ? 3 : 4) : (var == 0 && !kv8 ? 3 : 2); }

// ---------------------------------------------------------------------------
// bf16 MFMA kernel
// ---------------------------------------------------------------------------
// WIDE = false: 64 packed rows per workgroup, wavefront = (query block of 32 rows) x (half of each
//                64-key tile); the two halves are merged through LDS at the end.  For few rows.
//                Three tile buffers -- two tiles are in flight while a third is being computed -- or two (tile_buffers).
// WIDE (VAR 1, 2): 128 or 256 packed rows per workgroup (four or eight wavefronts), wavefront = 32 rows x the whole tile; staging one
//                tile in LDS is shared by twice as many MFMAs and nothing is merged at the end.
//                128 rows: two tile buffers, so that two workgroups share a compute unit; 256 rows: four, one workgroup per unit.
// Workgroups are numbered so that those which stream the same K/V (the row blocks of one
// (sequence, KV head, split)) sit on the same XCD, next to each other in its dispatch order, and
// share that XCD's L2: hardware hands workgroup L to XCD L % 8.  When the (sequence, KV head) pairs divide evenly
// over the eight XCDs, the key splits of a pair share an XCD as well: they read the same Q rows, which then come
// from memory once per pair instead of once per split.
//
// With more than one split, every workgroup leaves its partial (O, m, l) in the workspace in the
// accumulator's own register order (coalesced 16-byte stores), then takes a ticket from the counter
// of its (sequence, KV head, row block); the workgroup that draws the last ticket merges all the
// partials of those rows and writes O.  Nobody waits for anybody: a workgroup that is not last simply
// ends.  The counter is reset by the merging workgroup, so it is zero again when the kernel ends.
// Partial results of the key splits travel as bf16, or as fp32 (define to 0): bf16 halves the exchange and lets the merging
// workgroup take twice as many ranges in a trip to memory (merge_chunk); the extra rounding is of the size of the output's
// own (the output is bf16).
#ifndef OT_ATTN_PART_BF16
#define OT_ATTN_PART_BF16 1
#endif
// KV8: K and V arrive as FP8 E4M3 bytes with a scale factor per (sequence, KV head) each.  A tile is copied into LDS
// as it is (half the bytes), then every thread widens its sixteen-byte pieces to bf16 -- every E4M3 value is a bf16
// value -- into the layout the operand reads expect: in place, behind two more barriers per tile, or (256 rows) two tiles
// ahead from a ring of raw tiles into a ring of bf16 tiles, each lane the pieces that it has requested itself; the K factor
// joins the softmax scale, the V factor the final normalisation.  Everything else is the bf16 kernel.
//
// BAL (wide variants, batches of 2 to 64 sequences that fill the chip, each (sequence, KV head) in one piece): the
// sequences of a batch differ in length, workgroups are handed out in the order of their number, and a launch lasts
// as long as the compute unit that finishes last.  Every workgroup therefore reads all prefix lengths first (lane j
// = sequence j), ranks the sequences by length and takes the job that its number stands for in the order "longest
// first" -- the order in which handing jobs to whichever unit is free balances best.
template <int D, int VAR, bool KV8, bool BAL>
__global__ __launch_bounds__(VAR == 2 ? 512 : 256) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_mfma_kernel(
    // what the first loads need, as leading scalar arguments: the hardware hands these over in registers at
    // wavefront start (kernel-argument preload); they repeat fields of `a`
    const int32_t* a_prefix_len, const uint64_t* a_mask, const void* a_Q, const int a_splits, const unsigned a_inv_splits,
    const int a_kv_heads, const unsigned a_inv_kv_heads, const int a_n, const unsigned a_inv_n, const AttnKArgs a) {
    const int a_g = a.g, a_max_prefix = a.max_prefix, a_nk = a.nk, a_W = a.W, a_row_blocks = a.row_blocks;
    constexpr bool WIDE = VAR == 1 || VAR == 2;
    constexpr int NWAVES = VAR == 2 ? 8 : 4;
    constexpr int NT = 64 * NWAVES;        // threads
    constexpr int TK = 64;                 // keys per tile
    constexpr int CPR = D / 8;             // 16-byte chunks per row
    constexpr int SPR = D / 16;            // 32-byte segments per row
    // Where V's 32-byte segment g of key row r sits inside the row: at g ^ v_swizzle(r).  A transposed operand read
    // touches, per 32 lanes, four consecutive rows (r mod 4 = 0..3) and the two halves of a 32-column block (segments
    // 2d and 2d + 1); LDS serves 256 bytes = eight segments per cycle, so these eight must fall into eight different
    // 32-byte slots of a 256-byte window: the row's low bits go into the bits above the half bit (a plain g ^ (r mod 8)
    // put two of them into every slot it used: every such read took twice its time).
    auto v_swizzle = [](int r) { return D == 128 ? (r & 3) << 1 : ((r >> 1) & 1) << 1; };
    constexpr int SLABS = D / 16;          // 16-wide d slabs of the QK^T contraction
    constexpr int DB = D / 32;             // 32-wide d blocks of O^T
    constexpr int ESZ = KV8 ? 1 : 2;       // bytes per stored K/V element
    constexpr int CPRG = D * ESZ / 16;     // 16-byte chunks per row in global memory
    constexpr int CH = TK * CPRG / NT;     // 16-byte chunks per thread per tile (K or V)
    static_assert(CH >= 1, "a tile has at least one chunk per thread");
    constexpr int LPT = 2 * CH;            // asynchronous loads per thread per tile
    constexpr int NKB = WIDE ? 2 : 1;      // 32-key blocks per wavefront per tile
    constexpr int ROWS = VAR == 2 ? 256 : (WIDE ? 128 : 64);   // packed query rows per workgroup
    constexpr int NQB = ROWS / 32;         // query blocks per workgroup
    constexpr bool PIPE8 = KV8 && VAR == 2;   // tiles are widened two tiles ahead, into a ring of their own
    constexpr int NBUF = tile_buffers(VAR, KV8);
    constexpr int PD = PIPE8 ? NBUF : NBUF - 1;   // tiles requested ahead of the one being computed (PIPE8: being widened)
    static_assert(PD >= 1 && PD <= 3 && PD * LPT < 64, "prefetch depth fits the vmcnt counter");

    constexpr int BUF = TK * D;            // dwords of one staged tile: K [64][D] bf16, then V [64][D] bf16
    constexpr int RAW = KV8 ? BUF / 2 : BUF;  // the same as it is stored
    extern __shared__ __attribute__((aligned(16))) unsigned int s_buf[];   // [NBUF][BUF], PIPE8: then [NBUF][RAW]
    unsigned int* const s_raw = s_buf + (PIPE8 ? NBUF * BUF : 0);           // where requested tiles land
    constexpr int SLOT = PIPE8 ? RAW : BUF;
    __shared__ int s_last;
    constexpr int MST = DB * 16 + 4;       // floats per lane in the half-merge scratch (a multiple of four)
    static_assert(sizeof(unsigned int) * NBUF * BUF >= 2 * 64 * MST * 4, "merge scratch fits");

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int qb = WIDE ? wave : (wave & 1), kh = WIDE ? 0 : (wave >> 1);
    const int l32 = lane & 31, h = lane >> 5;
    // workgroup numbering: see above
    // grid (8 x row blocks, units / 8): hardware hands workgroups out with x running fastest
    const int xcd = blockIdx.x & 7, rb = blockIdx.x >> 3;
    int bz, split;
    int L_bal = 0;
    if constexpr (BAL) {
        static_assert(WIDE, "wide variants only");
        const int B = a.batch;                                   // 2..64, one key range per (sequence, KV head)
        const int Lj = lane < B ? a_prefix_len[lane] : 0;
        const int Tj = lane < B ? clamp_len(Lj, a_max_prefix) : -1;
        int rank = 0;                                            // sequences ahead of sequence j: longer ones, and equally long ones before it
        for (int i = 0; i < B; ++i) {
            const int Ti = __builtin_amdgcn_readlane(Tj, i);
            rank += (Ti > Tj || (Ti == Tj && i < lane)) ? 1 : 0;
        }
        const int job = blockIdx.y * 8 + xcd;                    // position in the order longest first
        const int q = fast_div(job, a_kv_heads, a_inv_kv_heads);
        if (q >= B) return;
        const int b_sel = (int)__builtin_ctzll(__ballot(rank == q && lane < B));
        L_bal = __builtin_amdgcn_readlane(Lj, b_sel);
        bz = b_sel * a_kv_heads + (job - q * a_kv_heads);
        split = 0;
    } else if (a.splits_share_xcd) {
        // (sequence, KV head) pairs dealt round over the XCDs, all splits of a pair on the same one
        const int round = fast_div(blockIdx.y, a_splits, a_inv_splits);
        split = blockIdx.y - round * a_splits;
        bz = round * 8 + xcd;
        if (bz >= a.batch * a_kv_heads) return;
    } else {
        const int unit = blockIdx.y * 8 + xcd;
        if (unit >= a.batch * a_kv_heads * a_splits) return;
        bz = fast_div(unit, a_splits, a_inv_splits);
        split = unit - bz * a_splits;
    }
    const int b = fast_div(bz, a_kv_heads, a_inv_kv_heads), hk = bz - b * a_kv_heads;
    const int n = a_n;
    // the prefix length decides which tiles this workgroup streams: fetched first (a scalar load, ahead of the
    // hand-issued loads below), used only when the tile requests are built
    const int L_raw = BAL ? L_bal : a_prefix_len[b];

    // this lane's query row; lanes past the last row work on a copy of it and store nothing
    const int rho = rb * ROWS + qb * 32 + l32;         // packed row inside the KV head
    const bool row_ok = rho < a_g * n;
    const int rho_c = row_ok ? rho : a_g * n - 1;
    const int head = fast_div(rho_c, n, a_inv_n);
    const int hq = hk * a_g + head;
    const int node = rho_c - head * n;

    // Q fragments (B operand of S^T = K Q^T; lane holds Q[row][16 s + 8 h .. +7]) are requested first, as
    // assembly like the tile requests below: the compiler does not know that they are in flight, so nothing
    // waits for them until the first tile does (s_waitcnt in tile_step; loads complete in order, Q is the
    // oldest).  The registers are handed to that wait as in/out operands, which keeps every use behind it.
    u32x4 qw[SLABS];
    {
        const unsigned short* qrow = (const unsigned short*)a_Q + (long long)b * a.qs[0] + (long long)hq * a.qs[1] +
                                     (long long)node * a.qs[2] + 8 * h;
#pragma unroll
        for (int s = 0; s < SLABS; ++s)
            asm volatile("global_load_dwordx4 %0, %1, off offset:%2" : "=&v"(qw[s]) : "v"(qrow), "n"(32 * s) : "memory");
    }
    // this lane's ancestor mask row: one 64-bit word per 64-key tree tile, requested with the tile and, like it,
    // delivered straight into LDS (s_mw: per buffer and wavefront the low words of the 64 lanes, then the high words)
    const uint64_t* const mask_row = a_mask + ((long long)b * n + node) * a_W;
    unsigned int* const s_mw = s_raw + NBUF * SLOT;                     // [NBUF][waves][2][64]

    const unsigned char* kp = (const unsigned char*)a.Kp + ((long long)b * a.kps[0] + (long long)hk * a.kps[1]) * ESZ;
    const unsigned char* vp = (const unsigned char*)a.Vp + ((long long)b * a.vps[0] + (long long)hk * a.vps[1]) * ESZ;
    const unsigned char* kt = (const unsigned char*)a.Kt + ((long long)b * a.kts[0] + (long long)hk * a.kts[1]) * ESZ;
    const unsigned char* vt = (const unsigned char*)a.Vt + ((long long)b * a.vts[0] + (long long)hk * a.vts[1]) * ESZ;

    // transpose-load addressing: key row and first column this lane points at inside a 4-key x 32-column block
    const int tr_j = (lane & 15) >> 2, tr_q = 4 * (lane & 3);
    // swizzle terms of this lane's operand reads: K chunk (2s + h) of row l32 -> position (2s) ^ kx;
    // V segment (2d + g1) of row 4h + tr_j (mod 4) -> position (2d) ^ vx
    const int kx = h ^ (l32 & (CPR - 1));
    const int vx = ((lane >> 4) & 1) ^ v_swizzle(4 * h + tr_j);
    // scores are kept raw; p = 2^(c s - ref), ref = the rounded product of c and the row's largest score so far.  What is already
    // summed follows a change of ref by 2^(ref - ref'): with the rounded products on both sides, since their rounding errors
    // (half a unit at 2^24) are in every p and have to cancel.  From |c s| = 2^31 on half a unit in the last place is more than
    // an exponent holds: the row is then not finite.  An 8-bit cache's K factor scales every score: it joins c.
    const float c = KV8 ? a.scale_log2 * a.k_scale[bz] : a.scale_log2;
    const float v_factor = KV8 ? a.v_scale[bz] : 1.f;
    // The fast loops have no branch for a row without a score above -inf so far: its reference there is the lowest finite number,
    // from which -inf gives p = 0 and any finite score an infinite p, which leaves the loop.
    constexpr float kNoRef = -3.402823466e38f;
    float ref = -INFINITY, l_run = 0.f;
    f32x16 oacc[DB];
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
        for (int v = 0; v < 16; ++v) oacc[d][v] = 0.f;

    // LDS slot sigma = cc * NT + tid (16 bytes each) holds key row sigma / CPR, chunk position sigma % CPR;
    // the chunk stored there is the one the swizzle maps to that position.  KSTEP rows separate cc and cc+1,
    // a multiple of 16, so the swizzle term is the same for every cc.
    // (KV8: the copy is not swizzled -- slot sigma holds chunk sigma % CPRG of row sigma / CPRG -- the widening is.)
    constexpr int KSTEP = NT / CPRG;
    const int kkey0 = tid / CPRG, pc = tid % CPRG;
    const int kcol = KV8 ? pc * 16 : (pc ^ (kkey0 & (CPR - 1))) * 16;                        // byte column; K: chunk c = pc ^ (r % 16)
    const int vcol = KV8 ? pc * 16 : (2 * ((pc >> 1) ^ v_swizzle(kkey0)) + (pc & 1)) * 16;  // V: segment g = (pc/2) ^ v_swizzle(r)
    const int wave_u = wave;
    // Request tile t: global memory -> LDS buffer `buf`, 16 bytes per lane and instruction, no registers in
    // between.  Full tiles address memory as (uniform base of the tile's rows) + (this lane's fixed 32-bit
    // offset), which costs no vector arithmetic.  Tiles that reach past the end of the keys (prefix tail,
    // last tree tile) compute per-lane addresses and re-read the last valid row for the rows past the end:
    // their scores are masked below, so their probabilities are exactly zero and the values only need to be
    // finite.  Written as assembly on purpose: the compiler does not track these loads, so it puts no wait
    // between them and the LDS reads of the tile being computed; completion is awaited explicitly, per tile,
    // with s_waitcnt vmcnt (loads complete in order) ahead of the barrier that publishes the buffer.
    const unsigned kofs_p = (unsigned)(kkey0 * (int)a.kps[2] * ESZ + kcol), vofs_p = (unsigned)(kkey0 * (int)a.vps[2] * ESZ + vcol);
    const unsigned kofs_t = (unsigned)(kkey0 * (int)a.kts[2] * ESZ + kcol), vofs_t = (unsigned)(kkey0 * (int)a.vts[2] * ESZ + vcol);
    const int L = clamp_len(L_raw, a_max_prefix);
    const int ptiles = (L + TK - 1) / TK, ttiles = (a_nk + TK - 1) / TK;
    int t0, t1;
    split_range(ptiles + ttiles, a_splits, a_inv_splits, split, t0, t1);
    auto request_tile = [&](int t, auto buf_c) {
        const int buf = buf_c;                 // a compile-time constant or, in the wide variant's fast loop, a value
        const bool tree = t >= ptiles;
        // the mask word of a tree tile travels ahead of the tile's K/V (older, so it has landed when the tile's
        // wait is over)
        if (tree && !PIPE8) {
            const unsigned lds_w = (unsigned)(size_t)(__attribute__((address_space(3))) void*)(s_mw + (buf * NWAVES + wave) * 128);
            const unsigned int* const wp = (const unsigned int*)(mask_row + (t - ptiles));
            asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dword %1, off" ::"s"(lds_w), "v"(wp) : "m0", "memory");
            asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dword %1, off" ::"s"(lds_w + 256), "v"(wp + 1) : "m0", "memory");
        }
        const int key0 = tree ? (t - ptiles) * TK : t * TK;
        const int last = (tree ? a_nk : L) - 1;
        const long long ks = (tree ? a.kts[2] : a.kps[2]) * ESZ;      // row strides in bytes
        const long long vs = (tree ? a.vts[2] : a.vps[2]) * ESZ;
        const unsigned char* kbase = tree ? kt : kp;
        const unsigned char* vbase = tree ? vt : vp;
        unsigned int* const lk = s_raw + buf * SLOT;
        unsigned int* const lv = lk + (PIPE8 ? RAW / 2 : TK * D / 2);
        if (key0 + TK - 1 <= last) {
            const unsigned kofs = tree ? kofs_t : kofs_p, vofs = tree ? vofs_t : vofs_p;
            const unsigned char* gk = kbase + (long long)key0 * ks;       // uniform: rows key0 + cc KSTEP of the tile
            const unsigned char* gv = vbase + (long long)key0 * vs;
            unsigned lds_k = (unsigned)(size_t)(__attribute__((address_space(3))) void*)(lk + wave_u * 256);
            unsigned lds_v = (unsigned)(size_t)(__attribute__((address_space(3))) void*)(lv + wave_u * 256);
#pragma unroll
            for (int cc = 0; cc < CH; ++cc) {                 // 16-byte slots cc * NT + wave * 64 + lane
                asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_k), "v"(kofs), "s"(gk) : "m0", "memory");
                asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_v), "v"(vofs), "s"(gv) : "m0", "memory");
                gk += KSTEP * ks; gv += KSTEP * vs;
                lds_k += NT * 16; lds_v += NT * 16;
            }
        } else {
#pragma unroll
            for (int cc = 0; cc < CH; ++cc) {
                const int slot0 = cc * NT + wave_u * 64;
                const unsigned lds_k = (unsigned)(size_t)(__attribute__((address_space(3))) void*)(lk + slot0 * 4);
                const unsigned lds_v = (unsigned)(size_t)(__attribute__((address_space(3))) void*)(lv + slot0 * 4);
                int row = key0 + kkey0 + cc * KSTEP;
                row = row < last ? row : last;
                const unsigned char* gk = kbase + row * ks + kcol;
                const unsigned char* gv = vbase + row * vs + vcol;
                asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_k), "v"(gk) : "m0", "memory");
                asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_v), "v"(gv) : "m0", "memory");
            }
        }
    };

    // The first PD tiles are requested at once.  A split with fewer tiles issues the same number of loads all the
    // same (one word each, into the unused buffer's mask-word slots: a load without a destination register): the
    // wait for Q below can then name a fixed count of younger requests.
    auto pad_requests = [&](int buf) {
        const unsigned lds_w = (unsigned)(size_t)(__attribute__((address_space(3))) void*)(s_mw + (buf * NWAVES + wave) * 128);
#pragma unroll
        for (int i = 0; i < LPT; ++i)
            asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dword %1, off" ::"s"(lds_w), "v"(a_prefix_len) : "m0", "memory");
    };
    // Sixteen E4M3 values as bf16, which holds each of them.  The conversion straight to bf16 is half the instructions: the
    // 64-row variant gains 5 to 9 % (16 rows x 30 heads x 10, 2336 keys 114 -> 102 us), the 128-row variant at head_dim 64 6 %.
    // At 128 that one gains 1 to 4 % at most shapes, but loses 10 % where ten row blocks share their keys (1264 rows x 4 heads
    // x 2, 1080 keys 22.4 -> 24.5), and stays with the longer way.
    auto widen = [](const u32x4& w, u32x4& lo, u32x4& hi) {
        unsigned int o[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (VAR != 1 || D == 64) {   // straight to bf16
                o[2 * i] = __builtin_bit_cast(unsigned int, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w[i], 1.f, false));
                o[2 * i + 1] = __builtin_bit_cast(unsigned int, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w[i], 1.f, true));
            } else {                               // over fp32
                const auto p01 = __builtin_amdgcn_cvt_pk_f32_fp8((int)w[i], false);     // bytes 0, 1 of the word
                const auto p23 = __builtin_amdgcn_cvt_pk_f32_fp8((int)w[i], true);      // bytes 2, 3
                o[2 * i] = (__float_as_uint(p01[0]) >> 16) | (__float_as_uint(p01[1]) & 0xffff0000u);
                o[2 * i + 1] = (__float_as_uint(p23[0]) >> 16) | (__float_as_uint(p23[1]) & 0xffff0000u);
            }
        }
        lo = u32x4{o[0], o[1], o[2], o[3]};
        hi = u32x4{o[4], o[5], o[6], o[7]};
    };
    // PIPE8: tile u has landed, this lane's pieces of it are widened into its place in the bf16 ring, and tile u + 3 is requested.
    // Every lane reads what it has asked for itself, so no barrier is needed in between.  Against the 128-row variant, which
    // widens every tile once per row block behind two barriers: 16 x 8 KV heads of 480 rows, 4096 keys +-25 % 182 -> 164 us.
    auto widen_ahead = [&](int u, int slot) {
        static_assert(!PIPE8 || CH == 1, "a piece of K and one of V per thread");
        if (u >= t1) return;
        const int ahead = t1 - 1 - u;
        if (ahead <= 0)      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        else if (ahead == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LPT) : "memory");
        else                 asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * LPT) : "memory");
        const unsigned char* const raw = (const unsigned char*)(s_raw + slot * SLOT) + tid * 16;
        unsigned short* const krow = (unsigned short*)(s_buf + slot * BUF) + kkey0 * D;
        unsigned short* const vrow = krow + TK * D;
        u32x4 lo, hi;
        widen(*(const u32x4*)raw, lo, hi);
        *(u32x4*)(krow + (((2 * pc) ^ (kkey0 & (CPR - 1))) << 3)) = lo;
        *(u32x4*)(krow + (((2 * pc + 1) ^ (kkey0 & (CPR - 1))) << 3)) = hi;
        widen(*(const u32x4*)(raw + RAW * 2), lo, hi);
        unsigned short* const vseg = vrow + ((pc ^ v_swizzle(kkey0)) << 4);
        *(u32x4*)vseg = lo;
        *(u32x4*)(vseg + 8) = hi;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // (the raw tile has been read)
        if (u + NBUF < t1) request_tile(u + NBUF, slot);
    };

    // KV8: widen the tile that has just landed in buffer `buf`, in place.  Every thread reads the sixteen-byte pieces
    // it owns (sixteen values each), the workgroup meets (the bf16 tile overwrites the bytes), the pieces are written
    // as bf16 where the operand reads expect them (K: 16-byte chunk c of row r at position c ^ (r mod 16); V: 32-byte
    // segment g at g ^ v_swizzle(r)), and the workgroup meets again.
    auto widen_tile = [&](int buf) {
        unsigned char* const rk = (unsigned char*)(s_buf + buf * BUF);
        unsigned char* const rv = rk + TK * D * 2;
        u32x4 wk[CH], wv[CH];
#pragma unroll
        for (int cc = 0; cc < CH; ++cc) {
            wk[cc] = *(const u32x4*)(rk + (cc * NT + tid) * 16);
            wv[cc] = *(const u32x4*)(rv + (cc * NT + tid) * 16);
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
        for (int cc = 0; cc < CH; ++cc) {
            const int sigma = cc * NT + tid, row = sigma / CPRG, c16 = sigma % CPRG;
            u32x4 lo, hi;
            widen(wk[cc], lo, hi);
            unsigned short* const krow = (unsigned short*)rk + row * D;
            *(u32x4*)(krow + (((2 * c16) ^ (row & (CPR - 1))) << 3)) = lo;
            *(u32x4*)(krow + (((2 * c16 + 1) ^ (row & (CPR - 1))) << 3)) = hi;
            widen(wv[cc], lo, hi);
            unsigned short* const vseg = (unsigned short*)rv + row * D + ((c16 ^ v_swizzle(row)) << 4);
            *(u32x4*)vseg = lo;
            *(u32x4*)(vseg + 8) = hi;
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    };
    if (t0 < t1) request_tile(t0, std::integral_constant<int, 0>{}); else pad_requests(0);
    if (PD > 1) { if (t0 + 1 < t1) request_tile(t0 + 1, std::integral_constant<int, (PD > 1 ? 1 : 0)>{}); else pad_requests(1); }
    if (PD > 2) { if (t0 + 2 < t1) request_tile(t0 + 2, std::integral_constant<int, (PD > 2 ? 2 : 0)>{}); else pad_requests(2); }
    // PIPE8: mask words do not travel with the tiles, whose places are taken again before they are computed: one tile ahead
    uint64_t next_word = 0;
    if (PIPE8 && max(t0, ptiles) < t1) next_word = mask_row[max(t0, ptiles) - ptiles];
    if (tid == 0 && hk == 0 && split == 0 && rb == 0) report_clamp(a.counters, L_raw, a_max_prefix);
    // Q has landed when at most the PD request groups issued behind it are outstanding (a tree tile's two mask
    // words are not counted: the wait is then on the safe side)
    wait_q<PD * LPT, SLABS>(qw);
    bf16x8 qf[SLABS];
#pragma unroll
    for (int s = 0; s < SLABS; ++s) qf[s] = __builtin_bit_cast(bf16x8, qw[s]);
    // One tile, out of buffer CUR.  In the narrow variant the buffer index is a compile-time constant (its loop is unrolled
    // NBUF times), so that every LDS address of the operand reads is a loop-invariant per-lane value plus an
    // immediate offset; a wide variant takes few tiles here.
    auto tile_step = [&](int t, auto cur_c) {
        const int CUR = cur_c;
        // buffer of tile t - 1 (= of tile t + PD); a constant again if CUR is one
        const auto PREV = [&](auto c) {
            if constexpr (std::is_same_v<decltype(c), int>) return (c + NBUF - 1) % NBUF;
            else return std::integral_constant<int, (decltype(c)::value + NBUF - 1) % NBUF>{};
        }(cur_c);
        // my requests for tile t have landed (younger ones may still be in flight); after the barrier
        // everybody's have, and everybody is done reading the buffer of tile t - 1
        // (a request group holds LPT tile loads, plus one mask word for a tree tile: allowing only
        // ahead * LPT younger loads to be outstanding is then on the safe side)
        const int ahead = t1 - 1 - t < PD - 1 ? t1 - 1 - t : PD - 1;
        const uint64_t word = next_word;
        if constexpr (PIPE8) {
            if (t >= ptiles && t + 1 < t1) next_word = mask_row[t + 1 - ptiles];
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            widen_ahead(t + 2, PREV);
        } else {
            if (ahead <= 0)      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
            else if (ahead == 1) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(LPT) : "memory");
            else                 asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(2 * LPT) : "memory");
            if (t + PD < t1) request_tile(t + PD, PREV);
            if constexpr (KV8) widen_tile(CUR);
        }

        const unsigned short* const s_k = (const unsigned short*)(s_buf + CUR * BUF);
        const unsigned short* const s_v = s_k + TK * D;

        const bool tree = t >= ptiles;
        const int key0 = tree ? (t - ptiles) * TK : t * TK;
        const int kend = tree ? a_nk : L;
        // visibility of the tile's 64 keys for this lane's query: keys that exist (a uniform bit run), and on
        // tree tiles the row's ancestor bits
        const bool masked = tree || key0 + TK > kend;
        uint64_t vis = kend - key0 >= TK ? ~0ull : ((1ull << (kend - key0)) - 1ull);
        if (tree && PIPE8) vis &= word;
        else if (tree) vis &= (uint64_t)s_mw[(CUR * NWAVES + wave) * 128 + lane] | ((uint64_t)s_mw[(CUR * NWAVES + wave) * 128 + 64 + lane] << 32);

        // one 32-key block at a time: S^T = K Q^T, online softmax, O^T += V^T P^T
#pragma unroll
        for (int j = 0; j < NKB; ++j) {
            const int kbi = WIDE ? j : kh;
            f32x16 sacc;
            u32x4 kfr[SLABS];
#pragma unroll
            for (int v = 0; v < 16; ++v) sacc[v] = 0.f;
#pragma unroll
            for (int s = 0; s < SLABS; ++s) kfr[s] = *(const u32x4*)(s_k + (32 * kbi + l32) * D + (((2 * s) ^ kx) << 3));
#pragma unroll
            for (int s = 0; s < SLABS; ++s)
                sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kfr[s]), qf[s], sacc, 0, 0, 0);
            // visibility; accumulator element v is key 32 kbi + 8 (v/4) + 4 h + v%4
            if (masked) {
                const unsigned int vw32 = (unsigned int)(kbi ? (vis >> 32) : vis) >> (4 * h);
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    // all ones if bit 8 (v/4) + v%4 is set, else zero; the score or -inf, chosen bit by bit
                    const unsigned int keep = (unsigned int)__builtin_amdgcn_sbfe((int)vw32, 8 * (v >> 2) + (v & 3), 1);
                    sacc[v] = __uint_as_float((__float_as_uint(sacc[v]) & keep) | (0xff800000u & ~keep));
                }
            }
            float tmax = sacc[0];
#pragma unroll
            for (int v = 1; v < 16; ++v) tmax = fmaxf(tmax, sacc[v]);
            tmax = xhalf_max(tmax);
            const float ref_new = fmaxf(ref, tmax * c);
            bf16x8 pf[2];
            if (ref_new == -INFINITY) {
#pragma unroll
                for (int v = 0; v < 16; ++v) pf[v >> 3][v & 7] = (__bf16)0.f;
            } else {
                const float alpha = __builtin_amdgcn_exp2f(ref - ref_new);            // ref = -inf gives 0
                float psum = 0.f;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float p = __builtin_amdgcn_exp2f(fmaf(sacc[v], c, -ref_new));
                    psum += p;
                    pf[v >> 3][v & 7] = (__bf16)p;
                }
                l_run = l_run * alpha + psum;
                ref = ref_new;
                if (__any(alpha != 1.f)) {       // the running maximum rarely moves after the first tiles
#pragma unroll
                    for (int d = 0; d < DB; ++d)
#pragma unroll
                        for (int v = 0; v < 16; ++v) oacc[d][v] *= alpha;
                }
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
#pragma unroll
                for (int d = 0; d < DB; ++d) {
                    // this lane needs column 32d+l32 of keys 32kbi+16u+4h+{0..3} and of the same +8.
                    // Transpose load: lanes 4j..4j+3 of a 16-lane group address the 32-byte segment
                    // [key j][16 columns]; lane i of the group receives column i of the 4 keys.
                    const unsigned short* seg = s_v + (32 * kbi + 16 * u + 4 * h + tr_j) * D + (((2 * d) ^ vx) << 4) + tr_q;
                    const s16x4 lo4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)seg);
                    const s16x4 hi4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(seg + 8 * D));
                    const s16x8 vw = __builtin_shufflevector(lo4, hi4, 0, 1, 2, 3, 4, 5, 6, 7);
                    oacc[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vw), pf[u], oacc[d], 0, 0, 0);
                }
            }
        }
    };
    int t_done = t0;           // tiles [t0, t_done) are consumed
    if constexpr (PIPE8) {                                     // the first two tiles, widened
        widen_ahead(t0, 0);
        widen_ahead(t0 + 1, 1);
    }
    if constexpr (VAR == 2) {
        // ---- fast loop of the 256-row variant over full prefix tiles: what the MFMA-bound shapes spend their time in.
        // The softmax reference of a row stays FIXED while no probability of a 32-key block comes out too large: p =
        // 2^(c s - ref) may exceed one, which fp32 sums and bf16 operands take in their stride, and O is never rescaled
        // inside the loop.  The loop is pipelined by 32-key blocks: in the phase of block j the matrix pipe forms S of
        // block j + 1 and adds P V of block j - 1 while the vector ALU takes the exponentials of block j, so that nothing
        // in a phase waits for anything of the same phase, and each matrix instruction has its share of the vector work
        // and of the operand reads beside it.  Operands of the next phase are read into a register as soon as its
        // instruction has been issued (half of a K block and a whole V block ahead), so tile t + 1 has to be there when
        // tile t begins.
        // Probabilities beyond the limit (every row's first block, then rarely) leave the loop before they are added: the
        // reference, O and l move up out here.
        // Measured (MI355X, the 128-row variant's loop, in which half of the matrix instructions had no vector work beside
        // them, before): 32 sequences x 8 KV heads of 1024 rows, 8448 keys of 128 1125 -> 1070 us (1.06 PFLOP/s); 16 x 8 of
        // 480 rows, 4156 keys 152 -> 137; 7 x 8 of 512 rows, 6428 keys 118 -> 105; 8 x 8 of 480 rows, 6060 keys of 64 79 -> 68;
        // 2 x 8 of 164 rows, 595 keys 21.0 -> 19.2.  Now a SIMD's two wavefronts need 2048 matrix cycles per tile (the
        // pipe is busy 52 % of the time), the operand reads of all eight 1030 cycles of the LDS (SQ_LDS_IDX_ACTIVE: 256 bytes a
        // cycle), which are not what bounds: 64 rows per wavefront, one wavefront per SIMD, halve them, and take 1139 us and 229
        // against 224 for a step of the 16 x 8 batch, since a wavefront by itself issues vector and matrix instructions one behind
        // the other.
        // Requests of the next tile spread over a phase instead of in one piece: 1051 us, but 140 at 16 x 8.
        constexpr int NS = SLABS, NP = 2 * DB, KR = NS / 2;     // instructions per phase for S, for P V; K operands ahead
        static_assert(NS == NP, "one P V instruction for each one of S");
        constexpr float kSumLimit = 16.f * 4096.f;              // of the sixteen probabilities of a lane
        const int t_full = min(t1, L / TK);                      // tiles below t_full are full prefix tiles
        // tile t + 1 has landed for this lane when only the requests of tile t + 2 are outstanding; after the barrier it has
        // for everybody, and everybody is done with tile t - 1, into whose buffer tile t + 3 goes
        // (PIPE8: tile t + 1 has been widened by everybody, and tile t + 2 is widened into the place of tile t - 1)
        int at = 0, at1 = 1;                                     // places of tiles t and t + 1 in the ring
        auto following = [](int at) { return at + 1 == NBUF ? 0 : at + 1; };
        auto stage = [&](int t) {
            if constexpr (PIPE8) {
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                widen_ahead(t + 2, following(at1));
                return;
            }
            if (t + 2 < t1) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(LPT) : "memory");
            else            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
            if (t + PD < t1) request_tile(t + PD, at == 0 ? NBUF - 1 : at - 1);
        };
        // LDS addresses of the operands, moved from tile to tile: K of tile t + 1, what is still to be read of K of tile t, V
        // of tile t; block 1 is at a fixed distance
        typedef const u32x4 __attribute__((address_space(3))) * lds_u32x4;
        typedef s16x4 __attribute__((address_space(3))) * lds_s16x4;
        const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) void*)s_buf;
        unsigned ka[NS], kc[NS - KR], va[DB];
#pragma unroll
        for (int s = 0; s < NS; ++s) ka[s] = lds0 + 2 * (l32 * D + (((2 * s) ^ kx) << 3));
#pragma unroll
        for (int d = 0; d < DB; ++d) va[d] = lds0 + 2 * (TK * D + (4 * h + tr_j) * D + (((2 * d) ^ vx) << 4) + tr_q);
        auto kfrag = [&](unsigned a, int kb) { return __builtin_bit_cast(bf16x8, *(lds_u32x4)(a + 2 * 32 * D * kb)); };
        auto vfrag = [&](int kb, int i) {
            // slab u, d block d: column 32d+l32 of keys 32kb+16u+4h+{0..3} and of the same +8 (transpose loads, see tile_step)
            const unsigned a = va[i % DB] + 2 * (32 * kb + 16 * (i / DB)) * D;
            const s16x4 lo4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)a);
            const s16x4 hi4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(a + 2 * 8 * D));
            return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo4, hi4, 0, 1, 2, 3, 4, 5, 6, 7));
        };
        auto row_max = [&](const f32x16& x) {                   // eight three-input maxima
            float m = fmaxf(fmaxf(x[0], x[1]), x[2]);
#pragma unroll
            for (int v = 3; v < 15; v += 2) m = fmaxf(fmaxf(m, x[v]), x[v + 1]);
            return xhalf_max(fmaxf(m, x[15]));
        };
        auto mma = [](const bf16x8& x, const bf16x8& y, f32x16& acc) { acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, y, acc, 0, 0, 0); };
        if (t0 < t_full) {
            bf16x8 kf[KR], vf[NP];
            u32x4 p0[2], p1[2];
            f32x16 s0, s1;
            // -ref by itself: with the sign as an operand modifier of the loop's multiply-adds 25 x 1 KV heads of 800 rows, 30000 keys of
            // 64 take 281 us instead of 274, 3 x 30 of 256 rows, 6000 keys 69.4 instead of 67.6
            float nref = 0.f;
            int t = t0;
            // reference, O and l move up to what block `s` needs
            auto move_up = [&](const f32x16& s) {
                const float ref_new = fmaxf(fmaxf(ref, row_max(s) * c), kNoRef);
                const float alpha = __builtin_amdgcn_exp2f(ref - ref_new);            // ref = -inf gives 0
                l_run *= alpha;
#pragma unroll
                for (int d = 0; d < DB; ++d)
#pragma unroll
                    for (int v = 0; v < 16; ++v) oacc[d][v] *= alpha;
                ref = ref_new;
                nref = -ref_new;
                asm volatile("" : "+v"(nref));
            };
            // a pair of probabilities, rounded to the MFMA's operand type, and their sum taken from the rounded pair (l then
            // matches what P V multiplies by)
            auto pair = [](float p, float q, float& sum) -> unsigned int {
                const bf16x2 pr = {(__bf16)p, (__bf16)q}, ones = {(__bf16)1.f, (__bf16)1.f};
                sum = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, sum, false);
                return __builtin_bit_cast(unsigned int, pr);
            };
            // One phase, block B of tile t: next = S of the block behind it, whose first KR operands are in kf; O += P V of the
            // block ahead of it, whose V operands are in vf; pc = 2^(c cur + nref).  Returns this lane's sum of pc.
            auto phase = [&](auto block_c, const f32x16& cur, f32x16& next, const u32x4 (&pp)[2], u32x4 (&pc)[2]) {
                constexpr int B = decltype(block_c)::value;
                __builtin_amdgcn_sched_barrier(0);
                float psum = 0.f;
                f32x16 acc;
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
                for (int i = 0; i < NS; ++i) {
                    mma(kf[i % KR], qf[i], acc);
                    kf[i % KR] = i < NS - KR ? (B ? kfrag(ka[i + KR], 0) : kfrag(kc[i], 1)) : kfrag(ka[i + KR - NS], B);
                    mma(vf[i], __builtin_bit_cast(bf16x8, pp[i / DB]), oacc[i % DB]);
                    vf[i] = vfrag(B, i);
                }
#pragma unroll
                for (int v = 0; v < 16; v += 2)
                    pc[v >> 3][(v & 7) >> 1] = pair(__builtin_amdgcn_exp2f(fmaf(cur[v], c, nref)), __builtin_amdgcn_exp2f(fmaf(cur[v + 1], c, nref)), psum);
                next = acc;
#pragma unroll
                for (int i = 0; i < NS; ++i) {                   // a matrix instruction, its share of the reads, its share of the rest
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 24 / NS, 0);
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 24 / NS, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
                return psum;
            };
            auto phase_a = [&]() { return phase(std::integral_constant<int, 0>{}, s0, s1, p1, p0); };
            auto phase_b = [&]() { return phase(std::integral_constant<int, 1>{}, s1, s0, p0, p1); };
            // behind phase B of tile t - 1: tile t
            auto next_tile = [&](int t) {
                at = at1;
                at1 = following(at);
                stage(t);
#pragma unroll
                for (int s = KR; s < NS; ++s) kc[s - KR] = ka[s];
#pragma unroll
                for (int s = 0; s < NS; ++s) ka[s] += at1 ? BUF * 4 : -(NBUF - 1) * BUF * 4;
#pragma unroll
                for (int d = 0; d < DB; ++d) va[d] += at ? BUF * 4 : -(NBUF - 1) * BUF * 4;
            };
            auto add_pv = [&]() {                    // P V of the block whose P is in p1 and whose V operands are in vf
#pragma unroll
                for (int i = 0; i < NP; ++i) mma(vf[i], __builtin_bit_cast(bf16x8, p1[i / DB]), oacc[i % DB]);
            };
            // S of the first block; its tile has landed when only the requests of the two behind it are outstanding
            if constexpr (PIPE8)  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            else if (t0 + 2 < t1) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(2 * LPT) : "memory");
            else if (t0 + 1 < t1) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(LPT) : "memory");
            else                  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
            for (int v = 0; v < 16; ++v) s0[v] = 0.f;
#pragma unroll
            for (int s = 0; s < NS; ++s) mma(kfrag(ka[s], 0), qf[s], s0);
            stage(t0);
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                if (s >= KR) kc[s - KR] = ka[s];
                ka[s] += BUF * 4;
            }
            // no block ahead: P and V of it are zero (V too, where zero times an infinity would not be)
            const u32x4 zero = {0u, 0u, 0u, 0u};
            auto no_v = [&]() {
#pragma unroll
                for (int i = 0; i < NP; ++i) vf[i] = __builtin_bit_cast(bf16x8, zero);
            };
            int moved = -1;                          // tile whose block 0 has set the reference: taken as it is (see below)
            while (t < t_full) {
                move_up(s0);
                moved = t;
                p1[0] = p1[1] = zero;
                no_v();
#pragma unroll
                for (int s = 0; s < KR; ++s) kf[s] = kfrag(ka[s] - (at1 ? BUF * 4 : -(NBUF - 1) * BUF * 4), 1);
                bool in_b = false;
                for (;;) {
                    float psum = phase_a();
                    asm volatile("" : "+s"(moved));     // (keeps the first tile of an entry from becoming a second loop body)
                    const uint64_t over = __ballot(psum > kSumLimit);      // (one test: each branch taken between the phases shows at 64)
                    if ((t == moved ? 0ull : over) != 0ull) break;
                    l_run += psum;
                    psum = phase_b();
                    if (__any(psum > kSumLimit)) { in_b = true; break; }
                    l_run += psum;
                    if (++t >= t_full) break;
                    next_tile(t);
                }
                if (in_b) {                          // P V of block 0 has been added; block 1 by itself
                    move_up(s1);
                    p0[0] = p0[1] = zero;
                    no_v();
#pragma unroll
                    for (int s = 0; s < KR; ++s) kf[s] = kfrag(ka[s], 0);
                    l_run += phase_b();
                    add_pv();
                    p1[0] = p1[1] = zero;
                    no_v();
                    if (++t < t_full) next_tile(t);
                }
            }
            add_pv();                                // the last block's, unless it has been added
            t_done = t_full;
        }
        for (int tt = t_done; tt < t1; ++tt) tile_step(tt, (tt - t0) % NBUF);       // the prefix tail and the tree tiles
    } else
    if constexpr (WIDE) {
        // ---- fast loop of the 128-row variant over full prefix tiles: what the MFMA-bound shapes spend their time in.
        // The softmax reference of a row stays FIXED while scores do not exceed it by more than kSlack (in units
        // of log2 e / scale): p = 2^(c s - ref) may then exceed one, which fp32 sums and bf16 operands take in
        // their stride, and O is never rescaled inside the loop -- the accumulators stay in their registers, the
        // loop body has no data-dependent path, and the two 32-key blocks of a tile are skewed against each other
        // so that the matrix pipe and the vector ALU work at the same time inside one wavefront (S of block 1
        // while the exponentials of block 0 are taken, P V of block 0 while those of block 1 are).  A score beyond
        // the slack (every row's first tile, then rarely) leaves the loop before anything of the tile is added;
        // the reference moves up, O and l are rescaled out here, and the loop is entered again at the same tile, which is then
        // taken as it is: nothing of it exceeds the new reference, but c s - ref of huge scores (1e9) may round past the
        // slack, again and again.
        constexpr float kSlack = 12.f;
        constexpr float kSumLimit = 16.f * 4096.f;          // sixteen terms of at most 2^kSlack
        static_assert(NBUF == 2, "the buffer of a tile is (t - t0) mod 2");
        // tile t has landed for this lane when only the requests of the tiles behind it are outstanding; after the
        // barrier it has for everybody, and everybody is done with the buffer that tile t + PD goes into
        auto stage_tile = [&](int t) {
            const int ahead = t1 - 1 - t < PD - 1 ? t1 - 1 - t : PD - 1;
            if (ahead <= 0)      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
            else if (ahead == 1) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(LPT) : "memory");
            else                 asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(2 * LPT) : "memory");
            if (t + PD < t1) request_tile(t + PD, (t + PD - t0) & (NBUF - 1));
            if constexpr (KV8) widen_tile((t - t0) & (NBUF - 1));
        };
        const int t_full = min(t1, L / TK);                      // tiles below t_full are full prefix tiles
        auto kfrag = [&](const unsigned short* s_k, int kb, int s) {
            return *(const u32x4*)(s_k + (32 * kb + l32) * D + (((2 * s) ^ kx) << 3));
        };
        auto vfrag = [&](const unsigned short* s_v, int kb, int u, int d) {
            // column 32d+l32 of keys 32kb+16u+4h+{0..3} and of the same +8 (transpose loads, see tile_step)
            const unsigned short* seg = s_v + (32 * kb + 16 * u + 4 * h + tr_j) * D + (((2 * d) ^ vx) << 4) + tr_q;
            const s16x4 lo4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)seg);
            const s16x4 hi4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(seg + 8 * D));
            return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo4, hi4, 0, 1, 2, 3, 4, 5, 6, 7));
        };
        auto row_max = [&](const f32x16& x) {                   // eight three-input maxima
            float m = fmaxf(fmaxf(x[0], x[1]), x[2]);
#pragma unroll
            for (int v = 3; v < 15; v += 2) m = fmaxf(fmaxf(m, x[v]), x[v + 1]);
            return xhalf_max(fmaxf(m, x[15]));
        };
        int t = t0;
        bool staged = false;                                      // tile t has been awaited and published
        float seen = -INFINITY;                                   // largest score of the tile that left the loop
        float m_run = -INFINITY;                                  // largest score that the reference was moved up for
        int moved = -1;                                           // tile that the reference was last moved up for
        while (t < t_full) {
            if (!staged) {
                stage_tile(t);
                staged = true;
            }
            {   // move the reference up to what tile t needs; O and l follow
                const unsigned short* const s_k = (const unsigned short*)(s_buf + ((t - t0) & (NBUF - 1)) * BUF);
                f32x16 sa, sb;
#pragma unroll
                for (int v = 0; v < 16; ++v) { sa[v] = 0.f; sb[v] = 0.f; }
#pragma unroll
                for (int s = 0; s < SLABS; ++s) {
                    sa = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kfrag(s_k, 0, s)), qf[s], sa, 0, 0, 0);
                    sb = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kfrag(s_k, 1, s)), qf[s], sb, 0, 0, 0);
                }
                m_run = fmaxf(m_run, fmaxf(row_max(sa), row_max(sb)));
                const float ref_new = fmaxf(fmaxf(ref, m_run * c), kNoRef);           // (the maximum keeps the product rounded)
                const float alpha = __builtin_amdgcn_exp2f(ref - ref_new);            // ref = -inf gives 0
                l_run *= alpha;
#pragma unroll
                for (int d = 0; d < DB; ++d)
#pragma unroll
                    for (int v = 0; v < 16; ++v) oacc[d][v] *= alpha;
                ref = ref_new;
            }
            moved = t;
            const float limit = m_run + kSlack / c;
            for (;;) {
                if (!staged) stage_tile(t);
                staged = true;
                const unsigned short* const s_k = (const unsigned short*)(s_buf + ((t - t0) & (NBUF - 1)) * BUF);
                const unsigned short* const s_v = s_k + TK * D;
                u32x4 kf[SLABS];
                bf16x8 va[2][DB], vb[2][DB];       // V operands of block 0 and of block 1
                f32x16 s0, s1;
#pragma unroll
                for (int s = 0; s < SLABS; ++s) kf[s] = kfrag(s_k, 0, s);
#pragma unroll
                for (int v = 0; v < 16; ++v) { s0[v] = 0.f; s1[v] = 0.f; }
#pragma unroll
                for (int s = 0; s < SLABS; ++s)
                    s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kf[s]), qf[s], s0, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int s = 0; s < SLABS; ++s) kf[s] = kfrag(s_k, 1, s);
                __builtin_amdgcn_sched_barrier(0);
                // S of block 1 in the matrix pipe, the exponentials of block 0 in the vector ALU, the V operands of
                // block 0 on their way.  One matrix instruction, then its share of the rest: the wavefront issues in
                // order, and a run of dependent MFMAs would otherwise hold everything else back until the last one.
#pragma unroll
                for (int s = 0; s < SLABS; ++s)
                    s1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kf[s]), qf[s], s1, 0, 0, 0);
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int d = 0; d < DB; ++d) va[u][d] = vfrag(s_v, 0, u, d);
                bf16x8 p0[2], p1[2];
                float psum = 0.f;
                const bf16x2 ones2 = {(__bf16)1.f, (__bf16)1.f};
#pragma unroll
                for (int v = 0; v < 16; v += 2) {
                    // a pair of probabilities, rounded to the MFMA's operand type, and their sum taken from the
                    // rounded pair with one dot-product instruction (l then matches what P V multiplies by)
                    const bf16x2 pr = {(__bf16)__builtin_amdgcn_exp2f(fmaf(s0[v], c, -ref)),
                                       (__bf16)__builtin_amdgcn_exp2f(fmaf(s0[v + 1], c, -ref))};
                    psum = __builtin_amdgcn_fdot2_f32_bf16(pr, ones2, psum, false);
                    p0[v >> 3][v & 7] = pr[0];
                    p0[v >> 3][(v & 7) + 1] = pr[1];
                }
                // (the empty statement is a use of P here: the compiler would otherwise move the exponentials behind
                // the test below, out of the shadow of the matrix instructions)
                asm volatile("" ::"v"(p0[0]), "v"(p0[1]), "v"(psum));
#pragma unroll
                for (int i = 0; i < SLABS; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, 4 * DB / SLABS, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 48 / SLABS, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
                seen = row_max(s1);
                // block 0 is tested on what its exponentials came to instead of on its scores: a probability beyond
                // 2^kSlack shows in the lane's sum (all terms are positive; an overflow gives +inf), which is there
                // anyway, while the maximum of sixteen scores costs a dozen instructions.  Nothing of the tile has
                // been added yet.  The bound is on the sum of sixteen terms, so single terms up to 2^kSlack pass
                // as before and a few somewhat larger ones may: the formats have the room.
                asm volatile("" : "+s"(moved));                   // (keeps the first tile of an entry from becoming a second loop body)
                if (t != moved && __any(seen > limit || psum > kSumLimit)) break;
                __builtin_amdgcn_sched_barrier(0);
                // P V of block 0 in the matrix pipe, the exponentials of block 1 in the vector ALU, the V operands of
                // block 1 on their way
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int d = 0; d < DB; ++d) oacc[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[u][d], p0[u], oacc[d], 0, 0, 0);
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int d = 0; d < DB; ++d) vb[u][d] = vfrag(s_v, 1, u, d);
#pragma unroll
                for (int v = 0; v < 16; v += 2) {
                    // a pair of probabilities, rounded to the MFMA's operand type, and their sum taken from the
                    // rounded pair with one dot-product instruction (l then matches what P V multiplies by)
                    const bf16x2 pr = {(__bf16)__builtin_amdgcn_exp2f(fmaf(s1[v], c, -ref)),
                                       (__bf16)__builtin_amdgcn_exp2f(fmaf(s1[v + 1], c, -ref))};
                    psum = __builtin_amdgcn_fdot2_f32_bf16(pr, ones2, psum, false);
                    p1[v >> 3][v & 7] = pr[0];
                    p1[v >> 3][(v & 7) + 1] = pr[1];
                }
#pragma unroll
                for (int i = 0; i < 2 * DB; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 48 / (2 * DB), 0);
                }
                __builtin_amdgcn_sched_barrier(0);
                l_run += psum;
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int d = 0; d < DB; ++d) oacc[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vb[u][d], p1[u], oacc[d], 0, 0, 0);
                staged = false;
                if (++t >= t_full) break;
            }
        }
        (void)seen;
        t_done = t;
        // the remaining tiles (the prefix tail and the tree tiles) take the general path, whose buffer index is a
        // compile-time constant: tile t sits in buffer (t - t0) mod NBUF
        for (int tt = t_done; tt < t1; ++tt) {
            if (((tt - t0) & 1) == 0) tile_step(tt, std::integral_constant<int, 0>{});
            else                      tile_step(tt, std::integral_constant<int, 1>{});
        }
    } else {
        static_assert(NBUF == 2 || NBUF == 3, "unrolled so");
        for (int t = t0; t < t1; t += NBUF) {
            tile_step(t, std::integral_constant<int, 0>{});
            if (t + 1 < t1) tile_step(t + 1, std::integral_constant<int, 1>{});
            if (NBUF > 2 && t + 2 < t1) tile_step(t + 2, std::integral_constant<int, (NBUF > 2 ? 2 : 0)>{});
        }
    }
    (void)t_done;

    l_run = xhalf_sum(l_run);
    if (!WIDE) {
        // merge the two key-half waves of each query block through LDS (all tiles are consumed)
        float* s_merge = (float*)s_buf;          // [2 qb][64 lanes][MST]
        float* mine = s_merge + (qb * 64 + lane) * MST;
        __syncthreads();
        if (kh == 1) {
#pragma unroll
            for (int d = 0; d < DB; ++d)
#pragma unroll
                for (int v4 = 0; v4 < 4; ++v4)
                    *(f32x4*)(mine + d * 16 + 4 * v4) =
                        f32x4{oacc[d][4 * v4], oacc[d][4 * v4 + 1], oacc[d][4 * v4 + 2], oacc[d][4 * v4 + 3]};
            *(f32x4*)(mine + DB * 16) = f32x4{ref, l_run, 0.f, 0.f};
        }
        __syncthreads();
        if (kh == 0) {
            const f32x4 ml2 = *(const f32x4*)(mine + DB * 16);
            const float ref2 = ml2.x, l2 = ml2.y;
            const float top = fmaxf(ref, ref2);
            float a1 = 0.f, a2 = 0.f;
            if (top != -INFINITY) {
                a1 = __builtin_amdgcn_exp2f(ref - top);
                a2 = __builtin_amdgcn_exp2f(ref2 - top);
            }
            l_run = l_run * a1 + l2 * a2;
            ref = top;
#pragma unroll
            for (int d = 0; d < DB; ++d)
#pragma unroll
                for (int v4 = 0; v4 < 4; ++v4) {
                    const f32x4 o2 = *(const f32x4*)(mine + d * 16 + 4 * v4);
                    oacc[d][4 * v4] = oacc[d][4 * v4] * a1 + o2.x * a2;
                    oacc[d][4 * v4 + 1] = oacc[d][4 * v4 + 1] * a1 + o2.y * a2;
                    oacc[d][4 * v4 + 2] = oacc[d][4 * v4 + 2] * a1 + o2.z * a2;
                    oacc[d][4 * v4 + 3] = oacc[d][4 * v4 + 3] * a1 + o2.w * a2;
                }
        }
    }
    const bool holder = WIDE || kh == 0;         // this wavefront holds finished (O, ref, l) of its 32 rows

    if (a_splits == 1) {
        if (holder && row_ok) {
            const float inv = l_run > 0.f ? v_factor / l_run : 0.f;
            unsigned short* orow =
                (unsigned short*)a.O + (long long)b * a.os[0] + (long long)hq * a.os[1] + (long long)node * a.os[2];
#pragma unroll
            for (int d = 0; d < DB; ++d)
#pragma unroll
                for (int v4 = 0; v4 < 4; ++v4) {
                    unsigned short o4[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        o4[e] = __builtin_bit_cast(unsigned short, (__bf16)(oacc[d][v4 * 4 + e] * inv));
                    uint2 pk;
                    pk.x = (unsigned)o4[0] | ((unsigned)o4[1] << 16);
                    pk.y = (unsigned)o4[2] | ((unsigned)o4[3] << 16);
                    *(uint2*)(orow + 32 * d + 8 * v4 + 4 * h) = pk;
                }
        }
        return;
    }

    // ---- several splits: leave the partial, take a ticket, the last one merges ----
    // Partials travel between workgroups (on different XCDs, each with its own L2) through device-scope
    // atomic stores and loads, which write through / read around the caches; a device-scope fence would
    // instead write back and invalidate the whole L2 once per workgroup.  Order: every wavefront waits
    // until its stores have completed (vmcnt), the workgroup meets at a barrier, then one thread takes the
    // ticket; the workgroup that sees the last ticket therefore reads completed partials only.
    // Only the live rows of a query block travel (a block holds live = min(32, g n - first row) of them):
    // part_o  [group][split][query block][e][64] x 8 bytes; e = (d block, group of four accumulator values as bf16)
    //         -- or (d block, pair of floats) when the exchange is fp32 -- and the live lanes of the two half-waves
    //         packed at the front of each 64-slot line (slot h live + l32): every store and load instruction touches
    //         one contiguous run, and nothing is moved for rows that do not exist
    // part_ml [group][split][query block][row] (ref, l) as two floats
    typedef unsigned long long u64;
    // EPS 64-bit elements per (lane, d block): pairs of floats, or with bf16 partials groups of four values
    constexpr int EPS = OT_ATTN_PART_BF16 ? 4 : 8;
    auto pack2 = [](float x, float y) -> u64 { return (u64)__float_as_uint(x) | ((u64)__float_as_uint(y) << 32); };
    auto pack4 = [](float x, float y, float z, float w) -> u64 {
        const bf16x2 lo = {(__bf16)x, (__bf16)y}, hi = {(__bf16)z, (__bf16)w};
        return (u64)__builtin_bit_cast(unsigned int, lo) | ((u64)__builtin_bit_cast(unsigned int, hi) << 32);
    };
    const int group = bz * a_row_blocks + rb;
    const int rows_all = a_g * n;
    if (holder && row_ok) {
        const int live = min(32, rows_all - (rb * ROWS + qb * 32));
        u64* po = (u64*)a.part_o + (((size_t)group * a_splits + split) * NQB + qb) * (DB * EPS * 64) + h * live + l32;
#pragma unroll
        for (int d = 0; d < DB; ++d)
#pragma unroll
            for (int e = 0; e < EPS; ++e) {
                const u64 w = OT_ATTN_PART_BF16
                                  ? pack4(oacc[d][4 * e % 16], oacc[d][(4 * e + 1) % 16], oacc[d][(4 * e + 2) % 16], oacc[d][(4 * e + 3) % 16])
                                  : pack2(oacc[d][2 * e], oacc[d][2 * e + 1]);
                __hip_atomic_store(po + (d * EPS + e) * 64, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        if (h == 0)                                                  // lanes l and l + 32 hold the same row
            __hip_atomic_store((u64*)a.part_ml + (((size_t)group * a_splits + split) * NQB + qb) * 32 + l32,
                               pack2(ref, l_run), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0)
        s_last = __hip_atomic_fetch_add(a.counters + group, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                         (unsigned)(a_splits - 1) ? 1 : 0;
    __syncthreads();
    if (!s_last) return;
    if (tid == 0) __hip_atomic_store(a.counters + group, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // for the next launch

    // merge: thread = (query block cq, lane) x DC of the DB d blocks, same register order as above
    constexpr int DC = WIDE ? DB : DB / 2;
    const int cq = WIDE ? wave : (wave & 1);
    const int d0 = WIDE ? 0 : (wave >> 1) * DC;
    const int rho2 = rb * ROWS + cq * 32 + l32;
    if (rho2 >= rows_all) return;                      // no row behind this lane (no barrier follows)
    const int live2 = min(32, rows_all - (rb * ROWS + cq * 32));
    // CHUNK splits at a time: all their loads are issued before the first one is used (each is a trip to
    // memory), and the running maximum M is carried from chunk to chunk like in the main loop.
    constexpr int CHUNK = merge_chunk(D, WIDE);
    static_assert(CHUNK * DC * EPS * 2 <= 96, "register budget");
    const u64* mlp = (const u64*)a.part_ml + ((size_t)group * a_splits * NQB + cq) * 32 + l32;
    const u64* pp = (const u64*)a.part_o + ((size_t)group * a_splits * NQB + cq) * (DB * EPS * 64) + d0 * EPS * 64 +
                    h * live2 + l32;
    float M = -INFINITY, Ls = 0.f;
    f32x16 acc[DC];
#pragma unroll
    for (int d = 0; d < DC; ++d)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[d][v] = 0.f;
    for (int s0 = 0; s0 < a_splits; s0 += CHUNK) {
        u64 ml[CHUNK], x[CHUNK][DC * EPS];
#pragma unroll
        for (int i = 0; i < CHUNK; ++i) {
            const int si = s0 + i < a_splits ? s0 + i : a_splits - 1;      // past the end: a copy, weight 0
            ml[i] = __hip_atomic_load(mlp + (size_t)si * NQB * 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
#pragma unroll
        for (int i = 0; i < CHUNK; ++i) {
            const int si = s0 + i < a_splits ? s0 + i : a_splits - 1;
            const u64* ps = pp + (size_t)si * NQB * (DB * EPS * 64);
#pragma unroll
            for (int e = 0; e < DC * EPS; ++e)
                x[i][e] = __hip_atomic_load(ps + e * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        float mi[CHUNK], m_new = M;
#pragma unroll
        for (int i = 0; i < CHUNK; ++i) {
            mi[i] = s0 + i < a_splits ? __uint_as_float((unsigned)ml[i]) : -INFINITY;
            m_new = fmaxf(m_new, mi[i]);
        }
        if (m_new == -INFINITY) continue;                                    // nothing visible so far
        const float alpha = __builtin_amdgcn_exp2f(M - m_new);                // M = -inf gives 0
        Ls *= alpha;
#pragma unroll
        for (int d = 0; d < DC; ++d)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[d][v] *= alpha;
#pragma unroll
        for (int i = 0; i < CHUNK; ++i) {
            const float w = mi[i] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mi[i] - m_new);
            Ls = fmaf(w, __uint_as_float((unsigned)(ml[i] >> 32)), Ls);
#pragma unroll
            for (int e = 0; e < DC * EPS; ++e) {
                const unsigned int lo = (unsigned)x[i][e], hi = (unsigned)(x[i][e] >> 32);
                if (OT_ATTN_PART_BF16) {
                    const int dd = e / EPS, v0 = 4 * (e % EPS);
                    acc[dd][v0] = fmaf(w, __uint_as_float(lo << 16), acc[dd][v0]);
                    acc[dd][v0 + 1] = fmaf(w, __uint_as_float(lo & 0xffff0000u), acc[dd][v0 + 1]);
                    acc[dd][v0 + 2] = fmaf(w, __uint_as_float(hi << 16), acc[dd][v0 + 2]);
                    acc[dd][v0 + 3] = fmaf(w, __uint_as_float(hi & 0xffff0000u), acc[dd][v0 + 3]);
                } else {
                    acc[e >> 3][2 * (e & 7)] = fmaf(w, __uint_as_float(lo), acc[e >> 3][2 * (e & 7)]);
                    acc[e >> 3][2 * (e & 7) + 1] = fmaf(w, __uint_as_float(hi), acc[e >> 3][2 * (e & 7) + 1]);
                }
            }
        }
        M = m_new;
    }
    {
        const int head2 = fast_div(rho2, n, a_inv_n);
        const int hq2 = hk * a_g + head2, node2 = rho2 - head2 * n;
        const float inv = Ls > 0.f ? v_factor / Ls : 0.f;
        unsigned short* orow =
            (unsigned short*)a.O + (long long)b * a.os[0] + (long long)hq2 * a.os[1] + (long long)node2 * a.os[2];
#pragma unroll
        for (int d = 0; d < DC; ++d)
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
                unsigned short o4[4];
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    o4[e] = __builtin_bit_cast(unsigned short, (__bf16)(acc[d][v4 * 4 + e] * inv));
                uint2 pk;
                pk.x = (unsigned)o4[0] | ((unsigned)o4[1] << 16);
                pk.y = (unsigned)o4[2] | ((unsigned)o4[3] << 16);
                *(uint2*)(orow + 32 * (d0 + d) + 8 * v4 + 4 * h) = pk;
            }
    }
}

// ---------------------------------------------------------------------------
// f32 kernel: fp32 matrix instructions throughout
// ---------------------------------------------------------------------------
// What bounds it: v_mfma_f32_32x32x2_f32 does 64 flop per cycle and SIMD, a sixteenth of the bf16 rate, so 32 query rows
// against 32 keys keep a SIMD busy for 8192 cycles (head_dim 128) over 32 KB of K/V: operands can come straight from
// memory into registers, one block ahead of their use, with no staging in LDS and no barrier in the loop.
//
// A wavefront takes 32 packed query rows (GQA: the rows of the heads that share a KV head are stacked, as in the bf16
// kernel) and every KS-th 32-key block of its workgroup's range; a workgroup is eight wavefronts = QB row blocks x KS key
// slices, whose results meet in LDS at the end.
//   S^T = K Q^T  A = K: lane (key l32, half h) holds K[key][8 j + 4 h + i], i = 0..3 -- one 16-byte load serves four
//                instructions (the order of the contraction is free); B = Q in the same order, from LDS
//   O^T += V^T P^T  B = register v of the accumulator: keys 8 (v/4) + 4 h + v%4 of the block, query l32; A = V of that
//                key, columns EV l32 .. EV l32 + EV - 1 (one load of a whole row per half-wave): instruction e of a key
//                pair yields output columns EV row + e
// Key ranges that are split over workgroups are merged by the workgroup that finishes last (tickets, as in the bf16
// kernel).
// Measured (MI355X, kernels replayed from a graph; before: one FMA per LDS operand pair, a merge launch): 32 heads x 128
// rows, 4096 keys of 128: 414 -> 109 us (78 TFLOP/s of 157); 8 KV heads x 480 rows x 4 sequences, 2048 keys: 795 -> 191 us;
// 4 heads x 16 rows, 128 keys of 64: 9.5 -> 10 us.  Few rows over few keys are a chain that the 32 x 32 blocks do not
// shorten: 33 rows over 128 keys of 128 13.4 -> 16.8 us, the longest loss seen over 88 shapes but for 512 workgroups of one
// row and one key each (9 -> 15 us).
template <int D, int QB, int KS>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_f32_kernel(
    const int32_t* a_prefix_len, const uint64_t* a_mask, const void* a_Q, const int a_splits, const unsigned a_inv_splits,
    const int a_kv_heads, const unsigned a_inv_kv_heads, const int a_n, const unsigned a_inv_n, const AttnKArgs a) {
    static_assert(QB * KS == 8, "eight wavefronts");
    constexpr int NT = 512, ROWS = 32 * QB, J = D / 8, EV = D / 32, QST = D + 4;
    typedef float fv __attribute__((ext_vector_type(EV)));
    typedef unsigned long long u64;
    extern __shared__ __attribute__((aligned(16))) float s_f[];      // Q [ROWS][QST]; later the exchange between key slices
    __shared__ int s_last;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, h = lane >> 5;
    const int qb = wave % QB, ks = wave / QB;
    const int xcd = blockIdx.x & 7, rb = blockIdx.x >> 3;            // numbering: see the bf16 kernel
    const int unit = blockIdx.y * 8 + xcd;
    if (unit >= a.batch * a_kv_heads * a_splits) return;
    const int bz = fast_div(unit, a_splits, a_inv_splits), split = unit - bz * a_splits;
    const int b = fast_div(bz, a_kv_heads, a_inv_kv_heads), hk = bz - b * a_kv_heads;
    const int L_raw = a_prefix_len[b];
    const int n = a_n, rows_all = a.g * n;
    const int L = clamp_len(L_raw, a.max_prefix);
    const int pblocks = (L + 31) / 32, T = pblocks + (a.nk + 31) / 32;
    int t0 = 0, t1 = T;
    if (a_splits > 1) {
        t0 = (int)((long long)T * split / a_splits);
        t1 = (int)((long long)T * (split + 1) / a_splits);
    }

    const int rho = rb * ROWS + qb * 32 + l32;                       // packed row inside the KV head
    const bool row_ok = rho < rows_all;
    const int rho_c = row_ok ? rho : rows_all - 1;
    const int head = fast_div(rho_c, n, a_inv_n), hq = hk * a.g + head, node = rho_c - head * n;
    const uint64_t* const mask_row = a_mask + ((long long)b * n + node) * a.W;
    const float* const kp = (const float*)a.Kp + (long long)b * a.kps[0] + (long long)hk * a.kps[1];
    const float* const vp = (const float*)a.Vp + (long long)b * a.vps[0] + (long long)hk * a.vps[1];
    const float* const kt = (const float*)a.Kt + (long long)b * a.kts[0] + (long long)hk * a.kts[1];
    const float* const vt = (const float*)a.Vt + (long long)b * a.vts[0] + (long long)hk * a.vts[1];

    f32x4 kr[J];
    fv vr[16];
    uint64_t mword = 0;
    // rows past the end of the keys repeat the last one: their scores are masked
    auto load_k = [&](int t) {
        const bool tree = t >= pblocks;
        const int key0 = 32 * (tree ? t - pblocks : t), last = (tree ? a.nk : L) - 1;
        const float* const row = (tree ? kt : kp) + (long long)min(key0 + l32, last) * (tree ? a.kts[2] : a.kps[2]) + 4 * h;
#pragma unroll
        for (int j = 0; j < J; ++j) kr[j] = *(const f32x4*)(row + 8 * j);
    };
    auto load_v = [&](int t) {
        const bool tree = t >= pblocks;
        const int key0 = 32 * (tree ? t - pblocks : t), last = (tree ? a.nk : L) - 1;
        const float* const base = (tree ? vt : vp) + EV * l32;
        const long long st = tree ? a.vts[2] : a.vps[2];
#pragma unroll
        for (int v = 0; v < 16; ++v) vr[v] = *(const fv*)(base + min(key0 + 8 * (v >> 2) + 4 * h + (v & 3), last) * st);
        mword = tree ? mask_row[key0 >> 6] : 0ull;
    };
    int t = t0 + ks;
    // Q is asked for ahead of K and V: it goes to LDS while they are under way, and the scores wait for K alone.  With it the
    // arguments that are in registers at the start, and divisions by multiplication but for a split's key range (two 64-bit ones):
    // 13 x 16 KV heads of 1024 rows, 253 keys of 128 363 -> 344 us, 14 x 2 of 944 rows 95 -> 89, 4 heads of 16 rows, 144 keys of 64
    // 9.92 -> 9.82, 0 to 7 % over 26 shapes, 1.5 % in the mean (ahead of the prefix length's use 15 x 8 KV heads of 36 rows, 4313 keys
    // of 64 96 -> 98 us, here 96.5)
    constexpr int QI = ROWS * D / 4 / NT;
    f32x4 qr[QI];
#pragma unroll
    for (int i = 0; i < QI; ++i) {
        const int rr = (i * NT + tid) / (D / 4), cc = ((i * NT + tid) % (D / 4)) * 4, r = min(rb * ROWS + rr, rows_all - 1);
        const int hh = fast_div(r, n, a_inv_n);
        qr[i] = *(const f32x4*)((const float*)a_Q + (long long)b * a.qs[0] + (long long)(hk * a.g + hh) * a.qs[1] +
                                (long long)(r - hh * n) * a.qs[2] + cc);
    }
    if (t < t1) { load_k(t); load_v(t); }                            // (slices that only wait must not ask for blocks: 2 to 9 % slower)
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < QI; ++i) {
        const int rr = (i * NT + tid) / (D / 4), cc = ((i * NT + tid) % (D / 4)) * 4;
        *(f32x4*)(s_f + rr * QST + cc) = rb * ROWS + rr < rows_all ? qr[i] : f32x4{0.f, 0.f, 0.f, 0.f};
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // (K and V stay under way)
    if (tid == 0 && hk == 0 && split == 0 && rb == 0) report_clamp(a.counters, L_raw, a.max_prefix);

    const float c = a.scale_log2;
    float ref = -INFINITY, l_run = 0.f;                              // ref: see the bf16 kernel
    f32x16 o[EV];
#pragma unroll
    for (int e = 0; e < EV; ++e)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[e][v] = 0.f;
    const float* const q_row = s_f + (qb * 32 + l32) * QST + 4 * h;
    for (; t < t1; t += KS) {
        f32x16 sc;
#pragma unroll
        for (int v = 0; v < 16; ++v) sc[v] = 0.f;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const f32x4 q = *(const f32x4*)(q_row + 8 * j);
#pragma unroll
            for (int i = 0; i < 4; ++i) sc = __builtin_amdgcn_mfma_f32_32x32x2f32(kr[j][i], q[i], sc, 0, 0, 0);
        }
        const int next = min(t + KS, t1 - 1);                        // (the last block is asked for twice)
        __builtin_amdgcn_sched_barrier(0);
        load_k(next);
        __builtin_amdgcn_sched_barrier(0);
        // visibility; accumulator element v is key 8 (v/4) + 4 h + v%4 of the block
        const bool tree = t >= pblocks;
        const int key0 = 32 * (tree ? t - pblocks : t), left = (tree ? a.nk : L) - key0;
        if (tree || left < 32) {
            unsigned vis = left >= 32 ? 0xffffffffu : (1u << left) - 1u;
            if (tree) vis &= (unsigned)(mword >> (key0 & 32));
            vis >>= 4 * h;
#pragma unroll
            for (int v = 0; v < 16; ++v) sc[v] = (vis >> (8 * (v >> 2) + (v & 3))) & 1u ? sc[v] : -INFINITY;
        }
        float tmax = sc[0];
#pragma unroll
        for (int v = 1; v < 16; ++v) tmax = fmaxf(tmax, sc[v]);
        const float ref_new = fmaxf(ref, xhalf_max(tmax) * c);
        if (ref_new == -INFINITY) {
#pragma unroll
            for (int v = 0; v < 16; ++v) sc[v] = 0.f;
        } else {
            const float alpha = __builtin_amdgcn_exp2f(ref - ref_new);       // ref = -inf gives 0
            float sum = 0.f;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                sc[v] = __builtin_amdgcn_exp2f(fmaf(sc[v], c, -ref_new));
                sum += sc[v];
            }
            l_run = l_run * alpha + sum;
            ref = ref_new;
            if (__any(alpha != 1.f)) {
#pragma unroll
                for (int e = 0; e < EV; ++e)
#pragma unroll
                    for (int v = 0; v < 16; ++v) o[e][v] *= alpha;
            }
        }
#pragma unroll
        for (int v = 0; v < 16; ++v)
#pragma unroll
            for (int e = 0; e < EV; ++e) o[e] = __builtin_amdgcn_mfma_f32_32x32x2f32(vr[v][e], sc[v], o[e], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        load_v(next);
        __builtin_amdgcn_sched_barrier(0);
    }
    l_run = xhalf_sum(l_run);

    // the key slices of a row block meet in LDS, halving their number every round; slices without a block take no part
    const int slices = min(KS, t1 - t0);
    if (slices > 1) {
        __syncthreads();                                             // (Q is no longer needed)
#pragma unroll
        for (int half = KS / 2; half >= 1; half /= 2) {
            if (slices <= half) continue;
            // [half x QB wavefronts][EV 4 + 1][64] x 16 bytes
            f32x4* const slot = (f32x4*)s_f + (size_t)((ks & (half - 1)) * QB + qb) * (EV * 4 + 1) * 64 + lane;
            if (ks >= half && ks < 2 * half && ks < slices) {
#pragma unroll
                for (int e = 0; e < EV; ++e)
#pragma unroll
                    for (int v4 = 0; v4 < 4; ++v4)
                        slot[(e * 4 + v4) * 64] = f32x4{o[e][4 * v4], o[e][4 * v4 + 1], o[e][4 * v4 + 2], o[e][4 * v4 + 3]};
                slot[EV * 4 * 64] = f32x4{ref, l_run, 0.f, 0.f};
            }
            __syncthreads();
            if (ks < half && ks + half < slices) {
                const f32x4 ml = slot[EV * 4 * 64];
                const float top = fmaxf(ref, ml.x);
                float a1 = 0.f, a2 = 0.f;
                if (top != -INFINITY) {
                    a1 = __builtin_amdgcn_exp2f(ref - top);
                    a2 = __builtin_amdgcn_exp2f(ml.x - top);
                }
                l_run = l_run * a1 + ml.y * a2;
                ref = top;
#pragma unroll
                for (int e = 0; e < EV; ++e)
#pragma unroll
                    for (int v4 = 0; v4 < 4; ++v4) {
                        const f32x4 x = slot[(e * 4 + v4) * 64];
#pragma unroll
                        for (int w = 0; w < 4; ++w) o[e][4 * v4 + w] = o[e][4 * v4 + w] * a1 + x[w] * a2;
                    }
            }
            if (half > 1) __syncthreads();
        }
    }

    // element v of o[0 .. EV-1] are columns EV (8 (v/4) + 4 h + v%4) .. + EV - 1 of row l32
    if (a.splits == 1) {
        if (ks == 0 && row_ok) {
            const float inv = l_run > 0.f ? 1.f / l_run : 0.f;
            float* const orow = (float*)a.O + (long long)b * a.os[0] + (long long)hq * a.os[1] + (long long)node * a.os[2];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                fv x;
#pragma unroll
                for (int e = 0; e < EV; ++e) x[e] = o[e][v] * inv;
                *(fv*)(orow + EV * (8 * (v >> 2) + 4 * h + (v & 3))) = x;
            }
        }
        return;
    }
    // part_o [group][split][ROWS][D], part_ml [group][split][ROWS] (ref, l): written through and read around the caches, in
    // the order stores - barrier - ticket (see the bf16 kernel)
    auto pack2 = [](float x, float y) -> u64 { return (u64)__float_as_uint(x) | ((u64)__float_as_uint(y) << 32); };
    const int group = bz * a.row_blocks + rb;
    if (ks == 0 && row_ok) {
        const size_t pr = ((size_t)group * a.splits + split) * ROWS + qb * 32 + l32;
        u64* const po = (u64*)(a.part_o + pr * D);
#pragma unroll
        for (int v = 0; v < 16; ++v)
#pragma unroll
            for (int e = 0; e < EV; e += 2)
                __hip_atomic_store(po + (EV * (8 * (v >> 2) + 4 * h + (v & 3)) + e) / 2, pack2(o[e][v], o[e + 1][v]), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        if (h == 0)
            __hip_atomic_store((u64*)a.part_ml + pr, pack2(ref, l_run), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0)
        s_last = __hip_atomic_fetch_add(a.counters + group, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                         (unsigned)(a.splits - 1) ? 1 : 0;
    __syncthreads();
    if (!s_last) return;
    if (tid == 0) __hip_atomic_store(a.counters + group, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // for the next launch
    const int live = min(ROWS, rows_all - rb * ROWS);
    const u64* const ml0 = (const u64*)a.part_ml + (size_t)group * a.splits * ROWS;
    const u64* const po0 = (const u64*)(a.part_o + (size_t)group * a.splits * ROWS * D);
    for (int i = tid; i < live * (D / 4); i += NT) {                 // four columns of a row per thread and round
        const int rr = i / (D / 4), cc = i % (D / 4);
        float M = -INFINITY, Ls = 0.f;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        for (int s0 = 0; s0 < a.splits; s0 += 8) {                   // eight splits per trip to memory
            u64 ml[8], x[8][2];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const size_t si = min(s0 + u, a.splits - 1);         // past the end: a copy, weight 0
                ml[u] = __hip_atomic_load(ml0 + si * ROWS + rr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                for (int e = 0; e < 2; ++e)
                    x[u][e] = __hip_atomic_load(po0 + (si * ROWS + rr) * (D / 2) + 2 * cc + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            float mi[8], m_new = M;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                mi[u] = s0 + u < a.splits ? __uint_as_float((unsigned)ml[u]) : -INFINITY;
                m_new = fmaxf(m_new, mi[u]);
            }
            if (m_new == -INFINITY) continue;
            const float alpha = __builtin_amdgcn_exp2f(M - m_new);
            Ls *= alpha;
            acc *= alpha;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const float w = mi[u] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mi[u] - m_new);
                Ls = fmaf(w, __uint_as_float((unsigned)(ml[u] >> 32)), Ls);
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    acc[2 * e] = fmaf(w, __uint_as_float((unsigned)x[u][e]), acc[2 * e]);
                    acc[2 * e + 1] = fmaf(w, __uint_as_float((unsigned)(x[u][e] >> 32)), acc[2 * e + 1]);
                }
            }
            M = m_new;
        }
        const float inv = Ls > 0.f ? 1.f / Ls : 0.f;
        const int r = rb * ROWS + rr, hh = r / n;
        *(f32x4*)((float*)a.O + (long long)b * a.os[0] + (long long)(hk * a.g + hh) * a.os[1] + (long long)(r - hh * n) * a.os[2] + 4 * cc) =
            acc * inv;
    }
}

__global__ void attn_clear_sync_kernel(unsigned int* p) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < OT_ATTN_SYNC_BYTES / 4) p[i] = 0u;
}

}  // namespace

static size_t align_up(size_t v, size_t al) { return (v + al - 1) / al * al; }

// Packed query rows per workgroup of the bf16 kernel: 64 (narrow: the wavefronts split each tile's keys), 128, or 256 --
// eight wavefronts then share every staged K/V tile, which halves the traffic into LDS per MFMA and leaves room for a ring
// of four tiles -- where the 256-row blocks are many or long enough: us at 128 / 256 rows, 16-bit cache of 128: 4 x 8 KV heads
// of 480 rows, 1060 keys 23.8 / 26.7, 2060 keys 34.6 / 33.7, 8060 keys 83 / 76; 1 x 8 of 480 rows, 8060 keys 33 / 45;
// 16 x 8 of 480 rows, 160 keys 18.4 / 18.7, 360 keys 29.1 / 25.0, 2060 keys 83 / 76; 8-bit cache: 2060 keys 84 / 74.  An 8-bit
// tile has to be widened two tiles ahead: a workgroup with few of them waits for that, each of several on a unit: 25 x 40 KV heads
// of 800 rows, 60 keys 159 / 207, 200 keys 259 / 303; 32 x 8 of 800 rows, 320 keys 78 / 87, 500 keys (nine tiles) 106 / 111;
// 1000 heads of 480 rows, 500 keys 237 / 230.  Nor does it pay to start one more round of 256-row blocks where half a round of
// 128-row ones does, unless tiles are many: 160 heads of 480 rows, 400 keys 46.6 / 49.8, 700 keys 61.5 / 65.2, 1500 keys 109 / 111,
// 6000 keys 360 / 358; 320 heads 73 / 79, 98 / 101, 180 / 171; 200 heads (almost two full rounds) 57 / 52, 75 / 67.
static int attn_rows_per_workgroup(const ot_attn_params& p, bool kv8, int tiles) {
    const int rows = p.q_heads / p.kv_heads * p.n;
    if (rows <= 64) return 64;
    if (rows <= 128 || (kv8 && p.head_dim == 64)) return 128;   // (64 one-byte rows of 64 have fewer pieces than 512 threads)
    const long long heads = (long long)p.batch * p.kv_heads, blocks = heads * ((rows + 255) / 256);
    const bool half_round = blocks > 256 && (heads * ((rows + 127) / 128) + 255) / 256 < 2 * ((blocks + 255) / 256);
    if (kv8 && ((tiles < 8 && blocks > 512) || (tiles < 20 && half_round))) return 128;
    return blocks >= 64 && blocks * tiles >= 2048 ? 256 : 128;
}

// `splits` ranges that take the same number of tiles (the last one possibly fewer)
static int even_out(int tiles, long long splits) {
    const int s = (int)std::max(1LL, std::min<long long>({splits, tiles, kMaxSplits})), per = (tiles + s - 1) / s;
    return (tiles + per - 1) / per;
}

// Key splits of the bf16 kernel: at least `least`, which is what a workspace has to hold, and `best` where it holds that.
// More splits shorten the streaming, but the workgroup that finishes last merges them all, 1.6 us
// for every trip to memory: as many as fill the 256 compute units once, and eight (the narrow variant: what one trip takes,
// at head_dim 128, six, two and more trips over long prefixes).  us by splits, one sequence unless noted:
//   64 rows x 8 heads, 128: 1016 keys 3: 14.5, 6: 11.3, 9: 12.6; 4008 keys 6: 19.5, 11: 16.5, 32: 21.1; 8016 keys 8: 26.7, 16: 21.0
//   64 rows x 8 heads, 64: 1016 keys 6: 9.8, 9: 9.2; 4016 keys 8: 13.6, 11: 12.0, 32: 16.3; two sequences 11: 12.9, 32: 23.7
//   200 rows x 8 heads in blocks of 128, 128: 250 keys 1: 12.5, 3: 14.1, 5: 14.3; 1050 keys 1: 25.6, 3: 18.9, 6: 17.3, 9: 19.1;
//   4050 keys 4: 30.4, 8: 23.8, 16: 25.8, 32: 34 to 45; 120 rows x 16 heads x 4, 4060 keys 4 (256 workgroups): 33.2, 8: 40.0;
//   50 rows x 32 heads, 64: 4050 keys 8 (256): 14.1, 16: 17.8
// Where one workgroup per unit leaves no split, the variants of which two fit a unit are split over those; two also hide each
// other's widening of 8-bit tiles (1264 rows x 4 heads x 2, 2158 keys of 128 3: 33.5, 6: 30.1; 120 rows x 16 x 4, 4120 of 64
// 4: 26.9, 8: 23.6).
struct AttnSplits { int least, best; };
static AttnSplits attn_splits(long long base, int tiles, int rows_wg, int row_blocks, int head_dim, bool kv8) {
    const bool wide = rows_wg > 64, two = rows_wg == 128 || (!wide && head_dim == 64);
    // Few tiles, 128-row blocks: a range of one tile each has nothing to stream behind and nothing to widen while it computes, and
    // pays for its merge.  us, one range / one a tile, 120 rows x 8 heads: 8-bit of 128, 120 keys 11.8 / 11.3, 190 keys 13.2 / 11.5,
    // 250 keys 14.9 / 12.5, 320 keys (three ranges) 13.6 / 12.6 and with 32 heads 13.9 / 13.8; 8-bit of 64, 250 keys 10.1 / 9.3;
    // 16-bit of 64, 190 keys 8.8 / 8.1, 250 keys 9.3 / 9.0, 11 x 2 heads of 240 rows, 134 keys 8.4 / 8.9; of 128, 190 keys 11.3 / 10.9, 250 keys 12.4 / 12.0, with 64 heads 11.7 /
    // 12.6.
    const bool one_each = rows_wg == 128 && tiles >= (kv8 ? 3 : 4) && tiles <= (kv8 ? 6 : 5) &&
                          base * tiles <= (tiles == 6 ? 96 : kv8 ? 256 : head_dim == 64 ? 128 : 48);
    if (tiles <= (wide || head_dim == 64 ? 5 : 1)) return {1, one_each ? tiles : 1};
    long long s = 256 / base;
    if (s < 2) s = two && tiles >= 24 ? 512 / base : 1;
    else if (kv8 && two && s >= 3 && s <= 5) s = 512 / base;
    const int most = wide ? 8 : merge_chunk(head_dim, false) * (head_dim == 128 ? 1 + tiles / 48 : 1);
    s = std::min<long long>(s, most);
    const int least = even_out(tiles, std::min<long long>(s, wide ? tiles / 2 : tiles));
    if (one_each) return {least, tiles};
    // 64 rows of 128, few heads: the second trip of six pays somewhat earlier than many heads let it.  us, six / up to twelve: 17 rows
    // x 8 heads, 1900 keys 12.6 / 11.5, 2720 keys 14.6 / 12.6, 8-bit 14.0 / 12.1, 17.0 / 13.5; 50 rows, 1900 keys 13.9 / 13.0, 2720
    // keys 15.8 / 14.3; x 16 heads, 1900 keys 14.0 / 14.3, 2720 keys 16.0 / 15.7
    if (!wide && head_dim == 128 && base <= 10 && tiles >= 28 && tiles < 48) return {least, even_out(tiles, 12)};
    if (least == 1 || !two || tiles < (kv8 ? 16 : 24)) return {least, least};
    // Longer prefixes, variants of which two workgroups fit a unit: what more ranges save grows with the prefix, what their merge
    // costs does not.  Both in units of the time that a tile takes a workgroup with a unit to itself (1.2 us at head_dim 128,
    // 0.8 at 64; 8-bit 1.6 and 1.0): with two workgroups to a unit a tile takes each `shared`, least where one widens while the
    // other computes, all of twice as long where each key is read once and memory is what bounds; the merge adds `merge` a range
    // (narrow: a trip of twelve), the rest of a launch some 8.  us, `least` / more ranges, one sequence unless noted:
    //   200 rows x 8 heads, 128: 16384 keys 8: 50.7, 16: 38.6; 32768 keys 8: 86.9, 16: 57.6, 32: 59.7; 131072 keys 307, 180, 158;
    //   8-bit 32768 keys 114, 70, 67; 64 wide 32768 keys 60.7, 39.7, 36.6; x 2 heads 32768 keys 84, 53, 44
    //   480 rows x 8 heads, 128: 8192 keys 8: 32.9, 16: 35.0; 32768 keys 90, 83; x 24 heads 8192 keys 2: 85.5, 5: 65.6
    //   120 rows x 100 heads, 128: 2048 keys 2: 33.3, 5: 36.2; 8192 keys 100, 90; 8-bit 1000 keys 26.7, 24.6; 8192 keys 112, 81
    //   64 rows x 8 heads, 64: 8192 keys 12: 15.1, 24: 15.2; 16384 keys 22.2, 18.7; 131072 keys 120, 24: 69, 32: 59
    const float shared = kv8 ? (wide ? 1.4f : 1.3f) : !wide ? 1.85f : head_dim == 64 ? 1.5f : row_blocks > 1 ? 1.6f : 2.f;
    auto time = [&](int x) {
        const bool one = base * x <= 256;
        const float merge = wide ? (head_dim == 128 ? (one ? 0.42f : 0.7f) : (one ? 0.3f : 0.54f)) * (kv8 ? 0.8f : 1.f) * x
                                 : (one ? 5.f : kv8 ? 6.f : 7.f) * ((x + 11) / 12);
        return (one ? 1.f : shared) * ((tiles + x - 1) / x) + merge + 8.f;
    };
    int best = least;
    float best_time = (tiles < 80 ? 0.89f : 0.94f) * time(least);        // (what the estimate is good for)
    for (int x = least + 1; x <= kMaxSplits && x <= tiles && base * x <= 512; ++x)
        if (even_out(tiles, x) == x && time(x) < best_time) { best = x; best_time = time(x); }
    return {least, best};
}

// Packed query rows per workgroup of the f32 kernel (its eight wavefronts = rows / 32 row blocks x key slices): as many as
// there are up to 128 where the row blocks alone fill the chip; fewer, with the rest of the wavefronts on the keys, where
// key ranges are split over workgroups -- 256 workgroups then leave at most 4 MB of partials.
static int f32_rows_per_workgroup(const ot_attn_params& p) {
    const int rows = p.q_heads / p.kv_heads * p.n, most = rows <= 32 ? 32 : (rows <= 64 ? 64 : 128);
    if (most == 32 || (long long)p.batch * p.kv_heads * ((rows + most - 1) / most) >= 256) return most;
    return p.head_dim == 64 ? 64 : 32;
}

AttnPlan plan_attention(const ot_attn_params& p, bool kv8, size_t room) {
    AttnPlan pl;
    pl.balance = 0;
    const int g = p.q_heads / p.kv_heads, nk = p.n_keys > 0 ? p.n_keys : p.n;
    int base, tile, rows_wg = 0, splits, least;
    if (p.dtype == OT_BF16) {
        tile = 64;
        const int tiles = (p.max_prefix + 63) / 64 + (nk + 63) / 64;
        rows_wg = attn_rows_per_workgroup(p, kv8, tiles);
        pl.row_blocks = (g * p.n + rows_wg - 1) / rows_wg;
        base = p.batch * p.kv_heads * pl.row_blocks;
        const AttnSplits sp = attn_splits(base, tiles, rows_wg, pl.row_blocks, p.head_dim, kv8);
        splits = sp.best;
        least = sp.least;
        // A batch that fills the chip with one key range per (sequence, KV head): the lengths are known on the
        // device only, where the workgroups take their jobs longest first (see the kernel).  Measured: 3 % faster on
        // ragged batches of one and a half to three rounds of workgroups; from four rounds on the rounds even the
        // lengths out by themselves and the ranking's extra trip to memory per workgroup costs 1 %.
        const int resident = rows_wg == 256 ? 256 : 512;   // workgroups that the chip holds at once
        if (rows_wg > 64 && p.batch > 1 && p.batch <= 64 && splits == 1 && base > resident / 2 && base < 4 * resident) pl.balance = 1;
    } else {
        // One workgroup per compute unit at a time (eight wavefronts, two per SIMD).  Splitting costs 5 us (partials through
        // memory, the merge), a 32 x 32 block 2 us of a SIMD at head_dim 64 and 4 at 128: what is at most two blocks per SIMD
        // stays whole, and a split has one block for every SIMD at least.  Measured, us, a split for every eight blocks with
        // prefix and tree rounded apart / this rule: 8 x 4 heads of 5 rows, 17 keys of 128 16.5 / 9.3; 4 heads of 16 rows, 1000
        // keys of 128 21.4 / 16.9; 4 sequences of 33 rows, 500 keys of 128 23.2 / 17.8; 8 x 8 heads of 60 rows, 128 keys of 128
        // 22.1 / 17.9; 4 x 4 heads of 128 rows, 128 keys of 64 18.6 / 14.6.
        rows_wg = f32_rows_per_workgroup(p);
        pl.row_blocks = (g * p.n + rows_wg - 1) / rows_wg;
        base = p.batch * p.kv_heads * pl.row_blocks;
        tile = 32;
        const int blocks = ((p.max_prefix + 31) / 32 + (nk + 31) / 32) * (rows_wg / 32);
        splits = blocks <= 8 ? 1 : std::min(256 / base, (blocks + 3) / 4);
    }
    const int max_tiles = (p.max_prefix + tile - 1) / tile + (nk + tile - 1) / tile;
    splits = even_out(max_tiles, splits);
    if (p.dtype != OT_BF16) least = splits;
    // partials are stored per workgroup (rows padded to the row block)
    const size_t rows = (size_t)base * rows_wg;
    const size_t part_elem = (p.dtype == OT_BF16 && OT_ATTN_PART_BF16) ? 2 : 4;
    const size_t fixed = OT_ATTN_SYNC_BYTES + 256, range = rows * (p.head_dim * part_elem + 2 * 4);   // (a multiple of 256)
    if (splits > least && fixed + splits * range > room) {
        const size_t held = room > fixed ? (room - fixed) / range : 0;      // fewer than `splits`
        splits = std::max(least, even_out(max_tiles, (long long)held));
    }
    pl.rows = rows_wg;
    pl.splits = splits;
    pl.part_o_bytes = splits > 1 ? align_up(rows * splits * p.head_dim * part_elem, 256) : 0;
    pl.part_ml_bytes = splits > 1 ? align_up(rows * splits * 2 * 4, 256) : 0;
    pl.bytes = OT_ATTN_SYNC_BYTES + pl.part_o_bytes + pl.part_ml_bytes + 256;
    return pl;
}

int launch_tree_attention(const ot_attn_params& p, const AttnPlan& plan, const void* Q, const void* Kp, const void* Vp,
                          const void* Kt, const void* Vt, const int32_t* prefix_len, const uint64_t* mask, void* O,
                          void* workspace, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1, const float* k_scale,
                          const float* v_scale) {
    const bool kv8 = k_scale != nullptr;
    AttnKArgs a;
    a.splits_share_xcd = 0;
    a.Q = Q; a.Kp = Kp; a.Vp = Vp; a.Kt = Kt; a.Vt = Vt;
    a.prefix_len = prefix_len; a.mask = mask; a.O = O;
    a.k_scale = k_scale; a.v_scale = v_scale;
    a.counters = (unsigned int*)workspace;
    a.part_o = (float*)((char*)workspace + OT_ATTN_SYNC_BYTES);
    a.part_ml = (float*)((char*)workspace + OT_ATTN_SYNC_BYTES + plan.part_o_bytes);
    a.batch = p.batch; a.kv_heads = p.kv_heads; a.g = p.q_heads / p.kv_heads;
    a.n = p.n; a.nk = p.n_keys > 0 ? p.n_keys : p.n; a.max_prefix = p.max_prefix; a.splits = plan.splits;
    a.W = OT_MASK_WORDS(a.nk);
    const float scale = p.softmax_scale != 0.f ? p.softmax_scale : 1.0f / sqrtf((float)p.head_dim);
    a.scale_log2 = scale * kLog2e;
    for (int i = 0; i < 3; ++i) {
        a.qs[i] = p.q_strides[i]; a.kps[i] = p.kp_strides[i]; a.vps[i] = p.vp_strides[i];
        a.kts[i] = p.kt_strides[i]; a.vts[i] = p.vt_strides[i]; a.os[i] = p.o_strides[i];
    }
    a.row_blocks = plan.row_blocks;
    auto magic = [](int d) { return d <= 1 ? 0u : (unsigned int)((0x100000000ull + (unsigned)d - 1) / (unsigned)d); };
    a.inv_splits = magic(a.splits); a.inv_kv_heads = magic(a.kv_heads); a.inv_n = magic(a.n);
#define OT_ATTN_ARGS a.prefix_len, a.mask, a.Q, a.splits, a.inv_splits, a.kv_heads, a.inv_kv_heads, a.n, a.inv_n, a
    if (p.dtype == OT_BF16) {
        const int rows_wg = plan.rows;
        const long long units = (long long)p.batch * p.kv_heads * plan.splits;
        const long long unit_groups = (units + 7) / 8;      // the same count either way when pairs % 8 == 0
        a.splits_share_xcd = (!plan.balance && plan.splits > 1 && ((long long)p.batch * p.kv_heads) % 8 == 0) ? 1 : 0;
        if (unit_groups > 65535 || 8LL * plan.row_blocks > 0x7fffffffLL) return OT_ERR_UNSUPPORTED;   // cannot happen within the limits
        if (plan.splits > 1 && (long long)p.batch * p.kv_heads * plan.row_blocks * 4 > OT_ATTN_STATUS_OFFSET)
            return OT_ERR_UNSUPPORTED;      // cannot happen: splits > 1 only with few workgroups
        const dim3 grid((unsigned)(8 * plan.row_blocks), (unsigned)unit_groups);
#define OT_ATTN_LAUNCH(DD, VV, K8, BB)                                                                       \
    do {                                                                                                   \
        const int nbuf = tile_buffers(VV, K8), nwaves = (VV) == 2 ? 8 : 4; \
        const int raw = (VV) == 2 && (K8) ? 32 * DD : 0;                                                   \
        const size_t lds = (size_t)nbuf * (64 * DD + raw + nwaves * 128) * sizeof(unsigned int);           \
        if (lds > 64 * 1024)                                                                               \
            OT_HIP_CHECK(hipFuncSetAttribute((const void*)attn_mfma_kernel<DD, VV, K8, BB>,                 \
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));       \
        if (ev0 || ev1) hipExtLaunchKernelGGL((attn_mfma_kernel<DD, VV, K8, BB>), grid, dim3(64 * nwaves), lds, s, ev0, ev1, 0, OT_ATTN_ARGS); \
        else hipLaunchKernelGGL((attn_mfma_kernel<DD, VV, K8, BB>), grid, dim3(64 * nwaves), lds, s, OT_ATTN_ARGS); \
    } while (0)
        const int var = rows_wg == 256 ? 2 : (rows_wg == 128 ? 1 : (units > 256 ? 3 : 0));   // (3: see tile_buffers)
        // (only wide variants take their jobs longest first; the 8-bit cache has no 256-row variant at head_dim 64)
#define OT_ATTN_PICK(DD, K8)                                                                                \
    do {                                                                                                    \
        constexpr int V2 = (K8) && (DD) == 64 ? 1 : 2, V3 = (K8) || (DD) == 64 ? 0 : 3;                     \
        if (var == 2)      { if (plan.balance) OT_ATTN_LAUNCH(DD, V2, K8, true); else OT_ATTN_LAUNCH(DD, V2, K8, false); } \
        else if (var == 1) { if (plan.balance) OT_ATTN_LAUNCH(DD, 1, K8, true); else OT_ATTN_LAUNCH(DD, 1, K8, false); } \
        else if (var == 3) OT_ATTN_LAUNCH(DD, V3, K8, false);                                               \
        else               OT_ATTN_LAUNCH(DD, 0, K8, false);                                                \
    } while (0)
        if (kv8) { if (p.head_dim == 128) OT_ATTN_PICK(128, true); else OT_ATTN_PICK(64, true); }
        else     { if (p.head_dim == 128) OT_ATTN_PICK(128, false); else OT_ATTN_PICK(64, false); }
#undef OT_ATTN_PICK
#undef OT_ATTN_LAUNCH
    } else {
        const int rows_wg = plan.rows;
        const long long unit_groups = ((long long)p.batch * p.kv_heads * plan.splits + 7) / 8;
        if (unit_groups > 65535 || 8LL * plan.row_blocks > 0x7fffffffLL) return OT_ERR_UNSUPPORTED;   // cannot happen within the limits
        if (plan.splits > 1 && (long long)p.batch * p.kv_heads * plan.row_blocks * 4 > OT_ATTN_STATUS_OFFSET)
            return OT_ERR_UNSUPPORTED;      // cannot happen: splits > 1 only with few workgroups
        const dim3 grid((unsigned)(8 * plan.row_blocks), (unsigned)unit_groups);
#define OT_F32_LAUNCH(DD, QQ, KK)                                                                                      \
    do {                                                                                                               \
        const size_t q = (size_t)32 * QQ * (DD + 4) * 4, x = (KK) > 1 ? (size_t)4 * (DD / 8 + 1) * 64 * 16 : 0;          \
        const size_t lds = q > x ? q : x;                                                                              \
        if (lds > 64 * 1024)                                                                                           \
            OT_HIP_CHECK(hipFuncSetAttribute((const void*)attn_f32_kernel<DD, QQ, KK>,                                  \
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));                   \
        if (ev0 || ev1) hipExtLaunchKernelGGL((attn_f32_kernel<DD, QQ, KK>), grid, dim3(512), lds, s, ev0, ev1, 0, OT_ATTN_ARGS);  \
        else hipLaunchKernelGGL((attn_f32_kernel<DD, QQ, KK>), grid, dim3(512), lds, s, OT_ATTN_ARGS);                             \
    } while (0)
#define OT_F32_PICK(DD)                                                                                                \
    do {                                                                                                               \
        if (rows_wg == 32) OT_F32_LAUNCH(DD, 1, 8);                                                                    \
        else if (rows_wg == 64) OT_F32_LAUNCH(DD, 2, 4);                                                               \
        else OT_F32_LAUNCH(DD, 4, 2);                                                                                  \
    } while (0)
        if (p.head_dim == 128) OT_F32_PICK(128); else OT_F32_PICK(64);
#undef OT_F32_PICK
#undef OT_F32_LAUNCH
    }
#undef OT_ATTN_ARGS
    OT_HIP_CHECK(hipGetLastError());
    return OT_OK;
}

}  // namespace ot

using namespace ot;

static int validate_attn(const ot_attn_params* p, bool kv8 = false) {
    if (!p) return OT_ERR_INVALID_ARG;
    if (p->batch < 1 || p->q_heads < 1 || p->kv_heads < 1 || p->n < 1 || p->max_prefix < 0) return OT_ERR_INVALID_ARG;
    if (p->q_heads % p->kv_heads) return OT_ERR_INVALID_ARG;
    if (p->dtype != OT_F32 && p->dtype != OT_BF16) return OT_ERR_INVALID_ARG;
    if (!(p->softmax_scale >= 0.f)) return OT_ERR_INVALID_ARG;
    if (p->head_dim != 64 && p->head_dim != 128) return OT_ERR_UNSUPPORTED;
    if (p->n > OT_MAX_NODES) return OT_ERR_UNSUPPORTED;
    if (p->n_keys < 0) return OT_ERR_INVALID_ARG;
    if (p->n_keys > OT_MAX_TREE_KEYS) return OT_ERR_UNSUPPORTED;
    if ((long long)p->batch * p->q_heads > 65535 || (long long)p->batch * p->q_heads * p->n > 0x7fffffffLL)
        return OT_ERR_UNSUPPORTED;
    if (kv8 && p->dtype != OT_BF16) return OT_ERR_INVALID_ARG;      // Q and O of the 8-bit cache variant are bf16
    const int64_t* st[6] = {p->q_strides, p->kp_strides, p->vp_strides, p->kt_strides, p->vt_strides, p->o_strides};
    for (int t = 0; t < 6; ++t) {
        const int vec = (kv8 && t >= 1 && t <= 4) ? 16 : (p->dtype == OT_BF16 ? 8 : 4);      // elements per 16 bytes
        for (int i = 0; i < 3; ++i)
            if (st[t][i] < 0 || st[t][i] % vec) return OT_ERR_INVALID_ARG;
        if (st[t][2] < p->head_dim) return OT_ERR_INVALID_ARG;
        if (st[t][2] > (1 << 22)) return OT_ERR_UNSUPPORTED;    // 64 rows of a tile are addressed with 32-bit offsets
    }
    return OT_OK;
}

// one workspace serves both caches, whose row blocks and key splits may differ
static size_t attn_bytes(const ot_attn_params& p, size_t room) {
    return std::max(plan_attention(p, false, room).bytes, p.dtype == OT_BF16 ? plan_attention(p, true, room).bytes : 0);
}

extern "C" {

size_t ot_attn_workspace_bytes(const ot_attn_params* p) {
    if (validate_attn(p) != OT_OK) return 0;
    // the library's own array goes on serving what it can hold with the fewest ranges
    const size_t full = attn_bytes(*p, SIZE_MAX);
    return full > OT_ATTN_SCRATCH_BYTES && attn_bytes(*p, 0) <= OT_ATTN_SCRATCH_BYTES ? attn_bytes(*p, OT_ATTN_SCRATCH_BYTES) : full;
}

size_t ot_attn_workspace_bytes_full(const ot_attn_params* p) { return validate_attn(p) != OT_OK ? 0 : attn_bytes(*p, SIZE_MAX); }

int ot_internal_attn_plan(const ot_attn_params* p, int32_t kv8, size_t room, int32_t* rows, int32_t* splits, int32_t* balance) {
    const int st = validate_attn(p, kv8 != 0);
    if (st != OT_OK) return st;
    const AttnPlan pl = plan_attention(*p, kv8 != 0, room);
    *rows = pl.rows; *splits = pl.splits; *balance = pl.balance;
    return OT_OK;
}

static int attention_entry(const ot_attn_params* p, const void* Q, const void* K_prefix, const void* V_prefix,
                           const void* K_tree, const void* V_tree, const int32_t* prefix_len, const uint64_t* mask,
                           void* O, void* workspace, size_t workspace_bytes, void* hip_stream, void* ev0, void* ev1,
                           const float* k_scale = nullptr, const float* v_scale = nullptr, bool kv8 = false) {
    int st = validate_attn(p, kv8);
    if (st != OT_OK) return st;
    if (kv8 && (!k_scale || !v_scale || ((uintptr_t)k_scale % 4) || ((uintptr_t)v_scale % 4))) return OT_ERR_INVALID_ARG;
    if (!Q || !K_tree || !V_tree || !prefix_len || !mask || !O || !workspace) return OT_ERR_INVALID_ARG;
    if (p->max_prefix > 0 && (!K_prefix || !V_prefix)) return OT_ERR_INVALID_ARG;
    const void* ptrs[7] = {Q, K_prefix, V_prefix, K_tree, V_tree, O, workspace};
    for (int i = 0; i < 7; ++i)
        if (ptrs[i] && ((uintptr_t)ptrs[i] % 16)) return OT_ERR_INVALID_ARG;
    if (((uintptr_t)prefix_len % 4) || ((uintptr_t)mask % 8)) return OT_ERR_INVALID_ARG;
    const AttnPlan plan = plan_attention(*p, kv8, workspace_bytes);
    if (workspace_bytes < plan.bytes) return OT_ERR_WORKSPACE_TOO_SMALL;
    return launch_tree_attention(*p, plan, Q, K_prefix, V_prefix, K_tree, V_tree, prefix_len, mask, O, workspace,
                                 (hipStream_t)hip_stream, (hipEvent_t)ev0, (hipEvent_t)ev1, kv8 ? k_scale : nullptr,
                                 kv8 ? v_scale : nullptr);
}

int ot_attn_workspace_prepare(void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (!workspace || ((uintptr_t)workspace % 16)) return OT_ERR_INVALID_ARG;
    if (workspace_bytes < OT_ATTN_SYNC_BYTES) return OT_ERR_WORKSPACE_TOO_SMALL;
    hipLaunchKernelGGL(attn_clear_sync_kernel, dim3(OT_ATTN_SYNC_BYTES / 4 / 256), dim3(256), 0, (hipStream_t)hip_stream,
                       (unsigned int*)workspace);
    OT_HIP_CHECK(hipGetLastError());
    return OT_OK;
}

int ot_tree_verify_attention(const ot_attn_params* p, const void* Q, const void* K_prefix, const void* V_prefix,
                             const void* K_tree, const void* V_tree, const int32_t* prefix_len, const uint64_t* mask,
                             void* O, void* workspace, size_t workspace_bytes, void* hip_stream) {
    return attention_entry(p, Q, K_prefix, V_prefix, K_tree, V_tree, prefix_len, mask, O, workspace, workspace_bytes,
                           hip_stream, nullptr, nullptr);
}

// ---------------------------------------------------------------------------
// Entry point for callers that cannot allocate: the workspace (ticket counters, status word, split partials) is a
// library-owned array in device memory.  Every GPU holds its own copy at its own address; host code never uses
// the array's name except to look that address up, once per device.
// ---------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[OT_ATTN_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices];       // device address of `scratch` on device i, null until looked up
}  // namespace

int ot_tree_verify_attention_noalloc(const ot_attn_params* p, const void* Q, const void* K_prefix, const void* V_prefix,
                                     const void* K_tree, const void* V_tree, const int32_t* prefix_len,
                                     const uint64_t* mask, void* O, void* hip_stream) {
    int st = validate_attn(p);
    if (st != OT_OK) return st;
    if (ot_attn_workspace_bytes(p) > (size_t)OT_ATTN_SCRATCH_BYTES) return OT_ERR_SCRATCH_LIMIT;
    int dev = -1;
    OT_HIP_CHECK(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return OT_ERR_UNSUPPORTED;
    void* ptr;
    {
        std::lock_guard<std::mutex> lock(g_scratch_mutex);
        if (!g_scratch_ptr[dev]) {
            // set-up, once per device, with that device current: the address of this device's copy of the array,
            // and its ticket counters and status word cleared (by a kernel, which a graph capture could record)
            void* found = nullptr;
            OT_HIP_CHECK(hipGetSymbolAddress(&found, HIP_SYMBOL(scratch)));
            if (!found || ((uintptr_t)found % 256)) return OT_ERR_HIP;
            hipLaunchKernelGGL(attn_clear_sync_kernel, dim3(OT_ATTN_SYNC_BYTES / 4 / 256), dim3(256), 0,
                               (hipStream_t)hip_stream, (unsigned int*)found);
            OT_HIP_CHECK(hipGetLastError());
            g_scratch_ptr[dev] = found;
        }
        ptr = g_scratch_ptr[dev];
    }
    return attention_entry(p, Q, K_prefix, V_prefix, K_tree, V_tree, prefix_len, mask, O, ptr, OT_ATTN_SCRATCH_BYTES,
                           hip_stream, nullptr, nullptr);
}

int ot_tree_verify_attention_fp8kv(const ot_attn_params* p, const void* Q, const void* K_prefix, const void* V_prefix,
                                   const void* K_tree, const void* V_tree, const float* k_scale, const float* v_scale,
                                   const int32_t* prefix_len, const uint64_t* mask, void* O, void* workspace,
                                   size_t workspace_bytes, void* hip_stream) {
    return attention_entry(p, Q, K_prefix, V_prefix, K_tree, V_tree, prefix_len, mask, O, workspace, workspace_bytes,
                           hip_stream, nullptr, nullptr, k_scale, v_scale, true);
}

int ot_tree_verify_attention_timed(const ot_attn_params* p, const void* Q, const void* K_prefix, const void* V_prefix,
                                   const void* K_tree, const void* V_tree, const int32_t* prefix_len,
                                   const uint64_t* mask, void* O, void* workspace, size_t workspace_bytes,
                                   void* hip_stream, void* kernel_begin_event, void* kernel_end_event) {
    return attention_entry(p, Q, K_prefix, V_prefix, K_tree, V_tree, prefix_len, mask, O, workspace, workspace_bytes,
                           hip_stream, kernel_begin_event, kernel_end_event);
}

}  // extern "C"
