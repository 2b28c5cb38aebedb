"""Parity of ot_build_tree / ot_tree_expand / ot_tree_finalize with the fp64 oracle (needs an MI355X).

Tree structure (tokens, parents, depths, masks, n_out) must be bit-exact; log p^ within 1e-5 absolute
and E within 1e-6 relative (fp32 exp-sum with fp64 combination, error budget ~1e-7 per row).
Inputs are regenerated with the next seed until every selection cut has a cross-parent gap > 1e-5."""
import numpy as np
import pytest

from oracle import opt_tree as ot_oracle
import workloads as wl
from tests import _util as U

pytestmark = pytest.mark.gpu


def _run(logits_stored, dtype, k, n, depth):
    from paper_2406_17276_amd import api
    import torch
    dev = U.to_device(logits_stored, dtype)
    tree = api.build_tree(dev, k, n, depth)
    torch.cuda.synchronize()
    return tree


@pytest.mark.parametrize("name", ["tiny", "7b", "13b"])
def test_full_config_single_sequence(name):
    w = wl.WORKLOADS[name]
    seed, logits, want = U.gapped_logits(w, 0)
    print(f"{name}: seed {seed}, min gap {min(t['min_gap'] for t in want):.3e}", flush=True)
    got = _run(logits, w.dtype, w.k, w.n, w.depth)
    U.assert_tree_equal(got, want, w.n)


def test_70b_shape_batched_subset():
    # full per-sequence shape (V=32000, d=10, k=8, n=60), 4 of the 16 sequences: the oracle stays in seconds
    w = wl.WORKLOADS["70b"]
    seed, logits, want = U.gapped_logits(w, 0, seqs=[0, 5, 10, 15])
    got = _run(logits, w.dtype, w.k, w.n, w.depth)
    U.assert_tree_equal(got, want, w.n)


def test_70b_full_batch_as_the_bench_launches_it():
    # all 16 sequences in one launch; sequences 0, 5, 10, 15 against the oracle, the invariants on every one
    w = wl.WORKLOADS["70b"]
    seed, _, want = U.gapped_logits(w, 0, seqs=[0, 5, 10, 15])
    logits = wl.make_logits(w, seed)
    got = _run(logits, w.dtype, w.k, w.n, w.depth)
    U.assert_tree_invariants(got, w.n, w.depth)
    import torch
    from paper_2406_17276_amd import api
    sub = api.alloc_tree(4, w.n)
    idx = torch.tensor([0, 5, 10, 15], device="cuda")
    for name in ("token", "parent", "depth", "score", "mask", "n_out", "expect"):
        getattr(sub, name).copy_(getattr(got, name)[idx])
    U.assert_tree_equal(sub, want, w.n)


@pytest.mark.timeout(900)
def test_large_budget_shape_full_depth_against_the_oracle():
    # The Large workload's own configuration for one sequence: vocabulary 128256 (four scan parts), k = 16, n = 256,
    # all 20 drafting steps, logits 5 N(0,1) with planted peaks.  The oracle needs about a minute for the 4625 rows.
    w = wl.WORKLOADS["large"]
    print("large, full depth: drawing the logits and running the oracle", flush=True)
    seed, logits, want = U.gapped_logits(w, 0, seqs=[0])
    print(f"large, full depth: seed {seed}, min gap {want[0]['min_gap']:.3g}; GPU build", flush=True)
    got = _run(logits, w.dtype, w.k, w.n, w.depth)
    assert want[0]["n_out"] == w.n
    U.assert_tree_equal(got, want, w.n)
    U.assert_tree_invariants(got, w.n, w.depth)


def test_large_budget_shape_full_depth_invariants():
    # n = 256, k = 16, 20 drafting steps, vocabulary 128256 (four scan parts): two more sequences, drawn on the
    # device, under the invariants of Algorithm 1's output (the oracle comparison at this size is the test above)
    import torch
    from paper_2406_17276_amd import api
    w = wl.WORKLOADS["large"]
    g = torch.Generator(device="cuda"); g.manual_seed(5)
    x = torch.empty((2, w.depth, w.n, w.vocab), dtype=torch.bfloat16, device="cuda")
    for t in range(w.depth):                                          # step by step: keeps the fp32 temporary small
        x[:, t] = (torch.randn((2, w.n, w.vocab), generator=g, device="cuda") * 3.0).to(torch.bfloat16)
    got = api.build_tree(x, w.k, w.n, w.depth)
    torch.cuda.synchronize()
    assert int(got.n_out.min()) == w.n
    U.assert_tree_invariants(got, w.n, w.depth)


def test_large_budget_shape_reduced_depth():
    # n=256 (4 mask words, 4 wavefronts), k=16, vocab 128256 split over 4 scan parts; 1 sequence, and
    # 6 instead of 20 drafting steps so that the oracle finishes in ~20 s
    import dataclasses
    w = dataclasses.replace(wl.WORKLOADS["large"], depth=6)
    seed, logits, want = U.gapped_logits(w, 0, seqs=[0])
    got = _run(logits, w.dtype, w.k, w.n, w.depth)
    U.assert_tree_equal(got, want, w.n)


def _random_case(V, k, n, d, B, dtype, seed, scale=3.0):
    g = np.random.default_rng(seed)
    for s in range(seed, seed + 16):
        x = (g.standard_normal((B, d, n, V)) * scale).astype(np.float32)
        stored = wl.store(x, dtype)
        want = U.oracle_trees(stored, dtype, k, n, d)
        if min(t["min_gap"] for t in want) > U.GAP:
            return stored, want
    raise RuntimeError("no gapped input")


@pytest.mark.parametrize("V,k,n,d,B,dtype", [
    (1000, 4, 16, 4, 3, "f32"),        # Tiny shape, batched
    (1001, 3, 7, 5, 2, "f32"),         # vocab not a multiple of the vector width -> scalar loads
    (777, 5, 33, 3, 2, "bf16"),
    (50, 16, 64, 3, 1, "f32"),         # k = 16, tiny vocab (most scan groups empty)
    (9000, 10, 50, 6, 2, "bf16"),      # 1024-thread scan with a ragged tail
    (40000, 6, 20, 4, 2, "bf16"),      # two scan parts + merge
    (70001, 2, 100, 9, 1, "f32"),      # three parts, unaligned vocab, 2 waves of selection
    (300, 1, 8, 5, 2, "f32"),          # k = 1: a chain, pool smaller than n
    (300, 4, 1, 3, 2, "f32"),          # n = 1
    (300, 2, 200, 4, 1, "f32"),        # n larger than the pool (2+4+8+16)
    (2048, 12, 130, 3, 2, "bf16"),     # 3 waves
    (512, 8, 256, 32, 1, "f32"),       # maximum n and depth
    (200, 16, 64, 26, 2, "f32"),       # one wavefront, but the row table exceeds LDS: general path
    (3000, 10, 64, 20, 1, "bf16"),     # one wavefront, deep tree, row table in LDS
    (400, 8, 60, 10, 16, "f32"),       # a batch of 70B-shaped trees
    (300, 16, 40, 2, 2, "f32"),        # depth 2: first cut at the second step
    (300, 3, 64, 7, 3, "f32"),         # frontier grows 1, 3, 9, 27, 64
    (300, 4, 64, 8, 50, "f32"),        # 17050 rows: more work items than workgroups (grid-stride scan)
    (262144, 16, 6, 2, 1, "bf16"),     # maximum vocabulary: eight scan parts per row, maximum k
])
def test_random_shapes_and_edges(V, k, n, d, B, dtype):
    stored, want = _random_case(V, k, n, d, B, dtype, seed=V + k + n)
    got = _run(stored, dtype, k, n, d)
    U.assert_tree_equal(got, want, n)


def test_constant_rows_exercise_every_tie_rule():
    # all logits equal: top-k ties by token id (candidate-list overflow path), layer cuts tie by
    # (parent slot, rank), the final cut ties by (depth, slot)
    for V, k, n, d, dtype in [(4096, 3, 10, 3, "f32"), (33000, 4, 9, 2, "bf16"), (64, 2, 5, 4, "f32")]:
        stored = wl.store(np.zeros((1, d, n, V), dtype=np.float32), dtype)
        want = U.oracle_trees(stored, dtype, k, n, d)
        got = _run(stored, dtype, k, n, d)
        U.assert_tree_equal(got, want, n)


def test_quantised_rows_with_many_exact_ties():
    g = np.random.default_rng(5)
    V, k, n, d = 5000, 8, 24, 4
    x = g.integers(-6, 7, size=(2, d, n, V)).astype(np.float32)      # 13 distinct values: huge tie groups
    x += (g.standard_normal((2, d, n, 1)) * 0.37).astype(np.float32)  # rows differ, ties inside rows stay
    stored = wl.store(x, "f32")
    want = U.oracle_trees(stored, "f32", k, n, d)
    assert min(t["min_gap"] for t in want) > U.GAP
    got = _run(stored, "f32", k, n, d)
    U.assert_tree_equal(got, want, n)


def test_strided_logits_view():
    import torch
    from paper_2406_17276_amd import api
    V, k, n, d, B = 1000, 4, 16, 4, 2
    stored, want = _random_case(V, k, n, d, B, "f32", seed=99)
    big = torch.zeros((B, d + 1, n + 3, V + 24), dtype=torch.float32, device="cuda")
    view = big[:, :d, :n, 8:8 + V]          # 16-byte aligned start, padded strides
    view.copy_(U.to_device(stored, "f32"))
    got = api.build_tree(view, k, n, d)
    torch.cuda.synchronize()
    U.assert_tree_equal(got, want, n)
    view2 = big[:, :d, :n, 3:3 + V]         # misaligned start: scalar-load path
    view2.copy_(U.to_device(stored, "f32"))
    got = api.build_tree(view2, k, n, d)
    torch.cuda.synchronize()
    U.assert_tree_equal(got, want, n)


def test_streaming_matches_oracle_layer_by_layer():
    """Drive expand() the way a decoder would: the rows of step t+1 depend on the frontier of step t."""
    import torch
    from paper_2406_17276_amd import api
    V, k, n, d, B = 3000, 5, 40, 6, 2

    def row_for(b, path):
        h = np.random.SeedSequence([1234, b, len(path)] + [int(p) + 1 for p in path])
        return (np.random.default_rng(h).standard_normal(V) * 3.0).astype(np.float32)

    builders = [ot_oracle.TreeBuilder(k, n) for _ in range(B)]
    paths = [[()] for _ in range(B)]
    stream = api.TreeStream(B, V, k, n, d, api.OT_F32)
    for t in range(d):
        F = len(paths[0])
        rows = np.zeros((B, n, V), dtype=np.float32)
        for b in range(B):
            for j, p in enumerate(paths[b]):
                rows[b, j] = row_for(b, p)
        ftok, fpar = stream.expand(torch.from_numpy(rows).cuda())
        torch.cuda.synchronize()
        ftok, fpar = ftok.cpu().numpy(), fpar.cpu().numpy()
        fcnt = stream.frontier_count.cpu().numpy()
        for b in range(B):
            tok, par = builders[b].expand(rows[b, :F].astype(np.float64))
            Fn = len(tok)
            assert fcnt[b] == Fn                       # rows the draft model owes for the next step
            np.testing.assert_array_equal(ftok[b, :Fn], tok)
            np.testing.assert_array_equal(fpar[b, :Fn], par)
            paths[b] = [paths[b][int(pj)] + (int(tk),) for tk, pj in zip(tok, par)]
    want = [bld.finalize() for bld in builders]
    assert min(wnt["min_gap"] for wnt in want) > U.GAP
    got = stream.finalize()
    torch.cuda.synchronize()
    U.assert_tree_equal(got, want, n)


def test_expected_length_grows_with_depth():
    # Thm. 3.2 on the GPU path: E of the depth-t tree is non-decreasing in t
    w = wl.WORKLOADS["tiny"]
    logits = wl.make_logits(w, 3)
    prev = 0.0
    for d in range(1, w.depth + 1):
        got = _run(logits, w.dtype, w.k, w.n, d)
        e = float(got.expect.cpu()[0])
        assert e >= prev - 1e-12
        prev = e


def test_repeated_calls_are_bit_identical():
    import torch
    w = wl.WORKLOADS["7b"]
    logits = wl.make_logits(w, 1)
    a = _run(logits, w.dtype, w.k, w.n, w.depth)
    for _ in range(3):
        b = _run(logits, w.dtype, w.k, w.n, w.depth)
        for f in ("token", "parent", "depth", "mask", "score", "expect"):
            assert torch.equal(getattr(a, f), getattr(b, f)), f


def test_adaptive_depth_matches_oracle():
    """Algorithm 1's loop through ot_tree_expand / ot_tree_esub / ot_tree_finalize: E_sub after every step,
    the go-on decision and the final tree of every sequence, for sequences that stop at different depths."""
    import torch
    from paper_2406_17276_amd import api
    V, k, n, dmax, B = 2000, 6, 30, 8, 5
    g = np.random.default_rng(77)
    # sequences differ in how peaked their rows are, hence in how fast E_sub saturates
    scales = np.array([0.5, 1.5, 3.0, 5.0, 8.0])
    delta = 0.01
    for attempt in range(8):
        x = (g.standard_normal((B, dmax, n, V)) * scales[:, None, None, None]).astype(np.float32)
        full = [ot_oracle.build_tree_adaptive(x[b].astype(np.float64), k, n, dmax, -1.0) for b in range(B)]
        gains = np.array([np.diff([0.0] + f["e_sub_trace"]) for f in full])
        margin = np.abs(gains - delta).min()              # no decision within rounding distance of delta
        want = [ot_oracle.build_tree_adaptive(x[b].astype(np.float64), k, n, dmax, delta) for b in range(B)]
        if margin > 1e-5 and min(w["min_gap"] for w in want) > U.GAP and len({w["steps"] for w in want}) >= 3:
            break
    else:
        raise RuntimeError("no suitable input")
    print("steps per sequence:", [w["steps"] for w in want], "delta", delta, flush=True)
    stream = api.TreeStream(B, V, k, n, dmax, api.OT_F32)
    dev = torch.from_numpy(x).cuda()
    active = [True] * B
    for t in range(dmax):
        stream.expand(dev[:, t])
        fcnt = stream.frontier_count.cpu().numpy()
        e_sub, go = stream.e_sub(delta)
        torch.cuda.synchronize()
        e_sub, go = e_sub.cpu().numpy(), go.cpu().numpy()
        for b in range(B):
            assert fcnt[b] == (min(n, k ** (t + 1)) if active[b] else 0)      # a stopped sequence asks for no rows
            if active[b]:
                assert e_sub[b] == pytest.approx(want[b]["e_sub_trace"][t], rel=1e-6)      # fp32 exp-sums behind every lse
                expect_go = t + 1 < want[b]["steps"] or (want[b]["steps"] == dmax and t + 1 == dmax and
                                                         np.diff([0.0] + want[b]["e_sub_trace"])[-1] > delta)
                assert bool(go[b]) == expect_go
                active[b] = bool(go[b])
            else:
                assert go[b] == 0
                assert e_sub[b] == pytest.approx(want[b]["e_sub_trace"][-1], rel=1e-6)    # frozen tree
        if not any(active):
            break
    got = stream.finalize()
    torch.cuda.synchronize()
    U.assert_tree_equal(got, want, n)


@pytest.mark.parametrize("V,k,n,d,B", [(1500, 4, 40, 7, 3),       # 280 pool indices: five mask words
                                       (600, 6, 100, 9, 2),       # 900 pool indices, two wavefronts per sequence
                                       (400, 16, 256, 20, 1)])    # the Large drafting shape: 5120 pool indices
def test_frontier_masks_of_the_drafting_phase_match_oracle(V, k, n, d, B):
    """ot_tree_frontier_mask after every expand: the incrementally kept ancestor masks over pool indices."""
    import torch
    from paper_2406_17276_amd import api
    for seed in range(5, 25):                              # inputs whose every cut has a gap the fp32 sums cannot flip
        g = np.random.default_rng(seed)
        x = (g.standard_normal((B, d, n, V)) * 3.0).astype(np.float32)
        want, builders = [], [ot_oracle.TreeBuilder(k, n) for _ in range(B)]
        for t in range(d):
            for b in range(B):
                F = builders[b].frontier_score.shape[0]
                builders[b].expand(x[b, t, :F].astype(np.float64))
            want.append([ot_oracle.frontier_masks(bld.layers, n, d) for bld in builders])
        if min(min(bld.cut_gaps) for bld in builders) > U.GAP:
            break
    else:
        raise RuntimeError("no gapped input")
    stream = api.TreeStream(B, V, k, n, d, api.OT_F32)
    dev = torch.from_numpy(x).cuda()
    for t in range(d):
        stream.expand(dev[:, t])
        m = stream.frontier_mask()
        torch.cuda.synchronize()
        m = m.cpu().numpy().view(np.uint64)
        for b in range(B):
            np.testing.assert_array_equal(m[b], want[t][b], err_msg=f"step {t}, sequence {b}")


@pytest.mark.parametrize("V,k,n,dmax,B,dtype,delta", [
    (2000, 6, 30, 8, 5, "f32", 0.01),
    (32000, 10, 50, 10, 2, "bf16", 0.02),      # 7B shape
    (500, 4, 64, 12, 3, "f32", 0.003),
    (900, 4, 100, 7, 4, "f32", 0.004),         # n > 64: the step-by-step form inside the call
    (3000, 16, 256, 5, 3, "bf16", 0.02),       # the widest frontier and k
    (70000, 3, 70, 6, 2, "f32", 0.01),         # rows of three scan parts
    (200, 16, 64, 26, 2, "f32", 0.002),        # one wavefront wide, but the row table exceeds LDS: step by step as well
])
def test_one_shot_adaptive_build_matches_oracle(V, k, n, dmax, B, dtype, delta):
    """ot_build_tree_adaptive: the stopping rule of Algorithm 1 applied inside the kernel."""
    import torch
    from paper_2406_17276_amd import api
    g = np.random.default_rng(V + n)
    scales = np.linspace(0.6, 7.0, B)
    for attempt in range(8):
        x = wl.store((g.standard_normal((B, dmax, n, V)) * scales[:, None, None, None]).astype(np.float32), dtype)
        x64 = wl.to_f64(x, dtype)
        full = [ot_oracle.build_tree_adaptive(x64[b], k, n, dmax, -1.0) for b in range(B)]
        gains = np.concatenate([np.diff([0.0] + f["e_sub_trace"]) for f in full])
        want = [ot_oracle.build_tree_adaptive(x64[b], k, n, dmax, delta) for b in range(B)]
        if np.abs(gains - delta).min() > 1e-5 and min(w["min_gap"] for w in want) > U.GAP:
            break
    else:
        raise RuntimeError("no suitable input")
    print("steps per sequence:", [w["steps"] for w in want], flush=True)
    got, steps, e_sub = api.build_tree_adaptive(U.to_device(x, dtype), k, n, dmax, delta)
    torch.cuda.synchronize()
    assert list(steps.cpu().numpy()) == [w["steps"] for w in want]
    np.testing.assert_allclose(e_sub.cpu().numpy(), [w["e_sub_trace"][-1] for w in want], rtol=1e-6)
    U.assert_tree_equal(got, want, n)


def test_one_shot_adaptive_build_with_a_threshold_nothing_passes_stops_after_one_step_at_any_width():
    import torch
    from paper_2406_17276_amd import api
    g = np.random.default_rng(5)
    x = g.standard_normal((2, 3, 100, 64)).astype(np.float32)
    got, steps, e_sub = api.build_tree_adaptive(torch.from_numpy(x).cuda(), 2, 100, 3, 10.0)
    torch.cuda.synchronize()
    assert list(steps.cpu().numpy()) == [1, 1]
    want = [ot_oracle.build_tree_adaptive(x[b].astype(np.float64), 2, 100, 3, 10.0) for b in range(2)]
    U.assert_tree_equal(got, want, 100)


@pytest.mark.parametrize("V,k,n,d,B,dtype,offset", [
    (8192, 4, 12, 3, 1, "bf16", 0), (8185, 4, 12, 3, 1, "bf16", 3),          # 256 threads: all of it; one vector too long
    (32768, 4, 12, 3, 1, "bf16", 0), (32761, 4, 12, 3, 1, "bf16", 5),        # 1024 threads, rows in registers
    (65536, 4, 12, 3, 1, "bf16", 8), (65529, 4, 12, 3, 1, "bf16", 1),        # rolling, 512 and 1024 threads
    (131072, 4, 12, 3, 1, "bf16", 0), (131065, 4, 12, 3, 1, "bf16", 7),      # one part; two
    (16385, 4, 12, 3, 1, "f32", 1), (32766, 16, 20, 3, 1, "f32", 2), (65533, 5, 12, 3, 1, "f32", 3),
    (8191, 16, 64, 7, 5, "bf16", 1),                                         # 1685 rows: rolling, 256 threads
    (4093, 16, 64, 7, 5, "f32", 3),
])
def test_scan_forms_at_the_ends_of_their_ranges_and_rows_at_any_alignment(V, k, n, d, B, dtype, offset):
    import torch
    from paper_2406_17276_amd import api
    stored, want = _random_case(V, k, n, d, B, dtype, seed=V + offset)
    dev = U.to_device(stored, dtype)
    big = torch.zeros((B, d, n, V + offset + (5 if V % 2 else 8)), dtype=dev.dtype, device="cuda")
    view = big[..., offset:offset + V]
    view.copy_(dev)
    got = api.build_tree(view, k, n, d)
    torch.cuda.synchronize()
    U.assert_tree_equal(got, want, n)


@pytest.mark.parametrize("V,B,dtype,offset,levels", [
    (16, 8, "f32", 0, 0), (61, 8, "bf16", 7, 0), (1000, 8, "f32", 1, 0), (1856, 8, "bf16", 0, 0),   # a wavefront per row ...
    (4096, 8, "bf16", 0, 0), (4089, 8, "bf16", 3, 0), (2048, 8, "f32", 0, 0), (2045, 8, "f32", 3, 0),   # ... its nearer end
    (8192, 37, "bf16", 0, 0), (8185, 37, "bf16", 5, 0), (4096, 37, "f32", 0, 0), (4093, 37, "f32", 1, 0),   # ... its farther end
    (3000, 8, "bf16", 1, 40), (3000, 8, "f32", 1, 2),              # 75 equal logits a level; more than the list holds
    (9000, 3, "bf16", 1, 0), (12000, 4, "f32", 2, 0),              # 256 threads from 768 and from 1125 rows on
])
def test_rows_in_great_numbers_match_the_same_rows_in_small_batches(V, B, dtype, offset, levels):
    """337 rows a sequence: all sequences at once take the forms for many rows, a sequence by itself the ones for few."""
    import torch
    from paper_2406_17276_amd import api
    k, n, d = 16, 64, 7
    g = torch.Generator(device="cuda")
    g.manual_seed(V + B)
    big = torch.randn((B, d, n, V + offset + (-(V + offset)) % 8), generator=g, device="cuda") * 3.0
    if levels:
        big = (big * levels / 24.0).round().clamp(-levels // 2, levels // 2)
    x = big.to(torch.bfloat16 if dtype == "bf16" else torch.float32)[..., offset:offset + V]
    got = api.build_tree(x, k, n, d)
    for b in range(0, B, max(1, B // 8)):
        want = api.build_tree(x[b:b + 1], k, n, d)
        torch.cuda.synchronize()
        for name in ("token", "parent", "depth", "mask", "n_out"):
            assert torch.equal(getattr(got, name)[b:b + 1], getattr(want, name)), (b, name)
        # both normalisers add up V terms in fp32 inside a vector and fp64 above it: 2^-24 times a few each
        torch.testing.assert_close(got.expect[b:b + 1], want.expect, rtol=2e-6, atol=0.0)


@pytest.mark.parametrize("k,n,d", [
    (16, 16, 6), (16, 17, 6),          # 256 candidates per step; more: 512 threads
    (16, 32, 5), (16, 33, 5),          # 512; two per thread
    (16, 64, 5), (16, 65, 5),          # 1024; 1024 threads
    (16, 128, 4), (16, 129, 4),        # 2048; four per thread
    (3, 85, 32),                       # 255 candidates, but a pool of more nodes than 256 threads take
    (16, 256, 32),                     # the largest pool
])
def test_selection_at_the_ends_of_each_number_of_threads(k, n, d):
    stored, want = _random_case(200, k, n, d, 2, "f32", seed=k + n + d, scale=2.0)
    got = _run(stored, "f32", k, n, d)
    U.assert_tree_equal(got, want, n)


@pytest.mark.parametrize("V,k,n,d,B", [
    (32000, 16, 256, 9, 2), (50001, 10, 200, 8, 2),       # one launch
    (32000, 16, 256, 24, 2), (50001, 10, 200, 16, 2),     # three; two, rows at odd addresses
])
def test_builds_in_several_launches_match_the_streaming_builder(V, k, n, d, B):
    """More than 384 MB of rows: the call goes in chunks of steps, the rows of finished sequences are left unread.  The
    streaming builder takes every step by itself."""
    import torch
    from paper_2406_17276_amd import api
    g = torch.Generator(device="cuda")
    g.manual_seed(V)
    x = torch.randn((B, d, n, V), generator=g, device="cuda")
    x *= torch.tensor([1.5, 5.0], device="cuda")[:, None, None, None]        # sequences that finish at different steps
    x = x.to(torch.bfloat16)
    for delta in (None, -1.0, 0.01, 0.3):
        ts = api.TreeStream(B, V, k, n, d, api.OT_BF16, "cuda")
        steps = torch.zeros(B, dtype=torch.int32)
        on = torch.ones(B, dtype=torch.bool)
        F = 1
        for t in range(d):
            ts.expand(x[:, t, :F].contiguous())
            F = min(n, k * F)
            steps += on.int()
            if delta is not None:
                _, go = ts.e_sub(delta)
                on &= go.cpu().bool()
        want = ts.finalize()
        if delta is None:
            got = api.build_tree(x, k, n, d)
        else:
            got, used, _ = api.build_tree_adaptive(x, k, n, d, delta)
            assert used.cpu().tolist() == steps.tolist()
        torch.cuda.synchronize()
        for name in ("token", "parent", "depth", "mask", "n_out"):
            assert torch.equal(getattr(got, name), getattr(want, name)), (delta, name)
        torch.testing.assert_close(got.expect, want.expect, rtol=1e-6, atol=0.0)


@pytest.mark.parametrize("V,k,n,d,B,dtype", [
    (300, 8, 12, 3, 2, "f32"), (20000, 16, 20, 3, 1, "bf16"),          # rows in registers: 256 and 1024 threads
    (40000, 16, 20, 3, 1, "bf16"), (8200, 16, 64, 7, 5, "bf16"),       # rolling: 512 threads; 256
    (140000, 16, 20, 3, 1, "bf16"),                                    # two parts and their merge
    (2500, 16, 16, 3, 1, "f32"),                                       # 1200 zeros: more candidates than the list holds
])
def test_zeros_of_either_sign_are_equal_logits(V, k, n, d, B, dtype):
    """Equal logits: the smaller token id first, so a -0 precedes a +0 of a larger token."""
    zeros = 1200 if V == 2500 else 24
    for seed in range(V, V + 16):
        g = np.random.default_rng(seed)
        x = -1.0 - np.abs(g.standard_normal((B, d, n, V)).astype(np.float32))
        for row in x.reshape(-1, V):
            row[g.choice(V, zeros, replace=False)] = np.where(g.random(zeros) < 0.5, np.float32(0.0), np.float32(-0.0))
        stored = wl.store(x, dtype)
        want = U.oracle_trees(stored, dtype, k, n, d)
        if min(t["min_gap"] for t in want) > U.GAP:
            break
    else:
        raise RuntimeError("no gapped input")
    U.assert_tree_equal(_run(stored, dtype, k, n, d), want, n)


@pytest.mark.parametrize("B,V,dtype", [
    (256, 32000, "bf16"), (64, 8000, "f32"),             # rows in registers
    (2048, 32000, "bf16"), (1600, 15000, "f32"),         # rolling: 256 threads
    (128, 60000, "bf16"), (64, 120000, "bf16"),          # 512, 1024
    (64, 200000, "bf16"), (64, 70000, "f32"),            # two parts
])
@pytest.mark.parametrize("sigma,peak", [(1.0, 0.0), (4.0, 6.0), (2.0, 20.0), (2.0, 30.0), (3.0, 40.0)])
def test_normaliser_of_flat_and_of_confident_rows(B, V, dtype, sigma, peak):
    """A tree of one node has E = p of its token, so log E = x - lse to the precision of the normaliser.  The term that
    dominates errs by 2^-23 (v_exp_f32, one unit in the last place) and by 2^-24 for the rounding of an exponent near 0;
    the fp32 additions on its way (13 at most) err by half a unit of a sum each, 2^-24 x sqrt(13) at random: 4e-7.  The
    sigma = 2, peak = 20 rows (one element among thousands that weigh as much) come closest."""
    import torch
    from paper_2406_17276_amd import api
    g = torch.Generator(device="cuda")
    g.manual_seed(B + V)
    x = torch.randn((B, V), generator=g, device="cuda") * sigma
    x[torch.arange(B, device="cuda"), torch.randint(0, V, (B,), generator=g, device="cuda")] += peak
    x = x.to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    ts = api.TreeStream(B, V, 1, 1, 1, api.OT_BF16 if dtype == "bf16" else api.OT_F32, "cuda")
    ts.expand(x[:, None, :])
    got = ts.finalize().expect.log()
    worst = 0.0
    for b in range(0, B, 128):
        y = x[b:b + 128].double()
        worst = max(worst, float((got[b:b + 128] - (y.max(1).values - torch.logsumexp(y, 1))).abs().max()))
    print(f"largest error of a normaliser: {worst:.2e}", flush=True)
    assert worst < 5e-7


@pytest.mark.parametrize("V,k,n,d", [(3000, 10, 50, 7), (3000, 10, 65, 7), (1000, 4, 200, 9), (1000, 16, 256, 6)])
def test_one_shot_and_streaming_builds_agree_on_e(V, k, n, d):
    """Both forms scan these rows the same way and add up p^ = e^(log p^) in fp64 over the same nodes, so E and E_sub differ
    by the order of at most 256 additions (2^-53 each) and by a unit or two of exp: 1e-13."""
    import torch
    from paper_2406_17276_amd import api
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    x = torch.randn((2, d, n, V), generator=g, device="cuda") * 3.0
    ts = api.TreeStream(2, V, k, n, d, api.OT_F32, "cuda")
    F = 1
    for t in range(d):
        ts.expand(x[:, t, :F].contiguous())
        F = min(n, k * F)
        e_sub, _ = ts.e_sub(-1.0)
    want = ts.finalize()
    got = api.build_tree(x, k, n, d)
    adaptive, _, got_sub = api.build_tree_adaptive(x, k, n, d, -1.0)
    torch.cuda.synchronize()
    assert torch.equal(got.token, want.token) and torch.equal(adaptive.token, want.token)
    for value, ref in ((got.expect, want.expect), (adaptive.expect, want.expect), (got_sub, e_sub)):
        torch.testing.assert_close(value, ref, rtol=1e-13, atol=0.0)


@pytest.mark.parametrize("k,n,d,dtype", [(4, 4, 10, "f32"), (4, 4, 32, "bf16"), (3, 20, 32, "f32"), (16, 64, 20, "f32"), (2, 80, 32, "f32")])
def test_streaming_tree_of_rows_with_one_token(k, n, d, dtype):
    """log p of a row's only token is 0 but for the rounding of the normaliser, above or below: no child comes before its parent."""
    import torch
    from paper_2406_17276_amd import api
    B, V = 4, 1000
    g = torch.Generator(device="cuda").manual_seed(n + d)
    x = torch.zeros((B, d, n, V), device="cuda")
    x.scatter_(3, torch.randint(0, V, (B, d, n, 1), generator=g, device="cuda"),
               30 + 60 * torch.rand((B, d, n, 1), generator=g, device="cuda"))
    x = x.to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    ts = api.TreeStream(B, V, k, n, d, api.OT_BF16 if dtype == "bf16" else api.OT_F32, "cuda")
    for t in range(d):
        ts.expand(x[:, t])
    got = ts.finalize()
    want = api.build_tree(x, k, n, d)
    torch.cuda.synchronize()
    U.assert_tree_invariants(got, n, d)
    for f in ("token", "parent", "depth", "mask", "n_out"):
        assert torch.equal(getattr(got, f), getattr(want, f)), f


def test_builds_of_more_threads_than_a_grid_holds():
    """2^24 + 3 sequences of one row: at 256 threads each more than 2^32 threads, in the scan as in the tree kernel."""
    import torch
    from paper_2406_17276_amd import api
    B, V = (1 << 24) + 3, 16
    x = torch.arange(V, device="cuda", dtype=torch.bfloat16).mul_(0.5).repeat(B, 1)
    best = torch.randint(0, V, (B,), generator=torch.Generator(device="cuda").manual_seed(5), device="cuda")
    x.scatter_(1, best[:, None], 9.0)
    want = torch.softmax(x[-4:].double(), 1).gather(1, best[-4:, None])[:, 0]
    for build in (lambda: api.build_tree(x[:, None, None], 1, 1, 1), lambda: api.build_tree_adaptive(x[:, None, None], 1, 1, 1, 0.1)[0]):
        tree = build()
        assert torch.equal(tree.token[:, 0], best.int())
        assert bool((tree.n_out == 1).all()) and bool((tree.parent == -1).all()) and bool((tree.mask == 1).all())
        torch.testing.assert_close(tree.expect[-4:], want, rtol=1e-6, atol=0.0)
        del tree
