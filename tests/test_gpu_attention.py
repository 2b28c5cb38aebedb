"""Parity of ot_tree_verify_attention with the fp64 oracle (needs an MI355X).
Bars: max-abs 1e-5 for f32 inputs, 2e-2 for bf16 inputs, against fp64 on the stored (rounded) inputs."""
import numpy as np
import pytest

from oracle import opt_tree as ot_oracle
from oracle import tree_attention as ta_oracle
import workloads as wl
from tests import _util as U

pytestmark = pytest.mark.gpu
TOL = {"f32": 1e-5, "bf16": 2e-2}


def _gpu_attention(x, mask, dtype, scale=0.0):
    import torch
    from paper_2406_17276_amd import api
    dev = {k: U.to_device(v, dtype) for k, v in x.items() if k != "prefix_len"}
    plen = torch.from_numpy(x["prefix_len"].astype(np.int32)).cuda()
    kp, vp = dev["K_prefix"], dev["V_prefix"]
    out = api.tree_verify_attention(dev["Q"], kp, vp, dev["K_tree"], dev["V_tree"], plen, U.mask_to_device(mask),
                                    softmax_scale=scale)
    torch.cuda.synchronize()
    return U.from_device_f64(out)


def _oracle_attention(x, mask, dtype, scale=None):
    f = {k: wl.to_f64(v, dtype) for k, v in x.items() if k != "prefix_len"}
    return ta_oracle.tree_verify_attention(f["Q"], f["K_prefix"], f["V_prefix"], f["K_tree"], f["V_tree"],
                                           x["prefix_len"], mask, scale)


def _shape(dtype, B, Hq, Hkv, D, L, n, ragged=0.0, name="t"):
    return wl.Workload(name, B, 8, 1, 1, n, dtype, "normal", 1.0, Hq, Hkv, D, L, ragged=ragged)


def _random_masks(B, n, seed, shape="random"):
    return np.stack([ot_oracle.ancestor_mask(wl.random_tree_parents(n, seed + b, shape)) for b in range(B)])


@pytest.mark.parametrize("name", ["tiny", "7b"])
def test_full_config_with_the_tree_built_by_the_oracle(name):
    w = wl.WORKLOADS[name]
    logits = wl.make_logits(w, 0)
    tree = U.oracle_trees(logits, w.dtype, w.k, w.n, w.depth)[0]
    mask = tree["mask"][None]
    x = wl.make_attention_inputs(w, 0)
    got = _gpu_attention(x, mask, w.dtype)
    want = _oracle_attention(x, mask, w.dtype)
    assert np.abs(got - want).max() < TOL[w.dtype]


def test_13b_shape_sampled_heads():
    # full shape on the GPU; the oracle checks 6 of the 40 heads
    w = wl.WORKLOADS["13b"]
    x = wl.make_attention_inputs(w, 1)
    mask = _random_masks(1, w.n, 7)
    got = _gpu_attention(x, mask, w.dtype)
    heads = [0, 7, 13, 22, 31, 39]
    sub = {k: (v[:, heads] if k != "prefix_len" else v) for k, v in x.items()}
    want = _oracle_attention(sub, mask, w.dtype)
    assert np.abs(got[:, heads] - want).max() < TOL[w.dtype]


def test_70b_shape_gqa_ragged_sampled():
    # GQA 64/8 heads, ragged prefixes around 4096, n=60; 3 sequences on the GPU, oracle on 2 KV groups of each
    w = wl.WORKLOADS["70b"]
    seqs = [0, 7, 12]
    x = wl.make_attention_inputs(w, 2, seqs=seqs)
    mask = _random_masks(len(seqs), w.n, 11)
    got = _gpu_attention(x, mask, w.dtype)
    g = w.q_heads // w.kv_heads
    for kvh in (1, 6):
        qh = list(range(kvh * g, kvh * g + g))
        sub = dict(Q=x["Q"][:, qh], K_prefix=x["K_prefix"][:, [kvh]], V_prefix=x["V_prefix"][:, [kvh]],
                   K_tree=x["K_tree"][:, [kvh]], V_tree=x["V_tree"][:, [kvh]], prefix_len=x["prefix_len"])
        want = _oracle_attention(sub, mask, w.dtype)
        assert np.abs(got[:, qh] - want).max() < TOL[w.dtype]


def test_large_budget_shape_one_kv_group():
    # n = 256 (4 mask words), 32/8 heads, prefix 8192: 1 sequence on the GPU, oracle on one KV group
    w = wl.WORKLOADS["large"]
    x = wl.make_attention_inputs(w, 3, seqs=[0])
    mask = _random_masks(1, w.n, 5)
    got = _gpu_attention(x, mask, w.dtype)
    qh = [8, 9, 10, 11]
    sub = dict(Q=x["Q"][:, qh], K_prefix=x["K_prefix"][:, [2]], V_prefix=x["V_prefix"][:, [2]],
               K_tree=x["K_tree"][:, [2]], V_tree=x["V_tree"][:, [2]], prefix_len=x["prefix_len"])
    want = _oracle_attention(sub, mask, w.dtype)
    assert np.abs(got[:, qh] - want).max() < TOL[w.dtype]


def _stored(t):
    """Device bf16 tensor -> host array of bf16 bit patterns (the stored form the oracle helpers take)."""
    import torch
    return t.contiguous().view(torch.int16).cpu().numpy().view(np.uint16)


@pytest.mark.parametrize("name,groups", [
    ("70b", [(0, 0), (3, 5), (9, 2), (15, 7)]),        # 16 sequences, GQA 64/8, ragged prefixes around 4096, n = 60
    ("large", [(0, 3), (31, 6)]),                      # 32 sequences, 32/8 heads, prefix 8192, n = 256
])
def test_full_batch_as_the_bench_launches_it_sampled_groups(name, groups):
    """The whole batch in one launch, inputs drawn on the device; the oracle recomputes sampled (sequence, KV head)
    groups from the slices it needs."""
    import torch
    from paper_2406_17276_amd import api
    w = wl.WORKLOADS[name]
    B, g = w.batch, w.q_heads // w.kv_heads
    gen = torch.Generator(device="cuda"); gen.manual_seed(17)
    draw = lambda *shape: torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16)
    Lmax = w.max_prefix()
    Q = draw(B, w.q_heads, w.n, w.head_dim)
    Kp, Vp = draw(B, w.kv_heads, Lmax, w.head_dim), draw(B, w.kv_heads, Lmax, w.head_dim)
    Kt, Vt = draw(B, w.kv_heads, w.n, w.head_dim), draw(B, w.kv_heads, w.n, w.head_dim)
    plen = wl.prefix_lengths(w, 4).astype(np.int32)
    mask = _random_masks(B, w.n, 23)
    out = api.tree_verify_attention(Q, Kp, Vp, Kt, Vt, torch.from_numpy(plen).cuda(), U.mask_to_device(mask))
    torch.cuda.synchronize()
    assert bool(torch.isfinite(out.float()).all())
    for b, kvh in groups:
        qh = slice(kvh * g, kvh * g + g)
        sub = dict(Q=_stored(Q[b:b + 1, qh]), K_prefix=_stored(Kp[b:b + 1, kvh:kvh + 1]),
                   V_prefix=_stored(Vp[b:b + 1, kvh:kvh + 1]), K_tree=_stored(Kt[b:b + 1, kvh:kvh + 1]),
                   V_tree=_stored(Vt[b:b + 1, kvh:kvh + 1]), prefix_len=plen[b:b + 1])
        want = _oracle_attention(sub, mask[b:b + 1], "bf16")
        got = U.from_device_f64(out[b:b + 1, qh])
        print(f"{name}: sequence {b}, KV head {kvh}: max-abs err {np.abs(got - want).max():.2e}", flush=True)
        assert np.abs(got - want).max() < TOL["bf16"]


@pytest.mark.parametrize("B,Hq,Hkv,D,n,lengths,plan", [
    (33, 16, 8, 128, 40, "ragged", (128, 1, 1)),        # 128-row blocks, 264 workgroups: one more round than the chip holds at once
    (64, 8, 4, 128, 70, "ragged", (256, 1, 1)),         # 256-row blocks, 256 workgroups, the largest batch that is ranked
    (40, 16, 8, 64, 33, "ties", (128, 1, 1)),           # head_dim 64; many equal lengths, some zero, some beyond the buffer
    (65, 8, 4, 128, 70, "ragged", (256, 1, 0)),         # one sequence too many for the ranking: the order of the sequences
])
def test_batches_that_take_their_jobs_longest_first(B, Hq, Hkv, D, n, lengths, plan):
    """Batches that fill the chip with one key range per (sequence, KV head): every workgroup ranks the sequences by
    prefix length on the device and takes its job in that order.  Whatever the order, every (sequence, KV head) must
    come out exactly once: all outputs are finite and non-zero, and sampled sequences (the longest, the shortest, ties,
    clamped ones) agree with the oracle."""
    import torch
    from paper_2406_17276_amd import api
    Lmax, g = 448, Hq // Hkv
    assert U.attention_plan(B, Hq, Hkv, D, n, Lmax) == plan
    rng = np.random.default_rng(B * 1000 + n)
    if lengths == "ragged":
        plen = rng.integers(1, Lmax + 1, size=B).astype(np.int32)
        plen[0], plen[B // 2], plen[B - 1] = Lmax, 1, Lmax // 2
    else:
        plen = rng.choice(np.array([0, 64, 64, 128, 200, 200, 200, Lmax], dtype=np.int32), size=B)
        plen[1], plen[2] = Lmax + 500, -7                     # clamped to Lmax and to 0 on the device
    eff = np.clip(plen, 0, Lmax)
    gen = torch.Generator(device="cuda"); gen.manual_seed(B + n)
    draw = lambda *shape: torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16)
    Q = draw(B, Hq, n, D)
    Kp, Vp = draw(B, Hkv, Lmax, D), draw(B, Hkv, Lmax, D)
    Kt, Vt = draw(B, Hkv, n, D), draw(B, Hkv, n, D)
    mask = _random_masks(B, n, 31)
    out = api.tree_verify_attention(Q, Kp, Vp, Kt, Vt, torch.from_numpy(plen).cuda(), U.mask_to_device(mask))
    torch.cuda.synchronize()
    of = out.float()
    assert bool(torch.isfinite(of).all())
    assert bool((of.abs().amax(dim=(2, 3)) > 0).all())          # no (sequence, head) was left out
    order = np.argsort(-eff, kind="stable")
    picks = sorted({int(order[0]), int(order[1]), int(order[B // 2]), int(order[-1]), 1, 2, B - 1})
    for b in picks:
        for kvh in (0, Hkv - 1):
            qh = slice(kvh * g, kvh * g + g)
            sub = dict(Q=_stored(Q[b:b + 1, qh]), K_prefix=_stored(Kp[b:b + 1, kvh:kvh + 1]),
                       V_prefix=_stored(Vp[b:b + 1, kvh:kvh + 1]), K_tree=_stored(Kt[b:b + 1, kvh:kvh + 1]),
                       V_tree=_stored(Vt[b:b + 1, kvh:kvh + 1]), prefix_len=eff[b:b + 1])
            want = _oracle_attention(sub, mask[b:b + 1], "bf16")
            got = U.from_device_f64(out[b:b + 1, qh])
            assert np.abs(got - want).max() < TOL["bf16"], (b, kvh, int(plen[b]))


@pytest.mark.parametrize("dtype,B,Hq,Hkv,D,L,n,ragged,shape", [
    ("f32", 2, 4, 4, 64, 128, 16, 0.0, "random"),
    ("f32", 2, 6, 2, 128, 77, 37, 0.3, "random"),      # GQA, ragged, n not a multiple of 16
    ("f32", 1, 2, 2, 64, 0, 20, 0.0, "random"),        # empty prefix
    ("f32", 1, 2, 1, 64, 300, 130, 0.0, "chain"),      # three mask words, chain = causal
    ("bf16", 2, 4, 4, 128, 200, 50, 0.2, "random"),
    ("bf16", 1, 8, 2, 128, 1000, 60, 0.0, "random"),   # packed GQA rows span several 64-row blocks
    ("bf16", 2, 4, 2, 64, 129, 33, 0.5, "random"),     # head_dim 64, ragged tails
    ("bf16", 1, 2, 2, 128, 0, 70, 0.0, "star"),        # empty prefix, two tree tiles
    ("bf16", 1, 4, 1, 128, 64, 256, 0.0, "random"),    # maximum n
    ("bf16", 1, 1, 1, 128, 5000, 1, 0.0, "random"),    # a single node
    ("bf16", 2, 4, 4, 64, 300, 40, 0.3, "random"),     # head_dim 64, 64-row workgroups, several splits
    ("bf16", 3, 2, 2, 128, 2000, 20, 0.9, "random"),   # very ragged: short sequences leave splits empty
    ("bf16", 1, 16, 1, 128, 700, 30, 0.0, "random"),   # 128-row workgroups, several splits, ragged last row block
])
def test_shapes_and_edges(dtype, B, Hq, Hkv, D, L, n, ragged, shape):
    w = _shape(dtype, B, Hq, Hkv, D, L, n, ragged)
    x = wl.make_attention_inputs(w, 4)
    mask = _random_masks(B, n, 3, shape)
    got = _gpu_attention(x, mask, dtype)
    want = _oracle_attention(x, mask, dtype)
    assert np.abs(got - want).max() < TOL[dtype]


def test_softmax_scale_override_and_unnormalised_inputs():
    w = _shape("f32", 1, 2, 2, 64, 90, 12)
    x = wl.make_attention_inputs(w, 6)
    x["Q"] = (x["Q"] * 4.0).astype(np.float32)          # large logits: exercises the running max
    mask = _random_masks(1, 12, 1)
    got = _gpu_attention(x, mask, "f32", scale=0.05)
    want = _oracle_attention(x, mask, "f32", scale=0.05)
    assert np.abs(got - want).max() < 1e-5


def test_strided_kv_cache_views():
    import torch
    from paper_2406_17276_amd import api
    w = _shape("bf16", 2, 4, 2, 128, 150, 24)
    x = wl.make_attention_inputs(w, 8)
    mask = _random_masks(2, 24, 2)
    want = _oracle_attention(x, mask, "bf16")
    dev = {k: U.to_device(v, "bf16") for k, v in x.items() if k != "prefix_len"}
    Lmax = dev["K_prefix"].shape[2]
    cache_k = torch.zeros((2, 2, Lmax + 40, 128 + 64), dtype=torch.bfloat16, device="cuda")
    cache_v = torch.zeros_like(cache_k)
    kview, vview = cache_k[:, :, 8:8 + Lmax, 64:], cache_v[:, :, 8:8 + Lmax, 64:]
    kview.copy_(dev["K_prefix"]); vview.copy_(dev["V_prefix"])
    plen = torch.from_numpy(x["prefix_len"]).cuda()
    out = api.tree_verify_attention(dev["Q"], kview, vview, dev["K_tree"], dev["V_tree"], plen, U.mask_to_device(mask))
    torch.cuda.synchronize()
    assert np.abs(U.from_device_f64(out) - want).max() < 2e-2


def test_prefix_length_is_clamped_on_device():
    w = _shape("f32", 1, 2, 2, 64, 40, 8)
    x = wl.make_attention_inputs(w, 9)
    mask = _random_masks(1, 8, 4)
    want = _oracle_attention(x, mask, "f32")
    y = dict(x); y["prefix_len"] = np.array([10_000], dtype=np.int32)
    got = _gpu_attention(y, mask, "f32")
    assert np.abs(got - want).max() < 1e-5


@pytest.mark.parametrize("dtype,D,L,n", [("f32", 64, 40, 8), ("bf16", 128, 300, 20)])
def test_clamped_prefix_length_is_reported_in_the_workspace_status_word(dtype, D, L, n):
    """A length outside [0, max_prefix] is clamped and sets bit 0 of the workspace's status word, which stays set
    until the workspace is prepared again; in-range lengths leave it clear."""
    import torch
    from paper_2406_17276_amd import api
    w = _shape(dtype, 3, 4, 2, D, L, n)
    x = wl.make_attention_inputs(w, 21)
    mask = _random_masks(3, n, 5)
    dev = {k: U.to_device(v, dtype) for k, v in x.items() if k != "prefix_len"}
    p = api.attn_params(dev["Q"], dev["K_prefix"], dev["V_prefix"], dev["K_tree"], dev["V_tree"])
    ws = api.attn_workspace(p, "cuda")
    call = lambda plen: api.tree_verify_attention(dev["Q"], dev["K_prefix"], dev["V_prefix"], dev["K_tree"], dev["V_tree"],
                                                  torch.tensor(plen, dtype=torch.int32, device="cuda"),
                                                  U.mask_to_device(mask), workspace=ws)
    good = call([L, L // 2, 0])
    assert api.attn_status(ws) == 0
    want = _oracle_attention(dict(x, prefix_len=np.array([L, L // 2, 0], dtype=np.int32)), mask, dtype)
    assert np.abs(U.from_device_f64(good) - want).max() < TOL[dtype]
    over = call([L, L + 1, 0])                                   # sequence 1 too long: clamped to L, flagged
    assert api.attn_status(ws) & api.OT_ATTN_STATUS_PREFIX_CLAMPED
    want = _oracle_attention(dict(x, prefix_len=np.array([L, L, 0], dtype=np.int32)), mask, dtype)
    assert np.abs(U.from_device_f64(over) - want).max() < TOL[dtype]
    call([L, L // 2, 0])
    assert api.attn_status(ws) & api.OT_ATTN_STATUS_PREFIX_CLAMPED        # sticky
    api._check(api.lib().ot_attn_workspace_prepare(ws.data_ptr(), ws.numel(), api._stream()), "prepare")
    call([L, -3, 0])                                             # negative: clamped to 0, flagged
    assert api.attn_status(ws) & api.OT_ATTN_STATUS_PREFIX_CLAMPED


def test_one_workspace_serves_consecutive_calls():
    """The split merge keeps ticket counters in the workspace and must leave them zero: the same prepared
    workspace is used for three calls in a row, the last one on a smaller problem."""
    import torch
    from paper_2406_17276_amd import api
    big = _shape("bf16", 1, 4, 4, 128, 900, 50)
    small = _shape("bf16", 1, 2, 2, 128, 260, 17)
    ws = None
    for w, seed in [(big, 11), (big, 12), (small, 13)]:
        x = wl.make_attention_inputs(w, seed)
        mask = _random_masks(w.batch, w.n, seed)
        dev = {k: U.to_device(v, "bf16") for k, v in x.items() if k != "prefix_len"}
        plen = torch.from_numpy(x["prefix_len"].astype(np.int32)).cuda()
        p = api.attn_params(dev["Q"], dev["K_prefix"], dev["V_prefix"], dev["K_tree"], dev["V_tree"])
        if ws is None:
            ws = api.attn_workspace(p, "cuda")
        assert api.attn_workspace_bytes(p) <= ws.numel()
        out = api.tree_verify_attention(dev["Q"], dev["K_prefix"], dev["V_prefix"], dev["K_tree"], dev["V_tree"],
                                        plen, U.mask_to_device(mask), workspace=ws)
        torch.cuda.synchronize()
        want = _oracle_attention(x, mask, "bf16")
        assert np.abs(U.from_device_f64(out) - want).max() < 2e-2
        assert int(ws[:4096].view(torch.int32).abs().sum().item()) == 0


@pytest.mark.parametrize("dtype,B,Hq,Hkv,D,L,k,n,d,upto", [
    ("f32", 2, 4, 2, 64, 90, 3, 12, 5, 4),          # 60 pool rows, one mask word
    ("f32", 1, 4, 2, 64, 50, 10, 50, 12, 12),        # f32 beyond eight mask words: 600 pool keys
    ("f32", 1, 2, 2, 128, 33, 16, 256, 7, 7),        # f32, the largest frontier: 1792 pool keys, 28 words
    ("bf16", 1, 8, 8, 128, 700, 10, 50, 10, 10),     # 7B-shaped drafting step: 50 queries, 500 pool keys, 8 words
    ("bf16", 2, 8, 2, 128, 300, 6, 40, 8, 6),        # packed GQA rows (128-row workgroups), 320 pool keys
    ("bf16", 1, 4, 4, 64, 0, 4, 64, 8, 3),           # no prefix, 512 pool keys of which 3 layers are filled
    ("bf16", 1, 4, 4, 128, 2048, 10, 64, 12, 12),    # the 13B drafting shape (four of its heads): 768 pool keys
    ("bf16", 2, 16, 2, 128, 700, 8, 60, 10, 10),     # the 70B drafting shape (two of its KV heads): 600 pool keys
    ("bf16", 1, 8, 2, 128, 512, 16, 256, 20, 20),    # the Large drafting shape (two of its KV heads): 5120 pool keys
])
def test_drafting_phase_attention_frontier_against_pool(dtype, B, Hq, Hkv, D, L, k, n, d, upto):
    """n frontier queries against the prefix and the K/V of all pool nodes (n_keys = depth * n), with the
    frontier masks of the drafting phase."""
    import torch
    from paper_2406_17276_amd import api
    g = np.random.default_rng(n + d)
    masks = []
    for b in range(B):
        bld = ot_oracle.TreeBuilder(k, n)
        for t in range(upto):
            bld.expand(g.standard_normal((bld.frontier_score.shape[0], 200)) * 2.0)
        masks.append(ot_oracle.frontier_masks(bld.layers, n, d))
    mask = np.stack(masks)
    w = _shape(dtype, B, Hq, Hkv, D, L, n, 0.2 if L else 0.0)
    x = wl.make_attention_inputs(w, 21)
    nk = d * n
    x["K_tree"] = wl.store(g.standard_normal((B, Hkv, nk, D)).astype(np.float32), dtype)
    x["V_tree"] = wl.store(g.standard_normal((B, Hkv, nk, D)).astype(np.float32), dtype)
    got = _gpu_attention(x, mask, dtype)
    want = _oracle_attention(x, mask, dtype)
    assert np.abs(got - want).max() < TOL[dtype]
    assert np.abs(want).max() > 0.01


@pytest.mark.parametrize("D", [64, 128])
def test_256_rows_against_a_drafting_pool(D):
    """13 sequences of 8 KV heads of 240 rows, two key ranges each, over the prefix and 600 pool keys: the second range has
    tree tiles only where the prefix is short.  Random masks, a few rows of which see no pool key."""
    B, Hq, Hkv, n, nk, L = 13, 32, 8, 60, 600, 700
    assert U.attention_plan(B, Hq, Hkv, D, n, L, n_keys=nk) == (256, 2, 0)
    x = wl.make_attention_inputs(_shape("bf16", B, Hq, Hkv, D, L, nk), 12)
    x["Q"] = np.ascontiguousarray(x["Q"][:, :, :n])
    x["prefix_len"][:] = [[700, 1, 64, 130, 448, 0, 200][b % 7] for b in range(B)]
    rng = np.random.default_rng(3)
    mask = rng.integers(0, 2 ** 64, size=(B, n, 10), dtype=np.uint64) & rng.integers(0, 2 ** 64, size=(B, n, 10), dtype=np.uint64)
    mask[:, ::17] = 0
    got = _gpu_attention(x, mask, "bf16")
    seqs, heads = [0, 3, 5, 8, 12], [0, 7]
    q = [h * 4 + i for h in heads for i in range(4)]
    sub = {k: v[seqs] if k == "prefix_len" else v[seqs][:, q if k == "Q" else heads] for k, v in x.items()}
    assert np.abs(got[seqs][:, q] - _oracle_attention(sub, mask[seqs], "bf16")).max() < TOL["bf16"]


def test_repeated_launches_are_bit_identical():
    """Split-heavy shape, 300 launches on one prepared workspace: the merge inside the kernel adds the splits
    in a fixed order, so every launch must reproduce the first bit for bit, and the ticket counters end at zero."""
    import torch
    from paper_2406_17276_amd import api
    w = _shape("bf16", 1, 8, 8, 128, 1000, 50)
    x = wl.make_attention_inputs(w, 31)
    mask = _random_masks(1, 50, 9)
    dev = {k: U.to_device(v, "bf16") for k, v in x.items() if k != "prefix_len"}
    plen = torch.from_numpy(x["prefix_len"].astype(np.int32)).cuda()
    pa = api.PreparedAttention(dev["Q"], dev["K_prefix"], dev["V_prefix"], dev["K_tree"], dev["V_tree"], plen,
                               U.mask_to_device(mask))
    st = torch.cuda.current_stream().cuda_stream
    pa(st)
    torch.cuda.synchronize()
    first = pa.out.clone()
    assert np.abs(U.from_device_f64(first) - _oracle_attention(x, mask, "bf16")).max() < 2e-2
    for it in range(300):
        pa(st)
        if it % 50 == 49:
            torch.cuda.synchronize()
            assert torch.equal(pa.out, first)
    assert int(pa.ws[:4096].view(torch.int32).abs().sum().item()) == 0


@pytest.mark.parametrize("B,Hq,Hkv,n,L,rows", [(2, 8, 2, 25, 1000, 128), (8, 16, 8, 75, 2000, 256), (2, 4, 4, 70, 1000, 128)])
def test_scores_that_jump_between_tiles(B, Hq, Hkv, n, L, rows):
    """The 128- and 256-row variants keep a row's softmax reference fixed while scores stay within a slack of it and
    move it up otherwise: key bands whose scores differ by factors of up to 400 (beyond what 2^x can hold in fp32
    relative to the first band) force that path again and again, in the middle of a split."""
    assert U.attention_plan(B, Hq, Hkv, 128, n, L)[0] == rows
    w = _shape("bf16", B, Hq, Hkv, 128, L, n)
    x = wl.make_attention_inputs(w, 31)
    kp = wl.bf16_bits_to_f32(x["K_prefix"]).copy()
    for lo, f in [(0, 0.1), (200, 1.0), (400, 8.0), (600, 0.5), (800, 40.0), (930, 3.0)]:
        kp[:, :, lo:] = wl.bf16_bits_to_f32(x["K_prefix"])[:, :, lo:] * f
    x["K_prefix"] = wl.store(kp, "bf16")
    mask = _random_masks(B, n, 8)
    got = _gpu_attention(x, mask, "bf16")
    assert np.isfinite(got).all()
    some = [0, B - 1]
    assert np.abs(got[some] - _oracle_attention({k: v[some] for k, v in x.items()}, mask[some], "bf16")).max() < TOL["bf16"]


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("L", [0, 1, 63, 64, 65, 128, 191, 192, 256, 320, 447, 1000])
def test_256_row_loop_with_few_full_tiles_and_jumps_in_either_block(D, L):
    """33 sequences of 4 KV heads (no key splits), 150 rows each: no, one, two, ... full prefix tiles ahead of the general
    path, and in half of the sequences a key band of far larger scores that starts inside a tile's first or second block."""
    B, Hkv, n, Lmax = 33, 4, 150, 1000
    assert U.attention_plan(B, Hkv, Hkv, D, n, Lmax) == (256, 1, 1)          # the plan goes by the rows that the cache has
    w = _shape("bf16", B, Hkv, Hkv, D, Lmax, n)
    x = wl.make_attention_inputs(w, 5)
    x["prefix_len"][:] = L
    kp = wl.bf16_bits_to_f32(x["K_prefix"]).copy()
    for b in range(1, B, 2):
        for at in (64 * (b % 3) + 8 * b % 64, 64 * (b % 5) + 70, 64 * (b % 7) + 40):
            kp[b, :, at:at + 9] *= 40.0
    x["K_prefix"] = wl.store(kp, "bf16")
    mask = _random_masks(B, n, 8)
    got = _gpu_attention(x, mask, "bf16")
    assert np.isfinite(got).all()
    some = sorted({0, 1, 2, 3, 5, 9, 17, B - 1})
    sub = {k: v[some] for k, v in x.items()}
    # the oracle works in 64 bits on the stored values; O, up to 4, and p, averaged over a row's keys, are rounded to 8 bits
    assert np.abs(got[some] - _oracle_attention(sub, mask[some], "bf16")).max() < TOL["bf16"]


@pytest.mark.parametrize("D", [64, 128])
def test_an_infinite_value_makes_its_own_column_infinite(D):
    """256 rows: one V element of a fully visible tile is infinite, in either block of a first or a later tile, with and
    without scores that move the softmax reference up on the way.  Every key has weight, so the column is infinite and the
    others are what they are without it."""
    B, Hkv, n, Lmax = 33, 4, 150, 1000
    assert U.attention_plan(B, Hkv, Hkv, D, n, Lmax)[0] == 256
    x = wl.make_attention_inputs(_shape("bf16", B, Hkv, Hkv, D, Lmax, n), 5)
    x["prefix_len"][:] = [[64, 128, 200, 447, 1000][b % 5] for b in range(B)]
    at = [[3, 40, 63][b % 3] if b % 5 == 0 else [3, 40, 69, 110][b % 4] for b in range(B)]
    kp = wl.bf16_bits_to_f32(x["K_prefix"]).copy()
    for b in range(1, B, 2):
        kp[b, :, 20:29] *= 6.0
        kp[b, :, 64 * (b % 3) + 36:64 * (b % 3) + 45] *= 6.0
    x["K_prefix"] = wl.store(kp, "bf16")
    mask = _random_masks(B, n, 8)
    some = list(range(0, B, 4)) + [1, 3, 7, 11]
    want = _oracle_attention({k: v[some] for k, v in x.items()}, mask[some], "bf16")
    vp = wl.bf16_bits_to_f32(x["V_prefix"]).copy()
    for b in range(B):
        vp[b, :, at[b], 7 * b % D] = np.inf if b % 2 else -np.inf
    x["V_prefix"] = wl.store(vp, "bf16")
    got = _gpu_attention(x, mask, "bf16")
    for b in range(B):
        assert (got[b, :, :, 7 * b % D] == (np.inf if b % 2 else -np.inf)).all(), (b, at[b])
    for i, b in enumerate(some):
        keep = np.arange(D) != 7 * b % D
        assert np.abs(got[b] - want[i])[..., keep].max() < TOL["bf16"], b


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("n", [70, 150])               # 128 rows per workgroup; 256
def test_scores_that_round_by_more_than_the_slack(D, n):
    """Scores of 1e9 in units of log2 e: a tile's own maximum minus itself rounds to anything up to 32 (64 from 2^30 on), so
    its probability to 2^32, which must not send the loops over full tiles back to that tile for ever.  Each row ends up as
    the V of its best key."""
    assert U.attention_plan(33, 4, 4, D, n, 1000)[0] == (256 if n == 150 else 128)
    w = _shape("bf16", 33, 4, 4, D, 1000, n)
    x = wl.make_attention_inputs(w, 6)
    x["prefix_len"][:] = 500
    for k in ("K_prefix", "K_tree"):
        x[k] = wl.store(wl.bf16_bits_to_f32(x[k]) * 2e8, "bf16")
    mask = _random_masks(33, n, 2)
    got = _gpu_attention(x, mask, "bf16")
    some = [0, 13, 32]
    want = _oracle_attention({k: v[some] for k, v in x.items()}, mask[some], "bf16")
    assert np.abs(got[some] - want).max() < TOL["bf16"]


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("n,rows", [(70, 128), (150, 256)])
def test_first_keys_that_score_minus_infinity_have_no_weight(D, n, rows):
    """The keys up to somewhere inside or beyond the first 32-key block or tile score -inf against every row (as do a few
    later ones): weight zero, and the row goes on from the first finite score."""
    B, Hkv, Lmax = 33, 4, 1000
    assert U.attention_plan(B, Hkv, Hkv, D, n, Lmax)[0] == rows
    x = wl.make_attention_inputs(_shape("bf16", B, Hkv, Hkv, D, Lmax, n), 5)
    x["prefix_len"][:] = [[64, 128, 200, 447, 1000][b % 5] for b in range(B)]
    q, kp = wl.bf16_bits_to_f32(x["Q"]).copy(), wl.bf16_bits_to_f32(x["K_prefix"]).copy()
    q[..., 0] = np.abs(q[..., 0]) + 0.01
    for b in range(B):
        kp[b, :, :[1, 31, 32, 33, 63, 64, 96, 128, 190][b % 9], 0] = -np.inf
        kp[b, :, 300:340, 0] = -np.inf
    x["Q"], x["K_prefix"] = wl.store(q, "bf16"), wl.store(kp, "bf16")
    mask = _random_masks(B, n, 8)
    got = _gpu_attention(x, mask, "bf16")
    some = sorted(set(range(0, B, 3)) | set(range(9)))
    assert np.abs(got[some] - _oracle_attention({k: v[some] for k, v in x.items()}, mask[some], "bf16")).max() < TOL["bf16"]


def large_exact_scores(B, Hkv, D, L, n, seed, first=2.0 ** 13):
    """Scores 2^26 + x, x a multiple of 8 that grows along the keys: exact in fp32, while c times a score is rounded to a
    multiple of 1/2 or 1 (in units of log2 e).  Keys differ in weight by 2^(c x): q = (2^13, 1, 0, ...), k = (2^13, x, 0, ...)."""
    rng = np.random.default_rng(seed)
    x = wl.make_attention_inputs(_shape("bf16", B, Hkv, Hkv, D, L, n), seed)
    for name, rows, base in (("K_prefix", L, 0), ("K_tree", n, 8 * (L // 100) + 8)):
        k = np.zeros((B, Hkv, rows, D), dtype=np.float32)
        k[..., 0] = first
        k[..., 1] = base + 8 * (np.arange(rows) // 100) + 8 * rng.integers(-3, 3, size=(B, Hkv, rows))
        x[name] = k
    x["Q"] = np.zeros((B, Hkv, n, D), dtype=np.float32)
    x["Q"][..., 0], x["Q"][..., 1] = 2.0 ** 26 / first, 1.0
    return x


@pytest.mark.parametrize("dtype,B,Hkv,D,L,n,rows", [
    ("bf16", 1, 2, 64, 700, 40, 64), ("bf16", 33, 8, 128, 700, 40, 64),      # 64 rows: key ranges; halves of a tile only
    ("bf16", 33, 4, 128, 500, 70, 128), ("bf16", 33, 4, 64, 1000, 150, 256), ("bf16", 33, 4, 128, 1000, 150, 256),
    ("f32", 1, 2, 64, 1000, 40, 64), ("f32", 2, 2, 128, 60, 33, 32),         # fp32: ranges; slices that meet in LDS
])
def test_weights_are_kept_when_the_reference_of_large_scores_moves(dtype, B, Hkv, D, L, n, rows):
    assert U.attention_plan(B, Hkv, Hkv, D, n, L, dtype)[0] == rows
    x = large_exact_scores(B, Hkv, D, L, n, 4)
    x["V_prefix"], x["V_tree"] = [wl.bf16_bits_to_f32(x[k]) for k in ("V_prefix", "V_tree")]
    x = {k: v if k == "prefix_len" else wl.store(v, dtype) for k, v in x.items()}
    mask = _random_masks(B, n, 2)
    got = _gpu_attention(x, mask, dtype)
    some = sorted({0, B // 2, B - 1})
    # bf16: as elsewhere.  fp32: a weight is off by the rounding of c, 2^-24 of exponents up to 40, and by its own rounding
    assert np.abs(got[some] - _oracle_attention({k: v[some] for k, v in x.items()}, mask[some], dtype)).max() < TOL[dtype]


@pytest.mark.parametrize("B,Hq,Hkv,D,L,n", [
    *[(1, 2, 2, D, 64 * t, 100) for D in (64, 128) for t in (1, 2, 3, 4, 5, 6, 8, 10, 12, 14, 30)],    # 128 rows: one, a tile each, three, ...
    (1, 2, 2, 128, 64 * 3 + 1, 40), (1, 2, 2, 128, 64 * 5, 40), (1, 2, 2, 128, 64 * 6, 40),       # 64 rows: as many splits as tiles,
    (1, 2, 2, 128, 3000, 64), (1, 2, 1, 128, 3008, 32), (1, 2, 1, 128, 6100, 32),                 # one, two and three trips of six
    (1, 2, 2, 64, 256, 40), (1, 2, 2, 64, 257, 40), (1, 2, 2, 64, 2000, 40),                      # 64 wide: no split; six; twelve
    (8, 8, 8, 128, 2000, 150), (6, 16, 16, 64, 1300, 130),                                        # 256 rows, four splits; two
])
def test_key_splits_and_their_merge(B, Hq, Hkv, D, L, n):
    if B > 1:
        assert U.attention_plan(B, Hq, Hkv, D, n, L)[:2] == (256, 256 // (B * Hkv))
    w = _shape("bf16", B, Hq, Hkv, D, L, n)
    x = wl.make_attention_inputs(w, 3)
    x["prefix_len"][-1] = max(1, L // 3)                      # splits without a key, where there is a second sequence
    mask = _random_masks(B, n, 5)
    got = _gpu_attention(x, mask, "bf16")
    seqs, heads = sorted({0, B - 1}), sorted({0, Hkv - 1})
    q = [h * (Hq // Hkv) + i for h in heads for i in range(Hq // Hkv)]
    sub = {k: v[seqs] if k == "prefix_len" else v[seqs][:, q if k == "Q" else heads] for k, v in x.items()}
    assert np.abs(got[seqs][:, q] - _oracle_attention(sub, mask[seqs], "bf16")).max() < TOL["bf16"]


@pytest.mark.parametrize("D,n,L", [(128, 100, 9000), (64, 100, 20000), (64, 40, 12000)])
def test_more_ranges_where_the_workspace_holds_them(D, n, L):
    """One sequence over a long prefix with the fewest ranges, some, and the best number, as three workspaces allow."""
    import torch
    from paper_2406_17276_amd import api
    x = wl.make_attention_inputs(_shape("bf16", 1, 2, 2, D, L, n), 3)
    mask = _random_masks(1, n, 5)
    want = _oracle_attention(x, mask, "bf16")
    dev = {k: U.to_device(v, "bf16") for k, v in x.items() if k != "prefix_len"}
    plen, md = torch.from_numpy(x["prefix_len"].astype(np.int32)).cuda(), U.mask_to_device(mask)
    rows, most, _ = U.attention_plan(1, 2, 2, D, n, L)
    few = U.attention_plan(1, 2, 2, D, n, L, room=0)[1]
    assert few < most
    for splits in (few, (few + most) // 2, most):
        room = 4096 + 256 + 2 * rows * splits * (2 * D + 8)
        assert few <= U.attention_plan(1, 2, 2, D, n, L, room=room)[1] <= splits
        ws = torch.full((room,), 255, dtype=torch.uint8, device="cuda")
        api._check(api.lib().ot_attn_workspace_prepare(ws.data_ptr(), ws.numel(), api._stream()), "prepare")
        out = api.tree_verify_attention(dev["Q"], dev["K_prefix"], dev["V_prefix"], dev["K_tree"], dev["V_tree"], plen, md, workspace=ws)
        torch.cuda.synchronize()
        assert np.abs(U.from_device_f64(out) - want).max() < TOL["bf16"], splits


@pytest.mark.parametrize("L", [1, 63, 64, 65, 128, 129, 192, 700])
@pytest.mark.parametrize("B,n", [(32, 33), (33, 33), (33, 64)])
def test_64_rows_in_great_numbers(B, n, L):
    """256 and 264 (sequence, KV head) pairs around the line between three tile buffers and two; two to twelve tiles."""
    w = _shape("bf16", B, 8, 8, 128, L, n)
    x = wl.make_attention_inputs(w, 4)
    x["prefix_len"][-1] = L // 2
    mask = _random_masks(B, n, 6)
    got = _gpu_attention(x, mask, "bf16")
    some = [0, 17, B - 1]
    assert np.abs(got[some] - _oracle_attention({k: v[some] for k, v in x.items()}, mask[some], "bf16")).max() < TOL["bf16"]


@pytest.mark.parametrize("B,Hq,Hkv,D,L,n", [
    (1, 2, 2, 64, 31, 32),             # 32 rows per workgroup, eight key slices; key blocks one short
    (1, 2, 2, 128, 33, 33),            # 33 rows in blocks of 32; one key past a block
    (1, 2, 1, 64, 1, 32),              # 64 rows, a single prefix key
    (2, 2, 2, 64, 500, 65),            # 64-row workgroups, key ranges split and merged
    (1, 4, 1, 128, 1500, 64),          # 256 rows in blocks of 32, split
    (4, 64, 64, 64, 20, 65),           # enough workgroups without splits: 128 rows, two key slices
    (4, 64, 64, 128, 32, 64),          # 64 rows, four key slices
    (4, 64, 64, 128, 5, 10),           # 32 rows, fewer key blocks than slices
    (1, 1, 1, 64, 1, 1), (1, 2, 2, 128, 64, 20), (1, 2, 2, 128, 96, 40), (1, 2, 2, 64, 128, 30),     # 2 to 7 key blocks,
    (1, 2, 2, 128, 160, 31),           # slices without a block in the meeting
    (1, 2, 2, 128, 200, 31), (1, 2, 2, 128, 225, 31),     # eight blocks in one workgroup; nine, split
    (1, 2, 2, 64, 64, 60), (1, 2, 2, 64, 65, 60),         # the same with 64 rows per workgroup
    (1, 1, 1, 128, 4100, 16),          # as many splits as a row block can have
])
def test_f32_row_blocks_and_key_slices_at_their_edges(B, Hq, Hkv, D, L, n):
    w = _shape("f32", B, Hq, Hkv, D, L, n)
    x = wl.make_attention_inputs(w, 9)
    mask = _random_masks(B, n, 5)
    got = _gpu_attention(x, mask, "f32")
    heads = sorted(set(np.linspace(0, Hkv - 1, 5).astype(int)))       # the oracle takes some of the KV heads
    q = [h * (Hq // Hkv) + i for h in heads for i in range(Hq // Hkv)]
    sub = {k: v if k == "prefix_len" else v[:, q if k == "Q" else heads] for k, v in x.items()}
    want = _oracle_attention(sub, mask, "f32")
    assert np.abs(got[:, q] - want).max() < TOL["f32"]
