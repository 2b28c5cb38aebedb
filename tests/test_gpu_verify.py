"""Parity of ot_verify_greedy / ot_kv_append with the oracle (needs an MI355X).  Integer results and the
moved K/V rows must be bit-exact."""
import numpy as np
import pytest

from oracle import opt_tree as ot_oracle
from oracle import verify as vf
import workloads as wl
from tests import _util as U

pytestmark = pytest.mark.gpu


def _target_rows(tree, n, V, g, agree, dtype):
    """Target logits [n + 1, V] whose most probable token at a position is, with probability `agree`, the token
    of one of that position's children in the draft tree."""
    x = (g.standard_normal((n + 1, V)) * 2.0).astype(np.float32)
    for pos in range(-1, n):
        kids = [i for i in range(tree["n_out"]) if tree["parent"][i] == pos]
        t = int(tree["token"][g.choice(kids)]) if kids and g.random() < agree else int(g.integers(V))
        x[pos + 1, t] = 12.0
    return wl.store(x, dtype)


@pytest.mark.parametrize("V,k,n,d,B,dtype,agree", [
    (1000, 4, 16, 4, 3, "f32", 0.8),
    (32000, 10, 50, 10, 2, "bf16", 0.9),       # 7B shape: 51 target rows per sequence
    (40000, 5, 70, 6, 2, "bf16", 0.95),        # two scan parts, two wavefronts of nodes
    (300, 1, 8, 8, 2, "f32", 1.0),             # a chain, accepted whole: A = n + 1
    (300, 3, 200, 3, 1, "f32", 0.5),           # n larger than the tree (n_out < n)
    (2000, 8, 256, 6, 1, "bf16", 0.9),         # maximum n
    (32000, 8, 60, 10, 16, "bf16", 0.9),       # the 70B batch: 16 sequences, 61 target rows each
])
def test_verify_and_append_match_oracle(V, k, n, d, B, dtype, agree):
    import torch
    from paper_2406_17276_amd import api
    g = np.random.default_rng(V + n)
    draft = wl.store((g.standard_normal((B, d, n, V)) * 3.0).astype(np.float32), dtype)
    trees = U.oracle_trees(draft, dtype, k, n, d)
    target = np.stack([_target_rows(trees[b], n, V, g, agree, dtype) for b in range(B)])
    want = [vf.greedy_verify(wl.to_f64(target[b], dtype), trees[b]["token"], trees[b]["parent"], trees[b]["n_out"])
            for b in range(B)]
    print("accepted lengths:", [w[0] for w in want], flush=True)

    tree_dev = api.alloc_tree(B, n)
    tree_dev.token.copy_(torch.from_numpy(np.stack([t["token"] for t in trees]).astype(np.int32)))
    tree_dev.parent.copy_(torch.from_numpy(np.stack([t["parent"] for t in trees]).astype(np.int32)))
    tree_dev.n_out.copy_(torch.tensor([t["n_out"] for t in trees], dtype=torch.int32))
    alen, anode, atok = api.verify_greedy(U.to_device(target, dtype), tree_dev)
    torch.cuda.synchronize()
    alen, anode, atok = alen.cpu().numpy(), anode.cpu().numpy(), atok.cpu().numpy()
    for b in range(B):
        A, nodes, toks = want[b]
        assert alen[b] == A
        assert list(anode[b, :A - 1]) == nodes and np.all(anode[b, A - 1:] == -1)
        assert list(atok[b, :A]) == toks and np.all(atok[b, A:] == -1)

    # K/V append: 2 KV heads, head_dim 64, room for all but the longest branch of sequence 0
    H, D, L0 = 2, 64, 37
    cap = L0 + max(1, want[0][0] - 2)
    w = wl.Workload("v", B, 8, 1, 1, n, dtype, "normal", 1.0, H, H, D, cap)
    x = wl.make_attention_inputs(w, 5)
    plen = np.full(B, L0, dtype=np.int32)
    kp, vp = U.to_device(x["K_prefix"], dtype), U.to_device(x["V_prefix"], dtype)
    kt, vt = U.to_device(x["K_tree"], dtype), U.to_device(x["V_tree"], dtype)
    new_len = api.kv_append(kp, vp, kt, vt, torch.from_numpy(plen).cuda(),
                            torch.from_numpy(alen).cuda(), torch.from_numpy(anode).cuda())
    torch.cuda.synchronize()
    got_k, got_v = U.from_device_f64(kp), U.from_device_f64(vp)
    for b in range(B):
        Kp, Vp = wl.to_f64(x["K_prefix"][b], dtype).copy(), wl.to_f64(x["V_prefix"][b], dtype).copy()
        L = vf.kv_append(Kp, Vp, wl.to_f64(x["K_tree"][b], dtype), wl.to_f64(x["V_tree"][b], dtype), L0, want[b][1])
        assert int(new_len[b]) == L
        np.testing.assert_array_equal(got_k[b], Kp)
        np.testing.assert_array_equal(got_v[b], Vp)


# ---------------------------------------------------------------------------------------------------------
# Random sampling: ot_verify_sample.  The kernel sums exp2 terms in fp32 per 16-byte vector and in fp64 above
# (relative error of a cumulative probability ~1e-6), so the uniform numbers are drawn with a margin of 1e-5
# to every boundary of the oracle's CDF; the drawn tokens and the walk must then be bit-exact.
SAMPLE_MARGIN = 1e-5


def _uniforms_with_margin(rows64, T, g):
    u = np.empty(len(rows64), dtype=np.float32)
    for r, row in enumerate(rows64):
        for _ in range(100):
            u[r] = np.float32(g.random())
            if u[r] < 1.0 and vf.sample_margin(row, T, float(u[r])) > SAMPLE_MARGIN:
                break
        else:
            raise RuntimeError("no uniform number with a margin")
    return u


def _tree_to_device(api, trees, B, n):
    import torch
    tree_dev = api.alloc_tree(B, n)
    tree_dev.token.copy_(torch.from_numpy(np.stack([t["token"] for t in trees]).astype(np.int32)))
    tree_dev.parent.copy_(torch.from_numpy(np.stack([t["parent"] for t in trees]).astype(np.int32)))
    tree_dev.n_out.copy_(torch.tensor([t["n_out"] for t in trees], dtype=torch.int32))
    return tree_dev


@pytest.mark.parametrize("V,k,n,d,B,dtype,agree,T", [
    (1000, 4, 16, 4, 3, "f32", 0.8, 1.0),
    (32000, 10, 50, 10, 2, "bf16", 0.9, 1.0),      # 7B shape
    (40000, 5, 70, 6, 2, "bf16", 0.95, 0.7),
    (300, 3, 200, 3, 1, "f32", 0.5, 1.5),          # n larger than the tree
    (32000, 8, 60, 10, 16, "bf16", 0.9, 0.8),      # the 70B batch
])
def test_sampled_verification_matches_oracle(V, k, n, d, B, dtype, agree, T):
    import torch
    from paper_2406_17276_amd import api
    g = np.random.default_rng(7 * V + n)
    draft = wl.store((g.standard_normal((B, d, n, V)) * 3.0).astype(np.float32), dtype)
    trees = U.oracle_trees(draft, dtype, k, n, d)
    target = np.stack([_target_rows(trees[b], n, V, g, agree, dtype) for b in range(B)])
    t64 = wl.to_f64(target, dtype)
    u = np.stack([_uniforms_with_margin(t64[b], T, g) for b in range(B)])
    want = [vf.sampled_verify(t64[b], T, u[b].astype(np.float64), trees[b]["token"], trees[b]["parent"],
                              trees[b]["n_out"]) for b in range(B)]
    print("accepted lengths:", [w[0] for w in want], flush=True)
    alen, anode, atok = api.verify_sample(U.to_device(target, dtype), torch.from_numpy(u).cuda(), T,
                                          _tree_to_device(api, trees, B, n))
    torch.cuda.synchronize()
    alen, anode, atok = alen.cpu().numpy(), anode.cpu().numpy(), atok.cpu().numpy()
    for b in range(B):
        A, nodes, toks = want[b]
        assert alen[b] == A
        assert list(anode[b, :A - 1]) == nodes and np.all(anode[b, A - 1:] == -1)
        assert list(atok[b, :A]) == toks and np.all(atok[b, A:] == -1)


@pytest.mark.parametrize("V,n,B,dtype,T,scale,masked", [
    (32000, 50, 2, "bf16", 1.0, 2.0, 0),           # 7B shape
    (128256, 12, 1, "bf16", 0.8, 3.0, 0),          # 251 segments: four per lane of the picking wavefront
    (262144, 3, 1, "bf16", 1.0, 3.0, 0),           # the largest supported row: 512 segments, eight per lane
    (1001, 20, 2, "f32", 1.3, 1.0, 0),             # rows not 16-byte aligned: element loads, ragged last vector
    (1003, 7, 1, "bf16", 0.9, 2.0, 0),             # the same for bf16 rows (2006 bytes apart)
    (5000, 9, 1, "bf16", 0.25, 1.5, 3000),         # 3000 tokens masked with -inf, among them whole segments
    (70, 5, 1, "f32", 4.0, 0.5, 0),                # less than one segment, nearly flat distribution
])
def test_every_row_draw_matches_oracle(V, n, B, dtype, T, scale, masked):
    """A chain whose node i carries the token the oracle draws at position i is accepted whole, so the produced
    tokens are the draws of all n + 1 rows."""
    import torch
    from paper_2406_17276_amd import api
    g = np.random.default_rng(V + n)
    x = (g.standard_normal((B, n + 1, V)) * scale).astype(np.float32)
    if masked:
        x[:, :, :2048] = -np.inf                                    # whole leading segments
        for b in range(B):
            for r in range(n + 1):
                x[b, r, g.choice(np.arange(2048, V), masked - 2048, replace=False)] = -np.inf
    target = wl.store(x, dtype)
    t64 = wl.to_f64(target, dtype)
    u = np.stack([_uniforms_with_margin(t64[b], T, g) for b in range(B)])
    u[:, 0] = 0.0                                                   # the first token with a positive probability
    draws = [[vf.sample_truth(t64[b, r], T, float(u[b, r])) for r in range(n + 1)] for b in range(B)]
    trees = [dict(token=np.array(draws[b][:n]), parent=np.arange(-1, n - 1), n_out=n) for b in range(B)]
    for b in range(B):
        assert vf.sampled_verify(t64[b], T, u[b].astype(np.float64), trees[b]["token"], trees[b]["parent"], n) == \
            (n + 1, list(range(n)), draws[b])
    alen, anode, atok = api.verify_sample(U.to_device(target, dtype), torch.from_numpy(u).cuda(), T,
                                          _tree_to_device(api, trees, B, n))
    torch.cuda.synchronize()
    assert list(alen.cpu().numpy()) == [n + 1] * B
    np.testing.assert_array_equal(atok.cpu().numpy(), np.array(draws))
    np.testing.assert_array_equal(anode.cpu().numpy(), np.tile(np.arange(n), (B, 1)))


def test_low_temperature_draw_is_the_greedy_result():
    import torch
    from paper_2406_17276_amd import api
    V, k, n, d, B, dtype = 4000, 6, 30, 5, 2, "bf16"
    g = np.random.default_rng(11)
    draft = wl.store((g.standard_normal((B, d, n, V)) * 3.0).astype(np.float32), dtype)
    trees = U.oracle_trees(draft, dtype, k, n, d)
    target = np.stack([_target_rows(trees[b], n, V, g, 0.9, dtype) for b in range(B)])
    tree_dev = _tree_to_device(api, trees, B, n)
    dev = U.to_device(target, dtype)
    u = torch.from_numpy(g.random((B, n + 1)).astype(np.float32)).cuda()
    a = api.verify_greedy(dev, tree_dev)
    b_ = api.verify_sample(dev, u, 0.02, tree_dev)                  # the boosted logit leads by > 2: e^-100
    torch.cuda.synchronize()
    for x, y in zip(a, b_):
        assert torch.equal(x, y)


def _at_offset(stored, dtype, offset):
    """The rows as a view that starts `offset` elements into a buffer, its rows offset + 5 elements longer."""
    import torch
    t = U.to_device(stored, dtype)
    flat = torch.zeros((*t.shape[:-1], t.shape[-1] + offset + 5), dtype=t.dtype, device="cuda")
    view = flat[..., offset:offset + t.shape[-1]]
    view.copy_(t)
    return view


@pytest.mark.parametrize("V,n,B,dtype,offset", [
    (8192, 255, 2, "bf16", 0),         # 256 threads per row by length; 512 rows
    (8200, 127, 1, "bf16", 1),         # 128 rows: 1024 threads; every row starts inside a vector
    (8201, 128, 1, "bf16", 7),         # 129 rows: 512 threads
    (8197, 255, 1, "f32", 3),          # 256 rows: still 512
    (8196, 128, 2, "f32", 2),          # 258 rows: 256 threads, several batches of vectors
    (5, 3, 1, "bf16", 6),              # a row shorter than a vector, across two of them
    (1, 1, 1, "f32", 1),
])
def test_every_row_result_at_any_alignment_and_width_of_workgroup(V, n, B, dtype, offset):
    """A chain that carries every row's ground truth is accepted whole, so the tokens are the results of all rows."""
    import torch
    from paper_2406_17276_amd import api
    g = np.random.default_rng(V + n)
    target = wl.store((g.standard_normal((B, n + 1, V)) * 2.0).astype(np.float32), dtype)
    t64 = wl.to_f64(target, dtype)
    u = np.stack([_uniforms_with_margin(t64[b], 1.0, g) for b in range(B)])
    rows = _at_offset(target, dtype, offset)
    for sampled in (False, True):
        truth = np.array([[vf.sample_truth(t64[b, r], 1.0, float(u[b, r])) if sampled else int(np.argmax(t64[b, r]))
                           for r in range(n + 1)] for b in range(B)])
        trees = [dict(token=truth[b, :n], parent=np.arange(-1, n - 1), n_out=n) for b in range(B)]
        dev = _tree_to_device(api, trees, B, n)
        alen, _, atok = (api.verify_sample(rows, torch.from_numpy(u).cuda(), 1.0, dev) if sampled
                         else api.verify_greedy(rows, dev))
        torch.cuda.synchronize()
        assert list(alen.cpu().numpy()) == [n + 1] * B
        np.testing.assert_array_equal(atok.cpu().numpy(), truth)


@pytest.mark.parametrize("V,dtype", [(70, "f32"), (8, "bf16"), (9001, "bf16")])
def test_rows_at_the_types_lowest_value_or_without_numbers(V, dtype):
    """Rows masked with the type's lowest value: alone they are a uniform distribution, beside an ordinary logit they
    weigh nothing.  Rows of NaNs have no ground truth, but name a token of the vocabulary."""
    import torch
    from paper_2406_17276_amd import api
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    low = torch.finfo(dt).min
    x = torch.full((1, 5, V), low, dtype=dt, device="cuda")
    x[0, 1, V // 2] = 1.0
    x[0, 2] = float("-inf")
    x[0, 3] = float("nan")
    x[0, 4, 0] = float("nan")
    want = [V // 3, V // 2, 0]
    u = torch.full((1, 5), (V // 3 + 0.5) / V, dtype=torch.float32, device="cuda")
    for sampled in (False, True):
        truth = want if sampled else [0, V // 2, 0]
        tree = _tree_to_device(api, [dict(token=np.array(truth + [0]), parent=np.arange(-1, 3), n_out=4)], 1, 4)
        alen, _, atok = api.verify_sample(x, u, 1.0, tree) if sampled else api.verify_greedy(x, tree)
        torch.cuda.synchronize()
        got = list(atok.cpu().numpy()[0])
        assert int(alen) >= 4 and got[:3] == truth
        assert all(0 <= t < V for t in got[:int(alen)])


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_nans_among_the_logits(dtype):
    """A NaN is never the most probable token; a 16-byte vector that holds one weighs nothing in the draw."""
    import torch
    from paper_2406_17276_amd import api
    V, n, vec = 9000, 40, 8 if dtype == "bf16" else 4
    g = np.random.default_rng(vec)
    stored = wl.store((g.standard_normal((1, n + 1, V)) * 2.0).astype(np.float32), dtype)
    at = g.integers(0, V, (n + 1, 200))
    at[:n // 2, 0] = wl.to_f64(stored, dtype)[0, :n // 2].argmax(1) ^ 1      # beside the best token
    rows = U.to_device(stored, dtype)
    greedy = wl.to_f64(stored, dtype)[0]
    drawn = greedy.copy()
    for r in range(n + 1):
        rows[0, r, torch.from_numpy(at[r]).cuda()] = float("nan")
        greedy[r, at[r]] = -np.inf
        drawn[r].reshape(-1, vec)[at[r] // vec] = -np.inf
    u = _uniforms_with_margin(drawn, 1.0, g)
    for sampled in (False, True):
        truth = np.array([vf.sample_truth(drawn[r], 1.0, float(u[r])) if sampled else int(np.argmax(greedy[r])) for r in range(n + 1)])
        tree = _tree_to_device(api, [dict(token=truth[:n], parent=np.arange(-1, n - 1), n_out=n)], 1, n)
        _, _, tok = (api.verify_sample(rows, torch.from_numpy(u[None]).cuda(), 1.0, tree) if sampled
                     else api.verify_greedy(rows, tree))
        np.testing.assert_array_equal(tok.cpu().numpy()[0], truth)


@pytest.mark.parametrize("V,dtype,sigma,peak,T", [
    (32000, "bf16", 2.0, 8.0, 0.3), (32000, "f32", 1.0, 0.0, 0.05),    # several wavefronts' and segments' references
    (128256, "bf16", 1.0, 0.0, 0.05), (128256, "bf16", 2.0, 8.0, 0.3),
    (3000, "bf16", 2.0, 30.0, 2.0),
])
def test_boundaries_of_the_sampled_distribution(V, dtype, sigma, peak, T):
    """Draws with uniform numbers next to a boundary of the CDF, 8192 of them within 4e-6 of it: where they change over is
    the boundary as the kernel has it.  A term near the reference errs by 2^-23 (v_exp_f32) and 2^-24 (its exponent), the
    sum of a vector by 7 x 2^-24 at most, both of a share of the whole that is below 1, and u is an fp32 number: 2.5e-7."""
    import torch
    from paper_2406_17276_amd import api
    g = torch.Generator(device="cuda")
    g.manual_seed(V)
    B, worst = 8192, 0.0
    for rep in range(12):
        x = torch.randn(V, generator=g, device="cuda") * sigma
        x[int(torch.randint(0, V, (1,), generator=g, device="cuda"))] += peak
        x = x.to(torch.bfloat16 if dtype == "bf16" else torch.float32)
        z = x.double() / T
        e = torch.exp(z - z.max())
        cdf = torch.cumsum(e, 0) / e.sum()
        for t in (int(torch.argmax(e)), int(torch.searchsorted(cdf, torch.tensor(0.02 + 0.075 * rep, device="cuda", dtype=torch.double)))):
            edge = float(cdf[t])
            if not 1e-4 < edge < 1.0 - 1e-5:
                continue
            u = (edge + (torch.arange(B, device="cuda", dtype=torch.double) - B / 2) * (8e-6 / B)).float()
            rows = torch.as_strided(x.repeat(2), (B, 2, V), (0, V, 1))            # every sequence: the same two rows
            tree = api.alloc_tree(B, 1)
            tree.token.fill_(-1), tree.parent.fill_(-1), tree.n_out.zero_()
            _, _, tok = api.verify_sample(rows, u[:, None].repeat(1, 2).contiguous(), T, tree)
            past = tok[:, 0] > t
            if bool(past.any()):
                worst = max(worst, edge - float(u[past].double().min()))
            if not bool(past.all()):
                worst = max(worst, float(u[~past].double().max()) - edge)
    print(f"largest error of a boundary: {worst:.2e}", flush=True)
    assert worst < 2.5e-7


@pytest.mark.parametrize("T", [1e-30, 1e-37, 2e-38, 1e-39, 1e-45])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_vanishing_temperatures_draw_the_most_probable_token(T, dtype):
    import torch
    from paper_2406_17276_amd import api
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    x = (torch.randn((4, 9, 5000), generator=g, device="cuda") * 3.0)
    x[1] -= 40.0
    x[2] += 40.0
    x.scatter_(2, torch.randint(0, 5000, (4, 9, 1), generator=g, device="cuda"), float(x.max()) + 20.0)
    x = x.to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    truth = x.float().argmax(2).cpu().numpy()
    tree = _tree_to_device(api, [dict(token=truth[b, :8], parent=np.arange(-1, 7), n_out=8) for b in range(4)], 4, 8)
    _, _, tok = api.verify_sample(x, torch.rand((4, 9), generator=g, device="cuda"), T, tree)
    np.testing.assert_array_equal(tok.cpu().numpy(), truth)


def test_verification_of_more_threads_than_a_grid_holds():
    """2^23 + 2 sequences of two rows: at 256 threads a row more than 2^32 threads."""
    import torch
    from paper_2406_17276_amd import api
    B, V = (1 << 23) + 2, 16
    g = torch.Generator(device="cuda").manual_seed(6)
    x = torch.zeros((B, 2, V), device="cuda", dtype=torch.bfloat16)
    best = torch.randint(0, V, (B, 2), generator=g, device="cuda")
    x.scatter_(2, best[..., None], 9.0)
    tree = api.alloc_tree(B, 1)
    hit = torch.rand(B, generator=g, device="cuda") < 0.5
    tree.token.copy_(torch.where(hit, best[:, 0], (best[:, 0] + 1) % V).int()[:, None])
    tree.parent.fill_(-1), tree.n_out.fill_(1)
    length, node, token = api.verify_greedy(x, tree)
    assert torch.equal(length, 1 + hit.int()) and torch.equal(node[:, 0], hit.int() - 1)
    assert torch.equal(token[:, 0], best[:, 0].int())
    assert torch.equal(token[:, 1], torch.where(hit, best[:, 1], torch.full_like(best[:, 1], -1)).int())


@pytest.mark.parametrize("n", [1, 63, 64, 65, 127, 128, 255, 256])
def test_walk_over_every_position(n):
    """A chain whose nodes have a sibling each that disagrees, a twin (the same token: the smaller index counts) or a node
    with a parent that does not exist behind them; cut off, or with nodes past n_out, at random."""
    import torch
    from paper_2406_17276_amd import api
    g = np.random.default_rng(n)
    B, V = 24, 16
    truth = g.integers(0, V, (B, n + 1)).astype(np.int32)
    token, parent, n_out = np.zeros((B, n), np.int32), np.zeros((B, n), np.int32), np.zeros(B, np.int32)
    want = []
    for b in range(B):
        cur, stop = -1, g.random() * 0.1 * (b % 3)
        for i in range(n):
            kind = g.random()
            parent[b, i], token[b, i] = cur, truth[b, cur + 1]
            if kind < 0.2:
                token[b, i] ^= 1                                   # disagrees
            elif kind < 0.3:
                parent[b, i] = int(g.choice([-7, -2, n, 10 ** 6, 2 ** 31 - 1, -2 ** 31]))
            elif kind < 0.4 and i > 0:
                parent[b, i], token[b, i] = parent[b, i - 1], token[b, i - 1]      # a twin
            elif g.random() >= stop:
                cur = i
        n_out[b] = n if b % 4 else int(g.integers(0, n + 1))
        path, cur = [], -1
        while True:
            kids = [i for i in range(n_out[b]) if parent[b, i] == cur and token[b, i] == truth[b, cur + 1]]
            if not kids:
                break
            cur = kids[0]
            path.append(cur)
        want.append(path)
    rows = torch.zeros((B, n + 1, V), device="cuda")
    rows.scatter_(2, torch.from_numpy(truth).long().cuda()[..., None], 3.0)
    tree = api.alloc_tree(B, n)
    tree.token.copy_(torch.from_numpy(token)), tree.parent.copy_(torch.from_numpy(parent)), tree.n_out.copy_(torch.from_numpy(n_out))
    length, node, tok = (t.cpu().numpy() for t in api.verify_greedy(rows, tree))
    for b, path in enumerate(want):
        A = len(path) + 1
        assert length[b] == A and list(node[b, :A - 1]) == path and (node[b, A - 1:] == -1).all()
        assert list(tok[b, :A]) == [truth[b, p + 1] for p in [-1] + path] and (tok[b, A:] == -1).all()


@pytest.mark.parametrize("B,H,n,D,dtype", [
    (1, 4, 256, 1024, "f32"), (2, 3, 256, 128, "bf16"), (1, 2, 129, 64, "f32"), (3, 1, 5, 8, "bf16"), (1, 1, 33, 4100, "f32"),
])
def test_append_of_long_branches(B, H, n, D, dtype):
    """Every node accepted, in reverse order, up to the cache's end."""
    import torch
    from paper_2406_17276_amd import api
    g = torch.Generator(device="cuda").manual_seed(n)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    Lmax, L = n + 20, [0, 17, 23][:B]                              # the last: room for n - 3 rows
    m = lambda rows: torch.randn((B, H, rows, D), generator=g, device="cuda").to(dt)
    kp, vp, kt, vt = m(Lmax), m(Lmax), m(n), m(n)
    wk, wv = kp.clone(), vp.clone()
    nodes = torch.arange(n - 1, -1, -1, dtype=torch.int32, device="cuda").repeat(B, 1)
    for b in range(B):
        rows = min(n, Lmax - L[b])
        wk[b, :, L[b]:L[b] + rows], wv[b, :, L[b]:L[b] + rows] = kt[b].flip(1)[:, :rows], vt[b].flip(1)[:, :rows]
    new = api.kv_append(kp, vp, kt, vt, torch.tensor(L, dtype=torch.int32, device="cuda"),
                        torch.full((B,), n + 1, dtype=torch.int32, device="cuda"), nodes)
    assert torch.equal(kp, wk) and torch.equal(vp, wv)
    assert new.cpu().tolist() == [min(l + n, Lmax) for l in L]
