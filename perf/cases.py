"""What a decoder that uses this library has it do, as timed cases.

Every case is one call sequence through the public binding (`paper_2406_17276_amd.api`) with the objects a serving
program keeps between calls (workspaces, output buffers, prepared calls).  Kinds:

  step    one-shot tree build, then the verification attention under the mask just built (the prepared-call form)
  build   one-shot tree build from the logits of all drafting steps
  adapt   the same with the stopping rule of Algorithm 1 inside the call
  draft   the streaming builder as a decoder drives it between draft-model forwards: begin, then per drafting step
          expand, drafting mask and the loop condition, finally the tree
  attn    tree attention on its own: verification (tree keys = nodes) or a drafting step (`pool` layers of keys),
          cache in the query's type or in 8 bits
  verify  target rows -> accepted branch (greedy or sampled) -> accepted K/V rows appended to the cache

Shapes named 7b, 13b, 70b, tiny and large are those of `workloads.py` in this repository.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2406_17276_amd import api

DEV = "cuda"


# ---------------------------------------------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------------------------------------------
def listed():
    return [
        # the smallest call pair: unit-test sized fp32 model, every microsecond is launch and host time
        dict(name="step_tiny_f32", kind="step", dtype="f32", batch=1, vocab=1000, depth=4, k=4, n=16, scale=3.0,
             q_heads=4, kv_heads=4, head_dim=64, prefix=128, ragged=0.0),
        # one user, one sequence, a 7B-shaped target: the step the benchmark's headline is quoted on
        dict(name="step_7b", kind="step", dtype="bf16", batch=1, vocab=32000, depth=10, k=10, n=50, scale=4.0,
             q_heads=32, kv_heads=32, head_dim=128, prefix=1024, ragged=0.0),
        # a serving batch: grouped-query target, 16 sequences of unequal length
        dict(name="step_70b_batch", kind="step", dtype="bf16", batch=16, vocab=32000, depth=10, k=8, n=60, scale=4.0,
             q_heads=64, kv_heads=8, head_dim=128, prefix=4096, ragged=0.25),
        # a draft head that emits all steps at once, depth decided by the rule, 13B-shaped
        dict(name="adapt_13b", kind="adapt", dtype="bf16", batch=1, vocab=32000, depth=12, k=10, n=64, scale=4.0,
             delta=0.2),
        # a vocabulary with a few added tokens: rows that start at odd addresses
        dict(name="build_odd_vocab", kind="build", dtype="bf16", batch=3, vocab=32003, depth=7, k=6, n=33, scale=4.0),
        # large node budget, long vocabulary, full batch: the largest stream of logits
        dict(name="build_large", kind="build", dtype="bf16", batch=32, vocab=128256, depth=20, k=16, n=256, scale=5.0),
        # the drafting loop of one sequence, one call per draft-model forward
        dict(name="draft_7b", kind="draft", dtype="bf16", batch=1, vocab=32000, depth=10, k=10, n=50, scale=4.0,
             delta=0.0),
        # the draft model's own attention in the last drafting step: 64 frontier tokens, 12 layers of pool keys
        dict(name="attn_draft_13b", kind="attn", dtype="bf16", cache="same", batch=1, n=64, pool=12, q_heads=40,
             kv_heads=40, head_dim=128, prefix=2048, ragged=0.0),
        # verification of the large node budget over long prefixes: bound by the matrix cores
        dict(name="attn_large", kind="attn", dtype="bf16", cache="same", batch=32, n=256, pool=1, q_heads=32,
             kv_heads=8, head_dim=128, prefix=8192, ragged=0.0),
        # the serving batch over a cache kept in 8 bits
        dict(name="attn_70b_8bit", kind="attn", dtype="bf16", cache="fp8", batch=16, n=60, pool=1, q_heads=64,
             kv_heads=8, head_dim=128, prefix=4096, ragged=0.25),
        # the end of a step, temperature 0, one sequence
        dict(name="verify_greedy_7b", kind="verify", dtype="bf16", mode="greedy", batch=1, vocab=32000, n=50,
             kv_heads=32, head_dim=128, prefix=1024),
        # the end of a step, temperature 1, the serving batch
        dict(name="verify_sample_70b", kind="verify", dtype="bf16", mode="sample", batch=16, vocab=32000, n=60,
             kv_heads=8, head_dim=128, prefix=4096),
    ]


def _log(rng, lo, hi):
    """An integer between lo and hi, spread over the logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_tree(rng, c):
    """Sizes of a tree build: generic vocabularies (a third of them not a multiple of anything), budgets and depths."""
    c["dtype"] = rng.choice(("bf16", "bf16", "bf16", "f32"))
    v = _log(rng, 1000, 131072)
    c["vocab"] = v if rng.random() < 1 / 3 else max(1000, v // 64 * 64)
    c["depth"] = rng.randint(3, 20)
    c["k"] = rng.randint(4, 16)
    c["n"] = _log(rng, 12, 256)
    c["scale"] = round(rng.uniform(3.0, 5.0), 2)
    c["batch"] = _log(rng, 1, 32)
    while c["batch"] > 1 and c["batch"] * c["depth"] * c["n"] * c["vocab"] > 2_000_000_000:
        c["batch"] -= 1


def _draw_attn(rng, c, batch=None):
    """Sizes of an attention call: multi-head and grouped-query shapes, one sequence to a batch."""
    g = rng.choice((1, 1, 4, 8))
    c["kv_heads"] = _log(rng, 4, 40) if g == 1 else rng.choice((2, 4, 8))
    c["q_heads"] = g * c["kv_heads"]
    c["head_dim"] = rng.choice((64, 128, 128))
    c["prefix"] = _log(rng, 100, 8192)
    c["ragged"] = rng.choice((0.0, 0.25))
    c["batch"] = _log(rng, 1, 32) if batch is None else batch
    most = 1e12 if c["dtype"] == "bf16" else 1e10
    while _attn_flops(c) > most and c["prefix"] > 128:
        c["prefix"] = max(128, c["prefix"] * 3 // 4)


def draw(rng):
    kind = rng.choice(("step", "step", "build", "adapt", "draft", "attn", "attn", "attn", "verify", "verify"))
    c = dict(kind=kind)
    if kind in ("step", "build", "adapt", "draft"):
        _draw_tree(rng, c)
    if kind == "adapt":
        c["delta"] = round(rng.uniform(0.02, 0.4), 3)
    if kind == "draft":
        c["delta"] = rng.choice((0.0, 0.05))
    if kind == "step":
        _draw_attn(rng, c, c["batch"])
    if kind == "attn":
        c["dtype"] = rng.choice(("bf16", "bf16", "bf16", "f32"))
        c["cache"] = rng.choice(("same", "fp8")) if c["dtype"] == "bf16" else "same"
        c["n"] = _log(rng, 8, 256)
        c["pool"] = 1 if rng.random() < 0.6 else rng.randint(2, 12)
        _draw_attn(rng, c)
    if kind == "verify":
        c["dtype"] = rng.choice(("bf16", "bf16", "f32"))
        c["mode"] = rng.choice(("greedy", "sample"))
        v = _log(rng, 1000, 131072)
        c["vocab"] = v if rng.random() < 1 / 3 else max(1000, v // 64 * 64)
        c["n"] = _log(rng, 12, 256)
        c["kv_heads"] = rng.choice((2, 4, 8, 32))
        c["head_dim"] = rng.choice((64, 128))
        c["prefix"] = _log(rng, 100, 8192)
        c["batch"] = _log(rng, 1, 32)
        while c["batch"] > 1 and c["batch"] * c["n"] * c["vocab"] > 300_000_000:
            c["batch"] -= 1
    return c


# ---------------------------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------------------------
def _torch_dtype(c):
    return torch.bfloat16 if c["dtype"] == "bf16" else torch.float32


def _frontier(c):
    F = [1]
    for _ in range(c["depth"]):
        F.append(min(c["n"], c["k"] * F[-1]))
    return F


def _generator(seed, tag):
    g = torch.Generator(device=DEV)
    g.manual_seed((seed * 1000003 + tag) & 0x7FFFFFFFFFFFFFFF)
    return g


def _step_rows(c, g, rows):
    """Draft-model rows of one drafting step: N(0, scale) logits with a planted peak (the workloads' recipe)."""
    x = torch.randn((c["batch"], rows, c["vocab"]), generator=g, device=DEV, dtype=torch.float32).mul_(c["scale"])
    idx = torch.randint(0, c["vocab"], (c["batch"], rows, 1), generator=g, device=DEV)
    x.scatter_add_(2, idx, torch.full(idx.shape, 6.0, dtype=torch.float32, device=DEV))
    return x.to(_torch_dtype(c))


def _logits(c, seed):
    """[batch, depth, n, vocab]; rows beyond a step's frontier are never read and stay as allocated."""
    g, F = _generator(seed, 1), _frontier(c)
    out = torch.empty((c["batch"], c["depth"], c["n"], c["vocab"]), dtype=_torch_dtype(c), device=DEV)
    for t in range(c["depth"]):
        out[:, t, :F[t]] = _step_rows(c, g, F[t])
    return out


def _prefix(c, seed):
    """Prefix lengths [batch] and the rows the cache has room for."""
    r = c.get("ragged", 0.0)
    u = np.random.RandomState(seed % (1 << 31)).uniform(-r, r, size=c["batch"])
    lens = np.round(c["prefix"] * (1.0 + u)).astype(np.int32)
    return torch.from_numpy(lens).to(DEV), int(round(c["prefix"] * (1.0 + r)))


def _random_parents(c, rs):
    """[batch, n] parents-first random trees, -1 = child of the root."""
    i = np.arange(c["n"])
    return np.floor(rs.random_sample((c["batch"], c["n"])) * (i + 1)).astype(np.int64) - 1


def _tree_mask(c, seed):
    """int64 [batch, n, words]: bit j of row i = key row j is node i or an ancestor.  pool > 1: row i is a frontier
    node of the last of `pool` layers of n nodes, its ancestors one per layer."""
    rs = np.random.RandomState((seed + 77) % (1 << 31))
    B, n, keys = c["batch"], c["n"], c["n"] * c["pool"]
    m = np.zeros((B, n, (keys + 63) // 64), dtype=np.uint64)
    bi = np.arange(B)[:, None]
    ni = np.arange(n)[None, :]
    one = np.uint64(1)
    if c["pool"] == 1:
        par = _random_parents(c, rs)
        for i in range(n):                                    # a parent's row is complete before its children's
            p = par[:, i]
            m[:, i] = np.where((p >= 0)[:, None], m[np.arange(B), np.maximum(p, 0)], np.uint64(0))
            m[:, i, i // 64] |= one << np.uint64(i % 64)
    else:
        slot = np.broadcast_to(ni, (B, n))
        for layer in range(c["pool"] - 1, -1, -1):
            key = layer * n + slot
            np.bitwise_or.at(m, (bi, ni, key // 64), one << (key % 64).astype(np.uint64))
            slot = rs.randint(0, n, size=(B, n))[bi, slot]    # parents in the layer above
    return torch.from_numpy(m.view(np.int64)).to(DEV)


def _attention(c, seed):
    g, dt = _generator(seed, 2), _torch_dtype(c)
    lens, room = _prefix(c, seed)
    B, H, D, keys = c["batch"], c["kv_heads"], c["head_dim"], c["n"] * c.get("pool", 1)

    def rows(h, r):
        return torch.randn((B, h, r, D), generator=g, device=DEV, dtype=torch.float32)
    a = dict(Q=rows(c["q_heads"], c["n"]).to(dt), K_prefix=rows(H, room), V_prefix=rows(H, room), K_tree=rows(H, keys),
             V_tree=rows(H, keys), prefix_len=lens)
    if c.get("cache") == "fp8":                               # one factor per (sequence, KV head): largest value -> 448
        for s in ("K", "V"):
            p, t = a[s + "_prefix"], a[s + "_tree"]
            f = torch.maximum(p.abs().amax((2, 3)), t.abs().amax((2, 3))) / 448.0
            for name, x in ((s + "_prefix", p), (s + "_tree", t)):
                a[name] = (x / f[:, :, None, None]).to(torch.float8_e4m3fn).view(torch.uint8)
            a[s.lower() + "_scale"] = f.contiguous()
    else:
        for name in ("K_prefix", "V_prefix", "K_tree", "V_tree"):
            a[name] = a[name].to(dt)
    return a


def _verify_inputs(c, seed):
    """A drafted tree and target rows that follow it: most nodes with a child have one the target agrees with, so a
    few tokens are accepted per step, as with a trained draft model."""
    rs = np.random.RandomState((seed + 5) % (1 << 31))
    B, n, V = c["batch"], c["n"], c["vocab"]
    par = _random_parents(c, rs)
    tok = np.stack([rs.permutation(V)[:n] for _ in range(B)])
    child = np.full((B, n + 1), -1, dtype=np.int64)           # by target row (0 = root, 1 + i = node i)
    for i in range(n - 1, -1, -1):
        child[np.arange(B), par[:, i] + 1] = i
    agree = (child >= 0) & (rs.random_sample(child.shape) < 0.85)
    g = _generator(seed, 3)
    x = torch.randn((B, n + 1, V), generator=g, device=DEV, dtype=torch.float32).mul_(4.0)
    b, r = np.nonzero(agree)
    x[torch.from_numpy(b).to(DEV), torch.from_numpy(r).to(DEV), torch.from_numpy(tok[b, child[b, r]]).to(DEV)] = \
        4.0 * math.sqrt(2.0 * math.log(V)) + 2.0
    tree = api.alloc_tree(B, n, DEV)
    tree.token.copy_(torch.from_numpy(tok.astype(np.int32)))
    tree.parent.copy_(torch.from_numpy(par.astype(np.int32)))
    tree.n_out.fill_(n)
    return x.to(_torch_dtype(c)), tree, torch.rand((B, n + 1), generator=g, device=DEV)


def prepare(case, seed):
    c, s = case, dict(case=case)
    kind = c["kind"]
    if kind == "step":
        s["build"] = api.PreparedBuild(_logits(c, seed), c["k"], c["n"], c["depth"])
        a = _attention(c, seed)
        s["attn"] = api.PreparedAttention(a["Q"], a["K_prefix"], a["V_prefix"], a["K_tree"], a["V_tree"], a["prefix_len"],
                                          s["build"].out.mask)
    elif kind in ("build", "adapt"):
        s["logits"] = _logits(c, seed)
        s["out"] = api.alloc_tree(c["batch"], c["n"], DEV)
        need = api.build_workspace_bytes(api.build_params(s["logits"], c["k"], c["n"], c["depth"]))
        s["ws"] = torch.empty(need, dtype=torch.uint8, device=DEV)
    elif kind == "draft":
        g, F = _generator(seed, 1), _frontier(c)
        s["rows"] = [_step_rows(c, g, F[t]) for t in range(c["depth"])]       # what the draft model's forwards return
    elif kind == "attn":
        s.update(_attention(c, seed))
        s["mask"] = _tree_mask(c, seed)
        s["O"] = torch.empty_like(s["Q"])
        s["ws"] = api.attn_workspace(api.attn_params(s["Q"], s["K_prefix"], s["V_prefix"], s["K_tree"], s["V_tree"]), DEV)
    elif kind == "verify":
        s["target"], s["tree"], s["u"] = _verify_inputs(c, seed)
        dt, g = _torch_dtype(c), _generator(seed, 4)
        room = c["prefix"] + c["n"]

        def rows(r):
            return torch.randn((c["batch"], c["kv_heads"], r, c["head_dim"]), generator=g, device=DEV).to(dt)
        s["kv"] = (rows(room), rows(room), rows(c["n"]), rows(c["n"]))
        s["len"] = torch.full((c["batch"],), c["prefix"], dtype=torch.int32, device=DEV)
        t = s["target"]
        p = api.VerifyParams(c["batch"], c["vocab"], c["n"], api.OT_BF16 if c["dtype"] == "bf16" else api.OT_F32,
                             t.stride(0), t.stride(1))
        size = api.lib().ot_verify_workspace_bytes if c["mode"] == "greedy" else api.lib().ot_verify_sample_workspace_bytes
        s["ws"] = torch.empty(int(size(p)), dtype=torch.uint8, device=DEV)
    return s


# ---------------------------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------------------------
def _tree_fields(t):
    return dict(token=t.token, parent=t.parent, depth=t.depth, score=t.score, mask=t.mask, n_out=t.n_out, expect=t.expect)


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "step":
        stream = torch.cuda.current_stream().cuda_stream
        s["build"](stream)
        s["attn"](stream)
        return dict(tree=_tree_fields(s["build"].out), O=s["attn"].out)
    if kind == "build":
        return _tree_fields(api.build_tree(s["logits"], c["k"], c["n"], c["depth"], out=s["out"], workspace=s["ws"]))
    if kind == "adapt":
        tree, steps, e = api.build_tree_adaptive(s["logits"], c["k"], c["n"], c["depth"], c["delta"], out=s["out"],
                                                 workspace=s["ws"])
        return dict(tree=_tree_fields(tree), steps=steps, e_sub=e)
    if kind == "draft":
        ts = api.TreeStream(c["batch"], c["vocab"], c["k"], c["n"], c["depth"],
                            api.OT_BF16 if c["dtype"] == "bf16" else api.OT_F32, DEV)
        for t in range(c["depth"]):
            token, parent = ts.expand(s["rows"][t])
            mask = ts.frontier_mask()
            e, go = ts.e_sub(c["delta"])
        return dict(tree=_tree_fields(ts.finalize()), token=token, parent=parent, count=ts.frontier_count, mask=mask,
                    e_sub=e, go_on=go)
    if kind == "attn":
        if c["cache"] == "fp8":
            return api.tree_verify_attention_fp8kv(s["Q"], s["K_prefix"], s["V_prefix"], s["K_tree"], s["V_tree"],
                                                   s["k_scale"], s["v_scale"], s["prefix_len"], s["mask"], out=s["O"],
                                                   workspace=s["ws"])
        return api.tree_verify_attention(s["Q"], s["K_prefix"], s["V_prefix"], s["K_tree"], s["V_tree"],
                                         s["prefix_len"], s["mask"], out=s["O"], workspace=s["ws"])
    if c["mode"] == "greedy":
        length, node, token = api.verify_greedy(s["target"], s["tree"], workspace=s["ws"])
    else:
        length, node, token = api.verify_sample(s["target"], s["u"], 1.0, s["tree"], workspace=s["ws"])
    kp, vp, kt, vt = s["kv"]
    new_len = api.kv_append(kp, vp, kt, vt, s["len"], length, node)
    return dict(length=length, node=node, token=token, new_len=new_len, K=kp, V=vp)


# ---------------------------------------------------------------------------------------------------------------
# what a pass cannot do without, and how close another correct implementation comes
# ---------------------------------------------------------------------------------------------------------------
def _esize(c):
    return 2 if c["dtype"] == "bf16" else 4


def _attn_flops(c):
    return 4.0 * c["batch"] * c["q_heads"] * c["n"] * (c["prefix"] + c["n"] * c.get("pool", 1)) * c["head_dim"]


def _attn_bytes(c):
    keys = c["n"] * c.get("pool", 1)
    cache = 1 if c.get("cache") == "fp8" else _esize(c)
    kv = 2 * c["batch"] * c["kv_heads"] * (c["prefix"] + keys) * c["head_dim"] * cache
    qo = 2 * c["batch"] * c["q_heads"] * c["n"] * c["head_dim"] * _esize(c)
    return kv + qo + c["batch"] * c["n"] * ((keys + 63) // 64) * 8


def _build_bytes(c):
    rows = sum(_frontier(c)[:c["depth"]])
    return c["batch"] * (rows * c["vocab"] * _esize(c) + c["n"] * (16 + 8 * ((c["n"] + 63) // 64)))


def _build_flops(c):
    return 3.0 * c["batch"] * sum(_frontier(c)[:c["depth"]]) * c["vocab"]     # maximum, exponential, sum per logit


def work(case):
    c, kind = case, case["kind"]
    if kind == "attn":
        return dict(bytes=_attn_bytes(c), flops=_attn_flops(c))
    if kind == "step":
        return dict(bytes=_build_bytes(c) + _attn_bytes(c), flops=_build_flops(c) + _attn_flops(c))
    if kind in ("build", "adapt"):
        return dict(bytes=_build_bytes(c), flops=_build_flops(c))
    if kind == "draft":
        words = (c["depth"] * c["n"] + 63) // 64
        return dict(bytes=_build_bytes(c) + c["batch"] * c["depth"] * c["n"] * (8 + 8 * words), flops=_build_flops(c))
    rows = c["batch"] * (c["n"] + 1)
    per = 1.0 if c["mode"] == "greedy" else 3.0
    return dict(bytes=rows * c["vocab"] * _esize(c) + rows * 16, flops=per * rows * c["vocab"])


def tolerance(case):
    c, kind = case, case["kind"]
    if kind == "verify":
        if c["mode"] == "greedy":
            return "exact"
        # a uniform number within 1e-7 of a boundary of the cumulative sum may fall on either side
        return dict(rel=1e-2, differ=0.01)
    if kind in ("attn", "step"):
        return dict(rel=1e-2, max=0.1) if c["dtype"] == "bf16" else dict(rel=1e-5, max=2e-4)
    return dict(rel=1e-5, max=2e-4)          # 32-bit scores of a tree whose whole numbers are exact
