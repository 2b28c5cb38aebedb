"""Parity of ot_tree_verify_attention_fp8kv (K/V cache in FP8 E4M3 bytes, one scale per sequence and KV head) with
the fp64 oracle on the values those bytes stand for (needs an MI355X).  Bar: max-abs 2e-2 (bf16 Q, P and O), as for
the bf16 cache."""
import numpy as np
import pytest

from oracle import opt_tree as ot_oracle
from oracle import tree_attention as ta_oracle
import workloads as wl
from tests import _util as U
from tests.test_gpu_attention import large_exact_scores

pytestmark = pytest.mark.gpu
TOL = 2e-2


def _masks(B, n, seed, shape="random"):
    return np.stack([ot_oracle.ancestor_mask(wl.random_tree_parents(n, seed + b, shape)) for b in range(B)])


def _inputs(B, Hq, Hkv, D, L, n, ragged, seed):
    w = wl.Workload("f8", B, 8, 1, 1, n, "bf16", "normal", 1.0, Hq, Hkv, D, L, ragged=ragged)
    x = wl.make_attention_inputs(w, seed)
    kp, kt, ks = wl.quantise_cache_e4m3(x["K_prefix"], x["K_tree"], "bf16")
    vp, vt, vs = wl.quantise_cache_e4m3(x["V_prefix"], x["V_tree"], "bf16")
    return dict(Q=x["Q"], K_prefix=kp, V_prefix=vp, K_tree=kt, V_tree=vt, k_scale=ks, v_scale=vs,
                prefix_len=x["prefix_len"])


def _gpu(x, mask, scale=0.0, views=None):
    import torch
    from paper_2406_17276_amd import api
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    kv = {k: dev(x[k]) for k in ("K_prefix", "V_prefix", "K_tree", "V_tree")}
    if views:
        kv = views(kv)
    out = api.tree_verify_attention_fp8kv(U.to_device(x["Q"], "bf16"), kv["K_prefix"], kv["V_prefix"], kv["K_tree"],
                                          kv["V_tree"], dev(x["k_scale"]), dev(x["v_scale"]),
                                          dev(x["prefix_len"].astype(np.int32)), U.mask_to_device(mask),
                                          softmax_scale=scale)
    torch.cuda.synchronize()
    return U.from_device_f64(out)


def _oracle(x, mask, scale=None, heads=None):
    q = wl.to_f64(x["Q"], "bf16")
    return ta_oracle.tree_verify_attention_fp8kv(q, x["K_prefix"], x["V_prefix"], x["K_tree"], x["V_tree"],
                                                 x["k_scale"], x["v_scale"], x["prefix_len"], mask,
                                                 wl.e4m3_bits_to_f32, scale)


@pytest.mark.parametrize("B,Hq,Hkv,D,L,n,ragged,shape", [
    (2, 4, 4, 64, 150, 20, 0.0, "random"),       # one query head per KV head, 64 wide
    (1, 8, 8, 128, 1000, 50, 0.0, "random"),     # 128 wide, several key splits
    (2, 16, 2, 128, 700, 60, 0.2, "random"),     # GQA 8:1, 480 packed rows: 128-row blocks, ragged prefixes
    (1, 8, 2, 64, 300, 40, 0.0, "chain"),        # GQA 4:1, 64 wide, a chain (every ancestor visible)
    (1, 8, 8, 64, 0, 33, 0.0, "star"),           # no prefix at all: tree keys only
    (3, 4, 2, 128, 65, 256, 0.5, "random"),      # the largest tree, short ragged prefixes (tree tiles dominate)
    (1, 2, 2, 128, 63, 1, 0.0, "random"),        # a single node
    (33, 16, 8, 128, 150, 40, 0.5, "random"),    # a batch that fills the chip: jobs taken longest first
])
def test_shapes_and_edges(B, Hq, Hkv, D, L, n, ragged, shape):
    x = _inputs(B, Hq, Hkv, D, L, n, ragged, 5)
    mask = _masks(B, n, 3, shape)
    got = _gpu(x, mask)
    want = _oracle(x, mask)
    assert np.abs(got - want).max() < TOL


@pytest.mark.parametrize("L", [1, 63, 64, 65, 128, 129, 192, 700])
def test_64_rows_in_great_numbers(L):
    """264 (sequence, KV head) pairs, two workgroups to a compute unit; two to twelve tiles through two buffers."""
    x = _inputs(33, 8, 8, 128, L, 40, 0.0, 7)
    x["prefix_len"][-1] = L // 2
    mask = _masks(33, 40, 9)
    got = _gpu(x, mask)
    some = [0, 17, 32]
    assert np.abs(got[some] - _oracle({k: v[some] for k, v in x.items()}, mask[some])).max() < TOL


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("L,n", [(120, 100), (190, 100), (250, 100), (250, 130)])
def test_a_range_for_every_tile(D, L, n):
    """128-row blocks over few tiles; in the second sequence some ranges have no key."""
    x = _inputs(2, 4, 2, D, L, n // 2, 0.0, 3)
    x["prefix_len"][-1] = L // 3
    mask = _masks(2, n // 2, 4)
    tiles = -(-L // 64) + -(-(n // 2) // 64)
    assert U.attention_plan(2, 4, 2, D, n // 2, L, kv8=True) == (128, tiles, 0)
    assert np.abs(_gpu(x, mask) - _oracle(x, mask)).max() < TOL


@pytest.mark.parametrize("L", [0, 1, 63, 64, 65, 128, 191, 192, 256, 320, 447, 1000])
def test_256_rows_with_few_tiles_and_jumps_in_either_block(L):
    """150 rows a KV head, no key splits: fewer and more tiles than the ring of widened tiles holds, and in half of the
    sequences key bands of far larger scores."""
    assert U.attention_plan(33, 4, 4, 128, 150, 1000, kv8=True) == (256, 1, 1)       # (by the rows that the cache has)
    x = _inputs(33, 4, 4, 128, 1000, 150, 0.0, 5)
    x["prefix_len"][:] = L
    for b in range(1, 33, 2):                                  # the largest value of both signs
        for at in (64 * (b % 3) + 8 * b % 64, 64 * (b % 5) + 70, 64 * (b % 7) + 40):
            band = x["K_prefix"][b, :, at:at + 9]
            band[...] = (band & 0x80) | 0x7E
    mask = _masks(33, 150, 8)
    got = _gpu(x, mask)
    assert np.isfinite(got).all()
    some = sorted({0, 1, 2, 3, 5, 9, 17, 32})
    assert np.abs(got[some] - _oracle({k: v[some] for k, v in x.items()}, mask[some])).max() < TOL


@pytest.mark.parametrize("B,Hq,Hkv,n,nk,L,strided,plan", [
    (8, 8, 8, 150, 150, 2000, False, (256, 4, 0)),       # key ranges: empty ones, ones that begin among the tree tiles
    (65, 6, 3, 70, 70, 600, True, (256, 1, 0)),          # a batch too large to be ranked; K and V as views
    (13, 32, 8, 60, 600, 700, False, (256, 2, 0)),       # a drafting pool of ten tiles
])
def test_256_rows_in_ranges_unranked_and_against_a_pool(B, Hq, Hkv, n, nk, L, strided, plan):
    import torch
    D, g = 128, Hq // Hkv
    assert U.attention_plan(B, Hq, Hkv, D, n, L, n_keys=nk if nk != n else 0, kv8=True) == plan
    x = _inputs(B, Hq, Hkv, D, L, nk, 0.0, 7)
    x["Q"] = np.ascontiguousarray(x["Q"][:, :, :n])
    x["prefix_len"][:] = [[L, 0, 1, 64, 130, 500, L - 1, 200][b % 8] for b in range(B)]
    rng = np.random.default_rng(3)
    W = (nk + 63) // 64
    mask = rng.integers(0, 2 ** 64, size=(B, n, W), dtype=np.uint64) & rng.integers(0, 2 ** 64, size=(B, n, W), dtype=np.uint64)
    mask[:, ::17] = 0

    def views(kv):
        pre = torch.stack([kv["K_prefix"], kv["V_prefix"]], dim=3)
        tre = torch.stack([kv["K_tree"], kv["V_tree"]], dim=3)
        return dict(K_prefix=pre[:, :, :, 0], V_prefix=pre[:, :, :, 1], K_tree=tre[:, :, :, 0], V_tree=tre[:, :, :, 1])

    got = _gpu(x, mask, views=views if strided else None)
    seqs, heads = sorted({0, 1, 2, 3, 4, 6, B - 1}), [0, Hkv - 1]
    q = [h * g + i for h in heads for i in range(g)]
    sub = {k: v[seqs] if k == "prefix_len" else v[seqs][:, q if k == "Q" else heads] for k, v in x.items()}
    assert np.abs(got[seqs][:, q] - _oracle(sub, mask[seqs])).max() < TOL


def test_the_70b_batch_on_sampled_groups():
    """16 sequences of 8 KV heads of 480 rows, ragged prefixes around 4096, inputs drawn on the device: 256-row blocks, jobs
    longest first."""
    import torch
    from paper_2406_17276_amd import api
    w = wl.WORKLOADS["70b"]
    B, Hkv, g, D, n, L = w.batch, w.kv_heads, w.q_heads // w.kv_heads, w.head_dim, w.n, w.max_prefix()
    assert U.attention_plan(B, Hkv * g, Hkv, D, n, L, kv8=True) == (256, 1, 1)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(17)
    draw = lambda rows: (torch.randn((B, Hkv, rows, D), generator=gen, device="cuda") * 64).to(torch.float8_e4m3fn).view(torch.uint8)
    kv = dict(K_prefix=draw(L), V_prefix=draw(L), K_tree=draw(n), V_tree=draw(n))
    Q = torch.randn((B, Hkv * g, n, D), generator=gen, device="cuda").to(torch.bfloat16)
    ks, vs = [(torch.rand((B, Hkv), generator=gen, device="cuda") + 0.5) / 64 for _ in range(2)]
    plen, mask = wl.prefix_lengths(w, 4).astype(np.int32), _masks(B, n, 23)
    out = api.tree_verify_attention_fp8kv(Q, kv["K_prefix"], kv["V_prefix"], kv["K_tree"], kv["V_tree"], ks, vs,
                                          torch.from_numpy(plen).cuda(), U.mask_to_device(mask))
    torch.cuda.synchronize()
    assert bool(torch.isfinite(out.float()).all())
    host = lambda t: t.cpu().numpy()
    for b, h in [(0, 0), (3, 5), (9, 2), (15, 7), (int(plen.argmax()), 1), (int(plen.argmin()), 6)]:
        sub = {k: host(v[b:b + 1, h:h + 1]) for k, v in kv.items()}
        sub.update(Q=host(Q[b:b + 1, h * g:h * g + g].view(torch.int16)).view(np.uint16), k_scale=host(ks[b:b + 1, h:h + 1]),
                   v_scale=host(vs[b:b + 1, h:h + 1]), prefix_len=plen[b:b + 1])
        got = U.from_device_f64(out[b:b + 1, h * g:h * g + g])
        assert np.abs(got - _oracle(sub, mask[b:b + 1])).max() < TOL, (b, h)


def test_scores_that_round_by_more_than_the_slack():
    """As in the 16-bit cache's test of this name: scores of 1e9, here from the K factors."""
    assert U.attention_plan(33, 4, 4, 128, 150, 1000, kv8=True)[0] == 256
    x = _inputs(33, 4, 4, 128, 1000, 150, 0.0, 6)
    x["prefix_len"][:] = 500
    x["k_scale"] = (x["k_scale"] * np.float32(2e8)).astype(np.float32)
    mask = _masks(33, 150, 2)
    got = _gpu(x, mask)
    some = [0, 13, 32]
    want = _oracle({k: v[some] for k, v in x.items()}, mask[some])
    # a row is the V of its best key, whose probability is any number here: rounded to 8 significant bits, like O
    assert (np.abs(got[some] - want) <= 1.01 * 2 * 2.0 ** -8 * np.abs(want) + 1e-6).all()


@pytest.mark.parametrize("n,rows", [(40, 64), (70, 128), (150, 256)])
def test_weights_are_kept_when_the_reference_of_large_scores_moves(n, rows):
    """As in the 16-bit cache's test of this name: scores 2^26 + x, exact in fp32, from K bytes 2^8 and x."""
    B, Hkv, D, L = 33, 4, 128, 1000
    assert U.attention_plan(B, Hkv, Hkv, D, n, L, kv8=True)[0] == rows
    x = large_exact_scores(B, Hkv, D, L, n, 4, first=2.0 ** 8)
    kp, kt = wl.f32_to_e4m3_bits(x["K_prefix"]), wl.f32_to_e4m3_bits(x["K_tree"])       # multiples of 8 up to 128: exact
    vp, vt, vs = wl.quantise_cache_e4m3(x["V_prefix"], x["V_tree"], "bf16")
    x = dict(Q=wl.store(x["Q"], "bf16"), K_prefix=kp, V_prefix=vp, K_tree=kt, V_tree=vt, k_scale=np.ones_like(vs), v_scale=vs,
             prefix_len=x["prefix_len"])
    mask = _masks(B, n, 2)
    got = _gpu(x, mask)
    some = [0, 16, 32]
    assert np.abs(got[some] - _oracle({k: v[some] for k, v in x.items()}, mask[some])).max() < TOL


def test_every_byte_code_and_uneven_scales():
    """Rows holding all 254 finite byte codes (both zeros, subnormals, +-448), scales far from 1 that differ between
    K and V and between heads, and an explicit softmax scale."""
    B, Hq, Hkv, D, L, n = 1, 4, 2, 128, 200, 24
    x = _inputs(B, Hq, Hkv, D, L, n, 0.0, 9)
    codes = np.arange(256, dtype=np.uint8)
    codes[0x7F], codes[0xFF] = 0x7E, 0xFE                      # the two NaN codes are not cache values
    for t in ("K_prefix", "V_prefix", "K_tree", "V_tree"):
        x[t][0, :, 3, :] = codes[:128]
        x[t][0, :, 4, :] = codes[128:]
        x[t][0, :, 5, :] = codes[::-1][:128]
    x["k_scale"] = np.array([[2.0 ** -9, 3.1e-3]], dtype=np.float32)
    x["v_scale"] = np.array([[0.75, 40.0]], dtype=np.float32)
    mask = _masks(B, n, 1)
    got = _gpu(x, mask, scale=0.05)
    want = _oracle(x, mask, scale=0.05)
    ref = np.abs(want).max(axis=(2, 3), keepdims=True)          # V of head group 1 is of order 40 * 448
    assert (np.abs(got - want) / np.maximum(ref, 1.0)).max() < TOL


def test_strided_cache_views():
    """K and V as the two halves of one [B,Hkv,rows,2,D] byte allocation: row stride 2*D bytes."""
    import torch
    B, Hq, Hkv, D, L, n = 2, 8, 4, 64, 130, 18
    x = _inputs(B, Hq, Hkv, D, L, n, 0.0, 2)

    def views(kv):
        pre = torch.stack([kv["K_prefix"], kv["V_prefix"]], dim=3)
        tre = torch.stack([kv["K_tree"], kv["V_tree"]], dim=3)
        return dict(K_prefix=pre[:, :, :, 0], V_prefix=pre[:, :, :, 1], K_tree=tre[:, :, :, 0], V_tree=tre[:, :, :, 1])

    mask = _masks(B, n, 8)
    assert np.abs(_gpu(x, mask, views=views) - _oracle(x, mask)).max() < TOL


def test_full_7b_and_a_70b_shaped_group():
    """The 7B verification shape whole (32 heads, prefix 1024, n = 50), and one sequence of the 70B shape (64 query
    heads on 8 KV heads, prefix near 4096, n = 60) checked on two KV groups."""
    w = wl.WORKLOADS["7b"]
    x = _inputs(1, w.q_heads, w.kv_heads, w.head_dim, w.prefix, w.n, 0.0, 4)
    mask = _masks(1, w.n, 2)
    assert np.abs(_gpu(x, mask) - _oracle(x, mask)).max() < TOL
    w = wl.WORKLOADS["70b"]
    x = _inputs(1, w.q_heads, w.kv_heads, w.head_dim, w.prefix, w.n, 0.0, 6)
    mask = _masks(1, w.n, 4)
    got = _gpu(x, mask)
    g = w.q_heads // w.kv_heads
    for kvh in (0, 5):
        qh = list(range(kvh * g, kvh * g + g))
        sub = dict(Q=x["Q"][:, qh], prefix_len=x["prefix_len"],
                   **{k: x[k][:, [kvh]] for k in ("K_prefix", "V_prefix", "K_tree", "V_tree", "k_scale", "v_scale")})
        assert np.abs(got[:, qh] - _oracle(sub, mask)).max() < TOL


def test_scales_of_one_on_bytes_that_hold_bf16_representable_values_match_the_bf16_cache_path():
    """Every E4M3 value is a bf16 value: with scales of 1 the 8-bit entry point must agree with the bf16 entry point
    fed the widened cache, to the bf16 output's rounding (the two differ only in where the scale is applied)."""
    import torch
    from paper_2406_17276_amd import api
    B, Hq, Hkv, D, L, n = 2, 8, 2, 128, 500, 30
    x = _inputs(B, Hq, Hkv, D, L, n, 0.1, 12)
    x["k_scale"][:] = 1.0
    x["v_scale"][:] = 1.0
    mask = _masks(B, n, 6)
    got8 = _gpu(x, mask)
    wide = {k: U.to_device(wl.f32_to_bf16_bits(wl.e4m3_bits_to_f32(x[k])), "bf16")
            for k in ("K_prefix", "V_prefix", "K_tree", "V_tree")}
    out = api.tree_verify_attention(U.to_device(x["Q"], "bf16"), wide["K_prefix"], wide["V_prefix"], wide["K_tree"],
                                    wide["V_tree"], torch.from_numpy(x["prefix_len"].astype(np.int32)).cuda(),
                                    U.mask_to_device(mask))
    torch.cuda.synchronize()
    got16 = U.from_device_f64(out)
    scale = np.maximum(np.abs(got16), 1.0)
    assert (np.abs(got8 - got16) / scale).max() < 2.0 ** -6
