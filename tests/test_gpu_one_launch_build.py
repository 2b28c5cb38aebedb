"""Builds whose scan and drafting are one launch (needs an MI355X), at the ends of the ranges of its forms: the trees must be
those of the two launches of the timed entry point bit for bit (the scan's forms and the order of every sum are the same), on a
workspace of any contents, again on the workspace that a build has left, and also where the drafting workgroup gives up waiting at once
and the workgroup of the last row drafts instead."""
import ctypes as C

import pytest

pytestmark = pytest.mark.gpu

FIELDS = ("token", "parent", "depth", "score", "mask", "n_out", "expect")


def _logits(V, n, d, B, dtype, seed, ragged=0):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    x = torch.randn((B, d, n, V + ragged), generator=g, device="cuda").mul_(3.5)
    x.scatter_add_(3, torch.randint(0, V, (B, d, n, 1), generator=g, device="cuda"), torch.full((B, d, n, 1), 6.0, device="cuda"))
    return x.to(torch.bfloat16 if dtype == "bf16" else torch.float32)[..., :V]


class _Build:
    def __init__(self, x, k, n, d):
        import torch
        from paper_2406_17276_amd import api
        self.x, self.p = x, api.build_params(x, k, n, d)
        g = torch.Generator(device="cuda")
        g.manual_seed(5)
        self.ws = torch.randint(0, 256, (api.build_workspace_bytes(self.p),), generator=g, device="cuda", dtype=torch.uint8)
        self.out = api.alloc_tree(self.p.batch, n)
        self.steps = torch.empty(self.p.batch, dtype=torch.int32, device="cuda")
        self.e = torch.empty(self.p.batch, dtype=torch.float64, device="cuda")

    def __call__(self, polls, delta=None):
        import torch
        from paper_2406_17276_amd import api
        for f in FIELDS:
            getattr(self.out, f).fill_(-7)
        one, o = C.c_int32(-1), self.out.c_struct()
        st = api.lib().ot_internal_build_tree(
            C.byref(self.p), C.c_int32(delta is not None), C.c_double(delta or 0.0), C.c_void_p(self.x.data_ptr()),
            C.c_void_p(self.ws.data_ptr()), C.c_size_t(self.ws.numel()), C.byref(o), C.c_void_p(self.steps.data_ptr()),
            C.c_void_p(self.e.data_ptr()), C.c_int32(polls), C.byref(one), C.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert st == 0, st
        torch.cuda.synchronize()
        return one.value, [getattr(self.out, f).clone() for f in FIELDS] + ([self.steps.clone(), self.e.clone()] if delta is not None else [])


def _equal(a, b):
    import torch
    return all(torch.equal(x.view(torch.uint8), y.view(torch.uint8)) for x, y in zip(a, b))


def _streamed(x, k, n, d, delta):
    """Algorithm 1's loop by the streaming calls: tree fields, steps drafted and last E_sub of every sequence."""
    import torch
    from paper_2406_17276_amd import api
    ts = api.TreeStream(x.shape[0], x.shape[3], k, n, d, api.OT_BF16 if x.dtype == torch.bfloat16 else api.OT_F32, "cuda")
    steps, last = None, None
    for t in range(d):
        ts.expand(x[:, t])
        e, go = ts.e_sub(delta)
        if t == 0:
            steps, last, live = torch.ones_like(go), e.clone(), go.clone()
        else:
            steps, last, live = steps + live, torch.where(live != 0, e, last), go.clone()
    tree = ts.finalize()
    torch.cuda.synchronize()
    return [getattr(tree, f) for f in FIELDS], steps, last


@pytest.mark.parametrize("V,k,n,d,B,dtype,ragged", [
    (1000, 4, 16, 4, 1, "f32", 0),          # 256 threads a row; one candidate each
    (8192, 16, 32, 5, 3, "bf16", 0),        # its longest row, two candidates each (512)
    (8184, 2, 200, 10, 2, "bf16", 1),       # rows at any alignment; more than 64 nodes, pool of many
    (500, 3, 1, 12, 32, "f32", 0),          # one node, the most sequences
    (8193, 10, 50, 10, 1, "bf16", 0),       # 1024 threads; one candidate each by 512 of them
    (32000, 16, 64, 4, 2, "bf16", 0),       # 1024 candidates
    (32003, 6, 33, 7, 3, "bf16", 3),
    (20000, 9, 65, 5, 2, "f32", 0),         # 640 threads draft
    (40000, 16, 64, 3, 2, "bf16", 0),       # 512 threads, rolling; two candidates each
    (33000, 5, 20, 6, 2, "f32", 0),         # 1024 threads, rolling
    (131072, 4, 9, 4, 2, "bf16", 0),        # the longest row of one part
])
def test_one_launch_equals_two(V, k, n, d, B, dtype, ragged):
    x = _logits(V, n, d, B, dtype, V + n, ragged)
    want = _timed(x, k, n, d)
    build = _Build(x, k, n, d)
    for polls in (30000, 30000, 0, 1, 30000):
        print(V, k, n, d, B, dtype, "polls", polls, flush=True)
        one, got = build(polls)
        assert one == 1
        assert _equal(got, want), polls
    fields, steps, e = _streamed(x, k, n, d, 0.05)
    first = None
    for polls in (30000, 0, 30000):
        one, got = build(polls, 0.05)
        assert one == 1
        first = first or got
        assert _equal(got, first), polls
    for f, a, b in zip(FIELDS, first, fields):
        # E and the scores: normalisers whose fp32 terms were added in another order (scan forms differ with the number of rows)
        assert a.allclose(b, rtol=1e-6, atol=1e-6) if f in ("score", "expect") else a.equal(b), f
    assert first[-2].equal(steps) and first[-1].allclose(e, rtol=1e-6, atol=0)


@pytest.mark.parametrize("V,k,n,d,B,dtype", [
    (1000, 1, 16, 6, 1, "f32"), (4000, 8, 32, 2, 1, "bf16"), (131080, 4, 9, 3, 1, "bf16"), (1000, 4, 16, 4, 33, "f32"),
    (4000, 16, 33, 4, 1, "bf16"), (32000, 16, 65, 4, 1, "bf16"),
])
def test_builds_that_go_in_two_launches(V, k, n, d, B, dtype):
    build = _Build(_logits(V, n, d, B, dtype, 3), k, n, d)
    one, got = build(30000)
    assert one == 0
    assert _equal(build(30000)[1], got)


def test_replays_of_a_captured_build_with_other_inputs():
    import torch
    from paper_2406_17276_amd import api
    V, k, n, d, B = 9000, 8, 40, 6, 2
    x = _logits(V, n, d, B, "bf16", 1)
    ws = torch.empty(api.build_workspace_bytes(api.build_params(x, k, n, d)), dtype=torch.uint8, device="cuda")
    out = api.alloc_tree(B, n)
    api.build_tree(x, k, n, d, out=out, workspace=ws)
    torch.cuda.synchronize()
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.stream(side), torch.cuda.graph(graph, stream=side):
        for _ in range(2):
            api.build_tree(x, k, n, d, out=out, workspace=ws)
    for replay in range(4):
        x.copy_(_logits(V, n, d, B, "bf16", 10 + replay))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        got = [getattr(out, f).clone() for f in FIELDS]
        assert _equal(_timed(x, k, n, d), got), replay


def _timed(x, k, n, d):
    """The same trees by scan and drafting as two launches."""
    import torch
    from paper_2406_17276_amd import api
    ref = api.PreparedBuild(x, k, n, d)
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    for e in ev:
        e.record()
    ref.timed(torch.cuda.current_stream().cuda_stream, ev[0].cuda_event, ev[1].cuda_event)
    torch.cuda.synchronize()
    return [getattr(ref.out, f).clone() for f in FIELDS]


@pytest.mark.parametrize("V,k,n,d,B,dtype,ragged", [
    (1000, 4, 16, 4, 1, "f32", 0),          # steps of one launch: 256 threads a row
    (8184, 16, 64, 5, 3, "bf16", 1),        # the most nodes, more than ten candidates a node
    (8184, 16, 65, 5, 3, "bf16", 1),        # 65 nodes: two launches a step
    (8192, 11, 64, 4, 4, "bf16", 0),        # 256 rows in the last steps: the most that go in one launch
    (8192, 8, 52, 4, 5, "bf16", 0),         # 260: two launches there
    (32000, 10, 50, 10, 1, "bf16", 0),      # 1024 threads
    (9000, 4, 32, 5, 8, "f32", 0),          # 256 rows of 1024 threads
    (40000, 8, 20, 5, 4, "bf16", 0),        # 512 threads, rolling
    (131072, 12, 9, 3, 2, "bf16", 0),       # the longest row of one part
    (131080, 3, 9, 3, 2, "bf16", 0),        # two parts
])
def test_streaming_steps_equal_the_one_shot_build(V, k, n, d, B, dtype, ragged):
    import torch
    from paper_2406_17276_amd import api
    x = _logits(V, n, d, B, dtype, 3 * V + n, ragged)
    want = api.build_tree(x, k, n, d)
    F = api.frontier_sizes(k, n, d)
    for go in (range(2)):                   # a second builder on the memory that the first has left
        ts = api.TreeStream(B, V, k, n, d, api.OT_BF16 if dtype == "bf16" else api.OT_F32, "cuda")
        for t in range(d):
            print(V, k, n, d, B, dtype, "step", t, flush=True)
            ts.expand(x[:, t])
            torch.cuda.synchronize()
            assert ts.frontier_count.tolist() == [F[t + 1]] * B
        got = ts.finalize()
        torch.cuda.synchronize()
        for f in ("token", "parent", "depth", "mask", "n_out"):
            assert torch.equal(getattr(got, f), getattr(want, f)), f
        # fp32 roundings of doubles that differ in the last places (scan forms differ with the number of rows)
        assert torch.allclose(got.score, want.score, rtol=1e-6, atol=1e-6)
        del ts


def test_a_stopped_sequence_stays_as_it_is_in_steps_of_one_launch():
    import torch
    from paper_2406_17276_amd import api
    V, k, n, d, B = 2000, 6, 30, 5, 3
    x = _logits(V, n, d, B, "bf16", 11)
    x[1] = 0
    x[1, ..., 7] = 60.0                     # one token has all of the probability: E grows by one node a step, of which nearly none adds
    ts = api.TreeStream(B, V, k, n, d, api.OT_BF16, "cuda")
    counts = []
    for t in range(d):
        ts.expand(x[:, t])
        e, go = ts.e_sub(1.0)
        torch.cuda.synchronize()
        counts.append((ts.frontier_count.tolist(), go.tolist()))
    tree, steps, _ = api.build_tree_adaptive(x, k, n, d, 1.0)
    got = ts.finalize()
    torch.cuda.synchronize()
    for b in range(B):
        for t in range(d):
            assert (counts[t][0][b] == 0) == (t >= int(steps[b])), (b, t, counts, steps)
    for f in ("token", "parent", "depth", "mask", "n_out"):
        assert torch.equal(getattr(got, f), getattr(tree, f)), f


@pytest.mark.parametrize("V,k,n,d,B,dtype", [
    (8184, 2, 200, 10, 2, "bf16"),          # seven steps that keep all of their candidates, and so have one barrier each
    (1000, 2, 200, 14, 1, "bf16"),          # 1455 rows: marking them takes 23 trips
    (9000, 4, 65, 6, 3, "f32"),             # 1024 threads; more than 64 nodes
    (1000, 4, 16, 4, 1, "f32"),
])
def test_a_wait_that_is_given_up_at_any_step(V, k, n, d, B, dtype):
    import torch
    build = _Build(_logits(V, n, d, B, dtype, 17), k, n, d)
    _, want = build(30000)
    words = [0x9d3f5be1c7604a2b - 2**64, 0x6b1e88d2f0957c43, 0x5c27f4a98e61d03b]      # kRowThere, kRowLate, kMarksMade
    for polls in range(24):
        print(V, k, n, d, B, dtype, "polls", polls, flush=True)
        one, got = build(polls)
        assert one == 1
        assert _equal(got, want), polls
        left = build.ws[:build.ws.numel() // 8 * 8].view(torch.int64)
        assert not any(bool((left == w).any()) for w in words), polls


# Rows that one workgroup scans in the same form however many there are
FORMS = [
    (8000, 6, 33, 5, "bf16"),               # 256 threads, rows in registers
    (20000, 12, 70, 4, "f32"),              # 1024
    (40000, 8, 20, 5, "bf16"),              # 512 threads, rolling
    (100000, 5, 9, 6, "bf16"),              # 1024, rolling
]


@pytest.mark.parametrize("V,k,n,d,dtype", FORMS)
@pytest.mark.parametrize("what", ["masked", "few", "none", "lowest", "nan"])
def test_masked_tokens_and_nans(V, k, n, d, dtype, what):
    import torch
    x = _logits(V, n, d, 2, dtype, V + k)
    g = torch.Generator(device="cuda")
    g.manual_seed(k)
    if what == "masked":                    # nine tokens in ten, whole vectors among them
        x[torch.rand(x.shape, generator=g, device="cuda") < 0.9] = -float("inf")
        x[..., 64:4096] = -float("inf")
    elif what == "few":                     # fewer tokens than children
        x[0, :, ::2, 3:] = -float("inf")
    elif what == "none":
        x[0, 0], x[1, 1, ::3] = -float("inf"), -float("inf")
    elif what == "lowest":
        x[0, :, ::2, k // 2:] = torch.finfo(x.dtype).min
    else:                                   # outside of what is promised, but the same in every form; a wavefront of them in a row
        x[torch.rand(x.shape, generator=g, device="cuda") < 1e-3] = float("nan")
        x[1, 1, 1, 1024:2048] = float("nan")
    want = _timed(x, k, n, d)
    build = _Build(x, k, n, d)
    one, got = build(30000)
    assert one == 1
    assert _equal(got, want)
    if what != "nan":
        fields, steps, e = _streamed(x, k, n, d, -1.0)
        for f, a, b in zip(FIELDS, got, fields):
            if f not in ("score", "expect"):
                assert a.equal(b), f


@pytest.mark.parametrize("V,k,n,d,dtype", FORMS)
@pytest.mark.parametrize("delta", [-1.0, 0.02, 0.3])
def test_adaptive_build_equals_two_launches(V, k, n, d, dtype, delta):
    x = _logits(V, n, d, 1, dtype, V + n)
    one, got = _Build(x, k, n, d)(30000, delta)
    two, want = _Build(x.expand(33, -1, -1, -1), k, n, d)(30000, delta)       # more than 32 sequences
    assert (one, two) == (1, 0)
    for a, b in zip(got, want):
        for i in range(33):
            assert _equal([a[:1]], [b[i:i + 1]])


@pytest.mark.parametrize("V,k,n,d,dtype", [c for c in FORMS if c[2] <= 64])
@pytest.mark.parametrize("masked", [False, True])
def test_streaming_steps_equal_two_launches(V, k, n, d, dtype, masked):
    import torch
    from paper_2406_17276_amd import api
    x = _logits(V, n, d, 1, dtype, V + 2 * n)
    if masked:
        x[..., 5:V // 2] = -float("inf")
        x[:, 2, ::2, 2:] = -float("inf")
        x[:, 1, 1] = -float("inf")
    got = []
    for B in (1, 300):                      # more than 256 rows: two launches a step
        ts = api.TreeStream(B, V, k, n, d, api.OT_BF16 if dtype == "bf16" else api.OT_F32, "cuda")
        step = []
        for t in range(d):
            ts.expand(x[:, t].expand(B, -1, -1))
            step += [a.clone() for a in (ts.frontier_token, ts.frontier_parent, ts.frontier_count, ts.frontier_mask())]
            step += [a.clone() for a in ts.e_sub(-1.0)]
        tree = ts.finalize()
        torch.cuda.synchronize()
        got.append(step + [getattr(tree, f) for f in FIELDS])
    for a, b in zip(*got):
        for i in (0, 1, 299):
            assert _equal([a[:1]], [b[i:i + 1]])


def test_builds_on_two_streams_at_once():
    import torch
    from paper_2406_17276_amd import api
    cases = [(8192, 4, 40, 7, 4, "bf16"), (32000, 10, 50, 10, 2, "bf16")]
    jobs = []
    for V, k, n, d, B, dtype in cases:
        x = _logits(V, n, d, B, dtype, V)
        jobs.append((_timed(x, k, n, d), [api.PreparedBuild(x, k, n, d) for _ in range(2)], torch.cuda.Stream()))
    torch.cuda.synchronize()
    for _ in range(50):                     # each on its stream, its two workspaces in turn
        for _, builds, stream in jobs:
            for build in builds:
                build(stream.cuda_stream)
    torch.cuda.synchronize()
    for want, builds, _ in jobs:
        for build in builds:
            assert _equal([getattr(build.out, f) for f in FIELDS], want)
