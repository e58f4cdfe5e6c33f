"""The projection as a kernel of its own in half precision -- more than 32 sequences, or a capture on a context
without query words -- in front of the scans that otherwise hold it: folded and rotary, plain and equalised, one
workgroup a pair and split pairs, and the layer step.  Lists equal those of the calls one by one, bit for bit, on
the ordinary route and with every wait given up at once."""
import pytest
import torch

import ig_workloads as wl
from ig_case import make_case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2406_19707_amd as ig
    c = ig.Context(0)
    yield c
    c.close()


def uploaded(ctx, cfg, B, H, d, N, ratio, gain, bias):
    from ig_gpu import Uploaded
    w = wl.shrink(wl.WORKLOADS[cfg], B=B, H=H, d=d, N=N, ratio=ratio, n_cal=2 * d, heavy_count=16)
    return Uploaded(ctx, make_case(w, gain=gain, bias=bias))


def lists(BH, N):
    return torch.full((BH, N), -1, dtype=torch.int32, device="cuda"), torch.full((BH,), -1, dtype=torch.int32, device="cuda")


def same(got, want):
    (idx, cnt), (idx0, cnt0) = got, want
    assert torch.equal(cnt, cnt0)
    kept = torch.arange(idx.shape[1], device="cuda")[None, :] < cnt0[:, None]
    assert torch.equal(idx[kept], idx0[kept])


def profiled(ctx, f):
    import paper_2406_19707_amd as ig
    ctx.ig_profile_begin()
    f()
    ctx.ig_profile_end()
    return {k: ctx.ig_profile_read(getattr(ig, k))[1] for k in ("IG_K_PROJECT", "IG_K_FINALIZE", "IG_K_SCAN", "IG_K_LAYER")}


def on_every_route(ctx, call, want):
    for limit in (-1, 100, 0):
        ctx.ig_set_wait_limit(limit)
        try:
            same(call(), want)
        finally:
            ctx.ig_set_wait_limit(0)


# cfg, B, H, d, N, ratio, gain, bias
SHAPES = [
    (3, 36, 4, 64, 1500, 0.6, 30.0, True),       # rotary, r 38, one tile a wave
    (3, 33, 4, 128, 4096, 0.3, 30.0, False),     # rotary, r 38, two tiles a wave
    (3, 34, 4, 128, 2100, 0.2, 30.0, True),      # rotary, r 25, two tiles a wave, the last one part of a tile
    (5, 33, 2, 64, 9000, 0.4, 40.0, False),      # rotary, r 25, split pairs
    (2, 40, 4, 64, 2700, 0.6, 12.0, True),       # folded, r 38, streaming form
    (2, 33, 2, 64, 9000, 0.6, 10.0, False),      # folded, r 38, split pairs
    (2, 35, 1, 64, 4700, 0.3, 8.0, True),        # folded, r 19 at run time, split pairs
    (2, 40, 4, 64, 1100, 0.3, 8.0, False),       # folded, r 19, block-loading form
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "-".join(map(str, s)))
def test_lists_of_more_than_32_sequences(ctx, shape):
    print("case", shape, flush=True)
    up = uploaded(ctx, *shape)
    w, N = up.c.w, up.c.N
    s0, s1 = (torch.zeros((w.B, w.H, N), device="cuda") for _ in range(2))
    want, q_p = lists(w.B * w.H, N), torch.zeros((w.B, w.H, up.c.r), device="cuda")
    ctx.ig_project(up.desc, up.x, up.wq, up.bias, up.A_p, up.pos, q_p)
    ctx.ig_scan_select(up.desc, q_p, up.slab, want[0], N, want[1], s0)
    assert bool((want[1] > 0).all())

    def call(scores=None):
        got = lists(w.B * w.H, N)
        ctx.ig_speculate(up.desc, up.x, up.wq, up.bias, up.A_p, up.pos, up.slab, got[0], N, got[1], scores)
        return got
    launches = profiled(ctx, lambda: same(call(s1), want))
    assert launches["IG_K_PROJECT"] == 1 and launches["IG_K_FINALIZE"] == 0 and launches["IG_K_SCAN"] == 1
    assert torch.equal(s0, s1)
    on_every_route(ctx, call, want)


@pytest.mark.parametrize("shape", [SHAPES[0], SHAPES[1], SHAPES[2], SHAPES[4]], ids=lambda s: "-".join(map(str, s)))
def test_equalised_lists_of_more_than_32_sequences(ctx, shape):
    print("case", shape, flush=True)
    up = uploaded(ctx, *shape)
    w, N = up.c.w, up.c.N
    want, thr = lists(w.B * w.H, N), lists(w.B * w.H, N)
    q_p, scores = torch.zeros((w.B, w.H, up.c.r), device="cuda"), torch.zeros((w.B, w.H, N), device="cuda")
    ctx.ig_project(up.desc, up.x, up.wq, up.bias, up.A_p, up.pos, q_p)
    ctx.ig_scan_select(up.desc, q_p, up.slab, thr[0], N, thr[1], scores)
    ctx.ig_equalize_heads(up.desc, scores, thr[1], 0.2, want[0], N, want[1])

    def call():
        got = lists(w.B * w.H, N)
        ctx.ig_speculate_equalized(up.desc, up.x, up.wq, up.bias, up.A_p, up.pos, up.slab, 0.2, got[0], N, got[1], None)
        return got
    launches = profiled(ctx, lambda: same(call(), want))
    assert launches["IG_K_PROJECT"] == 1 and launches["IG_K_FINALIZE"] == 0 and launches["IG_K_SCAN"] == 1
    on_every_route(ctx, call, want)


@pytest.mark.parametrize("cfg,B,H,d,N,ratio,gain,joint", [
    (2, 36, 4, 64, 1300, 0.3, 6.0, True),
    (2, 33, 4, 64, 3000, 0.6, 12.0, False),
    (3, 36, 4, 64, 2700, 0.6, 30.0, False),
])
def test_layer_step_of_more_than_32_sequences(ctx, cfg, B, H, d, N, ratio, gain, joint):
    up = uploaded(ctx, cfg, B, H, d, N, ratio, gain, True)
    BH = B * H
    this = lists(BH, N)
    ctx.ig_speculate(up.desc, up.x, up.wq, up.bias, up.A_p, up.pos, up.slab, this[0], N, this[1])

    def rows():
        return [torch.zeros(s, dtype=torch.float16, device="cuda") for s in ((BH, N, d), (BH, N, d), (B, H, d))]
    want, got, nxt = rows(), rows(), lists(BH, N)
    ctx.ig_gather_attention(up.desc, up.q, up.K, up.V, *this[:1], N, this[1], want[0], want[1], up.k_new, up.v_new, want[2])

    def step():
        ctx.ig_layer_step(up.desc, up.x, up.wq, up.bias, up.A_p, up.pos, up.slab, nxt[0], nxt[1], up.q, up.K, up.V, this[0],
                          this[1], N, got[0], got[1], up.k_new, up.v_new, got[2])
    for limit in (0, -1, 100):
        for t in (*got, *nxt):
            t.fill_(-1)
        for g in got[:2]:
            g.zero_()
        ctx.ig_set_wait_limit(limit)
        try:
            launches = profiled(ctx, step)
        finally:
            ctx.ig_set_wait_limit(0)
        assert launches["IG_K_PROJECT"] == 1 and launches["IG_K_LAYER"] == (1 if joint else 0)
        same(nxt, this)
        assert all(torch.equal(g, r) for g, r in zip(got, want))


@pytest.mark.parametrize("cfg,H,d,N,ratio,gain", [
    (2, 4, 64, 2700, 0.6, 12.0),         # split pairs
    (2, 4, 64, 900, 0.3, 8.0),           # block-loading form
    (3, 40, 64, 1500, 0.6, 30.0),        # rotary prologue
])
def test_captured_without_query_words(cfg, H, d, N, ratio, gain):
    """A context that has only served more than 32 sequences holds every workspace of a smaller batch but the query
    words: a capture takes the projection as a kernel of its own, allocates nothing, and its replays, with eager work
    on the same context between them, give the lists of the joined launch."""
    import paper_2406_19707_amd as ig
    print("case", cfg, H, d, N, ratio, flush=True)
    ctx, other = ig.Context(0), ig.Context(0)
    large, up = uploaded(ctx, cfg, 36, H, d, N, ratio, gain, True), uploaded(other, cfg, 4, H, d, N, ratio, gain, True)
    big, want, got = lists(36 * H, N), lists(4 * H, N), lists(4 * H, N)

    def call(c, u, out):
        c.ig_speculate(u.desc, u.x, u.wq, u.bias, u.A_p, u.pos, u.slab, out[0], N, out[1])
    call(ctx, large, big)
    call(other, up, want)
    torch.cuda.synchronize()
    held = ctx.ig_workspace_bytes()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=torch.cuda.Stream()):
        call(ctx, up, got)
    assert ctx.ig_workspace_bytes() == held
    for _ in range(3):
        for t in got:
            t.fill_(-1)
        call(ctx, large, big)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        same(got, want)
    joined = lists(4 * H, N)
    call(ctx, up, joined)                # outside the capture the words are allocated
    assert ctx.ig_workspace_bytes() > held
    same(joined, want)
    for c in (ctx, other):
        assert c.ig_check_status() == ig.IG_OK
        c.close()
