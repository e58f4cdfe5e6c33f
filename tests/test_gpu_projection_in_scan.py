"""The projection inside the scan's launch (ig_speculate, ig_speculate_equalized and ig_layer_step in half
precision): lists equal to those of the two separate calls, ig_project and ig_scan_select, bit for bit -- both add
the same partial sums in the same order -- on the ordinary route, with every wait given up at once (each workgroup
works its query out alone), with waits so short that some run out and some do not, and on the ordinary route again
on the words these left behind."""
import numpy as np
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


# cfg, B, H, d, N, N_cap, ratio, gain, bias
SHAPES = [
    (2, 1, 3, 64, 500, 500, 0.06, 6.0, False),        # r 3: window of 4; 6 K blocks, so K slices of one and none
    (2, 2, 5, 64, 1100, 1200, 0.11, 6.0, True),       # r 7: window of 8, heads that straddle column blocks
    (2, 1, 4, 64, 2048, 2048, 0.18, 6.0, False),      # r 11: window of 12, four whole tiles
    (2, 3, 4, 64, 700, 700, 1.0, 6.0, True),          # r 64: three turns of 20 and 4 more; a wave without a tile
    (2, 17, 2, 128, 513, 600, 0.3, 8.0, False),       # 17 sequences: two blocks of 16 in two workgroups, the second one row
    (2, 18, 36, 128, 300, 300, 0.3, 8.0, True),       # 4608 columns (9 K blocks a slice): both blocks in one wave; 648 pairs
    (2, 32, 4, 64, 600, 600, 0.3, 6.0, False),        # 32 sequences, 128 pairs
    (2, 6, 32, 64, 3000, 3000, 0.3, 8.0, False),      # 6 tiles, run-time r: workgroups of 8 waves
    (2, 5, 26, 64, 4096, 4096, 1.0, 6.0, True),       # 8 tiles, r 64, workgroups of 8 waves, two whole quarters each
    (2, 4, 32, 64, 1024, 1024, 0.6, 8.0, False),      # r 38, 128 pairs
    (2, 8, 16, 64, 2700, 3000, 0.6, 12.0, True),      # r 38, 6 tiles: streaming form, one workgroup a pair
    (2, 2, 8, 64, 9000, 9000, 0.6, 10.0, False),      # split pairs, 4 tiles a workgroup
    (2, 3, 5, 64, 4700, 4800, 0.3, 8.0, True),        # split pairs, r at run time
    (2, 1, 2, 64, 130000, 130000, 0.4, 20.0, False),  # 16 tiles a workgroup
    (3, 8, 16, 64, 4096, 4096, 0.6, 30.0, False),     # rotary, one workgroup a pair
    (3, 4, 32, 64, 1500, 1500, 0.6, 30.0, True),      # rotary, one tile a wave; bias
    (5, 2, 40, 128, 20000, 20000, 0.2, 40.0, False),  # rotary, split pairs
    (3, 20, 8, 128, 2500, 2500, 0.3, 30.0, False),    # rotary, 20 sequences
]


def _case(cfg, B, H, d, N, N_cap, ratio, gain, bias):
    w = wl.shrink(wl.WORKLOADS[cfg], B=B, H=H, d=d, N=N, ratio=ratio, n_cal=2 * d, heavy_count=16)
    return make_case(w, gain=gain, bias=bias, N_cap=N_cap)


def _same(got, want):
    (idx, cnt), (idx0, cnt0) = got, want
    assert np.array_equal(cnt, cnt0)
    for i in range(len(cnt0)):
        assert np.array_equal(idx[i, :cnt0[i]], idx0[i, :cnt0[i]]), i


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "-".join(map(str, s)))
def test_lists_equal_those_of_the_separate_calls(ctx, shape):
    import paper_2406_19707_amd as ig
    from ig_gpu import Uploaded
    c = _case(*shape)
    print("case", shape, "r", c.r, flush=True)
    up, w = Uploaded(ctx, c), c.w

    def call(together, scores=None):
        idx = torch.full((w.B * w.H, c.N), -1, dtype=torch.int32, device="cuda")
        cnt = torch.full((w.B * w.H,), -1, dtype=torch.int32, device="cuda")
        if together:
            ctx.ig_speculate(up.desc, up.x, up.wq, up.bias, up.A_p, up.pos, up.slab, idx, c.N, cnt, scores)
        else:
            q_p = torch.zeros((w.B, w.H, c.r), device="cuda")
            ctx.ig_project(up.desc, up.x, up.wq, up.bias, up.A_p, up.pos, q_p)
            ctx.ig_scan_select(up.desc, q_p, up.slab, idx, c.N, cnt, scores)
        torch.cuda.synchronize()
        return idx.cpu().numpy(), cnt.cpu().numpy()

    s0, s1 = (torch.zeros((w.B, w.H, c.N), device="cuda") for _ in range(2))
    want = call(False, s0)
    ctx.ig_profile_begin()
    got = call(True, s1)
    ctx.ig_profile_end()
    assert ctx.ig_profile_read(ig.IG_K_PROJECT)[1] == 0, "this shape is meant to take one launch"
    _same(got, want)
    assert torch.equal(s0, s1)
    for limit in (-1, 1, -1, 100, 300):
        ctx.ig_set_wait_limit(limit)
        try:
            _same(call(True), want)
        finally:
            ctx.ig_set_wait_limit(0)
        _same(call(True), want)
    assert ctx.ig_check_status() == ig.IG_OK


@pytest.mark.parametrize("shape", [SHAPES[9], SHAPES[10], SHAPES[15], SHAPES[14]], ids=lambda s: "-".join(map(str, s)))
def test_equalised_lists_on_every_route(ctx, shape):
    import paper_2406_19707_amd as ig
    from ig_gpu import Uploaded
    c = _case(*shape)
    up, w = Uploaded(ctx, c), c.w

    def call():
        idx = torch.full((w.B * w.H, c.N), -1, dtype=torch.int32, device="cuda")
        cnt, thr = (torch.full((w.B * w.H,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
        ctx.ig_speculate_equalized(up.desc, up.x, up.wq, up.bias, up.A_p, up.pos, up.slab, 0.2, idx, c.N, cnt, thr)
        torch.cuda.synchronize()
        return idx.cpu().numpy(), cnt.cpu().numpy()

    idx = torch.full((w.B * w.H, c.N), -1, dtype=torch.int32, device="cuda")
    cnt, thr = (torch.full((w.B * w.H,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
    q_p, scores = torch.zeros((w.B, w.H, c.r), device="cuda"), torch.zeros((w.B, w.H, c.N), device="cuda")
    ctx.ig_project(up.desc, up.x, up.wq, up.bias, up.A_p, up.pos, q_p)
    ctx.ig_scan_select(up.desc, q_p, up.slab, idx, c.N, thr, scores)
    ctx.ig_equalize_heads(up.desc, scores, thr, 0.2, idx, c.N, cnt)
    torch.cuda.synchronize()
    want = idx.cpu().numpy(), cnt.cpu().numpy()
    _same(call(), want)
    for limit in (-1, 100):
        ctx.ig_set_wait_limit(limit)
        try:
            _same(call(), want)
        finally:
            ctx.ig_set_wait_limit(0)
        _same(call(), want)
    assert ctx.ig_check_status() == ig.IG_OK


@pytest.mark.parametrize("d,r_ratio,B,H", [(64, 0.05, 3, 4), (64, 0.3, 18, 4), (128, 0.3, 2, 6), (32, 0.5, 2, 8)])
def test_layer_step_in_one_launch_on_every_route(ctx, d, r_ratio, B, H):
    """The joint launch with the projection in it: lists and outputs equal to the calls one by one."""
    from ig_gpu import Uploaded
    c = _case(2, B, H, d, 1300, 1300, r_ratio, 6.0, True)
    up, w = Uploaded(ctx, c), c.w
    BH, t16 = B * H, torch.float16

    def bufs():
        return dict(idx=torch.full((BH, c.N), -1, dtype=torch.int32, device="cuda"),
                    cnt=torch.full((BH,), -1, dtype=torch.int32, device="cuda"),
                    K=torch.zeros((BH, c.N, d), dtype=t16, device="cuda"), V=torch.zeros((BH, c.N, d), dtype=t16, device="cuda"),
                    out=torch.zeros((B, H, d), dtype=t16, device="cuda"))

    first = bufs()
    ctx.ig_speculate(up.desc, up.x, up.wq, up.bias, None, None, up.slab, first["idx"], c.N, first["cnt"])
    want = bufs()
    ctx.ig_gather_attention(up.desc, up.q, up.K, up.V, first["idx"], c.N, first["cnt"], want["K"], want["V"], up.k_new,
                            up.v_new, want["out"])
    torch.cuda.synchronize()
    want_lists = first["idx"].cpu().numpy(), first["cnt"].cpu().numpy()
    for limit in (0, -1, 100, 0):
        got = bufs()
        ctx.ig_set_wait_limit(limit)
        try:
            ctx.ig_layer_step(up.desc, up.x, up.wq, up.bias, None, None, up.slab, got["idx"], got["cnt"], up.q, up.K, up.V,
                              first["idx"], first["cnt"], c.N, got["K"], got["V"], up.k_new, up.v_new, got["out"])
            torch.cuda.synchronize()
        finally:
            ctx.ig_set_wait_limit(0)
        _same((got["idx"].cpu().numpy(), got["cnt"].cpu().numpy()), want_lists)
        assert torch.equal(got["K"], want["K"]) and torch.equal(got["V"], want["V"]) and torch.equal(got["out"], want["out"])
