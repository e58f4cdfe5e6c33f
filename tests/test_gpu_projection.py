"""The partial query (ig_project, ig_project_indexed) against float64 at the edges of its kernels: batch rows
around the blocks of 16 and around the powers of two of the FMA kernel, column blocks that do not fill a
workgroup, K slices of uneven length, heads of more than 256 columns behind the rotation.

Bound: the D-term float32 sum and the bias, (D + 2) 2^-24 of the sum of magnitudes (products of half values
are exact in float32); behind a rotation (done in double, rounded once) the same again over the d columns."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2406_19707_amd as ig
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = ig.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("dtype,H,d,r,rope,bias", [
    ("f16", 5, 64, 19, False, True),       # 6 column blocks: the second workgroup half empty; D = 320
    ("f16", 32, 128, 38, False, False),    # 76 blocks, 16 K slices of 8
    ("f16", 72, 128, 3, False, True),      # K slices of 18 pieces: over 16 batch rows without the LDS copy
    ("f16", 3, 80, 7, False, True),        # D = 240, no multiple of 32: FMA kernel
    ("f32", 4, 64, 19, False, False),
    ("f32", 7, 24, 24, False, True),
    ("f16", 4, 64, 38, True, True),
    ("f16", 2, 512, 100, True, False),     # two columns a thread
    ("f32", 3, 320, 256, True, True),      # one group of 256 outputs, more rows than are fetched ahead
    ("f16", 1, 64, 20, False, True),       # two partial sums
    ("f16", 2, 64, 30, True, False),       # four; 8 rows of A_p a thread
    ("f16", 3, 96, 96, True, True),        # 48 rows: 24 and three times 8
])
@pytest.mark.parametrize("B", [1, 2, 3, 5, 8, 9, 16, 17, 32, 33, 65, 100])
def test_partial_query_against_float64(ctx, dtype, H, d, r, rope, bias, B):
    import paper_2406_19707_amd as ig
    print(f"case {dtype} H{H} d{d} r{r} rope {rope} B{B}", flush=True)
    rng = np.random.default_rng(H * d + r + B)
    D, npdt = H * d, np.float16 if dtype == "f16" else np.float32
    x = rng.standard_normal((B, D)).astype(npdt)
    W = (rng.standard_normal((D, D)) / np.sqrt(D)).astype(npdt)
    idx = np.stack([np.sort(rng.choice(d, r, replace=False)) for _ in range(H)]).astype(np.int32)
    bv = rng.standard_normal(D if rope else H * r).astype(np.float32) if bias else None
    A = rng.standard_normal((H, d, r)).astype(np.float32) if rope else None
    pos = rng.integers(0, 40000, B).astype(np.int32) if rope else None
    desc = ig.IgDesc(B=B, H=H, d=d, r=r, N=8, dtype=ig.IG_F16 if dtype == "f16" else ig.IG_F32, rope=int(rope))
    dev = lambda a: None if a is None else torch.from_numpy(a).cuda()  # noqa: E731
    xd, Wd, idxd, bd, Ad, pd = map(dev, (x, W, idx, bv, A, pos))
    wq = torch.empty(ig.ig_wq_bytes(desc), dtype=torch.uint8, device="cuda")
    ctx.ig_wq_build(desc, Wd, idxd, wq)
    outs = [torch.full((B, H, r), float("nan"), device="cuda")]
    ctx.ig_project(desc, xd, wq, bd, Ad, pd, outs[0])
    if not rope and (d * x.itemsize) % 16 == 0:
        outs.append(torch.full((B, H, r), float("nan"), device="cuda"))
        ctx.ig_project_indexed(desc, xd, Wd, idxd, bd, outs[1])
    torch.cuda.synchronize()

    x64, W64 = x.astype(np.float64), W.astype(np.float64)
    q, mag = x64 @ W64, np.abs(x64) @ np.abs(W64)
    eps = (D + 2) * 2.0 ** -24
    if rope:
        b64 = 0.0 if bv is None else bv.astype(np.float64)
        q, err = (q + b64).reshape(B, H, d), (eps * (mag + np.abs(b64))).reshape(B, H, d)
        half = d // 2
        ang = pos[:, None] * 10000.0 ** (-2.0 * np.arange(half) / d)
        cs, sn = np.cos(ang)[:, None], np.sin(ang)[:, None]
        a, c = q[..., :half], q[..., half:]
        rot = np.concatenate([a * cs - c * sn, c * cs + a * sn], -1)
        e = err[..., :half] + err[..., half:]
        rerr = np.concatenate([e, e], -1) + 2.0 ** -24 * np.abs(rot)
        A64 = A.astype(np.float64)
        ref = np.einsum("bhc,hck->bhk", rot, A64)
        bound = np.einsum("bhc,hck->bhk", rerr + (d + 2) * 2.0 ** -24 * np.abs(rot), np.abs(A64))
    else:
        cols = (np.arange(H)[:, None] * d + idx).reshape(-1)
        b64 = 0.0 if bv is None else bv.astype(np.float64)
        ref, bound = (q[:, cols] + b64).reshape(B, H, r), (eps * (mag[:, cols] + np.abs(b64))).reshape(B, H, r)
    for o in outs:
        assert np.all(np.abs(o.cpu().numpy().astype(np.float64) - ref) <= bound)


# Small folded models: one kernel multiplies the weight, scans and selects (ig_speculate), with the sums of
# the three in the same order as the separate calls: the same scores and lists, bit for bit.  On both sides
# of its limits (32768 bytes of a head's weight columns, r = 64, four tiles).
@pytest.mark.parametrize("dtype,B,H,d,r,N,bias", [
    ("f32", 1, 4, 64, 19, 512, False), ("f32", 3, 4, 64, 19, 1024, True), ("f32", 2, 3, 8, 1, 1, True),
    ("f32", 2, 8, 64, 19, 700, True), ("f32", 1, 4, 48, 48, 257, False), ("f32", 1, 3, 64, 64, 1024, True),
    ("f32", 1, 3, 64, 64, 1025, False), ("f32", 5, 2, 80, 51, 300, True), ("f32", 5, 2, 80, 52, 300, False), ("f32", 1, 2, 128, 65, 300, False),
    ("f16", 2, 3, 80, 24, 700, True), ("f16", 40, 1, 8, 8, 2048, False), ("f16", 2, 5, 72, 64, 513, True),
    ("f16", 1, 3, 8, 3, 2049, False)])
def test_small_models_project_in_the_scan(ctx, dtype, B, H, d, r, N, bias):
    import paper_2406_19707_amd as ig
    print(f"case {dtype} B{B} H{H} d{d} r{r} N{N}", flush=True)
    torch.manual_seed(B + H * d + N)
    t, D = (torch.float16 if dtype == "f16" else torch.float32), H * d
    desc = ig.IgDesc(B=B, H=H, d=d, r=r, N=N, N_cap=N + 300, dtype=ig.IG_F16 if dtype == "f16" else ig.IG_F32, scale=0.4, alpha=3.0)
    W = (torch.randn(D, D, device="cuda") / D ** 0.5).to(t)
    idx = torch.stack([torch.randperm(d, device="cuda")[:r].sort().values for _ in range(H)]).to(torch.int32).contiguous()
    bv = torch.randn(H * r, device="cuda") if bias else None
    x, K = torch.randn(B, D, device="cuda").to(t), torch.randn(B, H, N + 300, d, device="cuda").to(t)
    wq = torch.empty(ig.ig_wq_bytes(desc), dtype=torch.uint8, device="cuda")
    slab = torch.empty(ig.ig_slab_bytes(desc), dtype=torch.uint8, device="cuda")
    ctx.ig_wq_build(desc, W, idx, wq)
    ctx.ig_slab_build(desc, K, ig.IG_MEM_DEVICE, idx, slab)

    def lists(stride, run):
        sel = torch.full((B * H, stride), -1, dtype=torch.int32, device="cuda")
        cnt = torch.full((B * H,), -1, dtype=torch.int32, device="cuda")
        scores = torch.full((B, H, N), float("nan"), device="cuda")
        run(sel, stride, cnt, scores)
        torch.cuda.synchronize()
        return sel.cpu().numpy(), cnt.cpu().numpy(), scores.cpu().numpy(), ctx.ig_check_status()

    def apart(sel, stride, cnt, scores):
        q_p = torch.zeros((B, H, r), device="cuda")
        ctx.ig_project(desc, x, wq, bv, None, None, q_p)
        ctx.ig_scan_select(desc, q_p, slab, sel, stride, cnt, scores)

    for stride in (N, max(1, N // 7)):
        one = lists(stride, lambda *a: ctx.ig_speculate(desc, x, wq, bv, None, None, slab, *a))
        two = lists(stride, apart)
        assert one[3] == two[3] and all(np.array_equal(u, v) for u, v in zip(one[:3], two[:3]))
        assert np.all(one[1] >= 1)
