"""Lists at the edges of the row slices that fetch and attention are cut into (a batch of a workgroup's
loads, or 128 rows, but no more than two batches; 16 slices at most), for every row length the attention has a form for, against
float64.

Bound of an attention output: a logit is a d-term float32 sum, scaled, and goes through exp, so it is off by
at most (d + 4) 2^-24 sum|q k| scale + 2^-22; a weight by that factor, twice with the normaliser; the weighted
sum of n rows by n 2^-23 more; and the result is rounded to its type."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

ROWS = [0, 1, 2, 31, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 513, 1023, 1024, 1025, 2047, 2048, 2049, 4095, 4096, 4097, 4300, 4500]


@pytest.fixture(scope="module")
def ctx():
    import paper_2406_19707_amd as ig
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = ig.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("dtype,d", [("f16", 8), ("f16", 32), ("f16", 64), ("f16", 128), ("f16", 256), ("f16", 512),
                                     ("f32", 4), ("f32", 32), ("f32", 64), ("f32", 128), ("f32", 256), ("f16", 96), ("f32", 512)])
@pytest.mark.parametrize("stride,new_row", [(4500, True), (4500, False), (200, True)])
def test_lists_at_slice_edges(ctx, dtype, d, stride, new_row):
    check(ctx, dtype, d, stride, new_row, ROWS, 4500)


def test_many_lists_of_long_rows(ctx):
    # 1024-byte rows: 64 of them a slice up to 255 lists, 128 from there
    check(ctx, "f32", 256, 300, True, [0, 1, 63, 64, 65, 127, 128, 129, 255, 256, 257, 300] * 22, 300)


def check(ctx, dtype, d, stride, new_row, lengths, N):
    import paper_2406_19707_amd as ig
    print(f"case {dtype} d{d} stride {stride} new {new_row}", flush=True)
    rng = np.random.default_rng(d + stride)
    npdt, half = (np.float16, True) if dtype == "f16" else (np.float32, False)
    B, H = 2, len(lengths) // 2
    q, kn, vn = (rng.standard_normal((B, H, d)).astype(npdt) for _ in range(3))
    K, V = (rng.standard_normal((B * H, N, d)).astype(npdt) for _ in range(2))
    cnt = np.minimum(np.array(lengths, np.int32)[rng.permutation(len(lengths))], stride).astype(np.int32)
    idx = np.zeros((B * H, stride), np.int32)
    for i, n in enumerate(cnt):
        idx[i, :n] = np.sort(rng.choice(N, n, replace=False))
    scale = 0.7 / np.sqrt(d)
    desc = ig.IgDesc(B=B, H=H, d=d, r=1, N=N, dtype=ig.IG_F16 if half else ig.IG_F32, scale=scale)
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    qd, knd, vnd, Kd, Vd, idxd, cntd = map(dev, (q, kn, vn, K, V, idx, cnt))
    new = (knd, vnd) if new_row else (None, None)
    tdt = torch.float16 if half else torch.float32
    fill = lambda: torch.full((B * H, stride, d), 7.0, dtype=tdt, device="cuda")  # noqa: E731
    Ks, Vs, Kf, Vf = fill(), fill(), fill(), fill()
    ctx.ig_gather_kv(desc, Kd, Vd, ig.IG_MEM_DEVICE, idxd, stride, cntd, Ks, Vs)
    attend = d != 96 and (dtype, d) != ("f32", 512)   # (rows of 16 * 2^k bytes, at most 1024)
    outs = [torch.zeros((B, H, d), dtype=tdt, device="cuda") for _ in range(3)]
    if attend:
        ctx.ig_sparse_attention(desc, qd, Ks, Vs, cntd, stride, *new, outs[0])
        ctx.ig_sparse_attention_indexed(desc, qd, Kd, Vd, idxd, stride, cntd, *new, outs[1])
        ctx.ig_gather_attention(desc, qd, Kd, Vd, idxd, stride, cntd, Kf, Vf, *new, outs[2])
    torch.cuda.synchronize()
    assert ctx.ig_check_status() == ig.IG_OK
    for i, n in enumerate(cnt):
        for src, copies in ((K, (Ks, Kf)), (V, (Vs, Vf))):
            for c in copies[:2 if attend else 1]:
                got = c[i].cpu().numpy()
                assert np.array_equal(got[:n], src[i, idx[i, :n]]) and np.all(got[n:] == 7.0), (i, n)
        if not attend:
            continue
        b, h = divmod(i, H)
        k64, v64 = K[i, idx[i, :n]].astype(np.float64), V[i, idx[i, :n]].astype(np.float64)
        if new_row:
            k64, v64 = np.vstack([k64, kn[b, h][None]]), np.vstack([v64, vn[b, h][None]])
        rows = len(k64)
        if rows == 0:
            for o in outs:
                assert np.all(o[b, h].cpu().numpy() == 0)
            continue
        q64 = q[b, h].astype(np.float64)
        l = k64 @ q64 * np.float64(np.float32(scale))
        p = np.exp(l - l.max())
        p /= p.sum()
        ref = p @ v64
        off = (d + 4) * 2.0 ** -24 * (np.abs(k64) @ np.abs(q64)).max() * scale + 2.0 ** -22
        bound = (2 * off + rows * 2.0 ** -23) * (p @ np.abs(v64)) + (2.0 ** -11 if half else 2.0 ** -24) * np.abs(ref) + 2.0 ** -24
        for o in outs:
            assert np.all(np.abs(o[b, h].cpu().numpy().astype(np.float64) - ref) <= bound), (i, n)
