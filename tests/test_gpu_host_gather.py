"""Prefetch from a pinned host pool: lists of every length side by side (empty, one row, more rows than a workgroup
takes), totals below, at and above one unit a thread and one turn of the whole grid, rows of 16 bytes to 1 KiB, lists
longer than the stride, slots outside the pool.  Copies are bit-exact and nothing else is written."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2406_19707_amd as ig
    c = ig.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("B,H,d,dtype,N,counts", [
    (1, 1, 128, "f16", 40, [0]),
    (1, 3, 128, "f16", 40, [0, 1, 0]),
    (1, 2, 128, "f16", 640, [639, 1]),            # 640 rows = 10240 units: 40 workgroups of 256 just full
    (1, 2, 128, "f16", 642, [640, 1]),            # one row more
    (2, 5, 64, "f16", 300, "uneven"),             # 8 units a row
    (1, 7, 8, "f16", 500, "uneven"),              # one unit a row
    (3, 4, 96, "f16", 200, "uneven"),             # 12 units a row: no power of two
    (1, 3, 256, "f32", 150, "uneven"),            # 64 units a row
    (5, 100, 16, "f32", 60, "uneven"),            # more lists than threads
    (1, 4, 128, "f16", 100, [100, 100, 100, 100]),
])
def test_rows_are_copied_exactly(ctx, B, H, d, dtype, N, counts):
    import paper_2406_19707_amd as ig
    print("case", B, H, d, dtype, N, counts, flush=True)
    rng = np.random.default_rng(N + d)
    BH, tdt = B * H, torch.float16 if dtype == "f16" else torch.float32
    K, V = (torch.from_numpy(rng.standard_normal((BH, N, d))).to(tdt).pin_memory() for _ in range(2))
    cnt = np.array(counts if counts != "uneven" else np.minimum(N, rng.pareto(0.6, BH) * 3).astype(int))
    stride = max(1, int(cnt.max()) - 5) if counts == "uneven" else N        # (the longest lists are cut at the stride)
    idx = np.zeros((BH, stride), np.int64)
    for i in range(BH):
        n = min(cnt[i], stride)
        idx[i, :n] = np.sort(rng.choice(N, n, replace=False))
    shown = idx.copy()
    if counts == "uneven":
        shown[np.argmax(cnt), 0] = -7                # a slot outside the pool is clamped into it
        idx[np.argmax(cnt), 0] = 0
    desc = ig.IgDesc(B=B, H=H, d=d, r=1, N=N, dtype=ig.IG_F16 if dtype == "f16" else ig.IG_F32)
    Ks, Vs = (torch.full((BH, stride, d), 9.0, dtype=tdt, device="cuda") for _ in range(2))
    ctx.ig_gather_kv(desc, K, V, ig.IG_MEM_HOST_PINNED, torch.from_numpy(shown).to(torch.int32).cuda(), stride,
                     torch.from_numpy(cnt).to(torch.int32).cuda(), Ks, Vs)
    torch.cuda.synchronize()
    for pool, got in ((K, Ks.cpu()), (V, Vs.cpu())):
        for i in range(BH):
            n = min(cnt[i], stride)
            assert torch.equal(got[i, :n], pool[i, torch.from_numpy(idx[i, :n])]), i
            assert torch.all(got[i, n:] == 9.0), i
