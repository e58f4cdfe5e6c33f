"""GPU parity of the prefill-side partial weight index (ig_partial_index_device) against the
oracle's column ranking (Section 4.3 "Prefill Stage").  The GPU sums in float32, the oracle in
double: the kept sets must agree except for columns whose oracle sums lie within 1e-5 (relative)
of the r-th largest sum."""
import numpy as np
import pytest
import torch

from oracle import ig_oracle as o

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2406_19707_amd as ig
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = ig.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("H,d,n,ratio,dtype,with_keys", [
    (32, 128, 2048, 0.3, "f16", True),
    (4, 64, 512, 0.3, "f32", False),
    (5, 96, 333, 0.2, "f16", True),      # ragged rows / columns
    (2, 256, 40, 0.5, "f32", True),
    (3, 8, 7, 0.3, "f32", False),        # fewer rows than row chunks
])
def test_kept_columns_match_the_oracle(ctx, H, d, n, ratio, dtype, with_keys):
    import paper_2406_19707_amd as ig
    print(f"case H{H} d{d} n{n} ratio {ratio} {dtype} keys {with_keys}", flush=True)
    rng = np.random.default_rng(H * 1000 + d + n)
    npdt = np.float16 if dtype == "f16" else np.float32
    col_gain = rng.uniform(0.2, 3.0, (1, H * d))
    Qs = (rng.standard_normal((n, H * d)) * col_gain).astype(npdt)
    Ks = (rng.standard_normal((n, H * d)) * col_gain[:, ::-1]).astype(npdt) if with_keys else None
    ref = o.partial_index(Qs.astype(np.float32), None if Ks is None else Ks.astype(np.float32), H, ratio)
    r = ref.shape[1]
    idx = torch.full((H, r), -1, dtype=torch.int32, device="cuda")
    q_dev = torch.from_numpy(Qs).cuda()
    k_dev = None if Ks is None else torch.from_numpy(Ks).cuda()
    code = ig.IG_F16 if dtype == "f16" else ig.IG_F32
    ctx.ig_partial_index_device(code, H, d, n, q_dev, k_dev, ratio, idx)
    torch.cuda.synchronize()
    got = idx.cpu().numpy()
    again = torch.full_like(idx, -1)
    ctx.ig_partial_index_device(code, H, d, n, q_dev, k_dev, ratio, again)
    torch.cuda.synchronize()
    assert torch.equal(idx, again)                               # repeatable bit for bit
    sums = np.abs(Qs.astype(np.float64)).sum(0) + (0 if Ks is None else np.abs(Ks.astype(np.float64)).sum(0))
    for h in range(H):
        assert np.all(np.diff(got[h]) > 0) and got[h][0] >= 0 and got[h][-1] < d
        diff = np.setxor1d(got[h], ref[h])
        if diff.size:
            c = sums[h * d:(h + 1) * d]
            cut = np.sort(c)[::-1][r - 1]
            assert np.all(np.abs(c[diff] - cut) <= 1e-5 * cut), (h, diff)


def test_equal_sums_keep_the_lower_columns(ctx):
    import paper_2406_19707_amd as ig
    Qs = torch.ones((16, 2 * 64), dtype=torch.float32, device="cuda")
    idx = torch.zeros((2, 19), dtype=torch.int32, device="cuda")
    ctx.ig_partial_index_device(ig.IG_F32, 2, 64, 16, Qs, None, 0.3, idx)
    torch.cuda.synchronize()
    assert np.array_equal(idx.cpu().numpy(), np.tile(np.arange(19, dtype=np.int32), (2, 1)))


def test_error_paths(ctx):
    import paper_2406_19707_amd as ig
    buf = torch.zeros(4096, dtype=torch.uint8, device="cuda")
    p = buf.data_ptr()
    call = lambda *a: ctx.call("ig_partial_index_device", *a)  # noqa: E731
    assert call(ig.IG_F32, 2, 300, 4, p, None, 0.3, p, 0) == ig.IG_ESHAPE       # d > 256
    assert call(9, 2, 64, 4, p, None, 0.3, p, 0) == ig.IG_EDTYPE
    assert call(ig.IG_F32, 2, 64, 4, None, None, 0.3, p, 0) == ig.IG_EINVAL
    assert call(ig.IG_F32, 2, 64, 4, p, None, 0.0, p, 0) == ig.IG_EINVAL
    assert call(ig.IG_F32, 2, 2, 4, p, None, 0.3, p, 0) == ig.IG_ESHAPE         # floor(0.3 * 2) = 0


@pytest.mark.parametrize("dtype,H,d,n", [("f16", 3, 64, 100), ("f16", 3, 7, 33), ("f32", 2, 128, 31), ("f32", 5, 3, 600)])
def test_arrays_of_any_alignment_give_the_same_columns(ctx, dtype, H, d, n):
    """Wide loads need 8- or 16-byte rows and addresses; the same rows one element further in memory, and
    rows of odd length, take the one-column-a-lane form, which adds in the same order: equal results."""
    import paper_2406_19707_amd as ig
    rng = np.random.default_rng(n + d)
    tdt = torch.float16 if dtype == "f16" else torch.float32
    code = ig.IG_F16 if dtype == "f16" else ig.IG_F32
    Q, K = (torch.from_numpy(rng.standard_normal((n, H * d))).to(tdt) for _ in range(2))
    got = []
    for shift in (0, 1):
        bufs = [torch.zeros(n * H * d + 8, dtype=tdt, device="cuda") for _ in range(2)]
        q, k = (b[shift: shift + n * H * d] for b in bufs)
        q.copy_(Q.reshape(-1)), k.copy_(K.reshape(-1))
        idx = torch.full((H, int(0.4 * d)), -1, dtype=torch.int32, device="cuda")
        ctx.ig_partial_index_device(code, H, d, n, q, k, 0.4, idx)
        torch.cuda.synchronize()
        got.append(idx.cpu().numpy())
    assert np.array_equal(got[0], got[1])
    sums = np.abs(Q.double().numpy()).sum(0) + np.abs(K.double().numpy()).sum(0)
    for h in range(H):
        c = sums[h * d:(h + 1) * d]
        cut = np.sort(c)[::-1][got[0].shape[1] - 1]
        assert np.all(c[got[0][h]] >= cut * (1 - 1e-5))


@pytest.mark.parametrize("H,d", [(3, 64), (2, 128), (2, 250)])
def test_rows_with_nan_or_infinity_keep_r_columns(ctx, H, d):
    """Columns whose sum is NaN or infinite are kept first, the earlier ones before the later, and never more
    than r: nothing is written past a head's entries."""
    import paper_2406_19707_amd as ig
    n, r = 40, d // 4
    rng = np.random.default_rng(d)
    Q = rng.standard_normal((n, H, d)).astype(np.float32)
    Q[3, 0, [1, d // 2, d - 1]] = np.nan              # fewer than r
    Q[5, 0, 7] = np.inf
    Q[0, H - 1, d // 8:] = np.nan                     # more than r
    buf = torch.full((H * r + 256,), -7, dtype=torch.int32, device="cuda")
    print(f"case H{H} d{d} r{r}", flush=True)
    ctx.ig_partial_index_device(ig.IG_F32, H, d, n, torch.from_numpy(Q.reshape(n, H * d)).cuda(), None, 0.25, buf)
    torch.cuda.synchronize()
    got = buf.cpu().numpy()
    assert np.all(got[H * r:] == -7)
    sums = np.abs(Q.astype(np.float64)).sum(0)
    sums[~np.isfinite(sums)] = np.inf
    for h in range(H):
        want = np.sort(np.argsort(-sums[h], kind="stable")[:r])
        assert np.array_equal(got[h * r:(h + 1) * r], want), h


@pytest.mark.parametrize("n", [1, 32, 33, 129, 512, 513, 1025, 2049, 2600])
@pytest.mark.parametrize("dtype", ["f16", "f32"])
def test_row_counts_at_the_edges_of_a_waves_share(ctx, dtype, n):
    """A wave sums a quarter of one of 32 row ranges, 4, 8 or 16 rows at a time: counts at which waves or ranges
    are left without rows, a turn is just full or one row over, and a second turn starts.  float32 sums of n
    positive terms are within n * 2^-24 of the exact ones, whatever the order."""
    import paper_2406_19707_amd as ig
    H, d, r = 3, 64, 19
    rng = np.random.default_rng(n)
    npdt = np.float16 if dtype == "f16" else np.float32
    Q, K = (rng.standard_normal((n, H * d)).astype(npdt) for _ in range(2))
    idx = torch.full((H, r), -1, dtype=torch.int32, device="cuda")
    ctx.ig_partial_index_device(ig.IG_F16 if dtype == "f16" else ig.IG_F32, H, d, n, torch.from_numpy(Q).cuda(),
                                torch.from_numpy(K).cuda(), 0.3, idx)
    got = idx.cpu().numpy()
    sums = np.abs(Q.astype(np.float64)).sum(0) + np.abs(K.astype(np.float64)).sum(0)
    tol = 4 * n * 2.0 ** -24
    for h in range(H):
        c = sums[h * d:(h + 1) * d]
        cut = np.sort(c)[::-1][r - 1]
        assert np.all(np.diff(got[h]) > 0)
        assert np.all(c[got[h]] >= cut * (1 - tol))
        assert np.all(np.delete(c, got[h]) <= cut * (1 + tol))
