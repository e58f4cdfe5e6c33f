"""GPU parity of the offline skewing on the device (ig_skew_device) against the oracle's skew
(Section 4.2, Eq. 2 and Eq. 3).  A is only unique up to the spectrum's gaps, so the comparison goes
through what the paper fixes: A_h orthogonal, Q_h A_h has orthogonal columns of norms sigma
(descending, equal to the oracle's), Q~ K~^T = Q K^T; and element-wise where the singular values
are well separated."""
import numpy as np
import pytest
import torch

import ig_workloads as wl
from oracle import ig_oracle as o

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2406_19707_amd as ig
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = ig.Context(0)
    yield c
    c.close()


def skew_on_gpu(ctx, Qcal, H):
    n, D = Qcal.shape
    d = D // H
    A = torch.zeros((H, d, d), device="cuda")
    sigma = torch.zeros((H, d), device="cuda")
    ctx.ig_skew_device(D, H, n, torch.from_numpy(np.ascontiguousarray(Qcal, dtype=np.float32)).cuda(), A, sigma)
    torch.cuda.synchronize()
    return A.cpu().numpy().astype(np.float64), sigma.cpu().numpy().astype(np.float64), ctx.ig_check_status()


def check_invariants(Qcal, H, A, sigma, ref_sigma):
    n, D = Qcal.shape
    d = D // H
    rng = np.random.default_rng(0)
    K = rng.standard_normal((64, D))
    for h in range(H):
        Ah = A[h]
        assert np.abs(Ah.T @ Ah - np.eye(d)).max() <= 2e-6
        Qh = Qcal[:, h * d:(h + 1) * d].astype(np.float64)
        gram = (Qh @ Ah).T @ (Qh @ Ah)
        scale = max(1.0, gram.max())
        assert np.abs(gram - np.diag(np.diag(gram))).max() <= 2e-5 * scale       # columns orthogonal
        assert np.all(np.diff(sigma[h]) <= 1e-6 * sigma[h, 0])                   # descending
        assert np.abs(sigma[h] - ref_sigma[h]).max() <= 1e-4 * ref_sigma[h, 0]
        Kh = K[:, h * d:(h + 1) * d]
        full = Qh @ Kh.T
        assert np.abs((Qh @ Ah) @ (Kh @ Ah).T - full).max() <= 1e-5 * np.abs(full).max()
        assert np.all(np.abs(Ah).argmax(0) == (Ah * np.sign(Ah[np.abs(Ah).argmax(0), np.arange(d)])).argmax(0))


@pytest.mark.parametrize("cfg,H,d", [(1, 4, 64), (2, 4, 128), (2, 3, 32)])
def test_matches_the_oracle_on_workload_calibration_queries(ctx, cfg, H, d):
    w = wl.shrink(wl.WORKLOADS[cfg], H=H, d=d)
    print(f"case {w.name} H{H} d{d} n_cal {w.n_cal}", flush=True)
    Qcal = (wl.calibration_input(w) @ wl.projection_weight(w, "Wq")).astype(np.float32)
    ref = o.skew(None, None, Qcal, H)
    A, sigma, status = skew_on_gpu(ctx, Qcal, H)
    assert status == 0
    check_invariants(Qcal, H, A, sigma, ref["sigma"].astype(np.float64))
    # element-wise on the columns whose singular value is separated from its neighbours
    for h in range(H):
        s = ref["sigma"][h].astype(np.float64)
        gap = np.minimum(np.abs(np.diff(s, prepend=np.inf)), np.abs(np.diff(s, append=-np.inf))) / s[0]
        cols = gap > 1e-3
        assert cols.sum() >= d // 4
        assert np.abs(A[h][:, cols] - ref["A"][h][:, cols]).max() <= 2e-3


def test_fewer_rows_than_columns_still_gives_an_orthogonal_basis(ctx):
    rng = np.random.default_rng(5)
    H, d, n = 2, 64, 20                       # rank 20 < d: the null space is completed arbitrarily
    Qcal = rng.standard_normal((n, H * d)).astype(np.float32)
    ref = o.skew(None, None, Qcal, H)
    A, sigma, status = skew_on_gpu(ctx, Qcal, H)
    assert status == 0
    for h in range(H):
        assert np.abs(A[h].T @ A[h] - np.eye(d)).max() <= 2e-6
        assert np.abs(sigma[h][:n] - ref["sigma"][h][:n]).max() <= 1e-4 * ref["sigma"][h][0]
        assert np.all(sigma[h][n:] <= 1e-3 * sigma[h][0])
        Qh = Qcal[:, h * d:(h + 1) * d].astype(np.float64)
        assert np.abs((Qh @ A[h]) @ (Qh @ A[h]).T - Qh @ Qh.T).max() <= 1e-5 * np.abs(Qh @ Qh.T).max()


def test_error_paths(ctx):
    import paper_2406_19707_amd as ig
    buf = torch.zeros(1 << 16, dtype=torch.uint8, device="cuda")
    p = buf.data_ptr()
    assert ctx.call("ig_skew_device", 66, 2, 8, p, p, None, 0) == ig.IG_ESHAPE      # odd d
    assert ctx.call("ig_skew_device", 64, 3, 8, p, p, None, 0) == ig.IG_ESHAPE      # D % H
    assert ctx.call("ig_skew_device", 1024, 2, 8, p, p, None, 0) == ig.IG_ESHAPE    # d > 256
    assert ctx.call("ig_skew_device", 64, 2, 8, None, p, None, 0) == ig.IG_EINVAL


ROUNDED = 1.01 * 2.0 ** -23


@pytest.mark.parametrize("d,n,kind", [(2, 8, "full"), (30, 64, "full"), (64, 64, "full"), (66, 70, "graded"), (96, 1, "full"),
                                      (126, 400, "graded"), (128, 127, "full"), (128, 129, "graded"), (128, 40, "repeated"),
                                      (64, 33, "zero"), (130, 200, "full")])
def test_edges_of_the_kernels_against_64_bits(ctx, d, n, kind):
    """Heads around the tile and kernel edges (d = 64 / 66, 128 / 130), fewer rows than columns, repeated
    columns, an all-zero head, singular values over five decades: against numpy's SVD in 64 bits.
    Tolerances: A and sigma are float32 (2^-24 relative each).  Rounding moves a column of A by at most
    2^-24 of its length, so an inner product of two of them, and one through Q^T Q against sigma_0^2, by
    at most 2^-23; ROUNDED is that and 1 % for the arithmetic before the rounding.  sigma comes from the
    Gram matrix in 64 bits, whose smallest eigenvalues carry d * 2^-52 of the largest: 2e-7 of sigma_0
    covers both.
    (d = 130 takes the two-sided kernel, whose fixed 16 sweeps do not reach five decades: it reports
    IG_ENOCONV there, so that case has singular values of one size.)"""
    rng = np.random.default_rng(d * 1000 + n)
    H = 2
    Q = rng.standard_normal((n, H, d))
    if kind == "graded":
        Q *= 10.0 ** np.linspace(0, -5, d)
        Q = Q @ np.linalg.qr(rng.standard_normal((d, d)))[0]
    if kind == "repeated":
        Q[:, :, d // 2:] = Q[:, :, : d - d // 2]
    if kind == "zero":
        Q[:, 1] = 0
    Q32 = np.ascontiguousarray(Q.reshape(n, H * d), dtype=np.float32)
    A, sigma, status = skew_on_gpu(ctx, Q32, H)
    assert status == 0
    for h in range(H):
        Qh = Q32[:, h * d:(h + 1) * d].astype(np.float64)
        ref = np.zeros(d)
        ref[: min(n, d)] = np.linalg.svd(Qh, compute_uv=False)
        top = max(ref[0], 1e-30)
        assert np.abs(A[h].T @ A[h] - np.eye(d)).max() <= ROUNDED
        assert np.abs(sigma[h] - ref).max() <= 2e-7 * top
        gram = (Qh @ A[h]).T @ (Qh @ A[h])
        assert np.abs(gram - np.diag(np.diag(gram))).max() <= ROUNDED * top * top
        big = np.abs(A[h]).max(0)
        assert np.all(A[h].max(0) >= big * (1 - 1e-6))                 # largest entry positive


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("spread", [1e-1, 1e-2, 1e-3, 1e-4, 0.0])
def test_close_singular_values(ctx, d, spread):
    """Singular values within `spread` of each other, as near-orthonormal queries and a flat noise floor have
    them: the rotations of the last sweeps are large there however small the inner products are.  A must
    be as orthogonal as elsewhere, and each column the right singular vector: a vector is settled to
    the rounding of the matrix it comes from (d * 2^-52 of the largest eigenvalue, here and in numpy) over
    the distance of its eigenvalue to the next, a factor 2 under the singular values' own."""
    n, H = 4 * d, 2
    rng = np.random.default_rng(int(1e4 * spread) + d)
    heads = []
    for _ in range(H):
        U, W = np.linalg.qr(rng.standard_normal((n, d)))[0], np.linalg.qr(rng.standard_normal((d, d)))[0]
        heads.append((U * (1.0 + spread * np.linspace(1.0, 0.0, d))) @ W.T)
    Q32 = np.ascontiguousarray(np.concatenate(heads, 1), dtype=np.float32)
    A, sigma, status = skew_on_gpu(ctx, Q32, H)
    assert status == 0
    for h in range(H):
        Qh = Q32[:, h * d:(h + 1) * d].astype(np.float64)
        _, s, Vt = np.linalg.svd(Qh, full_matrices=False)
        print(f"case d{d} spread {spread} head {h}: A^T A - I {np.abs(A[h].T @ A[h] - np.eye(d)).max():.2e}", flush=True)
        assert np.abs(A[h].T @ A[h] - np.eye(d)).max() <= ROUNDED
        assert np.abs(sigma[h] - s).max() <= 2.0 ** -23 * s[0]
        gram = (Qh @ A[h]).T @ (Qh @ A[h])
        assert np.abs(gram - np.diag(np.diag(gram))).max() <= ROUNDED * s[0] ** 2
        gap = np.minimum(np.abs(np.diff(s, prepend=np.inf)), np.abs(np.diff(s, append=-np.inf))) / s[0]
        V = Vt.T * np.sign(Vt.T[np.abs(A[h]).argmax(0), np.arange(d)])
        settled = 2.0 ** -24 + 2 * d * 2.0 ** -52 / (2 * gap)
        assert np.all(np.abs(A[h] - V).max(0) <= settled), (np.abs(A[h] - V).max(0) / settled).max()


@pytest.mark.parametrize("d", [64, 128, 130])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_queries_that_are_not_finite_are_reported(ctx, d, bad):
    """As ig_skew_offline reports them; the other heads are not touched by it."""
    import paper_2406_19707_amd as ig
    rng = np.random.default_rng(d)
    n, H = 200, 3
    Q = rng.standard_normal((n, H * d)).astype(np.float32)
    A0, sigma0, status = skew_on_gpu(ctx, Q, H)
    assert status == ig.IG_OK
    Q[7, d + 5] = bad
    print(f"case d{d} {bad}", flush=True)
    A, sigma, status = skew_on_gpu(ctx, Q, H)
    assert status == ig.IG_ENOCONV and ctx.ig_check_status() == ig.IG_OK
    assert np.array_equal(A[[0, 2]], A0[[0, 2]]) and np.array_equal(sigma[[0, 2]], sigma0[[0, 2]])
    if d <= 128:
        assert np.isnan(A[1]).all() and np.isnan(sigma[1]).all()


@pytest.mark.parametrize("d", [34, 64, 96, 128])
@pytest.mark.parametrize("spread", [1e-3, 1e-4, 1e-5])
def test_many_heads_of_close_singular_values(ctx, d, spread):
    """Sixteen heads a case, so that some end their sweeps at the first look at all pairs and some at the second: every
    column settled as far as rounding and the distance of its eigenvalue allow (the bound of the test above)."""
    n, H = 4 * d, 16
    rng = np.random.default_rng(int(1e6 * spread) + d)
    heads = []
    for _ in range(H):
        U, W = np.linalg.qr(rng.standard_normal((n, d)))[0], np.linalg.qr(rng.standard_normal((d, d)))[0]
        heads.append((U * (1.0 + spread * np.linspace(1.0, 0.0, d))) @ W.T)
    Q32 = np.ascontiguousarray(np.concatenate(heads, 1), dtype=np.float32)
    A, sigma, status = skew_on_gpu(ctx, Q32, H)
    assert status == 0
    for h in range(H):
        _, s, Vt = np.linalg.svd(Q32[:, h * d:(h + 1) * d].astype(np.float64), full_matrices=False)
        assert np.abs(A[h].T @ A[h] - np.eye(d)).max() <= ROUNDED
        gap = np.minimum(np.abs(np.diff(s, prepend=np.inf)), np.abs(np.diff(s, append=-np.inf))) / s[0]
        V = Vt.T * np.sign(Vt.T[np.abs(A[h]).argmax(0), np.arange(d)])
        settled = 2.0 ** -24 + 2 * d * 2.0 ** -52 / (2 * gap)
        assert np.all(np.abs(A[h] - V).max(0) <= settled), (h, (np.abs(A[h] - V).max(0) / settled).max())
