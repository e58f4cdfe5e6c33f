"""The partial key cache on the GPU (ig_slab_build) against its layout spelled out in numpy, byte for byte:
per (sequence, head), tiles of 512 half (256 float32) tokens, inside a tile one run of tokens per kept
channel, zeros past the valid tokens."""
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


# row lengths on both sides of every chunk size, rows that are no power of two, one kept column and all
# of them, one token, a chunk's and a tile's edges, spare capacity
@pytest.mark.parametrize("dtype,d,r,N,N_cap", [
    ("f16", 8, 1, 1, 1), ("f16", 64, 19, 127, 127), ("f16", 96, 28, 513, 700), ("f16", 128, 38, 128, 1100),
    ("f16", 128, 128, 1024, 1024), ("f16", 136, 5, 65, 65), ("f16", 256, 76, 512, 513),
    ("f32", 4, 4, 31, 300), ("f32", 64, 19, 257, 257), ("f32", 68, 20, 64, 256), ("f32", 128, 38, 255, 600), ("f32", 256, 76, 33, 40)])
@pytest.mark.parametrize("pinned", [False, True])
def test_layout_byte_for_byte(ctx, dtype, d, r, N, N_cap, pinned):
    check(ctx, dtype, d, r, N, N_cap, pinned, 2, 3)      # (fewer workgroups than compute units: 32 tokens each)


# enough pairs for every compute unit: 128, 64 and 32 tokens a workgroup by the length of a row
@pytest.mark.parametrize("dtype,d,r,N,N_cap", [
    ("f16", 8, 1, 1, 1), ("f16", 64, 19, 127, 127), ("f16", 96, 28, 513, 700), ("f16", 128, 38, 128, 1100), ("f16", 136, 5, 65, 65),
    ("f16", 256, 76, 512, 513), ("f32", 4, 4, 31, 300), ("f32", 64, 19, 257, 257), ("f32", 68, 20, 64, 256), ("f32", 256, 76, 33, 40)])
def test_layout_of_many_pairs(ctx, dtype, d, r, N, N_cap):
    check(ctx, dtype, d, r, N, N_cap, False, 16, 9)


def check(ctx, dtype, d, r, N, N_cap, pinned, B, H):
    import paper_2406_19707_amd as ig
    print(f"case {dtype} d{d} r{r} N{N} cap{N_cap} pinned {pinned}", flush=True)
    rng = np.random.default_rng(d * 7 + r + N)
    npdt = np.float16 if dtype == "f16" else np.float32
    K = rng.standard_normal((B, H, N_cap, d)).astype(npdt)
    idx = np.stack([np.sort(rng.choice(d, r, replace=False)) for _ in range(H)]).astype(np.int32)
    desc = ig.IgDesc(B=B, H=H, d=d, r=r, N=N, N_cap=N_cap, dtype=ig.IG_F16 if dtype == "f16" else ig.IG_F32)
    tile = 512 if dtype == "f16" else 256
    nt = -(-N_cap // tile)
    ref = np.zeros((B, H, nt * tile, r), npdt)
    for h in range(H):
        ref[:, h, :N] = K[:, h, :N][:, :, idx[h]]
    ref = ref.reshape(B, H, nt, tile, r).transpose(0, 1, 2, 4, 3)
    Kt = torch.from_numpy(K)
    Kt = Kt.pin_memory() if pinned else Kt.cuda()
    slab = torch.full((ig.ig_slab_bytes(desc),), 0x5A, dtype=torch.uint8, device="cuda")
    ctx.ig_slab_build(desc, Kt, ig.IG_MEM_HOST_PINNED if pinned else ig.IG_MEM_DEVICE, torch.from_numpy(idx).cuda(), slab)
    torch.cuda.synchronize()
    assert np.array_equal(slab.cpu().numpy(), np.ascontiguousarray(ref).reshape(-1).view(np.uint8))
