"""Pool counters and victims at the edges of the kernels' batches (1024 list entries, 1024 or 4096 slots) and of their
16-byte loads (capacities that are no multiple of four, counters that lie on four bytes), bit-exact against the
oracle; what lies behind the valid slots and in front of an unaligned array stays as it is."""
import numpy as np
import pytest
import torch

from oracle import ig_oracle as o

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,N_cap,stride,shift", [
    (1, 1, 1, 0), (3, 4, 3, 0), (4, 4, 4, 1), (255, 257, 100, 0), (1023, 1024, 1023, 0), (1025, 1028, 1025, 0),
    (1025, 1027, 1024, 0), (4095, 4096, 2049, 0), (4096, 4096, 4096, 2), (4097, 4100, 4097, 0), (4097, 4099, 1025, 0)])
def test_batch_edges(N, N_cap, stride, shift):
    import paper_2406_19707_amd as ig
    print(f"case N{N}/{N_cap} stride {stride} counters {4 * shift} bytes off", flush=True)
    rng = np.random.default_rng(N + stride)
    BH, cmax = 7, 5
    ctx = ig.Context(0)
    d = ig.IgDesc(B=1, H=BH, d=64, r=8, N=N, N_cap=N_cap)
    counters = rng.integers(1, cmax, (BH, N_cap)).astype(np.int32)
    counters[:, N:] = 0                                  # never a victim, never halved
    counters[1, :N] = 3                                  # ties: the lowest slot
    flat = torch.full((BH * N_cap + shift,), 77, dtype=torch.int32, device="cuda")
    c_dev = flat[shift:].view(BH, N_cap)
    c_dev.copy_(torch.from_numpy(counters))
    victim = torch.full((BH,), -1, dtype=torch.int32, device="cuda")
    for most in (0, min(N, stride), min(N, stride), max(1, min(N, stride) // 2)):
        idx = rng.integers(-2, N + 3, (BH, stride)).astype(np.int32)        # (entries behind a list mean nothing)
        cnt = np.array([most if i % 2 else rng.integers(0, most + 1) for i in range(BH)], np.int32)
        for i, n in enumerate(cnt):
            idx[i, :n] = np.sort(rng.choice(N, n, replace=False))
        o.pool_touch(counters, idx, cnt, N, counter_max=cmax)
        ctx.ig_pool_touch(d, torch.from_numpy(idx).cuda(), stride, torch.from_numpy(cnt).cuda(), c_dev, cmax)
        ctx.ig_pool_victim(d, c_dev, victim)
        torch.cuda.synchronize()
        assert np.array_equal(c_dev.cpu().numpy(), counters)
        assert np.array_equal(victim.cpu().numpy(), o.pool_victim(counters, N))
        assert bool((flat[:shift] == 77).all())
    ctx.close()
