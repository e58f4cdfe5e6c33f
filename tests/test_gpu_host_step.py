"""The host-pool decode step in one launch a layer (ig_decode_step_overlapped on folded half-precision shapes of up to
four tiles): outputs bit for bit those of the three calls a layer in order, for one and more layers, two and three
buffer sets, inputs that are an earlier layer's output, and with the side stream's own work before and behind the step
ordered as if the prefetches ran there."""
import ctypes

import pytest
import torch

import ig_workloads as wl
from ig_case import make_case

pytestmark = pytest.mark.gpu


class Step:
    """L layers over pinned pools, as a program holds them."""

    def __init__(self, B, H, d, N, L, n_sets, ratio=0.3, new_row=True):
        import paper_2406_19707_amd as ig
        from ig_gpu import Uploaded
        self.ig, self.ctx, self.L, self.BH, self.N = ig, ig.Context(0), L, B * H, N
        w = wl.shrink(wl.WORKLOADS[4], B=B, H=H, d=d, N=N, ratio=ratio, n_cal=2 * d, heavy_count=12)
        self.up = [Uploaded(self.ctx, make_case(w, gain=12.0, layer=l), host_pool=True) for l in range(L)]
        self.d = self.up[0].desc
        self.x = [u.x for u in self.up]
        self.out = [torch.zeros((B, H, d), dtype=torch.float16, device="cuda") for _ in range(L)]
        self.sets = [self.buffers() for _ in range(n_sets)]
        self.new_row = new_row

    def buffers(self):
        h = torch.float16
        return dict(sel_idx=torch.zeros((self.BH, self.N), dtype=torch.int32, device="cuda"),
                    sel_cnt=torch.zeros(self.BH, dtype=torch.int32, device="cuda"),
                    K_sel=torch.zeros((self.BH, self.N, self.d.d), dtype=h, device="cuda"),
                    V_sel=torch.zeros((self.BH, self.N, self.d.d), dtype=h, device="cuda"))

    def run(self, main, side):
        ig = self.ig
        io = (ig.IgLayerIO * self.L)(*[
            ig.IgLayerIO(x=self.x[l].data_ptr(), slab=u.slab.data_ptr(), q=u.q.data_ptr(), Kpool=u.K.data_ptr(), Vpool=u.V.data_ptr(),
                         k_new=u.k_new.data_ptr() if self.new_row else None, v_new=u.v_new.data_ptr() if self.new_row else None,
                         out=self.out[l].data_ptr()) for l, u in enumerate(self.up)])
        bufs = (ig.IgBufferSet * len(self.sets))(*[ig.IgBufferSet(**{k: t.data_ptr() for k, t in s.items()}) for s in self.sets])
        self.ctx.ig_decode_step_overlapped(self.d, io, self.up[0].wq, self.up[0].bias, None, None, ig.IG_MEM_HOST_PINNED, bufs,
                                           self.N, main, side)

    def in_order(self):
        """The calls of the step on one stream, rehearsal l behind attention l - 2."""
        b = [self.buffers() for _ in range(self.L)]
        want = [torch.zeros_like(o) for o in self.out]
        x = [t for t in self.x]
        alias = [next((k for k in range(self.L) if x[l].data_ptr() == self.out[k].data_ptr()), None) for l in range(self.L)]

        def attend(l):
            u, t = self.up[l], b[l]
            new = (u.k_new, u.v_new) if self.new_row else (None, None)
            self.ctx.ig_gather_kv(self.d, u.K, u.V, self.ig.IG_MEM_HOST_PINNED, t["sel_idx"], self.N, t["sel_cnt"], t["K_sel"], t["V_sel"])
            self.ctx.ig_sparse_attention(self.d, u.q, t["K_sel"], t["V_sel"], t["sel_cnt"], self.N, *new, want[l])
        for l in range(self.L):
            src = x[l] if alias[l] is None else want[alias[l]].reshape(x[l].shape)
            self.ctx.ig_speculate(self.d, src, self.up[0].wq, self.up[0].bias, None, None, self.up[l].slab, b[l]["sel_idx"], self.N,
                                  b[l]["sel_cnt"])
            if l >= 1:
                attend(l - 1)
        attend(self.L - 1)
        torch.cuda.synchronize()
        return want, b


def check(s, want, b):
    torch.cuda.synchronize()
    assert s.ctx.ig_check_status() == s.ig.IG_OK
    for l in range(s.L):
        assert torch.equal(s.out[l], want[l]), l
    for l in range(max(0, s.L - len(s.sets)), s.L):
        t, r = s.sets[l % len(s.sets)], b[l]
        assert torch.equal(t["sel_cnt"], r["sel_cnt"])
        for i in range(s.BH):
            n = int(r["sel_cnt"][i])
            assert torch.equal(t["sel_idx"][i, :n], r["sel_idx"][i, :n])
            assert torch.equal(t["K_sel"][i, :n], r["K_sel"][i, :n]) and torch.equal(t["V_sel"][i, :n], r["V_sel"][i, :n])


@pytest.mark.parametrize("B,H,d,N,L,n_sets,ratio,new_row", [
    (1, 4, 128, 600, 1, 2, 0.3, True),
    (2, 8, 128, 1500, 2, 2, 0.3, False),
    (2, 8, 64, 2048, 5, 2, 0.3, True),
    (1, 8, 64, 700, 4, 3, 0.05, True),
    (17, 4, 128, 300, 3, 2, 0.2, True),       # two blocks of 16 sequences
    (3, 4, 32, 513, 3, 3, 1.0, False),        # rows of 64 bytes: the attention's general form; every column kept
])
def test_outputs_and_sets_are_those_of_the_calls_in_order(B, H, d, N, L, n_sets, ratio, new_row):
    s = Step(B, H, d, N, L, n_sets, ratio, new_row)
    want, b = s.in_order()
    main, side = torch.cuda.Stream(), torch.cuda.Stream()
    s.ctx.ig_profile_begin()
    s.run(main, side)
    s.ctx.ig_profile_end()
    assert s.ctx.ig_profile_read(s.ig.IG_K_LAYER)[1] == L, "this shape is meant to take a launch a layer"
    check(s, want, b)
    for limit in (-1, 0):                      # every rehearsal alone, then the ordinary route on what that left
        for o in s.out:
            o.zero_()
        torch.cuda.synchronize()
        s.ctx.ig_set_wait_limit(limit)
        s.run(main, side)
        s.ctx.ig_set_wait_limit(0)
        check(s, want, b)
    s.ctx.close()


@pytest.mark.parametrize("back", [2, 3])
def test_an_input_may_be_an_earlier_layers_output(back):
    s = Step(2, 4, 128, 900, 5, 2)
    s.x[4] = s.out[4 - back]
    want, b = s.in_order()
    s.run(torch.cuda.Stream(), torch.cuda.Stream())
    check(s, want, b)
    s.ctx.close()


def test_an_input_may_lie_in_its_own_layers_list():
    s = Step(2, 4, 128, 900, 4, 2)
    want, b = s.in_order()
    lists = s.sets[3 % 2]["sel_idx"]           # the fourth layer's
    n = s.x[3].numel()
    # (that set is the second layer's too: the step must find the input there, so its lists may not reach that far)
    reach = int(b[1]["sel_cnt"][-1])
    s.x[3] = lists.view(-1)[-(n // 2):].view(torch.float16).view_as(s.x[3])
    assert n // 2 < s.N - reach
    s.x[3].copy_(s.up[3].x)
    s.ctx.ig_profile_begin()
    s.run(torch.cuda.Stream(), torch.cuda.Stream())
    s.ctx.ig_profile_end()
    assert s.ctx.ig_profile_read(s.ig.IG_K_LAYER)[1] == 0, "the rehearsal must not project beside the scan that writes the list"
    check(s, want, b)
    s.ctx.close()


def test_the_side_streams_own_work_is_ordered_around_the_prefetches():
    s = Step(2, 8, 128, 1500, 3, 2)
    main, side = torch.cuda.Stream(), torch.cuda.Stream()
    want0, b0 = s.in_order()
    victims = [b0[l]["sel_idx"][:, 0].contiguous() for l in range(s.L)]
    before, after = ([torch.randn((2, 8, 128), device="cuda").half() for _ in range(s.L)] for _ in range(2))
    scratch = [u.slab.clone() for u in s.up]

    def overwrite(rows):                       # slots that the step selects, in the pinned pools, on the side stream
        with torch.cuda.stream(side):
            torch.cuda._sleep(3_000_000)
        for l, u in enumerate(s.up):
            s.ctx.ig_pool_replace(s.d, victims[l], rows[l], rows[l], u.idx, scratch[l], u.K, u.V, s.ig.IG_MEM_HOST_PINNED, None, side)

    overwrite(before)
    s.run(main, side)
    overwrite(after)
    main.synchronize()
    got = [o.clone() for o in s.out]
    torch.cuda.synchronize()
    for l, u in enumerate(s.up):               # the pools as the step must have found them
        s.ctx.ig_pool_replace(s.d, victims[l], before[l], before[l], u.idx, scratch[l], u.K, u.V, s.ig.IG_MEM_HOST_PINNED, None)
    torch.cuda.synchronize()
    want, _ = s.in_order()
    for l in range(s.L):
        assert torch.equal(got[l], want[l]) and not torch.equal(got[l], want0[l]), l
    s.ctx.close()
