// One launch for two independent pieces of a decode step (Section 4.1, Fig. 3(d): the next layer
// is speculated while the current one computes): the scan / threshold / list kernel of the NEXT
// layer's rehearsal and the one-pass prefetch + attention of THIS layer.  The scan needs the next
// layer's partial query (sums of the launch before this one, or words of projecting workgroups in the
// same grid) and the attention needs this layer's index lists (the launch of the previous step), so
// neither depends on the other, and both are short, latency-bound kernels: run as the halves of one
// grid they share the launch and overlap fully, without streams or events between them.  The first
// workgroups project, where the projection is in the grid, B*H run the scan body (4 waves, one tile
// each), the remaining ones the attention body; the bodies are those of the stand-alone kernels, so the
// results are the same bit for bit.
#include "scan_device.h"
#include "attn_device.h"

namespace {

template <typename T, int CH, int LG>
__global__ __launch_bounds__(256) void scan_next_attend_this(ScanArgs sa, AttnArgs aa, int scan_blocks) {
  if ((int)blockIdx.x < scan_blocks)
    scan_select_fused_body<T, CH, 4>(sa, blockIdx.x);
  else
    sparse_attention_body<T, true, LG>(aa, (int)blockIdx.x - scan_blocks);
}

// The same with the next layer's projection in front, in the grid's first p.blocks workgroups (project_device.h): the
// projection, 4.6 us on its own, then runs beside the attention, which does not depend on it (four layers of 256
// pairs of 2048 tokens 98.7 -> 88.6 us).  The attention's registers leave room for four workgroups a compute
// unit; the matrix operands must not take a fifth of them away.
template <int CH, int LG>
__global__ __launch_bounds__(256, 4) void project_scan_next_attend_this(ScanArgs sa, AttnArgs aa, ProjWords p, int scan_blocks) {
  __shared__ __attribute__((aligned(16))) float red[PROJECT_LDS];
  const int id = (int)blockIdx.x - p.blocks;
  if (id >= scan_blocks)
    sparse_attention_body<half_t, true, LG>(aa, id - scan_blocks);
  else if (id >= 0)
    scan_select_fused_body<half_t, CH, 4, true>(sa, id, &p, red);
  else
    project_publish<1>(p, blockIdx.x, red);
}

template <int LG>
int launch_projecting(ig_ctx *ctx, const ScanArgs &sa, const AttnArgs &aa, const ProjWords &p, int BH, int ch, hipStream_t s) {
  dim3 grid(p.blocks + BH + BH * slices_at_most((long)aa.stride + 1, aa.slice_log2, aa.most_log2)), block(256);
#define CASE(CHV)                                                              \
  case CHV: {                                                                  \
    auto k = project_scan_next_attend_this<CHV, LG>;                           \
    IG_LAUNCH(ctx, IG_K_LAYER, k, grid, block, s, sa, aa, p, BH);              \
    return IG_OK;                                                              \
  }
  switch (ch) {
    CASE(4) CASE(8) CASE(12)
    default: break;
  }
#undef CASE
  return ig_fail(ctx, IG_ESHAPE, "layer step: unsupported channel block %d", ch);
}

// One layer of a host-pool decode step in one launch (Fig. 3(d)): the prefetch of layer l over PCIe, the rehearsal of
// layer l + 1 and the attention of layer l - 1.  None of them depends on another: the prefetch reads the lists that the
// launch before this one wrote, the attention the rows that one fetched, and the rehearsal writes a list set that only
// the attention still uses, of which it has a copy of the counts.  What bounds it is the link.  On two streams the
// list had to wait 15 us for its prefetch and the rows 11 us for their attention, each a hand-over between queues,
// and the link with them: three layers of 64 lists, 12239 rows whose prefetches take 126 us back to back, 186 us a step,
// 156 so (issued on an idle GPU 213 and 187, of which the host 120 and 60).
template <int LG>
__global__ __launch_bounds__(256, 4) void prefetch_rehearse_attend(GatherArgs ga, ScanArgs sa, AttnArgs aa, ProjWords p,
                                                                   int gather_blocks, int scan_blocks) {
  extern __shared__ int pre[];
  __shared__ __attribute__((aligned(16))) float red[PROJECT_LDS];
  int id = blockIdx.x;
  if (id < gather_blocks) {
    gather_flat_body(ga, id, gather_blocks, pre);
    return;
  }
  id -= gather_blocks + p.blocks;
  if (id >= scan_blocks)
    sparse_attention_body<half_t, false, LG>(aa, id - scan_blocks);
  else if (id >= 0)
    scan_select_fused_body<half_t, 12, 4, true>(sa, id, &p, red);
  else
    project_publish<1>(p, id + p.blocks, red);
}

template <typename T, int LG>
int launch_t(ig_ctx *ctx, const ScanArgs &sa, const AttnArgs &aa, int BH, int ch, hipStream_t s) {
  dim3 grid(BH + BH * slices_at_most((long)aa.stride + 1, aa.slice_log2, aa.most_log2)), block(256);
#define CASE(CHV)                                                              \
  case CHV: {                                                                  \
    auto k = scan_next_attend_this<T, CHV, LG>;                                \
    IG_LAUNCH(ctx, IG_K_LAYER, k, grid, block, s, sa, aa, BH);                 \
    return IG_OK;                                                              \
  }
  switch (ch) {
    CASE(4) CASE(8) CASE(12)
    default: break;
  }
#undef CASE
  return ig_fail(ctx, IG_ESHAPE, "layer step: unsupported channel block %d", ch);
}

}  // namespace

// The joint launch takes the shapes whose scan is the 4-wave one-workgroup-per-(b,h) form.
bool ig_layer_step_is_joint(const ig_desc *d) {
  const int tile = ig_tile_tokens(d->dtype);
  return ig_scan_is_fused(d) && (d->N + tile - 1) / tile <= 4;
}

int ig_launch_scan_attend(ig_ctx *ctx, const ig_desc *d, const QSource &qs, const void *slab,
                          int32_t *sel_idx_next, int32_t *sel_cnt_next, const void *q,
                          const void *Kpool, const void *Vpool, const int32_t *sel_idx,
                          const int32_t *sel_cnt, int32_t sel_stride, const void *k_new,
                          const void *v_new, void *out, void *K_sel, void *V_sel, hipStream_t s) {
  if (qs.A_p) return ig_fail(ctx, IG_EINVAL, "layer step: the joint launch takes no rotary query source");
  ScanArgs sa;
  int rc = ig_scan_args(ctx, d, qs, slab, sel_idx_next, sel_stride, sel_cnt_next, nullptr, &sa);
  if (rc) return rc;
  AttnArgs aa;
  if ((rc = ig_attn_args(ctx, d, q, Kpool, Vpool, sel_idx, sel_stride, sel_cnt, d->N_cap, k_new, v_new, out,
                         K_sel, V_sel, &aa)))
    return rc;
  // at most 12 channel loads in flight per wave: the scan half then fits the attention half's occupancy
  // (B8 H32 N2048 shape: 22.2-22.4 us per launch with 20 loads in flight where 12 took 20.4-20.8; with
  // the attention as it is now 12 take 18.5)
  const int ch = ig_pick_ch(d->r, 12);
  const int BH = d->B * d->H;
  if (qs.proj) {
    if (d->dtype != IG_F16) return ig_fail(ctx, IG_EINVAL, "layer step: the projection joins half precision only");
    // (a rolling window here: the channel count need not be a multiple of it)
    const int win = d->r <= 4 ? 4 : (d->r <= 8 ? 8 : 12);
    if (aa.lpr_log2 == 3) return launch_projecting<3>(ctx, sa, aa, *qs.proj, BH, win, s);
    if (aa.lpr_log2 == 4) return launch_projecting<4>(ctx, sa, aa, *qs.proj, BH, win, s);
    return launch_projecting<-1>(ctx, sa, aa, *qs.proj, BH, win, s);
  }
  if (d->dtype == IG_F16) {
    if (aa.lpr_log2 == 3) return launch_t<half_t, 3>(ctx, sa, aa, BH, ch, s);
    if (aa.lpr_log2 == 4) return launch_t<half_t, 4>(ctx, sa, aa, BH, ch, s);
    return launch_t<half_t, -1>(ctx, sa, aa, BH, ch, s);
  }
  return aa.lpr_log2 == 4 ? launch_t<float, 4>(ctx, sa, aa, BH, ch, s) : launch_t<float, -1>(ctx, sa, aa, BH, ch, s);
}

// The host-pool step's launch takes the folded half-precision shapes whose scan is the 4-wave form with the
// projection in its launch.
bool ig_host_step_is_joint(const ig_desc *d, const ProjGeom &g) {
  const int tile = ig_tile_tokens(d->dtype);
  return d->dtype == IG_F16 && !d->rope && ig_scan_joins_projection(d, g) && (d->N + tile - 1) / tile <= 4;
}

// next: the rehearsal (qs.proj set) or NULL, prev: the attention or NULL
int ig_launch_host_step(ig_ctx *ctx, const ig_desc *d, const void *Kpool, const void *Vpool, const int32_t *sel_idx,
                        const int32_t *sel_cnt, int32_t sel_stride, void *K_sel, void *V_sel, int32_t *cnt_copy,
                        const IgHostNext *next, const IgHostPrev *prev, hipStream_t s) {
  GatherArgs ga;
  int rc = ig_gather_args(ctx, d, Kpool, Vpool, sel_idx, sel_stride, sel_cnt, K_sel, V_sel, &ga);
  if (rc) return rc;
  ga.cnt_copy = cnt_copy;
  ScanArgs sa{};
  ProjWords p{};
  int scan_blocks = 0, attn_blocks = 0;
  if (next) {
    QSource qs{nullptr, 1, 0, 0, next->bias, nullptr, nullptr, next->proj};
    if ((rc = ig_scan_args(ctx, d, qs, next->slab, next->sel_idx, sel_stride, next->sel_cnt, nullptr, &sa))) return rc;
    p = *next->proj;
    scan_blocks = d->B * d->H;
  }
  AttnArgs aa{};
  if (prev) {
    if ((rc = ig_attn_args(ctx, d, prev->q, prev->K_sel, prev->V_sel, nullptr, sel_stride, prev->cnt, sel_stride, prev->k_new,
                           prev->v_new, prev->out, nullptr, nullptr, &aa)))
      return rc;
    attn_blocks = aa.BH * slices_at_most((long)sel_stride + 1, aa.slice_log2, aa.most_log2);
  }
  dim3 grid((unsigned)(GATHER_FLAT_BLOCKS + p.blocks + scan_blocks + attn_blocks)), block(256);
  const int row16_log2 = __builtin_ctz(d->d * 2 / 16);
  auto k = row16_log2 == 3 ? prefetch_rehearse_attend<3> : (row16_log2 == 4 ? prefetch_rehearse_attend<4> : prefetch_rehearse_attend<-1>);
  IG_LAUNCH_LDS(ctx, IG_K_LAYER, k, grid, block, (unsigned)ig_gather_lds(d), s, ga, sa, aa, p, (int)GATHER_FLAT_BLOCKS, scan_blocks);
  return IG_OK;
}
