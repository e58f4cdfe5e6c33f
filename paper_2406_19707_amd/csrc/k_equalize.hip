// Head-equalised selection (Section 4.3 "Decoding Stage", closing sentences: every head of a
// layer fetches the same number of tokens, the average over the heads of the tokens between the
// maximum score and the threshold; Section 5.1 "Key Metric": at most 20 % of the cache per layer).
//
// Input: the speculated scores s [B,H,N] and the per-head threshold counts of ig_speculate.
// One workgroup per (sequence, head):
//   n      = clamp(floor(sum_h count[b,h] / H), 1, cap)
//   T      = the n-th largest score of the head, found exactly by a most-significant-digit radix
//            select on an order-preserving integer image of the float (at most 3 passes of 11 bits, one
//            2048-bin LDS histogram each).  The scores of a head stay in registers (KPT per thread)
//            when they fit; longer sequences re-read them from L2 in every pass.
//   list   = tokens with score > T, plus the earliest tokens with score == T until n are kept,
//            written in ascending token order with ballot / bit-count prefix ranks.
// Integer work after the scores: the result is exact for the scores given.
#include "ig_internal.h"

namespace {

// order-preserving image of a float: larger float <-> larger unsigned; -0 is folded onto +0
__device__ __forceinline__ unsigned score_key(float s) {
  const unsigned b = __float_as_uint(s + 0.0f);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

__device__ __forceinline__ int wave_total(int v) { return __builtin_amdgcn_readlane(wave_incl_scan(v), 63); }
// A chain of dependent steps rather than work (192 heads of 3000 tokens are 2.3 MB), so the steps are few: a
// wave owns KPT * 64 consecutive tokens, whose keys stay in registers; every wave searches the histogram for
// itself, which leaves one barrier in a pass; 11 bits a pass instead of 8 are a pass less, spread the sign,
// exponent and leading bits over enough bins for the LDS adds not to queue up, and mostly settle the list in
// two passes (when a bin is kept whole nothing below it matters); and the ordered compaction needs one
// barrier, for the waves' totals, instead of two for every THREADS tokens.  (With the scan before it, whose
// share is 3 to 7 us: 32 lists of 4096 tokens 26.3 -> 13.1 us, 192 of 3000 20.8 -> 13.3 us, 1120 of 2048
// 32.6 -> 26.0 us.)
template <int THREADS, int KPT>
__global__ __launch_bounds__(THREADS) void equalize_select(const float *__restrict__ scores,
                                                           const int32_t *__restrict__ thr_cnt,
                                                           int32_t *__restrict__ sel_idx,
                                                           int32_t *__restrict__ sel_cnt,
                                                           int32_t *status, FastDiv by_H, int N, int cap,
                                                           int stride) {
  constexpr int NW = THREADS / 64, U = KPT > 0 ? KPT : 8;
  __shared__ __attribute__((aligned(16))) unsigned hist[3][RADIX_WORDS];
  __shared__ int w_gt[NW], w_eq[NW];
  const int H = by_H.d, bh = blockIdx.x, b = by_H.div(bh);
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float *s = scores + (long)bh * N;
  const int32_t *cnts = thr_cnt + (long)b * H;
  // the wave's tokens t0 .. t1 - 1, a multiple of 64 but for the end of the sequence
  const int chunk = KPT > 0 ? KPT * 64 : ((N + THREADS - 1) / THREADS) * 64;
  const int t0 = min(N, w * chunk), t1 = min(N, t0 + chunk);

  // f(token, its key, whether there is such a token) in token order, 64 tokens a call
  float raw[U];
  auto load = [&](int t) {
#pragma unroll
    for (int i = 0; i < U; ++i) raw[i] = s[min(t + i * 64 + lane, N - 1)];
  };
  auto each = [&](auto &&f) {
    if constexpr (KPT > 0) {
#pragma unroll
      for (int i = 0; i < U; ++i) f(t0 + i * 64 + lane, score_key(raw[i]), t0 + i * 64 + lane < t1);
    } else {
      for (int t = t0; t < t1; t += U * 64) {
        load(t);
#pragma unroll
        for (int i = 0; i < U; ++i) f(t + i * 64 + lane, score_key(raw[i]), t + i * 64 + lane < t1);
      }
    }
  };
  if constexpr (KPT > 0) load(t0);

  // ---- n: truncated mean of the sequence's threshold counts, capped ----
  int part = cnts[min(lane, H - 1)];
  part = lane < H ? part : 0;
  for (int h = lane + 64; h < H; h += 64) part += cnts[h];
  for (int i = tid; i < 3 * RADIX_WORDS / 4; i += THREADS) reinterpret_cast<uint4 *>(&hist[0][0])[i] = make_uint4(0, 0, 0, 0);
  int need = max(1, min(min(by_H.div(max(0, wave_total(part))), cap), N));
  __syncthreads();

  // ---- radix select of the n-th largest key ----
  // T: the kept tokens are those with a key above T and the first `need` of those equal to it
  unsigned T = 0;
#pragma unroll
  for (int pass = 0; pass < 3; ++pass) {
    each([&](int, unsigned k, bool there) {
      if (there) radix_add(hist[pass], pass, k, T);
    });
    __syncthreads();
    bool whole;
    T |= radix_digit(hist[pass], lane, need, &whole) << radix_shift(pass);
    if (pass < 2 && whole && T > 0) {
      T -= 1;                      // the bin is kept whole: everything from its lowest key upwards
      need = 0;
      break;
    }
  }

  // ---- ordered compaction ----
  int gt = 0, eq = 0;
  each([&](int, unsigned k, bool there) {
    gt += __popcll(__ballot(there && k > T));
    eq += __popcll(__ballot(there && k == T));
  });
  if (lane == 0) {
    w_gt[w] = gt;
    w_eq[w] = eq;
  }
  __syncthreads();
  int gt_all = 0, eq_all = 0, pos = 0, eq_rank = 0;      // before this wave's tokens, and in all
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    const int g = w_gt[i], e = w_eq[i];
    pos += i < w ? g : 0;
    eq_rank += i < w ? e : 0;
    gt_all += g;
    eq_all += e;
  }
  pos = __builtin_amdgcn_readfirstlane(pos + min(eq_rank, need));
  eq_rank = __builtin_amdgcn_readfirstlane(eq_rank);
  int32_t *list = sel_idx + (long)bh * stride;
  each([&](int t, unsigned k, bool there) {
    const unsigned long long be = __ballot(there && k == T);
    const bool keep = there && (k > T || (k == T && eq_rank + lanes_below(be) < need));
    const unsigned long long bk = __ballot(keep);
    const int at = pos + lanes_below(bk);
    if (keep && at < stride) list[at] = t;
    pos += __popcll(bk);
    eq_rank += __popcll(be);
  });
  if (tid == 0) {
    const int kept = gt_all + min(eq_all, need);
    sel_cnt[bh] = min(kept, stride);
    if (kept > stride) atomicOr(status, IG_STATUS_CAPACITY);
  }
}

}  // namespace

int ig_launch_equalize(ig_ctx *ctx, const ig_desc *d, const float *scores, const int32_t *thr_cnt,
                       int cap, int32_t *sel_idx, int32_t sel_stride, int32_t *sel_cnt,
                       hipStream_t s) {
  const int BH = d->B * d->H;
#define EQ_CASE(THREADS, KPT)                                                                      \
  {                                                                                                \
    auto k = equalize_select<THREADS, KPT>;                                                        \
    IG_LAUNCH(ctx, IG_K_SELECT, k, dim3(BH), dim3(THREADS), s, scores, thr_cnt, sel_idx, sel_cnt,  \
              ctx->status, ig_fast_div(d->H), (int)d->N, cap, (int)sel_stride);                            \
    return IG_OK;                                                                                  \
  }
  // 512 threads while every workgroup has a compute unit's waves nearly to itself (192 lists of 3000 tokens
  // with their scan 16.0 -> 13.3 us, 20.8 us before both), 256 where several
  // workgroups share one anyway (1120 lists of 2048: 26.0 against 27.3 us with the scan)
  if (BH <= 512) {
    if (d->N <= 512 * 4) EQ_CASE(512, 4)
    if (d->N <= 512 * 8) EQ_CASE(512, 8)
  }
  if (d->N <= 256 * 8) EQ_CASE(256, 8)
  if (d->N <= 256 * 16) EQ_CASE(256, 16)
  if (d->N <= 1024 * 16) EQ_CASE(1024, 16)
  if (d->N <= 1024 * 32) EQ_CASE(1024, 32)
  EQ_CASE(1024, 0)
#undef EQ_CASE
}
