// Partial key cache construction (Section 4.3 "Prefill Stage"), prefetch of the selected K/V rows
// (Section 4.1, Section 4.3) and decode attention over the fetched rows (Section 2.1).
#include "attn_device.h"

namespace {

// ---- slab build ---------------------------------------------------------------------------------
// A workgroup takes CHUNK consecutive tokens of one (b,h): the full key rows (a kept column in every
// 64-byte line or nearly, so whole rows are what has to be read) come in 16-byte loads, all of a thread's
// in flight at once (also when the pool is pinned host memory), go to LDS row by row, and the kept channels
// are picked out of LDS and written to the tile's channel planes, 16 bytes = VEC consecutive tokens a lane.
// HBM-bound; CHUNK rows are 32 KiB in flight a workgroup and 34 KiB of LDS, four workgroups a compute
// unit.  256 pairs of 2048 tokens, 38 of 128 half columns (134 MB read, 40 MB written): 33 us
// = 5.3 TB/s, the rate of a large copy, against 43.8 us with 32 tokens a workgroup and 2-byte accesses on
// both sides of the LDS.
// The LDS row is padded by 8 bytes: consecutive tokens of one column then fall two banks apart.
template <typename T, int CHUNK, int U>     // U: row units a thread has in flight
__global__ __launch_bounds__(256) void slab_build(const T *__restrict__ Kpool,
                                                  const int32_t *__restrict__ idx,
                                                  T *__restrict__ slab, int H, int d, int r, int N,
                                                  int N_cap, int nTiles) {
  constexpr int TPL = Elem<T>::TPL;              // elements of a pool row per 16-byte unit
  constexpr int TILE = IG_WAVE * SlabElem<T>::TPL;
  constexpr int VEC = 16 / sizeof(T);            // tokens of a 16-byte store
  constexpr int PAD = 8 / sizeof(T);
  static_assert(TILE % CHUNK == 0 && CHUNK % VEC == 0, "a chunk lies inside one tile");
  extern __shared__ uint2 slab_lds[];            // [CHUNK][d + PAD] elements, then the kept columns [r]
  T *rows = reinterpret_cast<T *>(slab_lds);
  const int ldr = d + PAD;
  int32_t *cols = reinterpret_cast<int32_t *>(rows + CHUNK * ldr);
  const int bh = blockIdx.y, h = bh % H;
  const int t0 = blockIdx.x * CHUNK;
  const int upr = d / TPL;   // 16-byte units per row (d is a multiple of TPL)
  const int units = max(0, min(CHUNK, N - t0)) * upr;        // units of valid tokens: one contiguous run
  const uint4 *src = reinterpret_cast<const uint4 *>(Kpool + ((long)bh * N_cap + t0) * d);
  for (int j = threadIdx.x; j < r; j += 256)
    cols[j] = min(max(idx[h * r + j], 0), d - 1);            // an index outside the head is clamped, never followed
  for (int u0 = 0; u0 < CHUNK * upr; u0 += 256 * U) {
    uint4 v[U];
#pragma unroll
    for (int i = 0; i < U; ++i) {
      const int u = u0 + 256 * i + (int)threadIdx.x;
      v[i] = make_uint4(0, 0, 0, 0);
      if (u < units) v[i] = src[u];
    }
#pragma unroll
    for (int i = 0; i < U; ++i) {
      const int u = u0 + 256 * i + (int)threadIdx.x;
      if (u < CHUNK * upr) {
        uint2 *at = reinterpret_cast<uint2 *>(rows + (u / upr) * ldr + (u % upr) * TPL);
        at[0] = make_uint2(v[i].x, v[i].y);
        at[1] = make_uint2(v[i].z, v[i].w);
      }
    }
  }
  __syncthreads();
  T *out = slab + ((long)bh * nTiles + t0 / TILE) * r * TILE + t0 % TILE;
  constexpr int GROUPS = CHUNK / VEC;            // lanes that cover the chunk's run of one channel
  for (int u = threadIdx.x; u < GROUPS * r; u += 256) {
    const int j = u / GROUPS, tt = (u % GROUPS) * VEC;
    const T *col = rows + tt * ldr + cols[j];
    typename Elem<T>::vec o;
#pragma unroll
    for (int e = 0; e < VEC; ++e) o[e] = col[e * ldr];
    *reinterpret_cast<typename Elem<T>::vec *>(out + (long)j * TILE + tt) = o;
  }
}

// ---- append of the token just decoded (Section 2.1: the new key and value join the cache; Section
// 4.4: the matching partial key cache entry is updated with it) -------------------------------------
// One workgroup per (b,h): the K and V rows go to slot `slot` of the pools (16-byte units, device
// or mapped pinned host memory), the r kept channels of the key to the slab's channel planes.
template <typename T>
__global__ __launch_bounds__(64) void append_token(const T *__restrict__ k_new, const T *__restrict__ v_new,
                                                   const int32_t *__restrict__ idx, T *__restrict__ slab,
                                                   u128 *__restrict__ Kpool, u128 *__restrict__ Vpool,
                                                   int H, int d, int r, int N_cap, int nTiles, int slot_all,
                                                   const int32_t *__restrict__ slots,
                                                   int32_t *__restrict__ counters, int32_t restart) {
  constexpr int TPL = Elem<T>::TPL;
  constexpr int TILE = IG_WAVE * SlabElem<T>::TPL;
  const int bh = blockIdx.x, h = bh % H;
  // one slot for every pool (append) or the pool's own victim slot (replacement); a slot outside
  // the pool is ignored
  const int slot = slots ? slots[bh] : slot_all;
  if (slot < 0 || slot >= N_cap) return;
  if (counters && threadIdx.x == 0) counters[(long)bh * N_cap + slot] = restart;   // policy state of the new entry
  const int U = d / TPL;
  const u128 *kn = reinterpret_cast<const u128 *>(k_new + (long)bh * d);
  const u128 *vn = reinterpret_cast<const u128 *>(v_new + (long)bh * d);
  for (int c = threadIdx.x; c < U; c += 64) {
    Kpool[((long)bh * N_cap + slot) * U + c] = kn[c];
    Vpool[((long)bh * N_cap + slot) * U + c] = vn[c];
  }
  const int tile = slot / TILE, tin = slot % TILE;
  for (int j = threadIdx.x; j < r; j += 64)
    slab[((long)bh * nTiles + tile) * r * TILE + (long)j * TILE + tin] =
        k_new[(long)bh * d + min(max(idx[h * r + j], 0), d - 1)];
}

// ---- pool counters (Section 4.4, counter-based victim selection) ------------------------------------
// One workgroup per (b,h) pool.  touch: +1 (saturating) on the counter of every prefetched slot; a
// list holds a slot once, so plain stores suffice; if a counter reached the saturation value, all
// counters of the pool are halved after the increments.  victim: the slot with the smallest count
// among the N valid ones, the lowest slot on ties (minimum over count * 2^32 + slot).
//
// Bound by the chain of trips through memory, so what can be asked for early is: a thread's first TOUCH_BATCH list
// entries while the count is on its way (entries past it are not used), all counters of a batch together.
// 256 pools of 2048 slots, lists of 100 on average: 3.8 -> 3.3 us, of which an empty launch is 2.
constexpr int TOUCH_BATCH = 4;
__global__ __launch_bounds__(256) void pool_touch(const int32_t *__restrict__ sel_idx,
                                                  const int32_t *__restrict__ sel_cnt,
                                                  int32_t *__restrict__ counters, int stride, int N,
                                                  int N_cap, int counter_max) {
  const int bh = blockIdx.x;
  int32_t *c = counters + (long)bh * N_cap;
  const int32_t *list = sel_idx + (long)bh * stride;
  int t[TOUCH_BATCH];
  auto load_entries = [&](int j0) {
#pragma unroll
    for (int i = 0; i < TOUCH_BATCH; ++i) t[i] = list[min(j0 + 256 * i, stride - 1)];
  };
  load_entries(threadIdx.x);
  const int n = min(sel_cnt[bh], stride);
  int sat = 0;
  for (int j0 = threadIdx.x; j0 < n;) {
    int v[TOUCH_BATCH];
    bool ok[TOUCH_BATCH];
#pragma unroll
    for (int i = 0; i < TOUCH_BATCH; ++i) {
      ok[i] = j0 + 256 * i < n && t[i] >= 0 && t[i] < N;
      t[i] = ok[i] ? t[i] : 0;
      v[i] = c[t[i]];
    }
#pragma unroll
    for (int i = 0; i < TOUCH_BATCH; ++i)
      if (ok[i]) {
        const int u = min(v[i] + 1, counter_max);
        c[t[i]] = u;
        sat |= u >= counter_max;
      }
    if ((j0 += 256 * TOUCH_BATCH) < n) load_entries(j0);
  }
  if (__syncthreads_or(sat))
    for (int t = threadIdx.x; t < N; t += 256) c[t] >>= 1;
}

// LRU comparison policy (Section 4.4, Table 2): the last-use stamp of every prefetched slot becomes
// `now`; the victim kernel below then names the slot whose last use lies furthest back.
__global__ __launch_bounds__(256) void pool_touch_lru(const int32_t *__restrict__ sel_idx,
                                                      const int32_t *__restrict__ sel_cnt,
                                                      int32_t *__restrict__ stamps, int stride, int N,
                                                      int N_cap, int32_t now) {
  const int bh = blockIdx.x;
  const int n = min(sel_cnt[bh], stride);
  for (int j = threadIdx.x; j < n; j += 256) {
    const int t = sel_idx[(long)bh * stride + j];
    if (t >= 0 && t < N) stamps[(long)bh * N_cap + t] = now;
  }
}

// W: counters a load takes, 4 where every pool's counters lie on 16 bytes.  A batch of VICTIM_BATCH loads a thread is in
// flight together (2048 slots: one trip instead of one after another for every 256).
// 256 pools of 2048 slots 3.3 -> 2.8 us.
constexpr int VICTIM_BATCH = 4;
template <int W>
__global__ __launch_bounds__(256) void pool_victim(const int32_t *__restrict__ counters,
                                                   int32_t *__restrict__ victim, int N, int N_cap) {
  typedef int32_t vec __attribute__((ext_vector_type(W)));
  __shared__ unsigned long long best[4];
  const int bh = blockIdx.x, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const vec *c = reinterpret_cast<const vec *>(counters + (long)bh * N_cap);
  const int units = (N + W - 1) / W;                 // (W == 4: N_cap is a multiple, the last unit lies inside it)
  unsigned long long m = ~0ull;
  for (int u0 = threadIdx.x; u0 < units; u0 += 256 * VICTIM_BATCH) {
    vec v[VICTIM_BATCH];
#pragma unroll
    for (int i = 0; i < VICTIM_BATCH; ++i) v[i] = c[min(u0 + 256 * i, units - 1)];
#pragma unroll
    for (int i = 0; i < VICTIM_BATCH; ++i) {
      const int t0 = min(u0 + 256 * i, units - 1) * W;
#pragma unroll
      for (int e = 0; e < W; ++e) {
        const unsigned long long key = ((unsigned long long)(unsigned)v[i][e] << 32) | (unsigned)(t0 + e);
        m = t0 + e < N && key < m ? key : m;
      }
    }
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const unsigned long long u = __shfl_xor(m, o, 64);
    m = u < m ? u : m;
  }
  if (lane == 0) best[w] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < 4; ++k) m = best[k] < m ? best[k] : m;
    victim[bh] = (int32_t)(m & 0xFFFFFFFFull);
  }
}

// ---- gather, device-resident pool ---------------------------------------------------------------
// Row copies in 16-byte units, U units per row; grid B*H x slices (see work_item).  A thread's copies are
// issued in batches of GATHER_BATCH, so that index loads, then K and V row loads, are in flight
// together.
constexpr int GATHER_BATCH = 8;
__global__ __launch_bounds__(256) void gather_rows_sliced(
    const u128 *__restrict__ Kpool, const u128 *__restrict__ Vpool, const int32_t *__restrict__ sel_idx,
    const int32_t *__restrict__ sel_cnt, u128 *__restrict__ K_sel, u128 *__restrict__ V_sel, int N_cap,
    int stride, int slice_log2, FastDiv by_U, int H, int BH, FastDiv by_H, FastDiv by_BH) {
  const int U = by_U.d;
  int bh, slice;
  work_item(blockIdx.x, H, BH, by_H, by_BH, &bh, &slice);
  const int cnt = min(sel_cnt[bh], stride);
  int row0, row1, slices;
  if (!slice_range(cnt, slice, slice_log2, SLICE_MAX_LOG2, &row0, &row1, &slices) || row1 <= row0) return;
  const int32_t *list = sel_idx + (long)bh * stride + row0;
  const long src0 = (long)bh * N_cap * U, dst0 = ((long)bh * stride + row0) * U;
  const int total = (row1 - row0) * U;
  // Branch-free batches (so that all loads of a batch are issued before the first store): a unit
  // past the end is clamped to the last unit, which is then copied more than once with identical
  // bytes.
  for (int u0 = threadIdx.x; u0 < total; u0 += 256 * GATHER_BATCH) {
    u128 kv[GATHER_BATCH], vv[GATHER_BATCH];
    long src[GATHER_BATCH];
#pragma unroll
    for (int i = 0; i < GATHER_BATCH; ++i) {
      const int u = min(u0 + 256 * i, total - 1);
      const int rr = by_U.div(u), c = u - rr * U;
      src[i] = src0 + (long)min(max(list[rr], 0), N_cap - 1) * U + c;   // a slot outside the pool is clamped
    }
#pragma unroll
    for (int i = 0; i < GATHER_BATCH; ++i) {
      kv[i] = Kpool[src[i]];
      vv[i] = Vpool[src[i]];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < GATHER_BATCH; ++i) {
      const int u = min(u0 + 256 * i, total - 1);
      store_stream(K_sel + dst0 + u, kv[i]);
      store_stream(V_sel + dst0 + u, vv[i]);
    }
  }
}

// ---- gather, pinned-host pool (body in attn_device.h) --------------------------------------------
__global__ __launch_bounds__(256) void gather_rows_flat(GatherArgs A) {
  extern __shared__ int pre[];
  gather_flat_body(A, blockIdx.x, gridDim.x, pre);
}

// ---- attention (body in attn_device.h) ----------------------------------------------------------
template <typename T, bool INDEXED, int LG, bool LONG>
__global__ __launch_bounds__(256) void sparse_attention(AttnArgs A) {
  sparse_attention_body<T, INDEXED, LG, LONG>(A, blockIdx.x);
}

__global__ __launch_bounds__(256) void copy_bytes(const u128 *__restrict__ src, u128 *__restrict__ dst,
                                                  long n16) {
  long i = (long)blockIdx.x * 256 + threadIdx.x;
  const long step = (long)gridDim.x * 256;
  for (; i < n16; i += step) dst[i] = src[i];
}

// Plain streaming read: a wave reads 8 consecutive KiB (16 bytes per lane and load) and folds them;
// the result is stored only if it equals a value it practically never takes, so the loads stay.
__global__ __launch_bounds__(256) void read_bytes(const u128 *__restrict__ src, long n16,
                                                  unsigned *__restrict__ sink) {
  const long wave = ((long)blockIdx.x * 256 + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  const long base = wave * 512 + lane;
  u128 v[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = src[min(base + 64L * i, n16 - 1)];
  unsigned x = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) x ^= v[i].x ^ v[i].y ^ v[i].z ^ v[i].w;
  if (x == 0x9e3779b9u) sink[0] = x;
}

}  // namespace

int ig_launch_read(ig_ctx *ctx, const void *src, size_t bytes, hipStream_t s) {
  const long n16 = (long)(bytes / 16);
  const long waves = (n16 + 511) / 512;
  auto k = read_bytes;
  IG_LAUNCH(ctx, IG_K_READ, k, dim3((unsigned)((waves + 3) / 4)), dim3(256), s, (const u128 *)src, n16,
            (unsigned *)(ctx->status + 8));
  return IG_OK;
}

int ig_launch_slab_build(ig_ctx *ctx, const ig_desc *d, const void *Kpool, const int32_t *idx,
                         void *slab, bool host_pool, hipStream_t s) {
  const int tile = ig_tile_tokens(d->dtype);
  const int nTiles = (d->N_cap + tile - 1) / tile;
  if (d->d > 256) return ig_fail(ctx, IG_ESHAPE, "slab build: d = %d exceeds 256", d->d);
  // Chunk of tokens by row length, so that it stays at about 32 KiB, 8 loads a thread.  From a pinned pool 32 tokens,
  // one load a thread at a time: requests over the link beyond what its latency covers only slow it down (8 pairs
  // of 1500 tokens, 128 float32 columns, 6.1 MB: 116 us, with 32 KiB in flight a workgroup 144 us).
  const int esz = ig_elem_bytes(d->dtype), row = d->d * esz;
  // Calls with less than a workgroup for every compute unit, which last as long as one workgroup, also take fewer
  // tokens in each, and one load where that is all there is (2 pairs of 492 tokens, 64 half columns: 2.6 us with 128
  // tokens, 2.0 so).
  int chunk = host_pool ? 32 : (row <= 256 ? 128 : (row <= 512 ? 64 : 32));
  while (chunk > 32 && (long)d->B * d->H * nTiles * (tile / chunk) < 256) chunk /= 2;
  const bool one_load = chunk == 32 && row <= 128;
  const size_t lds = (size_t)chunk * (row + 8) + (size_t)d->r * sizeof(int32_t);
  dim3 grid(nTiles * tile / chunk, d->B * d->H), block(256);
#define SLAB(T, CHUNK, U)                                                                          \
  {                                                                                                \
    auto k = slab_build<T, CHUNK, U>;                                                              \
    IG_LAUNCH_LDS(ctx, IG_K_BUILD, k, grid, block, lds, s, (const T *)Kpool, idx, (T *)slab,       \
                  (int)d->H, (int)d->d, (int)d->r, (int)d->N, (int)d->N_cap, nTiles);              \
    return IG_OK;                                                                                  \
  }
  if (d->dtype == IG_F16) {
    if (host_pool || one_load) SLAB(half_t, 32, 1)
    if (chunk == 128) SLAB(half_t, 128, 8)
    if (chunk == 64) SLAB(half_t, 64, 8)
    if (chunk == 32) SLAB(half_t, 32, 8)
  } else {
    if (host_pool || one_load) SLAB(float, 32, 1)
    if (chunk == 128) SLAB(float, 128, 8)
    if (chunk == 64) SLAB(float, 64, 8)
    if (chunk == 32) SLAB(float, 32, 8)
  }
#undef SLAB
  return ig_fail(ctx, IG_ESHAPE, "slab build: rows of %d bytes", row);
}

int ig_launch_append(ig_ctx *ctx, const ig_desc *d, const void *k_new, const void *v_new,
                     const int32_t *idx, void *slab, void *Kpool, void *Vpool,
                     const int32_t *slots, int32_t *counters, int32_t restart, hipStream_t s) {
  const int tile = ig_tile_tokens(d->dtype);
  const int nTiles = (d->N_cap + tile - 1) / tile;
  dim3 grid(d->B * d->H), block(64);
  if (d->dtype == IG_F16) {
    auto k = append_token<half_t>;
    IG_LAUNCH(ctx, IG_K_BUILD, k, grid, block, s, (const half_t *)k_new, (const half_t *)v_new, idx,
              (half_t *)slab, (u128 *)Kpool, (u128 *)Vpool, (int)d->H, (int)d->d, (int)d->r,
              (int)d->N_cap, nTiles, (int)d->N, slots, counters, restart);
  } else {
    auto k = append_token<float>;
    IG_LAUNCH(ctx, IG_K_BUILD, k, grid, block, s, (const float *)k_new, (const float *)v_new, idx,
              (float *)slab, (u128 *)Kpool, (u128 *)Vpool, (int)d->H, (int)d->d, (int)d->r,
              (int)d->N_cap, nTiles, (int)d->N, slots, counters, restart);
  }
  return IG_OK;
}

int ig_launch_pool_touch(ig_ctx *ctx, const ig_desc *d, const int32_t *sel_idx, int32_t sel_stride,
                         const int32_t *sel_cnt, int32_t *counters, int counter_max, hipStream_t s) {
  auto k = pool_touch;
  IG_LAUNCH(ctx, IG_K_BUILD, k, dim3(d->B * d->H), dim3(256), s, sel_idx, sel_cnt, counters,
            (int)sel_stride, (int)d->N, (int)d->N_cap, counter_max);
  return IG_OK;
}

int ig_launch_pool_touch_lru(ig_ctx *ctx, const ig_desc *d, const int32_t *sel_idx, int32_t sel_stride,
                             const int32_t *sel_cnt, int32_t *stamps, int32_t now, hipStream_t s) {
  auto k = pool_touch_lru;
  IG_LAUNCH(ctx, IG_K_BUILD, k, dim3(d->B * d->H), dim3(256), s, sel_idx, sel_cnt, stamps,
            (int)sel_stride, (int)d->N, (int)d->N_cap, now);
  return IG_OK;
}

int ig_launch_pool_victim(ig_ctx *ctx, const ig_desc *d, const int32_t *counters, int32_t *victim,
                          hipStream_t s) {
  auto k = d->N_cap % 4 == 0 && (uintptr_t)counters % 16 == 0 ? pool_victim<4> : pool_victim<1>;
  IG_LAUNCH(ctx, IG_K_BUILD, k, dim3(d->B * d->H), dim3(256), s, counters, victim, (int)d->N,
            (int)d->N_cap);
  return IG_OK;
}

int ig_launch_gather(ig_ctx *ctx, const ig_desc *d, const void *Kpool, const void *Vpool,
                     const int32_t *sel_idx, int32_t sel_stride, const int32_t *sel_cnt,
                     void *K_sel, void *V_sel, int host_pool, hipStream_t s) {
  const int U = d->d * ig_elem_bytes(d->dtype) / 16;
  const int BH = d->B * d->H;
  if (!host_pool) {
    // rows of a slice: 1 << SLICE_LOG2, but no more than two batches of a workgroup's copies (see att_slice_log2)
    int slice_log2 = SLICE_LOG2;
    while (slice_log2 > 4 && ((long)U << slice_log2) > 2 * 256 * GATHER_BATCH) --slice_log2;
    dim3 grid(BH * slices_at_most(sel_stride, slice_log2, SLICE_MAX_LOG2)), block(256);
    auto k = gather_rows_sliced;
    IG_LAUNCH(ctx, IG_K_GATHER, k, grid, block, s, (const u128 *)Kpool, (const u128 *)Vpool, sel_idx,
              sel_cnt, (u128 *)K_sel, (u128 *)V_sel, (int)d->N_cap, (int)sel_stride, slice_log2, ig_fast_div(U),
              (int)d->H, BH, ig_fast_div(d->H), ig_fast_div(BH));
    return IG_OK;
  }
  GatherArgs A;
  int rc = ig_gather_args(ctx, d, Kpool, Vpool, sel_idx, sel_stride, sel_cnt, K_sel, V_sel, &A);
  if (rc) return rc;
  auto k = gather_rows_flat;
  IG_LAUNCH_LDS(ctx, IG_K_GATHER, k, dim3(GATHER_FLAT_BLOCKS), dim3(256), (unsigned)ig_gather_lds(d), s, A);
  return IG_OK;
}

bool ig_gather_fits(const ig_desc *d) { return ig_gather_lds(d) <= 60 * 1024; }
size_t ig_gather_lds(const ig_desc *d) { return ((size_t)d->B * d->H + 1) * sizeof(int); }

int ig_gather_args(ig_ctx *ctx, const ig_desc *d, const void *Kpool, const void *Vpool, const int32_t *sel_idx,
                   int32_t sel_stride, const int32_t *sel_cnt, void *K_sel, void *V_sel, GatherArgs *A) {
  if (!ig_gather_fits(d)) return ig_fail(ctx, IG_ESHAPE, "host gather: B*H = %d exceeds %d", d->B * d->H, 60 * 256 - 1);
  *A = GatherArgs{(const uint4 *)Kpool, (const uint4 *)Vpool, sel_idx, sel_cnt, (uint4 *)K_sel, (uint4 *)V_sel, nullptr,
                  (int)d->N_cap, (int)sel_stride, d->d * ig_elem_bytes(d->dtype) / 16, d->B * d->H,
                  ig_fast_div(d->d * ig_elem_bytes(d->dtype) / 16)};
  return IG_OK;
}

int ig_attn_fill(ig_ctx *ctx, const ig_desc *d, const void *q, const void *K, const void *V,
                 const int32_t *sel_idx, int32_t sel_stride, const int32_t *sel_cnt, int kv_rows,
                 const void *k_new, const void *v_new, void *out, void *K_out, void *V_out,
                 float *part, int32_t *counters, AttnArgs *A) {
  const int row_bytes = d->d * ig_elem_bytes(d->dtype);
  const int LPR = row_bytes / 16;
  if (row_bytes % 16 || LPR < 1 || LPR > 64 || (LPR & (LPR - 1)))
    return ig_fail(ctx, IG_ESHAPE, "attention: row of %d bytes must be 16 * 2^k bytes, at most 1024",
                   row_bytes);
  A->q = q;
  A->K = (const uint4 *)K;
  A->V = (const uint4 *)V;
  A->sel_idx = sel_idx;
  A->sel_cnt = sel_cnt;
  A->stride = sel_stride;
  A->kv_rows = kv_rows;
  A->lpr_log2 = __builtin_ctz(LPR);
  A->slice_log2 = att_slice_log2(A->lpr_log2, d->B * d->H);
  A->most_log2 = SLICE_MAX_LOG2;
  A->k_new = k_new;
  A->v_new = v_new;
  A->out = out;
  A->scale = d->scale;
  A->d = d->d;
  A->part = part;
  A->counters = counters;
  A->H = d->H;
  A->BH = d->B * d->H;
  A->by_H = ig_fast_div(d->H);
  A->by_BH = ig_fast_div(A->BH);
  A->K_out = sel_idx ? (uint4 *)K_out : nullptr;
  A->V_out = sel_idx ? (uint4 *)V_out : nullptr;
  return IG_OK;
}

int ig_attn_args(ig_ctx *ctx, const ig_desc *d, const void *q, const void *K, const void *V,
                 const int32_t *sel_idx, int32_t sel_stride, const int32_t *sel_cnt, int kv_rows,
                 const void *k_new, const void *v_new, void *out, void *K_out, void *V_out, AttnArgs *A) {
  const int BH = d->B * d->H;
  int rc = ig_ensure(ctx, (void **)&ctx->attn_part, &ctx->attn_part_bytes,
                     (size_t)BH * IG_SLICE_MAX_LONG * (d->d + 2) * sizeof(float));
  if (rc) return rc;
  if ((rc = ig_ensure_zeroed(ctx, (void **)&ctx->attn_cnt, &ctx->attn_cnt_bytes, (size_t)BH * sizeof(int32_t))))
    return rc;
  return ig_attn_fill(ctx, d, q, K, V, sel_idx, sel_stride, sel_cnt, kv_rows, k_new, v_new, out, K_out,
                      V_out, ctx->attn_part, ctx->attn_cnt, A);
}

// the attention kernel for a type and row length (see LG at sparse_attention_body)
template <bool INDEXED, bool LONG>
static void (*attention_kernel(int dtype, int lpr_log2))(AttnArgs) {
  if (dtype == IG_F16) {
    if (lpr_log2 == 3) return sparse_attention<half_t, INDEXED, 3, LONG>;
    if (lpr_log2 == 4) return sparse_attention<half_t, INDEXED, 4, LONG>;
    if (lpr_log2 == 5) return sparse_attention<half_t, INDEXED, 5, LONG>;
    return sparse_attention<half_t, INDEXED, -1, LONG>;
  }
  if (lpr_log2 == 4) return sparse_attention<float, INDEXED, 4, LONG>;
  if (lpr_log2 == 5) return sparse_attention<float, INDEXED, 5, LONG>;
  return sparse_attention<float, INDEXED, -1, LONG>;
}

int ig_launch_attention(ig_ctx *ctx, const ig_desc *d, const void *q, const void *K, const void *V,
                        const int32_t *sel_idx, int32_t sel_stride, const int32_t *sel_cnt,
                        int kv_rows_per_bh, const void *k_new, const void *v_new, void *out,
                        void *K_out, void *V_out, hipStream_t s) {
  AttnArgs A;
  int rc = ig_attn_args(ctx, d, q, K, V, sel_idx, sel_stride, sel_cnt, kv_rows_per_bh, k_new, v_new, out,
                        K_out, V_out, &A);
  if (rc) return rc;
  if (sel_idx) A.most_log2 = att_most_log2(A.slice_log2, A.BH, sel_stride < d->N ? sel_stride : d->N);
  dim3 grid(A.BH * slices_at_most((long)sel_stride + 1, A.slice_log2, A.most_log2)), block(256);
  const auto k = !sel_idx ? attention_kernel<false, false>(d->dtype, A.lpr_log2)
                          : (A.most_log2 == SLICE_MAX_LOG2 ? attention_kernel<true, false>(d->dtype, A.lpr_log2)
                                                           : attention_kernel<true, true>(d->dtype, A.lpr_log2));
  IG_LAUNCH(ctx, IG_K_ATTENTION, k, grid, block, s, A);
  return IG_OK;
}

// ---- attention without any allocation -----------------------------------------------------------
// For callers that cannot allocate (stream capture, serving loops, harnesses that forbid it): the
// per-slice softmax states and the per-(b,h) arrival counters of the attention kernel live in a
// file-scope device array instead of context workspaces.  Every GPU the library runs on holds its
// own copy of the array, at its own address, until the process ends; the address is looked up
// once per context (ig_create, with the context's device current) and host code only ever uses
// that address, never the array's name.  Layout: counters int32 [B*H] (padded to 256 bytes), then
// states float [B*H][IG_SLICE_MAX][d+2].
constexpr size_t STATIC_SCRATCH_BYTES = (size_t)16 << 20;
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];

namespace {
__global__ __launch_bounds__(256) void zero_words(int32_t *p, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0;
}
}  // namespace

int ig_static_scratch_bind(ig_ctx *ctx) {
  void *ptr = nullptr;
  hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  if (e != hipSuccess || !ptr) {
    ctx->static_scratch = nullptr;
    ctx->static_scratch_bytes = 0;
    return ig_hip_fail(ctx, e, "hipGetSymbolAddress(scratch)");
  }
  ctx->static_scratch = ptr;
  ctx->static_scratch_bytes = STATIC_SCRATCH_BYTES;
  return IG_OK;
}

int ig_launch_attention_static(ig_ctx *ctx, const ig_desc *d, const void *q, const void *K, const void *V,
                               int32_t sel_stride, const int32_t *sel_cnt, const void *k_new,
                               const void *v_new, void *out, hipStream_t s) {
  if (!ctx->static_scratch) return ig_fail(ctx, IG_EHIP, "the static scratch array was not bound on this device");
  const size_t BH = (size_t)d->B * d->H;
  const size_t cnt_bytes = (BH * sizeof(int32_t) + 255) / 256 * 256;
  const size_t need = cnt_bytes + BH * IG_SLICE_MAX * ((size_t)d->d + 2) * sizeof(float);
  if (need > ctx->static_scratch_bytes)
    return ig_fail(ctx, IG_ECAPACITY,
                   "ig_sparse_attention_static: B*H = %zu heads of d = %d need %zu bytes of slice states, "
                   "the static scratch array holds %zu", BH, d->d, need, ctx->static_scratch_bytes);
  int32_t *counters = reinterpret_cast<int32_t *>(ctx->static_scratch);
  float *part = reinterpret_cast<float *>(static_cast<unsigned char *>(ctx->static_scratch) + cnt_bytes);
  AttnArgs A;
  int rc = ig_attn_fill(ctx, d, q, K, V, nullptr, sel_stride, sel_cnt, sel_stride, k_new, v_new, out,
                        nullptr, nullptr, part, counters, &A);
  if (rc) return rc;
  // The array keeps whatever the last call left (a call that was cut short leaves counters
  // behind): the arrival counters start from zero on every call.  A fill kernel, not a memset, so
  // that the sequence can be captured into a graph.
  hipLaunchKernelGGL(zero_words, dim3((unsigned)((BH + 255) / 256)), dim3(256), 0, s, counters, (int)BH);
  dim3 grid((unsigned)(BH * slices_at_most((long)sel_stride + 1, A.slice_log2, A.most_log2))), block(256);
  hipLaunchKernelGGL((attention_kernel<false, false>(d->dtype, A.lpr_log2)), grid, block, 0, s, A);
  hipError_t le = hipGetLastError();
  if (le != hipSuccess) return ig_hip_fail(ctx, le, "sparse_attention (static scratch)");
  return IG_OK;
}

int ig_launch_copy(ig_ctx *ctx, const void *src, void *dst, size_t bytes, hipStream_t s) {
  long n16 = (long)(bytes / 16);
  long blocks = (n16 + 255) / 256;
  if (blocks > 16384) blocks = 16384;
  if (blocks < 1) blocks = 1;
  auto k = copy_bytes;
  IG_LAUNCH(ctx, IG_K_COPY, k, dim3((unsigned)blocks), dim3(256), s, (const u128 *)src, (u128 *)dst,
            n16);
  return IG_OK;
}
