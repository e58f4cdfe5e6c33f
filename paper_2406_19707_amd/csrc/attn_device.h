// Device side of the gather / attention kernels: 16-byte row units, the (b, h, slice) work-item
// mapping, and the body of the sparse attention kernel.  Shared by the attention kernels and by the
// kernel that runs a layer's attention next to the next layer's scan in one launch.
#ifndef IG_ATTN_DEVICE_H
#define IG_ATTN_DEVICE_H
#include <type_traits>
#include "ig_internal.h"

struct AttnArgs {
  const void *q;              // [B,H,d]
  const uint4 *K, *V;          // gathered rows [B*H, stride, d] or the pool [B*H, kv_rows, d] (INDEXED)
  const int32_t *sel_idx, *sel_cnt;
  int stride, kv_rows;
  int lpr_log2;               // a row is 1 << lpr_log2 pieces of 16 bytes
  int slice_log2;             // rows of a slice: see slice_range
  int most_log2;              // slices of a list at most, 1 << most_log2
  const void *k_new, *v_new;  // optional always-attended row
  void *out;
  float scale;
  int d;
  float *part;                // per-slice softmax states [B*H][1 << most_log2][d+2]
  int32_t *counters;          // per-(b,h) arrival counters, zero between calls
  int H, BH;
  FastDiv by_H, by_BH;
  uint4 *K_out, *V_out;        // INDEXED only: the rows read are also stored here (fused prefetch)
};

struct GatherArgs {
  const uint4 *Kpool, *Vpool;
  const int32_t *sel_idx, *sel_cnt;
  uint4 *K_sel, *V_sel;
  int32_t *cnt_copy;           // optional: the counts as they were, for a reader that runs beside their next writer
  int N_cap, stride, U, BH;    // U: 16-byte units of a row
  FastDiv by_U;
};

namespace {

typedef uint4 u128;

// Store for gathered rows.  Marked non-temporal: written with plain stores, the rows stay dirty in
// the last-level cache and their write-back lands in the next kernels (measured: the following
// partial key cache scan slows from 29 to 35 us on a 159 MB slab); streamed out, it does not.
__device__ __forceinline__ void store_stream(u128 *p, const u128 &v) {
  typedef unsigned int v4u __attribute__((ext_vector_type(4)));
  const v4u t = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(t, reinterpret_cast<v4u *>(p));
}

// ---- work split shared by gather and attention --------------------------------------------------
// Selected-token lists are very uneven (a few heads keep a thousand rows, most a few dozen), and
// one compute unit moves well under 100 GB/s, so a list is cut into slices of 1 << slice_log2 rows, or,
// when that would be more than 1 << most_log2 of them, into that many equal ones.  Every workgroup derives
// this from the device-side count, so the host never reads the counts; surplus workgroups leave at
// once.  They are most of a grid, so the way to the exit has no division in it: with the work item
// decoded by run-time divisions and slices of rows*s/slices, 320 lists of 250 rows on average took 28.6 us
// to copy instead of 26.5.
//
// Workgroups are handed to the 8 XCDs round-robin by linear id, and an XCD reaches only about an
// eighth of the HBM bandwidth, so the work has to be even per XCD, not just per compute unit:
// heavy lists cluster by head (and H is normally a multiple of 8), so mapping (b,h) -> id = b*H+h
// would send every slice of the heavy heads to the same XCD.  work_item() therefore decodes the
// linear id as slice = id / BH, t = id % BH, b = t / H, h = (t % H - b - 5*slice) mod H, which puts
// (b, h, slice) on XCD (h + b + 5*slice) % 8: the slices of one list, the sequences of one head and
// the heads of one sequence are each spread over all XCDs.
constexpr int SLICE_LOG2 = 7;
constexpr int SLICE_MAX_LOG2 = 4, SLICE_MAX_LONG_LOG2 = 5;
static_assert(IG_SLICE_MAX == 1 << SLICE_MAX_LOG2 && IG_SLICE_MAX_LONG == 1 << SLICE_MAX_LONG_LOG2, "");
__device__ __forceinline__ void work_item(int id, int H, int BH, const FastDiv &by_H, const FastDiv &by_BH, int *bh, int *slice) {
  const int s = by_BH.div(id), t = id - s * BH;
  const int b = by_H.div(t);
  int h = t - b * H - by_H.mod(b + 5 * s);
  if (h < 0) h += H;
  *bh = b * H + h;
  *slice = s;
}
__device__ __forceinline__ bool slice_range(int rows, int s, int slice_log2, int most_log2, int *row0, int *row1, int *slices) {
  const int most = 1 << most_log2;
  if (rows <= (most << slice_log2)) {
    const int n = max(1, (rows + (1 << slice_log2) - 1) >> slice_log2);
    *slices = n;
    *row0 = s << slice_log2;
    *row1 = min(rows, *row0 + (1 << slice_log2));
    return s < n;
  }
  const int per = (rows + most - 1) >> most_log2;
  *slices = most;
  *row0 = min(rows, s * per);
  *row1 = min(rows, *row0 + per);
  return true;
}
// workgroups per list that a list of at most `rows` rows can need
static inline int slices_at_most(long rows, int slice_log2, int most_log2) {
  const long n = (rows + (1l << slice_log2) - 1) >> slice_log2;
  return n < 1 ? 1 : (n < (1l << most_log2) ? (int)n : 1 << most_log2);
}

// ---- attention ----------------------------------------------------------------------------------
// grid B*H x slices_at_most() (see work_item), 4 waves per workgroup, one slice of the (b,h) list each.  A row of d
// elements is covered by LPR = d*sizeof(T)/16 lanes, 16 bytes each, so a wave step covers 64/LPR
// rows; waves interleave over the rows, and steps are issued in batches of ATT_BATCH so that a
// batch's K and V loads are all in flight before the first is used.  Every lane group keeps an
// online-softmax state (running max, normaliser, weighted sum for its 16-byte slice of V); states
// are merged across lane groups with shuffles and across waves through LDS, in a fixed order.
//
// A list with one slice writes its output directly.  With several slices each workgroup publishes
// its state (max, normaliser, d sums) with device-coherent stores and bumps a per-(b,h) counter;
// the workgroup that arrives last reads all states with device-coherent loads and merges them in
// slice order, so the result does not depend on arrival order.  Coherent stores and loads are used
// instead of a device-wide fence, which would write back and invalidate the whole L2 per
// workgroup (see the note at the counter bump below).  The counter is left at zero for the next
// call.
constexpr int ATT_BATCH = 8;
// rows of a slice: what one batch of a workgroup's loads covers, or 1 << SLICE_LOG2 where that is more, but no
// more than two batches where lists are few.  (Rows of 128 bytes, d = 64 in half precision: 256 a batch; a list of
// 129..256 such rows is then one workgroup that writes its output itself instead of two that meet: 192 lists of
// 120 rows on average 8.2 -> 5.8 us.  Rows of 1024 bytes: 32 a batch; the first of two slices is full whatever is
// left for the second, and one workgroup walking 128 rows sets the time of a list of 137: 32 such lists 18.5 ->
// 11.6 us.  With 256 lists and more every compute unit has one, and cutting lists of 100 rows in two only adds the
// meeting: 512 of them 23.8 -> 25.8 us.)
static inline int att_slice_log2(int lpr_log2, int lists) {
  const int batch_log2 = 2 + (6 - lpr_log2) + 3;     // 4 waves x 64 / LPR rows x ATT_BATCH steps
  if (batch_log2 >= SLICE_LOG2) return batch_log2;
  return batch_log2 + 1 < SLICE_LOG2 && lists < 256 ? batch_log2 + 1 : SLICE_LOG2;
}
static_assert(ATT_BATCH == 8, "att_slice_log2 counts on it");
// Slices of a list at most, as a power of two: 16, or 32 where lists can be longer than 16 slices and their rows come
// out of the pool through the list: the longest lists set the time, and a slice of more than one batch of loads is a
// second round of trips.  Whole steps with 16 and with 32, lists of rows of 256 bytes: 512 rotary lists of 4096 tokens
// 79.7 -> 77.4 us, 320 of 2500 50.0 -> 48.8, 256 of 8192 51.1 -> 49.4, 80 of 16384 92.4 -> 78.5, 128 of 9000 55.0 -> 50.7;
// 384 of 6000, rows of 128 bytes, 43.0 -> 41.4.  With fewer than 256 lists only where they can be four times as long as
// that: the larger grid costs 32 lists of 8192 tokens 0.5 us (17.3 -> 17.8), and they rarely hold one so long.
// The joint launches keep 16, whose larger grid costs each of them 1 us, and so does the attention over rows that
// have been fetched: it runs beside the prefetch of a host-pool step, which more workgroups hold up.
static inline int att_most_log2(int slice_log2, int lists, long longest) {
  const long rows = (long)IG_SLICE_MAX << slice_log2;
  return longest > (lists >= 256 ? rows : 4 * rows) ? SLICE_MAX_LONG_LOG2 : SLICE_MAX_LOG2;
}

template <typename T> __device__ __forceinline__ void to_float(const u128 &raw, float (&f)[Elem<T>::TPL]);
template <> __device__ __forceinline__ void to_float<half_t>(const u128 &raw, float (&f)[8]) {
  const half8 h = *reinterpret_cast<const half8 *>(&raw);
#pragma unroll
  for (int e = 0; e < 8; ++e) f[e] = (float)h[e];
}
template <> __device__ __forceinline__ void to_float<float>(const u128 &raw, float (&f)[4]) {
  const floatx4 v = *reinterpret_cast<const floatx4 *>(&raw);
#pragma unroll
  for (int e = 0; e < 4; ++e) f[e] = v[e];
}

__device__ __forceinline__ float exp_or_zero(float m, float M) { return (m == -INFINITY) ? 0.f : __expf(m - M); }
__device__ __forceinline__ void coherent_store(float *p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float coherent_load(const float *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}


// `id` is the linear work item (see work_item); the kernel passes blockIdx.x
// LG: log2 of the 16-byte pieces in a row where that is known at build time (the row lengths of 64, 128 and
// 256 half or 64 and 128 float32 columns), -1 otherwise.  With it a batch is straight-line code: the
// eight rows' reductions interleave instead of eight times asking which form to take (with the query not
// waited for before the rows are asked for: 1120 lists of 77 rows of 128 half columns 30.1 -> 24.3 us,
// 512 lists of 229 rows, 120 MB read and written, 33.3 -> 31.6 us, 192 lists of 120 rows of 64 columns
// 9.5 -> 5.3 us).
// LONG: lists are cut into 32 slices at most instead of 16 (att_most_log2).  A form of its own: with the limit and
// the merge's second pass decided at run time every attention of lists in several slices lost 0.3 us.
template <typename T, bool INDEXED, int LG, bool LONG = false>
__device__ __forceinline__ void sparse_attention_body(const AttnArgs &A, const int id) {
  const T *__restrict__ q = static_cast<const T *>(A.q);
  const u128 *__restrict__ K = A.K;
  const u128 *__restrict__ V = A.V;
  const int32_t *__restrict__ sel_idx = A.sel_idx;
  const int32_t *__restrict__ sel_cnt = A.sel_cnt;
  const int lpr_log2 = LG >= 0 ? LG : A.lpr_log2;
  const int stride = A.stride, kv_rows = A.kv_rows, LPR = 1 << lpr_log2, d = A.d;
  const T *__restrict__ k_new = static_cast<const T *>(A.k_new);
  const T *__restrict__ v_new = static_cast<const T *>(A.v_new);
  T *__restrict__ out = static_cast<T *>(A.out);
  const float scale = A.scale;
  float *part = A.part;
  int32_t *counters = A.counters;
  u128 *__restrict__ K_out = A.K_out;
  u128 *__restrict__ V_out = A.V_out;
  constexpr int TPL = Elem<T>::TPL;
  __shared__ float sm[4], sz[4];
  __shared__ float sacc[4][512];
  __shared__ int s_last;
  constexpr int most_log2 = LONG ? SLICE_MAX_LONG_LOG2 : SLICE_MAX_LOG2;
  int bh, slice;
  work_item(id, A.H, A.BH, A.by_H, A.by_BH, &bh, &slice);
  const int n = min(sel_cnt[bh], stride);
  const int rows = n + (k_new ? 1 : 0);
  int row0 = 0, row1 = 0, slices = 1;
  if (!slice_range(rows, slice, A.slice_log2, most_log2, &row0, &row1, &slices)) return;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int RPW = 64 >> lpr_log2;      // rows per wave step
  const int sub = lane >> lpr_log2, li = lane & (LPR - 1);
  // (not looked at before the first batch's loads are out)
  const u128 qraw = *reinterpret_cast<const u128 *>(q + (long)bh * d + li * TPL);
  float m = -INFINITY, z = 0.f, acc[TPL];
#pragma unroll
  for (int e = 0; e < TPL; ++e) acc[e] = 0.f;
  const long base = (long)bh * kv_rows * LPR;
  const int32_t *list = sel_idx + (long)bh * stride;
  const int rows_per_batch = 4 * RPW * ATT_BATCH;
  // Fused prefetch (K_out): the rows read from the pool are also the rows ig_gather_kv would copy.
  // With several slices the row stores of a slice's last batch are held back until the slice has
  // published its softmax state, so that the wait for that publication does not also wait for
  // 64 KiB of row stores to be acknowledged; they then travel while the counter round trip and
  // the final merge are under way.
  const bool fuse_store = INDEXED && K_out != nullptr;
  const bool defer = fuse_store && slices > 1;
  u128 kr[ATT_BATCH], vr[ATT_BATCH];
  int r_keep = -1;                       // first row of the batch whose stores are held back
  auto store_rows = [&](int r0) {
#pragma unroll
    for (int i = 0; i < ATT_BATCH; ++i) {
      const int j = r0 + (i * 4 + w) * RPW + sub;
      if (j < row1 && j < n) {
        const long o = ((long)bh * stride + j) * LPR + li;
        store_stream(K_out + o, kr[i]);
        store_stream(V_out + o, vr[i]);
      }
    }
  };
  for (int r0 = row0; r0 < row1; r0 += rows_per_batch) {
    // Branch-free loads, so that the whole batch is in flight at once: a step past the slice's end
    // re-reads the slice's last row and its logit is masked below; the new-token row is a pointer
    // select, not a branch.
    bool valid[ATT_BATCH];
    long rowoff[ATT_BATCH];
#pragma unroll
    for (int i = 0; i < ATT_BATCH; ++i) {
      // step i of wave w covers rows r0 + (i*4 + w)*RPW + sub
      const int j = r0 + (i * 4 + w) * RPW + sub;
      valid[i] = j < row1;
      const int jc = min(j, row1 - 1);
      const int jl = min(jc, max(n - 1, 0));
      rowoff[i] = INDEXED ? (long)min(max(list[jl], 0), kv_rows - 1) : (long)jl;   // a slot outside the pool is clamped
    }
#pragma unroll
    for (int i = 0; i < ATT_BATCH; ++i) {
      const int j = r0 + (i * 4 + w) * RPW + sub;
      const bool cached = min(j, row1 - 1) < n;
      const u128 *kp = cached ? K + base + rowoff[i] * LPR + li : reinterpret_cast<const u128 *>(k_new + (long)bh * d) + li;
      const u128 *vp = cached ? V + base + rowoff[i] * LPR + li : reinterpret_cast<const u128 *>(v_new + (long)bh * d) + li;
      kr[i] = *kp;
      vr[i] = *vp;
    }
    if (fuse_store) {
      if (defer && r0 + rows_per_batch >= row1) r_keep = r0;
      else store_rows(r0);
    }
    __builtin_amdgcn_sched_barrier(0);
    u128 qnow = qraw;
    keep_loaded(qnow);
    float qf[TPL];
    to_float<T>(qnow, qf);
#pragma unroll
    for (int e = 0; e < TPL; ++e) qf[e] *= scale;
    float l[ATT_BATCH];
    float bm = m;
#pragma unroll
    for (int i = 0; i < ATT_BATCH; ++i) {
      float kf[TPL];
      to_float<T>(kr[i], kf);
      float t = 0.f;
#pragma unroll
      for (int e = 0; e < TPL; ++e) t = fmaf(qf[e], kf[e], t);
      if constexpr (LG == 3) {
        t = row8_sum(t);
      } else if constexpr (LG >= 4) {
        t = row16_sum(t);
        if constexpr (LG == 5) t += __shfl_xor(t, 16, 64);
      } else {
        for (int o = 1; o < LPR; o <<= 1) t += __shfl_xor(t, o, 64);
      }
      l[i] = valid[i] ? t : -INFINITY;
      bm = fmaxf(bm, l[i]);
    }
    if (bm != -INFINITY) {
      const float f = exp_or_zero(m, bm);
      z *= f;
#pragma unroll
      for (int e = 0; e < TPL; ++e) acc[e] *= f;
#pragma unroll
      for (int i = 0; i < ATT_BATCH; ++i) {
        const float p = exp_or_zero(l[i], bm);
        float vf[TPL];
        to_float<T>(vr[i], vf);
        z += p;
#pragma unroll
        for (int e = 0; e < TPL; ++e) acc[e] = fmaf(p, vf[e], acc[e]);
      }
      m = bm;
    }
  }
  // merge the lane groups of the wave (lanes with equal li hold the same slice of V)
  for (int o = LPR; o < 64; o <<= 1) {
    const float m2 = __shfl_xor(m, o, 64), z2 = __shfl_xor(z, o, 64);
    const float M = fmaxf(m, m2);
    const float f1 = exp_or_zero(m, M), f2 = exp_or_zero(m2, M);
    z = z * f1 + z2 * f2;
#pragma unroll
    for (int e = 0; e < TPL; ++e) acc[e] = acc[e] * f1 + __shfl_xor(acc[e], o, 64) * f2;
    m = M;
  }
  if (lane < LPR) {
    if (lane == 0) { sm[w] = m; sz[w] = z; }
#pragma unroll
    for (int e = 0; e < TPL; ++e) sacc[w][lane * TPL + e] = acc[e];
  }
  __syncthreads();
  // merge the four waves: thread c owns output channel c
  const float M = fmaxf(fmaxf(sm[0], sm[1]), fmaxf(sm[2], sm[3]));
  float zc = 0.f;
#pragma unroll
  for (int k = 0; k < 4; ++k) zc += sz[k] * exp_or_zero(sm[k], M);
  if (slices == 1) {
    for (int c = threadIdx.x; c < d; c += 256) {
      float a = 0.f;
#pragma unroll
      for (int k = 0; k < 4; ++k) a += sacc[k][c] * exp_or_zero(sm[k], M);
      out[(long)bh * d + c] = (T)(zc > 0.f ? a / zc : 0.f);
    }
    return;
  }
  // several slices: publish this slice's state; the last arrival merges all of them
  float *mine = part + (((long)bh << most_log2) + slice) * (d + 2);
  for (int c = threadIdx.x; c < d; c += 256) {
    float a = 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k) a += sacc[k][c] * exp_or_zero(sm[k], M);
    coherent_store(mine + 2 + c, a);
  }
  if (threadIdx.x == 0) {
    coherent_store(mine, M);
    coherent_store(mine + 1, zc);
  }
  // Order between the state stores and the arrival counter.  The states are agent-scope atomic
  // stores (written through to the device's coherence point); every wave waits until its own
  // have been acknowledged there (s_waitcnt vmcnt(0)), the barrier then puts all waves' stores
  // before thread 0's counter bump, an agent-scope atomic performed at the same coherence point,
  // and the last arrival reads the states with agent-scope atomic loads issued after its bump
  // has returned.  The bump itself is relaxed: making it a release-acquire operation adds a
  // write-back and an invalidation of the whole L2 per workgroup, which was measured to double
  // the kernel (20 -> 50 us on 512 lists of 4096 tokens).  What this leans on is therefore the
  // hardware's handling of acknowledged write-through stores, not the language memory model.
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  // held-back row stores: waves 1..3 issue theirs now; wave 0, which waits for the counter and does
  // the final merge, issues its own only when it has nothing left to wait for
  if (w != 0 && r_keep >= 0) store_rows(r_keep);
  if (threadIdx.x == 0) {
    const int prev = __hip_atomic_fetch_add(&counters[bh], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_last = (prev == slices - 1);
    if (s_last) __hip_atomic_store(&counters[bh], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (w != 0) return;
  if (s_last) {
    // wave 0 of the last arrival: lane c owns output channels c, c + 64, ...; all loads of a pass
    // (independent, slices past the last read it again) are issued before any is used
    const float *all = part + ((long)bh << most_log2) * (d + 2);
    const float *state = all + (long)min(lane, slices - 1) * (d + 2);
    constexpr int CPP = 2;               // channels per lane and pass
    constexpr int SPP = 16;              // slices per pass: of 32, the others follow, in the same registers
    for (int c0 = lane; c0 - lane < d; c0 += 64 * CPP) {   // (all lanes stay: they hold the weights)
      float mk = coherent_load(state), zk = coherent_load(state + 1), a[CPP], zz = 0.f;
      int wbits = 0;
      auto pass = [&](auto first) {
        constexpr int k0 = decltype(first)::value;
        float ak[CPP][SPP];
#pragma unroll
        for (int q = 0; q < CPP; ++q)
#pragma unroll
          for (int k = 0; k < SPP; ++k)
            ak[q][k] = coherent_load(all + (long)min(k0 + k, slices - 1) * (d + 2) + 2 + min(c0 + 64 * q, d - 1));
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (k0 == 0) {
          // (One lane a slice works out its weight, and the loop below reads them one by one.  With every slice's
          // maximum, normaliser and weight in every lane this merge set the kernel's registers, 144 instead of 117,
          // three waves a SIMD instead of four: 1120 lists of 77 rows 26.2 -> 23.4 us.)
          mk = lane < slices ? mk : -INFINITY;
          zk = lane < slices ? zk : 0.f;
          const float wk = exp_or_zero(mk, wave_max(mk));
          wbits = __float_as_int(wk);
          const int zs = __float_as_int(row16_sum(zk * wk));     // (lanes past the last slice hold zeros)
          zz = __int_as_float(__builtin_amdgcn_readlane(zs, 0));
          if constexpr (LONG) zz += __int_as_float(__builtin_amdgcn_readlane(zs, 16));
        }
#pragma unroll
        for (int q = 0; q < CPP; ++q) {
          float t = k0 == 0 ? 0.f : a[q];
#pragma unroll
          for (int k = 0; k < SPP; ++k)
            t = fmaf(k0 + k < slices ? ak[q][k] : 0.f, __int_as_float(__builtin_amdgcn_readlane(wbits, k0 + k)), t);
          a[q] = t;
        }
      };
      pass(std::integral_constant<int, 0>{});
      if constexpr (LONG)
        if (slices > SPP) pass(std::integral_constant<int, SPP>{});
#pragma unroll
      for (int q = 0; q < CPP; ++q) {
        const int c = c0 + 64 * q;
        if (c < d) out[(long)bh * d + c] = (T)(zz > 0.f ? a[q] / zz : 0.f);
      }
    }
  }
  if (r_keep >= 0) store_rows(r_keep);
}


// ---- gather, pinned-host pool --------------------------------------------------------------------
// The rows of all lists are treated as one flat sequence and cut into equal ranges, one per
// workgroup: every workgroup reads the B*H counts (one coalesced read), builds their prefix sum in
// LDS, takes rows [T*g/G, T*(g+1)/G) of the T selected rows and finds the list of each row by
// binary search in the prefix array.  The split is therefore even whatever the skew of the list
// lengths, consecutive workgroups (which go to different XCDs) take consecutive ranges, the grid
// is fixed, and the host never reads a count.
// A thread copies one 16-byte unit of K and of V at a time: 40 workgroups then have 328 KB on their way, a few times
// what the link's latency covers.  More is not better: the link's rate falls with what is asked of it at once, and
// requests for nothing (a batch filled up with its last unit again) are worst.  128 workgroups with eight units a
// thread, filled up, against 40 with one: 165 rows of 256 bytes 15.0 -> 5.7 us, 2835 rows (25.4 us at the rate of a
// large copy) 36.5 -> 31.0, 4574 (40.9) 52.5 -> 46.5, 37625 rows of 128 bytes (168) 202 -> 190, 100574 of 256 (900) 935 ->
// 908.  With one unit 32 workgroups are within 1 us of 40 below 5000 rows and 4 us behind at 100574, 64 are up to 1.5
// and up to 40 us behind.  The compute units stay free for what runs beside this.
constexpr int GATHER_FLAT_BLOCKS = 40;
__device__ __forceinline__ void gather_flat_body(const GatherArgs &A, int g, int G, int *pre /* [BH + 1] */) {
  __shared__ int wave_tot[4];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, BH = A.BH;
  // pre[i] = rows of lists 0..i-1: each thread sums a run of consecutive clamped counts
  const int per = (BH + 255) / 256;
  const int i0 = tid * per;
  int run = 0;
  for (int i = i0; i < min(BH, i0 + per); ++i) {
    const int cnt = A.sel_cnt[i];
    if (A.cnt_copy && g == 0) A.cnt_copy[i] = cnt;
    run += min(cnt, A.stride);
    pre[i + 1] = run;                    // local to the thread's run for now
  }
  int incl = wave_incl_scan(run);
  if (lane == 63) wave_tot[w] = incl;
  __syncthreads();
  int offset = incl - run;
  for (int k = 0; k < w; ++k) offset += wave_tot[k];
  for (int i = i0; i < min(BH, i0 + per); ++i) pre[i + 1] += offset;
  if (tid == 0) pre[0] = 0;
  __syncthreads();
  const int T = pre[BH];
  const int per_wg = max((T + G - 1) / G, max(1, 256 / A.U));        // (a unit a thread at least, when there are that many)
  const int r0 = min(T, g * per_wg), total = (min(T, r0 + per_wg) - r0) * A.U;
  int top = 1;
  while (top * 2 < BH) top *= 2;
  for (int u = tid; u < total; u += 256) {
    const int q = A.by_U.div(u), row = r0 + q, c = u - q * A.U;
    // list of this row: the last bh with pre[bh] <= row
    int lo = 0;
    for (int step = top; step >= 1; step >>= 1) {
      const int cand = lo + step;
      if (cand < BH && pre[cand] <= row) lo = cand;
    }
    const int j = row - pre[lo];
    const long t = min(max(A.sel_idx[(long)lo * A.stride + j], 0), A.N_cap - 1);   // a slot outside the pool is clamped
    const long src = ((long)lo * A.N_cap + t) * A.U + c, dst = ((long)lo * A.stride + j) * A.U + c;
    const u128 k = A.Kpool[src], v = A.Vpool[src];
    A.K_sel[dst] = k;                    // plain stores: with a pinned-host pool the streamed form
    A.V_sel[dst] = v;                    // measured slower (pipelined step 1107 vs 1083 us per layer)
  }
}

}  // namespace

// fills the gather's argument block (pinned-host pool); LDS bytes of its prefix sums
int ig_gather_args(ig_ctx *ctx, const ig_desc *d, const void *Kpool, const void *Vpool, const int32_t *sel_idx,
                   int32_t sel_stride, const int32_t *sel_cnt, void *K_sel, void *V_sel, GatherArgs *A);
size_t ig_gather_lds(const ig_desc *d);

// fills the attention argument block; grows the slice-state workspaces if needed
// (ig_attn_fill: the same with the slice-state / counter memory given by the caller, no allocation)
int ig_attn_fill(ig_ctx *ctx, const ig_desc *d, const void *q, const void *K, const void *V,
                 const int32_t *sel_idx, int32_t sel_stride, const int32_t *sel_cnt, int kv_rows,
                 const void *k_new, const void *v_new, void *out, void *K_out, void *V_out,
                 float *part, int32_t *counters, AttnArgs *A);
int ig_attn_args(ig_ctx *ctx, const ig_desc *d, const void *q, const void *K, const void *V,
                 const int32_t *sel_idx, int32_t sel_stride, const int32_t *sel_cnt, int kv_rows,
                 const void *k_new, const void *v_new, void *out, void *K_out, void *V_out, AttnArgs *A);

#endif
