// Device side of the projection that runs inside the scan's launch: the workgroups that multiply the weight,
// the words through which the scanning workgroups get their partial query, and how one of them works
// it out alone.  Shared by the scan kernels and by the kernel that runs a layer's scan beside the previous
// layer's attention.
//
// The grid's first `blocks` workgroups project, the others scan.  A scanning workgroup asks for its first slab
// planes, waits for its query and goes on; the launch and the chain of round trips of a kernel of its
// own are gone, and the weight is read while the slab's first planes are on their way.
//
// A projecting workgroup takes 16 columns and a quarter of K, its four waves a K slice each (the slices of the
// stand-alone kernel); the waves' sums are added in LDS, so that a query entry crosses the chip as at most
// four partial sums instead of 16.  They travel as self-validating 8-byte words: "published" bit and float32
// value in one agent-scope atomic, so nothing has to be ordered against anything else, and no wave waits
// for a store to be acknowledged before it may raise a flag.
//
// Rehearsals of 32 heads of 128 columns, 38 kept, projection and scan one after the other and so: one sequence of
// 1999 tokens 8.6 -> 7.1 us, eight of 2048 13.4 -> 10.7, sixteen rotary ones of 4096 40.9 -> 38.6; 20 sequences
// of 56 heads 43.4 -> 42.2; four rotary ones of 40 heads and 32768 tokens 64.1 -> 62.7.  What is left is HBM: 73, 193, 205
// and 314 MB at 5 TB/s in the last four.  A launch less is also 3 us less of the host's time.
//
// Who clears the words: the reader does, once it has read them (the last split of a pair to be done where
// several read them), so between launches all of them are zero, also between the replays of a captured launch.
// The wait is bounded (ig_set_wait_limit).  A workgroup that gives up works its query out alone, with the same
// matrix instructions in the same order, and leaves its words as "abandoned"; the atomic exchange by which either side
// writes tells whoever comes second that the other has been there, and the second one clears the word.
#ifndef IG_PROJECT_DEVICE_H
#define IG_PROJECT_DEVICE_H
#include "ig_internal.h"

namespace {

constexpr unsigned long long WORD_PUBLISHED = 1ull << 63, WORD_ABANDONED = 1ull << 62;

// acc[i]: the wave's K slice `ks` times column block cblk and batch block nb + i (operands and result registers as
// in project_mfma).  KB pieces of the weight and NB * KB of x are in flight at a time.
template <int NB, int KB>
__device__ __forceinline__ void project_slice(const ProjWords &p, int cblk, int ks, int nb, int lane, floatx4 (&acc)[NB]) {
  const int kb0 = ks * p.kb_per, kb1 = min(p.nKblk, kb0 + p.kb_per);
  const half8 *wp = static_cast<const half8 *>(p.blob) + (long)cblk * p.nKblk * 64 + lane;
  const half_t *xp[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    acc[i] = floatx4{0.f, 0.f, 0.f, 0.f};
    xp[i] = static_cast<const half_t *>(p.x) + (long)min((nb + i) * 16 + (lane & 15), p.B - 1) * p.D + (lane >> 4) * 8;
  }
  for (int kb = kb0; kb < kb1; kb += KB) {
    half8 a[KB], b[NB][KB];
#pragma unroll
    for (int t = 0; t < KB; ++t) {
      const int kbt = min(kb + t, kb1 - 1);
      a[t] = wp[(long)kbt * 64];
#pragma unroll
      for (int i = 0; i < NB; ++i) b[i][t] = *reinterpret_cast<const half8 *>(xp[i] + kbt * 32);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < KB; ++t) {
      keep_loaded(a[t]);
#pragma unroll
      for (int i = 0; i < NB; ++i) keep_loaded(b[i][t]);
      if (kb + t < kb1) {
#pragma unroll
        for (int i = 0; i < NB; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[t], b[i][t], acc[i], 0, 0, 0);
      }
    }
  }
}

// The slices of quarter kq by the four waves of a group (waves 4 g .. 4 g + 3) into the group's
// red[wave][batch block][row][column]; a barrier follows.  (A wave past the last slice leaves zeros.)
template <int NB, int KB>
__device__ __forceinline__ void project_quarter(const ProjWords &p, int cblk, int kq, int nb, float *red) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((threadIdx.x >> 6) & 3);
  floatx4 acc[NB];
  project_slice<NB, KB>(p, cblk, kq * 4 + w, nb, lane, acc);
#pragma unroll
  for (int i = 0; i < NB; ++i)
    *reinterpret_cast<floatx4 *>(red + (w * NB + i) * 256 + (lane & 15) * 16 + (lane >> 4) * 4) = acc[i];
  __syncthreads();
}
template <int NB> __device__ __forceinline__ float quarter_sum(const float *red, int i, int e) {
  float t = red[i * 256 + e];
#pragma unroll
  for (int k = 1; k < 4; ++k) t += red[(k * NB + i) * 256 + e];
  return t;
}
__device__ __forceinline__ unsigned long long *query_words(const ProjWords &p, int bh) { return p.words + (long)bh * p.KQ * p.ld; }

// One projecting workgroup of NG groups of four waves, a work item (column block, quarter of K, NB blocks of 16 batch
// rows) each.  Workgroups are handed to the 8 XCDs round-robin by id: those of the same columns and K are 8 ids
// apart, so that the weight of a second batch block comes out of the L2.
template <int NB, int KB, int NG>
__device__ __forceinline__ void project_items(const ProjWords &p, int wg, float *red) {
  const int g = NG > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 8) : 0, t = threadIdx.x & 255;
  red += g * (NB * 1024);
  const int oct = p.by_8groups.div(wg), rest = wg - oct * 8 * p.groups, nb = (rest >> 3) * NB;
  const int id = (oct * 8 + (rest & 7)) * NG + g;
  const int at = p.by_KQ.div(id), kq = id - at * p.KQ;
  const int cblk = min(at, p.nCblk - 1);                    // (the item count is rounded up)
  project_quarter<NB, KB>(p, cblk, kq, nb, red);
  const int c = cblk * 16 + (t & 15);
  if (at >= p.nCblk || c >= p.C) return;
  const int h = p.by_width.div(c), j = c - h * p.width;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int b = (nb + i) * 16 + (t >> 4);
    if (b >= p.B) break;
    unsigned long long *word = query_words(p, b * p.H + h) + kq * p.ld + j;
    const unsigned long long v = WORD_PUBLISHED | __float_as_uint(quarter_sum<NB>(red, i, t));
    if (__hip_atomic_exchange(word, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == WORD_ABANDONED)
      __hip_atomic_store(word, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}
constexpr int PROJECT_LDS = 2 * 1024;      // floats a group of four waves needs
template <int NG> __device__ __forceinline__ void project_publish(const ProjWords &p, int wg, float *red /* NG * PROJECT_LDS */) {
  if (p.both) project_items<2, 5, NG>(p, wg, red);
  else project_items<1, 8, NG>(p, wg, red);
}

// Query entry j of pair bh for this lane (whole waves; lanes with live == false ask for nothing): waits for its
// words and adds them to acc in order.  false: the wait ran out for some lane of the wave.
__device__ __forceinline__ bool await_query(const ProjWords &p, int bh, int j, bool live, float &acc) {
  if (p.limit < 0) return false;
  const unsigned long long *word = query_words(p, bh) + j;
  const long t0 = wall_clock64();
  while (true) {
    unsigned long long v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v[k] = WORD_PUBLISHED;
      if (live) v[k] = __hip_atomic_load(word + min(k, p.KQ - 1) * p.ld, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (__ballot((v[0] & v[1] & v[2] & v[3] & WORD_PUBLISHED) != 0) == ~0ull) {
#pragma unroll
      for (int k = 0; k < 4; ++k) acc += k < p.KQ ? __uint_as_float((unsigned)v[k]) : 0.f;
      return true;
    }
    if (wall_clock64() - t0 > p.limit) return false;
    __builtin_amdgcn_s_sleep(2);
  }
}
// Clears pair bh's words for the next launch (whole waves; threads first, first + step, ...).  `seen`: all of them
// were seen published by the caller's workgroup.
__device__ __forceinline__ void clear_words(const ProjWords &p, int bh, int first, int step, bool seen) {
  unsigned long long *word = query_words(p, bh);
  for (int i = first; i < p.KQ * p.ld; i += step) {
    const int j = i - p.by_ld.div(i) * p.ld;
    if (j >= p.width) continue;                             // (never written)
    if (seen || __hip_atomic_exchange(word + i, WORD_ABANDONED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0ull)
      __hip_atomic_store(word + i, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}
// The slow route: the workgroup works out the query of (b, h) alone, into q[0 .. width-1], its bias included; a
// barrier follows.  (Further groups of four waves do the same as the first, in LDS of their own.)
__device__ __forceinline__ void own_query(const ProjWords &p, const float *bias, int b, int h, float *red, float *q) {
  const int c0 = h * p.width, n = b & 15, t = threadIdx.x;
  red += (threadIdx.x >> 8) * 1024;
  for (int cblk = c0 / 16; cblk * 16 < c0 + p.width; ++cblk) {
    const int c = cblk * 16 + t, j = c - c0;
    const bool mine = t < 16 && j >= 0 && j < p.width;
    float acc = mine && bias ? bias[c] : 0.f;
    for (int kq = 0; kq < p.KQ; ++kq) {
      project_quarter<1, 4>(p, cblk, kq, b >> 4, red);
      if (mine) acc += quarter_sum<1>(red, 0, n * 16 + t);
      __syncthreads();
    }
    if (mine) q[j] = acc;
  }
  __syncthreads();
}

}  // namespace

#endif
