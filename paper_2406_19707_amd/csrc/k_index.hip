// Partial weight index generation on the GPU (Section 4.3 "Prefill Stage"): per head, the
// r = floor(ratio*d) columns with the largest sum over the prompt's rows of |Q~| + |K~|.
//
// Two kernels, both with a fixed summation order (no floating-point atomics, so a run repeats
// bit for bit):
//   column_abs_sums   a lane takes VEC consecutive columns (8-byte loads in half precision, 16-byte in
//                     float32) and a wave a quarter of one of ROW_CHUNKS row ranges; one partial
//                     sum per column and range is written
//   top_columns       one workgroup per head: adds the ROW_CHUNKS partial sums of each column in
//                     order, ranks the d columns (column j beats c when its sum is larger, or
//                     equal with j < c), keeps ranks < r and writes them in ascending order
#include "ig_internal.h"

namespace {

constexpr int ROW_CHUNKS = 32;

// HBM-bound (the rows are read once).  What it takes is bytes in flight: the grid is small (D columns
// x 32 ranges), so the four waves of a workgroup take a quarter of the range each, and a lane issues the loads
// of U rows of both matrices before it adds the first; the waves' sums are added in wave order.  2048 rows of 4096
// half columns, queries and keys (33.5 MB): 55 us with 2-byte loads one row at a time, with top_columns 14.6 us
// with one wave a range (512 waves, 64 rows each in four turns), 10.1 us so (one turn of 16 rows).  U is the
// smallest of 4, 8 and 16 that takes a wave's rows in one turn: loads past the last row read it again (56
// heads of 128, 700 rows, 6 a wave: two turns of 4 are 0.8 us behind the one wave a range, one of 8 ahead of it).
// Arrays whose rows or addresses do not allow the wide loads go one column a lane.
template <typename T, int VEC, int U>
__global__ __launch_bounds__(256) void column_abs_sums(const T *__restrict__ Qs, const T *__restrict__ Ks,
                                                       float *__restrict__ part, int n, int D) {
  typedef T vec __attribute__((ext_vector_type(VEC)));
  __shared__ float wave_sums[4][VEC][64];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = (blockIdx.x * 64 + lane) * VEC, cc = min(c, D - VEC);      // (lanes past the last column repeat it)
  const int chunk = blockIdx.y;
  const int rows_per = (n + ROW_CHUNKS - 1) / ROW_CHUNKS, per = (rows_per + 3) / 4;
  const int i0 = chunk * rows_per + w * per, i1 = min(min(n, (chunk + 1) * rows_per), i0 + per);
  const T *Kp = Ks ? Ks : Qs;                // (without keys: read and not added)
  float acc[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) acc[e] = 0.f;
  for (int i = i0; i < i1; i += U) {
    vec q[U], k[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long at = (long)min(i + u, i1 - 1) * D + cc;     // past the end: the last row again, not added
      q[u] = *reinterpret_cast<const vec *>(Qs + at);
      k[u] = *reinterpret_cast<const vec *>(Kp + at);
    }
    __builtin_amdgcn_sched_barrier(0);       // (the compiler would trade loads in flight for registers)
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (i + u < i1) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          acc[e] += fabsf((float)q[u][e]);
          if (Ks) acc[e] += fabsf((float)k[u][e]);
        }
      }
    }
  }
#pragma unroll
  for (int e = 0; e < VEC; ++e) wave_sums[w][e][lane] = acc[e];
  __syncthreads();
  if (w == 0 && c < D) {
#pragma unroll
    for (int e = 0; e < VEC; ++e)
      part[(long)chunk * D + c + e] =
          ((wave_sums[0][e][lane] + wave_sums[1][e][lane]) + wave_sums[2][e][lane]) + wave_sums[3][e][lane];
  }
}

// One workgroup per head and a chain of dependent steps: the ROW_CHUNKS partial sums of a column in flight
// at once, the d * d comparisons spread over PARTS threads a column (3 us on 32 heads of 128
// columns; 6.3 us with one load after another and d comparisons a thread).
template <int DP>      // columns, rounded up to 64, 128 or 256
__global__ __launch_bounds__(1024) void top_columns(const float *__restrict__ part, int32_t *__restrict__ idx,
                                                    int d, int D, int r) {
  constexpr int PARTS = 1024 / DP, PER = DP / PARTS;
  __shared__ __align__(16) float sum[DP];
  __shared__ int below[PARTS][DP];
  __shared__ int wave_tot[DP / 64];
  const int h = blockIdx.x, c = threadIdx.x % DP, p = threadIdx.x / DP, lane = threadIdx.x & 63;
  if (p == 0) {
    float v[ROW_CHUNKS];
    const float *col = part + h * d + min(c, d - 1);
#pragma unroll
    for (int k = 0; k < ROW_CHUNKS; ++k) v[k] = col[(long)k * D];
    __builtin_amdgcn_sched_barrier(0);
    float acc = 0.f;
#pragma unroll
    for (int k = 0; k < ROW_CHUNKS; ++k) acc += v[k];
    // sums are >= 0: columns past d never win; one that is NaN ranks as infinite (compared as it is it would
    // be beaten by none and beat none, and more than r columns would be kept)
    sum[c] = c < d ? (acc >= 0.f ? acc : INFINITY) : -1.f;
  }
  __syncthreads();
  // columns that beat column c: a larger sum, or an equal one further left
  const float v = sum[c];
  int n = 0;
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int j = p * PER + u;
    const float o = sum[j];
    n += (o > v) || (o == v && j < c);
  }
  below[p][c] = n;
  __syncthreads();
  bool kept = false;
  unsigned long long bal = 0;
  if (p == 0) {
    int rank = 0;
#pragma unroll
    for (int k = 0; k < PARTS; ++k) rank += below[k][c];
    kept = c < d && rank < r;
    bal = __ballot(kept);
    if (lane == 0) wave_tot[c / 64] = __popcll(bal);
  }
  __syncthreads();
  if (kept) {
    int pos = lanes_below(bal);
    for (int k = 0; k < c / 64; ++k) pos += wave_tot[k];
    idx[h * r + pos] = c;
  }
}

}  // namespace

int ig_launch_partial_index(ig_ctx *ctx, int dtype, int H, int d, int n, const void *Qs, const void *Ks,
                            int r, float *part, int32_t *idx, hipStream_t s) {
  const int D = H * d;
  const size_t align = (size_t)D * ig_elem_bytes(dtype) | (uintptr_t)Qs | (uintptr_t)Ks;
  const int per = ((n + ROW_CHUNKS - 1) / ROW_CHUNKS + 3) / 4;       // rows a wave
#define SUMS(T, VEC)                                                                               \
  {                                                                                                \
    auto k = per <= 4 ? column_abs_sums<T, VEC, 4>                                                 \
                      : (per <= 8 ? column_abs_sums<T, VEC, 8> : column_abs_sums<T, VEC, 16>);     \
    IG_LAUNCH(ctx, IG_K_BUILD, k, dim3((D + 64 * VEC - 1) / (64 * VEC), ROW_CHUNKS), dim3(256), s, \
              (const T *)Qs, (const T *)Ks, part, n, D);                                           \
  }
  if (dtype == IG_F16) {
    if (align % 8 == 0) SUMS(half_t, 4) else SUMS(half_t, 1)
  } else {
    if (align % 16 == 0) SUMS(float, 4) else SUMS(float, 1)
  }
#undef SUMS
#define TOP(DP)                                                                                    \
  {                                                                                                \
    auto k2 = top_columns<DP>;                                                                     \
    IG_LAUNCH(ctx, IG_K_BUILD, k2, dim3(H), dim3(1024), s, (const float *)part, idx, d, D, r);     \
  }
  if (d <= 64) TOP(64) else if (d <= 128) TOP(128) else TOP(256)
#undef TOP
  return IG_OK;
}

size_t ig_partial_index_workspace(int H, int d) { return (size_t)ROW_CHUNKS * H * d * sizeof(float); }
