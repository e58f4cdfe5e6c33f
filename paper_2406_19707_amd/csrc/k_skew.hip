// Offline skewing on the GPU (Section 4.2 "Skewed Partial Weight", Eq. 2 and Eq. 3; Section 4.3
// "Prefetching Scheme"): per head, A_h = V of the SVD Q_h = U S V^T of the calibration queries.
//
// As in the host version, V is obtained from the Gram matrix: Q_h^T Q_h = V S^2 V^T.
//   gram_heads       G_h = Q_h^T Q_h in double on the matrix cores, one 16 x 16 tile of the upper
//                    triangle per workgroup
//   onesided_heads   d <= 128: one workgroup per head, everything in LDS and registers.  A pivoted
//                    Cholesky factor G = L L^T, then one-sided Jacobi rotations of L's columns until
//                    they are orthogonal: L J = V S, so the columns' norms are the singular values
//                    and the normalised columns are V; no second matrix is carried along.
//   jacobi_heads     d > 128 (the factor does not fit the LDS): cyclic two-sided Jacobi on G with V
//                    accumulated, both in device memory
// The eigenvalues are then ranked in descending order (the earlier column first on ties), each
// eigenvector's sign is chosen so that its largest-magnitude entry is positive, and A_h (float32)
// and the singular values are written.  All sums and rotations are double (the angles of onesided_heads
// float32: they steer the iteration, whose end does not depend on them), and what both leave is checked.
#include "ig_internal.h"

namespace {

constexpr int JACOBI_SWEEPS = 16;

typedef double double4v __attribute__((ext_vector_type(4)));

// One workgroup per 16 x 16 tile (ta <= tb) of G_h: the four waves take every fourth group of 4 rows
// of Q_h, 8 groups (16 loads of 4 bytes a lane) in flight at a time, and their sums are added in wave
// order.  Latency-bound: 512 rows are 32 matrix instructions a wave.  (One thread an entry, walking the
// rows, took 159 us on 32 heads of 128 columns and 512 rows.)
__global__ __launch_bounds__(256) void gram_heads(const float *__restrict__ Qcal, double *__restrict__ G,
                                                  int n, int D, int d, int T) {
  __shared__ double red[4][256];
  const int h = blockIdx.y;
  int ta = 0, rest = blockIdx.x;
  while (rest >= T - ta) { rest -= T - ta; ++ta; }
  const int tb = ta + rest;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int i = lane & 15, k = lane >> 4;
  // columns past the head and rows past the last are read clamped and multiplied as zeros
  const int ca = ta * 16 + i, cb = tb * 16 + i;
  const float *pa = Qcal + (long)h * d + min(ca, d - 1), *pb = Qcal + (long)h * d + min(cb, d - 1);
  double4v acc = {0.0, 0.0, 0.0, 0.0};
  constexpr int U = 8;
  for (int r0 = w * 4; r0 < n; r0 += 16 * U) {
    float a[U], b[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long at = (long)min(r0 + 16 * u + k, n - 1) * D;
      a[u] = pa[at];
      b[u] = pb[at];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in = r0 + 16 * u + k < n;
      const double av = in && ca < d ? (double)a[u] : 0.0, bv = in && cb < d ? (double)b[u] : 0.0;
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc, 0, 0, 0);
    }
  }
  // result register v of a lane: row v*4 + lane/16 of the tile, column lane%16
#pragma unroll
  for (int v = 0; v < 4; ++v) red[w][(v * 4 + k) * 16 + i] = acc[v];
  __syncthreads();
  const int t = threadIdx.x;
  const double g = ((red[0][t] + red[1][t]) + red[2][t]) + red[3][t];
  const int a = ta * 16 + t / 16, b = tb * 16 + t % 16;
  if (a < d && b < d) {
    G[((long)h * d + a) * d + b] = g;
    if (ta != tb) G[((long)h * d + b) * d + a] = g;
  }
}

// ---- d <= 128: pivoted Cholesky factor and one-sided Jacobi in LDS and registers -------------------
// Columns are rotated in pairs x, x ^ m for m = 1 .. DP-1 (every pair once a sweep).  A wave takes 16 pairs
// at a time: lane (part, g), g = lane % 16, holds every fourth row of column A_g and of its partner B_g in
// registers, so that a pair's inner product is RP = DP/4 multiply-adds and two cross-lane steps and every
// lane works out its own pair's rotation.  All m with the same highest bit that differ only in m's low
// (up to 4) bits run without leaving the registers: between two of them the B columns change lanes, by
// one DPP move (xor 1, 2, 7 or 15 inside 16 lanes reaches every pairing).  The 31 rounds inside the wave's own 32
// columns (m < 32) trade columns between the A and B registers instead of going through LDS (four instructions
// a register, against 3.3 us for a trip of both columns); then blocks of 16 meet, all m with the same highest
// bit with the A columns kept and only the B columns stored and loaded (6 such trips a sweep of 127 rounds at
// DP = 128, the points where the waves meet).
// Rotations are square-root free on the columns (two multiply-adds an element pair; the cosines
// are collected in a factor per column and multiplied in when it goes back to LDS).  Angles come from
// float32 (a rotation by a slightly wrong angle is still a rotation; its cosine is worked out in double),
// which leaves 1e-7 of a pair's inner product for the next sweep.
// When a sweep has met no cosine over 1e-6, S^T S is formed on the matrix cores (10 us) and every pair is looked at:
// cosines of at most 1e-13, where rounding leaves 1e-15, end the sweeps if each is also small against the distance
// of its pair's squared norms (1e-10 of it); if not, after one more sweep.  Nothing coarser will do: columns whose
// norms differ by less than their cosine are still turned by large angles, which carries what a later pair has
// left into a pair that was done already, and nearly equal singular values make their columns of V as much worse
// as they are close.  (With an end at a cosine of 1e-5, 128 singular values within 1e-3 of each other left A^T A
// 2.8e-7 from the identity and moved entries of V by 1e-3; with 1e-13 whatever the distance, 64 within 1e-4 of
// each other moved them by 3e-6.)
// Bound by the double-precision issue rate of the head's compute unit, one wave per SIMD: a round is
// 3 multiply-adds and 2 moves for each of RP rows and a chain of about 40 dependent operations.
// The pivoted factor matters: L's columns come out graded, which takes 8 sweeps where the columns of G
// itself take more than 20, and a head without full rank is found by a pivot at rounding level: those
// columns are left out of the rotations and V is completed to an orthonormal basis.
// Measured on 32 heads of 128 columns, with the Gram matrices: 0.72 to 0.76 ms; 0.92 with both columns through LDS at
// every highest bit and a ninth sweep that only looked, of which the kept A columns are worth 0.05, the trades
// 0.02 and the sweep 0.08.  Two-sided rotations of G and V through the L2 (jacobi_heads): 34.8 ms.
__device__ __forceinline__ double join_d(unsigned lo, unsigned hi) {
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
template <int CTRL> __device__ __forceinline__ double dpp_d(double v) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)u, CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(u >> 32), CTRL, 0xF, 0xF, true);
  return join_d((unsigned)lo, (unsigned)hi);
}
// sum over lanes l, l ^ 16, l ^ 32, l ^ 48, returned in each of them
__device__ __forceinline__ double sum_parts(double v) {
  typedef unsigned uint2v __attribute__((ext_vector_type(2)));
  unsigned long long u = (unsigned long long)__double_as_longlong(v);
  uint2v lo = __builtin_amdgcn_permlane16_swap((unsigned)u, (unsigned)u, false, false);
  uint2v hi = __builtin_amdgcn_permlane16_swap((unsigned)(u >> 32), (unsigned)(u >> 32), false, false);
  v = join_d(lo[0], hi[0]) + join_d(lo[1], hi[1]);
  u = (unsigned long long)__double_as_longlong(v);
  lo = __builtin_amdgcn_permlane32_swap((unsigned)u, (unsigned)u, false, false);
  hi = __builtin_amdgcn_permlane32_swap((unsigned)(u >> 32), (unsigned)(u >> 32), false, false);
  return join_d(lo[0], hi[0]) + join_d(lo[1], hi[1]);
}
template <int RP> __device__ __forceinline__ double column_dot(const double (&a)[RP], const double (&b)[RP]) {
  double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int k = 0; k < RP; ++k) s[k & 3] = fma(a[k], b[k], s[k & 3]);
  return sum_parts((s[0] + s[1]) + (s[2] + s[3]));
}
constexpr double FAR2 = 1e-12;             // a cosine of 1e-6, squared
// Tangent, cosine and 1 / cosine of the rotation that makes columns with squared norms al, be and inner
// product ga orthogonal (0, 1, 1 where they are to rounding); `far` is set when they were not nearly so.
__device__ __forceinline__ void rotation(double al, double be, double ga, double &t, double &c, double &ic, bool &far) {
  const double g2 = ga * ga, ab = al * be;
  far = far || g2 > FAR2 * ab;
  const float z = (float)(be - al) * __builtin_amdgcn_rcpf((float)(2.0 * ga)), az = fabsf(z);
  // (z^2 leaves float32's range where one column is far shorter than the other)
  float tf = __builtin_amdgcn_rcpf(az + (az < 1e9f ? __builtin_amdgcn_sqrtf(fmaf(z, z, 1.f)) : az));
  tf = z < 0.f ? -tf : tf;
  const bool turn = (g2 > 1e-30 * ab) & (fabsf(tf) <= 1.f);      // (no branch)
  tf = turn ? tf : 0.f;
  t = (double)tf;
  const double x = fma(t, t, 1.0), hx = -0.5 * x;
  double y = (double)__builtin_amdgcn_rsqf(fmaf(tf, tf, 1.f));
  y = y * fma(hx * y, y, 1.5);
  c = y * fma(hx * y, y, 1.5);
  ic = x * c;
}
// The 16 column pairs a wave has in registers: column = D x what they hold, I = 1 / D, n = squared norm.
template <int RP> struct Pair {
  double a[RP], b[RP], na, nb, Da, Ia, Db, Ib;
};
// Rounds X, X + 1, .. of `rounds` (1, 2, 4, 8 or 16): rotate every pair, move the B columns on.  Spelled out
// by recursion: a loop around the four kinds of move copies the columns at every turn.
template <int X, int RP>
__device__ __forceinline__ void rotate_rounds(Pair<RP> &P, int rounds, bool &far) {
  const double ga = column_dot<RP>(P.a, P.b) * (P.Da * P.Db);
  double t, c, ic;
  rotation(P.na, P.nb, ga, t, c, ic, far);
  const double ta = -t * (P.Db * P.Ia), tb = t * (P.Da * P.Ib);
#pragma unroll
  for (int k = 0; k < RP; ++k) {
    const double av = P.a[k];
    P.a[k] = fma(ta, P.b[k], av);
    P.b[k] = fma(tb, av, P.b[k]);
  }
  const double c2 = c * c, t2 = t * t, tg = 2.0 * t * ga;
  const double na = c2 * (fma(t2, P.nb, P.na) - tg);
  P.nb = c2 * (fma(t2, P.na, P.nb) + tg);
  P.na = na;
  P.Da *= c;
  P.Db *= c;
  P.Ia *= ic;
  P.Ib *= ic;
  if constexpr (X < 15) {
    if constexpr ((X & (X + 1)) == 0) {
      if (rounds == X + 1) return;
    }
    constexpr int CTRL = X % 2 == 0 ? DPP_QUAD_1032 : (X % 4 == 1 ? DPP_QUAD_2301 : (X == 7 ? DPP_ROW_MIRROR : DPP_ROW_HALF_MIRROR));
#pragma unroll
    for (int k = 0; k < RP; ++k) P.b[k] = dpp_d<CTRL>(P.b[k]);
    P.nb = dpp_d<CTRL>(P.nb);
    P.Db = dpp_d<CTRL>(P.Db);
    P.Ib = dpp_d<CTRL>(P.Ib);
    rotate_rounds<X + 1, RP>(P, rounds, far);
  }
}
// From pairs that differ in bit X of their column number to pairs that differ in bit X + 1: column A of the lanes
// with bit X of their number set and column B of those without change places, between lanes l and l ^ (1 << X).
template <int X> __device__ __forceinline__ int lane_xor(int v) {
  static_assert(X >= 0 && X < 4, "inside 16 lanes");
  if constexpr (X == 0) return __builtin_amdgcn_mov_dpp(v, DPP_QUAD_1032, 0xF, 0xF, true);
  if constexpr (X == 1) return __builtin_amdgcn_mov_dpp(v, DPP_QUAD_2301, 0xF, 0xF, true);
  if constexpr (X == 2) return __builtin_amdgcn_mov_dpp(__builtin_amdgcn_mov_dpp(v, DPP_ROW_HALF_MIRROR, 0xF, 0xF, true), 0x1B, 0xF, 0xF, true);
  return __builtin_amdgcn_mov_dpp(v, 0x128, 0xF, 0xF, true);       // row_ror:8
}
template <int X> __device__ __forceinline__ void trade(int &a, int &b, bool set) {
  const int got = lane_xor<X>(set ? a : b);
  a = set ? got : a;
  b = set ? b : got;
}
template <int X> __device__ __forceinline__ void trade(double &a, double &b, bool set) {
  const unsigned long long ua = (unsigned long long)__double_as_longlong(a), ub = (unsigned long long)__double_as_longlong(b);
  int al = (int)ua, ah = (int)(ua >> 32), bl = (int)ub, bh = (int)(ub >> 32);
  trade<X>(al, bl, set);
  trade<X>(ah, bh, set);
  a = join_d((unsigned)al, (unsigned)ah);
  b = join_d((unsigned)bl, (unsigned)bh);
}
// 1 / D anew, a dozen instructions: the product that rotate_rounds keeps drifts from it by some roundings a round, and
// a rotation whose columns' factors do not cancel is not quite orthogonal.  (Over the at most 64 rounds between two
// loads that is 1e-14 and was not seen in any result: 2.6e-8 from 64 bits either way.  But trading the product's two
// registers costs more than working it out: 32 heads of 128 columns 749 us with the product kept, 739 so.)
__device__ __forceinline__ double inverse_of(double D) {
  double y = __builtin_amdgcn_rcp(D);
  y = fma(fma(-D, y, 1.0), y, y);
  return fma(fma(-D, y, 1.0), y, y);
}
template <int X, int RP> __device__ __forceinline__ void regroup(Pair<RP> &P, int &ia, int &ib, int lane) {
  const bool set = (lane >> X) & 1;
#pragma unroll
  for (int k = 0; k < RP; ++k) trade<X>(P.a[k], P.b[k], set);
  trade<X>(P.na, P.nb, set);
  trade<X>(P.Da, P.Db, set);
  P.Ia = inverse_of(P.Da);
  P.Ib = inverse_of(P.Db);
  trade<X>(ia, ib, set);
}
__device__ __forceinline__ unsigned wave_max_u32(unsigned v) {
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, DPP_QUAD_1032, 0xF, 0xF, false));
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, DPP_QUAD_2301, 0xF, 0xF, false));
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, DPP_ROW_HALF_MIRROR, 0xF, 0xF, false));
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, DPP_ROW_MIRROR, 0xF, 0xF, false));
  const unsigned r0 = __builtin_amdgcn_readlane(v, 0), r1 = __builtin_amdgcn_readlane(v, 16);
  const unsigned r2 = __builtin_amdgcn_readlane(v, 32), r3 = __builtin_amdgcn_readlane(v, 48);
  return max(max(r0, r1), max(r2, r3));
}

// S^T S by the four waves, in tiles of 16 x 16 (the diagonal ones or those above): f(row, column, value) for
// each entry of a tile, rows and columns as in gram_heads (entries past the head's columns are zeros).
template <int DP, int LD, typename F>
__device__ __forceinline__ void gram_tiles(const double *S, int w, int g, int part, bool diagonal, F &&f) {
  constexpr int NBLK = DP / 16, RP = DP / 4;
  for (int t = w; t < (diagonal ? NBLK : NBLK * (NBLK - 1) / 2); t += 4) {
    int ta = diagonal ? t : 0, rest = diagonal ? 0 : t + 1;
    while (!diagonal && rest >= NBLK - ta) { rest -= NBLK - ta - 1; ++ta; }
    const double *va = S + (ta * 16 + g) * LD + part, *vb = S + ((ta + rest) * 16 + g) * LD + part;
    double4v acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 8
    for (int k = 0; k < RP; ++k) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(va[4 * k], vb[4 * k], acc, 0, 0, 0);
#pragma unroll
    for (int v = 0; v < 4; ++v) f(ta * 16 + v * 4 + part, (ta + rest) * 16 + g, acc[v]);
  }
}

template <int DP>
__global__ __launch_bounds__(256, 1) void onesided_heads(const double *__restrict__ Gall, float *__restrict__ A,
                                                         float *__restrict__ sigma, int32_t *status, int d) {
  constexpr int RP = DP / 4;               // rows a lane holds of a column
  constexpr int LD = DP + 2;               // column stride: 16 columns x 2 rows fall into different banks
  constexpr int NT = 256, NBLK = DP / 16;  // blocks of 16 columns; two to a wave: NBLK / 2 waves rotate
  constexpr int TR = DP / 16;              // the Cholesky update: a TR x TR tile of G a thread
  constexpr int MAX_SWEEPS = 30;
  __shared__ double S[DP * LD];            // column c, row r at c*LD + r
  __shared__ double lvec[DP], diag[DP];
  __shared__ unsigned key[DP];
  __shared__ int place[DP];
  const int h = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const double *G = Gall + (long)h * d * d;
  // ---- G into registers, scaled by a power of two so that the largest diagonal entry is in [0.5, 1) ----
  double T[TR][TR];
  const int rb = tid & 15, cb = tid >> 4;  // rows rb + 16 i, columns cb + 16 j
#pragma unroll
  for (int j = 0; j < TR; ++j)
#pragma unroll
    for (int i = 0; i < TR; ++i) {
      const int r = rb + 16 * i, c = cb + 16 * j;
      T[i][j] = r < d && c < d ? G[(long)c * d + r] : 0.0;
    }
  if (rb == cb) {
#pragma unroll
    for (int i = 0; i < TR; ++i) diag[rb + 16 * i] = T[i][i];
  }
  __syncthreads();
  double top = 0.0;
  bool finite = true;
  for (int e = lane; e < DP; e += 64) {
    top = fmax(top, diag[e]);
    finite = finite && diag[e] <= 1.7976931348623157e308;
  }
  if (__ballot(!finite)) {                 // (every wave looks at all of the diagonal)
    // a NaN or an infinity among the head's queries is in its column's diagonal entry: no matrix
    const float none = __int_as_float(0x7FC00000);
    for (int e = tid; e < d * d; e += NT) A[(long)h * d * d + e] = none;
    if (sigma && tid < d) sigma[(long)h * d + tid] = none;
    if (tid == 0) atomicOr(status, IG_STATUS_NOCONV);
    return;
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) top = fmax(top, __shfl_xor(top, o, 64));
  int ex = 0;
  if (top > 0.0) (void)frexp(top, &ex);
  top = ldexp(top, -ex);
#pragma unroll
  for (int j = 0; j < TR; ++j)
#pragma unroll
    for (int i = 0; i < TR; ++i) T[i][j] = ldexp(T[i][j], -ex);
  // A pivot is the largest remaining diagonal entry to 16 bits, the earlier row first: the key is the
  // entry's float32 image with the row in its low bits, 0 for rows that are used up.
  // Thread r < DP keeps row r's diagonal entry by itself (with the arithmetic of the tile that holds it).
  unsigned alive = (1u << TR) - 1;         // rows of the thread's tile that are not used up
  double own_diag = tid < DP ? ldexp(diag[tid], -ex) : 0.0;
  bool own_alive = true;
  __syncthreads();                         // diag is overwritten
  auto publish = [&]() {
    if (tid < DP) {
      const float v = (float)own_diag;
      diag[tid] = own_diag;
      key[tid] = own_alive && v > 0.f ? (__float_as_uint(v) & ~127u) | (unsigned)(127 - tid) : 0u;
    }
  };
  publish();
  __syncthreads();
  const double least = 2.3e-16 * top;      // a pivot no larger than G's rounding ends the factorisation
  int rank = 0;
  unsigned k0 = key[lane], k1 = DP > 64 ? key[64 % DP + lane] : 0u;
  for (int j = 0; j < d; ++j) {
    const unsigned k = wave_max_u32(max(k0, k1));      // the same in every wave
    if (k == 0u) break;
    const int p = 127 - (int)(k & 127u);
    const double best = diag[p];
    if (!(best > least)) break;
    // column p of what is left goes to LDS as it is; it is scaled by 1 / sqrt(best) at the end
    if (cb == (p & 15)) {
#pragma unroll
      for (int jj = 0; jj < TR; ++jj)
        if (jj == (p >> 4)) {
#pragma unroll
          for (int i = 0; i < TR; ++i) S[j * LD + rb + 16 * i] = ((alive >> i) & 1u) ? T[i][jj] : 0.0;
        }
    }
    if (tid == 0) lvec[j] = best;
    if (tid == p) own_alive = false;
    alive &= ~((rb == (p & 15) ? 1u : 0u) << (p >> 4));
    __syncthreads();
    double inv = __builtin_amdgcn_rcp(best);       // and two Newton steps
    inv = fma(fma(-best, inv, 1.0), inv, inv);
    inv = fma(fma(-best, inv, 1.0), inv, inv);
    if (tid < DP) {
      const double l = S[j * LD + tid];
      own_diag = fma(l, l * -inv, own_diag);
    }
    publish();
    double rr[TR], cc[TR];
#pragma unroll
    for (int i = 0; i < TR; ++i) {
      rr[i] = S[j * LD + rb + 16 * i];
      cc[i] = S[j * LD + cb + 16 * i] * -inv;
    }
    __syncthreads();
    // (the next pivot's keys come in under the update)
    k0 = key[lane];
    k1 = DP > 64 ? key[64 % DP + lane] : 0u;
#pragma unroll
    for (int jj = 0; jj < TR; ++jj)
#pragma unroll
      for (int i = 0; i < TR; ++i) T[i][jj] = fma(rr[i], cc[jj], T[i][jj]);
    rank = j + 1;
  }
  __syncthreads();
  for (int e = tid; e < DP * DP; e += NT) {
    const int c = e / DP;
    S[c * LD + e % DP] = c < rank ? S[c * LD + e % DP] * (1.0 / sqrt(lvec[c])) : 0.0;
  }
  __syncthreads();
  // ---- one-sided Jacobi sweeps ----
  const int g = lane & 15, part = lane >> 4;
  bool straight = false, square = false, seen_small = false;
  for (int sweep = 0; sweep < MAX_SWEEPS && !straight; ++sweep) {
    bool far = false;
    Pair<RP> P;
    double *pa = S, *pb = S;               // where the lane's columns A and B lie
    auto load_a = [&]() {
#pragma unroll
      for (int k = 0; k < RP; ++k) P.a[k] = pa[4 * k];
      P.na = column_dot<RP>(P.a, P.a);
      P.Da = P.Ia = 1.0;
    };
    auto load_b = [&]() {
#pragma unroll
      for (int k = 0; k < RP; ++k) P.b[k] = pb[4 * k];
      P.nb = column_dot<RP>(P.b, P.b);
      P.Db = P.Ib = 1.0;
    };
    auto store_a = [&]() {
#pragma unroll
      for (int k = 0; k < RP; ++k) pa[4 * k] = P.a[k] * P.Da;
    };
    auto store_b = [&]() {
#pragma unroll
      for (int k = 0; k < RP; ++k) pb[4 * k] = P.b[k] * P.Db;
    };
    // pairs inside the wave's own 32 columns, by the highest bit in which their numbers differ; ia, ib: which
    // columns the lane holds.  The rounds' moves (xor 1, 2, 1, 7, 1, 2, 1, 15, ...) have taken the B columns to where
    // lane g holds lane g ^ 0, 1, 2, 7 and 15's (bits below the pair's own: any order in there meets every pair).
    if (w < NBLK / 2) {
      int ia = 32 * w + 2 * g, ib = ia + 1;
      pa = S + ia * LD + part;
      pb = S + ib * LD + part;
      load_a();
      load_b();
      rotate_rounds<0, RP>(P, 1, far);
      regroup<0, RP>(P, ia, ib, lane);
      rotate_rounds<0, RP>(P, 2, far);
      ib = __shfl_xor(ib, 1, 64);
      regroup<1, RP>(P, ia, ib, lane);
      rotate_rounds<0, RP>(P, 4, far);
      ib = __shfl_xor(ib, 2, 64);
      regroup<2, RP>(P, ia, ib, lane);
      rotate_rounds<0, RP>(P, 8, far);
      ib = __shfl_xor(ib, 7, 64);
      regroup<3, RP>(P, ia, ib, lane);
      rotate_rounds<0, RP>(P, 16, far);
      ib = __shfl_xor(ib, 15, 64);
      pa = S + ia * LD + part;
      pb = S + ib * LD + part;
      store_a();
      store_b();
    }
    __syncthreads();
    // block b0 against block b0 ^ M.  All M with the same highest bit hb pair the blocks without that bit with
    // those that have it, so a wave keeps its block A through them.
    for (int hb = 1; (1 << hb) < NBLK; ++hb) {
      const int b0 = ((w >> hb) << (hb + 1)) | (w & ((1 << hb) - 1));
      pa = S + (b0 * 16 + g) * LD + part;
      if (w < NBLK / 2) load_a();
      for (int M = 1 << hb; M < 2 << hb; ++M) {
        if (w < NBLK / 2) {
          pb = S + ((b0 ^ M) * 16 + g) * LD + part;
          load_b();
          P.Ia = inverse_of(P.Da);
          rotate_rounds<0, RP>(P, 16, far);
          pb = S + ((b0 ^ M) * 16 + (g ^ 15)) * LD + part;
          store_b();
          if (M == (2 << hb) - 1) store_a();
        }
        __syncthreads();
      }
    }
    if (__syncthreads_or(far) && sweep + 1 < MAX_SWEEPS) continue;
    // S^T S on the matrix cores: the diagonal tiles give the squared norms, the others are held against them
    bool off13 = false, off9 = false, close = false;
    gram_tiles<DP, LD>(S, w, g, part, true, [&](int r, int c, double v) {
      if (r == c) diag[r] = v;
    });
    __syncthreads();
    const auto look = [&](int r, int c, double v) {
      const double nn = diag[r] * diag[c];
      off13 = off13 || (r != c && !(v * v <= 1e-26 * nn));
      off9 = off9 || (r != c && !(v * v <= 1e-18 * nn));
      // (how far the pair is from the vectors it stands for: its cosine over the distance of its squared norms)
      const double most = fmax(diag[r], diag[c]), apart = diag[r] - diag[c];
      close = close || (r != c && !(v * v * most * most <= 1e-20 * apart * apart * nn));
    };
    gram_tiles<DP, LD>(S, w, g, part, true, look);
    gram_tiles<DP, LD>(S, w, g, part, false, look);
    const bool small = __syncthreads_or(off13) == 0;
    square = __syncthreads_or(off9) == 0;
    straight = small && (__syncthreads_or(close) == 0 || seen_small);
    seen_small = small;
  }
  // ---- normalised columns (diag, the squared norms, and lvec now belong to columns) ----
  if (tid < DP) lvec[tid] = diag[tid] > 0.0 ? 1.0 / sqrt(diag[tid]) : 0.0;
  __syncthreads();
  for (int e = tid; e < DP * DP; e += NT) S[(e / DP) * LD + e % DP] *= lvec[e / DP];
  __syncthreads();
  // ---- a head without full rank: complete V, one unit vector at a time ----
  for (int c = rank; c < d; ++c) {
    // the unit vector that the columns so far cover least
    if (tid < d) {
      double rest = 1.0;
      for (int k = 0; k < c; ++k) rest -= S[k * LD + tid] * S[k * LD + tid];
      lvec[tid] = rest;
    }
    __syncthreads();
    int e = 0;
    for (int i = 1; i < d; ++i)
      if (lvec[i] > lvec[e]) e = i;
    __syncthreads();
    if (tid < DP) S[c * LD + tid] = tid == e ? 1.0 : 0.0;
    for (int pass = 0; pass < 2; ++pass) {
      __syncthreads();
      if (tid < c) {
        double dot = 0.0;
        for (int i = 0; i < d; ++i) dot = fma(S[tid * LD + i], S[c * LD + i], dot);
        lvec[tid] = dot;
      }
      __syncthreads();
      if (tid < d) {
        double v = S[c * LD + tid];
        for (int k = 0; k < c; ++k) v = fma(-lvec[k], S[k * LD + tid], v);
        S[c * LD + tid] = v;
      }
    }
    __syncthreads();
    double n2 = 0.0;
    for (int i = 0; i < d; ++i) n2 = fma(S[c * LD + i], S[c * LD + i], n2);
    __syncthreads();
    if (tid < d) S[c * LD + tid] *= 1.0 / sqrt(n2);
    __syncthreads();
  }
  // ---- what the result rests on: the cosines measured last, and for a completed V what V^T V is ----
  bool off = !square;
  if (rank < d) {
    const auto check = [&](int r, int c, double v) { off = off || !(fabs(v - (r == c && r < d ? 1.0 : 0.0)) <= 1e-9); };
    gram_tiles<DP, LD>(S, w, g, part, true, check);
    gram_tiles<DP, LD>(S, w, g, part, false, check);
  }
  if (__ballot(off) && lane == 0) atomicOr(status, IG_STATUS_NOCONV);
  // ---- rank the singular values (descending, the earlier column first on ties), fix signs, write ----
  if (tid < d) {
    const double nc = diag[tid];
    int at = 0;
    for (int i = 0; i < d; ++i) at += (diag[i] > nc) || (diag[i] == nc && i < tid);
    int arg = 0;
    for (int i = 1; i < d; ++i)
      if (fabs(S[tid * LD + i]) > fabs(S[tid * LD + arg])) arg = i;
    lvec[tid] = S[tid * LD + arg] < 0 ? -1.0 : 1.0;
    place[at] = tid;
    if (sigma) sigma[(long)h * d + at] = (float)sqrt(ldexp(nc, ex));
  }
  __syncthreads();
  float *Ah = A + (long)h * d * d;
  for (int e = tid; e < d * d; e += NT) {
    const int c = place[e % d];
    Ah[e] = (float)(lvec[c] * S[c * LD + e / d]);
  }
}

// ---- d > 128: two-sided Jacobi through device memory ------------------------------------------------
// One workgroup per head: cyclic two-sided Jacobi with a round-robin (tournament) ordering, so that the
// d/2 rotations of a round act on disjoint index pairs and run in parallel: rotations are computed from
// the current G, then applied to the columns of G and V, then to the rows of G, with a barrier after
// each phase.  The number of sweeps is fixed (no data-dependent loop); what is left off the diagonal
// afterwards is checked and flagged.  G and V live in the double-precision workspace in device memory.
__global__ __launch_bounds__(256) void jacobi_heads(double *__restrict__ Gall, double *__restrict__ Vall,
                                                    float *__restrict__ A, float *__restrict__ sigma,
                                                    int32_t *status, int d) {
  extern __shared__ double rot[];            // c[half], s[half], then int p[half], q[half]
  __shared__ double lam[256];
  __shared__ double s_off, s_diag;
  const int h = blockIdx.x, tid = threadIdx.x;
  const int half = d / 2, m = d - 1;
  double *cc = rot, *ss = rot + half;
  int *pp = reinterpret_cast<int *>(rot + 2 * half), *qq = pp + half;
  double *G = Gall + (long)h * d * d, *V = Vall + (long)h * d * d;
  for (int e = tid; e < d * d; e += 256) V[e] = (e / d == e % d) ? 1.0 : 0.0;
  __syncthreads();
  for (int sweep = 0; sweep < JACOBI_SWEEPS; ++sweep) {
    for (int r = 0; r < m; ++r) {
      // round r of the tournament: pair 0 is (r, d-1), pair k is ((r+k) mod m, (r-k) mod m)
      for (int k = tid; k < half; k += 256) {
        int p = k == 0 ? r : (r + k) % m;
        int q = k == 0 ? d - 1 : (r - k + m) % m;
        if (p > q) { const int t = p; p = q; q = t; }
        const double gpq = G[(long)p * d + q], gpp = G[(long)p * d + p], gqq = G[(long)q * d + q];
        double c = 1.0, s = 0.0;
        if (gpq != 0.0 && fabs(gpq) > 1e-17 * sqrt(fabs(gpp * gqq))) {
          const double theta = (gqq - gpp) / (2.0 * gpq);
          const double t = (theta >= 0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(theta * theta + 1.0));
          c = 1.0 / sqrt(t * t + 1.0);
          s = t * c;
        }
        cc[k] = c; ss[k] = s; pp[k] = p; qq[k] = q;
      }
      __syncthreads();
      // columns p, q of G and V (consecutive threads: the pairs of one row)
      for (int item = tid; item < half * d; item += 256) {
        const int i = item / half, k = item % half;
        const int p = pp[k], q = qq[k];
        const double c = cc[k], s = ss[k];
        double a = G[(long)i * d + p], b = G[(long)i * d + q];
        G[(long)i * d + p] = c * a - s * b;
        G[(long)i * d + q] = s * a + c * b;
        a = V[(long)i * d + p]; b = V[(long)i * d + q];
        V[(long)i * d + p] = c * a - s * b;
        V[(long)i * d + q] = s * a + c * b;
      }
      __syncthreads();
      // rows p, q of G (consecutive threads: consecutive columns)
      for (int item = tid; item < half * d; item += 256) {
        const int k = item / d, j = item % d;
        const int p = pp[k], q = qq[k];
        const double c = cc[k], s = ss[k];
        const double a = G[(long)p * d + j], b = G[(long)q * d + j];
        G[(long)p * d + j] = c * a - s * b;
        G[(long)q * d + j] = s * a + c * b;
      }
      __syncthreads();
    }
  }
  // what is left off the diagonal, against the largest eigenvalue
  if (tid == 0) { s_off = 0.0; s_diag = 0.0; }
  __syncthreads();
  {
    double off = 0.0, dg = 0.0;
    for (int e = tid; e < d * d; e += 256) {
      const double v = fabs(G[e]);
      if (!(v <= 1.7976931348623157e308)) off = __longlong_as_double(0x7FF0000000000000ll);   // (fmax drops a NaN)
      else if (e / d == e % d) dg = fmax(dg, v);
      else off = fmax(off, v);
    }
    // maxima of non-negative doubles: their bit patterns order like unsigned integers
    atomicMax(reinterpret_cast<unsigned long long *>(&s_off), (unsigned long long)__double_as_longlong(off));
    atomicMax(reinterpret_cast<unsigned long long *>(&s_diag), (unsigned long long)__double_as_longlong(dg));
  }
  __syncthreads();
  if (tid == 0 && s_off > 1e-9 * s_diag) atomicOr(status, IG_STATUS_NOCONV);
  // rank the eigenvalues (descending, the earlier column first on ties), fix signs, write out
  if (tid < d) lam[tid] = G[(long)tid * d + tid];
  __syncthreads();
  for (int j = tid; j < d; j += 256) {
    const double lj = lam[j];
    int rank = 0;
    for (int i = 0; i < d; ++i) rank += (lam[i] > lj) || (lam[i] == lj && i < j);
    int arg = 0;
    for (int i = 1; i < d; ++i)
      if (fabs(V[(long)i * d + j]) > fabs(V[(long)arg * d + j])) arg = i;
    const double sgn = V[(long)arg * d + j] < 0 ? -1.0 : 1.0;
    float *Ah = A + (long)h * d * d;
    for (int i = 0; i < d; ++i) Ah[(long)i * d + rank] = (float)(sgn * V[(long)i * d + j]);
    if (sigma) sigma[(long)h * d + rank] = (float)sqrt(fmax(0.0, lj));
  }
}

}  // namespace

// Gram matrices; for d > 128 also the eigenvectors under construction
size_t ig_skew_workspace(int H, int d) { return (size_t)(d > 128 ? 2 : 1) * H * d * d * sizeof(double); }

int ig_launch_skew(ig_ctx *ctx, int D, int H, int n_cal, const float *Qcal, double *ws, float *A,
                   float *sigma, hipStream_t s) {
  const int d = D / H;
  double *G = ws;
  const int T = (d + 15) / 16;
  auto k1 = gram_heads;
  IG_LAUNCH(ctx, IG_K_BUILD, k1, dim3(T * (T + 1) / 2, H), dim3(256), s, Qcal, G, n_cal, D, d, T);
  if (d <= 64) {
    auto k2 = onesided_heads<64>;
    IG_LAUNCH(ctx, IG_K_BUILD, k2, dim3(H), dim3(256), s, (const double *)G, A, sigma, ctx->status, d);
    return IG_OK;
  }
  if (d <= 128) {
    auto k2 = onesided_heads<128>;
    IG_LAUNCH(ctx, IG_K_BUILD, k2, dim3(H), dim3(256), s, (const double *)G, A, sigma, ctx->status, d);
    return IG_OK;
  }
  double *V = ws + (size_t)H * d * d;
  auto k2 = jacobi_heads;
  const size_t lds = (size_t)(d / 2) * (2 * sizeof(double) + 2 * sizeof(int));
  IG_LAUNCH_LDS(ctx, IG_K_BUILD, k2, dim3(H), dim3(256), lds, s, G, V, A, sigma, ctx->status, d);
  return IG_OK;
}
