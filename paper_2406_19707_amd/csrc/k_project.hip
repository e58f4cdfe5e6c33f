// Partial query projection (Section 4.3 "Decoding Stage": attention input of the previous layer
// times the partial query weight) and the small finalisation step (bias, rotary embedding and the
// partial skew A_h[:, idx_h] for models whose skew cannot be folded into W_Q).
//
// The projection reads the weight once (it is weight-read bound: B is 4..20 rows).  For half
// precision it runs on the matrix cores: the weight blob is stored in MFMA fragment order, so that
// every wave-wide load is one contiguous 1 KiB piece, the batch rows are the N side of a
// 16x16x32 MFMA, and K is split across waves to get enough waves in flight; the split-K partial
// sums are written out and added, in a fixed order, by the consumer.  float32 (and half with
// D % 32 != 0) uses a plain FMA kernel over the same split.
#include "ig_internal.h"

ProjGeom ig_proj_geom(const ig_desc *d) {
  ProjGeom g;
  const int D = d->H * d->d;
  g.C = d->rope ? D : d->H * d->r;
  g.nCblk = (g.C + 15) / 16;
  g.Cpad = g.nCblk * 16;
  g.NBtot = (d->B + 15) / 16;
  g.Bpad = g.NBtot * 16;
  g.mfma = d->dtype == IG_F16 && D % 32 == 0;
  const int units = g.mfma ? D / 32 : D;          // K units that can be split
  g.nKblk = g.mfma ? D / 32 : 0;
  // aim for >= 4096 waves (16 per compute unit: a wave then has a single batch of K blocks; measured
  // on a 4096 x 4096 weight, 8.8 -> 7.6 us against 2048 waves) but never more than IG_KS_MAX partial sums
  const int col_waves = g.mfma ? g.nCblk : (g.Cpad + 63) / 64;
  int ks = (4096 + col_waves - 1) / col_waves;
  if (ks > IG_KS_MAX) ks = IG_KS_MAX;
  if (ks > units) ks = units;
  if (ks < 1) ks = 1;
  g.kb_per = (units + ks - 1) / ks;
  g.KS = (units + g.kb_per - 1) / g.kb_per;
  return g;
}

namespace {

// ---- weight blob construction -------------------------------------------------------------------
// Column c of the blob is column colmap(c) of Wq: h*d + idx[h*r + j] for c = h*r + j (folded), or c
// itself (rope: every column kept).
__device__ __forceinline__ int colmap(int c, int d, int r, const int32_t *idx) {
  if (!idx) return c;
  int h = c / r, j = c % r;
  return h * d + min(max(idx[h * r + j], 0), d - 1);   // an index outside the head is clamped
}

// MFMA fragment order: piece (cblk, kblk) is 64 lanes x 8 halves; lane (kg = lane/16, i = lane%16)
// holds W[k = kblk*32 + kg*8 + e][col(cblk*16 + i)], e < 8.
__global__ void wq_build_mfma(const half_t *W, const int32_t *idx, half8 *blob, int D, int d, int r,
                              int C, int nCblk, int nKblk) {
  long g = (long)blockIdx.x * blockDim.x + threadIdx.x;
  long total = (long)nCblk * nKblk * 64;
  if (g >= total) return;
  int lane = g & 63;
  long piece = g >> 6;
  int kblk = piece % nKblk, cblk = piece / nKblk;
  int i = lane & 15, kg = lane >> 4;
  int c = cblk * 16 + i;
  half8 v;
  if (c < C) {
    int col = colmap(c, d, r, idx);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = W[(long)(kblk * 32 + kg * 8 + e) * D + col];
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (half_t)0;
  }
  blob[g] = v;
}

// Plain layout for the FMA kernel: blob[k][c], c < Cpad (zero padded).
template <typename T>
__global__ void wq_build_plain(const T *W, const int32_t *idx, T *blob, int D, int d, int r, int C,
                               int Cpad) {
  long g = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= (long)D * Cpad) return;
  int c = g % Cpad;
  long k = g / Cpad;
  blob[g] = (c < C) ? W[k * D + colmap(c, d, r, idx)] : (T)0;
}

// ---- projection ---------------------------------------------------------------------------------
// Wave (cblk, ks): part[ks][n][cblk*16 + i] = sum over its K blocks of W^T-fragment x x-fragment.
// A operand = weight piece (M side = 16 output columns), B operand = 16 batch rows of x.
// Result lane l, register v -> column cblk*16 + 4*(l/16) + v, batch row l%16.
template <int NB, int KB>
__global__ __launch_bounds__(256) void project_mfma(const half8 *__restrict__ blob,
                                                    const half_t *__restrict__ x,
                                                    float *__restrict__ part, int B, int D,
                                                    int nCblk, int nKblk, int kb_per, int Bpad,
                                                    int Cpad) {
  // grid (column blocks / 4, KS, batch blocks / NB): nothing to divide before the first load goes out
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int cblk = blockIdx.x * 4 + w, ks = blockIdx.y;
  if (cblk >= nCblk) return;
  const int nb0 = blockIdx.z * NB;
  const int n = lane & 15, kg = lane >> 4;
  const int kb0 = ks * kb_per, kb1 = min(nKblk, kb0 + kb_per);
  floatx4 acc[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) acc[i] = floatx4{0.f, 0.f, 0.f, 0.f};
  const half8 *wp = blob + ((long)cblk * nKblk) * 64 + lane;
  // (lanes of a batch row past the last read the last row: a row of x only reaches its own row of the result)
  const half_t *xp[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) xp[i] = x + (long)min((nb0 + i) * 16 + n, B - 1) * D + kg * 8;
  // K blocks are taken KB at a time: all weight pieces and x fragments of a batch are loaded before
  // the first MFMA, so a wave keeps KB * (1 + NB) KiB in flight (a block past the end is clamped
  // to the last one and its MFMA skipped).
  for (int kb = kb0; kb < kb1; kb += KB) {
    half8 a[KB], bfrag[NB][KB];
#pragma unroll
    for (int t = 0; t < KB; ++t) {
      const int kbt = min(kb + t, kb1 - 1);
      a[t] = wp[(long)kbt * 64];
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        bfrag[i][t] = *reinterpret_cast<const half8 *>(xp[i] + kbt * 32);
      }
    }
    __builtin_amdgcn_sched_barrier(0);   // (the compiler would trade loads in flight for registers)
#pragma unroll
    for (int t = 0; t < KB; ++t) {
      keep_loaded(a[t]);
#pragma unroll
      for (int i = 0; i < NB; ++i) keep_loaded(bfrag[i][t]);
      if (kb + t < kb1) {
#pragma unroll
        for (int i = 0; i < NB; ++i)
          acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[t], bfrag[i][t], acc[i], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    int row = (nb0 + i) * 16 + n;
    if (row < B) {                        // (the padding rows' sums are never read)
      float *o = part + ((long)ks * Bpad + row) * Cpad + cblk * 16 + kg * 4;
      *reinterpret_cast<floatx4 *>(o) = acc[i];
    }
  }
}

// The same product for more than 16 batch rows (NB blocks of 16) with the x fragments shared
// through LDS.  With NB = 2 the plain kernel above issues one weight load and two x loads per K
// block and needs three batches of loads per wave for the register budget; here the four waves of
// a workgroup (four neighbouring column blocks, the same K slice) stage the NB*16 rows of x for
// their K slice in LDS once, a wave keeps only its weight pieces in registers -- all of its K slice
// in flight at once, up to PKB pieces -- and reads each x fragment from LDS right before the MFMA
// that uses it.  grid (ceil(nCblk/4), KS); LDS row stride padded by 16 bytes so that the 16 rows a
// fragment read touches fall into different banks.
template <int NB, int PKB>
__global__ __launch_bounds__(256) void project_mfma_shared(const half8 *__restrict__ blob,
                                                           const half_t *__restrict__ x,
                                                           float *__restrict__ part, int B, int D,
                                                           int nCblk, int nKblk, int kb_per, int Bpad,
                                                           int Cpad, FastDiv by_ppr) {
  extern __shared__ uint4 xs[];                       // [NB*16 rows][kb_per*4 + 1] 16-byte pieces
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int ks = blockIdx.y;
  const int cblk_raw = blockIdx.x * 4 + w;
  const bool live = cblk_raw < nCblk;                 // a surplus wave still helps staging x
  const int cblk = min(cblk_raw, nCblk - 1);
  const int n = lane & 15, kg = lane >> 4;
  const int kb0 = ks * kb_per, kb1 = min(nKblk, kb0 + kb_per);
  const int nkb = kb1 - kb0;
  // x rows of the slice: loaded first, because they are needed first -- a wave's loads return in the
  // order it issued them -- then the weight pieces of the whole K slice.  (Rows past the last read the
  // last row, which only reaches rows of the result that are not written; pieces past a short last slice
  // read its last piece, which no product takes.)
  const int ppr = kb_per * 4, stride = ppr + 1;       // 16-byte pieces per row, padded stride
  const int pieces = NB * 16 * ppr;
  constexpr int XPT = NB * 16 * PKB * 4 / 256;         // x pieces per thread at most
  uint4 xv[XPT];
  int at[XPT];                                        // where the piece goes in xs
#pragma unroll
  for (int u = 0; u < XPT; ++u) {
    const int p = threadIdx.x + u * 256;
    const int row = by_ppr.div(p), c = p - row * ppr;
    at[u] = row * stride + c;
    xv[u] = *reinterpret_cast<const uint4 *>(x + (long)min(row, B - 1) * D + (long)kb0 * 32 + min(c, nkb * 4 - 1) * 8);
  }
  half8 a[PKB];
  const half8 *wp = blob + ((long)cblk * nKblk + kb0) * 64 + lane;
#pragma unroll
  for (int t = 0; t < PKB; ++t) a[t] = wp[(long)min(t, nkb - 1) * 64];
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < XPT; ++u) {
    keep_loaded(xv[u]);
    if ((int)threadIdx.x + u * 256 < pieces) xs[at[u]] = xv[u];
  }
  __syncthreads();
  if (!live) return;
  floatx4 acc[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) acc[i] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < PKB; ++t) {
    keep_loaded(a[t]);
    if (t < nkb) {
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const uint4 raw = xs[(i * 16 + n) * stride + t * 4 + kg];
        acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[t], *reinterpret_cast<const half8 *>(&raw), acc[i], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int row = i * 16 + n;
    if (row < B) {
      float *o = part + ((long)ks * Bpad + row) * Cpad + cblk * 16 + kg * 4;
      *reinterpret_cast<floatx4 *>(o) = acc[i];
    }
  }
}

// One thread per output column, NR batch rows per pass, K rows [ks*kb_per, ...).  Weight-read bound on
// paper; on the small shapes that come here it is a chain of round trips, so the weight elements of U rows
// of K are in flight before the first is used, and only the batch rows that exist are multiplied (NR, a
// power of two up to 16).  The x entries are wave-uniform: scalar loads.  (256 x 76 float32 weight, one
// sequence: 2.6 us, against 6.7 us with one row of K after another and 16 batch rows always.)
template <typename T, int NR>
__global__ __launch_bounds__(64) void project_fma(const T *__restrict__ blob, const T *__restrict__ x,
                                                  float *__restrict__ part, int B, int D, int kb_per,
                                                  int Bpad, int Cpad) {
  constexpr int U = 16;
  const int c = blockIdx.x * 64 + threadIdx.x;
  const int ks = blockIdx.y;
  const int n0 = blockIdx.z * NR;
  if (c >= Cpad) return;
  const int k0 = ks * kb_per, k1 = min(D, k0 + kb_per);
  float acc[NR];
#pragma unroll
  for (int i = 0; i < NR; ++i) acc[i] = 0.f;
  const T *xr[NR];                        // (rows past the last read the last row; their sums are not written)
#pragma unroll
  for (int i = 0; i < NR; ++i) xr[i] = x + (long)min(n0 + i, B - 1) * D;
  for (int k = k0; k < k1; k += U) {
    T wv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) wv[u] = blob[(long)min(k + u, k1 - 1) * Cpad + c];
    if (k + U <= k1) {
#pragma unroll
      for (int i = 0; i < NR; ++i)
#pragma unroll
        for (int u = 0; u < U; ++u) acc[i] = fmaf((float)xr[i][k + u], (float)wv[u], acc[i]);
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (k + u < k1) {
#pragma unroll
          for (int i = 0; i < NR; ++i) acc[i] = fmaf((float)xr[i][k + u], (float)wv[u], acc[i]);
        }
    }
  }
#pragma unroll
  for (int i = 0; i < NR; ++i)
    if (n0 + i < B) part[((long)ks * Bpad + n0 + i) * Cpad + c] = acc[i];
}

// ---- index-only partial weight ------------------------------------------------------------------
// Section 6.2 "Memory Consumption": instead of a second copy of the kept columns, only their
// indices are stored and the columns are taken from the full (skewed) query weight, which the
// model keeps on the GPU anyway.  Picking 2-byte columns out of a row-major matrix touches nearly
// every 64-byte line of it, so the kernel reads the rows of a head whole, with 16-byte loads, and
// multiplies all d columns (fp32 FMAs: B*D*D of them, below the time of the D*D read for B <= 16);
// the kept columns are picked from the result.
// Workgroup (h, ks, batch block): 4 waves; a wave-wide load covers 64/LPRp rows of the head's
// d-column span (LPR = 16-byte pieces per row, LPRp = LPR rounded up to a power of two).  The
// NBR batch rows of x for the K chunk are staged in LDS as float.  The sums over a wave's rows are
// folded with a butterfly, the four waves are added in wave order, and the split-K partial sums go
// to part[ks][row][h*r + j], the layout the scan and the finalisation read.
template <typename T, int NBR>
__global__ __launch_bounds__(256) void project_columns(const T *__restrict__ W, const T *__restrict__ x,
                                                       const int32_t *__restrict__ idx,
                                                       float *__restrict__ part, int B, int D, int d,
                                                       int r, int LPR, int LPRp, int k_per, int Bpad,
                                                       int Cpad) {
  constexpr int TPL = Elem<T>::TPL;
  constexpr int KC = 512;                  // K rows staged per chunk
  constexpr int U = NBR <= 8 ? 8 : 4;      // loads in flight per lane
  typedef typename Elem<T>::vec vec;
  __shared__ float xs[NBR * KC];
  __shared__ float red[NBR * 512];
  const int h = blockIdx.x, ks = blockIdx.y, n0 = blockIdx.z * NBR;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int RPW = 64 / LPRp;
  const int sub = lane / LPRp, li = lane % LPRp;
  const bool active = li < LPR;
  const int k0 = ks * k_per, k1 = min(D, k0 + k_per);
  float acc[NBR][TPL];
#pragma unroll
  for (int b = 0; b < NBR; ++b)
#pragma unroll
    for (int e = 0; e < TPL; ++e) acc[b][e] = 0.f;
  const T *wcol = W + (long)h * d + (active ? li : 0) * TPL;
  for (int kc = k0; kc < k1; kc += KC) {
    const int kn = min(KC, k1 - kc);
    __syncthreads();
    for (int b = 0; b < NBR; ++b) {
      const int row = n0 + b;
      for (int kk = tid; kk < kn; kk += 256)
        xs[b * KC + kk] = row < B ? (float)x[(long)row * D + kc + kk] : 0.f;
    }
    __syncthreads();
    const int steps = (kn + 4 * RPW - 1) / (4 * RPW);
    for (int s0 = 0; s0 < steps; s0 += U) {
      vec v[U];
      int kk[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = ((s0 + u) * 4 + w) * RPW + sub;
        const bool ok = active && k < kn;
        kk[u] = min(k, kn - 1);
        vec z = {};
        v[u] = ok ? *reinterpret_cast<const vec *>(wcol + (long)(kc + kk[u]) * D) : z;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float wf[TPL];
#pragma unroll
        for (int e = 0; e < TPL; ++e) wf[e] = (float)v[u][e];
#pragma unroll
        for (int b = 0; b < NBR; ++b) {
          const float xv = xs[b * KC + kk[u]];
#pragma unroll
          for (int e = 0; e < TPL; ++e) acc[b][e] = fmaf(xv, wf[e], acc[b][e]);
        }
      }
    }
  }
  // rows of one wave
  for (int o = LPRp; o < 64; o <<= 1) {
#pragma unroll
    for (int b = 0; b < NBR; ++b)
#pragma unroll
      for (int e = 0; e < TPL; ++e) acc[b][e] += __shfl_xor(acc[b][e], o, 64);
  }
  // the four waves, in wave order
  for (int ww = 0; ww < 4; ++ww) {
    if (w == ww && sub == 0 && active) {
#pragma unroll
      for (int b = 0; b < NBR; ++b)
#pragma unroll
        for (int e = 0; e < TPL; ++e) {
          const int at = b * 512 + li * TPL + e;
          red[at] = (ww == 0 ? 0.f : red[at]) + acc[b][e];
        }
    }
    __syncthreads();
  }
  for (int i = tid; i < NBR * r; i += 256) {
    const int b = i / r, j = i % r;
    const int row = n0 + b;
    const int col = min(max(idx[h * r + j], 0), d - 1);
    if (row < B) part[((long)ks * Bpad + row) * Cpad + h * r + j] = red[b * 512 + col];
  }
}

// The same for half precision on the matrix cores (D a multiple of 128): workgroup (128-column
// block, ks, batch blocks).  Lane (n = lane%16, kg = lane/16) of a wave loads, for 8 consecutive
// rows k, the 16 bytes holding columns 8n .. 8n+7 of the block (16 lanes cover one 256-byte row
// piece, a wave-wide step covers 32 rows), turns its 8x8 block of halves around in registers so
// that each of its 8 columns has 8 consecutive k, and issues 8 MFMAs 16x16x32 per batch block:
// MFMA j multiplies columns {8m + j} (A operand, m = lane%16) with the x fragment (B operand, 16
// batch rows).  Result register v of lane l in MFMA j: column 8*(4*(l/16) + v) + j, batch row l%16.
// The four waves take every fourth step; their sums are added in wave order through LDS.
template <int NB>
__global__ __launch_bounds__(256) void project_columns_mfma(const half_t *__restrict__ W,
                                                            const half_t *__restrict__ x,
                                                            const int32_t *__restrict__ idx,
                                                            float *__restrict__ part, int B, int D,
                                                            int H, int d, int r, int k_per, int Bpad,
                                                            int Cpad) {
  constexpr int RS = 129;                   // row stride of the LDS result tile (floats)
  __shared__ float red[NB * 16 * RS];
  const int cb = blockIdx.x, ks = blockIdx.y, nb0 = blockIdx.z * NB;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int n = lane & 15, kg = lane >> 4;
  const int k0 = ks * k_per, k1 = min(D, k0 + k_per);      // both multiples of 32
  floatx4 acc[NB][8];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  const half_t *wp = W + (long)cb * 128 + n * 8;
  // two steps per pass: 16 row loads of a lane are in flight before the first MFMA
  for (int kb = k0 + w * 32; kb < k1; kb += 256) {
    half8 rows[2][8], xf[2][NB];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      // (a step past the slice reads its last 32 rows again and is not multiplied; lanes of a batch row
      // past the last read the last row, which only reaches rows of the result that are not written)
      const int kt = min(kb + t * 128, k1 - 32) + kg * 8;
#pragma unroll
      for (int e = 0; e < 8; ++e) rows[t][e] = *reinterpret_cast<const half8 *>(wp + (long)(kt + e) * D);
#pragma unroll
      for (int i = 0; i < NB; ++i)
        xf[t][i] = *reinterpret_cast<const half8 *>(x + (long)min((nb0 + i) * 16 + n, B - 1) * D + kt);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
#pragma unroll
      for (int e = 0; e < 8; ++e) keep_loaded(rows[t][e]);
#pragma unroll
      for (int i = 0; i < NB; ++i) keep_loaded(xf[t][i]);
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      if (kb + t * 128 < k1) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          half8 a;
#pragma unroll
          for (int e = 0; e < 8; ++e) a[e] = rows[t][e][j];
#pragma unroll
          for (int i = 0; i < NB; ++i)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, xf[t][i], acc[i][j], 0, 0, 0);
        }
      }
    }
  }
  for (int ww = 0; ww < 4; ++ww) {
    if (w == ww) {
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int at = (i * 16 + n) * RS + 8 * (4 * kg + v) + j;
            red[at] = (ww == 0 ? 0.f : red[at]) + acc[i][j][v];
          }
    }
    __syncthreads();
  }
  // kept columns that fall into this block, for the heads that overlap it
  const int c_lo = cb * 128;
  const int h_lo = c_lo / d, h_hi = min(H - 1, (c_lo + 127) / d);
  for (int i = h_lo * r + tid; i < (h_hi + 1) * r; i += 256) {
    const int col = (i / r) * d + min(max(idx[i], 0), d - 1) - c_lo;
    if (col < 0 || col >= 128) continue;
    for (int b = 0; b < NB * 16; ++b) {
      const int row = nb0 * 16 + b;
      if (row < B) part[((long)ks * Bpad + row) * Cpad + i] = red[b * RS + col];
    }
  }
}

// ---- finalisation -------------------------------------------------------------------------------
// folded: q_p[b,h,j] = bias[h*r+j] + sum_s part[s][b][h*r+j]
// rope:   q[c] = bias[h*d+c] + sum_s part[s][b][h*d+c]; rotate pairs (c, c+d/2) by
//         pos[b]*theta^(-2c/d) (angle in double: positions reach 1e5 where float loses the phase);
//         q_p[b,h,k] = sum_c q_rot[c] * A_p[h][c][k]
// (Section 4.3 "Decoding Stage" for models whose skew cannot be folded into W_Q.)
// finalize_folded takes a sequence's H*r columns in a row (5760 heads of 12 columns: one workgroup a head 6.5 us, so
// 4.2).  finalize_query is a chain of dependent steps: 5.6 us for 160 heads of 128 columns while the compiler
// put conditions around its loads (one round trip after another), 4.3 us with every load of a thread in flight.
// KSM, PF: partial sums of a column and rows of A_p that a thread has in flight.  Loads past what there is, clamped
// to the last, cost nothing while latency sets the time and something where the chip is full, so a launch
// takes the smallest that fit: KS sums of 2, 4, 8, 12 or IG_KS_MAX, a share of the rows (d r / 256) of 8, 16 or 24.
// (32 heads of 64 columns, 96 sequences, r = 6: 15.1 -> 8.2 us; 16 heads of 128, 80 sequences, r = 128: 13.8 ->
// 9.0 us with the waves that have no pair to rotate out of the double arithmetic and 8 of the further rows at a time.)
template <int KSM>
__global__ __launch_bounds__(64) void finalize_folded(const float *__restrict__ part,
                                                       const float *__restrict__ bias,
                                                       float *__restrict__ q_p, int C, int KS,
                                                       long ks_stride, int Cpad, FastDiv by_blocks) {
  // (one wave a workgroup, so that few rows reach every compute unit: rows of 1024 columns, 80 of them, with four
  // waves 2 us more)
  const int b = by_blocks.div(blockIdx.x), c = by_blocks.mod(blockIdx.x) * 64 + threadIdx.x;
  if (c >= C) return;
  // split-K partial sums: all loads of a column issued together, added in a fixed order
  const float *p = part + (long)b * Cpad + c;
  float v[KSM];
#pragma unroll
  for (int s = 0; s < KSM; ++s) v[s] = p[(long)min(s, KS - 1) * ks_stride];
  q_p[(long)b * C + c] = add_partials<KSM>(bias ? bias[c] : 0.f, v, KS);
}
template <int KSM, int PF>
__global__ __launch_bounds__(256) void finalize_query(const float *__restrict__ part,
                                                      const float *__restrict__ bias,
                                                      const float *__restrict__ A_p,
                                                      const int32_t *__restrict__ pos,
                                                      float *__restrict__ q_p, int H, int d, int r,
                                                      int KS, long ks_stride, int Cpad,
                                                      double freq_step /* -(2/d) log2(theta) */,
                                                      FastDiv by_H, FastDiv by_r, int G, int per) {
  __shared__ float q[512];
  __shared__ float qr[512];
  __shared__ float psum[256];
  const int bh = blockIdx.x, b = by_H.div(bh), h = bh - b * H;
  const int t = threadIdx.x;
  // Rotary model.  The block is one chain of dependent steps, so everything it reads is put in
  // flight before the first step: the partial sums of its (up to two) columns, the position, and
  // the thread's rows of A_p, which do not depend on the query at all.
  // (Addresses are clamped and surplus values dropped where they are used: a condition around a load
  // becomes a branch, and loads behind branches were issued one round trip after another.  The second
  // column of a thread exists for d > 256 only.)
  float v[KSM], v2[KSM], bs, bs2 = 0.f;
  {
    const float *p = part + (long)b * Cpad + (long)h * d;
    const int c = min(t, d - 1);
#pragma unroll
    for (int s = 0; s < KSM; ++s) v[s] = p[(long)min(s, KS - 1) * ks_stride + c];
    bs = *(bias ? bias + h * d + c : p);
    if (d > 256) {
      const int c2 = min(t + 256, d - 1);
#pragma unroll
      for (int s = 0; s < KSM; ++s) v2[s] = p[(long)min(s, KS - 1) * ks_stride + c2];
      if (bias) bs2 = bias[h * d + c2];
    }
  }
  const int position = pos[b];
  // q_p[k] = sum_c qr[c] * A_p[h][c][k]: the threads are G groups of r; group g sums its share of
  // the rows c for output k (reads of A_p coalesce over k), then the groups are added in order
  // (G = 256 / r, r <= 256; per = ceil(d / G) rows each)
  const int g = by_r.div(t), k = t - g * r;
  const int c0 = g < G ? min(d, g * per) : d, c1 = g < G ? min(d, (g + 1) * per) : d;
  const float *ap = A_p + (long)h * d * r + k;
  float apf[PF];
#pragma unroll
  for (int i = 0; i < PF; ++i) apf[i] = ap[(long)min(c0 + i, d - 1) * r];
  __builtin_amdgcn_sched_barrier(0);
  // the angle's frequency depends on nothing that is loaded (d <= 512: one pair a thread; waves without a pair
  // skip the double arithmetic, which is most of the block's work where the chip is full)
  const int half = d / 2;
  double freq = 0.0, sn = 0.0, cs = 1.0;
  if (t < half) freq = exp2((double)t * freq_step);
  {
    const float acc = add_partials<KSM>(bias ? bs : 0.f, v, KS);
    if (t < d) q[t] = acc;
  }
  if (d > 256) {
    const float acc = add_partials<KSM>(bs2, v2, KS);
    if (t + 256 < d) q[t + 256] = acc;
  }
  if (t < half) rope_sincos((double)position * freq, &sn, &cs);
  __syncthreads();
  if (t < half) {
    float a = q[t], bb = q[t + half];
    qr[t] = (float)((double)a * cs - (double)bb * sn);
    qr[t + half] = (float)((double)bb * cs + (double)a * sn);
  }
  __syncthreads();
  float acc = 0.f;
#pragma unroll
  for (int i = 0; i < PF; ++i) {               // (a condition around the LDS read would be a branch)
    const float next = fmaf(qr[min(c0 + i, d - 1)], apf[i], acc);
    acc = c0 + i < c1 ? next : acc;
  }
  for (int c = c0 + PF; c < c1; c += 8) {      // (heads kept nearly whole: 8 more rows at a time)
    float more[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) more[i] = ap[(long)min(c + i, d - 1) * r];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float next = fmaf(qr[min(c + i, d - 1)], more[i], acc);
      acc = c + i < c1 ? next : acc;
    }
  }
  psum[t] = acc;
  __syncthreads();
  if (t < r) {
    float tot = 0.f;
    for (int gg = 0; gg < G; ++gg) tot += psum[gg * r + t];
    q_p[(long)bh * r + t] = tot;
  }
}

}  // namespace

int ig_launch_wq_build(ig_ctx *ctx, const ig_desc *d, const ProjGeom &g, const void *Wq,
                       const int32_t *idx, void *wq, hipStream_t s) {
  const int D = d->H * d->d;
  const int32_t *ix = d->rope ? nullptr : idx;
  if (g.mfma) {
    long total = (long)g.nCblk * g.nKblk * 64;
    auto k = wq_build_mfma;
    IG_LAUNCH(ctx, IG_K_BUILD, k, dim3((unsigned)((total + 255) / 256)), dim3(256), s,
              (const half_t *)Wq, ix, (half8 *)wq, D, (int)d->d, (int)d->r, g.C, g.nCblk, g.nKblk);
  } else if (d->dtype == IG_F16) {
    long total = (long)D * g.Cpad;
    auto k = wq_build_plain<half_t>;
    IG_LAUNCH(ctx, IG_K_BUILD, k, dim3((unsigned)((total + 255) / 256)), dim3(256), s,
              (const half_t *)Wq, ix, (half_t *)wq, D, (int)d->d, (int)d->r, g.C, g.Cpad);
  } else {
    long total = (long)D * g.Cpad;
    auto k = wq_build_plain<float>;
    IG_LAUNCH(ctx, IG_K_BUILD, k, dim3((unsigned)((total + 255) / 256)), dim3(256), s,
              (const float *)Wq, ix, (float *)wq, D, (int)d->d, (int)d->r, g.C, g.Cpad);
  }
  return IG_OK;
}

int ig_launch_project(ig_ctx *ctx, const ig_desc *d, const ProjGeom &g, const void *x,
                      const void *wq, float *part, hipStream_t s) {
  const int D = d->H * d->d;
  if (g.mfma) {
    const unsigned cols = (unsigned)((g.nCblk + 3) / 4);
    dim3 block(256);
    if (g.NBtot == 1) {
      auto k = project_mfma<1, 8>;
      IG_LAUNCH(ctx, IG_K_PROJECT, k, dim3(cols, g.KS), block, s, (const half8 *)wq, (const half_t *)x,
                part, (int)d->B, D, g.nCblk, g.nKblk, g.kb_per, g.Bpad, g.Cpad);
    } else if (g.NBtot == 2 && g.kb_per <= 16) {
      // 17..32 batch rows: x fragments through LDS, a wave's whole K slice of weights in flight
      auto k = project_mfma_shared<2, 16>;
      const size_t lds = (size_t)32 * (g.kb_per * 4 + 1) * 16;
      const dim3 grid(cols, (unsigned)g.KS);
      IG_LAUNCH_LDS(ctx, IG_K_PROJECT, k, grid, block, lds, s, (const half8 *)wq, (const half_t *)x, part,
                    (int)d->B, D, g.nCblk, g.nKblk, g.kb_per, g.Bpad, g.Cpad, ig_fast_div(g.kb_per * 4));
    } else if (g.NBtot == 2) {
      auto k = project_mfma<2, 6>;
      IG_LAUNCH(ctx, IG_K_PROJECT, k, dim3(cols, g.KS), block, s, (const half8 *)wq, (const half_t *)x,
                part, (int)d->B, D, g.nCblk, g.nKblk, g.kb_per, g.Bpad, g.Cpad);
    } else {
      // groups of up to 4 blocks of 16 batch rows, as even as they go: a block past the batch is read (its last
      // row again) and multiplied like any other (5120 columns, 37 rows: 24.4 us as 4 blocks, 22.8 as 3, 20.4 with
      // its K slice of 10 taken by 2)
      const int groups = (g.NBtot + 3) / 4;
      // K blocks at a time: as many of 4, 3 or 2 as leave the fewest loads past the slice, which many rows feel
      int kb = 4;
      for (int n = 3; n >= 2; --n)
        if ((g.kb_per + n - 1) / n * n < (g.kb_per + kb - 1) / kb * kb) kb = n;
      auto pick = [&](auto k4, auto k3, auto k2) { return kb == 4 ? k4 : (kb == 3 ? k3 : k2); };
      auto k = (g.NBtot + groups - 1) / groups == 3 ? pick(project_mfma<3, 4>, project_mfma<3, 3>, project_mfma<3, 2>)
                                                    : pick(project_mfma<4, 4>, project_mfma<4, 3>, project_mfma<4, 2>);
      IG_LAUNCH(ctx, IG_K_PROJECT, k, dim3(cols, g.KS, (unsigned)groups), block, s, (const half8 *)wq,
                (const half_t *)x, part, (int)d->B, D, g.nCblk, g.nKblk, g.kb_per, g.Bpad, g.Cpad);
    }
  } else {
    const int nr = d->B > 8 ? 16 : (d->B > 4 ? 8 : (d->B > 2 ? 4 : d->B));
    dim3 grid((g.Cpad + 63) / 64, g.KS, (d->B + nr - 1) / nr), block(64);
#define FMA_CASE(T, NR)                                                                            \
  if (nr == NR) {                                                                                  \
    auto k = project_fma<T, NR>;                                                                   \
    IG_LAUNCH(ctx, IG_K_PROJECT, k, grid, block, s, (const T *)wq, (const T *)x, part, (int)d->B,  \
              D, g.kb_per, g.Bpad, g.Cpad);                                                        \
  }
    if (d->dtype == IG_F16) {
      FMA_CASE(half_t, 1) FMA_CASE(half_t, 2) FMA_CASE(half_t, 4) FMA_CASE(half_t, 8) FMA_CASE(half_t, 16)
    } else {
      FMA_CASE(float, 1) FMA_CASE(float, 2) FMA_CASE(float, 4) FMA_CASE(float, 8) FMA_CASE(float, 16)
    }
#undef FMA_CASE
  }
  return IG_OK;
}

// Split of the index-only projection: enough workgroups for two per compute unit.  Half precision
// with D a multiple of 128 runs on the matrix cores (column blocks of 128, K slices that are
// multiples of 32, up to 4 batch blocks of 16 per workgroup); everything else on the FMA kernel
// (one head per workgroup, 8 or 16 batch rows).
static bool proj_columns_mfma(const ig_desc *d) { return d->dtype == IG_F16 && (d->H * d->d) % 128 == 0; }

int ig_proj_columns_ks(const ig_desc *d, int *k_per) {
  const int D = d->H * d->d;
  int wgs, unit;
  if (proj_columns_mfma(d)) {
    const int nbtot = (d->B + 15) / 16;
    wgs = (D / 128) * ((nbtot + 3) / 4);
    unit = 32;
  } else {
    const int nbr = d->B <= 8 ? 8 : 16;
    wgs = d->H * ((d->B + nbr - 1) / nbr);
    unit = 1;
  }
  const int units = D / unit;
  int ks = (512 + wgs - 1) / wgs;
  if (ks > IG_KS_MAX) ks = IG_KS_MAX;
  if (ks > units) ks = units;
  if (ks < 1) ks = 1;
  *k_per = (units + ks - 1) / ks * unit;
  return (D + *k_per - 1) / *k_per;
}

int ig_launch_project_columns(ig_ctx *ctx, const ig_desc *d, const ProjGeom &g, const void *x,
                              const void *W, const int32_t *idx, float *part, hipStream_t s) {
  const int D = d->H * d->d;
  int k_per = 0;
  const int KS = ig_proj_columns_ks(d, &k_per);
  if (proj_columns_mfma(d)) {
    const int nbtot = (d->B + 15) / 16;
    const int groups = (nbtot + 3) / 4, nb = (nbtot + groups - 1) / groups;      // (as in ig_launch_project)
    dim3 grid(D / 128, KS, groups), block(256);
#define PM_CASE(NB)                                                                                \
  {                                                                                                \
    auto k = project_columns_mfma<NB>;                                                             \
    IG_LAUNCH(ctx, IG_K_PROJECT, k, grid, block, s, (const half_t *)W, (const half_t *)x, idx,     \
              part, (int)d->B, D, (int)d->H, (int)d->d, (int)d->r, k_per, g.Bpad, g.Cpad);         \
    return IG_OK;                                                                                  \
  }
    if (nb == 1) PM_CASE(1)
    if (nb == 2) PM_CASE(2)
    if (nb == 3) PM_CASE(3)
    PM_CASE(4)
#undef PM_CASE
  }
  const int row_bytes = d->d * ig_elem_bytes(d->dtype);
  if (row_bytes % 16 || row_bytes / 16 > 64 || d->d > 512)
    return ig_fail(ctx, IG_ESHAPE, "index-only projection: d = %d needs 16-byte rows of at most 1 KiB", d->d);
  const int LPR = row_bytes / 16;
  int LPRp = 1;
  while (LPRp < LPR) LPRp <<= 1;
  const int nbr = d->B <= 8 ? 8 : 16;
  dim3 grid(d->H, KS, (d->B + nbr - 1) / nbr), block(256);
#define PC_CASE(T, NBR)                                                                            \
  {                                                                                                \
    auto k = project_columns<T, NBR>;                                                              \
    IG_LAUNCH(ctx, IG_K_PROJECT, k, grid, block, s, (const T *)W, (const T *)x, idx, part,         \
              (int)d->B, D, (int)d->d, (int)d->r, LPR, LPRp, k_per, g.Bpad, g.Cpad);               \
    return IG_OK;                                                                                  \
  }
  if (d->dtype == IG_F16) {
    if (nbr == 8) PC_CASE(half_t, 8)
    PC_CASE(half_t, 16)
  }
  if (nbr == 8) PC_CASE(float, 8)
  PC_CASE(float, 16)
#undef PC_CASE
}

int ig_launch_finalize(ig_ctx *ctx, const ig_desc *d, const ProjGeom &g, const float *part,
                       const float *bias, const float *A_p, const int32_t *pos, float *q_p,
                       hipStream_t s) {
  if (d->rope && d->d > 512) return ig_fail(ctx, IG_ESHAPE, "rope: d = %d exceeds 512", d->d);
#define BY_KS(K)                                                                                   \
  (g.KS <= 2 ? K(2) : (g.KS <= 4 ? K(4) : (g.KS <= 8 ? K(8) : (g.KS <= 12 ? K(12) : K(IG_KS_MAX)))))
  const long ks_stride = (long)g.Bpad * g.Cpad;
  if (!d->rope) {
    const int C = d->H * d->r;
#define FOLDED(KSM) finalize_folded<KSM>
    auto k = BY_KS(FOLDED);
#undef FOLDED
    const int blocks = (C + 63) / 64;
    IG_LAUNCH(ctx, IG_K_FINALIZE, k, dim3((unsigned)d->B * blocks), dim3(64), s, part, bias, q_p, C, g.KS, ks_stride,
              g.Cpad, ig_fast_div(blocks));
    return IG_OK;
  }
  const int G = 256 / d->r, per = (d->d + G - 1) / G;
  auto pick = [&](auto k8, auto k16, auto k24) { return per <= 8 ? k8 : (per <= 16 ? k16 : k24); };
#define QUERY(KSM) pick(finalize_query<KSM, 8>, finalize_query<KSM, 16>, finalize_query<KSM, 24>)
  auto k = BY_KS(QUERY);
#undef QUERY
#undef BY_KS
  IG_LAUNCH(ctx, IG_K_FINALIZE, k, dim3(d->B * d->H), dim3(256), s, part, bias, A_p, pos, q_p,
            (int)d->H, (int)d->d, (int)d->r, g.KS, ks_stride, g.Cpad,
            -2.0 / (double)d->d * log2((double)d->rope_theta), ig_fast_div(d->H), ig_fast_div(d->r), G, per);
  return IG_OK;
}
