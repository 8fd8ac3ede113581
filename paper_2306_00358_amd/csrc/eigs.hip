// Leading eigenpairs of the environment matrix M (n x n, symmetric positive
// semi-definite) in FP64 by block subspace iteration with Rayleigh-Ritz.
//
// The projector of one coarse-graining step needs only the D' leading
// eigenvectors of M (plus the next eigenvalue for the cut gap), while a full
// dense eigensolver spends most of its time in a memory-bound
// tridiagonalisation of all n = D^2 rows.  The environment spectrum decays
// fast, so iterating a block of p > D' vectors converges in a few sweeps at
// the rate lambda_{p+1} / lambda_{D'} per sweep.
//
// One sweep:  Y = V (M - sigma I)  (rows of V are the p basis vectors)
//             V = orth(Y) by shifted Cholesky-QR (Fukaya et al., "Shifted
//             Cholesky QR for computing the QR factorization of
//             ill-conditioned matrices", SIAM J. Sci. Comput. 42 (2020)):
//             G = Y Y^T + s I, G = R^T R, V = R^-T Y; the first two passes
//             factor the diagonally scaled G with s = 11 (n p + p(p+1)) u
//             trace, the third with s = 0.  (When M's spectrum falls to
//             rounding noise within the block -- deep in an ordered phase --
//             one shifted pass leaves a basis too ill-conditioned for an
//             unshifted Cholesky; a second shifted pass brings it within
//             reach, and the third restores orthonormality to rounding.)
//             V = R^-T Y is a blocked triangular solve (k_trsm_rows).
//             Before a check all three passes run.  Between checks V only
//             has to stay a well-conditioned basis of the same span: one
//             pass, then a second that the device reduces to R = I when G is
//             already the identity to 1e-2 -- after the first pass it is
//             typically so to 1e-7..1e-4, except in a solve's first sweep
//             (and once no such check misses, only the first sweep after a
//             check is checked).
// Check:      H = V (V M)^T, H = Z diag(theta) Z^T (Householder reduction to
//             tridiagonal form in one workgroup, k_sytrd_small, then divide
//             and conquer on the tridiagonal in another, k_stedc_small in
//             stedc.hip, and the reflectors applied to its rows,
//             k_backtransform),
//             Ritz vectors X = Z^T V, residuals |(Z^T Y)_i - theta_i X_i|.
// Converged when the residuals of the `need` leading pairs are below
// tol * theta_1; otherwise the sweeps continue from X.  The first check
// comes after q_first sweeps.  On convergence `enough` estimates the fewest
// sweeps that would have met the tolerance: the residual of the slowest
// needed pair shrinks by about theta_min / theta_need per sweep, so a result
// k such factors below tol was k sweeps more than necessary.  The caller
// starts the next solve of the same kind from that estimate plus one, so most
// solves take a single Rayleigh-Ritz without sweeping far past convergence.
// All products are FP64 MFMA GEMMs; the host reads p Ritz values and
// residuals per check.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "internal.h"

namespace hotrg {

typedef double d4 __attribute__((ext_vector_type(4)));

// deterministic start block: splitmix64 of the element index -> [-1, 1)
__global__ void k_seed_block(double* V, long long count, unsigned long long seed) {
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < count;
       e += (long long)gridDim.x * blockDim.x) {
    unsigned long long z = (unsigned long long)e + seed * 0x9E3779B97F4A7C15ULL;
    z += 0x9E3779B97F4A7C15ULL;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
    z ^= z >> 31;
    V[e] = (double)(z >> 11) * (2.0 / 9007199254740992.0) - 1.0;
  }
}

// G (p x p, row-major) -> RinvT = (R^-1)^T where G + s I = R^T R, s =
// shift_rel * trace(G).  One workgroup of 256 threads as a 16 x 16 grid;
// thread (ty, tx) keeps the elements (ty + 16a, tx + 16b), a, b < 8, of the
// working matrix in registers (p <= 128, p a multiple of 16; indices past p
// are clamped, and those registers are never published or stored).
//
// Blocked right-looking Cholesky with blocks of 8 columns: the owners of the
// block's 8 rows (final by then) publish them in LDS; thread c < p then
// factors the 8 x 8 diagonal block itself (the same operations on the same
// data in every such thread) and forms column c of the block rows of R by
// forward substitution, straight into R in LDS; after a second barrier every
// thread applies the rank-8 update to its elements.  The inverse X = R^-1 is
// eliminated from X = I block by block from the bottom the same way: thread c
// back-substitutes column c of the block's rows in place, and every row takes
// the rank-8 update with column j0.. of R (zero below the diagonal, so rows
// at and below the block are left alone; the block's rows then take their
// final values).  Two barriers per block of 8 columns.
//
// R starts as zeros in LDS, so every load below is unconditional: rows and
// columns that are already finished take updates nobody reads again, which
// costs less than the waits a load under a branch would.  X^T leaves through
// LDS for coalesced stores.  *fail is set if a pivot is not positive.
constexpr int kCholThreads = 256;

__device__ __forceinline__ void chol_inv_body(const double* __restrict__ G, int p,
                                              double shift_rel, int scale, double identity_tol,
                                              double* __restrict__ RinvT, int* fail) {
  extern __shared__ double lds[];
  double* R = lds;             // p * p: R (upper, zeros below), later X^T
  double* P = R + p * p;       // 2 x 8 x 128 published rows
  __shared__ int bad;
  __shared__ double dev[kCholThreads];
  __shared__ double dsc[128];  // diag(G)^-1/2 when scaling, else 1
  const int t = threadIdx.x;
  const int tx = t & 15, ty = t >> 4;
  const int pm = p - 1;
  double A[8][8];
#pragma unroll
  for (int a = 0; a < 8; ++a)
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const int i = min(ty + 16 * a, pm), k = min(tx + 16 * b, pm);
      A[a][b] = G[min(i, k) * p + max(i, k)];  // upper part, mirrored
    }
  if (identity_tol > 0.0) {
    // G already the identity to within identity_tol: R^-1 = I
    double d = 0.0;
#pragma unroll
    for (int a = 0; a < 8; ++a)
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        const int i = ty + 16 * a, k = tx + 16 * b;
        if (i < p && k < p) d = fmax(d, fabs(A[a][b] - (i == k ? 1.0 : 0.0)));
      }
    dev[t] = d;
    __syncthreads();
    double mx = 0.0;
    for (int i = 0; i < kCholThreads; ++i) mx = fmax(mx, dev[i]);
    if (mx <= identity_tol) {  // uniform: every thread reduced the same values
      for (int e = t; e < p * p; e += kCholThreads) RinvT[e] = (e / p == e % p) ? 1.0 : 0.0;
      return;
    }
  }
  for (int e = t; e < p * p; e += kCholThreads) R[e] = 0.0;
  // diagonal: the owners publish it
  if (tx == ty) {
#pragma unroll
    for (int a = 0; a < 8; ++a)
      if (ty + 16 * a < p) P[ty + 16 * a] = A[a][a];
  }
  if (t == 0) bad = 0;
  __syncthreads();
  // with `scale`, factor D^-1 G D^-1 (D = diag(G)^1/2) instead of G: the
  // columns' lengths drop out of the conditioning, and the scaling is put
  // back into the rows of R^-1 at the end
  if (t < 128) dsc[t] = (scale && t < p) ? 1.0 / sqrt(P[t]) : 1.0;
  __syncthreads();
  if (scale) {
#pragma unroll
    for (int a = 0; a < 8; ++a) {
      const double dr = dsc[min(ty + 16 * a, pm)];
#pragma unroll
      for (int b = 0; b < 8; ++b) A[a][b] *= dr * dsc[min(tx + 16 * b, pm)];
    }
  }
  // trace (of the matrix factored), every thread sums in the same order
  double tr = 0.0;
  if (scale)
    tr = (double)p;
  else
    for (int i = 0; i < p; ++i) tr += P[i];
  const double shift = shift_rel * tr;
  if (tx == ty) {
#pragma unroll
    for (int a = 0; a < 8; ++a) A[a][a] += shift;
  }
  __syncthreads();  // everyone has read the trace before P is reused

  const int nblk = p >> 3;
  for (int J = 0; J < nblk; ++J) {
    const int j0 = 8 * J, aj = j0 >> 4, tj = j0 & 15;
    double* Pb = P + (J & 1) * 1024;
    if (ty >= tj && ty < tj + 8) {
#pragma unroll
      for (int a = 0; a < 8; ++a)
        if (a == aj) {
#pragma unroll
          for (int b = 0; b < 8; ++b) Pb[(ty - tj) * 128 + tx + 16 * b] = A[a][b];
        }
    }
    __syncthreads();
    if (t < p && t >= j0) {
      // the 8 x 8 diagonal block: L[r][c] (c >= r) becomes R[j0+r][j0+c]
      double L[8][8], inv[8];
#pragma unroll
      for (int r = 0; r < 8; ++r)
#pragma unroll
        for (int c = r; c < 8; ++c) L[r][c] = Pb[r * 128 + j0 + c];
      bool ok = true;
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const double d = L[r][r];
        ok = ok && d > 0.0;
        // 1 / sqrt(d) from v_rsq_f64 and two Newton steps; sqrt(d) = d / sqrt(d)
        const double dd = d > 0.0 ? d : 1.0;
        double y = __builtin_amdgcn_rsq(dd);
        y = fma(y, fma(-0.5 * dd * y, y, 0.5), y);
        y = fma(y, fma(-0.5 * dd * y, y, 0.5), y);
        inv[r] = y;
        L[r][r] = dd * y;
#pragma unroll
        for (int c = r + 1; c < 8; ++c) L[r][c] *= inv[r];
#pragma unroll
        for (int r2 = r + 1; r2 < 8; ++r2)
#pragma unroll
          for (int c = r2; c < 8; ++c) L[r2][c] -= L[r][r2] * L[r][c];
      }
      if (!ok) bad = 1;
      if (t >= j0 + 8) {
        double v[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          double w = Pb[r * 128 + t];
#pragma unroll
          for (int m = 0; m < r; ++m) w -= L[m][r] * v[m];
          v[r] = w * inv[r];
          R[(j0 + r) * p + t] = v[r];
        }
      } else {
        const int cc = t - j0;  // column inside the block
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          double v = 0.0;
#pragma unroll
          for (int c = r; c < 8; ++c) v = cc == c ? L[r][c] : v;
          R[(j0 + r) * p + t] = v;
        }
      }
    }
    __syncthreads();
    if (bad) {
      if (t == 0) *fail = 1;
      return;  // uniform: every thread read the same flag after the barrier
    }
    // register rows / columns whose indices all lie before j0 + 8 are
    // finished: skip them (a uniform test)
    double Ri[8][8];
#pragma unroll
    for (int a = 0; a < 8; ++a) {
      if (16 * a + 15 < j0 + 8) continue;
      const int i = min(ty + 16 * a, pm);
#pragma unroll
      for (int r = 0; r < 8; ++r) Ri[a][r] = R[(j0 + r) * p + i];
    }
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      if (16 * b + 15 < j0 + 8) continue;
      const int k = min(tx + 16 * b, pm);
      double Rk[8];
#pragma unroll
      for (int r = 0; r < 8; ++r) Rk[r] = R[(j0 + r) * p + k];
#pragma unroll
      for (int a = 0; a < 8; ++a) {
        if (16 * a + 15 < j0 + 8) continue;
        double v = A[a][b];
#pragma unroll
        for (int r = 0; r < 8; ++r) v -= Ri[a][r] * Rk[r];
        A[a][b] = v;
      }
    }
  }
  // X = I in registers
#pragma unroll
  for (int a = 0; a < 8; ++a)
#pragma unroll
    for (int b = 0; b < 8; ++b) A[a][b] = (ty + 16 * a == tx + 16 * b) ? 1.0 : 0.0;
  __syncthreads();  // the last reads of P and R rows are done
  for (int J = nblk - 1; J >= 0; --J) {
    const int j0 = 8 * J, aj = j0 >> 4, tj = j0 & 15;
    double* Pb = P + (J & 1) * 1024;
    if (ty >= tj && ty < tj + 8) {
#pragma unroll
      for (int a = 0; a < 8; ++a)
        if (a == aj) {
#pragma unroll
          for (int b = 0; b < 8; ++b) Pb[(ty - tj) * 128 + tx + 16 * b] = A[a][b];
        }
    }
    __syncthreads();
    if (t < p) {  // column t of the block rows, back substitution in place
      double L[8][8], inv[8], x[8];
#pragma unroll
      for (int r = 0; r < 8; ++r) {
#pragma unroll
        for (int c = r; c < 8; ++c) L[r][c] = R[(j0 + r) * p + j0 + c];
        inv[r] = 1.0 / L[r][r];
        x[r] = Pb[r * 128 + t];
      }
#pragma unroll
      for (int r = 7; r >= 0; --r) {
        double v = x[r];
#pragma unroll
        for (int m = r + 1; m < 8; ++m) v -= L[r][m] * x[m];
        x[r] = v * inv[r];
        Pb[r * 128 + t] = x[r];
      }
    }
    __syncthreads();
    // X is upper triangular: the block's rows vanish before column j0, and
    // rows from j0 + 8 on are final; skip those register groups (uniform)
    double Xb[8][8];  // the block's final rows at the thread's own columns
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      if (16 * b + 15 < j0) continue;
#pragma unroll
      for (int r = 0; r < 8; ++r) Xb[b][r] = Pb[r * 128 + tx + 16 * b];
    }
#pragma unroll
    for (int a = 0; a < 8; ++a) {
      if (16 * a >= j0 + 8) continue;
      const int i = ty + 16 * a;
      const int ic = min(i, pm);
      double Rr[8];  // R[i][j0 + r]: zero for rows at or below the block
#pragma unroll
      for (int r = 0; r < 8; ++r) Rr[r] = R[ic * p + j0 + r];
      const bool in_blk = i >= j0 && i < j0 + 8;
      const int rb = i - j0;
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        if (16 * b + 15 < j0) continue;
        double v = A[a][b];
#pragma unroll
        for (int r = 0; r < 8; ++r) v -= Rr[r] * Xb[b][r];
        double xr = Xb[b][0];
#pragma unroll
        for (int r = 1; r < 8; ++r) xr = rb == r ? Xb[b][r] : xr;
        A[a][b] = in_blk ? xr : v;
      }
    }
  }
  __syncthreads();  // all reads of R are done: reuse it for X^T
#pragma unroll
  for (int a = 0; a < 8; ++a)
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const int i = ty + 16 * a, k = tx + 16 * b;
      // with scaling R = R^ D, so row i of R^-1 = D^-1 R^^-1 carries G_ii^-1/2
      if (i < p && k < p) R[k * p + i] = A[a][b] * dsc[i];
    }
  __syncthreads();
  for (int e = t; e < p * p; e += kCholThreads) RinvT[e] = R[e];
}


// Factor-only Cholesky of a sweep's Gram matrix (Q = R^-T D^-1 Y then comes
// from k_trsm_rows): R with R^T R = D^-1 G D^-1 + s I (`scale`; D = diag(G)^1/2) or
// G + s I, s = shift_rel * trace of the matrix factored, into Rout (p x p
// row-major, zeros below the diagonal) and D^-1 (ones without `scale`) into
// Rout + p * p; with identity_tol > 0 and G the identity to within it, R = I.
// One workgroup of GW x GW threads (GW = 32 for p <= 128, 16 for p <= 64:
// the same register tiles, and barriers over 4 waves instead of 16); thread
// (ty, tx) keeps the elements (ty + GW a, tx + GW b), a, b < 4, in registers
// (p a multiple of 16; indices past p are clamped and never published).  Blocks of 8
// columns: the owners of the block's 8 rows publish them in LDS; the first
// wave factors the 8 x 8 diagonal block, one column per lane, the values of
// other columns by readlane (1/sqrt of a pivot from v_rsq_f64 and two Newton
// steps), into LDS; after a second barrier thread c < p forms column c of the
// block's rows of R, into LDS (8 doubles per column) and Rout; after a third
// every thread takes the rank-8 update on its register tiles that still
// matter (not wholly finished, not wholly past p).  Only the current block
// lives in LDS, so four waves per SIMD fit with their register tiles.  *fail
// is set if a pivot is not positive.

// value of v in lane l of the wave (l uniform)
__device__ __forceinline__ double readlane_f64(double v, int l) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, l);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

template <int GW>
__global__ __launch_bounds__(GW * GW) void k_chol_factor(const double* __restrict__ G, int p,
                                                               double shift_rel, int scale,
                                                               double identity_tol,
                                                               double* __restrict__ Rout,
                                                               int* fail, int* missed) {
  __shared__ double Pb[8 * 128];                 // the block's rows of the working matrix
  __shared__ __align__(16) double Rb[128 * 8];   // the block's rows of R, by column
  __shared__ __align__(16) double Ls[64];
  __shared__ double dg[128], dsc[128], red[GW * GW / 64], Li[8];
  __shared__ int bad;
  const int t = threadIdx.x, tx = t % GW, ty = t / GW;
  const int pm = p - 1;
  double A[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int i = min(ty + GW * a, pm), k = min(tx + GW * b, pm);
      A[a][b] = G[min(i, k) * p + max(i, k)];  // upper part, mirrored
    }
  if (identity_tol > 0.0) {
    double d = 0.0;
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int i = ty + GW * a, k = tx + GW * b;
        if (i < p && k < p) d = fmax(d, fabs(A[a][b] - (i == k ? 1.0 : 0.0)));
      }
    for (int o = 32; o > 0; o >>= 1) d = fmax(d, __shfl_xor(d, o, 64));
    if ((t & 63) == 0) red[t >> 6] = d;
    __syncthreads();
    double mx = 0.0;
    for (int w = 0; w < GW * GW / 64; ++w) mx = fmax(mx, red[w]);
    if (mx <= identity_tol) {  // uniform: every thread reduced the same values
      for (int e = t; e < p * p; e += GW * GW) Rout[e] = (e / p == e % p) ? 1.0 : 0.0;
      if (t < p) Rout[p * p + t] = 1.0;
      return;
    }
    if (missed && t == 0) *missed += 1;  // the check found a real factorisation to do
  }
  if (tx == ty) {
#pragma unroll
    for (int a = 0; a < 4; ++a)
      if (ty + GW * a < p) dg[ty + GW * a] = A[a][a];
  }
  if (t == 0) bad = 0;
  __syncthreads();
  if (t < 128) dsc[t] = (scale && t < p) ? 1.0 / sqrt(dg[t]) : 1.0;
  // trace of the matrix factored, every thread summing in the same order
  double tr = 0.0;
  if (scale)
    tr = (double)p;
  else
    for (int i = 0; i < p; ++i) tr += dg[i];
  __syncthreads();
  if (scale) {
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const double dr = dsc[min(ty + GW * a, pm)];
#pragma unroll
      for (int b = 0; b < 4; ++b) A[a][b] *= dr * dsc[min(tx + GW * b, pm)];
    }
  }
  const double shift = shift_rel * tr;
  if (tx == ty) {
#pragma unroll
    for (int a = 0; a < 4; ++a) A[a][a] += shift;
  }

  const int nblk = p >> 3;
  for (int J = 0; J < nblk; ++J) {
    const int j0 = 8 * J, aj = j0 / GW, tj = j0 % GW;
    if (ty >= tj && ty < tj + 8) {
#pragma unroll
      for (int a = 0; a < 4; ++a)
        if (a == aj) {
#pragma unroll
          for (int b = 0; b < 4; ++b) Pb[(ty - tj) * 128 + tx + GW * b] = A[a][b];
        }
    }
    __syncthreads();
    if (t < 64) {
      // the 8 x 8 diagonal block, right-looking, one column per lane (lane
      // c0 < 8 keeps L[r][c0] -> R[j0+r][j0+c0] in x[r], zeros below the
      // diagonal; the other lanes repeat columns and are not used); the
      // pivot and L[r][r2] of another column come from readlane, so no step
      // waits on LDS
      const int c0 = t & 7;
      double x[8];
#pragma unroll
      for (int r = 0; r < 8; ++r) x[r] = r <= c0 ? Pb[r * 128 + j0 + c0] : 0.0;
      bool ok = true;
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const double d = readlane_f64(x[r], r);
        ok = ok && d > 0.0;
        const double dd = d > 0.0 ? d : 1.0;
        double y = __builtin_amdgcn_rsq(dd);
        y = fma(y, fma(-0.5 * dd * y, y, 0.5), y);
        y = fma(y, fma(-0.5 * dd * y, y, 0.5), y);
        x[r] = c0 == r ? dd * y : (c0 > r ? x[r] * y : x[r]);
        if (t == r) Li[r] = y;
#pragma unroll
        for (int r2 = r + 1; r2 < 8; ++r2) {
          const double lr = readlane_f64(x[r], r2);  // L[r][r2]
          if (c0 >= r2) x[r2] -= lr * x[r];
        }
      }
      if (t < 8) {
#pragma unroll
        for (int r = 0; r < 8; ++r) Ls[t * 8 + r] = x[r];  // column t: Ls[c * 8 + r] = L[r][c]
      }
      if (t == 0 && !ok) bad = 1;
    }
    __syncthreads();
    if (t < p) {
      // column t of the block's rows of R: forward substitution past the
      // block, the factor itself inside it, zeros before it
      double v[8];
      if (t >= j0 + 8) {
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          double w = Pb[r * 128 + t];
#pragma unroll
          for (int m = 0; m < r; ++m) w -= Ls[r * 8 + m] * v[m];
          v[r] = w * Li[r];
        }
      } else {
        const int cc = t - j0;
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] = cc >= 0 ? Ls[min(max(cc, 0), 7) * 8 + r] : 0.0;
      }
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        if (t >= j0) Rb[t * 8 + r] = v[r];
        Rout[(j0 + r) * p + t] = v[r];
      }
    }
    __syncthreads();
    if (bad) {
      if (t == 0) *fail = 1;
      return;  // uniform: every thread read the same flag after the barrier
    }
    // rank-8 update; register rows / columns wholly before j0 + 8 are
    // finished and those wholly past p hold only clamped copies: both are
    // skipped (uniform tests); the others take it even where an element is
    // finished -- nobody reads those again
#pragma unroll
    for (int h = 0; h < 8; h += 4) {  // two rank-4 halves keep the operands few
      double Ri[4][4];
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        if (GW * a + GW - 1 < j0 + 8 || GW * a >= p) continue;
        const int i = min(ty + GW * a, pm);
#pragma unroll
        for (int r = 0; r < 4; ++r) Ri[a][r] = Rb[i * 8 + h + r];
      }
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        if (GW * b + GW - 1 < j0 + 8 || GW * b >= p) continue;
        const int k = min(tx + GW * b, pm);
        double Rk[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) Rk[r] = Rb[k * 8 + h + r];
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          if (GW * a + GW - 1 < j0 + 8 || GW * a >= p) continue;
          double v = A[a][b];
#pragma unroll
          for (int r = 0; r < 4; ++r) v -= Ri[a][r] * Rk[r];
          A[a][b] = v;
        }
      }
    }
  }
  if (t < p) Rout[p * p + t] = dsc[t];
}

// Q = R^-T D^-1 Y for the rows of Y (p x n, row-major): with L = R^T (lower
// triangular), L Q = D^-1 Y is solved by blocks of 16 rows,
//   Q_b = L_bb^-1 (D_b^-1 Y_b - sum_{a<b} L_ba Q_a),
// where R and D^-1 are the output of k_chol_factor (R at Rf, D^-1 at
// Rf + p * p).  One workgroup per 64 columns; each of its 4 waves owns 16
// columns and keeps their Q blocks in registers: in the accumulator layout of
// v_mfma_f64_16x16x4f64 (lane j + 16 l holds rows l + 4 v of column j) value
// v of a lane is exactly the B operand the next products take at k step v,
// so the blocks never leave the registers until the end.  R is staged in LDS
// (the A operands of every wave) and the 16 x 16 inverses of the diagonal
// blocks are formed there by forward substitution, one column per thread.
// p a multiple of 16, at most 128; columns past n are computed but not
// stored.
constexpr int kTrsmCols = 64;
__global__ __launch_bounds__(256, 2) void k_trsm_rows(const double* __restrict__ Rf, int p,
                                                   const double* __restrict__ Y, int n,
                                                   double* __restrict__ Q) {
  extern __shared__ double lds[];
  double* Rs = lds;              // p x p
  double* Li = lds + p * p;      // p / 16 blocks of 16 x 16: Li[b][i][c]
  const double* dinv = Rf + p * p;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int nb = p >> 4;
  const int j = lane & 15, l = lane >> 4;
  const int col = blockIdx.x * kTrsmCols + wave * 16 + j;
  const int cc = col < n ? col : n - 1;
  // this lane's rows of D^-1 Y, loaded before anything waits on them
  d4 y[8];
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    if (b >= nb) break;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = 16 * b + l + 4 * v;
      y[b][v] = Y[(long long)r * n + cc];
    }
  }
  {
    // p * p is a multiple of 256 doubles: 16-byte copies, 8 in flight
    typedef double d2 __attribute__((ext_vector_type(2)));
    const d2* src = (const d2*)Rf;
    d2* dst = (d2*)Rs;
#pragma unroll 8
    for (int e = t; e < p * p / 2; e += 256) dst[e] = src[e];
  }
  __syncthreads();
  if (t < 16 * nb) {
    // column c of the inverse of L_bb, L_bb[i][j] = R[16b + j][16b + i]
    const int b = t >> 4, c = t & 15, o = 16 * b;
    double x[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      double v = i == c ? 1.0 : 0.0;
#pragma unroll
      for (int j = 0; j < i; ++j) v -= Rs[(o + j) * p + o + i] * x[j];
      x[i] = v / Rs[(o + i) * p + o + i];
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) Li[(b * 16 + i) * 16 + c] = x[i];
  }
  __syncthreads();
  d4 q[8];
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    if (b >= nb) break;
    d4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int a = 0; a < 8; ++a) {
      if (a >= b) break;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        // A[i][k] = L[16b + i][16a + 4s + k] = R[16a + 4s + k][16b + i], lane i + 16k
        const double av = Rs[(16 * a + 4 * s + l) * p + 16 * b + j];
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av, q[a][s], acc, 0, 0, 0);
      }
    }
    d4 x;
#pragma unroll
    for (int v = 0; v < 4; ++v) x[v] = dinv[16 * b + l + 4 * v] * y[b][v] - acc[v];
    d4 qb = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const double av = Li[(b * 16 + j) * 16 + 4 * s + l];
      qb = __builtin_amdgcn_mfma_f64_16x16x4f64(av, x[s], qb, 0, 0, 0);
    }
    q[b] = qb;
  }
  if (col < n) {
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      if (b >= nb) break;
#pragma unroll
      for (int v = 0; v < 4; ++v) Q[(long long)(16 * b + l + 4 * v) * n + col] = q[b][v];
    }
  }
}

// One workgroup per problem of a batch; a problem whose gate reads 0 (its
// eigensolve has converged, or it has no steps left) is skipped.
__global__ __launch_bounds__(kCholThreads) void k_chol_inv_b(const CholItem* __restrict__ items,
                                                             int pass, int full) {
  const CholItem& it = items[blockIdx.x];
  if (it.gate && *it.gate == 0) return;
  chol_inv_body(it.G, it.p, pass < 2 ? it.shift_rel : 0.0, pass < 2 ? 1 : 0,
                (pass == 0 || full) ? 0.0 : 1e-2, it.Rt, it.fail);
}

void launch_chol_inv_batched(const CholItem* d_items, int count, int pmax, int pass, bool full,
                             hipStream_t s) {
  static bool lds_set = [] {
    return hipFuncSetAttribute((const void*)k_chol_inv_b,
                               hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)(((size_t)128 * 128 + 2048) * sizeof(double))) == hipSuccess;
  }();
  (void)lds_set;
  const size_t lds = ((size_t)pmax * pmax + 2048) * sizeof(double);
  hipLaunchKernelGGL(k_chol_inv_b, dim3(count), dim3(kCholThreads), lds, s, d_items, pass,
                     full ? 1 : 0);
}

// Householder reduction of a small symmetric matrix to tridiagonal form in
// one workgroup, for the Rayleigh-Ritz step (its tridiagonal eigenproblem
// goes to the divide and conquer of k_stedc_small).  For k = 0 .. p-3 the
// entries of row k past the diagonal, x (the column, by symmetry), give v
// (v_0 = 1) and tau with (I - tau v v^T) x = beta e_1, and the trailing block
// takes A <- A - v w^T - w v^T, w = tau A v - (tau^2 / 2) (v^T A v) v (the
// standard symmetric two-sided update).  d (p) and e (p - 1) receive the
// tridiagonal and H the reflectors: v_k in row k (zero outside its columns
// k+1 ..), the taus in row p - 2; k_backtransform applies Q = H_0 H_1 ...
// H_{p-3} to the tridiagonal's eigenvectors.  Every loop has a fixed trip
// count and every sum a fixed order.
//
// What bounds it is the latency of one step's dependency chain, not its
// arithmetic, and after that the LDS instructions of all waves together, so
// the layout keeps both short: 4 waves, NC columns per lane (1 for p <= 64, 2
// up to 128); lane c of wave w holds A[w + 4 r][c (+ 64)] in registers.  A v is
// then one FMA per row and column with v_i as a scalar (readlane) and a sum of
// 4 partials through LDS; the update takes v_i, w_i the same way; the only
// cross-lane sums are |x|^2 and v^T A v.  The wave that owns row k+1 publishes
// it as soon as step k has updated it.  Two barriers per step, which wait
// for LDS only (lds_barrier): the global stores of v_k stay in flight, where
// a fenced barrier waits for them.  Square root and divisions come from
// v_rsq_f64 / v_rcp_f64 and Newton steps.  Against 8 lanes per row in up to 16
// waves with d, e stored to global memory as they are found (and Q^T
// accumulated at the end, an s_barrier over 16 waves alone 467 cycles): p = 64
// 172 -> 61 us, p = 128 415 -> 208 us, and 16 and 43 us for the back-transform
// (which replaces a 7 us product, or 30 us inside the divide and conquer).
// another lane of the same 8-lane group (DPP: quad_perm [1,0,3,2],
// quad_perm [2,3,0,1], row_half_mirror); every lane of the group is active
template <int kCtrl>
__device__ __forceinline__ double trd_dpp(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, kCtrl, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), kCtrl, 0xF, 0xF, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// sum over the 8-lane group, the same bits in every lane
__device__ __forceinline__ double trd_sum8(double v) {
  v += trd_dpp<0xB1>(v);
  v += trd_dpp<0x4E>(v);
  return v + trd_dpp<0x141>(v);
}

// sum over the wave, the same bits in every lane: rows of 16 lanes by DPP
// (the last step row_mirror), then across the rows
__device__ __forceinline__ double trd_sum64(double v) {
  v = trd_sum8(v);
  v += trd_dpp<0x140>(v);
  return (readlane_f64(v, 0) + readlane_f64(v, 16)) + (readlane_f64(v, 32) + readlane_f64(v, 48));
}

// 1 / sqrt(x) and 1 / x from the hardware estimates and two Newton steps
__device__ __forceinline__ double trd_rsq(double x) {
  double y = __builtin_amdgcn_rsq(x);
  y = fma(y, fma(-0.5 * x * y, y, 0.5), y);
  return fma(y, fma(-0.5 * x * y, y, 0.5), y);
}

__device__ __forceinline__ double trd_rcp(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = fma(y, fma(-x, y, 1.0), y);
  return fma(y, fma(-x, y, 1.0), y);
}

template <int NC>
__device__ __forceinline__ void sytrd_body(double* __restrict__ H, int p, double* __restrict__ d,
                                           double* __restrict__ e) {
  constexpr int R = 16 * NC;  // rows per wave
  __shared__ double xs[64 * NC], part[4][64 * NC];
  const int t = threadIdx.x, lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  double a[NC][R];  // a[q][r]: row w + 4 r, column lane + 64 q
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      const int i = w + 4 * r, c = lane + 64 * q;
      a[q][r] = (i < p && c < p) ? H[i * p + c] : 0.0;
    }
  // lane c keeps d, e and tau of the indices c (+ 64)
  double dl[NC], el[NC], tl[NC];
#pragma unroll
  for (int q = 0; q < NC; ++q) dl[q] = el[q] = tl[q] = 0.0;
  // H is in registers (waited for here, so that the loop holds no wait for
  // vector memory): its rows may take the reflectors
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (w == 0) {
#pragma unroll
    for (int q = 0; q < NC; ++q) xs[lane + 64 * q] = a[q][0];  // row 0
  }
  for (int k = 0; k + 2 < p; ++k) {
    lds_barrier();
    double x[NC], v[NC];
    double s2 = 0.0;
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      x[q] = xs[lane + 64 * q];
      s2 += lane + 64 * q > k ? x[q] * x[q] : 0.0;  // columns past p are zero
    }
    const double nrm2 = trd_sum64(s2);
    const double x0 = readlane_f64(NC == 2 && k + 1 >= 64 ? x[NC - 1] : x[0], (k + 1) & 63);
    double beta, tau, scale;
    if (nrm2 >= 0x1p-960) {
      const double y = trd_rsq(nrm2);
      beta = -copysign(nrm2 * y, x0);
      tau = 1.0 + fabs(x0) * y;  // (beta - x0) / beta, beta and x0 of opposite signs
      scale = trd_rcp(x0 - beta);
    } else if (nrm2 == 0.0) {
      beta = x0;
      tau = 0.0;
      scale = 0.0;
    } else {  // near the bottom of the range: the plain operations
      beta = -copysign(sqrt(nrm2), x0);
      tau = (beta - x0) / beta;
      scale = 1.0 / (x0 - beta);
    }
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      const int c = lane + 64 * q;
      v[q] = c == k + 1 ? 1.0 : (c > k + 1 ? x[q] * scale : 0.0);
      dl[q] = c == k ? x[q] : dl[q];
      el[q] = c == k ? beta : el[q];
      tl[q] = c == k ? tau : tl[q];
    }
    // (A v)_c over this wave's rows (v_i = 0 for the finished ones; groups of
    // four rows that are all finished are skipped: a uniform test)
    double vi[R];
    double acc[NC][2];
#pragma unroll
    for (int q = 0; q < NC; ++q) acc[q][0] = acc[q][1] = 0.0;
#pragma unroll
    for (int g = 0; g < R; g += 4) {
      if (4 * (g + 4) <= k + 1) continue;
#pragma unroll
      for (int r = g; r < g + 4; ++r) {
        vi[r] = readlane_f64(v[r >> 4], (w + 4 * r) & 63);
#pragma unroll
        for (int q = 0; q < NC; ++q)
          acc[q][r & 1] = fma(a[q][r], vi[r], acc[q][r & 1]);
      }
    }
#pragma unroll
    for (int q = 0; q < NC; ++q) part[w][lane + 64 * q] = acc[q][0] + acc[q][1];
    // the reflector's row of H (one wave, a different one each step)
    if (w == (k & 3)) {
#pragma unroll
      for (int q = 0; q < NC; ++q)
        if (lane + 64 * q < p) H[k * p + lane + 64 * q] = v[q];
    }
    lds_barrier();
    double ws[NC];
    double pv = 0.0;
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      const int c = lane + 64 * q;
      const double s = (part[0][c] + part[1][c]) + (part[2][c] + part[3][c]);
      ws[q] = c > k ? tau * s : 0.0;  // finished columns take no part
      pv = fma(ws[q], v[q], pv);
    }
    const double alpha = -0.5 * tau * trd_sum64(pv);
#pragma unroll
    for (int q = 0; q < NC; ++q) ws[q] = fma(alpha, v[q], ws[q]);
    const int r1 = (k + 1) >> 2;  // row k+1 in its wave, in the first group not skipped
#pragma unroll
    for (int g = 0; g < R; g += 4) {
      if (4 * (g + 4) <= k + 1) continue;
#pragma unroll
      for (int r = g; r < g + 4; ++r) {
        const double wi = readlane_f64(ws[r >> 4], (w + 4 * r) & 63);
#pragma unroll
        for (int q = 0; q < NC; ++q) a[q][r] = fma(-vi[r], ws[q], fma(-wi, v[q], a[q][r]));
      }
      if (g == (r1 & ~3) && w == ((k + 1) & 3)) {  // publish row k+1 for the next step
#pragma unroll
        for (int q = 0; q < NC; ++q) {
          const double y0 = a[q][g], y1 = a[q][g + 1], y2 = a[q][g + 2], y3 = a[q][g + 3];
          const double lo = (r1 & 1) ? y1 : y0, hi = (r1 & 1) ? y3 : y2;
          xs[lane + 64 * q] = (r1 & 2) ? hi : lo;
        }
      }
    }
  }
  // the last 2 x 2 block: its rows through LDS (xs holds row p - 2 already)
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const int c = lane + 64 * q;
    dl[q] = c == p - 2 ? xs[c] : dl[q];
    if (c == p - 2) el[q] = xs[p - 1];
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (w + 4 * r == p - 1) part[0][c] = a[q][r];
  }
  __syncthreads();
  if (w == 0) {
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      const int c = lane + 64 * q;
      if (c < p) d[c] = c == p - 1 ? part[0][c] : dl[q];
      if (c < p - 1) e[c] = el[q];
      if (c < p - 2) H[(p - 2) * p + c] = tl[q];
    }
  }
}

template <int NC>
__global__ __launch_bounds__(256) void k_sytrd_small(double* __restrict__ H, int p,
                                                          double* __restrict__ d,
                                                          double* __restrict__ e) {
  sytrd_body<NC>(H, p, d, e);
}

static void launch_sytrd(double* H, int p, double* d, double* e, hipStream_t s) {
  if (p <= 64)
    hipLaunchKernelGGL(k_sytrd_small<1>, dim3(1), dim3(256), 0, s, H, p, d, e);
  else
    hipLaunchKernelGGL(k_sytrd_small<2>, dim3(1), dim3(256), 0, s, H, p, d, e);
}

// Rows z of Zt (p x p, the tridiagonal's eigenvectors) become the rows Q z,
// Q = H_0 ... H_{p-3} from the reflectors sytrd_body leaves in V (p x p):
// for k = p-3 .. 0, z <- z - tau_k (v_k^T z) v_k.  Rows row0 .. row0 + rows -
// 1 of Zt; row c goes to out + c ldo, its first nout entries (out may be Zt:
// a row is read and written by the same lanes).  Eight lanes per row, 32 rows
// per workgroup, V in LDS; a step is 8 NC products per lane, an 8-lane sum
// and 8 NC updates, with the next v loaded meanwhile.  The rows are
// independent, so they spread over workgroups (compute units), where the
// accumulation of Q^T inside the reduction's own workgroup was bound by one
// compute unit's LDS reads of v.
constexpr int kBackRows = 32;
template <int NC>
__device__ __forceinline__ void backtransform_body(const double* __restrict__ V, int p,
                                                   const double* Zt, int row0, int rows,
                                                   double* out, long long ldo, int nout,
                                                   int block) {
  constexpr int W = 64 * NC, C = 8 * NC;
  extern __shared__ double Vs[];  // (p - 2) x W, columns past p zero
  __shared__ double taus[128];
  const int t = threadIdx.x;
  for (int x = t; x < (p - 2) * W; x += 256) {
    const int k = x / W, c = x % W;
    Vs[x] = c < p ? V[k * p + c] : 0.0;
  }
  if (t < p - 2) taus[t] = V[(p - 2) * p + t];
  const int g = block * kBackRows + (t >> 3), u = t & 7;
  const int row = row0 + (g < rows ? g : rows - 1);
  // columns 16 (r / 2) + 2 u + r % 2
  double z[C], v[C];
#pragma unroll
  for (int r = 0; r < C; ++r) {
    const int c = 16 * (r >> 1) + 2 * u + (r & 1);
    z[r] = c < p ? Zt[(long long)row * p + c] : 0.0;
  }
  __syncthreads();
  typedef double d2 __attribute__((ext_vector_type(2)));
  auto load = [&](int k, double (&x)[C]) {
#pragma unroll
    for (int r = 0; r < C; r += 2) {
      const d2 y = *(const d2*)(Vs + k * W + 8 * r + 2 * u);
      x[r] = y.x;
      x[r + 1] = y.y;
    }
  };
  load(p - 3, v);
  double tau = taus[p - 3];
  for (int k = p - 3; k >= 0; --k) {
    double vn[C];
    const int kn = k > 0 ? k - 1 : 0;
    load(kn, vn);
    const double tn = taus[kn];
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int r = 0; r < C; ++r) acc[r & 3] = fma(z[r], v[r], acc[r & 3]);
    const double y = tau * trd_sum8((acc[0] + acc[1]) + (acc[2] + acc[3]));
#pragma unroll
    for (int r = 0; r < C; ++r) z[r] = fma(-y, v[r], z[r]);
#pragma unroll
    for (int r = 0; r < C; ++r) v[r] = vn[r];
    tau = tn;
  }
  if (g < rows) {
#pragma unroll
    for (int r = 0; r < C; ++r) {
      const int c = 16 * (r >> 1) + 2 * u + (r & 1);
      if (c < nout) out[(long long)row * ldo + c] = z[r];
    }
  }
}

template <int NC>
__global__ __launch_bounds__(256) void k_backtransform(const double* __restrict__ V, int p,
                                                       const double* Zt, int row0, int rows,
                                                       double* out, long long ldo, int nout) {
  backtransform_body<NC>(V, p, Zt, row0, rows, out, ldo, nout, blockIdx.x);
}

static inline size_t back_lds(int p, int nc) { return (size_t)(p - 2) * 64 * nc * sizeof(double); }

// false when the launch's LDS cannot be had
static bool launch_backtransform(const double* V, int p, const double* Zt, int row0, int rows,
                                 double* out, hipStream_t s) {
  static const bool lds_set =
      hipFuncSetAttribute((const void*)k_backtransform<2>,
                          hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)back_lds(128, 2)) == hipSuccess;
  if (!lds_set || p < 3 || p > 128) return false;
  const dim3 grid((rows + kBackRows - 1) / kBackRows);
  if (p <= 64)
    hipLaunchKernelGGL(k_backtransform<1>, grid, dim3(256), back_lds(p, 1), s, V, p, Zt, row0,
                       rows, out, (long long)p, p);
  else
    hipLaunchKernelGGL(k_backtransform<2>, grid, dim3(256), back_lds(p, 2), s, V, p, Zt, row0,
                       rows, out, (long long)p, p);
  return true;
}

// Eigenpairs of a small symmetric matrix M (n x n, 3 <= n <= 128, row-major,
// overwritten): W ascending, rows n - rows .. n - 1 of Zt (n x n) <- the
// eigenvectors of the `rows` largest (row c for W[c]; the other rows are
// scratch); E (n doubles) is scratch, *info = 1 when a result is not finite.
// Three launches: the Householder reduction, the divide and conquer (one
// workgroup each) and the back-transform of the rows wanted.
bool dense_eig_small(double* M, int n, int rows, double* W, double* E, double* Zt, int* info,
                     hipStream_t s) {
  if (n < 3 || n > 128) return false;
  launch_sytrd(M, n, W, E, s);
  return tridiag_eig_small(W, E, n, W, Zt, info, s) &&
         launch_backtransform(M, n, Zt, n - rows, rows, Zt, s);
}

// The same reduction for every problem of a lockstep batch whose block
// eigensolver is still iterating: H (p x p) -> reflectors, diagonal into W,
// the off-diagonal into G (free during the Rayleigh-Ritz step).
template <int NC>
__global__ __launch_bounds__(256) void k_group_sytrd(const GroupStep* __restrict__ dsc) {
  const GroupStep& g = dsc[blockIdx.x];
  if (!g.ctl->iter) return;  // uniform
  sytrd_body<NC>(g.H, g.p, g.W, g.G);
}

void group_sytrd(const GroupStep* d, int count, int pmax, hipStream_t s) {
  if (pmax <= 64)
    hipLaunchKernelGGL(k_group_sytrd<1>, dim3(count), dim3(256), 0, s, d);
  else
    hipLaunchKernelGGL(k_group_sytrd<2>, dim3(count), dim3(256), 0, s, d);
}

// The tridiagonals' eigenvector rows (in Rt) back to the Rayleigh-Ritz
// matrices' rows, in place -- or, for environments diagonalised whole (dense),
// to the rows of X (n columns: the padded index is dropped).
template <int NC>
__global__ __launch_bounds__(256) void k_group_back(const GroupStep* __restrict__ dsc, int dense) {
  const GroupStep& g = dsc[blockIdx.y];
  if (!g.ctl->iter || (int)blockIdx.x * kBackRows >= g.p) return;  // uniform
  backtransform_body<NC>(g.H, g.p, g.Rt, 0, g.p, dense ? g.X : g.Rt, dense ? g.n : g.p,
                         dense ? g.n : g.p, blockIdx.x);
}

void group_back(const GroupStep* d, int count, int pmax, bool dense, hipStream_t s) {
  static const bool lds_set =
      hipFuncSetAttribute((const void*)k_group_back<2>,
                          hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)back_lds(128, 2)) == hipSuccess;
  (void)lds_set;
  const dim3 grid((pmax + kBackRows - 1) / kBackRows, count);
  if (pmax <= 64)
    hipLaunchKernelGGL(k_group_back<1>, grid, dim3(256), back_lds(pmax, 1), s, d, dense ? 1 : 0);
  else
    hipLaunchKernelGGL(k_group_back<2>, grid, dim3(256), back_lds(pmax, 2), s, d, dense ? 1 : 0);
}

__global__ void k_symmetrize_small(double* H, int p) {
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < p * p; e += gridDim.x * blockDim.x) {
    const int i = e / p, j = e % p;
    if (i < j) {
      const double v = 0.5 * (H[i * p + j] + H[j * p + i]);
      H[i * p + j] = v;
      H[j * p + i] = v;
    }
  }
}

// res[i] = |Yx[i,:] - theta[i] X[i,:]| (one block per row, fixed-order tree)
__global__ void k_ritz_residual(const double* __restrict__ Yx, const double* __restrict__ X,
                                const double* __restrict__ theta, int n, double* res) {
  __shared__ double red[256];
  const int i = blockIdx.x, t = threadIdx.x;
  const double th = theta[i];
  double s = 0.0;
  for (int j = t; j < n; j += 256) {
    const double d = Yx[(long long)i * n + j] - th * X[(long long)i * n + j];
    s += d * d;
  }
  red[t] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (t < o) red[t] += red[t + o];
    __syncthreads();
  }
  if (t == 0) res[i] = sqrt(red[0]);
}

static inline int splitk_chunk(int K) {
  // about 32 partial products, each K chunk a multiple of 16
  int c = (K + 31) / 32;
  c = (c + 15) / 16 * 16;
  return c < 16 ? 16 : c;
}

// K chunk of the block products V M (p x n times n x n) by 64 x 64 tiles:
// enough partial products for about 1024 workgroups (at least 4, at most
// 16), so that p = 128, n = 4096 takes 8 x 2 x 64 (four workgroups per CU
// hide each other's slab loads: 2% less eigensolver time than 4 x 2 x 64)
// and p = 64, n = 1024 takes 16 x 1 x 16 instead of the 64 workgroups of a
// 4-way split that left most of the chip idle
static inline int vm_chunk(int n, int p) {
  const int tiles = ((p + 63) / 64) * ((n + 63) / 64);
  const int parts = std::min(16, std::max(4, (1024 + tiles - 1) / tiles));
  return ((n + parts - 1) / parts + 15) / 16 * 16;
}

static inline size_t partial_doubles(int n, int p) {
  const size_t pn = (size_t)p * n, pp = (size_t)p * p;
  const size_t gram = (size_t)((n + splitk_chunk(n) - 1) / splitk_chunk(n)) * pp;
  const size_t vm = (size_t)((n + vm_chunk(n, p) - 1) / vm_chunk(n, p)) * pn;
  return gram > vm ? gram : vm;
}

size_t topk_workspace_doubles(int n, int p) {
  const size_t pn = (size_t)p * n, pp = (size_t)p * p;
  return 4 * pn + partial_doubles(n, p) + 4 * pp + 4 * (size_t)p + 16;
}

// Returns true and leaves theta (ascending, p values) in W and the Ritz
// vectors (rows, same order) in Xout (p x n) on convergence.
//
// The sweeps multiply by M - sigma I (the Rayleigh-Ritz products use M
// itself).  M is positive semidefinite and the unwanted eigenvalues lie in
// [0, lambda_{p+1}]; with sigma = lambda_{p+1} / 2 the worst of them shrinks
// by sigma / (lambda_need - sigma) per sweep instead of lambda_{p+1} /
// lambda_need.  *shift holds the sigma to start with (from an earlier solve
// of the same kind; 0 if none) and returns theta_min / 2 of the last
// Rayleigh-Ritz step (theta_min <= lambda_p, so sigma never exceeds half of
// a wanted eigenvalue).
//
// Between Rayleigh-Ritz steps a sweep orthonormalises with one shifted
// Cholesky-QR pass and checks the result with a second Gram matrix (a real
// second pass when it is not the identity to 1e-2).  When no check since the
// last Rayleigh-Ritz step needed that second pass, only the first sweep of
// the next group is checked; *nocheck carries that state to the next solve.
// Every Rayleigh-Ritz step still sees a basis from three passes, and its
// residuals decide convergence.
bool topk_eigs(const double* M, int n, int p, int need, double tol,
               int q_first, double* shift, int* nocheck, double* ws, double* W, double* Xout,
               int* dinfo, int* iters, int* enough, double* resid, hipStream_t s) {
  const size_t pn = (size_t)p * n, pp = (size_t)p * p;
  const int kc = splitk_chunk(n);
  const int kv = vm_chunk(n, p);
  double* V = ws;
  double* Y = V + pn;
  double* T2 = Y + pn;
  double* Yx = T2 + pn;
  double* part = Yx + pn;
  double* G = part + partial_doubles(n, p);
  double* Rt = G + pp;
  double* H = Rt + pp;
  double* E = H + pp;          // off-diagonal of the tridiagonal form (p - 1)
  double* res = E + pp;        // p
  int* fail = (int*)(res + p); // fail flag, then the count of checks that missed
  // a pass's Cholesky factor (p x p) at Rt and its row scaling (p) in the
  // first p entries of H, which only the Rayleigh-Ritz step uses
  double* Rf = Rt;
  const double u = std::ldexp(1.0, -53);
  const double shift_rel = 11.0 * ((double)n * p + (double)p * (p + 1)) * u;

  static bool lds_set = [] {
    return hipFuncSetAttribute((const void*)k_trsm_rows,
                               hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)(((size_t)128 * 128 + 128 * 16) * sizeof(double))) ==
           hipSuccess;
  }();
  const size_t trsm_lds = ((size_t)p * p + (size_t)p * 16) * sizeof(double);
  if (!lds_set || p > 128 || p % 16 != 0) return false;
  (void)hipMemsetAsync(fail, 0, 2 * sizeof(int), s);
  hipLaunchKernelGGL(k_seed_block, dim3(256), dim3(256), 0, s, V, (long long)pn, 12345ULL);

  // one orthonormalisation of rows of Y into V: shifted Cholesky-QR of the
  // column-scaled Gram matrix twice, then a plain pass -- all three before a
  // Rayleigh-Ritz check (`full`); between checks only the first two, the
  // second skipped on the device (R^-1 = I) when its Gram matrix is the
  // identity to 1e-2.
  auto orth = [&](const double* Yin, double* Vout, bool full, bool check) {
    const double* src = Yin;
    const int last = full ? 2 : (check ? 1 : 0);
    for (int pass = 0; pass <= last; ++pass) {
      gemm_f64_splitk(src, n, src, n, B_KCONTIG, G, p, p, p, n, kc, part, s);
      const double sh = pass < 2 ? shift_rel : 0.0, itol = (pass == 0 || full) ? 0.0 : 1e-2;
      if (p <= 64)
        hipLaunchKernelGGL(k_chol_factor<16>, dim3(1), dim3(256), 0, s, G, p, sh,
                           pass < 2 ? 1 : 0, itol, Rf, fail, fail + 1);
      else
        hipLaunchKernelGGL(k_chol_factor<32>, dim3(1), dim3(1024), 0, s, G, p, sh,
                           pass < 2 ? 1 : 0, itol, Rf, fail, fail + 1);
      double* dst = (pass == last) ? Vout : (src == T2 ? Y : T2);
      if (dst == src) dst = (src == Y) ? T2 : Y;
      hipLaunchKernelGGL(k_trsm_rows, dim3((n + kTrsmCols - 1) / kTrsmCols), dim3(256), trsm_lds,
                         s, (const double*)Rf, p, src, n, dst);
      src = dst;
    }
  };

  // Y = V (M - sigma I)
  double sigma = shift && *shift > 0.0 ? *shift : 0.0;
  auto vm = [&](const double* Vin, double* Yout, double sg) {
    gemm_f64_splitk(Vin, n, M, n, B_NCONTIG, Yout, n, p, n, n, kv, part, s,
                    sg > 0.0 ? Vin : nullptr, sg);
  };

  int it = 0, q = q_first > 0 ? q_first : 3;
  const int max_it = 80;
  double prev = 1e300;
  std::vector<double> th(p), rs(p);
  while (true) {
    const bool skip = nocheck && *nocheck;
    for (int r = 0; r < q; ++r) {
      vm(V, Y, sigma);
      orth(Y, V, r == q - 1, r == 0 || !skip);
      ++it;
    }
    // Rayleigh-Ritz
    vm(V, Y, 0.0);
    gemm_f64_splitk(V, n, Y, n, B_KCONTIG, H, p, p, p, n, kc, part, s);
    hipLaunchKernelGGL(k_symmetrize_small, dim3(16), dim3(256), 0, s, H, p);
    // tridiagonal form and its reflectors (over H), then divide and conquer
    // on the tridiagonal (Z^T into Rt, eigenvalues over its diagonal in W),
    // then the rows of Rt back to H's basis: the Ritz coefficients
    launch_sytrd(H, p, W, E, s);
    if (!tridiag_eig_small(W, E, p, W, Rt, dinfo, s)) return false;
    if (!launch_backtransform(H, p, Rt, 0, p, Rt, s)) return false;
    gemm_f64(Rt, p, V, n, B_NCONTIG, Xout, out_rowmajor(n), p, n, p, nullptr, s);
    gemm_f64(Rt, p, Y, n, B_NCONTIG, Yx, out_rowmajor(n), p, n, p, nullptr, s);
    hipLaunchKernelGGL(k_ritz_residual, dim3(p), dim3(256), 0, s, Yx, Xout, W, n, res);
    int hinfo[3] = {0, 0, 0};
    (void)hipMemcpyAsync(th.data(), W, p * sizeof(double), hipMemcpyDeviceToHost, s);
    (void)hipMemcpyAsync(rs.data(), res, p * sizeof(double), hipMemcpyDeviceToHost, s);
    (void)hipMemcpyAsync(&hinfo[0], dinfo, sizeof(int), hipMemcpyDeviceToHost, s);
    (void)hipMemcpyAsync(&hinfo[1], fail, 2 * sizeof(int), hipMemcpyDeviceToHost, s);
    if (hipStreamSynchronize(s) != hipSuccess) return false;
    if (hinfo[0] != 0 || hinfo[1] != 0) return false;
    if (nocheck) *nocheck = hinfo[2] == 0 ? 1 : 0;
    (void)hipMemsetAsync(fail + 1, 0, sizeof(int), s);
    const double t1 = th[p - 1];
    if (!(t1 > 0.0)) return false;
    double top = 0.0;
    for (int i = 0; i < need; ++i) top = std::fmax(top, rs[p - 1 - i] / t1);
    // the worst unwanted factor per sweep at the shift the sweeps used, and
    // the shift for the next ones
    const double lo = std::fmax(th[0], 0.0);
    double rate = th[p - need] > sigma ? std::fmax(lo - sigma, sigma) / (th[p - need] - sigma)
                                       : 0.5;
    rate = std::fmin(std::fmax(rate, 1e-6), 0.95);
    sigma = 0.5 * lo;
    if (shift) *shift = sigma;
    if (iters) *iters = it;
    if (resid) *resid = top;
    if (top <= tol) {
      // sweeps beyond the first that met tol: top / rate^k <= tol
      int extra = top > 0.0 ? (int)std::floor(std::log(top / tol) / std::log(rate)) : it;
      extra = extra < 0 ? 0 : extra;
      if (enough) *enough = it - extra < 1 ? 1 : it - extra;
      return true;
    }
    if (it >= max_it || !(top < 0.5 * prev)) return false;
    prev = top;
    // the sweeps to come run at the new shift
    rate = th[p - need] > sigma ? std::fmax(lo - sigma, sigma) / (th[p - need] - sigma) : 0.5;
    rate = std::fmin(std::fmax(rate, 1e-6), 0.95);
    q = (int)std::ceil(std::log(tol / top) / std::log(rate));
    q = q < 1 ? 1 : (q > max_it - it ? max_it - it : q);
    // continue from the Ritz vectors
    (void)hipMemcpyAsync(V, Xout, pn * sizeof(double), hipMemcpyDeviceToDevice, s);
  }
}

}  // namespace hotrg
