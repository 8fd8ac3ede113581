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
#include <cstring>
#include <vector>

#include "internal.h"

namespace hotrg {

typedef double d4 __attribute__((ext_vector_type(4)));

// deterministic start block: splitmix64 of the element index -> [-1, 1)
__global__ void k_seed_block(double* V, long long count, unsigned long long seed, int* fail) {
  if (blockIdx.x == 0 && threadIdx.x < 2) fail[threadIdx.x] = 0;
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

// value of v in lane l of the wave (l uniform)
__device__ __forceinline__ double readlane_f64(double v, int l) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, l);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// Cholesky factor of a sweep's Gram matrix (Q = R^-T D^-1 Y then comes from
// k_trsm_rows): R with R^T R = D^-1 G D^-1 + s I (`scale`; D = diag(G)^1/2) or
// G + s I, s = shift_rel * trace of the matrix factored.  Rout receives R (p x p
// row-major; right of the diagonal 16 x 16 blocks only, and in those the blocks'
// inverses) and D^-1 (ones without `scale`) at p * p; with identity_tol > 0 and G
// the identity to within it, R = I.  *fail is set if a pivot is not positive.
//
// One workgroup, p a multiple of 16 up to 16 NB.  The upper 16 x 16 tiles stay in
// MFMA accumulators (negated, one of a row per wave), and each of the p / 16 steps
// has two barriers: the owners publish the step's row of tiles, the first one or
// two waves factor it while others store the rows of the step before, and the
// tiles below take R^T R by MFMA.  What bounds the kernel is the chain of one
// pivot after the other (v_rcp_f64, two Newton steps, the next pivot's row; the
// square roots are off it), so a step keeps it inside a row of 16 lanes: lane c of
// each has column c of the diagonal block, which every row of lanes factors again,
// and each lane one column to the right of it or, the first 16, of the identity,
// whose solution is the block's inverse.  Values of another column come by DPP
// (through a scalar register, v_readlane, each costs its latency).  Against 8-wide
// steps with the matrix in the registers of 256 or 1024 threads, three fenced
// barriers each, and the inverses formed again by each workgroup of k_trsm_rows:
// p = 64 18.0 -> 9.9 us, p = 128 47 -> 20, k_trsm_rows (64 x 1024)
// 7.3 -> 5.2; in a batch, where the inverse of R was formed and multiplied by,
// 17.9 + 9 -> 4.5 + 3.4 (p = 48, converged problems included).
template <int NB>
struct CholLds {
  static constexpr int NW = NB > 4 ? 8 : 4;  // waves
  static constexpr int W = 16 * NB, S = W + 16;
  double P[16 * S];                  // the step's row of tiles
  double R[W * W];                   // rows of R; odd ones with columns ^ 16
  double dg[W], dsc[W], red[NW];
  __device__ static int at(int r, int c) { return r * W + (c ^ ((r & 1) << 4)); }
};

// value of v in lane I of the row of 16 lanes (DPP row_newbcast)
template <int I>
__device__ __forceinline__ double bcast16(double v) {
  return __builtin_amdgcn_update_dpp(v, v, 0x150 + I, 0xf, 0xf, true);
}

// 1 / d (v_rcp_f64, two Newton steps); of a pivot not positive it is not used
__device__ __forceinline__ double pivot_rcp(double d) {
  double q = __builtin_amdgcn_rcp(d);
  q = fma(q, fma(-d, q, 1.0), q);
  return fma(q, fma(-d, q, 1.0), q);
}

// Rows R2 .. E of a step's columns less their multiple of row R, m = row R over its
// pivot: row R of column R2 of the diagonal block times m.
template <int R, int R2, int E>
__device__ __forceinline__ void chol_elim(double (&xd)[16], double (&x)[16], double md, double m) {
  if constexpr (R2 <= E) {
    const double b = bcast16<R2>(xd[R]);
    xd[R2] = fma(-b, md, xd[R2]);
    x[R2] = fma(-b, m, x[R2]);
    chol_elim<R, R2 + 1, E>(xd, x, md, m);
  }
}
// From row R down, q = 1 / its pivot.  The next pivot's row goes first, and its
// chain then runs between the other rows'; the fence keeps the rows of later steps
// from being fetched before (256 registers and spills).
template <int R>
__device__ __forceinline__ bool chol_pivots(double (&xd)[16], double (&x)[16], double q, bool ok) {
  if constexpr (R < 15) {
    const double md = xd[R] * q, m = x[R] * q;
    chol_elim<R, R + 1, R + 1>(xd, x, md, m);
    const double d = bcast16<R + 1>(xd[R + 1]);
    const double next = pivot_rcp(d);
    chol_elim<R, R + 2, 15>(xd, x, md, m);
    __builtin_amdgcn_sched_barrier(0);
    return chol_pivots<R + 1>(xd, x, next, ok && d > 0.0);
  } else {
    return ok;
  }
}
// x[R] over the root of pivot R, y in lane R of each row of lanes
template <int R>
__device__ __forceinline__ void chol_scale(double (&x)[16], double y) {
  if constexpr (R < 16) {
    x[R] *= bcast16<R>(y);
    chol_scale<R + 1>(x, y);
  }
}

template <int NB>
__device__ __forceinline__ void chol_body(const double* __restrict__ G, int p, double shift_rel,
                                          int scale, double identity_tol,
                                          double* __restrict__ Rout, int* fail, int* missed,
                                          CholLds<NB>& L) {
  using LD = CholLds<NB>;
  typedef double d2 __attribute__((ext_vector_type(2)));
  constexpr int S = LD::S, NW = LD::NW, NT = 64 * NW, Q = NB / 2 + 1;
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int li = lane & 15, lg = lane >> 4, nb = p >> 4;
  double* Dout = Rout + (size_t)p * p;
  // this wave's tiles (ti, tk), ti <= tk: those with ti + tk = w modulo NB, from
  // the middle outwards (an odd w has one fewer); ti = -1 past the end
  static_assert(NB == NW, "one tile of a row per wave");
  int ti[Q], tk[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int a = ((w >> 1) - q) & (NB - 1), b = (w - a) & (NB - 1);
    const bool in = max(a, b) < nb && !((w & 1) && q == Q - 1);
    ti[q] = in ? min(a, b) : -1;
    tk[q] = in ? max(a, b) : 0;
  }
  d4 acc[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = 16 * max(ti[q], 0) + lg + 4 * v, k = 16 * tk[q] + li;
      acc[q][v] = G[min(i, k) * p + max(i, k)];  // upper part, mirrored
    }
  if (identity_tol > 0.0) {
    double d = 0.0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      if (ti[q] < 0) continue;
#pragma unroll
      for (int v = 0; v < 4; ++v)
        d = fmax(d, fabs(acc[q][v] - (ti[q] == tk[q] && lg + 4 * v == li ? 1.0 : 0.0)));
    }
    for (int o = 32; o > 0; o >>= 1) d = fmax(d, __shfl_xor(d, o, 64));
    if (lane == 0) L.red[w] = d;
    lds_barrier();
    double mx = 0.0;
#pragma unroll
    for (int i = 0; i < NW; ++i) mx = fmax(mx, L.red[i]);
    if (mx <= identity_tol) {  // uniform: every thread reduced the same values
      for (int e = t; e < p * p; e += NT) Rout[e] = (e / p == e % p) ? 1.0 : 0.0;
      if (t < p) Dout[t] = 1.0;
      return;
    }
    if (missed && t == 0) *missed += 1;  // the check found a real factorisation to do
  }
#pragma unroll
  for (int q = 0; q < Q; ++q)
    if (ti[q] == tk[q]) {
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (lg + 4 * v == li) L.dg[16 * ti[q] + li] = acc[q][v];
    }
  lds_barrier();
  // trace of the matrix factored, every thread summing in the same order
  double tr = (double)p;
  if (!scale) {
    tr = 0.0;
    for (int i = 0; i < p; ++i) tr += L.dg[i];
  }
  const double shift = shift_rel * tr;
  if (t < p) {
    double dv = 1.0;
    if (scale) {
      const double g = L.dg[t], h = -0.5 * g;
      dv = __builtin_amdgcn_rsq(g);
      dv = fma(dv, fma(h * dv, dv, 0.5), dv);
      dv = fma(dv, fma(h * dv, dv, 0.5), dv);
    }
    L.dsc[t] = dv;
    Dout[t] = dv;
  }
  lds_barrier();
#pragma unroll
  for (int q = 0; q < Q; ++q)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      double a = acc[q][v];
      if (scale) a *= L.dsc[16 * max(ti[q], 0) + lg + 4 * v] * L.dsc[16 * tk[q] + li];
      if (ti[q] == tk[q] && lg + 4 * v == li) a += shift;
      acc[q][v] = -a;
    }
  // rows of step J of R to Rout (wave `first` and up); in LDS the diagonal block's
  // place holds the inverse of the block of L, whose transpose goes out
  auto dump = [&](int J, int first) {
    const int c = 2 * lane, j0 = 16 * J;
    for (int r = j0 + w - first; r < j0 + 16; r += NW - first)
      if (c >= j0 && c < p) {
        const bool in = c < j0 + 16;
        const double a = L.R[in ? LD::at(c, r) : LD::at(r, c)];
        const double b = L.R[in ? LD::at(c + 1, r) : LD::at(r, c + 1)];
        *(d2*)(Rout + r * p + c) = d2{a, b};
      }
  };
  bool ok = true;
  for (int J = 0; J < nb; ++J) {
    const int j0 = 16 * J;
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if (ti[q] == J) {
#pragma unroll
        for (int v = 0; v < 4; ++v) L.P[(lg + 4 * v) * S + 16 * tk[q] + li] = -acc[q][v];
      }
    lds_barrier();
    if (64 * w < p - j0) {
      // own column e: of the identity below 16, then j0 + e, past p repeats of the
      // last one
      const int e = 64 * w + lane;
      const bool unit = e < 16;
      const int col = min(j0 + e, p - 1);
      double xd[16], x[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        xd[r] = L.P[r * S + j0 + li];
        x[r] = L.P[r * S + col];
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        asm volatile("" : "+v"(x[r]));  // all the loads, then the selects: not 16 branches
        if (unit) x[r] = r == e ? 1.0 : 0.0;
      }
      const double d0 = bcast16<0>(xd[0]);
      ok = chol_pivots<0>(xd, x, pivot_rcp(d0), ok && d0 > 0.0);
      double d = xd[15];  // pivot of row li
#pragma unroll
      for (int r = 0; r < 15; ++r) d = li == r ? xd[r] : d;
      double y = __builtin_amdgcn_rsq(d);
      const double h = -0.5 * d;
      y = fma(y, fma(h * y, y, 0.5), y);
      y = fma(y, fma(h * y, y, 0.5), y);
      chol_scale<0>(x, y);
      // (or the rows' arithmetic moves into the branch, with every b kept for it)
#pragma unroll
      for (int r = 0; r < 16; ++r) asm volatile("" : "+v"(x[r]));
      if (e < p - j0) {
#pragma unroll
        for (int r = 0; r < 16; ++r) L.R[LD::at(j0 + r, col)] = x[r];
      }
    } else if (w >= 2 && J > 0) {
      dump(J - 1, 2);
    }
    lds_barrier();
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if (ti[q] > J) {
        double fa[4], fb[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          fa[u] = L.R[LD::at(j0 + 4 * u + lg, 16 * ti[q] + li)];
          fb[u] = L.R[LD::at(j0 + 4 * u + lg, 16 * tk[q] + li)];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
          acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[u], fb[u], acc[q], 0, 0, 0);
      }
  }
  dump(nb - 1, 0);
  if (t == 0 && !ok) *fail = 1;
}

template <int NB>
__global__ __launch_bounds__(64 * CholLds<NB>::NW) void k_chol_factor(
    const double* __restrict__ G, int p, double shift_rel, int scale, double identity_tol,
    double* __restrict__ Rout, int* fail, int* missed) {
  __shared__ CholLds<NB> L;
  chol_body<NB>(G, p, shift_rel, scale, identity_tol, Rout, fail, missed, L);
}

// Q = R^-T D^-1 Y for the rows of Y (p x n, row-major): with L = R^T (lower
// triangular), L Q = D^-1 Y is solved by blocks of 16 rows,
//   Q_b = L_bb^-1 (D_b^-1 Y_b - sum_{a<b} L_ba Q_a),
// where R (with R_bb^-1 = L_bb^-T in the place of its diagonal blocks) and D^-1 are
// the output of k_chol_factor (R at Rf, D^-1 at Rf + p * p).  One workgroup per 64 columns; each of its 4 waves owns 16
// columns and keeps their Q blocks in registers: in the accumulator layout of
// v_mfma_f64_16x16x4f64 (lane j + 16 l holds rows l + 4 v of column j) value
// v of a lane is exactly the B operand the next products take at k step v,
// so the blocks never leave the registers until the end.  R is staged in LDS
// (the A operands of every wave).
// p a multiple of 16, at most 128; columns past n are computed but not
// stored.
constexpr int kTrsmCols = 64;
__device__ __forceinline__ void trsm_body(const double* __restrict__ Rf, int p,
                                          const double* __restrict__ Y, int n,
                                          double* __restrict__ Q) {
  extern __shared__ double lds[];
  double* Rs = lds;              // p x p
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
      const double av = Rs[(16 * b + 4 * s + l) * p + 16 * b + j];
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

__global__ __launch_bounds__(256, 2) void k_trsm_rows(const double* __restrict__ Rf, int p,
                                                      const double* __restrict__ Y, int n,
                                                      double* __restrict__ Q) {
  trsm_body(Rf, p, Y, n, Q);
}

// The same two for every problem of a batch; a problem whose eigensolve has
// converged, or that has no steps left, is skipped.
template <int NB>
__global__ __launch_bounds__(64 * CholLds<NB>::NW) void k_group_chol(
    const GroupStep* __restrict__ dsc, int pass, int full) {
  __shared__ CholLds<NB> L;
  const GroupStep& g = dsc[blockIdx.x];
  if (g.ctl->iter == 0) return;
  chol_body<NB>(g.G, g.p, pass < 2 ? g.shift_rel : 0.0, pass < 2 ? 1 : 0,
                (pass == 0 || full) ? 0.0 : 1e-2, g.Rt, &g.ctl->fail, nullptr, L);
}

__global__ __launch_bounds__(256, 2) void k_group_trsm(const GroupStep* __restrict__ dsc, int src,
                                                       int dst) {
  const GroupStep& g = dsc[blockIdx.y];
  if (g.ctl->iter == 0 || (int)blockIdx.x * kTrsmCols >= g.n) return;
  double* const b[3] = {g.V, g.Y, g.T2};
  trsm_body(g.Rt, g.p, b[src], g.n, b[dst]);
}

static bool trsm_lds_set() {
  static const bool ok = [] {
    const int bytes = (int)((size_t)128 * 128 * sizeof(double));
    return hipFuncSetAttribute((const void*)k_trsm_rows,
                               hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess &&
           hipFuncSetAttribute((const void*)k_group_trsm,
                               hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess;
  }();
  return ok;
}

void group_orth(const GroupStep* d, int count, int pmax, int max_n, int pass, bool full,
                GroupRows src, GroupRows dst, hipStream_t s) {
  (void)trsm_lds_set();
  if (pmax <= 64)
    hipLaunchKernelGGL(k_group_chol<4>, dim3(count), dim3(256), 0, s, d, pass, full ? 1 : 0);
  else
    hipLaunchKernelGGL(k_group_chol<8>, dim3(count), dim3(512), 0, s, d, pass, full ? 1 : 0);
  hipLaunchKernelGGL(k_group_trsm, dim3((max_n + kTrsmCols - 1) / kTrsmCols, count), dim3(256),
                     (size_t)pmax * pmax * sizeof(double), s, d, (int)src, (int)dst);
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
// 172 -> 59 us, p = 128 415 -> 205 us, and 14 and 41 us for the back-transform
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

// res[i] = |Yx[i,:] - theta[i] X[i,:]| (one block per row, fixed-order tree); and what
// the host reads of a Rayleigh-Ritz step beside them: theta at res + p, then the
// ints dinfo, fail[0] and fail[1], which starts again at 0.
__global__ void k_ritz_residual(const double* __restrict__ Yx, const double* __restrict__ X,
                                const double* __restrict__ theta, int n, double* res, int p,
                                const int* __restrict__ dinfo, int* fail) {
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
  if (t == 0) {
    res[i] = sqrt(red[0]);
    res[p + i] = th;
    if (i == 0) {
      int* flags = (int*)(res + 2 * p);
      flags[0] = *dinfo;
      flags[1] = fail[0];
      flags[2] = fail[1];
      fail[1] = 0;
    }
  }
}

// K chunk of the block products V M (p x n times n x n) that go by 64 x 64 tiles:
// enough partial products for about 1024 workgroups (at least 4, at most
// 16), so that p = 128, n = 4096 takes 8 x 2 x 64 (four workgroups per CU
// hide each other's slab loads: 2% less eigensolver time than 4 x 2 x 64)
static inline int vm_chunk(int n, int p) {
  const int tiles = ((p + 63) / 64) * ((n + 63) / 64);
  const int parts = std::min(16, std::max(4, (1024 + tiles - 1) / tiles));
  return ((n + parts - 1) / parts + 15) / 16 * 16;
}

static inline size_t partial_doubles(int n, int p) {
  if (block_product_small(p, n)) return 0;
  return (size_t)((n + vm_chunk(n, p) - 1) / vm_chunk(n, p)) * p * n;
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
// The sweeps between the first and the last of a group orthonormalise after every
// second product where theta_1 / theta_p of the last Rayleigh-Ritz step (*cond, 0:
// none) is at most 1e8: rounding leaves a row that should hold the eigenvalue
// lambda a part u of the leading vector, two products make it u (theta_1 / lambda)^2
// of the row, and up to 1 the next orthonormalisation takes it out without loss.
// 24 steps at D = 32: 40.1 -> 39.4 ms, two-sided Potts steps 14.8 -> 14.0 (after every
// third or fourth product, where the ratio allows it, 40.5 and 14.3: the checks then
// find work to do).
// Every Rayleigh-Ritz step still sees a basis from three passes, and its
// residuals decide convergence.
// Two products leave Gram entries of theta^4: theta_1 within kPairRange keeps them
// (theta_p^4 too) inside the range of doubles; past it every product is orthonormalised.
constexpr double kPairCond = 1e8, kPairRange = 0x1p200;

bool topk_eigs(const double* M, int n, int p, int need, double tol,
               int q_first, double* shift, int* nocheck, double* cond, double* ws, double* W,
               double* Xout, int* dinfo, int* iters, int* enough, double* resid, hipStream_t s) {
  const size_t pn = (size_t)p * n, pp = (size_t)p * p;
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
  double* res = E + pp;        // p, the host's copy of the eigenvalues (p) and flags (2)
  int* fail = (int*)(res + 2 * p + 2);  // fail flag, then the count of checks that missed
  // a pass's Cholesky factor (p x p) at Rt and its row scaling (p) in the
  // first p entries of H, which only the Rayleigh-Ritz step uses
  double* Rf = Rt;
  const double u = std::ldexp(1.0, -53);
  const double shift_rel = 11.0 * ((double)n * p + (double)p * (p + 1)) * u;

  const size_t trsm_lds = (size_t)p * p * sizeof(double);
  if (!trsm_lds_set() || p > 128 || p % 16 != 0) return false;
  hipLaunchKernelGGL(k_seed_block, dim3(256), dim3(256), 0, s, V, (long long)pn, 12345ULL, fail);

  // one orthonormalisation of rows of Y into V: shifted Cholesky-QR of the
  // column-scaled Gram matrix twice, then a plain pass -- all three before a
  // Rayleigh-Ritz check (`full`); between checks only the first two, the
  // second skipped on the device (R^-1 = I) when its Gram matrix is the
  // identity to 1e-2.
  auto orth = [&](const double* Yin, double* Vout, bool full, bool check) {
    const double* src = Yin;
    const int last = full ? 2 : (check ? 1 : 0);
    for (int pass = 0; pass <= last; ++pass) {
      gemm_f64_symmetric(src, src, n, G, p, n, SYM_UPPER, s);
      const double sh = pass < 2 ? shift_rel : 0.0, itol = (pass == 0 || full) ? 0.0 : 1e-2;
      if (p <= 64)
        hipLaunchKernelGGL(k_chol_factor<4>, dim3(1), dim3(256), 0, s, G, p, sh,
                           pass < 2 ? 1 : 0, itol, Rf, fail, fail + 1);
      else
        hipLaunchKernelGGL(k_chol_factor<8>, dim3(1), dim3(512), 0, s, G, p, sh,
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
    gemm_f64_block(Vin, M, Yout, p, n, sg, kv, part, s);
  };

  int it = 0, q = q_first > 0 ? q_first : 3;
  const int max_it = 80;
  double prev = 1e300;
  std::vector<double> host(2 * p + 2);
  while (true) {
    const bool skip = nocheck && *nocheck;
    const bool pairs = cond && *cond > 0.0 && *cond <= kPairCond;
    for (int r = 0; r < q;) {
      const bool two = pairs && r > 0 && r + 2 < q;
      vm(V, Y, sigma);
      if (two) vm(Y, T2, sigma);
      const bool check = r == 0 || (two && r == 1) || !skip;
      r += two ? 2 : 1;
      it += two ? 2 : 1;
      orth(two ? T2 : Y, V, r == q, check);
    }
    // Rayleigh-Ritz
    vm(V, Y, 0.0);
    gemm_f64_symmetric(V, Y, n, H, p, n, SYM_BOTH, s);
    // tridiagonal form and its reflectors (over H), then divide and conquer
    // on the tridiagonal (Z^T into Rt, eigenvalues over its diagonal in W),
    // then the rows of Rt back to H's basis: the Ritz coefficients
    launch_sytrd(H, p, W, E, s);
    if (!tridiag_eig_small(W, E, p, W, Rt, dinfo, s)) return false;
    if (!launch_backtransform(H, p, Rt, 0, p, Rt, s)) return false;
    gemm_f64_two(Rt, p, V, Y, n, Xout, Yx, p, n, p, s);
    hipLaunchKernelGGL(k_ritz_residual, dim3(p), dim3(256), 0, s, Yx, Xout, W, n, res, p, dinfo,
                       fail);
    // everything the host decides by in one copy: four cost 30 us more a step
    (void)hipMemcpyAsync(host.data(), res, (2 * p + 2) * sizeof(double), hipMemcpyDeviceToHost, s);
    if (hipStreamSynchronize(s) != hipSuccess) return false;
    const double *rs = host.data(), *th = rs + p;
    int hinfo[3];
    std::memcpy(hinfo, th + p, sizeof hinfo);
    if (hinfo[0] != 0 || hinfo[1] != 0) return false;
    if (nocheck) *nocheck = hinfo[2] == 0 ? 1 : 0;
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
    if (cond) *cond = lo > 0.0 && t1 <= kPairRange && t1 >= 1.0 / kPairRange ? t1 / lo : 0.0;
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
