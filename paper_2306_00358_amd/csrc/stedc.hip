// Eigenvalues and eigenvectors of a small symmetric tridiagonal matrix (the
// Rayleigh-Ritz matrix of the block eigensolver after Householder reduction,
// n <= 128) by divide and conquer, in one workgroup.
//
// Method (Cuppen's divide and conquer with the deflation and the
// eigenvector formula of Gu and Eisenstat).  Index range [a, b) splits at c
// into [a, c) and [c, b); with beta = e[c-1],
//   T = diag(T1', T2') + |beta| v v^T,  v = e_{c-1} + sign(beta) e_c,
// where T1' and T2' have |beta| taken off their diagonal entries c-1 and c.
// The tree halves every range down to leaves of at most 8 indices, so the
// diagonal entries at a leaf's ends lose the moduli of the off-diagonal
// entries that leave it up front.  The leaves are diagonalised by cyclic
// Jacobi sweeps, 8 lanes per leaf, all leaves at once.  A merge, given the children's eigenpairs (Z1, L1), (Z2,
// L2), solves diag(L1, L2) + rho z z^T with z = (last row of Z1,
// sign(beta) first row of Z2) / |.|, rho = |beta| |z|^2:
//   * deflation, scanning the poles in ascending order: a component with
//     rho |z_i| <= tol leaves (d_i, its column) unchanged; two poles closer
//     than tol after the rotation that zeroes one z component are rotated
//     (columns of Z too) and the zeroed one leaves;
//     tol = 8 u max(max |d|, rho);
//   * each remaining root lam_j of 1/rho + sum_i z_i^2 / (d_i - lam) = 0 lies
//     in (d_j, d_{j+1}) (the last in (d_K, d_K + rho |z|^2]) and is stored as
//     lam_j = d_o + tau_j with the nearer pole o as origin, so that every
//     d_i - lam_j = (d_i - d_o) - tau_j is accurate; tau comes from a
//     safeguarded iteration on a two-pole rational model of the secular
//     function (value and slope of the parts left and right of the root);
//   * z is recomputed from the roots (Gu-Eisenstat),
//     z_i^2 = (lam_i - d_i) / rho * prod_{j != i} (d_i - lam_j) / (d_i - d_j),
//     with the sign of the original z_i, so that the vectors
//     u_j = (z_i / (d_i - lam_j))_i / |.| are orthogonal to working accuracy;
//   * the merged block of Z becomes Z [u_1 .. u_K] in the columns of the
//     remaining poles (MFMA, v_mfma_f64_16x16x4f64, the u entries formed as
//     B operands), deflated columns staying where they are.
// All merges of one tree level run together.  Eigenvalues leave ascending (ties
// by index) in W and the eigenvectors as rows of Zt (row c = eigenvector of
// W[c]); info = 1 when a result is not finite.
//
// What bounds it is instruction issue and latency on one compute unit: the
// secular iterations (half of the time) and a fixed cost per level.  So: the
// three lowest levels are one Jacobi solve, 4 lanes per root and as many waves
// as that takes (4 up to n = 64, 8 above: barriers over 16 waves cost 467
// cycles), the sums over the poles left and right of a root in loops of their
// own, reciprocals by v_rcp_f64 and Newton steps instead of divisions, the
// deflation decided for all poles of a merge at once (only poles that do
// rotate are walked serially), an index's merge looked up once per level, and
// in the products the u entries of a column tile formed once for all its row
// tiles and the poles ordered by child, so that a row tile takes only those
// its rows have entries in.  Barriers order LDS only.
// n = 64: 107 -> 79 us, n = 128: 240 -> 152 us (1024 threads with 8 lanes per root,
// leaves of one index, a serial scan, every product over all poles).
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "internal.h"

namespace hotrg {

constexpr int kDcMax = 128;
constexpr int kDcLd = kDcMax + 1;  // row stride of Z in LDS (padded against bank conflicts)

typedef double dc4 __attribute__((ext_vector_type(4)));
typedef double dc2 __attribute__((ext_vector_type(2)));

// value of another lane of the same 4-lane group (DPP: quad_perm [1,0,3,2],
// quad_perm [2,3,0,1]); every lane of the group is active
template <int kCtrl>
__device__ __forceinline__ double dc_dpp(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, kCtrl, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), kCtrl, 0xF, 0xF, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// sum / product / maximum over a 4-lane group, the same bits in every lane
__device__ __forceinline__ double dc_sum4(double v) {
  v += dc_dpp<0xB1>(v);
  return v + dc_dpp<0x4E>(v);
}

__device__ __forceinline__ double dc_prod4(double v) {
  v *= dc_dpp<0xB1>(v);
  return v * dc_dpp<0x4E>(v);
}

__device__ __forceinline__ double dc_max4(double v) {
  v = fmax(v, dc_dpp<0xB1>(v));
  return fmax(v, dc_dpp<0x4E>(v));
}

// 1 / x: v_rcp_f64 refined by two Newton steps
__device__ __forceinline__ double dc_rcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = fma(-x, r, 1.0);
  r = fma(r, e, r);
  e = fma(-x, r, 1.0);
  return fma(r, e, r);
}

// estimates for the steps of the secular iteration (which its own test of the
// secular function accepts or not): 1 / x and sqrt(x), one Newton step each
__device__ __forceinline__ double dc_rcp1(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  return fma(r, fma(-x, r, 1.0), r);
}

__device__ __forceinline__ double dc_sqrt1(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double s = x * y;
  return x > 0.0 ? fma(0.5 * y, fma(-s, s, x), s) : 0.0;
}

// lane ^ M of the same 8-lane group (DPP: quad_perm, row_half_mirror = ^ 7)
template <int M>
__device__ __forceinline__ double dc_xor(double v) {
  if constexpr (M == 1) return dc_dpp<0xB1>(v);
  if constexpr (M == 2) return dc_dpp<0x4E>(v);
  if constexpr (M == 3) return dc_dpp<0x1B>(v);
  if constexpr (M == 7) return dc_dpp<0x141>(v);
  if constexpr (M > 3 && M < 7) return dc_dpp<0x141>(dc_xor<7 - M>(v));
  return v;
}

// One round of a cyclic Jacobi sweep on a symmetric 8 x 8 matrix held by 8
// lanes: lane u has b[k] = A[u ^ k][u] and the eigenvector columns v[k] =
// V[u ^ k][u].  The pairs of the round are (u, u ^ M).  In these coordinates
// a column rotation combines b[k] with the partner lane's b[k ^ M], a row
// rotation b[k] with b[k ^ M] of the same lane (with lane u ^ k's angle), all
// register indices fixed.  Both lanes of a pair form the angle from the same
// bits (the difference of the diagonals negated), so their c agree and their
// s are exact negatives.
template <int M>
__device__ __forceinline__ void dc_jacobi_round(double (&b)[8], double (&v)[8], int u) {
  const double apq = 0.5 * (b[M] + dc_xor<M>(b[M]));
  double h = dc_xor<M>(b[0]) - b[0], g = 2.0 * apq;
  if (fmax(fabs(h), fabs(g)) < 0x1p-400) {  // the angle does not depend on the scale
    h *= 0x1p500;
    g *= 0x1p500;
  }
  const double x = fma(h, h, g * g);
  double y = __builtin_amdgcn_rsq(x);
  y = fma(y, fma(-0.5 * x * y, y, 0.5), y);
  y = fma(y, fma(-0.5 * x * y, y, 0.5), y);
  double t = g * dc_rcp(fma(x, y, fabs(h)));
  // sign(h); at h = 0 the pair's lower lane takes +
  constexpr int hb = M >= 4 ? 4 : (M >= 2 ? 2 : 1);
  const bool neg = h < 0.0 || (h == 0.0 && (u & hb));
  t = neg ? -t : t;
  t = x > 0.0 && g != 0.0 ? t : 0.0;
  const double x1 = fma(t, t, 1.0);
  double c = __builtin_amdgcn_rsq(x1);
  c = fma(c, fma(-0.5 * x1 * c, c, 0.5), c);
  c = fma(c, fma(-0.5 * x1 * c, c, 0.5), c);
  const double s = t * c, diag = fma(-t, apq, b[0]);
  double n[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) n[k] = fma(c, b[k], -s * dc_xor<M>(b[k ^ M]));
  auto rows = [&](auto kc) {
    constexpr int k = decltype(kc)::value;
    if constexpr ((k ^ M) > k) {
      const double ck = dc_xor<k>(c), sk = dc_xor<k>(s);
      b[k] = fma(ck, n[k], -sk * n[k ^ M]);
      b[k ^ M] = fma(ck, n[k ^ M], sk * n[k]);
    }
  };
  rows(std::integral_constant<int, 0>{});
  rows(std::integral_constant<int, 1>{});
  rows(std::integral_constant<int, 2>{});
  rows(std::integral_constant<int, 3>{});
  rows(std::integral_constant<int, 4>{});
  rows(std::integral_constant<int, 5>{});
  rows(std::integral_constant<int, 6>{});
  b[0] = diag;
  b[M] = 0.0;
#pragma unroll
  for (int k = 0; k < 8; ++k) n[k] = fma(c, v[k], -s * dc_xor<M>(v[k ^ M]));
#pragma unroll
  for (int k = 0; k < 8; ++k) v[k] = n[k];
}

// node k of tree level D over n indices: [(k n) >> D, ((k + 1) n) >> D)
struct DcMerge {
  int a, b, c;
  bool real;  // both children non-empty
};

// the node of index s; magic = ceil(2^22 / n) (the quotient (((s + 1) << D) - 1) / n is
// exact: its numerator is below 2^15 and n <= 128)
__device__ __forceinline__ DcMerge dc_merge_of(int s, int D, int n, unsigned magic) {
  const int k = (int)(((unsigned)(((s + 1) << D) - 1) * magic) >> 22);
  DcMerge m;
  m.a = (k * n) >> D;
  m.b = ((k + 1) * n) >> D;
  m.c = ((2 * k + 1) * n) >> (D + 1);
  m.real = m.c > m.a && m.c < m.b;
  return m;
}

// bits [lo, hi) of a 128-bit mask in two words
__device__ __forceinline__ void dc_range(const unsigned long long* m, int lo, int hi,
                                         unsigned long long& w0, unsigned long long& w1) {
  auto below = [](int x) { return x >= 64 ? ~0ull : (x <= 0 ? 0ull : (1ull << x) - 1); };
  w0 = m[0] & below(hi) & ~below(lo);
  w1 = m[1] & below(hi - 64) & ~below(lo - 64);
}

// din may be W: it is read before the second barrier and W written after the
// last.  NT threads: 256 for n <= 64, 512 up to 128.
template <int NT>
__device__ __forceinline__ void stedc_body(const double* din, const double* ein, int n, double* W,
                                           double* __restrict__ Zt, int* __restrict__ info) {
  constexpr int NW = NT / 64, N = NT / 4;  // waves, largest n
  constexpr int S = 8;                     // product tiles per wave and level, at most
  extern __shared__ double Z[];            // n rows of kDcLd: Z[r * kDcLd + c]
  __shared__ double lam[N], e[N], zv[N];
  __shared__ double sd[N], sz[N];
  __shared__ __attribute__((aligned(16))) dc2 dz[N];  // remaining poles: d, z
  __shared__ __attribute__((aligned(16))) dc2 ot[N];  // roots: origin pole's d, tau
  __shared__ double zt[N], inrm[N];
  __shared__ double rc[N], rs[N];
  __shared__ double mrho[N], mtol[N], msc[N];
  __shared__ int scol[N], ndc[N], rp[N], rq[N];
  __shared__ int kcnt[N], rcnt[N], ord[N];
  __shared__ unsigned long long alive[2], trig[2], side1[2], side2[2];
  __shared__ int mixed[N], lst[N], cn1[N], cn2[N];
  __shared__ int tiles[64];
  __shared__ int ntiles, bad;
  const int t = threadIdx.x, lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const double eps = 1.1102230246251565e-16;  // 2^-53
  const unsigned magic = ((1u << 22) + n - 1) / n;

  int L = 0;
  while ((1 << L) < n) ++L;
  const int DL = L > 3 ? L - 3 : 0;  // level of the leaves (at most 8 indices each)

  for (int r = w; r < n; r += NW)
    for (int c = lane; c < n; c += 64) Z[r * kDcLd + c] = 0.0;
  if (t < n) {
    e[t] = t < n - 1 ? ein[t] : 0.0;
    // a pole that is not a number has no rank, and the place that it leaves in an order
    // is not written: it holds an index of the range all the same, never what LDS held
    scol[t] = 0;
    ord[t] = t;
  }
  if (t == 0) bad = 0;
  if (t < 2) alive[t] = trig[t] = 0;
  // leaf t / 8 (the lanes past the last leaf carry zeros)
  const int u8 = t & 7, leaf = t >> 3;
  int la = 0, ls = 0;
  double jb[8], jv[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    jb[k] = 0.0;
    jv[k] = k == 0 ? 1.0 : 0.0;
  }
  if (leaf < (1 << DL)) {
    la = (leaf * n) >> DL;
    ls = (((leaf + 1) * n) >> DL) - la;
    if (u8 < ls) {
      const int i = la + u8;
      double dv = din[i];
      if (u8 == 0 && i > 0) dv -= fabs(ein[i - 1]);
      if (u8 == ls - 1 && i < n - 1) dv -= fabs(ein[i]);
      const double el = u8 > 0 ? ein[i - 1] : 0.0, er = u8 < ls - 1 ? ein[i] : 0.0;
      jb[0] = dv;
#pragma unroll
      for (int k = 1; k < 8; ++k) jb[k] = (u8 ^ k) == u8 - 1 ? el : ((u8 ^ k) == u8 + 1 ? er : 0.0);
    }
  }
  lds_barrier();
  if (const int i = NT - 1 - t; i < n && !(fabs(din[i]) < INFINITY && fabs(e[i]) < INFINITY))
    bad = 1;  // (found by the last waves, beside the leaves)
  if (w * 8 < (1 << DL)) {  // uniform
    for (int it = 0; it < 12; ++it) {
      double off = 0.0, nrm = fabs(jb[0]);
#pragma unroll
      for (int k = 1; k < 8; ++k) off = fmax(off, fabs(jb[k]));
      off = fmax(off, dc_xor<1>(off));
      off = fmax(off, dc_xor<2>(off));
      off = fmax(off, dc_xor<7>(off));
      nrm = fmax(nrm, dc_xor<1>(nrm));
      nrm = fmax(nrm, dc_xor<2>(nrm));
      nrm = fmax(nrm, dc_xor<7>(nrm));
      // off-diagonal entries below a quarter unit of the leaf's norm stay
      if (!__any(off > 0.25 * eps * fmax(nrm, off))) break;
      dc_jacobi_round<1>(jb, jv, u8);
      dc_jacobi_round<2>(jb, jv, u8);
      dc_jacobi_round<3>(jb, jv, u8);
      dc_jacobi_round<4>(jb, jv, u8);
      dc_jacobi_round<5>(jb, jv, u8);
      dc_jacobi_round<6>(jb, jv, u8);
      dc_jacobi_round<7>(jb, jv, u8);
    }
    if (u8 < ls) {
      lam[la + u8] = jb[0];
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if ((u8 ^ k) < ls) Z[(la + (u8 ^ k)) * kDcLd + la + u8] = jv[k];
    }
  }
  lds_barrier();

  const int gs = t >> 2, u = t & 3;  // the index of this 4-lane group, its lane
  for (int D = DL - 1; D >= 0; --D) {
    const DcMerge g1 = dc_merge_of(t < n ? t : 0, D, n, magic);    // of index t
    const DcMerge g4 = dc_merge_of(gs < n ? gs : 0, D, n, magic);  // of index gs
    const bool on1 = t < n && g1.real, on4 = gs < n && g4.real;
    // (A) the coupling vector z of each merge, by column
    if (on1) {
      const double sg = e[g1.c - 1] < 0.0 ? -1.0 : 1.0;
      zv[t] = t < g1.c ? Z[(g1.c - 1) * kDcLd + t] : sg * Z[g1.c * kDcLd + t];
    }
    lds_barrier();
    // poles of each merge in ascending order (ties by column), 4 lanes per
    // index; the first index of a merge also forms |z|, rho and tol
    if (on4) {
      const double lv = lam[gs];
      int rk = 0;
#pragma unroll 4
      for (int i = g4.a + u; i < g4.b; i += 4) {
        const double li = lam[i];
        rk += (li < lv || (li == lv && i < gs)) ? 1 : 0;
      }
      rk += __builtin_amdgcn_update_dpp(0, rk, 0xB1, 0xF, 0xF, false);
      rk += __builtin_amdgcn_update_dpp(0, rk, 0x4E, 0xF, 0xF, false);
      if (u == 0) {
        sd[g4.a + rk] = lv;
        sz[g4.a + rk] = zv[gs];
        scol[g4.a + rk] = gs - g4.a;
      }
      if (gs == g4.a) {
        double s2 = 0.0, dmax = 0.0;
#pragma unroll 4
        for (int i = g4.a + u; i < g4.b; i += 4) {
          s2 += zv[i] * zv[i];
          dmax = fmax(dmax, fabs(lam[i]));
        }
        s2 = dc_sum4(s2);
        dmax = dc_max4(dmax);
        if (u == 0) {
          const double rho = fabs(e[g4.c - 1]) * s2;
          mrho[g4.a] = rho;
          msc[g4.a] = s2 > 0.0 ? 1.0 / sqrt(s2) : 0.0;
          mtol[g4.a] = 8.0 * eps * fmax(dmax, rho);
        }
      }
    }
    lds_barrier();
    // (B) deflation, position t of the ascending order: small components
    // leave at once; of the others (alive), those that would rotate with the
    // alive one before (trig) are found assuming nothing rotated before them
    double dv = 0.0, zs = 0.0;
    int col = 0;
    bool al = false;
    if (on1) {
      dv = sd[t];
      zs = sz[t] * msc[g1.a];
      col = scol[t];
      al = mrho[g1.a] * fabs(zs) > mtol[g1.a];
      sz[t] = zs;
      if (!al) lam[g1.a + col] = dv;
      mixed[t] = 0;  // column t: a rotation has given it entries of both children
    }
    if (w < 2 && w * 64 < N) {
      const unsigned long long m = __ballot(al);
      if (lane == 0) alive[w] = m;
    }
    lds_barrier();
    {
      bool tr = false;
      if (al) {
        unsigned long long w0, w1;
        dc_range(alive, g1.a, t, w0, w1);
        if (w0 | w1) {
          const int pv = w1 ? 127 - __clzll((long long)w1) : 63 - __clzll((long long)w0);
          const double pd = sd[pv], pz = sz[pv];
          tr = fabs(dv - pd) * fabs(pz * zs) <= mtol[g1.a] * (pz * pz + zs * zs);
        }
      }
      if (w < 2 && w * 64 < N) {
        const unsigned long long m = __ballot(tr);
        if (lane == 0) trig[w] = m;
      }
    }
    lds_barrier();
    // the rotations of a merge, one thread: from each triggering pole on,
    // the alive poles in order as long as they rotate (a rotated pole's new
    // d and z meet the next one's test); the zeroed pole of a pair leaves
    if (on1 && t == g1.a) {
      const int a = g1.a;
      const double tol = mtol[a];
      int R = 0;
      unsigned long long t0, t1, a0, a1;
      dc_range(trig, a, g1.b, t0, t1);
      dc_range(alive, a, g1.b, a0, a1);
      while (t0 | t1) {
        int s = t0 ? __ffsll((long long)t0) - 1 : 63 + __ffsll((long long)t1);
        int pv;
        {
          unsigned long long w0, w1;
          const unsigned long long av[2] = {a0, a1};
          dc_range(av, a, s, w0, w1);
          pv = w1 ? 127 - __clzll((long long)w1) : 63 - __clzll((long long)w0);
        }
        double pd = sd[pv], pz = sz[pv];
        bool go = true;
        while (go) {
          // pv and s rotate: pv leaves, s takes the joint component
          const double sv = sd[s], sw = sz[s];
          const double r = sqrt(pz * pz + sw * sw);
          const double cth = sw / r, sth = -pz / r;
          rp[a + R] = scol[pv];
          rq[a + R] = scol[s];
          rc[a + R] = cth;
          rs[a + R] = sth;
          if (mixed[a + scol[pv]] || mixed[a + scol[s]] ||
              (a + scol[pv] < g1.c) != (a + scol[s] < g1.c))
            mixed[a + scol[s]] = 1;
          ++R;
          lam[a + scol[pv]] = pd * cth * cth + sv * sth * sth;
          pd = pd * sth * sth + sv * cth * cth;
          pz = r;
          sd[s] = pd;
          sz[s] = pz;
          if (pv < 64) a0 &= ~(1ull << pv); else a1 &= ~(1ull << (pv - 64));
          if (s < 64) t0 &= ~(1ull << s); else t1 &= ~(1ull << (s - 64));
          pv = s;
          // the next alive pole against the rotated one
          unsigned long long w0, w1;
          const unsigned long long av[2] = {a0, a1};
          dc_range(av, s + 1, g1.b, w0, w1);
          go = false;
          if (w0 | w1) {
            s = w0 ? __ffsll((long long)w0) - 1 : 63 + __ffsll((long long)w1);
            const double nv = sd[s], nw = sz[s];
            go = fabs(nv - pd) * fabs(pz * nw) <= tol * (pz * pz + nw * nw);
            // decided here, whatever the test against the unrotated pole said
            if (s < 64) t0 &= ~(1ull << s); else t1 &= ~(1ull << (s - 64));
          }
        }
      }
      rcnt[a] = R;
      if (R > 0) {
        // other merges' bits share the words
        unsigned long long o0, o1;
        dc_range(alive, a, g1.b, o0, o1);
        if (o0 != a0) atomicAnd(&alive[0], ~(o0 & ~a0));
        if (o1 != a1) atomicAnd(&alive[1], ~(o1 & ~a1));
      }
      kcnt[a] = __popcll(a0) + __popcll(a1);
    }
    lds_barrier();
    // the remaining poles in order; (C) the deflating rotations on the rows of
    // each merged block; one wave lists the product tiles of the level
    // (the poles whose columns are of the first child only, and of the second)
    int pos = -1;
    bool in1 = false, in2 = false;
    if (on1 && ((alive[t >> 6] >> (t & 63)) & 1)) {
      unsigned long long w0, w1;
      dc_range(alive, g1.a, t, w0, w1);
      pos = __popcll(w0) + __popcll(w1);
      ndc[g1.a + pos] = col;
      dz[g1.a + pos] = dc2{sd[t], sz[t]};
      const bool mx = mixed[g1.a + col] != 0;
      in1 = !mx && g1.a + col < g1.c;
      in2 = !mx && g1.a + col >= g1.c;
    }
    if (w < 2 && w * 64 < N) {
      const unsigned long long m1 = __ballot(in1), m2 = __ballot(in2);
      if (lane == 0) {
        side1[w] = m1;
        side2[w] = m2;
      }
    }
    if (on1) {
      const int R = rcnt[g1.a];
      double* zr = Z + t * kDcLd + g1.a;
      for (int q = 0; q < R; ++q) {
        const int x = rp[g1.a + q], y = rq[g1.a + q];
        const double cq = rc[g1.a + q], sq = rs[g1.a + q];
        const double zx = zr[x], zy = zr[y];
        zr[x] = cq * zx + sq * zy;
        zr[y] = -sq * zx + cq * zy;
      }
    }
    if (w == NW - 1) {
      // lane k lists merge k's tiles (at most 64 merges, 64 tiles a level),
      // the row tiles of a column tile one after another
      const int k = lane;
      int cnt = 0, a = 0, rts = 1;
      if (k < (1 << D)) {
        a = (k * n) >> D;
        const int b = ((k + 1) * n) >> D, c = ((2 * k + 1) * n) >> (D + 1);
        if (c > a && c < b) {
          rts = (b - a + 15) / 16;
          cnt = rts * ((kcnt[a] + 15) / 16);
        }
      }
      int x = cnt;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(x, o, 64);
        if (k >= o) x += y;
      }
      for (int q = 0; q < cnt; ++q) tiles[x - cnt + q] = a | ((q % rts) << 8) | ((q / rts) << 12);
      if (k == 63) ntiles = x;
    }
    lds_barrier();
    // product order of a merge's poles: the first child's, the mixed ones, the
    // second child's
    if (on1) {
      const int a = g1.a;
      unsigned long long w0, w1, x0, x1;
      dc_range(side1, a, g1.b, w0, w1);
      dc_range(side2, a, g1.b, x0, x1);
      const int n1 = __popcll(w0) + __popcll(w1), n2 = __popcll(x0) + __popcll(x1);
      if (t == a) {
        cn1[a] = n1;
        cn2[a] = n2;
      }
      if (pos >= 0) {
        dc_range(side1, a, t, w0, w1);
        dc_range(side2, a, t, x0, x1);
        const int b1 = __popcll(w0) + __popcll(w1), b2 = __popcll(x0) + __popcll(x1);
        lst[a + (in1 ? b1 : (in2 ? kcnt[a] - n2 + b2 : n1 + pos - b1 - b2))] = pos;
      }
    }
    // (D) secular roots, 4 lanes per root
    const int a4 = g4.a, K = on4 ? kcnt[a4] : 0, j = gs - a4;
    const bool root = on4 && j < K;
    if (root) {
      const double rinv = 1.0 / mrho[a4];
      // sums of the secular function and of its slope over the poles left
      // (negative terms) and right of the root at tv, in the frame of origin org
      double psi = 0.0, dpsi = 0.0, phi = 0.0, dphi = 0.0;
      auto sums = [&](double org, double tv) {
        psi = dpsi = phi = dphi = 0.0;
        for (int i0 = 0; i0 < K; i0 += 16) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int i = i0 + 4 * q + u;
            const dc2 p = dz[a4 + (i < K ? i : j)];
            const double zq = i < K ? p.y : 0.0;
            // the terms left of the root are negative, those right of it positive
            const double r = zq * dc_rcp((p.x - org) - tv);
            const double f = zq * r, g = copysign(r * r, f);
            psi += fmin(f, 0.0);
            dpsi -= fmin(g, 0.0);
            phi += fmax(f, 0.0);
            dphi += fmax(g, 0.0);
          }
        }
        psi = dc_sum4(psi);
        dpsi = dc_sum4(dpsi);
        phi = dc_sum4(phi);
        dphi = dc_sum4(dphi);
      };
      const double dj = dz[a4 + j].x;
      int o;
      double lo, hi, tv, gap = 0.0;
      bool have = false;
      if (j < K - 1) {
        // the sign at the midpoint of (d_j, d_j+1) picks the nearer pole as
        // origin; the sums there start the iteration
        gap = dz[a4 + j + 1].x - dj;
        const double mid = 0.5 * gap;
        sums(dj, mid);
        have = true;
        if (rinv + psi + phi >= 0.0) {
          o = j;
          lo = 0.0;
          hi = mid;
          tv = mid;
        } else {
          o = j + 1;
          lo = -(gap - mid);
          hi = 0.0;
          tv = lo;
        }
      } else {
        double s2 = 0.0;
        for (int i = u; i < K; i += 4) s2 += dz[a4 + i].y * dz[a4 + i].y;
        o = K - 1;
        lo = 0.0;
        hi = mrho[a4] * dc_sum4(s2);
        tv = 0.5 * hi;
      }
      const double org = dz[a4 + o].x;
      const double oj = dj - org, oj1 = j < K - 1 ? dz[a4 + j + 1].x - org : 0.0;
      for (int it = 0; it < 80; ++it) {
        if (!have) sums(org, tv);
        have = false;
        const double f = rinv + psi + phi;
        if (!(fabs(f) < INFINITY)) {
          if (u == 0) bad = 1;
          break;
        }
        const double err = 8.0 * (fabs(psi) + fabs(phi) + rinv) + fabs(tv) * (dpsi + dphi);
        if (fabs(f) <= 4.0 * eps * err) break;
        if (f > 0.0)
          hi = fmin(hi, tv);
        else
          lo = fmax(lo, tv);
        // two-pole model f(tv + eta) ~ cf + s / (Dj - eta) + S / (Dj1 - eta)
        double eta;
        const double Dj = oj - tv;
        if (j < K - 1) {
          const double Dj1 = oj1 - tv;
          const double s = dpsi * Dj * Dj, S2 = dphi * Dj1 * Dj1;
          const double cf = f - dpsi * Dj - dphi * Dj1;
          const double qb = -(cf * (Dj + Dj1) + s + S2);
          const double qc = cf * Dj * Dj1 + s * Dj1 + S2 * Dj;
          const double sq = dc_sqrt1(fmax(qb * qb - 4.0 * cf * qc, 0.0));
          const double qq = -0.5 * (qb + copysign(sq, qb));
          // an infinite or NaN candidate is never inside (lo, hi)
          const double r1 = qq * dc_rcp1(cf), r2 = qc * dc_rcp1(qq);
          const bool in1 = tv + r1 > lo && tv + r1 < hi;
          const bool in2 = tv + r2 > lo && tv + r2 < hi;
          eta = in2 ? r2 : NAN;
          if (in1 && !(in2 && fabs(r2) <= fabs(r1))) eta = r1;
        } else {
          const double s = dpsi * Dj * Dj, cf = f - dpsi * Dj;
          eta = Dj + s * dc_rcp1(cf);
        }
        double nt = tv + eta;
        if (!(nt > lo && nt < hi)) nt = 0.5 * (lo + hi);
        if (nt == tv) break;
        // a step of relative size 2^-28 of the distance to the nearer pole
        // leaves a remainder of about its square: no need to look again
        const bool last = fabs(nt - tv) <= 0x1p-28 * fabs(nt);
        tv = nt;
        if (last) break;
      }
      if (u == 0) ot[gs] = dc2{org, tv};
    }
    lds_barrier();
    // (E) z recomputed from the roots
    if (root) {
      const dc2 pi = dz[a4 + j];
      double pr = 1.0;
#pragma unroll 4
      for (int i = u; i < K; i += 4) {
        const dc2 o = ot[a4 + i];
        const double dl = (pi.x - o.x) - o.y;
        const double den = i == j ? -mrho[a4] : pi.x - dz[a4 + i].x;
        pr *= dl * dc_rcp(den);
      }
      pr = dc_prod4(pr);
      if (u == 0) zt[gs] = copysign(sqrt(fmax(pr, 0.0)), pi.y);
    }
    lds_barrier();
    // (F) norms of the vectors (z_i / (d_i - lam_j))_i
    if (root) {
      const dc2 o = ot[gs];
      double s2 = 0.0;
#pragma unroll 4
      for (int i = u; i < K; i += 4) {
        const double q = zt[a4 + i] * dc_rcp((dz[a4 + i].x - o.x) - o.y);
        s2 += q * q;
      }
      s2 = dc_sum4(s2);
      if (u == 0) inrm[gs] = 1.0 / sqrt(s2);
    }
    lds_barrier();
    // (G) Z block <- Z block [u_1 .. u_K] in the remaining poles' columns: wave
    // w takes `per` consecutive tiles of the list, in runs of one column tile
    // whose u entries (B operands) are formed once for the run
    {
      const int li = lane & 15, lk = lane >> 4;
      const int nt = ntiles, rt0 = (((n + (1 << D) - 1) >> D) + 15) / 16;
      const int cols = (nt + rt0 - 1) / rt0;
      int per = rt0 * ((cols + NW - 1) / NW);
      if (per > S || per * NW < nt) per = (nt + NW - 1) / NW;
      dc4 acc[S];
      int tl[S];
#pragma unroll
      for (int q = 0; q < S; ++q) {
        const int ti = w * per + q;
        tl[q] = __builtin_amdgcn_readfirstlane(q < per && ti < nt ? tiles[ti] : -1);
        acc[q] = dc4{0.0, 0.0, 0.0, 0.0};
      }
#pragma unroll
      for (int q = 0; q < S; ++q) {
        if (tl[q] < 0 || (q > 0 && (tl[q] & ~0xf00) == (tl[q > 0 ? q - 1 : 0] & ~0xf00)))
          continue;  // none, or inside a run (uniform)
        const int a = tl[q] & 255, ct = (tl[q] >> 12) & 15;
        const int Ka = kcnt[a], jj = 16 * ct + li;
        const DcMerge g = dc_merge_of(a, D, n, magic);
        dc2 oj = dc2{0.0, 0.0};
        double nj = 0.0;
        if (jj < Ka) {
          oj = ot[a + jj];
          nj = inrm[a + jj];
        }
        // a tile's rows lie in the first child, the second or both: it needs the
        // poles [0, K - n2), [n1, K) or all of the product order
        const int n1 = cn1[a], e1 = Ka - cn2[a];
        // (the operands of the next steps are loaded ahead of this step's products)
        const int steps = (Ka + 3) / 4;
        auto pole = [&](int kk) {
          const int i = 4 * min(kk, steps - 1) + lk;
          return a + (i < Ka ? lst[a + i] : 0);
        };
        const double* zrow[S];  // this lane's row of each tile of the run
        bool rok[S];
        int lo[S], hi[S];       // the steps the tile takes
        int run = q;
#pragma unroll
        for (int x = q; x < S; ++x) {
          if (run < x || tl[x] < 0 || (tl[x] & ~0xf00) != (tl[q] & ~0xf00)) {
            lo[x] = steps;
            hi[x] = 0;
            zrow[x] = Z + a * kDcLd + a;
            rok[x] = false;
            continue;
          }
          run = x + 1;
          const int r0 = a + 16 * ((tl[x] >> 8) & 15), r = r0 + li;
          rok[x] = r < g.b;
          zrow[x] = Z + (rok[x] ? r : a) * kDcLd + a;
          lo[x] = r0 >= g.c ? n1 / 4 : 0;
          hi[x] = r0 + 16 <= g.c ? (e1 + 3) / 4 : steps;
        }
        int ic = pole(0), icn = pole(1);
        double pd = dz[ic].x, pz = zt[ic];
        int pc = ndc[ic], pcn = ndc[icn];
        double zr[S];
#pragma unroll
        for (int x = q; x < S; ++x) zr[x] = zrow[x][pc];
        for (int kk = 0; kk < steps; ++kk) {
          const bool in = 4 * kk + lk < Ka;
          const double ui = pz * dc_rcp((pd - oj.x) - oj.y) * nj;
          const double bv = in && jj < Ka ? ui : 0.0;
          double av[S];
#pragma unroll
          for (int x = q; x < S; ++x) {
            av[x] = in && rok[x] ? zr[x] : 0.0;
            zr[x] = zrow[x][pcn];
          }
          pd = dz[icn].x;
          pz = zt[icn];
          icn = pole(kk + 2);
          pcn = ndc[icn];
#pragma unroll
          for (int x = q; x < S; ++x)
            if (kk >= lo[x] && kk < hi[x])  // uniform
              acc[x] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[x], bv, acc[x], 0, 0, 0);
        }
      }
      lds_barrier();  // every read of the old block is done
#pragma unroll
      for (int q = 0; q < S; ++q) {
        if (tl[q] < 0) continue;
        const int a = tl[q] & 255, rt = (tl[q] >> 8) & 15, ct = (tl[q] >> 12) & 15;
        const DcMerge g = dc_merge_of(a, D, n, magic);
        const int jj = 16 * ct + li;
        if (jj >= kcnt[a]) continue;
        const int c = a + ndc[a + jj];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = a + 16 * rt + lk + 4 * v;
          if (r < g.b) Z[r * kDcLd + c] = acc[q][v];
        }
      }
      if (on1 && t - g1.a < kcnt[g1.a]) lam[g1.a + ndc[t]] = ot[t].x + ot[t].y;
    }
    lds_barrier();
  }

  // ascending order (ties by index)
  if (t < n) {
    const double lv = lam[t];
    int r = 0;
#pragma unroll 8
    for (int i = 0; i < n; ++i) {
      const double li = lam[i];
      r += (li < lv || (li == lv && i < t)) ? 1 : 0;
    }
    ord[r] = t;
    W[r] = lv;
    if (!(fabs(lv) < INFINITY)) bad = 1;
  }
  lds_barrier();
  for (int c = w; c < n; c += NW) {
    const int oc = ord[c];
    for (int r = lane; r < n; r += 64) Zt[c * n + r] = Z[r * kDcLd + oc];
  }
  if (t == 0) *info = bad;
}

template <int NT>
__global__ __launch_bounds__(NT, 2) void k_stedc_small(const double* din, const double* ein, int n,
                                                    double* W, double* __restrict__ Zt,
                                                    int* __restrict__ info) {
  stedc_body<NT>(din, ein, n, W, Zt, info);
}

// Every problem of a lockstep batch whose block eigensolver is still
// iterating: the tridiagonal (diagonal in W, off-diagonal in G) of its
// Rayleigh-Ritz matrix becomes W ascending and Rt = its eigenvectors as
// rows; a non-finite result marks the problem failed (it is then run again
// alone).
template <int NT>
__global__ __launch_bounds__(NT, 2) void k_group_stedc(const GroupStep* __restrict__ dsc) {
  const GroupStep& g = dsc[blockIdx.x];
  if (!g.ctl->iter) return;  // uniform
  __shared__ int bad_out;
  stedc_body<NT>(g.W, g.G, g.p, g.W, g.Rt, &bad_out);
  if (threadIdx.x == 0 && bad_out) g.ctl->fail = 1;  // thread 0 wrote bad_out itself
}

static inline size_t dc_lds(int n) { return (size_t)n * kDcLd * sizeof(double); }

// the dynamic LDS limit of the kernels' larger instances, once
static bool dc_lds_ok() {
  static const bool ok =
      hipFuncSetAttribute((const void*)k_stedc_small<512>,
                          hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)dc_lds(kDcMax)) == hipSuccess &&
      hipFuncSetAttribute((const void*)k_stedc_small<256>,
                          hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)dc_lds(64)) == hipSuccess &&
      hipFuncSetAttribute((const void*)k_group_stedc<512>,
                          hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)dc_lds(kDcMax)) == hipSuccess &&
      hipFuncSetAttribute((const void*)k_group_stedc<256>,
                          hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)dc_lds(64)) == hipSuccess;
  return ok;
}

void group_stedc(const GroupStep* d, int count, int pmax, hipStream_t s) {
  (void)dc_lds_ok();
  if (pmax <= 64)
    hipLaunchKernelGGL(k_group_stedc<256>, dim3(count), dim3(256), dc_lds(pmax), s, d);
  else
    hipLaunchKernelGGL(k_group_stedc<512>, dim3(count), dim3(512), dc_lds(pmax), s, d);
}

bool tridiag_eig_small(const double* d, const double* e, int n, double* W, double* Zt, int* info,
                       hipStream_t s) {
  if (!dc_lds_ok() || n < 1 || n > kDcMax) return false;
  if (n <= 64)
    hipLaunchKernelGGL(k_stedc_small<256>, dim3(1), dim3(256), dc_lds(n), s, d, e, n, W, Zt, info);
  else
    hipLaunchKernelGGL(k_stedc_small<512>, dim3(1), dim3(512), dc_lds(n), s, d, e, n, W, Zt, info);
  return hipGetLastError() == hipSuccess;
}

}  // namespace hotrg
