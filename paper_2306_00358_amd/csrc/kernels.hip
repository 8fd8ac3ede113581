// Bandwidth-bound and single-block kernels of one HOTRG step:
// operand preparation (leg transposition, normalisation, layouts), the
// environment symmetrisation, spectrum bookkeeping, projector extraction,
// and the FP64 log-norm accumulation (arXiv 2306.00358, Sec. 2).
#include <hip/hip_runtime.h>
#include <math.h>

#include "internal.h"

namespace hotrg {

static inline int nblocks(long long n, int t) {
  long long b = (n + t - 1) / t;
  return (int)(b < 65536 ? (b > 0 ? b : 1) : 65536);
}

__device__ __forceinline__ double ld_any(const void* p, long long i, bool f32) {
  return f32 ? (double)((const float*)p)[i] : ((const double*)p)[i];
}
__device__ __forceinline__ void st_any(void* p, long long i, double v, bool f32) {
  if (f32)
    ((float*)p)[i] = (float)v;
  else
    ((double*)p)[i] = v;
}

// ---------------------------------------------------------------- max|x| --
__global__ void k_maxabs(const void* x, long long n, bool f32, unsigned long long* maxbits) {
  double m = 0.0;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x)
    m = fmax(m, fabs(ld_any(x, i, f32)));
  for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o, 64));
  if ((threadIdx.x & 63) == 0) atomicMax(maxbits, (unsigned long long)__double_as_longlong(m));
}

void launch_maxabs(const void* x, long long n, bool is_f32, unsigned long long* maxbits,
                   hipStream_t s) {
  hipLaunchKernelGGL(k_maxabs, dim3(nblocks(n, 256) < 1024 ? nblocks(n, 256) : 1024), dim3(256),
                     0, s, x, n, is_f32, maxbits);
}

// acc[0] = ln n_0; the state's sticky failure flag (an int in acc[1]) is cleared
__global__ void k_init_acc(const unsigned long long* maxbits, double* acc) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    acc[0] = log(__longlong_as_double((long long)*maxbits));
    *(int*)(acc + 1) = 0;
  }
}

// *flag = 1: the failure the tests inject (a failed eigensolve stays visible
// until the state is finished)
__global__ void k_fail_flag(int* flag) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *flag = 1;
}

void launch_fail_flag(int* flag, hipStream_t s) {
  hipLaunchKernelGGL(k_fail_flag, dim3(1), dim3(64), 0, s, flag);
}

void launch_init_acc(const unsigned long long* maxbits, double* acc, hipStream_t s) {
  hipLaunchKernelGGL(k_init_acc, dim3(1), dim3(64), 0, s, maxbits, acc);
}

// ------------------------------------------------------------- operands --
__device__ __forceinline__ void st_rp(void* hi, void* lo, long long i, float v, int mode) {
  if (mode == RP_F32) {
    ((float*)hi)[i] = v;
  } else {
    const __bf16 h = (__bf16)v;
    ((__bf16*)hi)[i] = h;
    ((__bf16*)lo)[i] = (__bf16)(v - (float)h);
  }
}

// Log-norm and torus trace of the coarse tensor Tt (dims (dn,dy,dn,dy)), by one
// workgroup of 256 threads: acc[0] += w ln n_k; rec[0] = ln n_k, rec[3] =
// acc + w ln trace (NaN if trace <= 0), n_k from maxbits.
__device__ __forceinline__ void norm_body(const NormArgs& a, const unsigned long long* maxbits) {
  __shared__ double red[256];
  const int t = threadIdx.x;
  const double nk = __longlong_as_double((long long)*maxbits);
  double s = 0.0;
  const int cnt = a.dn * a.dy;
  for (int e = t; e < cnt; e += 256) {
    int i = e / a.dy, j = e % a.dy;
    s += ld_any(a.Tt, (((long long)i * a.dy + j) * a.dn + i) * a.dy + j, a.f32);
  }
  red[t] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (t < o) red[t] += red[t + o];
    __syncthreads();
  }
  if (t == 0) {
    double ln = log(nk);
    double c = a.acc[0] + a.w * ln;
    a.acc[0] = c;
    double tr = red[0] / nk;
    a.rec[0] = ln;
    a.rec[3] = tr > 0.0 ? c + a.w * log(tr) : __longlong_as_double(0x7ff8000000000000LL);
  }
}

// One operand of a step: element (l, u, r, d) of the tensor (dims n = (dx, dy,
// dx, dy)) is read at sum idx * sst, scaled by 1 / max|T~| and written at sum
// idx * dst in the operand's format (and at its natural position into an
// FP32 copy when one is given).  The dims ta (unit source stride) and tb (unit
// destination stride, or another one when that is ta) are tiled 32 x 32, one
// workgroup per tile and index pair of the other two dims o0, o1.  With
// different unit-stride dims the tile passes through LDS, so reads run along
// ta and writes along tb, both coalesced; otherwise both run along ta.
struct PrepPass {
  long long sst[4], dst[4];
  int n[4];
  int ta, tb, o0, o1;
  int tiles_a, tiles, blk0;  // tiles along ta, tiles of an index pair, first workgroup
  int mode;                  // RP_F32, RP_BF16X3 or kFmtF64
  void *hi, *lo;
  float* tn;
};

// A step's operands in one launch (each operand a range of workgroups), with
// the log-norm as its last workgroup: these are bandwidth-bound passes at
// large D and launches of a few us each at small D.
struct PrepSet {
  PrepPass p[4];
  int count, norm_blk;
  int blocks;  // workgroups with work: the grid's rows may end in others
  NormArgs norm;
  const void* src;
  bool src_f32;
  const unsigned long long* maxbits;  // null: scale 1
};

constexpr int kPrepRow = 1 << 20;

__global__ __launch_bounds__(256) void k_prep(PrepSet S) {
  __shared__ double tile[32][33];
  const int blk = (int)(blockIdx.y * gridDim.x + blockIdx.x);
  if (blk >= S.blocks) return;  // uniform
  if (blk == S.norm_blk) {  // uniform
    norm_body(S.norm, S.maxbits);
    return;
  }
  int q = 0;
  while (q + 1 < S.count && blk >= S.p[q + 1].blk0) ++q;
  const PrepPass& P = S.p[q];
  const double inv = S.maxbits ? 1.0 / __longlong_as_double((long long)*S.maxbits) : 1.0;
  const int na = P.n[P.ta], nb = P.n[P.tb];
  const int local = blk - P.blk0, pair = local / P.tiles, tl = local - pair * P.tiles;
  const int i1 = pair / P.n[P.o0], i0 = pair - i1 * P.n[P.o0];
  const int a0 = (tl % P.tiles_a) * 32, b0 = (tl / P.tiles_a) * 32;
  const long long sb = i0 * P.sst[P.o0] + i1 * P.sst[P.o1];
  const long long db = i0 * P.dst[P.o0] + i1 * P.dst[P.o1];
  const long long nat[4] = {(long long)P.n[1] * P.n[0] * P.n[1], (long long)P.n[0] * P.n[1], P.n[1],
                            1};
  const long long tb = i0 * nat[P.o0] + i1 * nat[P.o1];
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const bool direct = P.dst[P.ta] == 1;
  const long long sa = P.sst[P.ta], sbb = P.sst[P.tb], da = P.dst[P.ta], dbb = P.dst[P.tb];
  const long long ta = nat[P.ta], tbb = nat[P.tb];
  auto put = [&](int a, int b, double v) {
    const long long o = db + a * da + b * dbb;
    if (P.mode == kFmtF64) {
      ((double*)P.hi)[o] = v;
    } else {
      st_rp(P.hi, P.lo, o, (float)v, P.mode);
      if (P.tn) P.tn[tb + a * ta + b * tbb] = (float)v;
    }
  };
  for (int k = ty; k < 32; k += 8) {
    const int a = a0 + tx, b = b0 + k;
    double v = 0.0;
    if (a < na && b < nb) {
      v = ld_any(S.src, sb + a * sa + b * sbb, S.src_f32) * inv;
      if (direct) put(a, b, v);
    }
    tile[k][tx] = v;
  }
  if (direct) return;  // uniform
  __syncthreads();
  for (int k = ty; k < 32; k += 8) {
    const int b = b0 + tx, a = a0 + k;
    if (a < na && b < nb) put(a, b, tile[tx][k]);
  }
}

void launch_prep(const void* src, bool src_f32, bool rotate, int dx, int dy,
                 const unsigned long long* maxbits, const PrepOut* outs, int count,
                 const NormArgs* norm, hipStream_t s) {
  // index order (l, u, r, d); the source is T~ itself or, rotated, T~[u, l, d, r]
  const long long X = dx, Y = dy;
  const long long src_rot[4] = {Y * X, X * Y * X, 1, X};
  const long long src_nat[4] = {Y * X * Y, X * Y, Y, 1};
  const long long* sst = rotate ? src_rot : src_nat;
  PrepSet S{};
  S.count = count;
  S.src = src;
  S.src_f32 = src_f32;
  S.maxbits = maxbits;
  int blocks = 0;
  for (int o = 0; o < count; ++o) {
    PrepPass& P = S.p[o];
    const int n[4] = {dx, dy, dx, dy};
    int ta = 0, tb = -1;
    for (int i = 0; i < 4; ++i) {
      P.sst[i] = sst[i];
      P.dst[i] = outs[o].dst[i];
      P.n[i] = n[i];
    }
    for (int i = 0; i < 4; ++i)
      if (P.sst[i] == 1) ta = i;
    for (int i = 0; i < 4; ++i)
      if (P.dst[i] == 1 && i != ta) tb = i;
    if (tb < 0) tb = ta == 3 ? 2 : 3;  // the same unit-stride dim: any other one
    int rest[2], nr = 0;
    for (int i = 0; i < 4; ++i)
      if (i != ta && i != tb) rest[nr++] = i;
    P.ta = ta;
    P.tb = tb;
    P.o0 = rest[0];
    P.o1 = rest[1];
    P.tiles_a = (n[ta] + 31) / 32;
    P.tiles = P.tiles_a * ((n[tb] + 31) / 32);
    P.blk0 = blocks;
    P.mode = outs[o].mode;
    P.hi = outs[o].hi;
    P.lo = outs[o].lo;
    P.tn = outs[o].tn;
    blocks += P.tiles * n[rest[0]] * n[rest[1]];
  }
  S.norm_blk = -1;
  if (norm) {
    S.norm = *norm;
    S.norm_blk = blocks++;
  }
  S.blocks = blocks;
  // one row of workgroups, or several: a grid dimension holds fewer than 2^32 threads
  // (a leg of 23184 beside one of 1 takes more)
  const int row = blocks < kPrepRow ? blocks : kPrepRow;
  if (blocks > 0)
    hipLaunchKernelGGL(k_prep, dim3(row, (blocks + row - 1) / row), dim3(256), 0, s, S);
}

// Columns [from, ld) of `rows` rows of ld elements of es bytes, for each region
// (one grid row each) = 0: the padding of operands whose rows are longer than
// their contracted index, so that the products need no remainder in K.  Only
// the padding is written -- clearing the whole of a D^5 intermediate, as for
// D^2 not a multiple of 32, cost as much as a contraction's own stores.
__global__ __launch_bounds__(256) void k_zero_pads(PadSet S) {
  const PadRegion& R = S.r[blockIdx.y];
  const long long w = R.ld - R.from, total = R.rows * w;
  for (long long e = blockIdx.x * 256LL + threadIdx.x; e < total; e += gridDim.x * 256LL) {
    const long long row = e / w, o = row * R.ld + R.from + (e - row * w);
    if (R.es == 8)
      ((double*)R.p)[o] = 0.0;
    else if (R.es == 4)
      ((float*)R.p)[o] = 0.0f;
    else
      ((unsigned short*)R.p)[o] = 0;
  }
}

void PadSet::add(void* p, long long rows, long long ld, long long from, int es, hipStream_t s) {
  if (!p || rows <= 0 || from >= ld) return;
  if (count == kMax) launch(s);
  r[count++] = PadRegion{p, rows, ld, from, es};
}

void PadSet::launch(hipStream_t s) {
  if (count == 0) return;
  long long most = 1;
  for (int i = 0; i < count; ++i) {
    const long long t = r[i].rows * (r[i].ld - r[i].from);
    most = t > most ? t : most;
  }
  const long long blocks = (most + 255) / 256;
  hipLaunchKernelGGL(k_zero_pads, dim3((unsigned)(blocks < 2048 ? blocks : 2048), count), dim3(256),
                     0, s, *this);
  count = 0;
}

// The reflected tensor T'[l,u,r,d] = T[r,u,l,d] (FP64, dims (dx,dy,dx,dy)) in
// the natural layout and in the Xt layout [(l,d),(u,r)], rows of ld elements:
// the operands whose environment is that of the right pair of legs of T.
__global__ void k_prep_mirror(const double* __restrict__ T, int dx, int dy, long long ld,
                              double* Tn, double* Xt) {
  const long long total = (long long)dx * dy * dx * dy;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x) {
    long long q = e;
    int d = (int)(q % dy); q /= dy;
    int r = (int)(q % dx); q /= dx;
    int u = (int)(q % dy); q /= dy;
    int l = (int)q;
    const double v = T[(((long long)r * dy + u) * dx + l) * dy + d];
    Tn[((long long)l * dy + u) * ld + (long long)r * dy + d] = v;
    Xt[((long long)l * dy + d) * ld + (long long)u * dx + r] = v;
  }
}

void launch_prep_mirror(const double* T, int dx, int dy, long long ld, double* Tn, double* Xt,
                        hipStream_t s) {
  long long total = (long long)dx * dy * dx * dy;
  hipLaunchKernelGGL(k_prep_mirror, dim3(nblocks(total, 256)), dim3(256), 0, s, T, dx, dy, ld, Tn,
                     Xt);
}

__global__ void k_store(double* p, double v) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *p = v;
}

void launch_store(double* p, double v, hipStream_t s) {
  hipLaunchKernelGGL(k_store, dim3(1), dim3(64), 0, s, p, v);
}

// ------------------------------------------------------------ environment --
// M <- (M + M^T) / 2 by 32 x 32 tile pairs (I, J), I <= J: both tiles are
// read coalesced into LDS and written back, each entry 0.5 (M_rc + M_cr)
// with r < c the upper one; a diagonal tile is its own partner.
__global__ __launch_bounds__(256) void k_symmetrize(double* M, int n, double* trace) {
  const int I = blockIdx.y, J = blockIdx.x;
  if (I == (int)gridDim.x) {
    // the last row of workgroups: trace(M), by the first of them (the
    // diagonal is not written), fixed-order tree
    if (J > 0) return;  // uniform
    __shared__ double red[256];
    const int t = threadIdx.x;
    double s = 0.0;
    for (int i = t; i < n; i += 256) s += M[(long long)i * n + i];
    red[t] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
      if (t < o) red[t] += red[t + o];
      __syncthreads();
    }
    if (t == 0) *trace = red[0];
    return;
  }
  if (I > J) return;  // uniform
  __shared__ double A[32][33], B[32][33];  // tiles (I, J) and (J, I)
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const int r0 = I * 32, c0 = J * 32;
  for (int k = ty; k < 32; k += 8) {
    const int r = r0 + k, c = c0 + tx;
    A[k][tx] = (r < n && c < n) ? M[(long long)r * n + c] : 0.0;
    const int r2 = c0 + k, c2 = r0 + tx;
    B[k][tx] = (r2 < n && c2 < n) ? M[(long long)r2 * n + c2] : 0.0;
  }
  __syncthreads();
  for (int k = ty; k < 32; k += 8) {
    const int r = r0 + k, c = c0 + tx;  // in tile (I, J): M_rc = A[k][tx], M_cr = B[tx][k]
    if (r < n && c < n && r < c) M[(long long)r * n + c] = 0.5 * (A[k][tx] + B[tx][k]);
    const int r2 = c0 + k, c2 = r0 + tx;  // in tile (J, I), lower: upper partner (c2, r2)
    if (r2 < n && c2 < n && c2 < r2) M[(long long)r2 * n + c2] = 0.5 * (A[tx][k] + B[k][tx]);
  }
}

void launch_symmetrize(double* M, int n, double* trace, hipStream_t s) {
  const int T = (n + 31) / 32;
  hipLaunchKernelGGL(k_symmetrize, dim3(T, T + 1), dim3(256), 0, s, M, n, trace);
}

// --------------------------------------------------------------- spectrum --
// W: the cnt leading eigenvalues of M, ascending; lambda_m = W[cnt-1-m]
// (descending).  total = trace(M).  rec[1] = truncation error, rec[2] = cut
// gap, rec[4] = kept (as double), rec[5] = 0 (left environment).  Sums use a
// fixed-order tree.  A dense solve's *info (may be null) that is not zero
// sets the sticky flag.
__global__ void k_spectrum(const double* W, int cnt, int n, int dn, int trunc, double tau,
                           int spec_len, const double* total, double* spec_out, double* rec,
                           int* kept_out, const int* info, int* sticky) {
  __shared__ double red[256];
  __shared__ int kept_s;
  const int t = threadIdx.x;
  const double l1 = W[cnt - 1];
  if (t == 0) {
    int kept = dn;
    if (trunc == 1 && dn < n)
      while (kept > 0 && (W[cnt - kept] - W[cnt - 1 - kept]) <= tau * l1) --kept;
    kept_s = kept;
    *kept_out = kept;
    if (info && *info != 0) *sticky = 1;
  }
  __syncthreads();
  const int kept = kept_s;
  double kp = 0.0;
  for (int m = t; m < kept; m += 256) kp += W[cnt - 1 - m];
  red[t] = kp;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (t < o) red[t] += red[t + o];
    __syncthreads();
  }
  if (t == 0) {
    rec[1] = 1.0 - red[0] / total[0];
    rec[2] = dn < n ? (W[cnt - dn] - W[cnt - 1 - dn]) / l1 : -1.0;
    rec[4] = (double)kept;
    rec[5] = 0.0;
  }
  if (spec_out)
    for (int m = t; m < spec_len; m += 256) spec_out[m] = m < cnt ? W[cnt - 1 - m] / l1 : 0.0;
}

void launch_spectrum(const double* W, int cnt, int n, int dn, int trunc, double tau, int spec_len,
                     const double* total, double* spec_out, double* rec, int* kept,
                     const int* info, int* sticky, hipStream_t s) {
  hipLaunchKernelGGL(k_spectrum, dim3(1), dim3(256), 0, s, W, cnt, n, dn, trunc, tau, spec_len,
                     total, spec_out, rec, kept, info, sticky);
}

// ------------------------------------------------------------- projector --
// V: `cols` eigenvectors of M of length n, vector c at V[c*n .. c*n + n),
// ascending eigenvalue order.
// Ucan[(a*dx + b)*dn + i] = U[a,b,i] = vector cols-1-i (zero for i >= kept).
__global__ void k_isometry(const double* V, int cols, int n, int dn, const int* kept,
                           double* Ucan) {
  const int kp = *kept;
  long long total = (long long)n * dn;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x) {
    int i = (int)(e % dn);
    int row = (int)(e / dn);
    Ucan[e] = i < kp ? V[(long long)(cols - 1 - i) * n + row] : 0.0;
  }
}

void launch_isometry(const double* V, int cols, int n, int dn, const int* kept, double* Ucan,
                     hipStream_t s) {
  hipLaunchKernelGGL(k_isometry, dim3(nblocks((long long)n * dn, 256)), dim3(256), 0, s, V, cols,
                     n, dn, kept, Ucan);
}

// The projector in the layouts the contractions read.  U[a,b,i] is read at
// src + (a dx + b) sr + i si (eigenvector rows: sr = 1, si = -n from the last row;
// a canonical U: sr = dn, si = 1), zero for i >= *kept (kept may be null).
//   U1[(i,a)][b] = U[a,b,i], row length ld1      (A operand of the first contraction)
//   FP64:    U3[(d,e)][k] = U[e,d,k], row length ld3 (B operand of the last one)
//   reduced: U3[k][(d,e)] = U[e,d,k], row length ld3
// *clear (may be null) = 0: the max|T~| slot of the contractions that follow.
__global__ void k_layout_u(const double* src, long long sr, long long si, const int* kept, int dx,
                           int dn, int mode, void* u1hi, void* u1lo, void* u3hi, void* u3lo,
                           long long ld1, long long ld3, unsigned long long* clear) {
  const int kp = kept ? *kept : dn;
  const int n = dx * dx;
  const long long total = (long long)n * dn;
  if (clear && blockIdx.x == 0 && threadIdx.x == 0) *clear = 0ULL;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x) {
    const int ab = (int)(e % n), i = (int)(e / n);
    const int a = ab / dx, b = ab % dx;
    const double v = i < kp ? src[ab * sr + i * si] : 0.0;
    const long long o1 = ((long long)i * dx + a) * ld1 + b;
    const long long de = (long long)b * dx + a;  // (a,b) plays (e,d)
    if (mode == kFmtF64) {
      ((double*)u1hi)[o1] = v;
      ((double*)u3hi)[de * ld3 + i] = v;
    } else {
      st_rp(u1hi, u1lo, o1, (float)v, mode);
      st_rp(u3hi, u3lo, (long long)i * ld3 + de, (float)v, mode);
    }
  }
}

void launch_layout_u(const double* src, long long sr, long long si, const int* kept, int dx, int dn,
                     int mode, void* u1hi, void* u1lo, void* u3hi, void* u3lo, long long ld1,
                     long long ld3, unsigned long long* clear, hipStream_t s) {
  hipLaunchKernelGGL(k_layout_u, dim3(nblocks((long long)dx * dx * dn, 256)), dim3(256), 0, s, src,
                     sr, si, kept, dx, dn, mode, u1hi, u1lo, u3hi, u3lo, ld1, ld3, clear);
}

// ---------------------------------------------------------------- finish --
// ln Z / N = acc + w ln sum_{i,j} T[i,j,i,j]  (periodic trace, Sec. 2)
__global__ void k_finish(const void* Tn, bool f32, int dx, int dy, double w, const double* acc,
                         double* out) {
  __shared__ double red[256];
  const int t = threadIdx.x;
  double s = 0.0;
  const int cnt = dx * dy;
  for (int e = t; e < cnt; e += 256) {
    int i = e / dy, j = e % dy;
    s += ld_any(Tn, (((long long)i * dy + j) * dx + i) * dy + j, f32);
  }
  red[t] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (t < o) red[t] += red[t + o];
    __syncthreads();
  }
  if (t == 0)
    out[0] = red[0] > 0.0 ? acc[0] + w * log(red[0]) : __longlong_as_double(0x7ff8000000000000LL);
}

void launch_finish(const void* Tn, bool f32, int dx, int dy, double weight, const double* acc,
                   double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_finish, dim3(1), dim3(256), 0, s, Tn, f32, dx, dy, weight, acc, out);
}

__global__ void k_f32_to_f64(const float* x, double* y, long long n) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x)
    y[i] = (double)x[i];
}

void launch_f32_to_f64(const float* x, double* y, long long n, hipStream_t s) {
  hipLaunchKernelGGL(k_f32_to_f64, dim3(nblocks(n, 256)), dim3(256), 0, s, x, y, n);
}

}  // namespace hotrg
