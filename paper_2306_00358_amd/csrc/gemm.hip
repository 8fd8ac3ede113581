// Dense contractions of the HOTRG step as MFMA GEMMs for gfx950.
//
// Every contraction of a step (environment halves and combine, the three
// coarse contractions; Sec. 2 of arXiv 2306.00358) is a plain GEMM once its
// operands are laid out with the contracted legs contiguous; the index
// permutation that the next contraction needs is applied in the epilogue
// (OutMap), so no separate transpose pass touches the large intermediates.
//
// FP64: v_mfma_f64_16x16x4f64.  Lane layout of one 16x16x4 product
// (64 lanes): A[i][k] from lane i + 16k, B[k][j] from lane j + 16k, and the
// four accumulator values of lane L hold D[L/16 + 4v][L % 16], v = 0..3.
#include <hip/hip_runtime.h>

#include <cstdlib>

#include <map>
#include <mutex>
#include <type_traits>

#include "internal.h"
#include "lds_copy.h"

namespace hotrg {

typedef double d4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ long long map_row(const OutMap& o, int m) {
  int m2 = m % o.r2;
  int q = m / o.r2;
  int m1 = q % o.r1;
  int m0 = q / o.r1;
  return (long long)m0 * o.s0 + (long long)m1 * o.s1 + (long long)m2 * o.s2;
}

__device__ __forceinline__ long long map_col(const OutMap& o, int n) {
  int n2 = n % o.c2;
  int q = n / o.c2;
  int n1 = q % o.c1;
  int n0 = q / o.c1;
  return (long long)n0 * o.t0 + (long long)n1 * o.t1 + (long long)n2 * o.t2;
}

__device__ __forceinline__ void atomic_max_bits(unsigned long long* p, double v) {
  // |v| >= 0: the IEEE bit pattern of a non-negative double orders like
  // the value; NaN patterns compare above +inf and propagate.
  atomicMax(p, (unsigned long long)__double_as_longlong(v));
}

__device__ __forceinline__ double wave_max(double v) {
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}

// Block tile BM x BN, K slab BK; 4 waves in a 2 x 2 arrangement (two waves per
// SIMD promised to the compiler, which otherwise moves the accumulators to the
// accumulation registers and back every slab: 64 x 64 tiles 8% slower), each wave
// owns a (BM/2) x (BN/2) sub-tile made of 16x16 MFMA tiles.  Operand tiles
// go global -> registers -> LDS; the next slab's global loads are issued
// before the current slab's MFMAs so that they overlap.
template <int BM, int BN, int BK, int BL>
__device__ __forceinline__ void f64_tile(const double* __restrict__ A, long long lda,
                                         const double* __restrict__ B, long long ldb,
                                         double* __restrict__ C, const OutMap& om, int M, int N,
                                         int K, unsigned long long* maxbits, int m0, int n0) {
  constexpr int WM = BM / 2, WN = BN / 2, TM = WM / 16, TN = WN / 16;
  constexpr int A_PER = BM * BK / 256, B_PER = BN * BK / 256;
  static_assert(BM * BK % 256 == 0 && BN * BK % 256 == 0, "tile must split over 256 threads");
  __shared__ double As[BM][BK + 1];
  // B_NCONTIG: Bs[k][n]; B_KCONTIG: Bs[n][k] (padded against bank conflicts)
  __shared__ double Bs[BL == B_NCONTIG ? BK : BN][BL == B_NCONTIG ? BN : BK + 1];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;

  d4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};

  double ra[A_PER], rb[B_PER];

  auto load = [&](int k0) {
#pragma unroll
    for (int p = 0; p < A_PER; ++p) {
      int e = tid + 256 * p;
      int r = e / BK, c = e % BK;
      int gm = m0 + r, gk = k0 + c;
      ra[p] = (gm < M && gk < K) ? A[(long long)gm * lda + gk] : 0.0;
    }
#pragma unroll
    for (int p = 0; p < B_PER; ++p) {
      int e = tid + 256 * p;
      if (BL == B_NCONTIG) {
        int r = e / BN, c = e % BN;
        int gk = k0 + r, gn = n0 + c;
        rb[p] = (gk < K && gn < N) ? B[(long long)gk * ldb + gn] : 0.0;
      } else {
        int r = e / BK, c = e % BK;
        int gn = n0 + r, gk = k0 + c;
        rb[p] = (gk < K && gn < N) ? B[(long long)gn * ldb + gk] : 0.0;
      }
    }
  };
  auto store = [&]() {
#pragma unroll
    for (int p = 0; p < A_PER; ++p) {
      int e = tid + 256 * p;
      As[e / BK][e % BK] = ra[p];
    }
#pragma unroll
    for (int p = 0; p < B_PER; ++p) {
      int e = tid + 256 * p;
      if (BL == B_NCONTIG)
        Bs[e / BN][e % BN] = rb[p];
      else
        Bs[e / BK][e % BK] = rb[p];
    }
  };

  const int li = lane & 15, lk = lane >> 4;
  load(0);
  for (int k0 = 0; k0 < K; k0 += BK) {
    __syncthreads();
    store();
    __syncthreads();
    if (k0 + BK < K) load(k0 + BK);
#pragma unroll
    for (int kk = 0; kk < BK; kk += 4) {
      double a[TM], b[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) a[i] = As[wm * WM + i * 16 + li][kk + lk];
#pragma unroll
      for (int j = 0; j < TN; ++j)
        b[j] = (BL == B_NCONTIG) ? Bs[kk + lk][wn * WN + j * 16 + li]
                                 : Bs[wn * WN + j * 16 + li][kk + lk];
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
    }
  }

  // epilogue: scatter through the OutMap, track max |C|
  double mx = 0.0;
  long long coff[TN];
  bool cok[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    int n = n0 + wn * WN + j * 16 + li;
    cok[j] = n < N;
    coff[j] = cok[j] ? map_col(om, n) : 0;
  }
#pragma unroll
  for (int i = 0; i < TM; ++i) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      int m = m0 + wm * WM + i * 16 + lk + 4 * v;
      if (m >= M) continue;
      long long roff = map_row(om, m);
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        if (!cok[j]) continue;
        double x = acc[i][j][v];
        C[roff + coff[j]] = x;
        mx = fmax(mx, fabs(x));
      }
    }
  }
  if (maxbits) {
    mx = wave_max(mx);
    if (lane == 0) atomic_max_bits(maxbits, mx);
  }
}

template <int BM, int BN, int BK, int BL>
__global__ __launch_bounds__(256, 2) void k_gemm_f64(const double* __restrict__ A, long long lda,
                                                  const double* __restrict__ B, long long ldb,
                                                  double* __restrict__ C, OutMap om, int M, int N,
                                                  int K, unsigned long long* maxbits, int kchunk,
                                                  long long cstride) {
  // split-K: block z sums k in [z*kchunk, min((z+1)*kchunk, K)) into C + z*cstride
  if (kchunk > 0) {
    const int z = blockIdx.z;
    const int kb = z * kchunk;
    A += kb;
    B += BL == B_NCONTIG ? (long long)kb * ldb : kb;
    C += z * cstride;
    K = K - kb < kchunk ? K - kb : kchunk;
  }
  f64_tile<BM, BN, BK, BL>(A, lda, B, ldb, C, om, M, N, K, maxbits, blockIdx.y * BM,
                           blockIdx.x * BN);
}

// Sum of the waves' partial tiles in wave order (through red, NWV BT^2 doubles free
// of other data once every wave is here) into C, less sigma * sub, and the maximum.
// mirror: a symmetric C (row-major) from its upper triangle.
template <int BT, int NWV>
__device__ __forceinline__ void small_store(const d4 (&acc)[BT / 16][BT / 16], double* red,
                                            double* __restrict__ C, const OutMap& om, int m0,
                                            int n0, int M, int N, unsigned long long* maxbits,
                                            const double* __restrict__ sub, double sigma,
                                            bool mirror = false) {
  constexpr int TT = BT / 16, E = TT * TT * 256;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  // element e = ((i TT + j) 4 + v) 64 + lane of the tile
  double mx = 0.0;
  auto put = [&](int i, int j, int v, int ln, double x) {
    const int m = m0 + 16 * i + (ln >> 4) + 4 * v, n = n0 + 16 * j + (ln & 15);
    if (m < M && n < N && !(mirror && m > n)) {
      const long long o = map_row(om, m) + map_col(om, n);
      if (mirror) C[map_row(om, n) + map_col(om, m)] = x;
      if (sub) x -= sigma * sub[o];
      C[o] = x;
      mx = fmax(mx, fabs(x));
    }
  };
  if constexpr (NWV == 1) {
#pragma unroll
    for (int i = 0; i < TT; ++i)
#pragma unroll
      for (int j = 0; j < TT; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) put(i, j, v, lane, acc[i][j][v]);
  } else {
#pragma unroll
    for (int i = 0; i < TT; ++i)
#pragma unroll
      for (int j = 0; j < TT; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[w * E + ((i * TT + j) * 4 + v) * 64 + lane] = acc[i][j][v];
    lds_barrier();
#pragma unroll
    for (int e = tid; e < E; e += 64 * NWV) {
      double x = 0.0;
#pragma unroll
      for (int u = 0; u < NWV; ++u) x += red[u * E + e];
      put(e / (TT * 256), (e >> 8) % TT, (e >> 6) & 3, e & 63, x);
    }
  }
  if (maxbits) {
    mx = wave_max(mx);
    if (lane == 0) atomic_max_bits(maxbits, mx);
  }
}

// Small products: one BT x BT output tile per workgroup, its K split over the
// workgroup's NWV waves, operands loaded from global memory straight into the
// MFMA's registers (no LDS until the partial tiles of the waves are summed, in
// wave order).  Lane (i, g) = (lane % 16, lane / 16) takes k = 4 g .. 4 g + 3
// of each 16-wide slab (two 16-byte loads per row of A when VEC: even strides and
// 16-byte aligned bases; B_NCONTIG loads are 8 bytes, 16 lanes to a 128-byte
// line); wave w takes slabs w, w + NWV, ...  K need not be a multiple of
// anything: the last slab is loaded element by element with zeros past K.
// With sub, C -= sigma * sub (sub laid out like C, row-major).
// What bounds these products is latency and the few workgroups that larger
// tiles would give; past a few hundred workgroups the loads of A (64 cycles an
// instruction: 16 rows, each lane its own 16 bytes).  N-contiguous, against 4- to
// 16-way split K by 64 x 64 tiles with a launch for the partial sums:
// 64 x 1024 x 1024 14.1 -> 8.2 us, 96 x 2304 x 2304 46 -> 35 (where the split is the
// faster one: block_product_small); 4096 x 16 x 256 18 -> 5.2.
template <int BT, int NWV, bool VEC>
__device__ __forceinline__ void small_tile(const double* __restrict__ A, long long lda,
                                           const double* __restrict__ B, long long ldb,
                                           double* __restrict__ C, const OutMap& om, int m0, int n0,
                                           int M, int N, int K, unsigned long long* maxbits,
                                           const double* __restrict__ sub, double sigma,
                                           double* red) {
  constexpr int TT = BT / 16;
  typedef double d2 __attribute__((ext_vector_type(2)));
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lg = lane >> 4;
  const double *ar[TT], *br[TT];
#pragma unroll
  for (int i = 0; i < TT; ++i) {
    ar[i] = A + (long long)min(m0 + 16 * i + li, M - 1) * lda;
    const int n = min(n0 + 16 * i + li, N - 1);
    br[i] = B + n;
  }
  d4 acc[TT][TT];
#pragma unroll
  for (int i = 0; i < TT; ++i)
#pragma unroll
    for (int j = 0; j < TT; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};
  struct Frag {
    double a[TT][4], b[TT][4];
  };
  auto load = [&](int s, Frag& f) {
    const int k = 16 * s + 4 * lg;
#pragma unroll
    for (int i = 0; i < TT; ++i) {
#pragma unroll
      for (int t = 0; t < 4; t += 2) {
        if constexpr (VEC) {
          const d2 v = *(const d2*)(ar[i] + k + t);
          f.a[i][t] = v.x;
          f.a[i][t + 1] = v.y;
        } else {
          f.a[i][t] = ar[i][k + t];
          f.a[i][t + 1] = ar[i][k + t + 1];
        }
        f.b[i][t] = br[i][(long long)(k + t) * ldb];
        f.b[i][t + 1] = br[i][(long long)(k + t + 1) * ldb];
      }
    }
  };
  auto mul = [&](const Frag& f) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int i = 0; i < TT; ++i)
#pragma unroll
        for (int j = 0; j < TT; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(f.a[i][t], f.b[j][t], acc[i][j], 0, 0, 0);
  };
  const int full = K >> 4;
  int s = w;
  if (s < full) {
    // two slabs in flight ahead of the products
    Frag f0, f1;
    load(s, f0);
    load(s + NWV < full ? s + NWV : s, f1);
    for (; s < full; s += NWV) {
      Frag f2;
      load(s + 2 * NWV < full ? s + 2 * NWV : s, f2);
      mul(f0);
      f0 = f1;
      f1 = f2;
    }
  }
  if ((K & 15) && s == full) {  // uniform: the wave whose turn the last slab is
    Frag f;
    const int k = 16 * full + 4 * lg;
#pragma unroll
    for (int i = 0; i < TT; ++i)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const bool in = k + t < K;
        f.a[i][t] = in ? ar[i][k + t] : 0.0;
        f.b[i][t] = in ? br[i][(long long)(k + t) * ldb] : 0.0;
      }
    mul(f);
  }
  small_store<BT, NWV>(acc, red, C, om, m0, n0, M, N, maxbits, sub, sigma);
}

template <int BT, int NWV, bool VEC>
__global__ __launch_bounds__(64 * NWV, 2) void k_gemm_f64_small(
    const double* __restrict__ A, long long lda, const double* __restrict__ B, long long ldb,
    double* __restrict__ C, OutMap om, int M, int N, int K, unsigned long long* maxbits,
    const double* __restrict__ sub, double sigma, const double* __restrict__ A_2,
    double* __restrict__ C_2, const double* __restrict__ B_2) {
  __shared__ double red[NWV > 1 ? NWV * BT * BT : 1];
  if (blockIdx.z) {  // the second of two products
    A = A_2;
    B = B_2;
    C = C_2;
  }
  small_tile<BT, NWV, VEC>(A, lda, B, ldb, C, om, blockIdx.y * BT, blockIdx.x * BT, M, N, K,
                               maxbits, sub, sigma, red);
}

// The same with both operands K-contiguous: each wave copies its slabs to its own part of LDS (coalesced 128-byte rows, two
// stages, no barrier: it reads only what it copied) instead of loading them into
// registers 16 bytes a lane, 64 cycles an instruction, which bounded them: two
// products of 576^3 35 -> 22 us, of 400^3 19.8 -> 10.1, of 128^3 4.0 -> 3.1; 64 x 64
// x 1024 8.9 -> 5.2 (there by 32 partial products and a launch that sums them),
// 128 x 128 x 4096 16 -> 13.7.  Operands off 16 bytes or with odd strides are copied 4
// bytes a lane into the same places (64 x 64 x 1225: 8.3 us, by 32 partial products 9.1;
// 128 x 128 x 2025 11.9 and 11.3, x 8281 44 and 24: past legs of 45 a few us of a solve
// of milliseconds).  More stages take LDS that a second workgroup uses better (four:
// 576^3 27 us).
// With `sym` (a symmetric C) only tiles that reach the upper triangle are formed, and
// mirrored or not.
constexpr int kSmallStages = 2;
template <int BT, int NWV>
struct SmallK {
  static constexpr int NST = kSmallStages;
  static constexpr int kStage = 2 * BT * 128;  // bytes of a wave's slab of A and B
  static constexpr int kWave = NST * kStage > BT * BT * 8 ? NST * kStage : BT * BT * 8;
  static constexpr int kBytes = NWV * kWave;
};

template <int BT, int NWV, bool VEC>
__device__ __forceinline__ void small_k_tile(const double* __restrict__ A, long long lda,
                                             const double* __restrict__ B, long long ldb,
                                             double* __restrict__ C, const OutMap& om, int m0,
                                             int n0, int M, int N, int K,
                                             unsigned long long* maxbits, bool mirror,
                                             char* smem) {
  constexpr int TT = BT / 16, LOADS = VEC ? 2 * BT / 8 : BT, STAGE = SmallK<BT, NWV>::kStage;
  constexpr int NST = kSmallStages;
  typedef double d2 __attribute__((ext_vector_type(2)));
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lg = lane >> 4;
  char* const base = smem + w * SmallK<BT, NWV>::kWave;
  d4 acc[TT][TT];
#pragma unroll
  for (int i = 0; i < TT; ++i)
#pragma unroll
    for (int j = 0; j < TT; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};
  const int full = K >> 4;
  const int mine = full > w ? (full - w + NWV - 1) / NWV : 0;  // slabs w, w + NWV, ...
  auto issue = [&](int q) {
    char* st = base + (q % NST) * STAGE;
    const int k0 = 16 * (w + q * NWV);
    if constexpr (VEC) {
      load_kcontig<BT, 16, 1>(A, lda, m0, M, k0, st, 0, lane);
      load_kcontig<BT, 16, 1>(B, ldb, n0, N, k0, st + BT * 128, 0, lane);
    } else {
      load_kcontig_any<BT>(A, lda, m0, M, k0, st, lane);
      load_kcontig_any<BT>(B, ldb, n0, N, k0, st + BT * 128, lane);
    }
  };
  auto mul = [&](const double (&fa)[TT][4], const double (&fb)[TT][4]) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int i = 0; i < TT; ++i)
#pragma unroll
        for (int j = 0; j < TT; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[i][t], fb[j][t], acc[i][j], 0, 0, 0);
  };
  for (int q = 0; q < NST - 1; ++q)
    if (q < mine) issue(q);
  for (int q = 0; q < mine; ++q) {
    // slab q has landed; the NST - 2 after it may be pending
    if (q + NST - 1 <= mine)
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 2) * LOADS) : "memory");
    else
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const char* st = base + (q % NST) * STAGE;
    double fa[TT][4], fb[TT][4];
#pragma unroll
    for (int i = 0; i < TT; ++i) {
      const int r = 16 * i + li;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int c = (lg * 2 + u) ^ swz<16>(r);
        const d2 x = *(const d2*)(st + (r * 8 + c) * 16);
        const d2 y = *(const d2*)(st + BT * 128 + (r * 8 + c) * 16);
        fa[i][2 * u] = x.x;
        fa[i][2 * u + 1] = x.y;
        fb[i][2 * u] = y.x;
        fb[i][2 * u + 1] = y.y;
      }
    }
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the stage of slab q - 1 is free
    asm volatile("" ::: "memory");
    if (q + NST - 1 < mine) issue(q + NST - 1);
    mul(fa, fb);
  }
  if ((K & 15) && full % NWV == w) {  // uniform: the wave whose turn the last slab is
    double fa[TT][4], fb[TT][4];
#pragma unroll
    for (int i = 0; i < TT; ++i) {
      const double* ar = A + (long long)min(m0 + 16 * i + li, M - 1) * lda;
      const double* br = B + (long long)min(n0 + 16 * i + li, N - 1) * ldb;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int k = 16 * full + 4 * lg + t;
        fa[i][t] = k < K ? ar[k] : 0.0;
        fb[i][t] = k < K ? br[k] : 0.0;
      }
    }
    mul(fa, fb);
  }
  if (NWV > 1) lds_barrier();  // every wave is done with its stages
  small_store<BT, NWV>(acc, (double*)smem, C, om, m0, n0, M, N, maxbits, nullptr, 0.0, mirror);
}

template <int BT, int NWV, bool VEC>
__global__ __launch_bounds__(64 * NWV, 2) void k_gemm_f64_smallk(
    const double* __restrict__ A, long long lda, const double* __restrict__ B, long long ldb,
    double* __restrict__ C, OutMap om, int M, int N, int K, unsigned long long* maxbits,
    int sym, const double* __restrict__ A_2, double* __restrict__ C_2,
    const double* __restrict__ B_2) {
  __shared__ __attribute__((aligned(16))) char smem[SmallK<BT, NWV>::kBytes];
  if (sym && blockIdx.y > blockIdx.x) return;
  if (blockIdx.z) {  // the second of two products
    A = A_2;
    B = B_2;
    C = C_2;
  }
  small_k_tile<BT, NWV, VEC>(A, lda, B, ldb, C, om, blockIdx.y * BT, blockIdx.x * BT, M, N, K, maxbits,
                             sym == SYM_BOTH, smem);
}

// Grouped form over a device table of products (the block eigensolver of a batch of
// problems): workgroup b takes tile b - begin[i] (BT x BT tiles) of the item i whose
// range holds b; an item whose gate reads 0 skips its tiles.  Small tiles, because a
// batch of few problems leaves the chip idle by 64 x 64 ones over the whole of K (Gram
// matrices of 8 problems, 64 x 64 x 1024: 20 -> 3.6 us a launch, converged ones included).
// An item with a shift subtracts it times sub where `shifted` (the sweeps of the block
// eigensolver, Y = V (M - sigma I)).
template <int BT, int NWV, int BL>
__global__ __launch_bounds__(64 * NWV, 2) void k_gemm_f64_small_grouped(
    const F64Item* __restrict__ items, const int* __restrict__ begin, int count, int sym,
    int shifted) {
  __shared__ __attribute__((aligned(16))) char smem[SmallK<BT, NWV>::kBytes];
  int lo = 0, hi = count - 1;
  const int b = blockIdx.x;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (begin[mid] <= b) lo = mid; else hi = mid - 1;
  }
  const F64Item& it = items[lo];
  if (it.gate && *it.gate == 0) return;
  const int local = b - begin[lo], tn = (it.N + BT - 1) / BT;
  const int tm = local / tn, tc = local % tn;
  if (sym && tm > tc) return;
  if constexpr (BL == B_KCONTIG) {
    if ((it.lda | it.ldb) & 1 || ((uintptr_t)it.A | (uintptr_t)it.B) & 15)
      small_k_tile<BT, NWV, false>(it.A, it.lda, it.B, it.ldb, it.C, out_rowmajor(it.ldc), tm * BT,
                                   tc * BT, it.M, it.N, it.K, nullptr, sym == SYM_BOTH, smem);
    else
      small_k_tile<BT, NWV, true>(it.A, it.lda, it.B, it.ldb, it.C, out_rowmajor(it.ldc), tm * BT,
                                  tc * BT, it.M, it.N, it.K, nullptr, sym == SYM_BOTH, smem);
  } else {
    const double sg = shifted && it.sub ? it.shift[*it.step & 1] : 0.0;
    small_tile<BT, NWV, false>(it.A, it.lda, it.B, it.ldb, it.C, out_rowmajor(it.ldc), tm * BT,
                               tc * BT, it.M, it.N, it.K, nullptr, sg > 0.0 ? it.sub : nullptr, sg,
                               (double*)smem);
  }
}

int f64_group_tiles(const F64Item& it, int bl) {
  const int bt = bl == B_KCONTIG ? 16 : 32;
  return ((it.M + bt - 1) / bt) * ((it.N + bt - 1) / bt);
}

void gemm_f64_grouped(int bl, int sym, bool shifted, const F64Item* d_items, const int* d_begin,
                      int count, int tiles, hipStream_t s) {
  if (tiles <= 0) return;
  if (bl == B_KCONTIG)
    hipLaunchKernelGGL((k_gemm_f64_small_grouped<16, 8, B_KCONTIG>), dim3(tiles), dim3(512), 0, s,
                       d_items, d_begin, count, sym, 0);
  else
    hipLaunchKernelGGL((k_gemm_f64_small_grouped<32, 4, B_NCONTIG>), dim3(tiles), dim3(256), 0, s,
                       d_items, d_begin, count, 0, shifted ? 1 : 0);
}

static bool vec_ok(const double* p, long long ld) { return !(ld & 1) && !((uintptr_t)p & 15); }

template <int BT, int NWV>
static void launch_small(const double* A, long long lda, const double* B, long long ldb, int bl,
                         double* C, const OutMap& om, int M, int N, int K,
                         unsigned long long* maxbits, hipStream_t s, const double* sub,
                         double sigma, int sym, const double* A_2, double* C_2,
                         const double* B_2) {
  const dim3 grid((N + BT - 1) / BT, (M + BT - 1) / BT, A_2 ? 2 : 1), block(64 * NWV);
  const bool vec = vec_ok(A, lda) && vec_ok(A_2, lda) && (bl == B_NCONTIG || (vec_ok(B, ldb) && vec_ok(B_2, ldb)));
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, grid, block, 0, s, A, lda, B, ldb, C, om, M, N, K, maxbits, sub,
                       sigma, A_2, C_2, B_2);
  };
  if (bl == B_NCONTIG) {
    if (vec) go(k_gemm_f64_small<BT, NWV, true>);
    else go(k_gemm_f64_small<BT, NWV, false>);
  } else {
    auto gok = [&](auto kern) {
      hipLaunchKernelGGL(kern, grid, block, 0, s, A, lda, B, ldb, C, om, M, N, K, maxbits, sym,
                         A_2, C_2, B_2);
    };
    if (vec) gok(k_gemm_f64_smallk<BT, NWV, true>);
    else gok(k_gemm_f64_smallk<BT, NWV, false>);
  }
}

// C = A B (- sigma sub, N-contiguous) by small tiles; false for the products that belong to
// the larger ones.  The lines, both sides measured: up to 524288 outputs (729^2 K-
// contiguous: 28.6 us, 34 with 64 x 64 LDS tiles); short K with many tiles stays with the 64 x 64 ones (256 x 4096 x 16: 5.8
// us, 8.7 here).  16 x 16 tiles up to one per compute unit (256^3 N-contiguous: 5.5
// us, 8.7 with 32 x 32), K-contiguous to six (two of 400^3: 10.1 us, 12.3 with
// 32 x 32; two of 484^3: 17.3 and 14.5); four waves once each has a slab, eight with
// K of 256 and at most a tile per unit (64 x 64 x 1024: 5.2 us, 6.2 with four).
// `sym` (K-contiguous, a symmetric C): SymTiles.  A_2: a second product into C_2, of
// A_2 with B_2, or with itself.
static bool gemm_f64_small(const double* A, long long lda, const double* B, long long ldb, int bl,
                           double* C, const OutMap& om, int M, int N, int K,
                           unsigned long long* maxbits, hipStream_t s, const double* sub = nullptr,
                           double sigma = 0.0, int sym = 0, const double* A_2 = nullptr,
                           double* C_2 = nullptr, const double* B_2 = nullptr) {
  const long long t16 = (long long)((M + 15) / 16) * ((N + 15) / 16), mn = (long long)M * N;
  if (K < 1 || mn > 524288 || (K < 32 && t16 > 512)) return false;
  const int slabs = (K + 15) / 16;
  const bool t32 = bl == B_KCONTIG ? (A_2 ? 2 : 1) * t16 > 1536 : t16 > 256;
  auto go = [&](auto nw) {
    constexpr int NWV = decltype(nw)::value;
    if (!t32)
      launch_small<16, NWV>(A, lda, B, ldb, bl, C, om, M, N, K, maxbits, s, sub, sigma, sym, A_2,
                            C_2, B_2 ? B_2 : A_2);
    else if constexpr (NWV <= 4)
      launch_small<32, NWV>(A, lda, B, ldb, bl, C, om, M, N, K, maxbits, s, sub, sigma, sym, A_2,
                            C_2, B_2 ? B_2 : A_2);
  };
  if (bl == B_KCONTIG && slabs >= 16 && t16 <= 256)
    go(std::integral_constant<int, 8>{});
  else if (slabs >= 4)
    go(std::integral_constant<int, 4>{});
  else if (slabs >= 2)
    go(std::integral_constant<int, 2>{});
  else
    go(std::integral_constant<int, 1>{});
  return true;
}

bool gemm_f64_small_pair(const double* A1, const double* A2, long long lda, double* C1, double* C2,
                         const OutMap& om, int M, int K, hipStream_t s) {
  return gemm_f64_small(A1, lda, A1, lda, B_KCONTIG, C1, om, M, M, K, nullptr, s, nullptr, 0.0, 0,
                        A2, C2);
}

// Large-GEMM variant: 128 x 128 block tile, K slab BK = 32, LDS double
// buffered so that one barrier per slab separates the MFMAs of slab s from
// the LDS stores of slab s+1 (whose global loads were issued before the
// MFMAs of slab s).  TAG only gives each call site its own kernel symbol,
// so per-contraction times can be read from a kernel trace.
template <int BL, int TAG>
__global__ __launch_bounds__(256, 2) void k_gemm_f64_big(const double* __restrict__ A, long long lda,
                                                      const double* __restrict__ B, long long ldb,
                                                      double* __restrict__ C, OutMap om, int M,
                                                      int N, int K, unsigned long long* maxbits) {
  constexpr int BM = 128, BN = 128, BK = 32;
  constexpr int WM = BM / 2, WN = BN / 2, TM = WM / 16, TN = WN / 16;
  constexpr int A_PER = BM * BK / 256, B_PER = BN * BK / 256;
  constexpr int AS = BK + 1;                               // A row pitch (doubles)
  constexpr int BR = BL == B_NCONTIG ? BK : BN;            // B rows in LDS
  constexpr int BP = BL == B_NCONTIG ? BN : BK + 1;        // B row pitch
  __shared__ double As[2][BM * AS];
  __shared__ double Bs[2][BR * BP];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;

  d4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};

  double ra[A_PER], rb[B_PER];
  auto load = [&](int k0) {
#pragma unroll
    for (int p = 0; p < A_PER; ++p) {
      int e = tid + 256 * p;
      int r = e / BK, c = e % BK;
      int gm = m0 + r, gk = k0 + c;
      ra[p] = (gm < M && gk < K) ? A[(long long)gm * lda + gk] : 0.0;
    }
#pragma unroll
    for (int p = 0; p < B_PER; ++p) {
      int e = tid + 256 * p;
      if (BL == B_NCONTIG) {
        int r = e / BN, c = e % BN;
        int gk = k0 + r, gn = n0 + c;
        rb[p] = (gk < K && gn < N) ? B[(long long)gk * ldb + gn] : 0.0;
      } else {
        int r = e / BK, c = e % BK;
        int gn = n0 + r, gk = k0 + c;
        rb[p] = (gk < K && gn < N) ? B[(long long)gn * ldb + gk] : 0.0;
      }
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int p = 0; p < A_PER; ++p) {
      int e = tid + 256 * p;
      As[buf][(e / BK) * AS + e % BK] = ra[p];
    }
#pragma unroll
    for (int p = 0; p < B_PER; ++p) {
      int e = tid + 256 * p;
      if (BL == B_NCONTIG)
        Bs[buf][(e / BN) * BP + e % BN] = rb[p];
      else
        Bs[buf][(e / BK) * BP + e % BK] = rb[p];
    }
  };

  const int li = lane & 15, lk = lane >> 4;
  const int nslab = (K + BK - 1) / BK;
  load(0);
  store(0);
  __syncthreads();
  for (int s = 0; s < nslab; ++s) {
    const int cur = s & 1;
    if (s + 1 < nslab) load((s + 1) * BK);
    const double* as = As[cur];
    const double* bs = Bs[cur];
#pragma unroll
    for (int kk = 0; kk < BK; kk += 4) {
      double a[TM], b[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) a[i] = as[(wm * WM + i * 16 + li) * AS + kk + lk];
#pragma unroll
      for (int j = 0; j < TN; ++j)
        b[j] = (BL == B_NCONTIG) ? bs[(kk + lk) * BP + wn * WN + j * 16 + li]
                                 : bs[(wn * WN + j * 16 + li) * BP + kk + lk];
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    if (s + 1 < nslab) store(cur ^ 1);
    __syncthreads();
  }

  double mx = 0.0;
  long long coff[TN];
  bool cok[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    int n = n0 + wn * WN + j * 16 + li;
    cok[j] = n < N;
    coff[j] = cok[j] ? map_col(om, n) : 0;
  }
#pragma unroll
  for (int i = 0; i < TM; ++i) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      int m = m0 + wm * WM + i * 16 + lk + 4 * v;
      if (m >= M) continue;
      long long roff = map_row(om, m);
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        if (!cok[j]) continue;
        double x = acc[i][j][v];
        C[roff + coff[j]] = x;
        mx = fmax(mx, fabs(x));
      }
    }
  }
  if (maxbits) {
    mx = wave_max(mx);
    if (lane == 0) atomic_max_bits(maxbits, mx);
  }
}

template <int BM, int BN, int BK>
static void launch_f64(const double* A, long long lda, const double* B, long long ldb, int bl,
                       double* C, const OutMap& om, int M, int N, int K,
                       unsigned long long* maxbits, hipStream_t s, int kchunk = 0,
                       long long cstride = 0) {
  const int nz = kchunk > 0 ? (K + kchunk - 1) / kchunk : 1;
  dim3 grid((N + BN - 1) / BN, (M + BM - 1) / BM, nz);
  if (bl == B_NCONTIG)
    hipLaunchKernelGGL((k_gemm_f64<BM, BN, BK, B_NCONTIG>), grid, dim3(256), 0, s, A, lda, B, ldb,
                       C, om, M, N, K, maxbits, kchunk, cstride);
  else
    hipLaunchKernelGGL((k_gemm_f64<BM, BN, BK, B_KCONTIG>), grid, dim3(256), 0, s, A, lda, B, ldb,
                       C, om, M, N, K, maxbits, kchunk, cstride);
}

__global__ void k_sum_partials(const double* __restrict__ P, int parts, long long count,
                               long long stride, double* __restrict__ out,
                               const double* __restrict__ sub, double sigma) {
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < count;
       e += (long long)gridDim.x * blockDim.x) {
    double s = 0.0;
#pragma unroll 8
    for (int z = 0; z < parts; ++z) s += P[z * stride + e];
    if (sub) s -= sigma * sub[e];
    out[e] = s;
  }
}

void gemm_f64_symmetric(const double* A, const double* B, long long ld, double* C, int M, int K,
                        int sym, hipStream_t s) {
  // (never refused at these sizes)
  (void)gemm_f64_small(A, ld, B, ld, B_KCONTIG, C, out_rowmajor(M), M, M, K, nullptr, s, nullptr,
                       0.0, sym);
}

void gemm_f64_two(const double* A, long long lda, const double* B1, const double* B2,
                  long long ldb, double* C1, double* C2, int M, int N, int K, hipStream_t s) {
  if (gemm_f64_small(A, lda, B1, ldb, B_NCONTIG, C1, out_rowmajor(N), M, N, K, nullptr, s, nullptr,
                     0.0, 0, A, C2, B2))
    return;
  gemm_f64(A, lda, B1, ldb, B_NCONTIG, C1, out_rowmajor(N), M, N, K, nullptr, s);
  gemm_f64(A, lda, B2, ldb, B_NCONTIG, C2, out_rowmajor(N), M, N, K, nullptr, s);
}

bool block_product_small(int p, int n) {
  const long long t16 = (long long)((p + 15) / 16) * ((n + 15) / 16);
  const long long t32 = (long long)((p + 31) / 32) * ((n + 31) / 32);
  if (t16 <= 256) return !(n & 1) || n <= 640;
  return !(n & 1) && p > 64 && t32 <= (n < 3500 ? 256 : 512);
}

void gemm_f64_block(const double* V, const double* M, double* Y, int p, int n, double sigma,
                    int kchunk, double* partials, hipStream_t s) {
  const double* sub = sigma > 0.0 ? V : nullptr;
  if (block_product_small(p, n) &&
      gemm_f64_small(V, n, M, n, B_NCONTIG, Y, out_rowmajor(n), p, n, n, nullptr, s, sub, sigma))
    return;
  const long long count = (long long)p * n;
  const int parts = (n + kchunk - 1) / kchunk;
  launch_f64<64, 64, 16>(V, n, M, n, B_NCONTIG, partials, out_rowmajor(n), p, n, n, nullptr, s,
                         kchunk, count);
  const long long blocks = (count + 255) / 256;
  hipLaunchKernelGGL(k_sum_partials, dim3(blocks < 4096 ? (int)blocks : 4096), dim3(256), 0, s,
                     partials, parts, count, count, Y, sub, sigma);
}

template <int TAG>
static void launch_big(const double* A, long long lda, const double* B, long long ldb, int bl,
                       double* C, const OutMap& om, int M, int N, int K,
                       unsigned long long* maxbits, hipStream_t s) {
  dim3 grid((N + 127) / 128, (M + 127) / 128);
  if (bl == B_NCONTIG)
    hipLaunchKernelGGL((k_gemm_f64_big<B_NCONTIG, TAG>), grid, dim3(256), 0, s, A, lda, B, ldb, C,
                       om, M, N, K, maxbits);
  else
    hipLaunchKernelGGL((k_gemm_f64_big<B_KCONTIG, TAG>), grid, dim3(256), 0, s, A, lda, B, ldb, C,
                       om, M, N, K, maxbits);
}

// ------------------------------------------------------------- autotuner --
// Large products (M * N >= 2^20) pick their kernel by measurement: on the
// first call with a given shape, operand strides, layout, output map and tag,
// every applicable candidate runs three times on the caller's operands and
// stream, timed with HIP events (the faster of the last two counts: the
// first loads code and warms caches; single runs of the largest products
// spread by a few percent, as much as some candidates differ); the fastest
// is kept for the rest of the process and produces the output of that first
// call too.  Candidates differ only in
// tiling (same products, different summation order), so results agree to
// rounding.  HOTRG_AUTOTUNE=0 keeps the fixed rule below; HOTRG_GEMM_VARIANT
// forces one kernel.
namespace {

enum { C_LDS2 = 0, C_LDS3, C_LDS32, C_LDS_HALF, C_LDS_N64, C_LDS_N32, C_LDS64, C_LDS128, C_BIG,
       C_G128, C_G64, C_COUNT };

struct TuneKey {
  long long v[16];
  bool operator<(const TuneKey& o) const {
    for (int i = 0; i < 16; ++i)
      if (v[i] != o.v[i]) return v[i] < o.v[i];
    return false;
  }
};

std::mutex g_tune_mu;
std::map<TuneKey, int> g_tune;

bool autotune_on() {
  static const bool on = [] {
    const char* e = std::getenv("HOTRG_AUTOTUNE");
    return !(e && e[0] == '0');
  }();
  return on;
}

TuneKey make_key(int prec, long long lda, long long ldb, int bl, const OutMap& om, int M, int N,
                 int K, bool mx, int tag) {
  TuneKey k{};
  const long long v[16] = {prec, lda, ldb, bl, M, N, K, mx, tag, om.r1, om.r2, om.s0,
                           om.c1, om.c2, om.t0, om.s1 * 1000003LL + om.s2 + om.t1 * 7919LL + om.t2};
  for (int i = 0; i < 16; ++i) k.v[i] = v[i];
  return k;
}

// time each applicable candidate (faster of runs two and three); -1 if none
// applies
// The lock is held through a measurement, so each shape is measured once
// per process and every call sees the same choice.
template <class Run>
int tune(const TuneKey& key, int count, Run&& run, hipStream_t s, bool* tuned) {
  *tuned = false;
  std::lock_guard<std::mutex> lk(g_tune_mu);
  auto it = g_tune.find(key);
  if (it != g_tune.end()) return it->second;
  *tuned = true;
  hipEvent_t a, b;
  if (hipEventCreate(&a) != hipSuccess) return -1;
  if (hipEventCreate(&b) != hipSuccess) {
    (void)hipEventDestroy(a);
    return -1;
  }
  int best = -1;
  float best_ms = 0.f;
  for (int c = 0; c < count; ++c) {
    if (!run(c)) continue;  // not applicable to this shape
    float ms = 0.f;
    bool ok = true;
    for (int rep = 0; rep < 2 && ok; ++rep) {
      (void)hipEventRecord(a, s);
      run(c);
      (void)hipEventRecord(b, s);
      float t = 0.f;
      ok = hipEventSynchronize(b) == hipSuccess && hipEventElapsedTime(&t, a, b) == hipSuccess;
      if (ok && (rep == 0 || t < ms)) ms = t;
    }
    if (!ok) continue;
    if (best < 0 || ms < best_ms) {
      best = c;
      best_ms = ms;
    }
  }
  (void)hipEventDestroy(a);
  (void)hipEventDestroy(b);
  if (best >= 0) g_tune[key] = best;
  return best;
}

}  // namespace

void gemm_f64(const double* A, long long lda, const double* B, long long ldb, int blayout,
              double* C, const OutMap& om, int M, int N, int K, unsigned long long* maxbits,
              hipStream_t s, int tag) {
  if (M <= 0 || N <= 0) return;
  const bool no_tune = (tag & GEMM_NO_TUNE) != 0;
  tag &= ~GEMM_NO_TUNE;
  static const int forced = [] {
    const char* e = std::getenv("HOTRG_GEMM_VARIANT");
    return e ? std::atoi(e) : -1;
  }();
  auto cand = [&](int c) -> bool {
    switch (c) {
      case C_LDS2:
        return N >= 128 && gemm_f64_lds(A, lda, B, ldb, blayout, C, om, M, N, K, maxbits, s, tag, 1);
      case C_LDS3:
        return N >= 128 && K >= 64 &&
               gemm_f64_lds(A, lda, B, ldb, blayout, C, om, M, N, K, maxbits, s, tag, 3);
      case C_LDS32:
        return N >= 128 && gemm_f64_lds(A, lda, B, ldb, blayout, C, om, M, N, K, maxbits, s, tag, 0);
      case C_LDS_HALF:
        return N >= 128 && gemm_f64_lds(A, lda, B, ldb, blayout, C, om, M, N, K, maxbits, s, tag, 4);
      case C_LDS_N64:
        return N <= 64 && gemm_f64_lds(A, lda, B, ldb, blayout, C, om, M, N, K, maxbits, s, tag, 5);
      case C_LDS_N32:
        return N <= 64 && gemm_f64_lds(A, lda, B, ldb, blayout, C, om, M, N, K, maxbits, s, tag, 8);
      case C_LDS64:
        return gemm_f64_lds(A, lda, B, ldb, blayout, C, om, M, N, K, maxbits, s, tag, 6);
      case C_LDS128:
        return N >= 128 && gemm_f64_lds(A, lda, B, ldb, blayout, C, om, M, N, K, maxbits, s, tag, 7);
      case C_BIG:
        if (N < 128 || K < 64) return false;
        switch (tag) {
          case GEMM_TAG_C2:
            launch_big<GEMM_TAG_C2>(A, lda, B, ldb, blayout, C, om, M, N, K, maxbits, s);
            break;
          case GEMM_TAG_ENV:
            launch_big<GEMM_TAG_ENV>(A, lda, B, ldb, blayout, C, om, M, N, K, maxbits, s);
            break;
          default:
            launch_big<GEMM_TAG_OTHER>(A, lda, B, ldb, blayout, C, om, M, N, K, maxbits, s);
        }
        return true;
      case C_G128:
        if (N < 128) return false;
        launch_f64<128, 128, 16>(A, lda, B, ldb, blayout, C, om, M, N, K, maxbits, s);
        return true;
      default:
        launch_f64<64, 64, 16>(A, lda, B, ldb, blayout, C, om, M, N, K, maxbits, s);
        return true;
    }
  };
  if (forced < 0 &&
      gemm_f64_small(A, lda, B, ldb, blayout, C, om, M, N, K, maxbits, s))
    return;
  if (!no_tune && forced < 0 && autotune_on() && (long long)M * N >= (1LL << 20)) {
    bool tuned = false;
    const int c = tune(make_key(0, lda, ldb, blayout, om, M, N, K, maxbits != nullptr, tag),
                       C_COUNT, cand, s, &tuned);
    // the candidates' runs all reached the output max: start it again
    if (tuned && maxbits) (void)hipMemsetAsync(maxbits, 0, 8, s);
    if (c >= 0 && cand(c)) return;
  }
  // fixed rule: 256 x 128 tiles, three LDS stages for long K (one barrier per
  // slab, two slabs in flight), two for short K
  const int variant = forced >= 0 ? forced : (K >= 256 ? 3 : 1);
  if ((long long)M * N >= (1LL << 20) && (N >= 128 || ((variant == 5 || variant == 8) && N <= 64)) &&
      variant != 2 && gemm_f64_lds(A, lda, B, ldb, blayout, C, om, M, N, K, maxbits, s, tag, variant))
    return;
  // below the tuner's range: 64 x 64 tiles through LDS where they apply and
  // the slabs are enough to pipeline (1024 x 512 x 1024: 27 us, 33 staged
  // through registers)
  if (K >= 64 && (long long)M * N >= (1LL << 18) && (cand(C_LDS_N32) || cand(C_LDS64))) return;
  if ((long long)M * N >= (1LL << 22) && N >= 128 && K >= 64) {
    cand(C_BIG);
  } else if ((long long)M * N >= (1LL << 22) && N >= 128) {
    launch_f64<128, 128, 16>(A, lda, B, ldb, blayout, C, om, M, N, K, maxbits, s);
  } else {
    launch_f64<64, 64, 16>(A, lda, B, ldb, blayout, C, om, M, N, K, maxbits, s);
  }
}

// the autotuner's table, for the reduced-precision launcher
int tune_choice(int prec, long long lda, long long ldb, int bl, const OutMap& om, int M, int N,
                int K, unsigned long long* maxbits, int tag, int count,
                bool (*run)(void*, int), void* ctx, hipStream_t s) {
  if (!autotune_on()) return -1;
  bool tuned = false;
  const int c = tune(make_key(prec, lda, ldb, bl, om, M, N, K, maxbits != nullptr, tag), count,
                     [&](int k) { return run(ctx, k); }, s, &tuned);
  if (tuned && maxbits) (void)hipMemsetAsync(maxbits, 0, 8, s);
  return c;
}

}  // namespace hotrg
