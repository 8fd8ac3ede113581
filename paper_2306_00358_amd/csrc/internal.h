// Internal declarations of libhotrg: kernel launchers shared by the engine.
// Not part of the C ABI (see include/hotrg.h).
#pragma once

#include <hip/hip_runtime.h>
#include <rocblas/rocblas.h>
#include <stdint.h>

#include <atomic>

#include "../../include/hotrg.h"

namespace hotrg {

// A divisor 1 <= d < 2^31 of numbers 0 <= n < 2^31: with 2^l >= d > 2^(l-1) and
// mul = floor(2^32 (2^l - d) / d) + 1, n / d = (floor(mul n / 2^32) + n) / 2^l (the
// sum stays below 2^32).  Three instructions where the compiler's division by a
// number it does not know takes about thirty, two an output row and two a column:
// 13200 x 660 x 672 259 -> 247 us, 1089 x 21780 x 20 (20 x 33, C1) 85 -> 39.
struct Div {
  int d;
  unsigned mul;
  int l;
  __host__ __device__ constexpr Div(int v = 1) : d(v), mul(1), l(0) {
    while ((1LL << l) < v) ++l;
    mul = (unsigned)((((1ULL << l) - (unsigned)v) << 32) / (unsigned)v + 1);
  }
  __host__ __device__ operator int() const { return d; }
};
__device__ __forceinline__ int operator/(int n, const Div& v) {
  return (int)((__umulhi((unsigned)n, v.mul) + (unsigned)n) >> v.l);
}
__device__ __forceinline__ int operator%(int n, const Div& v) { return n - (n / v) * v.d; }

// Where a GEMM output element (m, n) is stored.  The row index is read as
// three mixed-radix digits m = (m0 * r1 + m1) * r2 + m2 and the column as
// n = (n0 * c1 + n1) * c2 + n2; the destination offset is
// m0*s0 + m1*s1 + m2*s2 + n0*t0 + n1*t1 + n2*t2.  This is how the index
// permutations between the contractions of one step are fused into the
// GEMM epilogues instead of separate transpose passes.
struct OutMap {
  Div r1, r2;
  long long s0, s1, s2;
  Div c1, c2;
  long long t0, t1, t2;
};

// Two-level map: m = mh * rr + ml -> mh*sh + ml*sl; n = nh * cr + nl -> nh*th + nl*tl.
__host__ __device__ inline OutMap omap2(int rr, long long sh, long long sl, int cr, long long th,
                                        long long tl) {
  OutMap o;
  o.r1 = 1; o.r2 = rr; o.s0 = sh; o.s1 = 0; o.s2 = sl;
  o.c1 = 1; o.c2 = cr; o.t0 = th; o.t1 = 0; o.t2 = tl;
  return o;
}

// Plain row-major output of an M x N matrix with leading dimension ld.
__host__ __device__ inline OutMap out_rowmajor(long long ld) { return omap2(1, ld, 0, 1, 1, 0); }

enum BLayout { B_NCONTIG = 0, B_KCONTIG = 1 };

// Call-site tags: large GEMMs get a kernel symbol per tag.  GEMM_NO_TUNE, or-ed
// into a tag, keeps the fixed tile rule (no timed candidate runs, no host wait).
enum GemmTag { GEMM_TAG_OTHER = 0, GEMM_TAG_ENV = 1, GEMM_TAG_C2 = 2, GEMM_NO_TUNE = 0x100 };

// C[map(m,n)] = sum_k A[m*lda + k] * B(k, n), FP64 MFMA.
// B(k, n) = B[k*ldb + n] for B_NCONTIG, B[n*ldb + k] for B_KCONTIG.
// maxbits (may be null): atomic max of |C| as the bit pattern of a
// non-negative double.
void gemm_f64(const double* A, long long lda, const double* B, long long ldb, int blayout,
              double* C, const OutMap& om, int M, int N, int K,
              unsigned long long* maxbits, hipStream_t s, int tag = GEMM_TAG_OTHER);

// C1 = A1 A1^T and C2 = A2 A2^T (M x K operands, K-contiguous) in one launch of
// small tiles; false where those do not apply.
bool gemm_f64_small_pair(const double* A1, const double* A2, long long lda, double* C1, double* C2,
                         const OutMap& om, int M, int K, hipStream_t s);

// One product of a grouped FP64 launch (device table): C (row-major, leading
// dimension ldc) = A B with B's layout given per launch; gate as for RpItem.
struct F64Item {
  const double* A;
  long long lda;
  const double* B;
  long long ldb;
  double* C;
  long long ldc;
  int M, N, K;
  const int* gate;
  // C -= shift[*step & 1] sub (laid out like C) where the launch asks for it and the
  // shift is positive (N-contiguous only)
  const double* sub;
  const double* shift;
  const int* step;
};
// Of a symmetric C (or all but rounding) only the tiles that reach the upper triangle:
enum SymTiles {
  SYM_NONE = 0,  // no: every tile
  SYM_UPPER,     // the lower triangle's tiles are left as they are
  SYM_BOTH       // the lower triangle mirrors the upper one
};
int f64_group_tiles(const F64Item& it, int bl);  // 16 x 16 (K-contiguous) or 32 x 32
void gemm_f64_grouped(int bl, int sym, bool shifted, const F64Item* d_items, const int* d_begin,
                      int count, int tiles, hipStream_t s);
// C (M x M, row-major) = A B^T, K-contiguous operands whose product is symmetric but for
// rounding, M at most 128; `sym` says what becomes of the lower triangle.
void gemm_f64_symmetric(const double* A, const double* B, long long ld, double* C, int M, int K,
                        int sym, hipStream_t s);
// C1 = A B1 and C2 = A B2 (N-contiguous, C row-major), in one launch where the small
// tiles apply.
void gemm_f64_two(const double* A, long long lda, const double* B1, const double* B2,
                  long long ldb, double* C1, double* C2, int M, int N, int K, hipStream_t s);

// Y = V (M - sigma I), the product of the block eigensolver (V p x n, p a multiple of
// 16, M n x n, all row-major and 16-byte aligned).
void gemm_f64_block(const double* V, const double* M, double* Y, int p, int n, double sigma,
                    int kchunk, double* partials, hipStream_t s);
// By one launch of small tiles, or else by 64 x 64 tiles with K in chunks of kchunk
// (products to `partials`, ceil(n / kchunk) p n doubles) and a launch that sums them.
// Small tiles take it while there are at most 256 of them, one a compute unit: 16 x 16
// (64 x 1024: 8.5 us, 13.3 in chunks; 32 x 1936: 19.7 and 19.0), or 32 x 32 where the 64
// x 64 ones would be of two rows (96 x 2304: 34.9 and 40.4; 128 x 1936: 31.8 and 33.6;
// not 64 x 1600: 26.0 and 20.8).  A second tile a unit costs more than the chunks' sum
// (128 x 2304: 53.7 and 42.6; 96 x 2916: 66 and 56) up to n = 3500; there two tiles
// hide each other's loads, and the chunks' n^2 has caught up (128 x 3600: 83 and 91,
// 96 x 5184: 116 and 150, level at 128 x 4096: 92 and 90).  Odd rows of V are loaded
// 8 bytes a lane: chunks from n = 641 on (64 x 625: 8.7 and 11.9; x 729: 12.9 and 11.1;
// 96 x 2025: 45 and 33; 64 x 4225: 131 and 64).
bool block_product_small(int p, int n);

// Direct-to-LDS FP64 GEMM (gemm_lds.hip); returns false if the operands do
// not meet its alignment / K-multiple requirements.  variant 0: 4 waves,
// 128 x 128 tile, K slab 32; variant 1: 8 waves, 256 x 128 tile, K slab 16;
// variant 3: the same with three stages; 4: 4 waves, 128 x 128; 5: 512 x 64;
// 6: 4 waves, 64 x 64, three stages; 7: 8 waves, 128 x 128, four stages; 8: 4
// waves, 64 x 32, four stages.
bool gemm_f64_lds(const double* A, long long lda, const double* B, long long ldb, int blayout,
                  double* C, const OutMap& om, int M, int N, int K, unsigned long long* maxbits,
                  hipStream_t s, int tag, int variant);
// C = A A^T (M x M, A M x K K-contiguous) from the upper-triangle tiles with
// mirrored stores, and C_2 = A_2 A_2^T in the same launch when A_2 is given;
// false where it does not apply.
bool gemm_f64_syrk(const double* A, long long lda, double* C, const OutMap& om, int M, int K,
                   hipStream_t s, const double* A_2 = nullptr, double* C_2 = nullptr);

// Tile order of a launch over tm x tn output tiles.  Workgroups are handed
// round-robin to the 8 XCDs, each with its own L2.  With group gm > 0 the
// XCD that receives workgroup b takes a contiguous eighth of the tiles,
// walked gm row panels at a time (all of a group's rows for one column
// panel, then the next column panel), so that the workgroups resident on an
// XCD share a few row panels of A and column panels of B.  gm = 0:
// row-major order.
__device__ __forceinline__ void tile_order(int tm, int tn, int b, int gm, int& im, int& in) {
  if (gm <= 0) {
    im = b / tn;
    in = b - im * tn;
    return;
  }
  const int T = tm * tn;
  const int t = (T & 7) ? b : (b & 7) * (T >> 3) + (b >> 3);
  const int g = t / (gm * tn);
  const int rows = min(gm, tm - g * gm);
  const int r = t - g * gm * tn;
  im = g * gm + r % rows;
  in = r / rows;
}

// Workgroup barrier that orders LDS accesses only: global loads and stores in
// flight are not waited for.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ---- reduced-precision contractions (gemm_rp.hip) ----
enum RpMode { RP_F32 = 0, RP_BF16X3 = 1 };
enum RpOut { RP_OUT_F32 = 0, RP_OUT_SPLIT = 1, RP_OUT_F64 = 2 };
// An operand: one float array (RP_F32) or bf16 arrays hi and lo (RP_BF16X3).
struct RpOperand {
  const void* hi;
  const void* lo;
};
// C[map(m,n)] = sum_k A[m][k] B[n][k]; rows of lda / ldb elements (multiples
// of 8, zero past the true K); K a multiple of 32.  Output as float, split
// bf16 (C = hi, Clo = lo) or double.  Returns false if a requirement fails.
// Autotuner table shared by the GEMM launchers: the fastest of `count`
// candidates (run(ctx, c) launches candidate c, false if it does not apply)
// for this shape, measured on first use; -1 if tuning is off.  If it had to
// measure, *maxbits (when given) is zeroed again for the final run.
int tune_choice(int prec, long long lda, long long ldb, int bl, const OutMap& om, int M, int N,
                int K, unsigned long long* maxbits, int tag, int count,
                bool (*run)(void*, int), void* ctx, hipStream_t s);
bool gemm_rp(int mode, const RpOperand& A, long long lda, const RpOperand& B, long long ldb,
             int out, void* C, void* Clo, const OutMap& om, int M, int N, int K,
             unsigned long long* maxbits, hipStream_t s, int tag);
inline long long pad32(long long k) { return (k + 31) / 32 * 32; }

// Row lengths of the FP64 operands of a step with dims (dx, dy) and D' = dn.  A
// contracted index of 128 or more is padded with zeros to a multiple of 16, the
// K slab of the direct-to-LDS tiles, which refuse other K (and odd strides of an
// N-contiguous operand); smaller ones go to the small tiles, which take any K.
// D = 50 (K = 2500): C1, C2, C3 29.7 ms by register-staged tiles, 26.8 padded.
inline long long pad16(long long k) { return k < 128 ? k : (k + 15) / 16 * 16; }
struct F64Ld {
  long long p;   // (r,d), (u,r), (a,c): environment operands, X1 and K of C2
  long long tp;  // columns (l,e) of C2's B
  long long n;   // (d,e): X2 and K of C3
  long long u3;  // columns k of C3's B
  long long k2;  // (e,f): the environment halves
};
inline F64Ld f64_ld(int dx, int dy, int dn) {
  const long long P = (long long)dx * dy, n = (long long)dx * dx;
  return F64Ld{pad16(P), P < 128 ? P : P + (P & 1), pad16(n), n < 128 ? dn : dn + (dn & 1LL),
               pad16((long long)dy * dy)};
}
// the same, nothing padded
inline F64Ld f64_ld_plain(int dx, int dy, int dn) {
  const long long P = (long long)dx * dy;
  return F64Ld{P, P, (long long)dx * dx, dn, (long long)dy * dy};
}

// One product of a grouped launch (device table): the operands and output
// of gemm_rp, and a gate (device int, may be null) that skips the product's
// tiles while it reads 0.
struct RpItem {
  RpOperand A;
  long long lda;
  RpOperand B;
  long long ldb;
  void* C;
  void* Clo;
  OutMap om;
  int M, N, K;
  unsigned long long* maxbits;
  const int* gate;
};
// Workgroups of an item under tile configuration cfg (0: 256 x 256,
// 1: 256 x 128 two stages, 2: 256 x 128 three stages): its output tiles,
// rounded up to a multiple of 8.
int rp_group_tiles(const RpItem& it, int cfg);
// One launch over `tiles` tiles; d_begin[i] is the first tile of item i
// (ascending, d_begin[0] = 0).  Requirements per item as for gemm_rp.
void gemm_rp_grouped(int mode, int out, int cfg, const RpItem* d_items, const int* d_begin,
                     int count, int tiles, hipStream_t s);

// All eigenpairs of the symmetric tridiagonal (d, e), n <= 128, in one
// workgroup (divide and conquer): eigenvalues ascending into W (which may be
// d), eigenvectors as the rows of Zt (n x n); *info = 1 if a result is not
// finite.  False when the launch fails.
bool tridiag_eig_small(const double* d, const double* e, int n, double* W, double* Zt, int* info,
                       hipStream_t s);
// Eigenpairs of a small symmetric matrix (3 <= n <= 128, row-major,
// overwritten): W ascending, rows n - rows .. n - 1 of Zt (n x n) <- the
// eigenvectors of the `rows` largest; E (n) scratch; false when not
// applicable or the launch fails.
bool dense_eig_small(double* M, int n, int rows, double* W, double* E, double* Zt, int* info,
                     hipStream_t s);

// ---- small kernels (kernels.hip) ----
void launch_maxabs(const void* x, long long n, bool is_f32, unsigned long long* maxbits, hipStream_t s);
void launch_init_acc(const unsigned long long* maxbits, double* acc, hipStream_t s);
// The tests' injected eigensolver failure: *flag = 1.
void launch_fail_flag(int* flag, hipStream_t s);
// Operands of a step from the tensor `src` (f64 or f32; legs transposed
// (l,u,r,d) -> (u,l,d,r) with `rotate`, divided by the maximum in *maxbits when
// given), each at its own strides over (l, u, r, d) and in its own format
// (RP_F32, RP_BF16X3: hi and lo; kFmtF64: hi), `tn` an FP32 copy in natural
// order (may be null); one launch.  With `norm` the launch also takes the step's
// log-norm and torus estimate from the coarse tensor.
constexpr int kFmtF64 = 2;
struct PrepOut {
  void* hi;
  void* lo;
  float* tn;
  int mode;
  long long dst[4];
};
struct NormArgs {
  const void* Tt;  // coarse tensor (dims (dn,dy,dn,dy))
  bool f32;
  int dn, dy;
  double w;        // 2^-k
  double* acc;
  double* rec;
};
void launch_prep(const void* src, bool src_f32, bool rotate, int dx, int dy,
                 const unsigned long long* maxbits, const PrepOut* outs, int count,
                 const NormArgs* norm, hipStream_t s);
void launch_prep_mirror(const double* T, int dx, int dy, long long ld, double* Tn, double* Xt,
                        hipStream_t s);
// Padding to clear, several regions a launch (launched by itself when full).
struct PadRegion {
  void* p;
  long long rows, ld, from;  // columns [from, ld) of each row
  int es;                    // element size: 2, 4 or 8
};
struct PadSet {
  static constexpr int kMax = 8;
  PadRegion r[kMax];
  int count = 0;
  void add(void* p, long long rows, long long ld, long long from, int es, hipStream_t s);
  void launch(hipStream_t s);
};
void launch_store(double* p, double v, hipStream_t s);
// M <- (M + M^T) / 2 and *trace = trace(M)
void launch_symmetrize(double* M, int n, double* trace, hipStream_t s);
// W: the `cnt` leading eigenvalues of M in ascending order (cnt <= n);
// total: trace(M) (device scalar).
void launch_spectrum(const double* W, int cnt, int n, int dn, int trunc, double tau, int spec_len,
                     const double* total, double* spec_out, double* rec, int* kept,
                     const int* info, int* sticky, hipStream_t s);
// V: `cols` eigenvectors of length n, vector c at V[c*n], ascending order.
void launch_isometry(const double* V, int cols, int n, int dn, const int* kept, double* Ucan,
                     hipStream_t s);
size_t topk_workspace_doubles(int n, int p);
bool topk_eigs(const double* M, int n, int p, int need, double tol,
               int q_first, double* shift, int* nocheck, double* cond, double* ws, double* W, double* Xout,
               int* dinfo, int* iters, int* enough, double* resid, hipStream_t s);
void launch_layout_u(const double* src, long long sr, long long si, const int* kept, int dx, int dn,
                     int mode, void* u1hi, void* u1lo, void* u3hi, void* u3lo, long long ld1,
                     long long ld3, unsigned long long* clear, hipStream_t s);
void launch_finish(const void* Tn, bool f32, int dx, int dy, double weight, const double* acc,
                   double* out, hipStream_t s);
void launch_f32_to_f64(const float* x, double* y, long long n, hipStream_t s);

// ---- lockstep batch engine (group.hip) ----
constexpr int kGroupRec = 6;  // doubles per step record (as the engine's)
// Per-problem control block, updated by the kernels of a sweep.
struct GroupCtl {
  int active;  // the problem has steps left
  int iter;    // its block eigensolver is still iterating in this step
  int fail;    // sticky: eigensolver budget exhausted or a Cholesky pivot <= 0
  int k;       // steps done
};
// Per-problem descriptor of a run (device memory, fixed while it runs).
struct GroupStep {
  GroupCtl* ctl;
  int n, dn, dy, p, need, trunc, spec_len, K;
  double tau, tol;
  const double* M;  // environment (n x n)
  double* trace;
  double* W;
  double* X;
  int* kept;
  double *V, *Y, *T2, *Yx, *G, *Rt, *H, *res;
  double* recs;
  double* spec;
  double* acc;
  const void* Tt;
  int tt_f32;
  unsigned long long* maxbits;
  double* shift;  // sweep shift per step parity (theta_min / 2 of the last Rayleigh-Ritz)
  double shift_rel;  // of the shifted Cholesky-QR passes
};
// Shifted Cholesky-QR of the iterating problems: dst = R^-T D^-1 src with R, D of
// the Gram matrix G (p <= 128, a multiple of 16).  Pass 0 and 1 factor the
// diagonally scaled, shifted G, pass 2 the plain one; pass 1 between checks
// (!full) takes R = I when G is the identity to 1e-2.  A non-positive pivot sets
// ctl->fail.
enum GroupRows { ROWS_V, ROWS_Y, ROWS_T2 };
void group_orth(const GroupStep* d, int count, int pmax, int max_n, int pass, bool full,
                GroupRows src, GroupRows dst, hipStream_t s);
void group_begin(const GroupStep* d, int count, hipStream_t s);
void group_seed(const GroupStep* d, int count, long long max_pn, hipStream_t s);
// Rayleigh-Ritz matrices H (p x p, p a multiple of 16, <= 128) of the
// iterating problems: Householder reduction (diagonal into W, off-diagonal
// into G, reflectors over H), divide and conquer (W ascending, Rt <- the
// tridiagonal's eigenvector rows), back-transform (Rt <- H's eigenvector
// rows; with `dense` X <- them, n columns each)
void group_sytrd(const GroupStep* d, int count, int pmax, hipStream_t s);
void group_stedc(const GroupStep* d, int count, int pmax, hipStream_t s);
void group_back(const GroupStep* d, int count, int pmax, bool dense, hipStream_t s);
void group_resid(const GroupStep* d, int count, bool last, hipStream_t s);
void group_restart(const GroupStep* d, int count, long long max_pn, hipStream_t s);
// whole small environments (n <= 128, p = n rounded up to even) by the same kernels
void group_dense(const GroupStep* d, int count, int pmax, hipStream_t s);
void group_spectrum(const GroupStep* d, int count, hipStream_t s);
void group_norm(const GroupStep* d, int count, hipStream_t s);
void group_advance(const GroupStep* d, int count, hipStream_t s);

// ---- engine hooks used by the scheduler (sched.cpp) ----
// C1 -> C2 -> C3 in FP64 on caller buffers with rows as `ld` says, padding zero
// (X1: dn*dy*dx rows, X2: dn*dy*dy rows; Tt: dn*dy*dn*dy); *maxbits, cleared by the caller's layout kernel, receives
// max|Tt|.
void coarse_f64_into(hotrg_ctx* c, const double* Tn, const double* Tp, const double* U1,
                     const double* U3, int dx, int dy, int dn, const F64Ld& ld, double* X1,
                     double* X2, double* Tt, unsigned long long* maxbits, int tag_flags);
hipStream_t ctx_stream(const hotrg_ctx* c);
// Allocation-free entry point's scratch (noalloc.hip): look up this device's
// copy of the static array once (call with the device current).
void noalloc_init_device(int device);
// hotrg_run with a cancellation flag checked between steps.
hotrg_status run_problem(hotrg_ctx* c, const hotrg_model_params* params, const hotrg_opts* o,
                         hotrg_result* res, const std::atomic<bool>* cancel);
void ctx_trim(hotrg_ctx* c);  // release the step workspace
double ctx_seconds(const hotrg_ctx* c);
int ctx_device(const hotrg_ctx* c);
size_t ctx_budget(const hotrg_ctx* c);
bool& ctx_plain(hotrg_ctx* c);  // states made from now on: unpadded FP64 rows
int& ctx_workers(hotrg_ctx* c);
int& ctx_test_fail_step(hotrg_ctx* c);  // failure-injection hook, 0: off
void*& ctx_sched(hotrg_ctx* c);
void sched_shutdown(hotrg_ctx* c);
const char* last_error_text();
void set_last_error(const char* m);

}  // namespace hotrg
