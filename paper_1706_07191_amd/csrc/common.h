// Internal declarations shared by the HIP translation units of libbrsvd (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "brsvd.h"

namespace brsvd {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef double doublex4 __attribute__((ext_vector_type(4)));

constexpr int kMaxL = 512;       // largest sketch width l = k + p
constexpr int kTile = 16;        // MFMA tile edge (v_mfma_f32_16x16x4_f32)

// Padded panel width: every internal thin panel is rows x Lp, row-major, Lp a multiple of 16,
// columns l..Lp-1 kept at zero, so the GEMM kernels need no column masking on their inputs.
inline int padded_l(int l) { return (l + kTile - 1) / kTile * kTile; }
inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

#define BRSVD_HIP_TRY(expr)                         \
  do {                                              \
    hipError_t e__ = (expr);                        \
    if (e__ != hipSuccess) return BRSVD_ERR_HIP;    \
  } while (0)

#define BRSVD_TRY(expr)                 \
  do {                                  \
    int s__ = (expr);                   \
    if (s__ != BRSVD_OK) return s__;    \
  } while (0)

// Products of l x l factors: the waves of a workgroup that share the contraction of one 16 x 16 tile.  Adds their accumulators in wave order, the sum
// is in wave 0, for which it returns true.
constexpr int kTileWaves = 8;
__device__ __forceinline__ bool sum_over_waves(doublex4& acc, double (*part)[256], int lane, int wave) {
#pragma unroll
  for (int v = 0; v < 4; ++v) part[wave][64 * v + lane] = acc[v];
  __syncthreads();
  if (wave != 0) return false;
#pragma unroll
  for (int w = 1; w < kTileWaves; ++w)
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[v] += part[w][64 * v + lane];
  return true;
}

// ---- thin-panel GEMMs (gemm_thin.hip) ------------------------------------------------------
// Optional events for per-kernel timing of one call: stop directly behind the MFMA kernel launch(es), sum_stop behind the
// split-sum kernels that follow (recorded even when there is nothing to sum).  The caller records the start.
struct KernelEvents {
  hipEvent_t stop, sum_stop;
};

// Y (rows x ncols, ldy) = A (rows x K, lda) * X (K x Lp padded panel, ldx = Lp).
// scratch holds partial sums when the launch is split along K.  fp32 and fp64 (esz = element size).
uint64_t gemm_an_scratch_bytes(int64_t rows, int64_t K, int Lp, int esz = 4);
// Bytes of the partial panels that are used where the scratch is also enough for gemm_at of the same A (small products are cut further then).
uint64_t gemm_an_split_bytes(int64_t rows, int64_t K, int Lp, int esz = 4);
int gemm_an(const float* A, int64_t lda, int64_t rows, int64_t K, const float* X, int Lp,
            float* Y, int64_t ldy, int ncols, void* scratch, uint64_t scratch_bytes,
            hipStream_t stream, const KernelEvents* ev = nullptr);
int gemm_an(const double* A, int64_t lda, int64_t rows, int64_t K, const double* X, int Lp,
            double* Y, int64_t ldy, int ncols, void* scratch, uint64_t scratch_bytes,
            hipStream_t stream, const KernelEvents* ev = nullptr);

// Z (n x Lp padded panel) (+)= A^T * Q; A is rows x n (lda), Q is rows x Lp.  The row range is
// cut at multiples of block_rows (the row blocks of the method) and each block into equal
// sub-ranges; partial panels are summed in row order, so the result does not depend on timing.
uint64_t gemm_at_scratch_bytes(int64_t rows, int64_t n, int Lp, int64_t block_rows, int esz = 4);
int gemm_at(const float* A, int64_t lda, int64_t rows, int64_t n, const float* Q, int Lp,
            float* Z, bool accumulate, int64_t block_rows, void* scratch, uint64_t scratch_bytes,
            hipStream_t stream, const KernelEvents* ev = nullptr);
int gemm_at(const double* A, int64_t lda, int64_t rows, int64_t n, const double* Q, int Lp,
            double* Z, bool accumulate, int64_t block_rows, void* scratch, uint64_t scratch_bytes,
            hipStream_t stream, const KernelEvents* ev = nullptr);

// Work partition of Y = A X (described at k_gemm_an): C chunks per tile, whole and leftover row tiles, f main splits,
// tail strips of x chunks, j of them per workgroup.
struct AnShape {
  int C, whole, lt, f, x, j;
};
// The part of workgroup b: chunks [c0, c1) of nseg row tiles from first_tile on, into Y or into partial panel `slot`.
struct AnWork {
  int first_tile, nseg, c0, c1, slot;
  bool partial;
};
__host__ __device__ inline AnWork an_work(const AnShape& sh, int b) {
  AnWork w;
  w.nseg = 1;
  w.slot = 0;
  w.partial = true;
  const int C = sh.C;
  if (b < sh.whole) {
    w.first_tile = b; w.c0 = 0; w.c1 = C; w.partial = false;
  } else if (b < sh.whole + sh.lt * sh.f) {
    const int idx = b - sh.whole, s = idx % sh.f;
    w.first_tile = sh.whole + idx / sh.f;
    w.c0 = (int)((int64_t)s * (C - sh.x) / sh.f);
    w.c1 = (int)((int64_t)(s + 1) * (C - sh.x) / sh.f);
    w.slot = s;
  } else {
    const int i = b - sh.whole - sh.lt * sh.f, left = sh.whole + sh.lt;
    w.first_tile = sh.whole + i * sh.j;
    w.nseg = sh.j < left - w.first_tile ? sh.j : left - w.first_tile;
    w.c0 = C - sh.x; w.c1 = C; w.slot = sh.f;
  }
  return w;
}
AnShape an_shape(int T, int C, int S, int min_piece, int min_strip);

// ---- pieces of the planners and the split sum, shared by gemm_thin.hip and gemm_split.hip ----
struct NGroups {
  int groups, nt;   // column groups per launch sequence, n-tiles per group
};
NGroups column_groups(int Lp, int esz);
double traffic_weight(int nt);
int pick_splits(int64_t tiles, int slots, int64_t units, double out_over_in, double traffic_weight, int max_splits);
int reduce_splits_f32(float* part, int nsplit, int64_t split_stride, int64_t rows, int ncols, int64_t ldi, float* out,
                      int64_t ldo, bool accumulate, hipStream_t stream);

// ---- the same two products for wide fp32 panels on the 16-bit matrix cores (gemm_split.hip, gemm_half.hip) ----
// out x K (an) or K x out (at) is the part of A multiplied; pack is device memory for the split right panel.
// Taken for contractions of at least 512 and 2^22 elements of A, from 48 padded columns on.  Measured, plain fp32 kernel and this one
// (us, A X / A^T Q): 100000x50000 l=272 20944 / 21274 and 12640 / 13114; 20000x20000 l=110 877 / 791 and 514 / 514; 89083x2783 l=97
// 583 / 748 and 336 / 343; 76800x2000 l=40 189 / 197 and 165 / 148; 4000x4000 l=48 36.8 / 30.9 and 31.9 / 25.6.  Below, the extra
// launches cost what the product saves, or the read of A bounds both: 2000x1000 l=60 21.2 / 23.6 and 24.2 / 18.0, 1024x1024 l=300
// 79 / 35.6 and 73 / 36.8, 100000x50000 l=16 3287 / 3266 and 3911 / 3373.
// At 32 padded columns both kernels are near the read of A, and what decides is how they cut and read it (l = 24):
//   A X: this one reads 64 bytes of a row at a time and loses where rows do not start on lines of 128 bytes: 20000x20004 338 and
//     374, 30000x20003 510 and 567, 60000x8007 431 and 468; or where they are short or few: 20000x8000 137 and 143, 8000x16000 113 and
//     118, 1000x8000 25 and 32.  From 14000 columns and 20000 rows on, on lines, it is level or ahead: 20000x20000 306 and 309,
//     30000x14848 343 and 338, 60000x20000 887 and 873, 20000x50016 739 and 716.
//   A^T Q: rows that vectors of 16 bytes do not fit cost the plain kernel a third: 60000x8007 507 and 349, 5003x1001 l=32 29 and 24.
//     Otherwise few rows of A leave the plain one with too few workgroups, 1000x8000 24 and 21, 4000x10000 46 and 39, 6000x20000 112
//     and 94, 2000x50000 95 and 87, and for many its panels are larger, 20000x20000 307 and 274, 60000x20000 832 and 813; between, the
//     plain one is ahead: 12000x14000 128 and 138, 30000x8000 170 and 182, 4000x50000 160 and 173, 8000x24000 144 and 152.
constexpr int64_t kSplitMinK = 512, kSplitMinOut = 64, kSplitMinLp = 32, kSplitMinA = 1 << 22;
struct SplitPlan {
  int tile, groups, nt, nsplit, wgs;           // rows (columns of A) per workgroup, column groups, tiles per group, partial panels
  AnShape sh;                                  // an
  int64_t partial_rows;                        // an: rows of the partial panels
  int col_tiles, blocks, blocks_per_sub;       // at: column tiles, blocks of 32 rows in all and per sub-range
};
SplitPlan split_an_plan(int64_t rows, int64_t K, int Lp, uint64_t scratch_bytes);
SplitPlan split_at_plan(int64_t rows, int64_t n, int Lp, uint64_t scratch_bytes);
bool split_fits(bool at, const float* A, int64_t out, int64_t K, int Lp, int64_t lda, uint64_t pack_bytes);
int split_parts(bool at, int64_t out, int64_t K, int Lp);   // 16-bit numbers an operand is split into, with all the scratch it can use
// X (K x xcols, leading dimension ldx) and Q (rows x qcols, ldq) need no padding; Lp = padded width of the partial panels.  whole: three
// bf16 numbers, which hold all 24 bits of an operand, whatever its length.
int split_gemm_an(const float* A, int64_t lda, int64_t rows, int64_t K, const float* X, int64_t ldx, int xcols, int Lp,
                  float* Y, int64_t ldy, int ncols, void* scratch, uint64_t scratch_bytes, void* pack,
                  uint64_t pack_bytes, hipStream_t stream, const KernelEvents* ev = nullptr, bool whole = false);
int split_gemm_at(const float* A, int64_t lda, int64_t rows, int64_t n, const float* Q, int64_t ldq, int qcols, int Lp,
                  float* Z, int64_t ldz, int ncols, bool accumulate, void* scratch, uint64_t scratch_bytes, void* pack,
                  uint64_t pack_bytes, hipStream_t stream, const KernelEvents* ev = nullptr, bool whole = false);

// Launch plans as numbers (see brsvd_gemm_plan in the C ABI).
void gemm_an_plan_describe(int64_t rows, int64_t K, int Lp, int esz, int32_t out[12]);
void gemm_at_plan_describe(int64_t rows, int64_t n, int Lp, int64_t block_rows, int esz, int32_t out[12]);

// dst (rows x Lp, zero padded) <- src (rows x l dense)
int pad_panel(const float* src, int64_t rows, int l, float* dst, int Lp, hipStream_t stream);
int pad_panel(const double* src, int64_t rows, int l, double* dst, int Lp, hipStream_t stream);
// dst (rows x l dense) (+)= src (rows x Lp) restricted to the first l columns
int unpad_panel(const float* src, int64_t rows, int Lp, int l, float* dst, bool accumulate, hipStream_t stream);
int unpad_panel(const double* src, int64_t rows, int Lp, int l, double* dst, bool accumulate, hipStream_t stream);
// dst (l x rows, ld = rows) <- transpose of src (rows x Lp) restricted to the first l columns
int transpose_panel(const float* src, int64_t rows, int Lp, int l, float* dst, hipStream_t stream);
int transpose_panel(const double* src, int64_t rows, int Lp, int l, double* dst, hipStream_t stream);

// ---- orthonormalisation (orth.hip, tsqr.hip) -----------------------------------------------
// T = element type of the panels (float or double); the l x l factors are fp64 either way.
template <typename T>
struct OrthWorkT {
  double* gram_part;   // gram_chunks_max slots of Lp x Lp partial Gram sums (orth_gram_slots)
  int gram_chunks_max;
  double* G;           // Lp x Lp
  double* R[2];        // upper-triangular factors of the two CholeskyQR sweeps (stride Lp)
  T* Rinv;             // Lp x Lp zero-padded inverse factor in the panels' type (right operand of the apply GEMM)
  bool G_of_panel = false;   // G is already the Gram matrix of the panel that is orthonormalised next (an_gram)
  int* flags;          // device: [0] = breakdown flag (0 = none, else 1 + column), [1] = the last basis was far from orthonormal (orth_basis)
  void* gemm_scratch;
  uint64_t gemm_scratch_bytes;
  void* tsqr_work;     // TSQR scratch; otherwise partial Gram sums
  uint64_t tsqr_bytes;
  // Optional companion panel (comp_rows x Lp): every R^-1 applied to the panel being orthonormalised
  // is applied to it as well (comp <- comp * R^-1, ping-ponging with comp_tmp; the result is in comp).
  T* comp = nullptr;
  T* comp_tmp = nullptr;
  int64_t comp_rows = 0;
};
typedef OrthWorkT<float> OrthWork;
// out (rows x ncols, leading dimension ldo) = P X; P: rows x Lp padded panel, X: zero-padded Lp x Lp factor.  scratch as for gemm_an.
template <typename T>
int apply_panel(const T* P, int64_t rows, int Lp, const T* X, T* out, int64_t ldo, int ncols, void* scratch, uint64_t scratch_bytes,
                hipStream_t stream);
// Y (rows x Lp) = A X with the Gram matrix of Y in w.G, for tall matrices of short rows: the next orthonormalisation by CholeskyQR on w starts from
// there.
bool an_gram_fits(int64_t rows, int64_t K, int Lp, int esz);
int an_gram(const float* A, int64_t lda, int64_t rows, int64_t K, const float* X, int Lp, float* Y, OrthWork& w, hipStream_t stream,
            const KernelEvents* ev);
// Applies the current w.Rinv to the companion panel, if any.
template <typename T> int apply_to_companion(OrthWorkT<T>& w, int Lp, hipStream_t stream);
uint64_t orth_gram_slots(int64_t rows, int Lp);   // Lp x Lp fp64 slots of partial Gram sums for such a panel
uint64_t tsqr_work_bytes(int64_t rows, int Lp);
// Orthonormalises the columns of P (rows x Lp padded panel, rows >= l).  tmp is a second
// rows x Lp buffer; *result is set to whichever of P / tmp holds the orthonormal panel.
// Rtot (stride Lp, fp64, may be null) receives the triangular factor with P_in = Q * Rtot.
// Asynchronous: a CholeskyQR breakdown is only reported through w.flags[0] on the device.
// final_basis = false: the panel only seeds the next power half step (one CholeskyQR sweep).
template <typename T>
int orth_panel(T* P, T* tmp, int64_t rows, int l, int Lp, int method, bool final_basis, OrthWorkT<T>& w,
               double* Rtot, T** result, hipStream_t stream);
// The same for a basis that reaches the output, with the last l x l factor left to the caller: the orthonormal basis of P is panel * left (left
// null: the panel itself), and with want_R P = panel * R1, left^-1 = R2 (null if left is).  left: room for an Lp x Lp factor; Rtot: for
// an fp64 one, used with want_R only.  settle: panel is next to orthonormal by itself; w.Rinv and w.flags[1] are used for it.
template <typename T>
struct Basis {
  T* panel;
  const T* left;
  const double *R1, *R2;
};
template <typename T>
int orth_basis(T* P, T* tmp, int64_t rows, int l, int Lp, int method, OrthWorkT<T>& w, T* left, double* Rtot, bool want_R, bool settle,
               Basis<T>* out, hipStream_t stream);
// Pieces shared between the CholeskyQR and the Householder-tree routes (orth.hip, tsqr.hip).
template <typename T>
int cholqr_sweeps(T* P, T* tmp, int64_t rows, int l, int Lp, int nsweeps, OrthWorkT<T>& w, double* Rtot,
                  T** result, hipStream_t stream, bool strict_last, bool publish_R = false);
template <typename T>
int chol_inv_factored(double* G, int l, int Lp, double* Rout, T* Rinv, int* flags, hipStream_t stream);
template <typename T>
int tsqr_panel(T* P, T* tmp, int64_t rows, int l, int Lp, OrthWorkT<T>& w, double* Rtot, T** result,
               hipStream_t stream);
// C = A B, upper triangular l x l factors (strides Lp)
template <typename TB>
int triu_mul(const double* A, const TB* B, int l, int Lp, double* C, hipStream_t stream);
// *out (device) = min |R_ii| / max |R_ii| of the l x l triangular factor R (stride Lp)
int diag_ratio(const double* R, int l, int Lp, double* out, hipStream_t stream);

// ---- small SVD (small_svd.hip) -------------------------------------------------------------
struct SvdWork {
  double* W;     // Lp x Lp rows being orthogonalised
  double* sig;   // 3 * Lp
  int* info;     // device, eight: [0] sweeps, [1] converged, the others for the iteration itself
};
// The work of the block Jacobi iteration in the order in which its workgroups take it: a ticket is one of the P = nblk2 / 2 block
// pairs of one of the nblk2 - 1 rounds of a sweep (from 0).  Its turn comes once all tickets of the rounds before are done.
struct JacobiTicket {
  int sweep, round, pair, before;    // before: tickets of the earlier rounds
};
__host__ __device__ inline JacobiTicket jacobi_ticket(int ticket, int nblk2) {
  const int P = nblk2 / 2, r = ticket / P;
  return JacobiTicket{r / (nblk2 - 1), r % (nblk2 - 1), ticket - r * P, r * P};
}
// What a ticket is, when its turn has come and `last` is the latest sweep (from 1) that turned a pair above the settled bar: that sweep
// is not the one before, or there have been enough: no more rotations, and the tickets that would have been the next two rounds
// work out the norms and the ranks.
enum { JACOBI_ROTATE = 0, JACOBI_NORMS, JACOBI_RANKS, JACOBI_END };
__host__ __device__ inline int jacobi_work(const JacobiTicket& k, int last, int max_sweeps) {
  if (k.sweep == 0 || (last >= k.sweep && k.sweep < max_sweeps)) return JACOBI_ROTATE;
  return k.round == 0 ? JACOBI_NORMS : (k.round == 1 ? JACOBI_RANKS : JACOBI_END);
}
// R (l x l fp64, stride ldr): R = Ur diag(S) Vr^T.  Writes S (descending) as fp64 and/or in the
// panels' type TO, the zero-padded (Lp x Lp) operands XV = Vr and XU = Ur used by the lifts (type TO),
// and optional dense fp64 l x l Ur / Vr.  Skips the work when *breakdown_flag != 0.
// open: the lifts' panels are not orthonormal yet (see Basis): XV = left Vr (left null: Vr) and XU = Rx Vr / diag(S), Rx upper triangular with
// stride ldr; there are no dense results then.
template <typename TO>
struct OpenFactors {
  const TO* left;
  const double* Rx;
};
template <typename TO>
int small_svd(const double* R, int ldr, int l, int Lp, SvdWork& w, const int* breakdown_flag,
              double* S, TO* S32, TO* XV, TO* XU, double* Ur, double* Vr, hipStream_t stream, const OpenFactors<TO>* open = nullptr);

// ---- robust-PCA elementwise kernels (rpca.hip) ---------------------------------------------
// Number of doubles of partial-sum scratch the reductions below need.
uint64_t rpca_part_doubles(int64_t m, int64_t n);
// scal[0] = max |M_ij|, scal[1] = ||M||_F^2 (device doubles).  T = float or double throughout.
template <typename T> int rpca_norms(const T* M, int64_t count, double* part, double* scal, hipStream_t stream);
// Y0 = M * inv_J, X0 = M - S0 + Y0 * inv_mu with S0 = 0
template <typename T>
int rpca_init(const T* M, int64_t count, T inv_J, T inv_mu, T* Y, T* X, hipStream_t stream);
// Fused update after the SVD of X_i: with L = U diag(shrink(sig, 1/mu)) Vt (contraction over l) and
// S = shrink(M - L + Yin/mu, lambda/mu) formed in registers, writes Yout = Yin + mu (M - L - S), the next SVD input
// X = M - S + Yout/mu_next and per-workgroup partial sums of ||M-L-S||_F^2 into `part` (*nparts_out of them); L and
// S themselves are not stored.  U is m x l (ld l), Vt is l x n (ld n); Yout may be Yin.  rpca_residual_sum then adds
// the partial sums into *resid2_out in a fixed order.
template <typename T>
int rpca_update(const T* M, const T* U, const T* sig, const T* Vt, int64_t m, int64_t n, int l, T mu, T lambda,
                T mu_next, const T* Yin, T* Yout, T* X, double* part, int* nparts_out, hipStream_t stream);
int rpca_residual_sum(double* part, int nparts, double* resid2_out, hipStream_t stream);
// L and S of the iteration that used (U, sig, Vt, mu) and read the multiplier Yin, with the arithmetic of rpca_update.
// Lout may be Yin.
template <typename T>
int rpca_finalize(const T* M, const T* U, const T* sig, const T* Vt, int64_t m, int64_t n, int l, T mu, T lambda,
                  const T* Yin, T* Lout, T* S, hipStream_t stream);
// `iters` steps x = z / |z|, y = A x, z = A^T y of the power method, z = x0 at first; *y2 (device) = |y|^2 of the last.  z: n elements of
// workspace.  For rows that a workgroup can hold, and scratch for at least 64 parts of z (power_fits).
template <typename T> bool power_fits(int64_t m, int64_t n, uint64_t scratch_bytes);
template <typename T>
int power_method(const T* A, int64_t lda, int64_t m, int64_t n, const T* x0, int iters, T* z, void* scratch, uint64_t scratch_bytes,
                 double* y2, hipStream_t stream);
// P[0..count) *= 1 / sqrt(*s2) (device scalar; a zero scalar zeroes P, NaN makes it NaN).
template <typename T> int scale_rsqrt(T* P, int64_t count, const double* s2, hipStream_t stream);

// ---- device-side Gaussian generator (philox.hip) -------------------------------------------
// Rows [row0, row0 + rows) of the m x l matrix Omega(seed) (Philox4x32-10 + Box-Muller, element
// e = row*l + col from output e&3 of counter e>>2) into out (rows x ld, columns l..ld-1 zeroed).
template <typename T>
int philox_normal(uint64_t seed, int64_t row0, int64_t rows, int l, T* out, int ld, hipStream_t stream);

// ---- machine probes (probe.hip) -------------------------------------------------------------
int probe(int kind, void* buf, uint64_t amount, double* seconds, double* work, hipStream_t stream);

}  // namespace brsvd
