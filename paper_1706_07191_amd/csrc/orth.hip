// Orthonormalisation of tall thin panels (Alg. 1 step 3, Alg. 2 line 6) on gfx950.
//
// Main route: CholeskyQR.  G = P^T P is accumulated in fp64 (products of fp32 values are exact in fp64), factored
// G = R^T R in fp64, and P <- P * R^-1 is one more thin GEMM on the MFMA path.  A basis that reaches the output gets a second
// factor, which goes into the l x l factors that the panel meets later (orth_basis) or is applied too (orth_panel).  Pivots
// that fall below a relative threshold are clamped in every sweep but the last one of an output basis; there such a pivot
// raises the breakdown flag and the caller switches to the Householder-based TSQR route (tsqr.hip).
// The paper orthonormalises with a TSQR-based CAQR; range(P) -- all the method needs -- is the
// same for any orthonormalisation.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "common.h"

namespace brsvd {

// ---- Gram matrix -----------------------------------------------------------------------------
// G = P^T P on the fp64 matrix cores (v_mfma_f64_16x16x4_f64; products of fp32 values are exact in
// fp64; the panel may also be fp64).  The columns are cut into blocks of up to four tiles of 16; grid = (row chunks, pairs bi <= bj of
// blocks).  Lane (r, g) of a wave takes W neighbouring columns of row g of four rows with one load, W r .. W r + W - 1 of the block's 16 W: number t
// of them is its operand of tile t, whose columns are thus t, W + t, 2 W + t, ...; the same value is the A operand (entry [i = r][k = g] of the
// transposed tile) and the B operand ([k = g][j = r]), so the panel goes from global memory straight into the MFMA operands, in lines.
// The eight waves of a workgroup take AH steps of four rows at a time round-robin, the next ones' loads under way, and
// add their accumulators through LDS in wave order; the chunks are added by k_gram_sum.
// Accumulator layout of the instruction: component v of lane (r, g) is entry [g + 4*v][r].
// Measured, with one load of four bytes per tile and step, and this (us):
// 2073600x32 83 and 64, 76800x32 20 and 9, 40000x64 28 and 19, 20000x112 18.5 and 15, 100000x160 91 and 65, 100000x272 226 and 175, fp64 15872x80
// 12.7 and 8.2.
constexpr int kGramWaves = 8;

__device__ __forceinline__ doublex4 mfma_f64(double a, double b, doublex4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// W neighbouring numbers of a row.
template <typename T, int W>
__device__ __forceinline__ void load_run(const T* p, T (&v)[W]) {
  if constexpr (W == 2 || W == 4) {
    typedef T vec __attribute__((ext_vector_type(W)));
    const vec x = *(const vec*)p;
#pragma unroll
    for (int t = 0; t < W; ++t) v[t] = x[t];
  } else {
#pragma unroll
    for (int t = 0; t < W; ++t) v[t] = p[t];
  }
}

// The sums of WAVES waves' accumulators, in wave order, to the workgroup's part Go of G: block of columns ci .. ci + 16 TI, cj .. cj + 16 TJ.  red:
// room for two tiles per wave.
template <int TI, int TJ, bool DIAG, int WAVES, int TILES>
__device__ __forceinline__ void gram_store(const doublex4 (&acc)[TILES], int Lp, int ci, int cj, double* red, double* Go, int tid) {
  const int lane = tid & 63, wave = tid >> 6;
  constexpr int PASS = TILES < 2 ? TILES : 2;
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = DIAG ? i : 0; j < TJ; ++j) {
      const int t = DIAG ? i * TI - i * (i - 1) / 2 + j - i : i * TJ + j;
#pragma unroll
      for (int v = 0; v < 4; ++v) red[(wave * PASS + t % PASS) * 256 + 64 * v + lane] = acc[t][v];
      if (t % PASS != PASS - 1 && t + 1 != TILES) continue;
      __syncthreads();
      // entry e of tile tt; the thread also writes the entry's mirror image where that lies in an upper tile and no tile of its own has it
      const int e = tid & 255;
#pragma unroll
      for (int h = tid >> 8; h < PASS; h += WAVES / 4) {
        const int tt = t - t % PASS + h;
        if (tt > t) continue;
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) s += red[(w * PASS + h) * 256 + e];
        int ti = 0, tj = tt;
        while (tj >= (DIAG ? TI - ti : TJ)) { tj -= DIAG ? TI - ti : TJ; ++ti; }
        if (DIAG) tj += ti;
        const int x = ci + TI * (((e & 63) >> 4) + 4 * (e >> 6)) + ti, y = cj + TJ * (e & 15) + tj;
        if (!DIAG || x / 16 <= y / 16) Go[(int64_t)x * Lp + y] = s;
        if (DIAG && ti != tj && y / 16 <= x / 16) Go[(int64_t)y * Lp + x] = s;
      }
      __syncthreads();
    }
}

// The part of a chunk, rows [rbeg, rend), in the block of columns ci .. ci + 16 TI, cj .. cj + 16 TJ of G.
template <typename T, int TI, int TJ, bool DIAG>
__device__ __forceinline__ void gram_block(const T* P, int Lp, int ci, int cj, int64_t rbeg, int64_t rend, double* red, double* Go, int tid) {
  constexpr int AH = TI <= 2 ? 4 : 2, BJ = DIAG ? 1 : TJ, TILES = DIAG ? TI * (TI + 1) / 2 : TI * TJ;
  const int lane = tid & 63, wave = tid >> 6, r = lane & 15, g = lane >> 4;
  doublex4 acc[TILES];
#pragma unroll
  for (int t = 0; t < TILES; ++t) acc[t] = doublex4{0.0, 0.0, 0.0, 0.0};
  T an[AH][TI], bn[AH][BJ];
  const T *pi = P + ci + TI * r, *pj = P + cj + TJ * r;
  auto load = [&](int64_t row0) {
#pragma unroll
    for (int s = 0; s < AH; ++s) {
      const int64_t off = (row0 + 4 * s + g) * Lp;
      load_run(pi + off, an[s]);
      if constexpr (!DIAG) load_run(pj + off, bn[s]);
    }
  };
  auto multiply = [&](const T (&a0)[AH][TI], const T (&b0)[AH][BJ]) {
#pragma unroll
    for (int s = 0; s < AH; ++s) {
      double a[TI], b[TJ];
#pragma unroll
      for (int t = 0; t < TI; ++t) a[t] = (double)a0[s][t];
#pragma unroll
      for (int t = 0; t < TJ; ++t) b[t] = DIAG ? a[t % TI] : (double)b0[s][t % BJ];
      int t = 0;
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = DIAG ? i : 0; j < TJ; ++j) { acc[t] = mfma_f64(a[i], b[j], acc[t]); ++t; }
    }
  };
  constexpr int STEP = 4 * AH;
  int64_t row0 = rbeg + STEP * wave;
  if (row0 + STEP <= rend) load(row0);
#pragma nounroll
  for (; row0 + STEP <= rend; row0 += STEP * kGramWaves) {
    T a[AH][TI], b[AH][BJ];
#pragma unroll
    for (int s = 0; s < AH; ++s) {
#pragma unroll
      for (int t = 0; t < TI; ++t) a[s][t] = an[s][t];
      if constexpr (!DIAG) {
#pragma unroll
        for (int t = 0; t < BJ; ++t) b[s][t] = bn[s][t];
      }
    }
    const int64_t next = row0 + STEP * kGramWaves;
    load(next + STEP <= rend ? next : row0);               // under way while these rows are multiplied (the last time round: not used)
    multiply(a, b);
  }
  if (row0 < rend) {                                       // the chunk's last rows, fewer than a step
#pragma unroll
    for (int s = 0; s < AH; ++s) {
      const int64_t row = row0 + 4 * s + g, off = min(row, rend - 1) * Lp;
      load_run(pi + off, an[s]);
#pragma unroll
      for (int t = 0; t < TI; ++t) an[s][t] = row < rend ? an[s][t] : T(0);
      if constexpr (!DIAG) load_run(pj + off, bn[s]);
    }
    // (a row that is not there meets zeros on one side; on the other it is a copy of one that is, which may not be finite)
    if constexpr (!DIAG) {
#pragma unroll
      for (int s = 0; s < AH; ++s)
#pragma unroll
        for (int t = 0; t < TJ; ++t) bn[s][t] = row0 + 4 * s + g < rend ? bn[s][t] : T(0);
    }
    multiply(an, bn);
  }
  gram_store<TI, TJ, DIAG, kGramWaves>(acc, Lp, ci, cj, red, Go, tid);
}

// MAXB: tiles of a block at most; 1 to 3 where that is the whole matrix.
template <typename T, int MAXB>
__global__ void __launch_bounds__(kGramWaves * 64)
k_gram(const T* __restrict__ P, int64_t rows, int Lp, int64_t rows_per_chunk, double* __restrict__ Gpart) {
  __shared__ double red[kGramWaves * 2 * 256];
  const int tid = threadIdx.x;
  const int64_t rbeg = (int64_t)blockIdx.x * rows_per_chunk, rend = min(rows, rbeg + rows_per_chunk);
  double* Go = Gpart + (int64_t)blockIdx.x * Lp * Lp;
  if constexpr (MAXB < 4) {
    gram_block<T, MAXB, MAXB, true>(P, Lp, 0, 0, rbeg, rend, red, Go, tid);
  } else {
    // blocks of equal size, or one tile more: two and three tiles for five in all, otherwise three and four (or a single one of four)
    const int NT = Lp / 16, nb = (NT + 3) / 4;
    int bi = 0, rem = blockIdx.y;
    while (rem >= nb - bi) { rem -= nb - bi; ++bi; }
    const int bj = bi + rem, t0 = bi * NT / nb, t1 = bj * NT / nb, ni = (bi + 1) * NT / nb - t0, nj = (bj + 1) * NT / nb - t1;
#define CALL(NI, NJ, DIAG) gram_block<T, NI, NJ, DIAG>(P, Lp, 16 * t0, 16 * t1, rbeg, rend, red, Go, tid)
    if (bi == bj) {
      if (ni == 4) CALL(4, 4, true);
      else if (ni == 3) CALL(3, 3, true);
      else CALL(2, 2, true);
    } else if (ni == 4) {
      if (nj == 4) CALL(4, 4, false);
      else CALL(4, 3, false);
    } else if (ni == 3) {
      if (nj == 4) CALL(3, 4, false);
      else CALL(3, 3, false);
    } else {
      CALL(2, 3, false);
    }
#undef CALL
  }
}

// ---- Cholesky factor and its inverse ---------------------------------------------------------
// One workgroup; everything is fp64, in 16 x 16 tiles on v_mfma_f64_16x16x4_f64.  G = R^T R is eliminated with the
// identity beside it: the row operations that turn G into R turn the identity into E = R^-T, so the inverse needs no
// pass of its own.  With E_kk = R_kk^-T, step k is
//   pan_c   = E_kk M_kc for every column tile c: R_kc for c > k, E_kc for c < k  (pan_k = E_kk)
//   M_ic   -= R_ki^T pan_c for the rows i > k, columns c <= k (E) and c >= i (what is left of G)
// where M holds G in its upper tiles and E in its lower ones (zero before step c).  Row k is final after its panel:
// R and R^-1 = E^T are written out from there.  The diagonal tile of the next step is updated and
// factored by wave 0 while the other waves finish the update of step k, which takes the chain of 16 pivots
// off the path of everything else: a step is the longer of the two plus the panel and two barriers.
//
// What bounds it: the chain of pivots (375 cycles each: a matrix instruction, two lane reads, a reciprocal with two
// Newton steps, the scale of the row) up to l of 128, where M is in LDS; above that M stays in global memory (L2) and the
// tile updates, 2 l^3 / 3 flops on one CU, take over.  Measured (us with the launch; before: the factorisation with
// row-wise panel solves, then a recursive inversion): l = 20 19.8 -> 11.3, 60 38.0 -> 20.2, 110 73.7 -> 33.1,
// 128 87.4 -> 38.9, 160 151 -> 65, 272 383 -> 208, 400 895 -> 562.  Since then padding needs no pivots: l = 20 9.4 -> 8.3.
// A pivot <= tol * its original diagonal entry is clamped to that value (lenient) or sets
// flag[0] = 1 + column of its tile and ends the kernel.
// A matrix close to the identity, as in the second sweep of CholeskyQR and after a Householder tree, needs no elimination: for G = I + E, and N the
// strict upper triangle and half the diagonal of E, the factor is R = I + N - H, H the strict upper triangle and half the diagonal of N^T N,
// and R^-1 = I - N, to the orders |E|_F^3 and |E|_F^2.  R^-1 is rounded to the panels' precision, R stays in fp64.  Taken where |E|_F is at most
// `near_eye` (near_eye_of).  Measured, elimination and this with R (us): l = 20 8.0 and 4.0, 72 21 and 7.0, 97 30 and 11, 110 31 and 11, 160 62 and
// 29, 272 192 and 97, 400 526 and 255; without R 7.6 and 3.4, 21 and 4.7, 28 and 7.3, 30 and 6.2, 58 and 12, 177 and 28, 494 and 61.
// far_inv: if |E|_F is above kFarFromEye, R^-1 goes there, the identity into its own place and 1 into flag[1], otherwise 0 (see k_apply_far).
constexpr int kNB = 16;
constexpr double kFarFromEye = 0.1;
constexpr int kCholLdsMaxLp = 128;    // largest padded size whose fp64 matrix fits the LDS

// Row strides (in doubles): 16 modulo 32 puts the four rows a wave reads at once on distinct banks; the matrix of
// the largest sizes has no room for that and takes two doubles of padding.
static constexpr int chol_ldp(int Lp) { return Lp % 32 == 0 ? Lp + 16 : Lp; }
static constexpr int chol_ldm(int Lp) { return Lp % 32 == 0 ? (Lp < 128 ? Lp + 16 : Lp + 2) : Lp; }
static constexpr size_t chol_lds_bytes(int Lp, bool in_lds) {
  return sizeof(double) * ((size_t)kNB * (kNB + 1) + Lp + (size_t)kNB * chol_ldp(Lp) + (in_lds ? (size_t)Lp * chol_ldm(Lp) : 0));
}

// Broadcast of lane `src` (a compile-time constant after unrolling): two scalar lane reads.
__device__ __forceinline__ double shfl_d(double v, int src) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), src);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), src);
  return __hiloint2double(hi, lo);
}
// 1/sqrt(x) and 1/x: hardware seed plus two Newton steps (full fp64 accuracy for normal x).
__device__ __forceinline__ double rsqrt_fast(double x) {
  double y = __builtin_amdgcn_rsq(x);
  const double h = 0.5 * x;
  y = fma(y, fma(-h * y, y, 0.5), y);
  y = fma(y, fma(-h * y, y, 0.5), y);
  return y;
}
__device__ __forceinline__ double rcp_fast(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = fma(y, fma(-x, y, 1.0), y);
  y = fma(y, fma(-x, y, 1.0), y);
  return y;
}

// One wave: factors the diagonal tile D (upper triangle) and inverts the factor, both in the accumulator layout of the
// matrix instruction (component v of lane (r, g) is entry [g + 4 v][r]).  The elimination is D = L d L^T without square
// roots: row j of D sits in component j >> 2 of the lanes of group j & 3, which is where the instruction expects
// contraction index j & 3 of both operands, so a pivot step is one instruction for D and one for the identity E,
//   D -= (row_j / d_j)^T row_j,  E -= (row_j / d_j)^T E_j   (first operand masked to the rows below j),
// with no value moved between lanes.  The next pivot is taken from the old tile, d_(j+1) = D_(j+1,j+1) -
// D_(j,j+1)^2 / d_j, so its reciprocal is worked out while the instruction runs.  Rows are scaled by 1/sqrt(d)
// at the end: D = R_kk, E = R_kk^-T.  cnt: rows of the tile that are not padding (those are rows of the identity and need no pivots).  FACTORED: D
// is already R_kk.  d0: original diagonal of the tile.  Returns false if a pivot had to be clamped.
template <bool FACTORED>
__device__ __forceinline__ bool chol_diag_wave(doublex4& D, doublex4& E, const double* d0, double tol, int lane, int cnt) {
  const int r = lane & 15, g = lane >> 4;
  const double floors = tol * d0[r];
  doublex4 ds;
#pragma unroll
  for (int v = 0; v < 4; ++v) { E[v] = g + 4 * v == r ? 1.0 : 0.0; ds[v] = 1.0; }
  int clamped = 0;
  auto pivot = [&](int j, double d) {
    if (FACTORED) return d;
    const double floor_ = shfl_d(floors, j);
    const bool low = !(d > floor_);
    clamped |= low;
    return low ? (floor_ > 0.0 ? floor_ : 1.0) : d;            // an all-zero column keeps R_jj = 1
  };
  double d = pivot(0, shfl_d(D[0], 0)), inv = rcp_fast(d);
#pragma unroll
  for (int j = 0; j < kNB; ++j) {
    const bool mine = g == (j & 3);
    ds[j >> 2] = mine ? d : ds[j >> 2];
    if (j + 1 >= cnt) break;
    if (j + 1 < kNB) {
      const double x = shfl_d(D[j >> 2], 16 * (j & 3) + j + 1), dn = shfl_d(D[(j + 1) >> 2], 16 * ((j + 1) & 3) + j + 1);
      const double a = mine && r > j ? D[j >> 2] * -inv : 0.0;
      if (!FACTORED) D = mfma_f64(a, D[j >> 2], D);
      // the chain of the next pivot between the two matrix instructions: the second would wait for the first otherwise,
      // and everything behind it
      __builtin_amdgcn_sched_barrier(0);
      d = pivot(j + 1, FACTORED ? dn : fma(-x * inv, x, dn));
      inv = rcp_fast(d);
      __builtin_amdgcn_sched_barrier(0);
      E = mfma_f64(a, E[j >> 2], E);
    }
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int i = g + 4 * v;
    const double sc = FACTORED ? rcp_fast(ds[v]) : rsqrt_fast(ds[v]);
    E[v] *= sc;
    if (!FACTORED) D[v] = i == r ? ds[v] * sc : D[v] * sc;
    D[v] = i <= r ? D[v] : 0.0;
  }
  return clamped == 0;
}

template <bool IN_LDS, bool FACTORED, typename TO>
__global__ void __launch_bounds__(1024)
k_chol_inv(double* __restrict__ G, int l, int Lp, double* __restrict__ Rout, TO* __restrict__ Rinv_out,
           int* __restrict__ flag, double tol, int lenient, double near_eye, TO* __restrict__ far_inv) {
  extern __shared__ double smem[];
  __shared__ int bad;
  __shared__ double off_eye[16];
  const int ldp = chol_ldp(Lp), ld = IN_LDS ? chol_ldm(Lp) : Lp;
  double* e = smem;                                // 16 x 17: E_kk
  double* d0 = e + kNB * (kNB + 1);                // Lp: original diagonal
  double* pan = d0 + Lp;                           // 16 x ldp
  double* M = IN_LDS ? pan + kNB * ldp : G;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
  const int r = lane & 15, g = lane >> 4, nb = Lp / kNB;
  if (flag[0] != 0) return;           // an earlier panel already broke down: results are void anyway
  if (tid == 0) bad = 0;

  // The matrix is padded to Lp x Lp with an identity block; R^-1 is zero below its diagonal tiles and in the padding.
  for (int idx = tid; idx < Lp * Lp; idx += blockDim.x) Rinv_out[idx] = TO(0);
  double e2 = 0.0;                    // |G - I|_F^2
  for (int t = wave; t < nb * (nb + 1) / 2; t += nw) {
    int ti = 0, rem = t;
    while (rem >= nb - ti) { rem -= nb - ti; ++ti; }
    const int tj = ti + rem, col = kNB * tj + r;
    double v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int row = kNB * ti + g + 4 * q;
      const bool in = row < l && col < l;
      v[q] = G[(int64_t)(in ? row : 0) * Lp + (in ? col : 0)];
      if (!in) v[q] = row == col ? 1.0 : 0.0;
      const double e = v[q] - (row == col ? 1.0 : 0.0);
      e2 = fma(ti == tj ? e : 2.0 * e, e, e2);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int row = kNB * ti + g + 4 * q;
      if (IN_LDS || row >= l || col >= l) M[(int64_t)row * ld + col] = v[q];
      if (row == col) d0[row] = v[q];
    }
  }
  if (!FACTORED && near_eye > 0.0) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) e2 += __shfl_xor(e2, off, 64);
    if (lane == 0) off_eye[wave] = e2;
    __syncthreads();
    e2 = 0.0;
    for (int w = 0; w < nw; ++w) e2 += off_eye[w];
    if (far_inv) {
      const bool far = !(e2 <= kFarFromEye * kFarFromEye);
      if (tid == 0) flag[1] = far;
      if (far) {
        for (int idx = tid; idx < Lp * Lp; idx += blockDim.x) far_inv[idx] = TO(0);
        for (int i = tid; i < l; i += blockDim.x) Rinv_out[(int64_t)i * Lp + i] = TO(1);
        Rinv_out = far_inv;
      }
    }
    if (e2 <= near_eye * near_eye) {  // (not when it is NaN)
      const bool second = Rout && e2 > 1.6e-17;            // otherwise H is less than a rounding
      auto n_at = [&](int i, int j) {
        const double v = M[(int64_t)i * ld + j];
        return i < j ? v : (i == j ? 0.5 * (v - 1.0) : 0.0);
      };
      for (int t = wave; t < nb * (nb + 1) / 2; t += nw) {
        int ti = 0, rem = t;
        while (rem >= nb - ti) { rem -= nb - ti; ++ti; }
        const int tj = ti + rem, col = kNB * tj + r;
        doublex4 h = {0.0, 0.0, 0.0, 0.0};
        if (second) {
          double a[4], b[4];
          const double *pa = M + (int64_t)g * ld + kNB * ti + r, *pb = M + (int64_t)g * ld + col;
          for (int k = 0; k < ti; ++k) {                     // tiles above the diagonal ones: N is E there
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) { a[kk] = pa[4 * kk * ld]; b[kk] = pb[4 * kk * ld]; }
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) h = mfma_f64(a[kk], b[kk], h);
            pa += kNB * ld;
            pb += kNB * ld;
          }
#pragma unroll
          for (int kk = 0; kk < 4; ++kk) {
            a[kk] = n_at(kNB * ti + 4 * kk + g, kNB * ti + r);
            b[kk] = n_at(kNB * ti + 4 * kk + g, col);
          }
#pragma unroll
          for (int kk = 0; kk < 4; ++kk) h = mfma_f64(a[kk], b[kk], h);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int row = kNB * ti + g + 4 * v;
          if (row >= l || col >= l) continue;
          const double d = row == col ? 1.0 : 0.0, n = n_at(row, col);
          if (row <= col) Rinv_out[(int64_t)row * Lp + col] = (TO)(d - n);
          if (Rout) {
            Rout[(int64_t)row * Lp + col] = row <= col ? d + (n - (row == col ? 0.5 : 1.0) * h[v]) : 0.0;
            if (ti < tj) Rout[(int64_t)col * Lp + row] = 0.0;
          }
        }
      }
      return;
    }
  }
  // the diagonal tile of step k (wave 0), its factor stored, E_kk left for the panel
  auto diagonal = [&](int k, doublex4 D) {
    doublex4 E;
    const bool ok = chol_diag_wave<FACTORED>(D, E, d0 + kNB * k, tol, lane, min(kNB, l - kNB * k));
    if (!ok && !lenient && lane == 0) bad = kNB * k + 1;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = g + 4 * v, row = kNB * k + i, col = kNB * k + r;
      e[i * (kNB + 1) + r] = E[v];
      if (Rout && row < l && col < l) Rout[(int64_t)row * Lp + col] = D[v];
    }
  };

  // Step k = -1 only factors the first diagonal tile (one copy of that long code serves every step).
  for (int k = -1; k < nb; ++k) {
    __syncthreads();                  // E_kk is in place, the update of step k - 1 is complete
    if (bad) {
      if (tid == 0) flag[0] = bad;
      return;
    }
    // ---- panel: row k of R and of E, and their stores ----
    const int row0 = kNB * k;
    for (int c = k < 0 ? nb : wave; c < nb; c += nw) {
      const int c0 = kNB * c;
      doublex4 acc = {0.0, 0.0, 0.0, 0.0};
      if (c == k) {
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[v] = e[(g + 4 * v) * (kNB + 1) + r];
      } else if (FACTORED && c > k) {
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[v] = M[(int64_t)(row0 + g + 4 * v) * ld + c0 + r];
      } else {
        double b[4];
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) b[kk] = M[(int64_t)(row0 + 4 * kk + g) * ld + c0 + r];
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) acc = mfma_f64(e[r * (kNB + 1) + 4 * kk + g], b[kk], acc);
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = row0 + g + 4 * v, j = c0 + r;
        pan[(g + 4 * v) * ldp + j] = acc[v];
        if (i < l && j < l) {
          if (c > k) { if (Rout) { Rout[(int64_t)i * Lp + j] = acc[v]; Rout[(int64_t)j * Lp + i] = 0.0; } }
          else Rinv_out[(int64_t)j * Lp + i] = (TO)acc[v];
        }
      }
    }
    __syncthreads();
    // ---- update of the rows below, a few tiles at a time so that their loads overlap ----
    const int a = nb - 1 - k;                       // rows left
    auto update = [&](int i, int c, doublex4 acc) {
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        const double* p = pan + (4 * kk + g) * ldp + r;
        acc = mfma_f64(-p[kNB * i], p[kNB * c], acc);
      }
      return acc;
    };
    auto load = [&](int i, int c) {
      doublex4 t = {0.0, 0.0, 0.0, 0.0};
      if (c != k) {
#pragma unroll
        for (int v = 0; v < 4; ++v) t[v] = M[(int64_t)(kNB * i + g + 4 * v) * ld + kNB * c + r];
      }
      return t;
    };
    if (wave == 0) {
      if (a > 0) {
        doublex4 t = load(k + 1, k + 1);
        if (!FACTORED && k >= 0) t = update(k + 1, k + 1, t);
        __builtin_amdgcn_s_setprio(3);
        diagonal(k + 1, t);
        __builtin_amdgcn_s_setprio(0);
      }
    } else if (k >= 0 && (!IN_LDS || (wave & 3) != 0)) {
      // small matrices: the pivot chain has its SIMD (every fourth wave) to itself
      // row i = k + 1 + q: k + 1 tiles of E, then the tiles i..nb - 1 of G (not the first one of all: wave 0 has it)
      const int helpers = IN_LDS ? nw - nw / 4 : nw - 1;
      int q = 0, pos = IN_LDS ? wave - 1 - (wave >> 2) : wave - 1, width = k + 1 + (FACTORED ? 0 : a - 1);
      constexpr int BATCH = 4;
      while (q < a) {
        int ti[BATCH], tc[BATCH];
        doublex4 t[BATCH];
#pragma unroll
        for (int b = 0; b < BATCH; ++b) {
          while (q < a && pos >= width) { pos -= width; ++q; width = k + 1 + (FACTORED ? 0 : a - q); }
          const int i = k + 1 + q;
          ti[b] = q < a ? i : -1;
          tc[b] = pos <= k ? pos : i + (pos - (k + 1)) + (q == 0 ? 1 : 0);
          if (ti[b] >= 0) t[b] = load(ti[b], tc[b]);
          pos += helpers;
        }
#pragma unroll
        for (int b = 0; b < BATCH; ++b) {
          if (ti[b] < 0) continue;
          t[b] = update(ti[b], tc[b], t[b]);
#pragma unroll
          for (int v = 0; v < 4; ++v) M[(int64_t)(kNB * ti[b] + g + 4 * v) * ld + kNB * tc[b] + r] = t[b][v];
        }
      }
    }
  }
}

// C = A B of upper triangular l x l factors (strides Lp), a workgroup per tile of 16 x 16; what lies below their diagonals is not looked at.
// What bounds it: the latency of the loads, so eight waves share the contraction (v_mfma_f64_16x16x4_f64).  Measured (us with the launch,
// one thread per entry before): l = 30 4.3 -> 2.8, 110 11.9 -> 5.1, 160 12.7 -> 6.0, 272 18.2 -> 5.6.
template <typename TB>
__global__ void __launch_bounds__(kTileWaves * 64)
k_triu_mul(const double* __restrict__ A, const TB* __restrict__ B, int l, int Lp, double* __restrict__ C) {
  __shared__ double part[kTileWaves][256];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15, g = lane >> 4;
  const int i0 = kNB * blockIdx.y, j0 = kNB * blockIdx.x, row = i0 + r, col = j0 + r;
  doublex4 acc = {0.0, 0.0, 0.0, 0.0};
  double an[4], bn[4];
  auto load = [&](int k0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int k = k0 + 4 * q + g;
      const bool ina = row <= k && k < l && row < l, inb = k <= col && col < l;
      an[q] = A[(int64_t)(ina ? row : 0) * Lp + (ina ? k : 0)];
      bn[q] = (double)B[(int64_t)(inb ? k : 0) * Lp + (inb ? col : 0)];
      if (!ina) an[q] = 0.0;
      if (!inb) bn[q] = 0.0;
    }
  };
  load(i0 + kNB * wave);
  for (int k0 = i0 + kNB * wave; k0 <= j0; k0 += kTileWaves * kNB) {
    double a[4], b[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) { a[q] = an[q]; b[q] = bn[q]; }
    load(k0 + kTileWaves * kNB);
#pragma unroll
    for (int q = 0; q < 4; ++q) acc = mfma_f64(a[q], b[q], acc);
  }
  if (!sum_over_waves(acc, part, lane, wave)) return;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int i = i0 + g + 4 * v;
    if (i < l && col < l) C[(int64_t)i * Lp + col] = acc[v];
  }
}

// Slots of Lp x Lp doubles for partial sums in the workspace (its size is what callers' budgets were chosen for): enough for a Gram matrix that has
// nothing else, after a Householder tree.
constexpr int kGramFan = 64;
uint64_t orth_gram_slots(int64_t rows, int Lp) {
  const int nbk = (Lp + 63) / 64, pairs = nbk * (nbk + 1) / 2;
  int64_t c = std::min<int64_t>(ceil_div(rows, 64), 64);
  c = std::min<int64_t>(c, std::max<int64_t>(1, ceil_div(1024, pairs)));
  const int64_t cap = std::min<int64_t>(std::max(2048 / pairs, 1), (64ll << 20) / ((int64_t)Lp * Lp * 8));
  const int64_t tall = std::min<int64_t>(rows / 1024, cap);
  c = std::max<int64_t>(std::max(c, tall), 1);
  return (uint64_t)(c > kGramFan ? c + ceil_div(c, kGramFan) : c);
}
// Row chunks of the Gram kernel: of 64 rows at least (eight per wave), and as many as give every CU a workgroup: one where all blocks of tiles are
// of a size, more where a chunk's pairs of blocks are not, so that the short ones fill the gaps.  Two per CU for the tallest narrow panels, whose
// workgroups have rows enough. Measured (us with the sum, workgroups in all: 256 / 512 / 1024): 76800x32 10.2 / 11.6 / 12.6, 2073600x32 76 / 71 /
// 79, 40000x64 15 / 20 / 20 (23 with 64), 20000x112 16.7 / 17.3 / 16.5 (20 with 192), 89083x112 38 / 39 / 45, 100000x160 73 / 69 / 78, 100000x272
// 192 / 181 / 170, 50000x272 104 / 99 / 97; chunks of 64 / 128 / 256 rows: 2000x32 5.8 / 8.0 / 7.4, 12000x64 11.8 / 11.4 / 14.0, 2783x112 10.4 /
// 11.7 / 15.0.
static int64_t gram_chunks(int64_t rows, int pairs) {
  const int64_t wgs = pairs > 6 ? 1024 : pairs > 3 || (pairs == 1 && rows >= (1 << 20)) ? 512 : 256;
  return std::min<int64_t>(ceil_div(rows, 64), std::max<int64_t>(1, wgs / pairs));
}

// G = the sum of the chunks' parts.  A workgroup takes 32 entries of the upper tiles; each is added up by 32 threads, thread s the chunks s, s + 32,
// ... in order, and then their sums in order: the result does not depend on timing.
// What bounds it: the latency of the loads, which come from all dies.  One thread per entry, over all entries, in two launches from 65 (small
// factors: 257) chunks on, and this (us): l = 30 3.1 and 2.6, 72 7.3 and 4.8, 110 9.1 and 4.8, 160 10.5 and 5.1, 272 14.4 and 11.0; 76800x32 (75
// chunks) 6.1 and 4.6, 2073600x32 (2025) 11.2 and 11.6.
__global__ void __launch_bounds__(1024)
k_gram_sum(const double* __restrict__ part, int chunks, int Lp, double* __restrict__ G) {
  __shared__ double sums[32][33];
  const int e = threadIdx.x & 31, slice = threadIdx.x >> 5, NT = Lp / 16;
  int i = 0, j = (int)(blockIdx.x >> 3);           // eight workgroups per tile
  while (j >= NT - i) { j -= NT - i; ++i; }
  j += i;
  const int in_tile = (int)(blockIdx.x & 7) * 32 + e, row = 16 * i + (in_tile >> 4), col = 16 * j + (in_tile & 15);
  const double* p = part + (int64_t)row * Lp + col;
  double s = 0.0;
#pragma unroll 16
  for (int c = slice; c < chunks; c += 32) s += p[(int64_t)c * Lp * Lp];
  sums[slice][e] = s;
  __syncthreads();
  if (slice != 0) return;
#pragma unroll
  for (int k = 1; k < 32; ++k) s += sums[k][e];
  G[(int64_t)row * Lp + col] = s;
}

// Where the partial sums lie, and for how many chunks there is room: in the work area of the Householder tree, unless that is in use.
struct GramPlace {
  double* part;
  int64_t room;
};
template <typename T>
static GramPlace gram_place(const OrthWorkT<T>& w, int Lp) {
  const int64_t slot = (int64_t)Lp * Lp * 8, tree = (int64_t)w.tsqr_bytes / slot;
  return tree > w.gram_chunks_max ? GramPlace{(double*)w.tsqr_work, tree} : GramPlace{w.gram_part, w.gram_chunks_max};
}
static int gram_sum(const double* part, int chunks, int Lp, double* G, hipStream_t stream) {
  const int nt = Lp / 16;
  hipLaunchKernelGGL(k_gram_sum, dim3(nt * (nt + 1) / 2 * 8), dim3(1024), 0, stream, part, chunks, Lp, G);
  BRSVD_HIP_TRY(hipGetLastError());
  return BRSVD_OK;
}

template <typename T>
static int gram(const T* P, int64_t rows, int Lp, OrthWorkT<T>& w, hipStream_t stream) {
  if (w.G_of_panel) {                  // came with the product that wrote the panel
    w.G_of_panel = false;
    return BRSVD_OK;
  }
  const int nt = Lp / 16, nb = (nt + 3) / 4, pairs = nb * (nb + 1) / 2;
  const GramPlace at = gram_place(w, Lp);
  double* part = at.part;
  int chunks = (int)std::min(gram_chunks(rows, pairs), at.room);
  if (chunks < 1) return BRSVD_ERR_BUDGET;
  int64_t rpc = ceil_div(rows, chunks);
  rpc = ceil_div(rpc, 8) * 8;
  chunks = (int)ceil_div(rows, rpc);
  dim3 grid(chunks, pairs), block(kGramWaves * 64);
  switch (nt) {
    case 1: hipLaunchKernelGGL((k_gram<T, 1>), grid, block, 0, stream, P, rows, Lp, rpc, part); break;
    case 2: hipLaunchKernelGGL((k_gram<T, 2>), grid, block, 0, stream, P, rows, Lp, rpc, part); break;
    case 3: hipLaunchKernelGGL((k_gram<T, 3>), grid, block, 0, stream, P, rows, Lp, rpc, part); break;
    default: hipLaunchKernelGGL((k_gram<T, 4>), grid, block, 0, stream, P, rows, Lp, rpc, part); break;
  }
  BRSVD_HIP_TRY(hipGetLastError());
  return gram_sum(part, chunks, Lp, w.G, stream);
}

// lenient != 0: pivots below tol * (original diagonal) are clamped and the factorisation goes on;
// otherwise such a pivot raises the breakdown flag and ends the kernel.
template <typename TO>
static int chol_inv(double* G, int l, int Lp, double* Rout, TO* Rinv, int* flags, double tol, hipStream_t stream,
                    int factored = 0, int lenient = 0, double near_eye = 0.0, TO* far_inv = nullptr) {
  const bool in_lds = Lp <= kCholLdsMaxLp;
  const size_t lds = chol_lds_bytes(Lp, in_lds);
  // a step has at most one panel tile per wave up to 16 column tiles; two tiles leave work for four waves only
  const int threads = Lp <= 32 ? 256 : (Lp <= 64 ? 512 : 1024);
  auto launch = [&](auto kern, size_t max_lds, bool* attr_set) -> int {
    if (!*attr_set) {
      BRSVD_HIP_TRY(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)max_lds));
      *attr_set = true;
    }
    hipLaunchKernelGGL(kern, dim3(1), dim3(threads), lds, stream, G, l, Lp, Rout, Rinv, flags, tol, lenient, near_eye, far_inv);
    BRSVD_HIP_TRY(hipGetLastError());
    return BRSVD_OK;
  };
  static bool attr_set[4] = {false, false, false, false};
  const size_t most_lds = chol_lds_bytes(kCholLdsMaxLp, true), most = chol_lds_bytes(kMaxL, false);
  if (factored)
    return in_lds ? launch(k_chol_inv<true, true, TO>, most_lds, attr_set) : launch(k_chol_inv<false, true, TO>, most, attr_set + 1);
  return in_lds ? launch(k_chol_inv<true, false, TO>, most_lds, attr_set + 2)
                : launch(k_chol_inv<false, false, TO>, most, attr_set + 3);
}

template <typename T>
int chol_inv_factored(double* G, int l, int Lp, double* Rout, T* Rinv, int* flags, hipStream_t stream) {
  return chol_inv<T>(G, l, Lp, Rout, Rinv, flags, 0.0, stream, 1);
}

// ---- panel times an Lp x Lp factor ----------------------------------------------------------
// out = P X for a narrow fp32 panel (rows x Lp, Lp = 16 NT): no staging and no barrier.  A wave holds all of X in registers and walks
// over tiles of 16 rows, the next tile's loads in flight under the matrix instructions (v_mfma_f32_16x16x4_f32).  X is the first
// operand: lane (r, g) holds X[16j + 4g + i][16t + r] for the instructions (j, i) of tile t, and the 16 bytes P[r][16j + 4g ..] of its
// row; its results are out[r][16t + 4g ..], 16 bytes again.
// What bounds it: the panel's read and write.  k_gemm_an, made for long contractions, takes chunks of 64 indices with a barrier
// each, half of them padding at 32 columns.  Measured, k_gemm_an and this (us, padded columns): 2073600x32 132 and 105 (5.1 TB/s),
// 400000x48 37.6 and 32.2, 76800x32 9.1 and 6.4, 2000x32 4.5 and 1.8 to 3.9; with four tiles 1000000x64 125 and 131.
template <int NT>
__global__ void __launch_bounds__(256)
k_apply(const float* __restrict__ P, int64_t rows, const float* __restrict__ X, float* __restrict__ out, int64_t ldo, int ncols) {
  constexpr int Lp = 16 * NT;
  typedef floatx4 floatx4u __attribute__((aligned(4)));
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int64_t tiles = (rows + 15) / 16, stride = (int64_t)gridDim.x * 4;
  int64_t tile = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (tile >= tiles) return;
  auto load = [&](int64_t t, floatx4 (&a)[NT]) {
    const float* p = P + min(t * 16 + r, rows - 1) * Lp + 4 * g;
#pragma unroll
    for (int j = 0; j < NT; ++j) a[j] = *(const floatx4*)(p + 16 * j);
  };
  floatx4 next[NT];
  load(tile, next);
  float x[NT][NT][4];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) x[t][j][i] = X[(16 * j + 4 * g + i) * Lp + 16 * t + r];
  for (; tile < tiles; tile += stride) {
    floatx4 a[NT], acc[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) { a[j] = next[j]; acc[j] = floatx4{0.f, 0.f, 0.f, 0.f}; }
    if (tile + stride < tiles) load(tile + stride, next);
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[t][j][i], a[j][i], acc[t], 0, 0, 0);
    const int64_t row = tile * 16 + r;
    if (row < rows) {
      float* o = out + row * ldo;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int col = 16 * t + 4 * g;
        if (col + 4 <= ncols) {
          *(floatx4u*)(o + col) = acc[t];
        } else {
#pragma unroll
          for (int v = 0; v < 4; ++v)
            if (col + v < ncols) o[col + v] = acc[t][v];
        }
      }
    }
  }
}

// Between LDS accesses of the lanes of one wave to each other's numbers: those before it are done and seen by all lanes.  (The hardware keeps a
// wave's LDS accesses in order; this keeps the compiler to it.)
__device__ __forceinline__ void wave_exchange() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The same with the Gram matrix of what is written, for the second sweep of CholeskyQR: that saves a read of the panel.  A wave puts each tile in
// LDS (its own place, no barrier) and takes it up again in the order of the Gram kernel's operands; Gpart as there, one part per workgroup.
// What bounds it: the panel's read and write, as before; the fp64 matrix instructions run under them.  Measured, product, Gram matrix and its sum,
// and with this (us): 2073600x32 101 + 61 + 5 and 101 + 5, 76800x32 5.5 + 5 + 4.6 and 9 + 4.6, 2000x32 3.3 + 3.4 + 2.7 and 4.5 + 2.7.
// It also does Y = A X with the Gram matrix of Y for tall matrices of short rows (K up to 128, KT tiles of 16; rows at any element address): all of
// X is in registers there as well.  A lane whose four indices lie behind K repeats the row's last ones and meets zeros of X.  k_gemm_an, Gram
// matrix and sum, and this (us): 2073600x100 l=20 214 + 61 + 5 and 208 + 4.
// Waves of a workgroup: eight, two of whose workgroups fit a CU, up to 64 indices; four where registers run out (SVD runs, q = 1, with four and
// eight, us: 1000000x64 l = 32 750 and 731, 1000000x100 828 and 859, 2073600x96 1415 and 1492).
template <int KT> constexpr int rows_gram_waves() { return KT <= 4 ? 8 : 4; }
template <int KT, int NT>
__global__ void __launch_bounds__(rows_gram_waves<KT>() * 64)
k_rows_gram(const float* __restrict__ A, int64_t lda, int64_t rows, int K, const float* __restrict__ X, float* __restrict__ out,
            double* __restrict__ Gpart) {
  constexpr int Lp = 16 * NT, TILES = NT * (NT + 1) / 2, LD = Lp + 4, WAVES = rows_gram_waves<KT>();
  typedef floatx4 floatx4u __attribute__((aligned(4)));
  __shared__ __align__(16) float place[WAVES][16 * LD];
  __shared__ double red[WAVES * 2 * 256];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r = lane & 15, g = lane >> 4;
  const int64_t tiles = (rows + 15) / 16, stride = (int64_t)gridDim.x * WAVES;
  int64_t tile = (int64_t)blockIdx.x * WAVES + wave;
  const bool whole = (K & 3) == 0;                 // no lane's four indices straddle K
  auto load = [&](int64_t t, floatx4 (&a)[KT]) {
    const float* p = A + min(t * 16 + r, rows - 1) * lda;
#pragma unroll
    for (int j = 0; j < KT; ++j) {
      const int k = 16 * j + 4 * g;
      if (j < KT - 1 || whole) {
        a[j] = *(const floatx4u*)(p + min(k, K - 4));
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) a[j][i] = p[min(k + i, K - 1)];
      }
    }
  };
  floatx4 next[KT];
  load(min(tile, tiles - 1), next);
  float x[NT][KT][4];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int j = 0; j < KT; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int k = 16 * j + 4 * g + i;
        const float v = X[min(k, K - 1) * Lp + 16 * t + r];
        x[t][j][i] = k < K ? v : 0.f;
      }
  doublex4 gram[TILES];
#pragma unroll
  for (int t = 0; t < TILES; ++t) gram[t] = doublex4{0.0, 0.0, 0.0, 0.0};
  float* mine = place[wave];
#pragma nounroll
  for (; tile < tiles; tile += stride) {
    floatx4 a[KT], acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < KT; ++j) a[j] = next[j];
    load(min(tile + stride, tiles - 1), next);
#pragma unroll
    for (int j = 0; j < KT; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[t][j][i], a[j][i], acc[t], 0, 0, 0);
    const int64_t row = tile * 16 + r;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (row < rows) *(floatx4*)(out + row * Lp + 16 * t + 4 * g) = acc[t];
      *(floatx4*)(mine + r * LD + 16 * t + 4 * g) = row < rows ? acc[t] : floatx4{0.f, 0.f, 0.f, 0.f};
    }
    wave_exchange();
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      double b[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) b[t] = (double)mine[(4 * s + g) * LD + NT * r + t];
      int t = 0;
#pragma unroll
      for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = i; j < NT; ++j) { gram[t] = mfma_f64(b[i], b[j], gram[t]); ++t; }
    }
    wave_exchange();                               // the next tile goes where this one was read
  }
  gram_store<NT, NT, true, WAVES>(gram, Lp, 0, 0, red, Gpart + (int64_t)blockIdx.x * Lp * Lp, tid);
}

// out = A X and w.G = out^T out, where both are one kernel.
template <int KT, int NT>
static int rows_gram(const float* A, int64_t lda, int64_t rows, int K, const float* X, float* out, OrthWork& w, hipStream_t stream) {
  constexpr int WAVES = rows_gram_waves<KT>(), Lp = 16 * NT;
  const GramPlace at = gram_place(w, Lp);
  const int64_t most = rows >= (1 << 20) ? 512 : 256;      // two and one per CU
  const int chunks = (int)std::min(std::min<int64_t>(ceil_div(rows, 16 * WAVES), most), at.room);
  if (chunks < 1) return BRSVD_ERR_BUDGET;
  hipLaunchKernelGGL((k_rows_gram<KT, NT>), dim3(chunks), dim3(WAVES * 64), 0, stream, A, lda, rows, K, X, out, at.part);
  BRSVD_HIP_TRY(hipGetLastError());
  return gram_sum(at.part, chunks, Lp, w.G, stream);
}
// The panel times a factor: fp32 panels of up to three tiles.
static bool apply_gram_fits(int Lp, int esz) { return esz == 4 && Lp <= 48; }
static int apply_gram(const float* P, int64_t rows, int Lp, const float* X, float* out, OrthWork& w, hipStream_t stream) {
  switch (Lp / 16) {
    case 1: return rows_gram<1, 1>(P, Lp, rows, Lp, X, out, w, stream);
    case 2: return rows_gram<2, 2>(P, Lp, rows, Lp, X, out, w, stream);
    default: return rows_gram<3, 3>(P, Lp, rows, Lp, X, out, w, stream);
  }
}
// A X: rows of up to 128 numbers, and some wavefronts for every CU.  SVD runs, q = 1, with the product and the Gram matrix apart and in one (us):
// 4200x48 l = 32 252 and 245, 16384x128 270 and 263, 131072x96 l = 16 252 and 255, 131072x128 l = 32 343 and 339, 1000000x48 l = 32 745 and 707,
// 1000000x64 744 and 736, 1000000x128 903 and 875, 2073600x48 l = 16 801 and 757, 2073600x80 l = 32 1476 and 1317; of 74 shapes from 4200x48
// to 2073600x100 all but 131072x96 l = 16 gain 1 to 11 percent.  Fewer rows are matters of launches, and the small products' plan cuts them.
bool an_gram_fits(int64_t rows, int64_t K, int Lp, int esz) { return esz == 4 && Lp <= 32 && K >= 4 && K <= 128 && rows >= 4096; }
int an_gram(const float* A, int64_t lda, int64_t rows, int64_t K, const float* X, int Lp, float* Y, OrthWork& w, hipStream_t stream,
            const KernelEvents* ev) {
  if (!an_gram_fits(rows, K, Lp, 4)) return BRSVD_ERR_ARG;
  int status = BRSVD_ERR_ARG;
#define CALL(KT)                                                            \
  case KT:                                                                  \
    status = Lp == 16 ? rows_gram<KT, 1>(A, lda, rows, (int)K, X, Y, w, stream)  \
                      : rows_gram<KT, 2>(A, lda, rows, (int)K, X, Y, w, stream); \
    break;
  switch (ceil_div(K, 16)) {
    CALL(1) CALL(2) CALL(3) CALL(4) CALL(5) CALL(6) CALL(7) CALL(8)
  }
#undef CALL
  if (ev) {
    BRSVD_HIP_TRY(hipEventRecord(ev->stop, stream));
    BRSVD_HIP_TRY(hipEventRecord(ev->sum_stop, stream));
  }
  w.G_of_panel = status == BRSVD_OK;
  return status;
}

template <typename T>
int apply_panel(const T* P, int64_t rows, int Lp, const T* X, T* out, int64_t ldo, int ncols, void* scratch, uint64_t scratch_bytes,
                hipStream_t stream) {
  if constexpr (std::is_same<T, float>::value) {
    // from 64 columns on the matrix cores bound both kernels, and more of X than this takes too many registers
    if (Lp <= 48) {
      const dim3 grid((unsigned)std::min<int64_t>(ceil_div(rows, 64), 2048)), block(256);   // eight workgroups of four waves per CU
      switch (Lp / 16) {
        case 1: hipLaunchKernelGGL(k_apply<1>, grid, block, 0, stream, P, rows, X, out, ldo, ncols); break;
        case 2: hipLaunchKernelGGL(k_apply<2>, grid, block, 0, stream, P, rows, X, out, ldo, ncols); break;
        default: hipLaunchKernelGGL(k_apply<3>, grid, block, 0, stream, P, rows, X, out, ldo, ncols); break;
      }
      BRSVD_HIP_TRY(hipGetLastError());
      return BRSVD_OK;
    }
  }
  return gemm_an(P, Lp, rows, Lp, X, Lp, out, ldo, ncols, scratch, scratch_bytes, stream);
}
template int apply_panel<float>(const float*, int64_t, int, const float*, float*, int64_t, int, void*, uint64_t, hipStream_t);
template int apply_panel<double>(const double*, int64_t, int, const double*, double*, int64_t, int, void*, uint64_t, hipStream_t);

// P <- P X for X upper triangular, in place, if *far is set.  A wave takes 16 rows into LDS and all columns from there, one tile of 16 after the
// other.  What bounds it: mostly the launch, as *far is not set (us: 2000x32 2.2, 20000x112 and 2073600x32 3.9); where it is, a wave's loads of X
// (2073600x32 254, 20000x112 24, 100000x272 347, fp64 15872x80 18; in the SVD of a matrix of rank 2, q = 1, against the two applications of a basis
// that is always orthonormalised twice: 2073600x100 l = 20 1676 and 1843, 20000x5000 l = 110 1535 and 1627, 100000x4000 l = 272 9495 and 9826).
template <typename T>
__global__ void __launch_bounds__(64)
k_apply_far(T* P, int64_t rows, int Lp, const T* __restrict__ X, const int* __restrict__ far) {
  if (*far == 0) return;
  extern __shared__ __align__(16) char far_smem[];
  T* place = (T*)far_smem;
  const int LD = Lp + 16 / (int)sizeof(T), lane = threadIdx.x, r = lane & 15, g = lane >> 4;
  constexpr int V = 16 / sizeof(T);
  typedef T vec __attribute__((ext_vector_type(V)));
  for (int64_t row0 = (int64_t)blockIdx.x * 16; row0 < rows; row0 += (int64_t)gridDim.x * 16) {
    const int n = (int)min((int64_t)16, rows - row0), units = Lp / V;
    T* p = P + row0 * Lp;
    __syncthreads();
    for (int u = lane; u < 16 * units; u += 64) {
      const int i = u / units;
      *(vec*)(place + i * LD + (u - i * units) * V) = *(const vec*)(p + (int64_t)min(i, n - 1) * Lp + (u - i * units) * V);
    }
    __syncthreads();
    for (int c0 = 0; c0 < Lp; c0 += 16) {
      typename std::conditional<sizeof(T) == 8, doublex4, floatx4>::type acc = {0, 0, 0, 0};
      for (int k0 = 0; k0 <= c0; k0 += 16) {
        T a[4], b[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          a[q] = place[r * LD + k0 + 4 * q + g];
          b[q] = X[(int64_t)(k0 + 4 * q + g) * Lp + c0 + r];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if constexpr (sizeof(T) == 8) acc = mfma_f64(a[q], b[q], acc);
          else acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[q], b[q], acc, 0, 0, 0);
        }
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = sizeof(T) == 8 ? g + 4 * v : 4 * g + v;
        if (i < n) p[(int64_t)i * Lp + c0 + r] = acc[v];
      }
    }
  }
}
template <typename T>
static int apply_far(T* P, int64_t rows, int Lp, const T* X, const int* far, hipStream_t stream) {
  static bool attr_set = false;
  if (!attr_set) {
    BRSVD_HIP_TRY(hipFuncSetAttribute((const void*)k_apply_far<T>, hipFuncAttributeMaxDynamicSharedMemorySize, 16 * (kMaxL * (int)sizeof(T) + 16)));
    attr_set = true;
  }
  const int64_t wgs = std::min<int64_t>(ceil_div(rows, 16), 2048);
  hipLaunchKernelGGL(k_apply_far<T>, dim3((unsigned)wgs), dim3(64), 16 * (Lp * sizeof(T) + 16), stream, P, rows, Lp, X, far);
  BRSVD_HIP_TRY(hipGetLastError());
  return BRSVD_OK;
}

template <typename T>
int apply_to_companion(OrthWorkT<T>& w, int Lp, hipStream_t stream) {
  if (!w.comp) return BRSVD_OK;
  BRSVD_TRY(apply_panel(w.comp, w.comp_rows, Lp, w.Rinv, w.comp_tmp, Lp, Lp, w.gemm_scratch, w.gemm_scratch_bytes, stream));
  T* t = w.comp; w.comp = w.comp_tmp; w.comp_tmp = t;
  return BRSVD_OK;
}

// *out = min_i |R_ii| / max_i |R_ii| of an l x l triangular factor (stride Lp): how far the last column
// of the factored panel sits below the first.  One wave.
__global__ void __launch_bounds__(64)
k_diag_ratio(const double* __restrict__ R, int l, int Lp, double* __restrict__ out) {
  double lo = INFINITY, hi = 0.0;
  for (int i = threadIdx.x; i < l; i += 64) {
    const double d = fabs(R[(int64_t)i * Lp + i]);
    lo = fmin(lo, d);
    hi = fmax(hi, d);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, off, 64));
    hi = fmax(hi, __shfl_xor(hi, off, 64));
  }
  if (threadIdx.x == 0) *out = hi > 0.0 ? lo / hi : 0.0;
}

int diag_ratio(const double* R, int l, int Lp, double* out, hipStream_t stream) {
  hipLaunchKernelGGL(k_diag_ratio, dim3(1), dim3(64), 0, stream, R, l, Lp, out);
  BRSVD_HIP_TRY(hipGetLastError());
  return BRSVD_OK;
}

template <typename TB>
int triu_mul(const double* A, const TB* B, int l, int Lp, double* C, hipStream_t stream) {
  const unsigned nt = (unsigned)ceil_div(l, kNB);
  hipLaunchKernelGGL(k_triu_mul<TB>, dim3(nt, nt), dim3(kTileWaves * 64), 0, stream, A, B, l, Lp, C);
  BRSVD_HIP_TRY(hipGetLastError());
  return BRSVD_OK;
}
template int triu_mul<float>(const double*, const float*, int, int, double*, hipStream_t);
template int triu_mul<double>(const double*, const double*, int, int, double*, hipStream_t);

constexpr double kPivotTol = 1e-12;
// |G - I|_F up to which the factor of G (l x l) is not eliminated.  R, in fp64, is then off by at most |E|_F^3 / 2, a quarter of a rounding for each
// of the l steps of an elimination, its inverse by |E|_F^2 / 2, which in the panels' precision is a hundredth of a rounding (8e-10 of 6e-8 at l =
// 272) and a seventh (8e-18 of 1.1e-16).  First sweeps of panels with conditions up to a few hundred leave 5e-7 to 2e-5 in fp32.
template <typename T> double near_eye_of(int l) { return sizeof(T) == 4 ? cbrt(l * 0x1p-52) : 4e-9; }
// Only the last sweep of a basis that reaches the output must succeed without clamped pivots (its
// input is then already nearly orthonormal, so a small pivot there means the panel really lost
// rank to working precision).  Earlier sweeps, and the single sweep of an intermediate panel, clamp:
// the numerically dependent directions of an exactly rank-deficient panel -- the paper's own test
// inputs have rank k < l -- come out as damped rounding noise, which the next sweep or the next
// power step treats like any other direction; P = Q R holds exactly either way.
template <typename T>
int cholqr_sweeps(T* P, T* tmp, int64_t rows, int l, int Lp, int nsweeps, OrthWorkT<T>& w, double* Rtot,
                  T** result, hipStream_t stream, bool strict_last, bool publish_R) {
  T* src = P;
  T* dst = tmp;
  for (int sweep = 0; sweep < nsweeps; ++sweep) {
    BRSVD_TRY(gram<T>(src, rows, Lp, w, stream));
    const int lenient = (sweep + 1 < nsweeps || !strict_last) ? 1 : 0;
    double* Rs = (Rtot || publish_R) ? w.R[sweep] : nullptr;      // the factor is only written out when someone reads it
    BRSVD_TRY(chol_inv<T>(w.G, l, Lp, Rs, w.Rinv, w.flags, kPivotTol, stream, 0, lenient, lenient ? 0.0 : near_eye_of<T>(l)));
    BRSVD_TRY(apply_panel(src, rows, Lp, w.Rinv, dst, Lp, Lp, w.gemm_scratch, w.gemm_scratch_bytes, stream));
    BRSVD_TRY(apply_to_companion<T>(w, Lp, stream));
    T* t = src; src = dst; dst = t;
  }
  *result = src;
  if (Rtot) {
    if (nsweeps == 2) {
      BRSVD_TRY(triu_mul(w.R[1], w.R[0], l, Lp, Rtot, stream));
    } else {
      BRSVD_HIP_TRY(hipMemcpyAsync(Rtot, w.R[0], (size_t)Lp * Lp * sizeof(double), hipMemcpyDeviceToDevice, stream));
    }
  }
  return BRSVD_OK;
}

template <typename T>
int orth_panel(T* P, T* tmp, int64_t rows, int l, int Lp, int method, bool final_basis, OrthWorkT<T>& w,
               double* Rtot, T** result, hipStream_t stream) {
  if (rows < l) return BRSVD_ERR_ARG;
  if (method == BRSVD_ORTH_TSQR) return tsqr_panel<T>(P, tmp, rows, l, Lp, w, Rtot, result, stream);
  // A panel that only seeds the next power half step needs a well-conditioned basis, not one
  // orthonormal to working precision: one CholeskyQR sweep (fp64 Gram) leaves ||Q^T Q - I|| of
  // order eps32 * cond(P).  The bases that reach the output (Q behind U, W_B behind V) get two.
  return cholqr_sweeps<T>(P, tmp, rows, l, Lp, final_basis ? 2 : 1, w, Rtot, result, stream, final_basis);
}

// The second sweep of CholeskyQR, G2 = Q1^T Q1 = R2^T R2, without its pass over the panel Q2 = Q1 R2^-1: everything that follows is a product of Q1
// with an l x l factor or a product from the left that R2^-1 can be multiplied to afterwards.  R2 is close to the identity (where a pivot was
// clamped, to a diagonal matrix times a well-conditioned one), so little is lost by taking R2^-1 to the other side.
// settle: of a basis Q that A is multiplied by.  A column of Q1 whose pivot was clamped is rounding, and as much along the columns before it as
// across them; A^T Q1 then holds A's largest values there, and their rounding stays when R2^-1 takes them out: zero singular values came out as
// 1e-7 to 9e-7 of the largest (fp64 8e-16 to 2e-14) in the place of 4e-8 (7e-17) at most.  So Q1 <- Q1 R2^-1 and left = I after all where Q1 is far
// from orthonormal.
template <typename T>
int orth_basis(T* P, T* tmp, int64_t rows, int l, int Lp, int method, OrthWorkT<T>& w, T* left, double* Rtot, bool want_R, bool settle,
               Basis<T>* out, hipStream_t stream) {
  if (rows < l) return BRSVD_ERR_ARG;
  out->panel = nullptr;
  if (method == BRSVD_ORTH_TSQR) {
    *out = Basis<T>{nullptr, nullptr, want_R ? Rtot : nullptr, nullptr};
    return tsqr_panel<T>(P, tmp, rows, l, Lp, w, want_R ? Rtot : nullptr, &out->panel, stream);
  }
  if constexpr (std::is_same<T, float>::value) {
    if (apply_gram_fits(Lp, 4) && !w.comp) {
      BRSVD_TRY(gram<T>(P, rows, Lp, w, stream));
      BRSVD_TRY(chol_inv<T>(w.G, l, Lp, want_R ? w.R[0] : nullptr, w.Rinv, w.flags, kPivotTol, stream, 0, 1));
      BRSVD_TRY(apply_gram(P, rows, Lp, w.Rinv, tmp, w, stream));
      out->panel = tmp;
    }
  }
  if (!out->panel) {
    BRSVD_TRY(cholqr_sweeps<T>(P, tmp, rows, l, Lp, 1, w, nullptr, &out->panel, stream, false, want_R));
    BRSVD_TRY(gram<T>(out->panel, rows, Lp, w, stream));
  }
  BRSVD_TRY(chol_inv<T>(w.G, l, Lp, want_R ? w.R[1] : nullptr, left, w.flags, kPivotTol, stream, 0, 0, near_eye_of<T>(l),
                        settle ? w.Rinv : nullptr));
  if (settle) BRSVD_TRY(apply_far<T>(out->panel, rows, Lp, w.Rinv, w.flags + 1, stream));
  out->left = left;
  out->R1 = want_R ? w.R[0] : nullptr;
  out->R2 = want_R ? w.R[1] : nullptr;
  return BRSVD_OK;
}

#define BRSVD_ORTH_INSTANTIATE(T)                                                                               \
  template int chol_inv_factored<T>(double*, int, int, double*, T*, int*, hipStream_t);                         \
  template int apply_to_companion<T>(OrthWorkT<T>&, int, hipStream_t);                                          \
  template int cholqr_sweeps<T>(T*, T*, int64_t, int, int, int, OrthWorkT<T>&, double*, T**, hipStream_t, bool, \
                                bool);                                                                          \
  template int orth_panel<T>(T*, T*, int64_t, int, int, int, bool, OrthWorkT<T>&, double*, T**, hipStream_t);   \
  template int orth_basis<T>(T*, T*, int64_t, int, int, int, OrthWorkT<T>&, T*, double*, bool, bool, Basis<T>*, \
                                hipStream_t);
BRSVD_ORTH_INSTANTIATE(float)
BRSVD_ORTH_INSTANTIATE(double)
#undef BRSVD_ORTH_INSTANTIATE

}  // namespace brsvd
