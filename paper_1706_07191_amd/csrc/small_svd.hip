// SVD of the small l x l factor (Alg. 1 step 5 / Alg. 2 line 11) by one-sided (Hestenes) Jacobi.
//
// With B^T = W_B * R (thin QR of the n x l panel), R = Ur * diag(s) * Vr^T gives
// B = Vr * diag(s) * (W_B Ur)^T, i.e. the small left factor is Vr and V = W_B * Ur.
// The rows of a working copy W of R are rotated in pairs (round-robin schedule) until they are
// mutually orthogonal: then W = diag(s) Vr^T, so s_i is the norm of row i and Vr's column i the
// normalised row i; Ur = R Vr diag(1/s) follows from one small product.  Everything is fp64.
#include <cstdlib>

#include "common.h"

namespace brsvd {

constexpr int kMaxSweeps = 40;

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Pair pi of round-robin step `step` among L2 (even) players.
__device__ __forceinline__ void rr_pair(int pi, int step, int L2, int& a, int& b) {
  const int N = L2 - 1;
  if (pi == 0) { a = N; b = step; }
  else {
    a = step + pi; if (a >= N) a -= N;
    b = step - pi; if (b < 0) b += N;
  }
  if (a > b) { int t = a; a = b; b = t; }
}

// 1/sqrt(x) and 1/x for positive normal x: hardware seed plus two Newton steps (full fp64).
__device__ __forceinline__ double rsqrt_nr(double x) {
  double y = __builtin_amdgcn_rsq(x);
  const double h = 0.5 * x;
  y = fma(y, fma(-h * y, y, 0.5), y);
  y = fma(y, fma(-h * y, y, 0.5), y);
  return y;
}
__device__ __forceinline__ double rcp_nr(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = fma(y, fma(-x, y, 1.0), y);
  y = fma(y, fma(-x, y, 1.0), y);
  return y;
}

// Sweeps end when a whole sweep met no pair with |cos| above kSettled: all cosines are then of the order
// l * kSettled^2 after that sweep's rotations (quadratic convergence), of the order of rounding, so
// a further sweep that would only confirm it is not run.
// With results delivered in single precision the bar is lower: a last sweep whose largest cosine was below
// kSettledF32 leaves cosines of the order l * kSettledF32^2 = 1e-8, an order of magnitude below what the fp32
// lifts U = Q V_R and V = W_B U_R can show, and that saves one sweep of the seven to eight an l of 100 to 300 takes.
// Row rotations turn everything above rounding: what is left counts times s_i / s_j in U = R V / s.  (A bar of 1e-13 from 33 rows on, whose skipped
// rotations save their traffic, left V of fp64 runs with l = 40 off by 7e-12 at a condition of 64 and 3e-8 at 1e6, now 2e-14 and 5e-11, and of fp32
// runs on sketches of lower rank than their width by 7e-5, now 5e-7; small SVD of SVD runs, with it and now, us: fp32 l = 33 136 and 139, 40 158 and
// 158, 48 179 and 179, fp64 151 and 154, 173 and 176, 197 and 203.)  On the 32 x 32 Gram matrix a rotation costs the same whether it turns or not:
// there is no bar.
constexpr double kTolRows = 1e-16;
constexpr double kSettled = 1e-8;
constexpr double kSettledF32 = 1e-5;
// In the last sweeps most block pairs have nothing left to rotate.  One is left as it is, for the price of its Gram matrix, when the inner
// product of every two of its rows is at most kIdle (results in single precision: kIdleF32) of the smaller of their squared norms.  Rows i
// and j that keep a product g leave g / (s_i s_j) in V^T V, but U = R V / s carries that times s_i / s_j: the bar is on g / s_j^2, which
// holds for both whatever the condition of R.  kIdle is near the rounding of a cosine; kIdleF32 leaves U and V within 1e-8 of
// orthogonal, where the rounding of the panels leaves 2e-7.  The results' defects are the same to two digits with and without the bars
// (l = 30 to 400, s_1 / s_l from 64 to 1e6; fp64 2e-15 to 1e-13).  (4e-9 and 1e-15 on the cosines left V of the SVD off by 3e-6 and 4e-14 at l =
// 200 and a condition of 1e4, by 6e-4 and 1e-10 at 1e6.)
// Over 32 rows, everything rotated and with the bars (us of the small SVD of an SVD run): fp32 l = 72 326 and 289, 97 450 and 431, 110 450 and
// 431, 160 742 and 637, 272 1664 and 1555 (with 1e-12 72 304, 97 447, 110 430, 160 694, 272 1570); fp64 l = 110 532 and 504, 160 737 and 703, 272
// 1897 and 1798.  Calls for dense factors (brsvd_small_svd) take any matrix, not the graded R of a range finder, and hardly ever meet an
// idle pair (a panel's R, condition 100, without and with: l = 72 524 and 537, 110 693 and 711, 160 1081 and 1091): no bar for those.
constexpr double kIdle = 1e-15, kIdleF32 = 4e-9;
constexpr int kIdleFrom = 3;                       // earlier sweeps (from 0) have none
// Rotation (c, s) that makes two rows with squared norms al, be and inner product ga orthogonal:
// with zeta = (be - al) / (2 ga), t = sign(zeta) / (|zeta| + sqrt(1 + zeta^2)), c = 1/sqrt(1+t^2),
// s = c t, written so that it needs one reciprocal and two reciprocal square roots.
// Returns false (identity) when |ga| <= tol * sqrt(al * be); big: above the settled bar.
__device__ __forceinline__ bool rotation_exact(double al, double be, double ga, double tol2, double settled2, double& c,
                                         double& s, bool& big) {
  c = 1.0; s = 0.0;
  big = ga * ga > settled2 * al * be;
  if (!(ga * ga > tol2 * al * be)) return false;
  const double tau = be - al, g2 = 2.0 * ga;
  const double hh = fma(tau, tau, g2 * g2);
  const double h = hh * rsqrt_nr(hh);
  const double t = copysign(g2, g2 * tau >= 0.0 ? 1.0 : -1.0) * rcp_nr(fabs(tau) + h);
  c = rsqrt_nr(fma(t, t, 1.0));
  s = c * t;
  return true;
}

// A value from another lane of the row of 16 (CTRL: the lane pattern).
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  int lo = __double2loint(v), hi = __double2hiint(v);
  lo = __builtin_amdgcn_update_dpp(0, lo, CTRL, 0xf, 0xf, true);
  hi = __builtin_amdgcn_update_dpp(0, hi, CTRL, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
// Sum over the 16 lanes of a DPP row, result in every lane of the row.
__device__ __forceinline__ double row16_sum(double v) {
  v += dpp_f64<0x128>(v);   // row_ror:8
  v += dpp_f64<0x124>(v);   // row_ror:4
  v += dpp_f64<0x4E>(v);    // quad_perm [2,3,0,1]
  v += dpp_f64<0xB1>(v);    // quad_perm [1,0,3,2]
  return v;
}

// Whether row j comes before row i in the descending order of their norms: NaN first, equal ones by index, so that the ranks are a
// permutation whatever the norms are.  Norms are not negative, so their bit patterns are in the same order, with NaN above
// infinity; and without branches the loads of the loops around this stay in flight together (7 us at l = 30).
__device__ __forceinline__ bool ranks_before(double sj, int j, double si, int i) {
  const unsigned long long kj = __double_as_longlong(sj), ki = __double_as_longlong(si);
  return (kj > ki) | ((kj == ki) & (j < i));
}

// Singular values (row norms), their descending order, and the final rows, written to global.
template <int NTHREADS>
__device__ void publish(const double* W, int ld, int l, int Lp, double* Wg, double* sig, int* order_sh,
                        int tid, int lane, int wave) {
  for (int i = wave; i < l; i += NTHREADS / 64) {
    double s2 = 0.0;
    for (int e = lane; e < l; e += 64) { double x = W[(int64_t)i * ld + e]; s2 = fma(x, x, s2); }
    s2 = wave_sum(s2);
    if (lane == 0) sig[Lp + i] = sqrt(s2);
  }
  __syncthreads();
  for (int i = tid; i < l; i += NTHREADS) {
    const double si = sig[Lp + i];
    int rank = 0;
    for (int j = 0; j < l; ++j) rank += ranks_before(sig[Lp + j], j, si, i);
    order_sh[rank] = i;
  }
  __syncthreads();
  for (int i = tid; i < l; i += NTHREADS) {
    sig[i] = sig[Lp + order_sh[i]];
    sig[2 * Lp + i] = (double)order_sh[i];
  }
  if (Wg != W)
    for (int idx = tid; idx < l * l; idx += NTHREADS) {
      int i = idx / l, c = idx - i * l;
      Wg[(int64_t)i * Lp + c] = W[(int64_t)i * ld + c];
    }
}

// Sum over groups of 8 lanes (half a DPP row), result in every lane of the group.
__device__ __forceinline__ double row8_sum(double v) {
  v += dpp_f64<0xB1>(v);    // quad_perm [1,0,3,2]
  v += dpp_f64<0x4E>(v);    // quad_perm [2,3,0,1]
  v += dpp_f64<0x141>(v);   // row_half_mirror
  return v;
}

// ---- up to 16 and 33 to 48 rows: row rotations in LDS ---------------------------------------------------------------------------------
// Each group of 16 lanes owns one row pair per step, so a wave handles 4 pairs with one instruction stream: 8 pairs take 128 threads,
// 32 take 512.  EPL = elements of a row per lane = ceil(l / 16).
// Pair schedule of a sweep (every pair of rows met exactly once): the index range is halved
// recursively.  At a level, every segment [base, base + n) is cut into a top half of h = ceil(n/2) rows
// and a bottom half; in step s top row i meets bottom row (i + s) mod h, so h steps pair every top with
// every bottom of the segment; the next level does the same inside both halves, all segments side by
// side (l-1 .. l+1 steps in all).  Within a level a group keeps its top row in registers and only the
// bottom rows travel through LDS, which halves the LDS traffic of the round-robin schedule.
constexpr int LPP = 16;
constexpr int kRowsMaxL = 16;                      // row rotations up to here, with one block of 16 rows, and with three

template <int EPL, int PAIRS>       // PAIRS = the most of a step: 8 up to 16 rows, 24 up to 40 (eight segments of 5), 32 up to 48
__global__ void __launch_bounds__(PAIRS * LPP)
k_jacobi_rows(const double* __restrict__ R, int ldr, int l, int Lp, double* __restrict__ Wg,
             double* __restrict__ sig, int* __restrict__ info, const int* __restrict__ breakdown_flag,
             double tol, double settled) {
  extern __shared__ double W[];
  __shared__ int rotated, top;
  __shared__ int order_sh[kMaxL];
  constexpr int NT = PAIRS * LPP, LEV = EPL == 1 ? 4 : 6;      // levels: 16 8 4 2, 40 20 10 5 3 2
  __shared__ short tb_top[LEV][PAIRS], tb_bb[LEV][PAIRS], tb_bs[LEV][PAIRS], tb_hi[LEV][PAIRS];
  __shared__ short seg_base[2][1 << LEV], seg_size[2][1 << LEV];
  __shared__ int lev_steps[LEV];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (breakdown_flag && breakdown_flag[0] != 0) {
    if (tid == 0) { info[0] = 0; info[1] = 0; }
    return;
  }
  const int ld = l;
  // The bars compare squares of squared norms.  Where even those of the largest entry would be close to the smallest double, all entries are
  // multiplied by a power of two (and by its inverse in the end).
  if (tid == 0) top = 0;
  __syncthreads();
  int most = 0;
  for (int idx = tid; idx < l * l; idx += NT) {
    int i = idx / l, c = idx - i * l;
    const double v = R[(int64_t)i * ldr + c];
    W[i * ld + c] = v;
    most = max(most, __double2hiint(v) >> 20 & 0x7ff);
  }
  atomicMax(&top, most);
  __syncthreads();
  const int shift = top > 823 ? 0 : 1023 - top;
  if (shift != 0)
    for (int idx = tid; idx < l * l; idx += NT) W[idx] = ldexp(W[idx], shift);
  // schedule tables: per level and group, the top row, the bottom half [bb, bb + bs) and (h << 8) | i
  if (tid == 0) { seg_base[0][0] = 0; seg_size[0][0] = (short)l; }
  for (int lev = 0; lev < LEV; ++lev) {
    const int nseg = 1 << lev, cur = lev & 1;
    if (tid < PAIRS) tb_top[lev][tid] = -1;
    __syncthreads();
    if (tid < nseg) {
      const int base = seg_base[cur][tid], size = seg_size[cur][tid];
      const int h = (size + 1) >> 1, nb = size - h;
      if (size >= 2) {
        int off = 0;
        for (int k = 0; k < tid; ++k) { const int sz = seg_size[cur][k]; if (sz >= 2) off += (sz + 1) >> 1; }
        for (int i = 0; i < h; ++i) {
          const int gid = off + i;
          if (gid < PAIRS) {
            tb_top[lev][gid] = (short)(base + i); tb_bb[lev][gid] = (short)(base + h);
            tb_bs[lev][gid] = (short)nb; tb_hi[lev][gid] = (short)((h << 8) | i);
          }
        }
      }
      seg_base[cur ^ 1][2 * tid] = (short)base; seg_size[cur ^ 1][2 * tid] = (short)h;
      seg_base[cur ^ 1][2 * tid + 1] = (short)(base + h); seg_size[cur ^ 1][2 * tid + 1] = (short)nb;
    }
    if (tid == 0) {
      int mx = 0;
      for (int k = 0; k < nseg; ++k) { const int sz = seg_size[cur][k]; if (sz >= 2) mx = max(mx, (sz + 1) >> 1); }
      lev_steps[lev] = mx;
    }
    __syncthreads();
  }
  const int pi = tid / LPP;
  const int rl = tid % LPP;
  const double tol2 = tol * tol, settled2 = settled * settled;
  int sweeps = 0, converged = (l < 2);
  __syncthreads();
  while (!converged && sweeps < kMaxSweeps) {
    if (tid == 0) rotated = 0;
    __syncthreads();
    bool any = false;
    for (int lev = 0; lev < LEV; ++lev) {
      const int steps = lev_steps[lev];
      if (steps == 0) continue;                        // uniform over the workgroup
      const int top = tb_top[lev][pi], bb = tb_bb[lev][pi], bs = tb_bs[lev][pi];
      const int h = tb_hi[lev][pi] >> 8, i0 = tb_hi[lev][pi] & 255;
      double x[EPL];
#pragma unroll
      for (int e = 0; e < EPL; ++e) {
        const int col = rl + LPP * e;
        x[e] = (top >= 0 && col < l) ? W[top * ld + col] : 0.0;
      }
      for (int step = 0; step < steps; ++step) {
        int j = i0 + step;
        if (j >= h) j -= h;
        const bool valid = top >= 0 && step < h && j < bs;
        const double* wb = W + (bb + j) * ld;
        double y[EPL], al = 0.0, be = 0.0, ga = 0.0;
#pragma unroll
        for (int e = 0; e < EPL; ++e) {
          const int col = rl + LPP * e;
          y[e] = (valid && col < l) ? wb[col] : 0.0;
          al = fma(x[e], x[e], al);
          be = fma(y[e], y[e], be);
          ga = fma(x[e], y[e], ga);
        }
        al = row16_sum(al); be = row16_sum(be); ga = row16_sum(ga);
        double c, s;
        bool big;
        const bool rot = rotation_exact(al, be, ga, tol2, settled2, c, s, big) && valid;
        any |= big && valid;
        if (rot) {
          double* wbw = W + (bb + j) * ld;
#pragma unroll
          for (int e = 0; e < EPL; ++e) {
            const int col = rl + LPP * e;
            const double xn = c * x[e] - s * y[e];
            if (col < l) wbw[col] = s * x[e] + c * y[e];
            x[e] = xn;
          }
        }
        __syncthreads();
      }
      if (top >= 0) {
#pragma unroll
        for (int e = 0; e < EPL; ++e) {
          const int col = rl + LPP * e;
          if (col < l) W[top * ld + col] = x[e];
        }
      }
      __syncthreads();
    }
    if (any) rotated = 1;
    __syncthreads();
    ++sweeps;
    converged = (rotated == 0);
    __syncthreads();
  }
  if (shift != 0) {
    for (int idx = tid; idx < l * l; idx += NT) W[idx] = ldexp(W[idx], -shift);
    __syncthreads();
  }
  publish<NT>(W, ld, l, Lp, Wg, sig, order_sh, tid, lane, wave);
  if (tid == 0) { info[0] = sweeps; info[1] = converged; }
}

// ---- Jacobi by blocks of rows -------------------------------------------------------------------------------------
// The rows are cut into blocks of kJB = 16 and pairs of blocks are orthogonalised at a time: the Gram matrix of the 32
// rows (fp64 matrix cores), one sweep of rotations on that 32 x 32 matrix alone, accumulated in an orthogonal J, and
// the rows replaced by J^T times the rows (matrix cores again).  A rotation then touches 32 numbers of the Gram
// matrix and of J instead of two whole rows, and needs no inner products: its step is a read of four matrix entries
// per thread, the rotation, and a write.  The Gram matrix is formed afresh from the rows for every pair of blocks, so
// what the two-sided updates lose never accumulates; singular values keep the relative accuracy of plain row rotations
// (simulated at condition 1e6, 1e10, 1e14: 8e-15, 9e-15, 8e-13, plain rotations 9e-15, 1.3e-14, 8e-13).
// A row whose squared norm is not finite is set aside: it is zero while the others are rotated (one of its products with them would make
// the whole block NaN) and comes back at the end with its own norm, as when rows are rotated, where no comparison with it holds.
// A sweep is a round robin over the block pairs.  Its first round rotates all 496 pairs of the 32 rows (31 steps of
// 16 disjoint pairs), the others the 256 pairs across the two blocks (16 steps).
//   l <= 32: one block pair, rows in LDS for all sweeps (k_jacobi_small);
//   otherwise: one workgroup per block pair, rows in global memory, one launch (k_jacobi_rounds).
// Row rotations stay ahead (us of the kernels of a call on an R of the range finder / of a panel with a geometric spectrum, this
// against row rotations)
//   up to 16 rows, where the 31 steps of a sweep are more than their l: l = 4 41 / 19 and 52 / 22, 8 52 / 32 and 77 / 42, 12 53 / 46 and
//   75 / 62, 14 54 / 52 and 76 / 61, 16 54 / 54 and 76 / 74; on the other side 17 66 / 80 and 77 / 93, 20 67 / 84 and 78 / 98;
//   and with three blocks, where a fourth block goes round that is padding (us of a call of brsvd_small_svd, on a panel's R / on one of equal
//   columns): l = 33 - / 132 and 193, 40 - / 165 and 219, 41 196 and 286 / 172 and 227, 44 195 and 288 / 177 and 233, 48 196 and 281 / 186
//   and 271.
// (One sweep more or less, 28 us at l = 33 to 48, is by chance.  The figures up to 20 rows are with 1024 threads for the row rotations, of which
// most only met the others at the barriers; with those they need a call takes 63 us in the place of 77 at l = 16.)
// What bounds it: the latency of a step, 640 cycles from barrier to barrier -- 130 until the rotations are read from LDS, 60 for the
// new inner product, 190 for the 13 dependent operations of the rotation, the rest its way back to LDS -- and of the meeting of the
// workgroups.  At l = 110 a round takes 25 thousand cycles: 11.2 the 16 steps, 3.2 the Gram matrix, 4.1 J^T times the rows, 2.5 the load
// of the rows and 3.7 the meeting (it was 29.7: 15.6, 4.9, 4.0, 2.2 and 4.7).  What made the difference: the matrix instructions
// accumulate in vector registers, for which the kernel must ask for two waves per SIMD (with one, the compiler keeps accumulators in the
// other half of the register file and moves all 16 of them to and fro around every four products); J on waves of its own;
// a step without branches; a shorter chain; a ticket drawn ahead, one acquire for all waves (each costs 250 cycles).
// Measured (us of the kernels, before and now): l = 24 68 -> 57, 30 85 -> 70, 48 199 -> 171 (row rotations before), 64 245 -> 206, 72 367 ->
// 329 (row rotations before), 97 555 -> 447, 110 558 -> 451, 128 580 -> 464, 160 1312 -> 1040, 272 2197 -> 1686, 400 6078 -> 4454.
// Since then SVD runs pass over pairs with nothing left to rotate (kIdle).
constexpr int kJB = 16;
constexpr int kJN = 2 * kJB;                      // rows of a block pair
// Place of entry (x, y) of the Gram matrix and of J: odd rows have their halves exchanged, so that the two rows of 16
// consecutive columns that half a wave touches, and 16 consecutive diagonal entries, lie on distinct banks.
__device__ __forceinline__ int jat(int x, int y) { return x * kJN + (y ^ ((x & 1) << 4)); }
constexpr int kJThreads = 512;                    // threads per block pair: two per pair (i, j) of pairs of rows, for the Gram matrix and for J
constexpr int kJWork = 3 * kJN * kJN + 128;       // doubles of LDS per block pair: two Gram buffers, J, rotations

__device__ __forceinline__ doublex4 mfma_f64(double a, double b, doublex4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Rotation (c, s) that makes two rows with squared norms al, be and inner product ga orthogonal: tan of the smaller
// angle, t = 2 ga / (tau +- sqrt(tau^2 + 4 ga^2)), tau = be - al.  The denominator is worked out in single precision: that only
// leaves 1e-7 of the inner product, while c and s, which have to be orthogonal, follow from t in double.  The numerator stays
// in double: rows whose norms are more than 2^126 apart need a t below the single-precision range.
// Everything is scaled by the power of two of the larger norm.  It bounds the inner product, so the scaling and all else that does
// not depend on ga is ready before ga is (RotationOf), and 13 dependent operations lead from ga to (c, s).
// Two rows of norm zero, or of one norm and a product below 1e-18 of it, have a denominator of 1e-18 at least, and |t| <= 1.
struct RotationOf {
  double eight, ab;       // 8 / 2^e with the sign of tau, 2^e the power of two of the larger norm; 64 al be / 2^(2 e)
  float tf, hh;           // 4 |tau| / 2^e and its square
};
// The power of two of a squared norm, kept where 8 / 2^e is a normal number: its biased exponent (a norm that rounding has made
// negative counts as zero).
__device__ __forceinline__ int norm_exponent(double al) { return min(max(__double2hiint(al) >> 20, 3), 2046); }
__device__ __forceinline__ RotationOf rotation_of(double al, int eal, double be, int ebe) {
  const int hi = (2049 - max(eal, ebe)) << 20;
  const double four = __hiloint2double(hi - (1 << 20), 0), as = al * four, bs = be * four, tau = bs - as;
  const float tf = fabsf((float)tau);
  return RotationOf{__hiloint2double(hi | (__double2hiint(tau) & 0x80000000), 0), 4.0 * as * bs, tf, fmaf(tf, tf, 1e-36f)};
}
// big: |ga| above the settled bar.  Returns t.
__device__ __forceinline__ double rotation(const RotationOf& p, double ga, double settled2, double& c, double& s, bool& big) {
  const double gd = ga * p.eight;                          // 8 ga / 2^e
  big = gd * gd > settled2 * p.ab;
  const float gf = (float)gd;
  const float inv = __builtin_amdgcn_rcpf(p.tf + __builtin_amdgcn_sqrtf(fmaf(gf, gf, p.hh)));
  const double t = gd * (double)inv;
  // c = 1 / sqrt(1 + t^2) from a single-precision seed y by one step of third order (2^-22 -> below 2^-64)
  const float ts = gf * inv;
  const double y = (double)__builtin_amdgcn_rsqf(fmaf(ts, ts, 1.f)), ty = t * y;
  const double e = fma(-ty, ty, fma(-y, y, 1.0)), w = fma(0.375 * e, e, 0.5 * e);
  c = fma(y, w, y);
  s = fma(ty, w, ty);
  return t;
}

// Value of the next lane, cyclically among each H lanes.
template <int H>
__device__ __forceinline__ double next_lane(double v, int lane) {
  if constexpr (H == 16) return dpp_f64<0x12F>(v);           // row_ror:15
  else if constexpr (H == 8) {
    const double up = dpp_f64<0x101>(v), back = dpp_f64<0x117>(v);     // row_shl:1, row_shr:7
    return (lane & 7) == 7 ? back : up;
  }
  else if constexpr (H == 4) return dpp_f64<0x39>(v);        // quad_perm [1,2,3,0]
  else if constexpr (H == 2) return dpp_f64<0xB1>(v);        // quad_perm [1,0,3,2]
  else return v;
}

// The eight waves of a block pair form the Gram matrix of its rows in buffer 0 of work; row(x) is the LDS address of row x, cols (a
// multiple of 16) its length.  It is symmetric: three tiles.  A matrix instruction of this kind keeps its SIMD busy for 64 cycles or
// more, so the work is dealt out evenly over the SIMDs: the first three quarters of the columns go to one SIMD for each tile, shared
// by its two waves w and w + 4, and the last quarter of all three tiles to wave 3 on the fourth.
template <typename Row>
__device__ __forceinline__ void gram_32(Row row, int cols, double* work, int t) {
  const int lane = t & 63, w = t >> 6, r = lane & 15, g = lane >> 4, q = w & 3, m = cols / 16;
  doublex4 acc[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) acc[k] = doublex4{0.0, 0.0, 0.0, 0.0};
  double* part = work + kJN * kJN + lane;        // partial tiles: those of waves 4, 5, 6, then the three of wave 3
  if (q < 3) {
    const double *lo = row((q == 2 ? kJB : 0) + r) + g, *hi = row((q == 0 ? 0 : kJB) + r) + g;
    const int mid = 3 * m / 2, end = w < 4 ? mid : 3 * m;
    int k = w < 4 ? 0 : mid;
    for (; k + 2 <= end; k += 2) {
      const double x0 = lo[4 * k], x1 = lo[4 * k + 4], y0 = hi[4 * k], y1 = hi[4 * k + 4];
      acc[0] = mfma_f64(x0, y0, acc[0]);
      acc[1] = mfma_f64(x1, y1, acc[1]);
    }
    if (k < end) acc[0] = mfma_f64(lo[4 * k], hi[4 * k], acc[0]);
    acc[0] += acc[1];
    if (w >= 4) {
#pragma unroll
      for (int v = 0; v < 4; ++v) part[256 * q + 64 * v] = acc[0][v];
    }
  } else if (w == 3) {
    const double *lo = row(r) + g, *hi = row(kJB + r) + g;
    for (int k = 3 * m; k < 4 * m; ++k) {
      const double x = lo[4 * k], y = hi[4 * k];
      acc[0] = mfma_f64(x, x, acc[0]);
      acc[1] = mfma_f64(x, y, acc[1]);
      acc[2] = mfma_f64(y, y, acc[2]);
    }
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int v = 0; v < 4; ++v) part[768 + 256 * k + 64 * v] = acc[k][v];
  }
  __syncthreads();
  if (w < 3) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int x = (w == 2 ? kJB : 0) + g + 4 * v, y = (w == 0 ? 0 : kJB) + r;
      const double s = (acc[0][v] + part[256 * w + 64 * v]) + part[768 + 256 * w + 64 * v];
      work[jat(x, y)] = s;
      if (w == 1) work[jat(y, x)] = s;
    }
  }
}

// The 32 rows in groups of 2 H: rotates all pairs of a row of the first half of a group with a row of its second half, in H steps
// (row x of the one with row (x + step) mod H of the other), on the Gram matrix in buffer 0 of work, and updates J (fresh: J is
// the identity so far).  Everything but the rotations lives in registers: the first 256 threads hold the 2 x 2 blocks of the pairs
// i and j, the others two rows of J each.  From one step to the next the rows of the second halves move up by one pair, i.e. columns come
// from the next lane and rows through LDS from the thread of the next pair.  The thread (i, i) works out the next rotation of
// pair i as soon as it has the new inner product: the squared norms follow from those before, al - t ga and be + t ga, so
// a step is one read, two multiplications and two multiply-adds, the rotation and one write between two barriers.  store: the Gram matrix is left in
// buffer 0.  Every thread of the workgroup calls it; the caller's barriers separate it from what is around it.
// Returns whether a rotation was above the settled bar.
template <int H>
__device__ __forceinline__ bool cross_pairs(double* work, int t, bool fresh, bool store, double settled2) {
  const int i = (t >> 4) & 15, j = t & 15, up = (i & ~(H - 1)) | ((i + 1) & (H - 1));
  auto top = [](int k) { return (k & ~(H - 1)) + k; };       // 2 H (k / H) + k mod H; the partner at step 0 is H rows below
  double* G = work;
  double2* T = (double2*)(work + kJN * kJN);                 // two buffers of 256
  double* J = work + 2 * kJN * kJN;
  double2* C = (double2*)(J + kJN * kJN);                    // two buffers of 16 x {c, s}
  double2* B = C + 32;                                       // two buffers of 16 x {squared norm, its exponent} of the second rows
  if (t >= 256) {
    const int f0 = jat(i, top(j)), f1 = jat(i, top(j) + H), h0 = f0 + kJB * kJN, h1 = f1 + kJB * kJN;   // rows i, 16 + i
    double p0, p1, q0, q1;
    if (fresh) {
      p0 = top(j) == i; p1 = top(j) + H == i; q0 = top(j) == kJB + i; q1 = top(j) + H == kJB + i;
    } else {
      p0 = J[f0]; p1 = J[f1]; q0 = J[h0]; q1 = J[h1];
    }
    __syncthreads();
    auto move = [&](int buf) {
      const double2 rj = C[buf + j];
      const double u = rj.y * p0 + rj.x * p1, w = rj.y * q0 + rj.x * q1;
      p0 = rj.x * p0 - rj.y * p1;
      q0 = rj.x * q0 - rj.y * q1;
      p1 = next_lane<H>(u, j);
      q1 = next_lane<H>(w, j);
      __syncthreads();
    };
#pragma unroll 1
    for (int step = 0; step + 1 < H; step += 2) { move(0); move(16); }
    if (H == 1) move(0);
    // H moves have brought every column home
    J[f0] = p0;
    J[f1] = p1;
    J[h0] = q0;
    J[h1] = q1;
    return false;
  }
  const int e0 = jat(top(i), top(j)), e1 = jat(top(i), top(j) + H);
  const int e2 = jat(top(i) + H, top(j)), e3 = jat(top(i) + H, top(j) + H);
  double a = G[e0], b = G[e1], bt = G[e2], cc = G[e3];
  const bool diag = i == j;
  bool any = false;
  double al = a;
  int eal = norm_exponent(al);
  T[16 * up + j] = double2{bt, cc};                          // where step 0 looks for them
  auto next_rotation = [&](const RotationOf& of, double be, double ga, int buf) {
    double c, s;
    bool big;
    const double tg = rotation(of, ga, settled2, c, s, big) * ga;
    any |= big && diag;
    al -= tg;
    eal = norm_exponent(al);
    double be_new = be + tg;
    int ebe = norm_exponent(be_new);
    asm volatile("" : "+v"(c), "+v"(s), "+v"(be_new), "+v"(ebe));      // before the branch, not in it
    if (diag) {
      C[buf + i] = double2{c, s};
      B[buf + i] = double2{be_new, __hiloint2double(ebe, 0)};
    }
  };
  next_rotation(rotation_of(al, eal, cc, norm_exponent(cc)), cc, b, 0);
  __syncthreads();
  // One step.  The chain that everything waits for -- the rotations read, the new inner product, the next rotation,
  // its store -- comes without a branch, so that the compiler lays the rest of the step into its gaps.
  auto move = [&](int buf, bool more) {
    const double2 rj = C[buf + j], ri = C[buf + i], be = B[buf + up];
    const double2 v = T[16 * (buf + up) + j];
    bt = v.x;
    cc = v.y;
    const RotationOf of = rotation_of(al, eal, be.x, __double2hiint(be.y));
    const double x0 = rj.x * a - rj.y * b, x1 = rj.y * a + rj.x * b;
    const double y0 = rj.x * bt - rj.y * cc, y1 = rj.y * bt + rj.x * cc;
    b = next_lane<H>(ri.x * x1 - ri.y * y1, j);
    a = ri.x * x0 - ri.y * y0;
    T[16 * (buf ^ 16) + t] = double2{ri.y * x0 + ri.x * y0, next_lane<H>(ri.y * x1 + ri.x * y1, j)};
    if (more) next_rotation(of, be.x, b, buf ^ 16);
    __syncthreads();
  };
#pragma unroll 1
  for (int step = 0; step + 2 < H; step += 2) { move(0, true); move(16, true); }
  if (H > 1) move(0, true);
  move(H > 1 ? 16 : 0, false);
  if (store) {                                               // H moves have brought every row and column home
    const double2 v = T[(H & 1) * 256 + 16 * up + j];
    G[e0] = a;
    G[e1] = b;
    G[e2] = v.x;
    G[e3] = v.y;
  }
  return any;
}

// Whether an inner product in the Gram matrix in buffer 0 of work, of all pairs of the 32 rows or of those across the two blocks, is
// above the idle bar (or not a number).  Every thread of the workgroup calls it.
__device__ __forceinline__ bool busy_32(const double* work, int t, bool all, double idle) {
  __syncthreads();
  bool busy = false;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int e = t + q * kJThreads, x = e >> 5, y = e & 31;
    if (x < y && (all || (x < kJB && y >= kJB)))
      busy |= !(fabs(work[jat(x, y)]) <= idle * fmin(work[jat(x, x)], work[jat(y, y)]));
  }
  return __syncthreads_or(busy);
}

// One sweep of rotations on the Gram matrix in buffer 0 of work: all pairs of the 32 rows, or those across the two blocks.  fresh, store: as for
// cross_pairs.
__device__ __forceinline__ bool sweep_32(double* work, int t, bool all, double settled2, bool fresh = true, bool store = false) {
  bool any = false;
  __syncthreads();
  if (all) {
    any |= cross_pairs<8>(work, t, fresh, true, settled2);
    __syncthreads();
    any |= cross_pairs<4>(work, t, false, true, settled2);
    __syncthreads();
    any |= cross_pairs<2>(work, t, false, true, settled2);
    __syncthreads();
    any |= cross_pairs<1>(work, t, false, true, settled2);
    __syncthreads();
  }
  any |= cross_pairs<16>(work, t, !all && fresh, store, settled2);
  __syncthreads();
  return any;
}

// The 16 columns from c0 on of J^T times the rows of a block pair (one wave): out(x, col, value) for the 32 x 16 entries.
template <typename Row, typename Out>
__device__ __forceinline__ void apply_32(Row row, const double* J, int c0, int lane, Out out) {
  const int r = lane & 15, g = lane >> 4;
  doublex4 acc[2];
  acc[0] = acc[1] = doublex4{0.0, 0.0, 0.0, 0.0};
  double b[kJN / 4];
#pragma unroll
  for (int k = 0; k < kJN / 4; ++k) b[k] = row(4 * k + g)[c0 + r];
#pragma unroll
  for (int k = 0; k < kJN; k += 4) {
    acc[0] = mfma_f64(J[jat(k + g, r)], b[k / 4], acc[0]);
    acc[1] = mfma_f64(J[jat(k + g, kJB + r)], b[k / 4], acc[1]);
  }
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int v = 0; v < 4; ++v) out(kJB * m + g + 4 * v, c0 + r, acc[m][v]);
}

// Bytes of LDS of a block pair: its rows have Lp columns (padding zero) and a stride of Lp + 2 doubles, which spreads the 16
// rows a wave reads over the banks.
static constexpr size_t jacobi_lds_bytes(int Lp) { return sizeof(double) * ((size_t)kJN * (Lp + 2) + kJWork); }

// Up to 32 rows: one workgroup, one block pair.  A sweep is 31 steps, and a third as much for the Gram matrix and J^T times the rows, which
// two sweeps on one Gram matrix need once (us, before and with it: l = 30 55 and 50, 20 67 and 64).  That matrix does not tell when to
// stop: what is left of two rows that were nearly parallel is lost in it, and may be far from orthogonal.  After a pair of sweeps whose second
// one met nothing above the bar, a fresh Gram matrix without anything above the idle bar ends the iteration, or a single sweep on it decides.
constexpr int kTwoSweeps = 4;                      // from sweep 0 to 4, two at a time
__global__ void __launch_bounds__(kJThreads, 2)
k_jacobi_small(const double* __restrict__ R, int ldr, int l, int Lp, double* __restrict__ Wg, double* __restrict__ sig,
               int* __restrict__ info, const int* __restrict__ breakdown_flag, double settled, double idle) {
  extern __shared__ __align__(16) double W[];
  __shared__ int rotated;
  __shared__ int order_sh[kJN];
  const int t = threadIdx.x, ld = Lp + 2;
  if (breakdown_flag && breakdown_flag[0] != 0) {
    if (t == 0) { info[0] = 0; info[1] = 0; }
    return;
  }
  constexpr int XN = kJN / (kJThreads / 32);
  unsigned aside = 0;                                  // bit q: row (t >> 5) + q (kJThreads / 32) is set aside
  double first[XN];
#pragma unroll
  for (int q = 0; q < XN; ++q) {
    const int i = (t >> 5) + q * (kJThreads / 32), c = t & 31;      // Lp <= 32: a lane has one entry of a row
    first[q] = R[(int64_t)min(i, l - 1) * ldr + min(c, l - 1)];
    if (i >= l || c >= l) first[q] = 0.0;
  }
#pragma unroll
  for (int q = 0; q < XN; ++q) {
    const int i = (t >> 5) + q * (kJThreads / 32), c = t & 31;
    double v = first[q];
    // (an entry whose square is near the largest double: nothing rotates against such a row)
    if ((unsigned)(__ballot(!(fabs(v) < 0x1p509)) >> (t & 32))) { aside |= 1u << q; v = 0.0; }
    if (c < Lp) W[i * ld + c] = v;
  }
  double* work = W + kJN * ld;
  int sweeps = 0, converged = (l < 2), quiet = 0;      // quiet: the second of a pair of sweeps met nothing above the bar
  auto row = [&](int x) { return W + x * ld; };
  while (!converged && sweeps < kMaxSweeps) {
    if (t == 0) rotated = 0;
    __syncthreads();
    gram_32(row, Lp, work, t);
    if (quiet && !busy_32(work, t, true, idle)) {        // uniform over the workgroup
      converged = 1;
      break;
    }
    const bool two = sweeps < kTwoSweeps && !quiet;
    if (two) {
      sweep_32(work, t, true, settled * settled, true, true);
      ++sweeps;
    }
    if (sweep_32(work, t, true, settled * settled, !two)) rotated = 1;
    for (int c0 = kJB * (t >> 6); c0 < Lp; c0 += (kJThreads / 64) * kJB)
      apply_32(row, work + 2 * kJN * kJN, c0, t & 63, [&](int x, int c, double v) { row(x)[c] = v; });
    __syncthreads();
    ++sweeps;
    quiet = rotated == 0;
    converged = quiet && !two;
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < kJN / (kJThreads / 32); ++q) {
    const int i = (t >> 5) + q * (kJThreads / 32), c = t & 31;
    if ((aside >> q & 1) && i < l && c < l) W[i * ld + c] = R[(int64_t)i * ldr + c];
  }
  __syncthreads();
  publish<kJThreads>(W, ld, l, Lp, Wg, sig, order_sh, t, t & 63, t >> 6);
  if (t == 0) { info[0] = sweeps; info[1] = converged; }
}

// ---- more than 32 rows: one workgroup per pair of blocks ---------------------------------------------------------------
// info: [0] sweeps done, [1] converged, [2] tickets done, [3] last sweep (from 1) with a rotation above the bar, [4] nothing to do,
// [5] a workgroup has given up waiting, [6] tickets taken.
// One workgroup of 128 threads per row; sig[Lp + i]: the squared norm of a row that is set aside, otherwise 0.
__global__ void __launch_bounds__(128)
k_jacobi_init(const double* __restrict__ R, int ldr, int l, int Lp, double* __restrict__ W, double* __restrict__ sig,
              int* __restrict__ info, const int* __restrict__ breakdown_flag) {
  __shared__ double part[2];
  const int c = threadIdx.x, i = blockIdx.x;
  if (i == 0 && c < 8) info[c] = c == 4 && breakdown_flag && breakdown_flag[0] != 0;
  double v[kMaxL / 128], s2 = 0.0;
#pragma unroll
  for (int q = 0; q < kMaxL / 128; ++q) {
    const int cc = c + 128 * q;
    v[q] = i < l && cc < l ? R[(int64_t)i * ldr + cc] : 0.0;
    s2 = fma(v[q], v[q], s2);
  }
  s2 = wave_sum(s2);
  if ((c & 63) == 0) part[c >> 6] = s2;
  __syncthreads();
  s2 = part[0] + part[1];
  const bool aside = !isfinite(s2);
  if (c == 0) sig[Lp + i] = aside ? s2 : 0.0;
#pragma unroll
  for (int q = 0; q < kMaxL / 128; ++q) {
    const int cc = c + 128 * q;
    if (cc < Lp) W[(int64_t)i * Lp + cc] = aside ? 0.0 : v[q];
  }
}

// Ticks of the 100 MHz clock after which a workgroup stops waiting for the others (20 s).  Those it waits for are running (see
// k_jacobi_rounds) and need some 30 us; the limit only makes sure that every wait ends (the call then reports that the
// iteration did not converge).
constexpr unsigned long long kMeetTicks = 2000000000ull;
constexpr int kWaitStores = 0x0f70;              // s_waitcnt: no vector memory operation outstanding, the other counters as they are

// The 32 rows of the block pair at rows rI and rJ of W, to LDS; rows from l on are zero.  64 H columns at a time are under way.
template <int H>
__device__ __forceinline__ void load_pair(const double* W, int l, int Lp, int rI, int rJ, double* sh, int ld, int t) {
  constexpr int XN = kJN / (kJThreads / 32);
  for (int c0 = 2 * (t & 31); c0 < Lp; c0 += 64 * H) {
    double2 v[XN][H];
#pragma unroll
    for (int q = 0; q < XN; ++q) {
      const int x = (t >> 5) + q * (kJThreads / 32), i = x < kJB ? rI + x : rJ + x - kJB;
      const double* src = W + (int64_t)min(i, l - 1) * Lp;
#pragma unroll
      for (int h = 0; h < H; ++h) v[q][h] = *(const double2*)(src + min(c0 + 64 * h, Lp - 2));
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < XN; ++q) {
      const int x = (t >> 5) + q * (kJThreads / 32), i = x < kJB ? rI + x : rJ + x - kJB;
#pragma unroll
      for (int h = 0; h < H; ++h)
        if (c0 + 64 * h < Lp) *(double2*)(sh + x * ld + c0 + 64 * h) = i < l ? v[q][h] : double2{0.0, 0.0};
    }
  }
}

// All sweeps in one launch.  The workgroups (nblk2 / 2 of them; any number will do) take tickets in order, one after the other, and
// start on one when all tickets of the rounds before are done.  A workgroup therefore only waits for lower tickets, which
// running ones hold, and the lowest of these waits for nothing: the iteration goes on however few of the workgroups find room on
// the device, on a stream with a few CUs or beside kernels that fill the rest.
// A ticket is drawn while the one before it is worked on.  A workgroup works through its tickets in their order, so the lowest
// unfinished one is still always at work or about to be.
// The rows travel through global memory between rounds; they are stored at the scope of the device, past the L2 of an XCD, which
// leaves the releases at a meeting little to write back (2 to 4 % of the whole).  With a launch per round, and the host looking at the
// convergence flag, l = 160 took 1980 us and 272 4280 us.  Eight times the workgroups with all but every eighth leaving at
// once, to keep the rest on one XCD, gains 5 % below 128 and loses up to 13 % above.
__global__ void __launch_bounds__(kJThreads, 2)
k_jacobi_rounds(const double* R, int ldr, double* W, int l, int Lp, int nblk2, double settled, double idle, double* sig, int* info) {
  extern __shared__ __align__(16) double sh[];
  __shared__ int next, state;
  const int t = threadIdx.x, ld = Lp + 2;
  if (info[4]) return;
  double* work = sh + kJN * ld;
  auto row = [&](int x) { return sh + x * ld; };
  int ticket = 0;
  int* drawn = info + 6;
  asm("" : "+v"(drawn));      // one that is known to be uniform makes the compiler wait for the result where it is asked for
  if (t == 0) ticket = __hip_atomic_fetch_add(drawn, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  for (;;) {
    if (t == 0) {
      const int before = jacobi_ticket(ticket, nblk2).before;
      const unsigned long long start = wall_clock64();
      int now;
      // the tickets done and the latest sweep with a rotation above the bar, in one load
      for (;;) {
        const unsigned long long both = __hip_atomic_load((unsigned long long*)(info + 2), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        now = (int)(both >> 32);
        if ((int)both >= before) break;
        if (wall_clock64() - start > kMeetTicks || __hip_atomic_load(info + 5, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
          __hip_atomic_store(info + 5, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          now = -1;
          break;
        }
      }
      next = ticket;
      state = now;
      // one wave acquires for the workgroup: what it invalidates is shared by all of them, and the others start behind the barrier
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
    if (state < 0) return;
    const JacobiTicket k = jacobi_ticket(__builtin_amdgcn_readfirstlane(next), nblk2);
    const int last = __builtin_amdgcn_readfirstlane(state), what = jacobi_work(k, last, kMaxSweeps);
    if (t == 0 && what != JACOBI_END) ticket = __hip_atomic_fetch_add(drawn, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (what == JACOBI_ROTATE) {
      int I, J;
      rr_pair(k.pair, k.round, nblk2, I, J);
      const int rI = I * kJB, rJ = J * kJB;             // I < J; the last blocks may be all padding
      auto grow = [&](int x) { return x < kJB ? rI + x : rJ + x - kJB; };
      if (rI < l && (k.round == 0 || rJ < l)) {         // uniform over the workgroup
        if (Lp <= 128) load_pair<2>(W, l, Lp, rI, rJ, sh, ld, t);
        else load_pair<4>(W, l, Lp, rI, rJ, sh, ld, t);
        __syncthreads();
        gram_32(row, Lp, work, t);
        const bool busy = idle == 0.0 || k.sweep < kIdleFrom || busy_32(work, t, k.round == 0, idle);   // uniform over the workgroup
        if (busy && sweep_32(work, t, k.round == 0, settled * settled) && last <= k.sweep)
          __hip_atomic_fetch_max(info + 3, k.sweep + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        for (int c0 = kJB * (t >> 6); busy && c0 < Lp; c0 += (kJThreads / 64) * kJB)
          apply_32(row, work + 2 * kJN * kJN, c0, t & 63, [&](int x, int c, double v) {
            if (grow(x) < l) __hip_atomic_store(W + (int64_t)grow(x) * Lp + c, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          });
      }
    } else {
      if (what == JACOBI_END) return;
      // the rows of the blocks 2 pair and 2 pair + 1, eight lanes a row: their norms, then their places in the descending order
      const int i = t < 256 ? 2 * kJB * k.pair + (t >> 3) : l, e0 = t & 7;
      if (what == JACOBI_NORMS) {
        double s2 = 0.0;
        const double left = i < l ? sig[Lp + i] : 0.0;      // not zero: a row that was set aside
        if (i < l)
          for (int e = e0; e < l; e += 8) {
            if (left != 0.0) W[(int64_t)i * Lp + e] = R[(int64_t)i * ldr + e];
            const double v = W[(int64_t)i * Lp + e];
            s2 = fma(v, v, s2);
          }
        s2 = row8_sum(s2);
        if (i < l && e0 == 0) sig[Lp + i] = sqrt(left != 0.0 ? left : s2);
      } else {
        if (i < l) {
          const double si = sig[Lp + i];
          int rank = 0;
          for (int j = e0; j < l; j += 8) rank += ranks_before(sig[Lp + j], j, si, i);
          for (int off = 4; off > 0; off >>= 1) rank += __shfl_xor(rank, off, 8);
          if (e0 == 0) { sig[rank] = si; sig[2 * Lp + rank] = (double)i; }
        }
        if (k.pair == 0 && t == 0) { info[0] = k.sweep; info[1] = last < k.sweep; }
      }
    }
    // Each wave waits for its own stores before the barrier, which does not wait for them; then one releases for all.
    __builtin_amdgcn_s_waitcnt(kWaitStores);
    __syncthreads();
    if (t == 0) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      __hip_atomic_fetch_add(info + 2, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}


// Sorted factors.  Vr[t][i] = W[o_i][t] / s_i;  Ur[kk][i] = sum_t R[kk][t] Vr[t][i] / s_i.
// XV / XU: zero-padded Lp x Lp right operands of the lifts; Ur / Vr: optional dense fp64.  left: XV = left Vr; upper: R (then not the matrix
// whose SVD this is) and left are upper triangular.
// A workgroup per tile of 16 x 16 of XU (blockIdx.z = 0) or XV, on v_mfma_f64_16x16x4_f64: lane (r, g) holds R[kk + r][t + g] and W[o_(i+r)][t + g],
// which come from other dies' work, at a latency of a microsecond and more; eight waves share the contraction for that.
// Measured (us with the launch; one thread per entry before, without the product for XV): l = 30 6.0 -> 4.7, 110 13.4 -> 7.7, 272 42.8 -> 13.9.
template <typename TO>
__global__ void __launch_bounds__(kTileWaves * 64)
k_svd_outputs(const double* __restrict__ R, int ldr, int upper, const TO* __restrict__ left, const double* __restrict__ W,
              const double* __restrict__ sig, int l, int Lp, double* __restrict__ S, TO* __restrict__ S32, TO* __restrict__ XV,
              TO* __restrict__ XU, double* __restrict__ Ur, double* __restrict__ Vr, const int* __restrict__ breakdown_flag) {
  if (breakdown_flag && breakdown_flag[0] != 0) return;   // nothing was computed
  __shared__ double part[kTileWaves][256];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15, g = lane >> 4;
  const int kk0 = kTile * blockIdx.y, i = kTile * blockIdx.x + r;
  const bool isv = blockIdx.z != 0;
  const int o = min(max((int)sig[2 * Lp + min(i, l - 1)], 0), l - 1);   // stays in range even for NaN input
  const double s = i < l ? sig[min(i, l - 1)] : 0.0;
  const double* wrow = W + (int64_t)o * Lp;
  doublex4 acc = {0.0, 0.0, 0.0, 0.0};
  const int arow = min(kk0 + r, l - 1);
  auto product = [&](const auto* A, int lda) {
    const auto* a0 = A + (int64_t)arow * lda;
    double an[4], bn[4];
    auto load = [&](int t0) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int t = t0 + 4 * q + g, tc = min(t, l - 1);
        an[q] = (double)a0[tc];
        bn[q] = wrow[tc];
        if (t >= l) bn[q] = 0.0;
        if (t >= l || (upper && t < arow)) an[q] = 0.0;
      }
    };
    int t0 = (upper ? kk0 : 0) + kTile * wave;
    load(t0);
    for (; t0 < l; t0 += kTileWaves * kTile) {
      double a[4], b[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) { a[q] = an[q]; b[q] = bn[q]; }
      load(t0 + kTileWaves * kTile);
#pragma unroll
      for (int q = 0; q < 4; ++q) acc = mfma_f64(a[q], b[q], acc);
    }
  };
  if (!isv) {
    product(R, ldr);
  } else if (left) {
    product(left, Lp);
  } else if (wave == 0) {
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[v] = wrow[min(kk0 + g + 4 * v, l - 1)];
  }
  if (!sum_over_waves(acc, part, lane, wave)) return;
  const double div = isv ? s : s * s;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int kk = kk0 + g + 4 * v;
    const bool in = kk < l && i < l;
    const double x = in && s > 0.0 ? acc[v] / div : 0.0;
    TO* X = isv ? XV : XU;
    double* D = isv ? Vr : Ur;
    if (X) X[(int64_t)kk * Lp + i] = (TO)x;
    if (D && in) D[(int64_t)kk * l + i] = x;
    if (isv && kk == 0 && i < l) {
      if (S) S[i] = s;
      if (S32) S32[i] = (TO)s;
    }
  }
}

static int jacobi_global(const double* R, int ldr, int l, int Lp, SvdWork& w, const int* breakdown_flag, double settled, double idle,
                         hipStream_t stream) {
  static bool attr_set = false;
  if (!attr_set) {
    BRSVD_HIP_TRY(hipFuncSetAttribute((const void*)k_jacobi_rounds, hipFuncAttributeMaxDynamicSharedMemorySize,
                                      (int)jacobi_lds_bytes(kMaxL)));
    attr_set = true;
  }
  hipLaunchKernelGGL(k_jacobi_init, dim3(Lp), dim3(128), 0, stream, R, ldr, l, Lp, w.W, w.sig, w.info, breakdown_flag);
  const int nblk = (int)ceil_div(l, kJB), nblk2 = (nblk + 1) & ~1;
  hipLaunchKernelGGL(k_jacobi_rounds, dim3(nblk2 / 2), dim3(kJThreads), jacobi_lds_bytes(Lp), stream, R, ldr, w.W, l, Lp, nblk2,
                     settled, idle, w.sig, w.info);
  BRSVD_HIP_TRY(hipGetLastError());
  return BRSVD_OK;
}

template <typename TO>
int small_svd(const double* R, int ldr, int l, int Lp, SvdWork& w, const int* breakdown_flag, double* S,
              TO* S32, TO* XV, TO* XU, double* Ur, double* Vr, hipStream_t stream, const OpenFactors<TO>* open) {
  if (l < 1 || l > kMaxL || (open && (!open->Rx || Ur || Vr))) return BRSVD_ERR_ARG;
  // fp64 factors or singular values asked for: the strict bar; single-precision results only: the relaxed one
  const double settled = (sizeof(TO) == 4 && !S && !Ur && !Vr) ? kSettledF32 : kSettled;
  const double idle = settled == kSettledF32 ? kIdleF32 : kIdle;
  const int nblk = (l + kJB - 1) / kJB;
  if (l <= kRowsMaxL || nblk == 3) {
    auto kern = nblk == 1 ? k_jacobi_rows<1, 8> : l <= 40 ? k_jacobi_rows<3, 24> : k_jacobi_rows<3, 32>;
    const int threads = LPP * (nblk == 1 ? 8 : l <= 40 ? 24 : 32);
    hipLaunchKernelGGL(kern, dim3(1), dim3(threads), (size_t)l * l * sizeof(double), stream, R, ldr, l, Lp, w.W, w.sig, w.info,
                       breakdown_flag, kTolRows, settled);
    BRSVD_HIP_TRY(hipGetLastError());
  } else if (l <= kJN) {
    hipLaunchKernelGGL(k_jacobi_small, dim3(1), dim3(kJThreads), jacobi_lds_bytes(Lp), stream, R, ldr, l, Lp, w.W, w.sig, w.info,
                       breakdown_flag, settled, idle);
    BRSVD_HIP_TRY(hipGetLastError());
  } else {
    BRSVD_TRY(jacobi_global(R, ldr, l, Lp, w, breakdown_flag, settled, Ur || Vr ? 0.0 : idle, stream));
  }
  const dim3 tiles(Lp / kTile, Lp / kTile, 2);
  hipLaunchKernelGGL(k_svd_outputs<TO>, tiles, dim3(kTileWaves * 64), 0, stream, open ? open->Rx : R, ldr, open ? 1 : 0,
                     open ? open->left : nullptr, w.W, w.sig, l, Lp, S, S32, XV, XU, Ur, Vr, breakdown_flag);
  BRSVD_HIP_TRY(hipGetLastError());
  return BRSVD_OK;
}

template int small_svd<float>(const double*, int, int, int, SvdWork&, const int*, double*, float*, float*, float*,
                              double*, double*, hipStream_t, const OpenFactors<float>*);
template int small_svd<double>(const double*, int, int, int, SvdWork&, const int*, double*, double*, double*, double*,
                               double*, double*, hipStream_t, const OpenFactors<double>*);

}  // namespace brsvd
