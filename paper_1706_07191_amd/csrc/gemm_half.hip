// The products of gemm_split.hip for contractions that are long enough (the rule and what it was measured on: half_fits there) with
// two fp16 numbers in the place of three bf16 ones: every operand is scaled by a power of two and split,
//
//   2^e a = h + l,   h = fp16(2^e a), l = fp16(2^e a - h),  both rounded to nearest
//
// (11 + 11 significant bits and the sign of l: of the 24 bits of a at most the last one is lost, for a quarter of the numbers).  Of
// the four products l*h + h*l + h*h are taken, the fourth is below 2^-22 of |a||x| and 2^-25 on average: three
// v_mfma_f32_16x16x32_f16 do what takes six v_mfma_f32_16x16x32_bf16 of the same cost.
//
// Range.  fp16 ends at 2^-24, so a number is only held to its 23 bits down to 2^-17 of the largest one under the same scale, below to
// an error of 2^-39 of that one.  The scale of A belongs to a row (A^T Q: a column) and a step of 64 contraction indices, that of the
// panel to a step.  With M and N the largest of the two, such errors come to at most 2^-39 M N for each index of either operand that is
// that small, and that is little beside the step's sum of |a||x| as long as enough large numbers meet:
//   - of the 16 runs of four successive indices in a row's step, 14 or more hold a number of at least 2^-7 M;
//   - a column of the panel has no more than 11 of its 64 entries below 2^-9 N, or is zero.
// Each of those 11 takes the large number of one run, so at least 3 are left: the sum of |a||x| is at least 3 * 2^-16 M N, and the
// (50 + 11) 2^-39 M N are less than 2^-18.6 of it.  With the 2^-21 that the split itself and l*l may lose, a step's sum is off by less
// than 2^-18 of |a||x|, what 64 rounded fp32 additions may lose, whatever the numbers are.  (The last two steps of a contraction
// may have as few as 32 indices.  Of those the first 32 count: 7 of 8 runs, 5 entries, and less than 2^-17 is lost.)  Of N(0, 1) entries a
// step of a row fails with a chance below 10^-16, one of a panel of 272 columns below 10^-11 (of 32 indices 2 * 10^-5).
// A row's step that fails, or whose scales' product leaves the range of fp32, is multiplied as zeros and noted; the wave that did so adds
// its 64 products in fp32 at the end.  bf16 numbers (which hold every range) take over
//   - where a column of the panel fails, or it has an infinity, or one of the up to 64 rows per step that the packing looks at fails: all
//     workgroups leave their parts to k_split_fix_*;
//   - where a wave meets more steps with such rows than it can note (kMaxNoted), or more rows in all than it is worth (kMaxRows): what its
//     workgroup has done is done again.
// Measured, six bf16 products and this (us, A X / A^T Q, 60000x6000 l=110): N(0, 1) entries 491 / 480 and 401 / 376, one of them 10^6 477 / 470
// and 390 / 378 (744 / 551 when its workgroup did its part again), 24 of them 479 / 484 and 407 / 493 (sampled in A^T Q), half of A zero
// 470 / 480 and 511 / 485.
//
// Accuracy.  A step's six products are added into one register tile, which is then added to the running sum by rounded fp32
// fused multiply-adds: half as many additions as in gemm_split.hip, whose error is the larger part of both.  Measured: half_fits.
#include "split.h"

namespace brsvd {

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

struct Frag2 { uintx4 p[2]; };       // h, l of eight contraction indices

__device__ __forceinline__ floatx4 mfma_f16(uintx4 a, uintx4 b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}
// Pair q (elements 2q, 2q + 1) of a fragment; scale is a power of two.
__device__ __forceinline__ void half_pair(float a, float b, float scale, Frag2& f, int q) {
  a *= scale;
  b *= scale;
  const f16x2 h = __builtin_convertvector(floatx2{a, b}, f16x2);
  f.p[0][q] = __builtin_bit_cast(unsigned, h);
  const f16x2 l = __builtin_convertvector(floatx2{a - (float)h[0], b - (float)h[1]}, f16x2);
  f.p[1][q] = __builtin_bit_cast(unsigned, l);
}

constexpr int kHalfEarly = 8;                     // see EARLY
constexpr int kHalfStep = 2 * kSplitB;            // contraction indices per step: one scale, one block sum
constexpr unsigned kExpMask = 0x7f800000u, kExpOne = 1u << 23;
constexpr unsigned kUntame = 0x100;               // bit of the upper half of a step's word: not fit for this
constexpr int kMaxNoted = 31, kMaxRows = 64, kSampled = 64;
// Scales: the largest number becomes one in [2^14, 2^15), i.e. it is multiplied by 2^(14 - (E - 127)) with its exponent field E, at
// least 15 (then 2^126, and even subnormal numbers are held whole).  A block sum is multiplied by 2^(E_A - 141 + E_X - 141), whose
// exponent field is E_A + E_X - 155.  The upper half of a step's word holds E_X.

// Largest over the four groups of 16 lanes.
__device__ __forceinline__ unsigned max_groups(unsigned v) {
  const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = max((unsigned)a[0], (unsigned)a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return max((unsigned)b[0], (unsigned)b[1]);
}
// Largest over the 16 lanes of a row.
template <int CTRL>
__device__ __forceinline__ float max_ror(float x) {
  return fmaxf(x, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xf, 0xf, true)));
}
__device__ __forceinline__ float max_row(float x) { return max_ror<0x121>(max_ror<0x122>(max_ror<0x124>(max_ror<0x128>(x)))); }

__device__ __forceinline__ int sum_groups(int v) {
  const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = (int)a[0] + (int)a[1];
  const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return (int)b[0] + (int)b[1];
}
// The test of a row's step, see above: run = the largest of each four successive indices that this lane holds (the other groups of lanes
// hold the rest), m = the largest of the step; returns how many of the lane's are large, min_runs of them in all groups pass.  whole: 64
// indices, otherwise the first 32 count.  (Where 2^-7 m rounds to zero, m is so small that fp16 holds every number of the row whole.)
constexpr float kLargeRun = 0x1p-7f, kLargeEntry = 0x1p-9f;
constexpr int kMaxSmall = 11, kMaxSmallHalf = 5;
__device__ __forceinline__ int min_runs(bool whole) { return whole ? 14 : 7; }
__device__ __forceinline__ int large_runs(const float (&run)[4], bool whole, unsigned& m) {
  m = max_groups(__float_as_uint(fmaxf(fmaxf(run[0], run[1]), fmaxf(run[2], run[3]))));
  const float thr = __uint_as_float(m) * kLargeRun;
  const int n0 = (run[0] >= thr ? 1 : 0) + (run[1] >= thr ? 1 : 0), n1 = (run[2] >= thr ? 1 : 0) + (run[3] >= thr ? 1 : 0);
  return n0 + (whole ? n1 : 0);
}

// Packed panel: [step][column tile][block of the step][h, l][lane][8 fp16], 4 KiB per step and tile of 16 columns.  One workgroup per step
// of 64 rows, PER tiles of columns per wave.  Also clears the flags, and looks at the step in up to 64 rows (AT: columns) of A, 16 per
// wave, so that a matrix of many magnitudes is not found out by every workgroup of the product on its own.
// What bounds it: the latency of its loads and of two reductions (20000 x 110 9.5 us, 100000 x 272 56 us).
template <int PER>
__global__ void __launch_bounds__(1024)
k_half_pack(const float* __restrict__ src, int64_t K, int64_t ld, int cols, int nt_total, uintx4* __restrict__ out,
            unsigned* __restrict__ words, int* __restrict__ flags, int64_t nflags, const float* __restrict__ A, int64_t lda, int64_t count_a,
            int at) {
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, threads = (int64_t)gridDim.x * blockDim.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6, r = lane & 15, g = lane >> 4;
  const int64_t chunk = blockIdx.x, blocks = 2 * (int64_t)gridDim.x;
  __shared__ unsigned top;
  __shared__ int untame;
  if (threadIdx.x == 0) { top = 0; untame = 0; }
  const bool whole = chunk < whole_steps(K);
  float v[PER][16];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int col = 16 * (wave + i * waves) + r;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int64_t blk = 2 * chunk + (e >> 3), k = block_start(blk, K) + ((e >> 2) & 1) * 16 + 4 * g + (e & 3);
      v[i][e] = k >= block_first(blk, K) && col < cols ? src[k * ld + col] : 0.f;
    }
  }
  bool bad = false;
  if (wave < kSampled / 16) {
    const int64_t row = (chunk * 2654435761u + threadIdx.x / 64 * 16 + r) % count_a;             // of A (column, if at)
    float run[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float* p = A + (at ? row : row * lda);
      const int64_t k = block_start(2 * chunk + (q >> 1), K) + (q & 1) * 16 + 4 * g, step = at ? lda : 1;
      run[q] = fmaxf(fmaxf(fabsf(p[k * step]), fabsf(p[(k + 1) * step])), fmaxf(fabsf(p[(k + 2) * step]), fabsf(p[(k + 3) * step])));
    }
    unsigned m;
    bad = sum_groups(large_runs(run, whole, m)) < min_runs(whole);
  }
  for (int64_t i = id; i < nflags; i += threads) flags[i] = 0;
  __syncthreads();
  float most = 0.f;                                                       // (fmaxf leaves NaN out)
#pragma unroll
  for (int i = 0; i < PER; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) most = fmaxf(most, fabsf(v[i][e]));
  const unsigned wave_max = max_groups(__float_as_uint(max_row(most)));
  if (lane == 0) atomicMax(&top, wave_max);
  __syncthreads();
  const unsigned gmax = top;
  const unsigned ex = gmax == 0 ? 127u << 23 : max(gmax & kExpMask, 15u << 23);
  const float scale = __uint_as_float((268u << 23) - ex), thr = __uint_as_float(gmax) * kLargeEntry;
  const int need = whole ? kHalfStep - kMaxSmall : kHalfStep / 2 - kMaxSmallHalf;
  unsigned first = 0;
  bad |= gmax >= kExpMask;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int nt = wave + i * waves;
    if (nt >= nt_total) break;
    Frag2 f[2];
    bool any_nan[2] = {false, false};
    float cm = 0.f;
    int count = 0;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      any_nan[e >> 3] |= v[i][e] != v[i][e];
      cm = fmaxf(cm, fabsf(v[i][e]));
      count += fabsf(v[i][e]) >= thr && (whole || e < 8) ? 1 : 0;
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) half_pair(v[i][2 * q], v[i][2 * q + 1], scale, f[q >> 2], q & 3);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const unsigned long long b = __ballot(any_nan[s]);                   // bit 16 * g + r
      const unsigned word = (unsigned)(b | b >> 16 | b >> 32 | b >> 48) & 0xffffu;
      if (nt == 0 && s == 0) first = word;
      else if (lane == 0) words[nt * blocks + 2 * chunk + s] = word;
#pragma unroll
      for (int p = 0; p < 2; ++p) out[((chunk * nt_total + nt) * 4 + 2 * s + p) * kFragU + lane] = f[s].p[p];
    }
    count += __shfl_xor(count, 16, 64);
    count += __shfl_xor(count, 32, 64);
    cm = __uint_as_float(max_groups(__float_as_uint(cm)));
    bad |= cm != 0.f && count < need;
  }
  if (bad) untame = 1;
  __syncthreads();
  if (threadIdx.x == 0) words[2 * chunk] = first | (ex >> 23 | (untame ? kUntame : 0)) << 16;
}

struct HalfPanel {
  const uintx4* panel;     // of the launch's columns
  int64_t stride;          // 16-byte units of one step
  const unsigned* words;
  int *flags, *redo;
  int c0;                  // the first of the launch's columns
  // all columns, and the panel as it was
  uintx4* all;
  const float* X;
  int64_t ld, steps;
  int cols, nt_total;
};
// In LDS: the steps with rows that were left out, and these rows as bits, for each wave; one more entry than it may hold, which is
// written for the steps without.
typedef uint2 Noted[8][kMaxNoted + 1];

// Workgroup: as in gemm_split.hip, WR x WC waves of MT tiles of 16 rows (AT: columns of A) and NTW tiles of the panel's columns; but the
// panel is the first operand of the instruction and A the second, so that a lane's results belong to one row and that row's scale
// is in the lane that split it.
//
// What bounds it: below 15 column tiles, and with 4 alone, the latency of the loads of A.  With 17 the chip is at its power limit (1.65 GHz),
// but the matrix cores are only 47 % busy (the six bf16 products: 63 to 67 % at the same clock); where the rest of the power goes is not
// established -- from 11 tiles on both columns of waves load, scan and split the same rows, and A X keeps 8 to 88 bytes a lane in scratch
// (13 to 17 tiles).  As there, everything else is spread over the stream of matrix
// instructions: the panel's fragments from LDS, the block sums, the scale of the next step (all of its part of A has to be there:
// in the middle of the step), its split, the loads, and the hand-over of the panel, in parts to need fewer registers.  The code of a
// step has no branch, also not for the rows that are left out: the compiler would put off sums past it and run out of registers (25 more
// per column tile).
// Measured, six bf16 products and this (us of the whole product, A X / A^T Q): 100000x50000 l=272 12982 / 13720 and 9315 / 9678;
// 20000x20000 l=110 579 / 534 and 473 / 397, l=64 407 / 386 and 354 / 320; 89083x2783 l=97 346 / 342 and 302 / 273.  (Without the test of every
// row's step, which numbers beside larger ones need, 2 % less.)
template <bool AT, int NT, int NTW, int MT, int WR, int WC>
__device__ __forceinline__ int half_tile(const SplitTile& s, const HalfPanel& panel, uintx4* lds, Noted& notes, int wave, int wr,
                                         int nt0) {
  constexpr int NTH = WR * WC * 64;
  constexpr int BUF = NT * 4 * kFragU;                 // 16-byte units of one staged step
  // units a thread hands over per step, XH of them on their way at a time (the last ones may repeat the end of the buffer)
  constexpr int XU = (BUF + NTH - 1) / NTH, XH = XU <= 3 ? XU : XU == 4 ? 2 : XU <= 6 || XU == 9 ? 3 : 4, XPT = (XU + XH - 1) / XH * XH;
  constexpr int SL = NTW * 6;                          // slots of matrix instructions per step
  // With registers to spare a load of A is issued as soon as its target is split; otherwise all of a step's at its start.
  constexpr bool EARLY = NTW <= kHalfEarly;
  constexpr int SCAN = EARLY ? SL / 2 : SL * 5 / 8;    // the slot before the split of the next step's part of A
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
  const int w0 = s.first + wr * (MT * 16);             // first row (column) of this wave

  unsigned off[AT ? 1 : MT];
  int c0 = 0;
  if constexpr (AT) {
    c0 = max(0, min(w0 + MT * r, s.count - MT));
    off[0] = (unsigned)((4 * g * s.lda + c0) * 4);
  } else {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) off[mt] = (unsigned)(((min(w0 + mt * 16 + r, s.count - 1) - s.first) * s.lda + 4 * g) * 4);
  }
  typedef float vecM __attribute__((ext_vector_type(MT)));
  typedef vecM vecMu __attribute__((aligned(4)));
  typedef floatx4 floatx4u __attribute__((aligned(4)));

  floatx4 acc[MT][NTW], t[2][MT];
  floatx4 ra[MT][4];                                   // Y = A X: [tile][quarter step] four indices of one row
  vecM rq[16];                                         // Z = A^T Q: [index] MT columns of one row of A
  Frag2 fa[MT][2], fb[MT][2];                          // [tile][block of the step]
  uintx4 xr[XH];
  float scale[MT], inv[MT], inv_next[MT];              // of the step being split; of the block sums of a step and of the next
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
    for (int nt = 0; nt < NTW; ++nt) acc[mt][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
  }
  const int b0 = (int)s.b0, K = (int)s.K, empty = (int)empty_block(s.K);
  const int last = s.blocks / 2 - 1, whole_end = whole_steps(s.K) - (int)(s.b0 / 2);
  // (written by an earlier kernel: a scalar load, which does not wait for the loads of A as a vector load would)
  const auto* sw = (const __attribute__((address_space(4))) unsigned*)(panel.words + s.b0);
  auto step_scale = [&](int c) { return ((sw[2 * c] >> 16 & 0xff) - 155u) << 23; };
  auto xid = [&](int x) { return min(tid + x * NTH, BUF - 1); };
  auto block_base = [&](int c, int sub) {
    const int64_t k0 = block_start(b0 + 2 * c + sub, empty, K);
    return (const char*)(s.A + (AT ? k0 * s.lda : k0));
  };
  auto elem = [&](int mt, int q, int i) -> float {     // element i of quarter q of the step
    if constexpr (AT) return rq[4 * q + i][mt];
    else return ra[mt][q][i];
  };
  // the loads that become possible once pairs 0..p of the step have been split
  auto load_a = [&](int p, const char* b0, const char* b1) {
    if constexpr (AT) {
      if (p % MT == MT - 1) {
        const int e0 = 2 * (p / MT);                   // this pair of rows is done in every tile
#pragma unroll
        for (int e = e0; e < e0 + 2; ++e)
          rq[e] = *(const vecMu*)((e < 8 ? b0 : b1) + (int64_t)(((e >> 2) & 1) * 16 + (e & 3)) * s.lda * 4 + off[0]);
      }
    } else {
      const int mt = p >> 3, q = (p >> 1) & 3;
      if (p & 1) ra[mt][q] = *(const floatx4u*)((q < 2 ? b0 : b1) + (q & 1) * 64 + off[mt]);
    }
  };
  auto split_a = [&](int p, Frag2 (&f)[MT][2]) {
    const int mt = AT ? p % MT : p >> 3, pr = AT ? p / MT : p & 7, q = pr >> 1, i = 2 * (pr & 1);   // pair pr of the 16 elements
    half_pair(elem(mt, q, i), elem(mt, q, i + 1), scale[mt], f[mt][q >> 1], pr & 3);
  };
  // The scale of each row (column) for step c; those that fail are left out and noted.
  auto scan = [&](unsigned sx, int c) {
    const bool whole = c < whole_end;
    unsigned rows = 0, most[MT];
    int large = 0;                                     // of all rows' counts, in bytes
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      float run[4];
#pragma unroll
      for (int q = 0; q < 4; ++q)
        run[q] = fmaxf(fmaxf(fabsf(elem(mt, q, 0)), fabsf(elem(mt, q, 1))), fmaxf(fabsf(elem(mt, q, 2)), fabsf(elem(mt, q, 3))));
      large += large_runs(run, whole, most[mt]) << (8 * mt);
    }
    large = sum_groups(large);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const unsigned m = most[mt];
      bool bad = (large >> (8 * mt) & 0xff) < min_runs(whole);
      const unsigned eb = m == 0 ? 127u << 23 : max(m & kExpMask, 15u << 23);
      const int comb = (int)(eb + sx);
      bad |= m != 0 && (unsigned)comb - kExpOne > 253u * kExpOne;
      scale[mt] = bad ? 0.f : __uint_as_float((268u << 23) - eb);
      inv_next[mt] = __int_as_float(max((int)kExpOne, min(comb, (int)(254u << 23))));
      rows |= ((unsigned)__ballot(bad) & 0xffffu) << (16 * mt);            // the same in all groups of lanes
    }
    return rows;
  };
  unsigned own = 0;                                    // rows (columns) that are stored, as bits like those of a note
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int row = AT ? c0 + mt : w0 + mt * 16 + r;
    own |= ((unsigned)__ballot(row < s.count && (!AT || row >= w0 + MT * r)) & 0xffffu) << (16 * mt);
  }
  int noted = 0;                                       // without a branch, see step
  auto note = [&](int c, unsigned rows) {
    rows &= own;
    notes[wave][min(noted, kMaxNoted)] = uint2{(unsigned)c, rows};
    noted += rows != 0;
  };
  const uintx4* xb = panel.panel + s.b0 / 2 * panel.stride;
  {
    const char *p0 = block_base(0, 0), *p1 = block_base(0, 1);
    static_for<0, 8 * MT>([&](auto p) { load_a(p, p0, p1); });
    static_for<0, XPT>([&](auto x) { lds[xid(x)] = xb[xid(x)]; });
    const int c1 = min(1, last);
    static_for<0, XH>([&](auto x) { xr[x] = xb[c1 * panel.stride + xid(x)]; });
    note(0, scan(step_scale(0), 0));
    p0 = block_base(c1, 0);
    p1 = block_base(c1, 1);
    static_for<0, 8 * MT>([&](auto p) { split_a(p, fa); if (EARLY) load_a(p, p0, p1); });
  }
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) inv[mt] = inv_next[mt];
  __syncthreads();

  auto step = [&](int c, const Frag2 (&cf)[MT][2], Frag2 (&nf)[MT][2]) __attribute__((always_inline)) {
    const uintx4* bb = lds + (c & 1) * BUF + nt0 * (4 * kFragU) + lane;
    uintx4* nxt = lds + ((c & 1) ^ 1) * BUF;
    const int c1 = min(c + 1, last), c2 = min(c + 2, last);
    const uintx4 *x1 = xb + c1 * panel.stride, *x2 = xb + c2 * panel.stride;
    const char *p0 = block_base(EARLY ? c2 : c1, 0), *p1 = block_base(EARLY ? c2 : c1, 1);
    const unsigned sx = step_scale(c1);
    uintx4 b[2][2];
#pragma unroll
    for (int p = 0; p < 2; ++p) b[0][p] = bb[p * kFragU];
    static_for<0, SL>([&](auto slot) __attribute__((always_inline)) {
      constexpr int sl = decltype(slot)::value, nt = sl / 6, i = sl % 6;
      constexpr int u2 = sl / 3, sub = u2 & 1, j = sl % 3;               // l*h, h*l, h*h of the first block and of the second
      constexpr int pa = j == 0 ? 1 : 0, px = j == 1 ? 1 : 0;
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        t[nt & 1][mt] = mfma_f16(b[u2 & 1][px], cf[mt][sub].p[pa], i == 0 ? floatx4{0.f, 0.f, 0.f, 0.f} : t[nt & 1][mt]);
      if constexpr (!EARLY) {
        constexpr int n = SL / 6;
        if constexpr (sl < n) {
#pragma unroll
          for (int p = sl * (8 * MT) / n; p < (sl + 1) * (8 * MT) / n; ++p) load_a(p, p0, p1);
        }
      }
      if constexpr (sl == SCAN) {
        // without a branch: one would let the compiler put off what stands before it
        const unsigned rows = scan(sx, c1);
        note(c1, c < last ? rows : 0);
      }
      if constexpr (sl > SCAN) {
        constexpr int u = sl - SCAN - 1, n = SL - SCAN - 1;
#pragma unroll
        for (int p = u * (8 * MT) / n; p < (u + 1) * (8 * MT) / n; ++p) { split_a(p, nf); if (EARLY) load_a(p, p0, p1); }
      }
      // the next step's packed panel goes to LDS in parts, each requested when the one before is handed over
#pragma unroll
      for (int x = sl * XPT / SL; x < (sl + 1) * XPT / SL; ++x) {
        nxt[xid(x)] = xr[x % XH];
        xr[x % XH] = x + XH < XPT ? x1[xid(x + XH)] : x2[xid(x + XH - XPT)];
      }
      // the previous tile's block sum
      if constexpr (nt > 0) {
#pragma unroll
        for (int e = i * (4 * MT) / 6; e < (i + 1) * (4 * MT) / 6; ++e)
          acc[e >> 2][nt - 1][e & 3] = fmaf(t[(nt + 1) & 1][e >> 2][e & 3], inv[e >> 2], acc[e >> 2][nt - 1][e & 3]);
      }
      if constexpr (u2 + 1 < 2 * NTW && j < 2) b[(u2 + 1) & 1][j] = bb[((u2 + 1) * 2 + j) * kFragU];
    });
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[mt][NTW - 1][v] = fmaf(t[(NTW - 1) & 1][mt][v], inv[mt], acc[mt][NTW - 1][v]);
      inv[mt] = inv_next[mt];
    }
  };
  int c = 0;
#pragma nounroll
  for (; c < last; c += 2) {
    step(c, fa, fb);
    step(c + 1, fb, fa);
  }
  if (c == last) step(c, fa, fb);
  if (noted > kMaxNoted) return kRedo;
  int left_out = 0;
  for (int i = 0; i < noted; ++i) left_out += __popc(notes[wave][i].y);
  if (left_out > kMaxRows) return kRedo;

  // lane (r, g) holds columns 4g..4g+3 of every tile of the panel, for row (column of A) r
  float worst = 0.f;                                   // NaN as soon as one result is not finite
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int row = AT ? c0 + mt : w0 + mt * 16 + r;
    const bool valid = own >> (16 * mt + r) & 1;         // (a column belongs to the lane that has it first)
    if (valid) {
      float* o = s.out + (int64_t)row * s.ldo;
#pragma unroll
      for (int nt = 0; nt < NTW; ++nt) {
        const int col = (nt0 + nt) * 16 + 4 * g;
        const floatx4 y = acc[mt][nt];
        if (col + 4 <= s.ncols) {
          *(floatx4u*)(o + col) = y;
          worst += (y[0] * 0.f + y[1] * 0.f) + (y[2] * 0.f + y[3] * 0.f);
        } else {
#pragma unroll
          for (int v = 0; v < 4; ++v)
            if (col + v < s.ncols) { o[col + v] = y[v]; worst += y[v] * 0.f; }
        }
      }
    }
  }
  // What was left out: a row's 64 numbers in the lanes, the panel's columns across them.
  if (left_out > 0) {
    __threadfence_block();                             // other lanes have stored what is added to
    for (int i = 0; i < noted; ++i) {
      const int c = __builtin_amdgcn_readfirstlane(notes[wave][i].x);
      const int64_t k0 = block_index(s.b0 + 2 * c, s.K) * kSplitB;
      const int n = (int)(min(s.K, block_index(s.b0 + 2 * c + 2, s.K) * kSplitB) - k0);
      for (unsigned rows = __builtin_amdgcn_readfirstlane(notes[wave][i].y); rows; rows &= rows - 1) {
        const int mt = (__ffs(rows) - 1) / 16, rr = (__ffs(rows) - 1) % 16;
        const int row = AT ? max(0, min(w0 + MT * rr, s.count - MT)) + mt : w0 + mt * 16 + rr;
        const int64_t k = k0 + min(lane, n - 1);
        const float own = AT ? s.A[k * s.lda + row] : s.A[(row - s.first) * s.lda + k];
        const int a = __float_as_int(lane < n ? own : 0.f);
        for (int j = 0; j < NTW * 16; j += 64) {         // (all lanes: v_readlane reads those beyond the last column too)
          const int col = nt0 * 16 + j + lane, xcol = min(panel.c0 + col, panel.cols - 1);
          const float* p = panel.X + k0 * panel.ld + xcol;
          float sum[4] = {0.f, 0.f, 0.f, 0.f};
          for (int k = 0; k < n; k += 16) {
            float v[16];
#pragma unroll
            for (int e = 0; e < 16; ++e) v[e] = p[min(k + e, n - 1) * panel.ld];
#pragma unroll
            for (int e = 0; e < 16; ++e) sum[e & 3] = fmaf(__int_as_float(__builtin_amdgcn_readlane(a, k + e)), v[e], sum[e & 3]);
          }
          if (j + lane < NTW * 16 && col < s.ncols && panel.c0 + col < panel.cols) s.out[(int64_t)row * s.ldo + col] += (sum[0] + sum[1]) + (sum[2] + sum[3]);
        }
      }
    }
  }
  return !(worst == 0.f) ? kNotFinite : 0;
}

template <bool AT, int NT, int MT, int WR, int WC>
__device__ __forceinline__ int half_tile_waves(const SplitTile& s, const HalfPanel& panel, uintx4* lds, Noted& notes) {
  constexpr int NTW = (NT + WC - 1) / WC;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = wave % WR, wc = wave / WR;
  if constexpr (NT % WC == 0) {
    return half_tile<AT, NT, NTW, MT, WR, WC>(s, panel, lds, notes, wave, wr, wc * NTW);
  } else {
    if (wc == 0) return half_tile<AT, NT, NTW, MT, WR, WC>(s, panel, lds, notes, wave, wr, 0);
    return half_tile<AT, NT, NTW - 1, MT, WR, WC>(s, panel, lds, notes, wave, wr, NTW);
  }
}

// Whether a step of the panel or of the sampled rows is not fit for this product: then all workgroups leave their parts, and pack the panel in bf16 numbers in
// the place of these before they go.  (All threads.)
__device__ __forceinline__ bool half_leave(const HalfPanel& x, int64_t K, int wg, int wgs) {
  int bad = 0;
  for (int64_t i = threadIdx.x; i < x.steps; i += blockDim.x) bad |= x.words[2 * i] >> 16 & kUntame;
  if (!__syncthreads_or(bad)) return false;
  const int64_t fragments = 2 * x.steps * x.nt_total, waves = blockDim.x >> 6;
  for (int64_t i = wg * waves + (threadIdx.x >> 6); i < fragments; i += wgs * waves) {
    const int64_t blk = i / x.nt_total;
    split_pack_fragment(x.X, K, x.ld, x.cols, blk, (int)(i - blk * x.nt_total), x.all + i * (3 * kFragU));
  }
  if (threadIdx.x == 0) x.redo[wg] = kRedoPacked;
  return true;
}

// Y = A X and partial panel blockIdx.y of Z = A^T Q: the parts of the workgroups of k_split_an and k_split_at.
template <int NT, int MT, int WR, int WC>
__global__ void __launch_bounds__(WR * WC * 64)
k_half_an(const float* __restrict__ A, int64_t lda, int rows, int K, HalfPanel x, float* __restrict__ Y, int64_t ldy, int ncols,
          float* __restrict__ Part, int64_t ldp, int64_t split_stride, AnShape sh) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  __shared__ Noted notes;
  constexpr int TR = WR * MT * 16;
  const AnWork w = an_work(sh, blockIdx.x);
  if (half_leave(x, K, blockIdx.x, gridDim.x)) return;
  for (int seg = 0; seg < w.nseg; ++seg) {
    SplitTile s;
    s.first = (w.first_tile + seg) * TR;
    s.A = A + (int64_t)s.first * lda;
    s.lda = lda;
    s.K = K;
    s.b0 = 2 * (int64_t)w.c0;
    s.blocks = 2 * (w.c1 - w.c0);
    s.count = rows;
    s.out = w.partial ? Part + (int64_t)w.slot * split_stride - (int64_t)sh.whole * TR * ldp : Y;
    s.ldo = w.partial ? ldp : ldy;
    s.ncols = w.partial ? NT * 16 : ncols;
    const int found = half_tile_waves<false, NT, MT, WR, WC>(s, x, (uintx4*)lds_raw, notes);
    if (found & kNotFinite) x.flags[blockIdx.x % kSplitFlags] = 1;
    if (found & kRedo) x.redo[blockIdx.x] = kRedoRaw;
    __syncthreads();                                   // before the next strip reuses the staging buffers
  }
}

template <int NT, int MT, int WR, int WC>
__global__ void __launch_bounds__(WR * WC * 64)
k_half_at(const float* __restrict__ A, int64_t lda, int64_t rows, int n, HalfPanel x, float* __restrict__ Zpart, int64_t ldz,
          int64_t split_stride, int blocks, int blocks_per_sub) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  __shared__ Noted notes;
  SplitTile s;
  s.A = A;
  s.lda = lda;
  s.K = rows;
  s.b0 = (int64_t)blockIdx.y * blocks_per_sub;
  s.blocks = min(blocks_per_sub, blocks - (int)s.b0);
  s.first = blockIdx.x * (WR * MT * 16);
  s.count = n;
  s.out = Zpart + (int64_t)blockIdx.y * split_stride;
  s.ldo = ldz;
  s.ncols = NT * 16;
  const int wg = blockIdx.y * gridDim.x + blockIdx.x;
  if (half_leave(x, rows, wg, gridDim.x * gridDim.y)) return;
  const int found = half_tile_waves<true, NT, MT, WR, WC>(s, x, (uintx4*)lds_raw, notes);
  if (found & kNotFinite) x.flags[wg % kSplitFlags] = 1;
  if (found & kRedo) x.redo[wg] = kRedoRaw;
}

// ---- host side --------------------------------------------------------------------------------------------------
#define BRSVD_HALF_SWITCH(nt, tile, CALL)                                                                        \
  if (nt == 10 && tile == 4 * kSplitMT * 16) { CALL(10, 4, 2); } else                                            \
  switch (nt) {                                                                                                  \
    case 2: CALL(2, 8, 1); break; case 3: CALL(3, 8, 1); break; case 4: CALL(4, 8, 1); break; case 5: CALL(5, 8, 1); break;                    \
    case 6: CALL(6, 8, 1); break; case 7: CALL(7, 8, 1); break; case 8: CALL(8, 8, 1); break;                    \
    case 9: CALL(9, 8, 1); break; case 10: CALL(10, 8, 1); break; case 11: CALL(11, 4, 2); break;                \
    case 12: CALL(12, 4, 2); break; case 13: CALL(13, 4, 2); break; case 14: CALL(14, 4, 2); break;              \
    case 15: CALL(15, 4, 2); break; case 16: CALL(16, 4, 2); break; case 17: CALL(17, 4, 2); break;              \
    default: return BRSVD_ERR_ARG;                                                                               \
  }

template <typename K>
static int half_lds(K kern, int nt, bool* done) {
  if (!*done) {
    BRSVD_HIP_TRY(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 2 * nt * 4 * kFragU * 16));
    *done = true;
  }
  return BRSVD_OK;
}

int half_pack(const float* A, int64_t lda, int64_t count, int64_t K, int Lp, bool at, const HalfPacked& x, hipStream_t stream) {
  const int nt = Lp / 16;                                 // at most kMaxL / 16 = 32: two tiles for each of 16 waves
  const dim3 grid((unsigned)split_chunks(K));
  if (nt <= 16)
    hipLaunchKernelGGL(k_half_pack<1>, grid, dim3(64 * nt), 0, stream, x.X, K, x.ldx, x.xcols, nt, (uintx4*)x.panel, x.words, x.flags,
                       x.nflags, A, lda, count, (int)at);
  else
    hipLaunchKernelGGL(k_half_pack<2>, grid, dim3(64 * ((nt + 1) / 2)), 0, stream, x.X, K, x.ldx, x.xcols, nt, (uintx4*)x.panel, x.words,
                       x.flags, x.nflags, A, lda, count, (int)at);
  BRSVD_HIP_TRY(hipGetLastError());
  return BRSVD_OK;
}

// The column tiles from c0 / 16 on.
static HalfPanel half_panel(const HalfPacked& x, int64_t K, int Lp, int c0) {
  return HalfPanel{(const uintx4*)x.panel + (c0 / 16) * 4 * kFragU, (int64_t)(Lp / 16) * 4 * kFragU, x.words, x.flags, x.redo, c0,
                   (uintx4*)x.panel, x.X, x.ldx, split_chunks(K), x.xcols, Lp / 16};
}

int half_an(const float* A, int64_t lda, int64_t rows, int64_t K, const HalfPacked& x, int Lp, int c0, int nt, int tile, float* Y,
            int64_t ldy, int ncols, float* part, int64_t stride, const AnShape& sh, int wgs, hipStream_t stream) {
#define CALL(N, WR, WC)                                                                                              \
  {                                                                                                                  \
    if (tile != WR * kSplitMT * 16) return BRSVD_ERR_ARG;                                                            \
    auto kern = k_half_an<N, kSplitMT, WR, WC>;                                                                      \
    static bool done = false;                                                                                        \
    BRSVD_TRY(half_lds(kern, N, &done));                                                                             \
    hipLaunchKernelGGL(kern, dim3(wgs), dim3(WR * WC * 64), 2 * N * 4 * kFragU * 16, stream, A, lda, (int)rows, (int)K, \
                       half_panel(x, K, Lp, c0), Y, ldy, ncols, part, (int64_t)Lp, stride, sh);                      \
  }
  BRSVD_HALF_SWITCH(nt, tile, CALL)
#undef CALL
  BRSVD_HIP_TRY(hipGetLastError());
  return BRSVD_OK;
}

int half_at(const float* A, int64_t lda, int64_t rows, int64_t n, const HalfPacked& x, int Lp, int c0, int nt, int tile,
            float* part, int64_t stride, int col_tiles, int nsplit, int blocks, int blocks_per_sub, hipStream_t stream) {
#define CALL(N, WR, WC)                                                                                              \
  {                                                                                                                  \
    if (tile != WR * kSplitMT * 16) return BRSVD_ERR_ARG;                                                            \
    auto kern = k_half_at<N, kSplitMT, WR, WC>;                                                                      \
    static bool done = false;                                                                                        \
    BRSVD_TRY(half_lds(kern, N, &done));                                                                             \
    hipLaunchKernelGGL(kern, dim3(col_tiles, nsplit), dim3(WR * WC * 64), 2 * N * 4 * kFragU * 16, stream, A, lda, rows, (int)n, \
                       half_panel(x, rows, Lp, c0), part, (int64_t)Lp, stride, blocks, blocks_per_sub);              \
  }
  BRSVD_HALF_SWITCH(nt, tile, CALL)
#undef CALL
  BRSVD_HIP_TRY(hipGetLastError());
  return BRSVD_OK;
}

}  // namespace brsvd
