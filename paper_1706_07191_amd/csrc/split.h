// Shared by the two families of products with split operands: gemm_split.hip (three bf16 numbers) and gemm_half.hip (two scaled
// fp16 numbers).  Both cut the work alike, so that one can take over a workgroup's part from the other.
#pragma once
#include <algorithm>

#include "common.h"

namespace brsvd {

typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

constexpr int kSplitB = 32;          // contraction indices per block
constexpr int kFragU = 64;           // 16-byte units of one operand fragment (16 x 32 numbers of 16 bits)
// Flags of the workgroups that met a result that is not finite, and behind them of those that met a row (Z = A^T Q: a column) of
// A with small elements only.  A workgroup beyond the last one shares a flag with an earlier one; where the other raised it,
// its own results are only looked at in vain.  (What a workgroup left undone in gemm_half.hip is a word of its own.)
constexpr int kSplitFlags = 4096;
constexpr int kNotFinite = 1, kSmall = 2, kRedo = 4;

// Blocks are taken in twos.  Where their number is odd an empty one stands before the last two, so that the first of any two is whole.
// Block `blk` covers the contraction indices from block_first on (K for the empty one).  It is read from block_start on: the last one is
// moved back so that it ends with the range, and the indices the block before has already covered are zero in the packed panel.
// Neither operand is then ever read outside its range, and A needs no masks.  K >= 3 * kSplitB.
__host__ __device__ inline int64_t empty_block(int64_t K) {
  const int64_t n = (K + kSplitB - 1) / kSplitB;
  return n & 1 ? n - 2 : n;
}
__host__ __device__ inline int64_t block_index(int64_t blk, int64_t K) { return blk > empty_block(K) ? blk - 1 : blk; }
__host__ __device__ inline int64_t block_first(int64_t blk, int64_t K) { return blk == empty_block(K) ? K : block_index(blk, K) * kSplitB; }
__host__ __device__ inline int64_t block_start(int64_t blk, int64_t K) {
  const int64_t k = block_index(blk, K) * kSplitB;
  return k < K - kSplitB ? k : K - kSplitB;
}
// The same in 32 bits (split_fits), which is all that scalar instructions compare: in 64 the addresses take vector registers.
__host__ __device__ inline int block_start(int blk, int empty, int K) {
  const int k = (blk - (blk > empty ? 1 : 0)) * kSplitB;
  return k < K - kSplitB ? k : K - kSplitB;
}
// The twos of blocks before those that may have less than 64 indices.
__host__ __device__ inline int whole_steps(int64_t K) {
  const int n = (int)((K + kSplitB - 1) / kSplitB);
  return n & 1 ? (n - 3) / 2 : (int)(K / (2 * kSplitB));
}

template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// Elements from 2^-95 on have one of these exponent bits set.  They are split without loss, and their parts times anything of
// ordinary size stay clear of the subnormal numbers; the third part of an element below 2^-110 would not fit bf16 (2^-133).
constexpr unsigned kWholeBits = 0x70000000u;

struct Frag3 { uintx4 p[3]; };       // h, m, l of eight contraction indices

__device__ __forceinline__ unsigned pack_bf16(float a, float b) {
  return __builtin_bit_cast(unsigned, __builtin_convertvector(floatx2{a, b}, bf16x2));
}
// Pair q (elements 2q, 2q + 1) of a fragment.
__device__ __forceinline__ void split_pair(float a, float b, Frag3& f, int q) {
  const unsigned ua = __float_as_uint(a), ub = __float_as_uint(b);
  f.p[0][q] = __builtin_amdgcn_perm(ub, ua, 0x07060302u);              // the two upper halves
  float ra = a - __uint_as_float(ua & 0xffff0000u), rb = b - __uint_as_float(ub & 0xffff0000u);
  const unsigned m = pack_bf16(ra, rb);
  f.p[1][q] = m;
  ra -= __uint_as_float(m << 16);
  rb -= __uint_as_float(m & 0xffff0000u);
  f.p[2][q] = pack_bf16(ra, rb);
}

// Splits eight entries of one column; a column with small elements only in the block is made NaN (whole waves).
__device__ __forceinline__ Frag3 split_panel_fragment(const float (&v)[8]) {
  Frag3 f;
  unsigned bits = 0;
#pragma unroll
  for (int e = 0; e < 8; ++e) bits |= __float_as_uint(v[e]);
#pragma unroll
  for (int q = 0; q < 4; ++q) split_pair(v[2 * q], v[2 * q + 1], f, q);
  bits |= __shfl_xor(bits, 16, 64);
  bits |= __shfl_xor(bits, 32, 64);
  if (!(bits & kWholeBits) && (bits & 0x7fffffffu)) f.p[0][0] = 0x7fc07fc0u;
  return f;
}
// Packed panel: [block][column tile][h, m, l][lane][8 bf16], i.e. 3 KiB per block and tile of 16 columns; an even number of
// blocks.  src: K x cols, leading dimension ld; columns cols.. are zero.  One fragment by one wave; returns the columns with a NaN.
__device__ __forceinline__ unsigned split_pack_fragment(const float* __restrict__ src, int64_t K, int64_t ld, int cols, int64_t blk, int nt,
                                                        uintx4* __restrict__ o) {
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4, col = 16 * nt + r;
  const int64_t k0 = block_start(blk, K);
  float v[8];
  bool any_nan = false;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int64_t k = k0 + (e >> 2) * 16 + 4 * g + (e & 3);
    v[e] = k >= block_first(blk, K) && col < cols ? src[k * ld + col] : 0.f;
    any_nan |= v[e] != v[e];
  }
  const unsigned long long b = __ballot(any_nan);                      // bit 16 * g + r
  const Frag3 f = split_panel_fragment(v);
#pragma unroll
  for (int p = 0; p < 3; ++p) o[p * kFragU + lane] = f.p[p];
  return (unsigned)(b | b >> 16 | b >> 32 | b >> 48) & 0xffffu;
}

// What one workgroup multiplies: `blocks` blocks (even) of the contraction from block `b0` on, and where its result goes.
struct SplitTile {
  const float* A;        // Y = A X: first row of the tile;  Z = A^T Q: first row of A
  int64_t lda;
  int64_t K;             // length of the contraction
  int64_t b0;
  int blocks;
  int first, count;      // first row (column) of the tile and how many rows (columns) the output has in all
  float* out;            // row `first` of the output is out + first * ldo
  int64_t ldo;
  int ncols;
  int* whole;            // set for the rows (columns) with an element that is split without loss
};

// ---- host side --------------------------------------------------------------------------------------------------
struct SplitCfg { int wr, wc, tile; };
constexpr int kSplitMT = 2;
// Up to ten column tiles one wave holds them all (accumulators of 2 x 10 tiles); wider panels take two columns of waves, i.e. half as many
// rows per workgroup.  Registers: three bf16 numbers take all 256 for A X from 9 tiles on and 36 to 212 bytes a lane of scratch (none with
// 12 tiles), for A^T Q up to 228 and 88 bytes with 15 and 17 tiles; two fp16 ones all for A X from 9 tiles on and 8 to 88 bytes with 13 to
// 17, for A^T Q up to 245 and none.
static SplitCfg split_cfg(int nt) {
  return nt <= 10 ? SplitCfg{8, 1, 8 * kSplitMT * 16} : SplitCfg{4, 2, 4 * kSplitMT * 16};
}
constexpr int kSplitSlots = 256;                        // one workgroup of eight waves per CU
static int64_t split_chunks(int64_t K) { return ceil_div(K, 2 * kSplitB); }
// The packed panel, behind it the words that say which columns have a NaN, and the flags of the product's workgroups and of the
// `out` rows (columns) of A.
struct PackLayout {
  uint64_t nan, flags, whole, bytes;
};
static PackLayout pack_layout(int64_t out, int64_t K, int Lp) {
  const uint64_t tiles = (uint64_t)split_chunks(K) * 2 * (Lp / 16);
  PackLayout o;
  o.nan = tiles * 3 * kFragU * 16;
  o.flags = o.nan + tiles * 4;
  o.whole = o.flags + 2 * kSplitFlags * 4;
  o.bytes = o.whole + (uint64_t)out * 4;
  return o;
}

// ---- gemm_half.hip ----
// words: those of k_split_pack (which columns of a fragment have a NaN), whose upper halves hold the scale of each step of 64 indices in
// the first column tile's.  redo: what a workgroup left undone (nothing, kRedoRaw or kRedoPacked).
constexpr int kRedoRaw = 1, kRedoPacked = 2;
struct HalfPacked {
  void* panel;
  unsigned* words;
  int *flags, *redo;
  int64_t nflags;          // words of both
  const float* X;
  int64_t ldx;
  int xcols;
};
// Packs X (K indices) and clears the flags; A (its `count` rows or columns of the output) is sampled.
int half_pack(const float* A, int64_t lda, int64_t count, int64_t K, int Lp, bool at, const HalfPacked& x, hipStream_t stream);
// Column tiles [c0 / 16, c0 / 16 + nt) of the panel; Y, part and ncols are those of column c0.
int half_an(const float* A, int64_t lda, int64_t rows, int64_t K, const HalfPacked& x, int Lp, int c0, int nt, int tile, float* Y,
            int64_t ldy, int ncols, float* part, int64_t stride, const AnShape& sh, int wgs, hipStream_t stream);
int half_at(const float* A, int64_t lda, int64_t rows, int64_t n, const HalfPacked& x, int Lp, int c0, int nt, int tile,
            float* part, int64_t stride, int col_tiles, int nsplit, int blocks, int blocks_per_sub, hipStream_t stream);

}  // namespace brsvd
