// The two thin products of gemm_thin.hip for wide fp32 panels over large A (more than 32 columns, and 17 to 32 where it pays; the rule
// and what it was measured on: common.h) on the bf16 matrix cores -- the shorter contractions, and what gemm_half.hip leaves of the
// longer ones -- with every fp32 operand split exactly into three bf16 numbers:
//
//   a = h + m + l,   h = the upper 16 bits of a (8 significant bits), m = bf16(a - h), l = a - h - m
//
// (24 significant bits = 8 + 8 + 8, so nothing of a is lost from 2^-110 on; l of a smaller number would have bits below 2^-133,
// where bf16 ends.  Rows of A or columns of a panel with no larger element are multiplied in fp32 after all: k_split_repair_an.)
// Of the nine products of two such sums the six above 2^-24 are taken, l*h + h*l + m*m + m*h + h*m + h*h: six
// v_mfma_f32_16x16x32_bf16 do the work of eight v_mfma_f32_16x16x4_f32 in 96 cycles instead of 256.  The dropped products are
// below 2^-22 of |a||x| at most and 2^-26 on average, and random in sign.
//
// Accuracy.  The bf16 instruction truncates its sum to fp32 instead of rounding it, which over a long contraction
// would add up to a bias (K = 20000, entries N(0.5, 1): 5e-6, against 2.2e-6 for the fp32 instruction).  So the six
// products of one block of 32 contraction indices are added into a register tile that starts from zero, smallest
// products first -- only the last one can truncate anything that matters -- and that tile is added to the
// running sum by rounded fp32 additions.  That makes K/32 additions where the fp32 instruction makes K/4 or more:
// measured error against fp64, this kernel and the fp32 instruction: K = 112 6.1e-8 and 1.9e-7, K = 1000 1.2e-7
// and 5.5e-7, K = 20000 4.7e-7 and 2.5e-6 (N(0,1) entries); K = 20000, N(0.5,1): 3.8e-7 and 2.2e-6.  Where a sum has few terms
// there are no additions to save, and the truncation shows: one entry in a row of A 4.1e-8 and 2.5e-8 (the rounding of a
// single product), one in a hundred (K = 1000 and 4000) 7.1e-8 and 5.4e-8, 9.9e-8 and 7.3e-8.
//
// Both products are one kernel.  The contraction runs over blocks of 32 (columns of A for Y = A X, rows of A for
// Z = A^T Q); the right panel is split once per call into the operand layout of the instruction (k_split_pack), A is
// split in registers on its way into the matrix cores:
//   operands: lane = 16*g + r holds eight contraction indices 4*g + {0..3}, 16 + 4*g + {0..3} of the block (any
//   assignment is allowed as long as both operands share it), for row / column r; D: component v of lane (r, g) is
//   entry [4*g + v][r].
#include "split.h"

namespace brsvd {

__device__ __forceinline__ floatx4 mfma_bf16(uintx4 a, uintx4 b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
// bits |= a | b in one instruction: as plain code the compiler puts it off and keeps a and b in registers (20 more, and spills).
__device__ __forceinline__ void or3(unsigned& bits, float a, float b) {
  asm("v_or3_b32 %0, %0, %1, %2" : "+v"(bits) : "v"(a), "v"(b));
}

struct PackedPanel {                  // written by k_split_pack; panel points to the first column tile
  static constexpr int kUnits = 1;    // 16-byte units a thread hands over at a time
  typedef uintx4 Unit;
  const uintx4* panel;
  int64_t stride;                     // 16-byte units of one block
  template <int NT>
  __device__ __forceinline__ void load(Unit& u, int id, int64_t blk, int64_t) const {
    u = panel[blk * stride + min(id, NT * 3 * kFragU - 1)];
  }
  template <int NT>
  __device__ __forceinline__ void store(const Unit& u, int id, int64_t, int64_t, uintx4* buf) const {
    buf[min(id, NT * 3 * kFragU - 1)] = u;
  }
};
// nan: [column tile][block], a bit for each column with a NaN.  Also clears the flags of the product's workgroups and of the rows of A.
// Where a column has small elements only in a block, its part of the panel is made NaN, so that its results are taken from the repair.
__global__ void __launch_bounds__(256)
k_split_pack(const float* __restrict__ src, int64_t K, int64_t ld, int cols, int nt_total, int64_t blocks,
             uintx4* __restrict__ out, unsigned* __restrict__ nan, int* __restrict__ flags, int64_t nflags) {
  const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
  for (int64_t i = id; i < nflags; i += (int64_t)gridDim.x * 256) flags[i] = 0;
  const int64_t tile = id >> 6, blk = tile / nt_total;
  if (blk >= blocks) return;
  const int nt = (int)(tile - blk * nt_total);
  const unsigned b = split_pack_fragment(src, K, ld, cols, blk, nt, out + tile * (3 * kFragU));
  if ((threadIdx.x & 63) == 0) nan[nt * blocks + blk] = b;
}
struct RawPanel {
  static constexpr int kUnits = 3;
  struct Unit { float v[8]; };
  const float* X;
  int64_t ld;
  int cols;
  template <int NT>
  __device__ __forceinline__ void load(Unit& u, int id, int64_t blk, int64_t K) const {
    const int lane = id & 63, nt = min(id >> 6, NT - 1);
    const float* p = X + block_start(blk, K) * ld + min(16 * nt + (lane & 15), cols - 1);
#pragma unroll
    for (int e = 0; e < 8; ++e) u.v[e] = p[((e >> 2) * 16 + 4 * (lane >> 4) + (e & 3)) * ld];
  }
  template <int NT>
  __device__ __forceinline__ void store(const Unit& u, int id, int64_t blk, int64_t K, uintx4* buf) const {
    const int lane = id & 63, nt = min(id >> 6, NT - 1);
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int64_t k = block_start(blk, K) + (e >> 2) * 16 + 4 * (lane >> 4) + (e & 3);
      v[e] = k >= block_first(blk, K) && 16 * nt + (lane & 15) < cols ? u.v[e] : 0.f;
    }
    const Frag3 f = split_panel_fragment(v);
#pragma unroll
    for (int p = 0; p < 3; ++p) buf[(nt * 3 + p) * kFragU + lane] = f.p[p];
  }
};

// Workgroup: WR x WC waves; wave (wr, wc) owns MT tiles of 16 rows (AT: columns of A) and NTW tiles of the panel's
// columns.  Wave column 0 owns the first NTW tiles, wave column 1 the rest; the waves of one SIMD are one of each.
//
// What bounds it: the matrix cores and the power they may draw (16 cycles per instruction, 204 of them per
// 32 x 32 x 272 block step; the clock falls to 1.7-1.9 GHz under full load), so everything else is spread over the
// stream of matrix instructions in small portions between scheduling barriers: the reads of the next tile's panel
// fragments from LDS, the addition of the previous tile's block sum, the split of the next block's part of A with
// the loads of the block after that, and the hand-over of the next block's packed panel from registers to LDS.  One barrier
// per block.  A first version that did these things between the blocks ran at 75-85 % of this one.
//
// Panel: a packed one (PackedPanel), or the panel as it is (RawPanel: its part of a block is split on its way to LDS).
template <bool AT, int NT, int NTW, int MT, int WR, int WC, typename Panel>
__device__ __forceinline__ int split_tile(const SplitTile& s, const Panel& panel, uintx4* lds, int wr, int nt0) {
  constexpr int NTH = WR * WC * 64;
  constexpr int BUF = NT * 3 * kFragU;                 // 16-byte units of one staged block
  constexpr int XPT = (BUF / Panel::kUnits + NTH - 1) / NTH;
  constexpr int SL = NTW * 6;                          // slots of matrix instructions per block
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
  const int w0 = s.first + wr * (MT * 16);             // first row (column) of this wave

  // Byte offsets of this lane's loads from a uniform base (below 2^32: see split_fits).  Rows past the end repeat the last one, columns past the end the
  // last MT; their results are not stored.
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

  floatx4 acc[MT][NTW], t[2][MT], tl[MT];
  floatx4 ra[MT][2];                                   // Y = A X: [tile][half block] four indices of one row
  vecM rq[8];                                          // Z = A^T Q: [index] MT columns of one row of A
  Frag3 fa[MT], fb[MT];
  typename Panel::Unit xr[XPT];
  unsigned bits[MT];                                   // of all elements of A this lane has split, by row (AT: column)
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    tl[mt] = floatx4{0.f, 0.f, 0.f, 0.f};
    bits[mt] = 0;
#pragma unroll
    for (int nt = 0; nt < NTW; ++nt) acc[mt][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
  }
  const int last = s.blocks - 1, b0 = (int)s.b0, K = (int)s.K, empty = (int)empty_block(s.K);
  auto load_x = [&](int x, int c) { panel.template load<NT>(xr[x], tid + x * NTH, s.b0 + c, s.K); };
  auto store_x = [&](int x, int c, uintx4* buf) { panel.template store<NT>(xr[x], tid + x * NTH, s.b0 + c, s.K, buf); };
  // base of block c: A + k0 (row part of the address is in off) or A + k0 * lda
  auto block_base = [&](int c) {
    const int64_t k0 = block_start(b0 + c, empty, K);
    return (const char*)(s.A + (AT ? k0 * s.lda : k0));
  };
  // the loads that become possible once pairs 0..p of the block have been split
  auto load_a = [&](int p, const char* base) {
    if constexpr (AT) {
      if (p % MT == MT - 1) {
        const int q = p / MT;                          // pair q of every tile is done: rows 2q, 2q + 1 are free
#pragma unroll
        for (int e = 2 * q; e < 2 * q + 2; ++e)
          rq[e] = *(const vecMu*)(base + (int64_t)((e >> 2) * 16 + (e & 3)) * s.lda * 4 + off[0]);
      }
    } else {
      if (p & 1) ra[p >> 2][(p >> 1) & 1] = *(const floatx4u*)(base + ((p >> 1) & 1) * 64 + off[p >> 2]);
    }
  };
  auto split_a = [&](int p, Frag3 (&f)[MT]) {
    if constexpr (AT) {
      const int q = p / MT, mt = p % MT;
      split_pair(rq[2 * q][mt], rq[2 * q + 1][mt], f[mt], q);
      or3(bits[mt], rq[2 * q][mt], rq[2 * q + 1][mt]);
    } else {
      const int mt = p >> 2, q = p & 3;
      split_pair(ra[mt][q >> 1][2 * (q & 1)], ra[mt][q >> 1][2 * (q & 1) + 1], f[mt], q);
      or3(bits[mt], ra[mt][q >> 1][2 * (q & 1)], ra[mt][q >> 1][2 * (q & 1) + 1]);
    }
  };

  {
    const char* base = block_base(0);
    static_for<0, XPT>([&](auto x) { load_x(x, 0); });
    static_for<0, 4 * MT>([&](auto p) { load_a(p, base); });
    static_for<0, XPT>([&](auto x) { store_x(x, 0, lds); load_x(x, 1); });
    base = block_base(1);
    static_for<0, 4 * MT>([&](auto p) { split_a(p, fa); load_a(p, base); });
  }
  __syncthreads();

  auto block = [&](int c, const Frag3 (&cf)[MT], Frag3 (&nf)[MT]) __attribute__((always_inline)) {
    const uintx4* bb = lds + (c & 1) * BUF + nt0 * (3 * kFragU) + lane;
    uintx4* nxt = lds + ((c & 1) ^ 1) * BUF;
    const int c2 = min(c + 2, last);
    const char* base2 = block_base(c2);
    uintx4 b[2][3];
#pragma unroll
    for (int p = 0; p < 3; ++p) b[0][p] = bb[p * kFragU];
    static_for<0, SL>([&](auto slot) __attribute__((always_inline)) {
      constexpr int sl = decltype(slot)::value, nt = sl / 6, i = sl % 6;
      constexpr int pa = i == 0 ? 2 : (i == 2 || i == 3 ? 1 : 0);        // l m h of A: l*h, h*l, m*m, m*h, h*m, h*h
      constexpr int pb = i == 1 ? 2 : (i == 2 || i == 4 ? 1 : 0);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        t[nt & 1][mt] = mfma_bf16(cf[mt].p[pa], b[nt & 1][pb], i == 0 ? floatx4{0.f, 0.f, 0.f, 0.f} : t[nt & 1][mt]);
      // split of the next block's part of A, and the loads of the block after it into the freed registers
#pragma unroll
      for (int p = sl * (4 * MT) / SL; p < (sl + 1) * (4 * MT) / SL; ++p) { split_a(p, nf); load_a(p, base2); }
      // the next block's packed panel goes to LDS, the one after it is requested
#pragma unroll
      for (int x = sl * XPT / SL; x < (sl + 1) * XPT / SL; ++x) { store_x(x, min(c + 1, last), nxt); load_x(x, c2); }
      // the previous tile's block sum
      constexpr int pv = (nt + NTW - 1) % NTW;
#pragma unroll
      for (int e = i * (4 * MT) / 6; e < (i + 1) * (4 * MT) / 6; ++e)
        acc[e >> 2][pv][e & 3] += nt == 0 ? tl[e >> 2][e & 3] : t[(nt + 1) & 1][e >> 2][e & 3];
      if constexpr (nt + 1 < NTW && i < 3) b[(nt + 1) & 1][i] = bb[((nt + 1) * 3 + i) * kFragU];
    });
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) tl[mt] = t[(NTW - 1) & 1][mt];
    __syncthreads();
  };
#pragma nounroll
  for (int c = 0; c < s.blocks; c += 2) {
    block(c, fa, fb);
    block(c + 1, fb, fa);
  }
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) acc[mt][NTW - 1] += tl[mt];

  float worst = 0.f;                                   // NaN as soon as one result is not finite
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = 4 * g + v;
      // row i of tile mt is the mt-th of the MT columns lane i loaded (AT; a column belongs to the lane that has it first), or row 16 * mt + i
      const int row = AT ? max(0, min(w0 + MT * i, s.count - MT)) + mt : w0 + mt * 16 + i;
      const bool valid = row < s.count && (!AT || row >= w0 + MT * i);
      if (valid) {
        float* o = s.out + (int64_t)row * s.ldo;
#pragma unroll
        for (int nt = 0; nt < NTW; ++nt) {
          const int col = (nt0 + nt) * 16 + r;
          const float y = acc[mt][nt][v];
          if (col < s.ncols) { o[col] = y; worst += y * 0.f; }
        }
      }
    }
  // rows with an element that is split whole, and whether one has only smaller ones
  int found = !(worst == 0.f) ? kNotFinite : 0;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    unsigned b = bits[mt] | __shfl_xor(bits[mt], 16, 64);
    b |= __shfl_xor(b, 32, 64);
    const int row = AT ? c0 + mt : min(w0 + 16 * mt + r, s.count - 1);
    if (b & kWholeBits) s.whole[row] = 1;
    else if (b & 0x7fffffffu) found |= kSmall;
  }
  return found;
}

template <bool AT, int NT, int MT, int WR, int WC, typename Panel>
__device__ __forceinline__ int split_tile_waves(const SplitTile& s, const Panel& panel, uintx4* lds) {
  constexpr int NTW = (NT + WC - 1) / WC;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = wave % WR, wc = wave / WR;
  if constexpr (NT % WC == 0) {
    return split_tile<AT, NT, NTW, MT, WR, WC>(s, panel, lds, wr, wc * NTW);
  } else {
    if (wc == 0) return split_tile<AT, NT, NTW, MT, WR, WC>(s, panel, lds, wr, 0);
    return split_tile<AT, NT, NTW - 1, MT, WR, WC>(s, panel, lds, wr, NTW);
  }
}

// Y = A X.  Work partition and partial panels as in k_gemm_an (AnShape), in chunks of two blocks.
template <int NT, int MT, int WR, int WC>
__global__ void __launch_bounds__(WR * WC * 64)
k_split_an(const float* __restrict__ A, int64_t lda, int rows, int K, const uintx4* __restrict__ XP, int64_t xstride,
           float* __restrict__ Y, int64_t ldy, int ncols, float* __restrict__ Part, int64_t ldp, int64_t split_stride,
           AnShape sh, int* __restrict__ flags, int* __restrict__ whole) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  constexpr int TR = WR * MT * 16;
  const AnWork w = an_work(sh, blockIdx.x);
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
    s.whole = whole;
    const int found = split_tile_waves<false, NT, MT, WR, WC>(s, PackedPanel{XP, xstride}, (uintx4*)lds_raw);
    if (found & kNotFinite) flags[blockIdx.x % kSplitFlags] = 1;
    if (found & kSmall) flags[kSplitFlags + blockIdx.x % kSplitFlags] = 1;
    __syncthreads();                                   // before the next strip reuses the staging buffers
  }
}

// Partial panel blockIdx.y of Z = A^T Q: blocks [y * blocks_per_sub, ...) of the rows.
template <int NT, int MT, int WR, int WC>
__global__ void __launch_bounds__(WR * WC * 64)
k_split_at(const float* __restrict__ A, int64_t lda, int64_t rows, int n, const uintx4* __restrict__ QP, int64_t xstride,
           float* __restrict__ Zpart, int64_t ldz, int64_t split_stride, int blocks, int blocks_per_sub,
           int* __restrict__ flags, int* __restrict__ whole) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
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
  s.whole = whole;
  const int found = split_tile_waves<true, NT, MT, WR, WC>(s, PackedPanel{QP, xstride}, (uintx4*)lds_raw);
  int* flag = flags + (blockIdx.y * gridDim.x + blockIdx.x) % kSplitFlags;
  if (found & kNotFinite) flag[0] = 1;
  if (found & kSmall) flag[kSplitFlags] = 1;
}

// Products with infinities, NaN or overflow: a split infinity is inf + NaN + NaN, and inf times the zero low parts
// of a short number is NaN, so where a result of the kernels above is not finite it is worked out once more with plain fp32
// multiplications.  So are the rows (AT: columns) of A that have elements below 2^-95 only, whose third parts bf16 may not hold:
// next to a larger element what they lose is below the rounding of that one's products.  (Columns of the panel with such
// elements only in a block of 32 are packed as NaN, which brings them here too.)  One workgroup per workgroup of the product, with the same part of the contraction and the same place for the
// result; it leaves at once when that one met nothing (about 3 us for the launch).  Otherwise it goes through pieces of 32 rows
// (AT: columns of A) and 64 columns of the panel and redoes those that have a result that is not finite in a column of the
// panel without a NaN: with one, it is NaN as it should be.  So a bad entry of A costs its rows or columns and a bad panel
// nothing.
// What bounds a piece: the latency of its operands, which come straight from global memory; so the eight waves share the
// contraction.  Measured (us of the whole product, A X / A^T Q; plain kernels in brackets; before, when every tile of the product was
// taken once more as soon as one entry was not finite):
//                            finite                     one infinity in A                         an infinity in every row and column
//   4000 x 4000 l=48         34 / 31 (41 / 40)          47 / 45 (41 / 40; before 429 / 526)       111 / 104
//   20000 x 8000 l=110       210 / 212 (377 / 358)      338 / 472 (388 / 365; 7749 / 12884)       831 / 1516
//   30000 x 20000 l=272      1836 / 1725 (2752 / 2835)  3025 / 4044 (2600 / 2815; 68574 / 97456)  7143 / 8865
struct SplitRepair {
  const float *A, *X;      // X: K x xcols, leading dimension ldx
  int64_t lda, ldx, K;
  int xcols, count, tile, nt_total;
  const unsigned* nan;     // [column tile][block]
  int64_t blocks;
  const int *flags, *whole;
};
constexpr int kRepairNT = 4, kRepairWaves = 8, kMaxTiles = kMaxL / kTile;
constexpr int kRepairMaxPieces = 256 / 32 * (kMaxTiles / kRepairNT);   // a tile has at most 256 rows (columns of A)

// Whether the piece at rows w0.. of the output and column tiles nt0.. has a result that its columns do not explain (one wave).
__device__ __forceinline__ bool repair_needed(const SplitRepair& p, int w0, int nt0, bool small, const unsigned* xnan,
                                              const float* out, int64_t ldo, int ncols) {
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  if (small && __any(p.whole[min(w0 + (lane & 31), p.count - 1)] == 0)) return true;
  float worst = 0.f;                                     // NaN as soon as one is not finite
#pragma unroll
  for (int nt = 0; nt < kRepairNT; ++nt) {
    const int tile = min(nt0 + nt, p.nt_total - 1), col = 16 * tile + r;
    const bool look = col < ncols && !(xnan[tile] >> r & 1);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float y = out[(int64_t)min(w0 + 4 * i + g, p.count - 1) * ldo + min(col, ncols - 1)];
      worst += look ? y * 0.f : 0.f;
    }
  }
  return __any(!(worst == 0.f));
}

// One piece by all waves: rows w0.. of the output (a multiple of 32), column tiles nt0.., contraction [kbeg, kend).
template <bool AT>
__device__ __forceinline__ void repair_piece(const SplitRepair& p, int w0, int nt0, int64_t kbeg, int64_t kend,
                                             floatx4* sum, float* out, int64_t ldo, int ncols) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15, g = lane >> 4;
  // the waves take equal parts of the contraction, multiples of 32, and add their sums in a fixed order
  const int64_t part = (kend - kbeg + 32 * kRepairWaves - 1) / (32 * kRepairWaves) * 32;
  const int64_t k_first = min(kend, kbeg + wave * part), k_last = min(kend, k_first + part);
  floatx4 acc[2][kRepairNT];
#pragma unroll
  for (int mt = 0; mt < 2; ++mt)
#pragma unroll
    for (int nt = 0; nt < kRepairNT; ++nt) acc[mt][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
  // lane (r, g) holds the contraction indices k0 + 4 g + {0..3} and k0 + 16 + 4 g + {0..3} of row r and of column r
  float a[2][8], x[kRepairNT][8];
  typedef floatx4 floatx4u __attribute__((aligned(4)));
  auto load = [&](int64_t k0, auto whole) {              // whole: all 32 indices are below kend
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int64_t kk = k0 + (e >> 2) * 16 + 4 * g + (e & 3);
      const bool in = whole || kk < k_last;
      const int64_t k = in ? kk : k_last - 1;
#pragma unroll
      for (int mt = 0; mt < 2; ++mt) {
        const int64_t row = min(w0 + 16 * mt + r, p.count - 1);
        if (AT || !whole) {
          const float v = AT ? p.A[k * p.lda + row] : p.A[row * p.lda + k];
          a[mt][e] = in ? v : 0.f;
        } else if (e % 4 == 0) {
          const floatx4 v = *(const floatx4u*)(p.A + row * p.lda + k);
#pragma unroll
          for (int i = 0; i < 4; ++i) a[mt][e + i] = v[i];
        }
      }
#pragma unroll
      for (int nt = 0; nt < kRepairNT; ++nt) {
        const int col = 16 * (nt0 + nt) + r;
        const float v = p.X[k * p.ldx + min(col, p.xcols - 1)];
        x[nt][e] = in && col < p.xcols ? v : 0.f;
      }
    }
  };
  auto add = [&]() {
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int nt = 0; nt < kRepairNT; ++nt)
          acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[mt][e], x[nt][e], acc[mt][nt], 0, 0, 0);
  };
  int64_t k0 = k_first;
#pragma nounroll
  for (; k0 + 32 <= k_last; k0 += 32) {
    load(k0, std::true_type{});
    __builtin_amdgcn_sched_barrier(0);
    add();
  }
  if (k0 < k_last) {
    load(k0, std::false_type{});
    add();
  }
#pragma unroll
  for (int h = kRepairWaves / 2; h > 0; h /= 2) {
    __syncthreads();
    if (wave >= h && wave < 2 * h) {
#pragma unroll
      for (int i = 0; i < 2 * kRepairNT; ++i) sum[((wave - h) * 2 * kRepairNT + i) * 64 + lane] = acc[i / kRepairNT][i % kRepairNT];
    }
    __syncthreads();
    if (wave < h) {
#pragma unroll
      for (int i = 0; i < 2 * kRepairNT; ++i) acc[i / kRepairNT][i % kRepairNT] += sum[(wave * 2 * kRepairNT + i) * 64 + lane];
    }
  }
  if (wave != 0) return;
#pragma unroll
  for (int mt = 0; mt < 2; ++mt)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = w0 + 16 * mt + 4 * g + v;
      if (row >= p.count) continue;
#pragma unroll
      for (int nt = 0; nt < kRepairNT; ++nt) {
        const int col = 16 * (nt0 + nt) + r;
        if (nt0 + nt < p.nt_total && col < ncols) out[(int64_t)row * ldo + col] = acc[mt][nt][v];
      }
    }
}

// The tile of rows (columns of A) from `first` on, over `blocks` blocks of the contraction from b0 on.
template <bool AT>
__device__ __forceinline__ void repair_tile(const SplitRepair& p, int first, int64_t b0, int blocks, bool small, const unsigned* xnan,
                                            float* out, int64_t ldo, int ncols) {
  __shared__ floatx4 sum[kRepairWaves / 2 * 2 * kRepairNT * 64];
  __shared__ int redo[kRepairMaxPieces];
  // (the blocks are an even number: the first is not the empty one)
  const int64_t kbeg = block_index(b0, p.K) * kSplitB, kend = min(p.K, block_index(b0 + blocks, p.K) * kSplitB);
  const int strips = (p.nt_total + kRepairNT - 1) / kRepairNT, pieces = (min(p.tile, p.count - first) + 31) / 32 * strips;
  for (int i = threadIdx.x >> 6; i < pieces; i += kRepairWaves) {
    const bool bad = repair_needed(p, first + i / strips * 32, i % strips * kRepairNT, small, xnan, out, ldo, ncols);
    if ((threadIdx.x & 63) == 0) redo[i] = bad;
  }
  __syncthreads();
  for (int i = 0; i < pieces; ++i)
    if (redo[i])
      repair_piece<AT>(p, first + i / strips * 32, i % strips * kRepairNT, kbeg, kend, sum, out, ldo, ncols);
  __syncthreads();                                       // before the next tile's `redo`
}

// Which columns of the panel have a NaN in the blocks [b0, b0 + blocks).
__device__ __forceinline__ void nan_columns(const SplitRepair& p, int64_t b0, int blocks, unsigned* xnan) {
  const int lane = threadIdx.x & 63;
  for (int nt = threadIdx.x >> 6; nt < p.nt_total; nt += kRepairWaves) {
    unsigned m = 0;
    for (int b = lane; b < blocks; b += 64) m |= p.nan[nt * p.blocks + b0 + b];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m |= __shfl_xor(m, off, 64);
    if (lane == 0) xnan[nt] = m;
  }
  __syncthreads();
}

__global__ void __launch_bounds__(kRepairWaves * 64)
k_split_repair_an(SplitRepair p, float* __restrict__ Y, int64_t ldy, int ncols, float* __restrict__ Part, int64_t ldp,
                  int64_t split_stride, AnShape sh) {
  __shared__ unsigned xnan[kMaxTiles];
  const int* flag = p.flags + blockIdx.x % kSplitFlags;
  const bool small = flag[kSplitFlags] != 0;
  if (flag[0] == 0 && !small) return;
  const AnWork w = an_work(sh, blockIdx.x);
  const int64_t b0 = 2 * (int64_t)w.c0;
  const int blocks = 2 * (w.c1 - w.c0);
  nan_columns(p, b0, blocks, xnan);
  float* out = w.partial ? Part + (int64_t)w.slot * split_stride - (int64_t)sh.whole * p.tile * ldp : Y;
  for (int seg = 0; seg < w.nseg; ++seg)
    repair_tile<false>(p, (w.first_tile + seg) * p.tile, b0, blocks, small, xnan, out, w.partial ? ldp : ldy, w.partial ? (int)ldp : ncols);
}

__global__ void __launch_bounds__(kRepairWaves * 64)
k_split_repair_at(SplitRepair p, float* __restrict__ Zpart, int64_t ldz, int64_t split_stride, int blocks_per_sub) {
  __shared__ unsigned xnan[kMaxTiles];
  const int* flag = p.flags + (blockIdx.y * gridDim.x + blockIdx.x) % kSplitFlags;
  const bool small = flag[kSplitFlags] != 0;
  if (flag[0] == 0 && !small) return;
  const int64_t b0 = (int64_t)blockIdx.y * blocks_per_sub;
  const int blocks = (int)min((int64_t)blocks_per_sub, p.blocks - b0);
  nan_columns(p, b0, blocks, xnan);
  repair_tile<true>(p, blockIdx.x * p.tile, b0, blocks, small, xnan, Zpart + (int64_t)blockIdx.y * split_stride, ldz, (int)ldz);
}

// What is left of a product of gemm_half.hip: the workgroups that gave up do their part with bf16 numbers, then (and where a result
// was not finite) the repair above, for the column tiles of one launch.  Which rows have small elements only is decided within the
// workgroup's part, so the result does not depend on what the others have come to.  No work for ordinary numbers (about 3 us for the
// launch).
struct SplitFix {
  SplitRepair p;           // of the launch's columns
  PackedPanel panel;       // the same columns, in bf16 numbers if a word of redo is kRedoPacked
  const int* redo;
};
template <bool AT, int NT, int MT, int WR, int WC>
__device__ __forceinline__ void split_fix(const SplitFix& f, SplitTile s, int redo, uintx4* lds) {
  __shared__ unsigned xnan[kMaxTiles];
  __shared__ int whole[MT + WR * MT * 16], found;        // (the last MT columns of A may begin before the tile)
  SplitRepair p = f.p;
  if (threadIdx.x < MT + WR * MT * 16) whole[threadIdx.x] = 0;
  if (threadIdx.x == 0) found = 0;
  __syncthreads();
  s.whole = whole + MT - s.first;                        // addressed like the words of all rows
  int mine = 0;
  if (redo == kRedoPacked) mine = split_tile_waves<AT, NT, MT, WR, WC>(s, f.panel, lds);
  else if (redo == kRedoRaw) mine = split_tile_waves<AT, NT, MT, WR, WC>(s, RawPanel{p.X, p.ldx, p.xcols}, lds);
  if (mine) atomicOr(&found, mine);
  __threadfence_block();
  __syncthreads();
  if (redo && found == 0) return;
  const bool small = found & kSmall;
  p.whole = s.whole;
  nan_columns(p, s.b0, s.blocks, xnan);
  repair_tile<AT>(p, s.first, s.b0, s.blocks, small, xnan, s.out, s.ldo, s.ncols);
}

template <int NT, int MT, int WR, int WC>
__global__ void __launch_bounds__(WR * WC * 64)
k_split_fix_an(SplitFix f, float* __restrict__ Y, int64_t ldy, int ncols, float* __restrict__ Part, int64_t ldp, int64_t split_stride,
               AnShape sh) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  constexpr int TR = WR * MT * 16;
  const int redo = f.redo[blockIdx.x];
  if (!redo && f.p.flags[blockIdx.x % kSplitFlags] == 0) return;
  const AnWork w = an_work(sh, blockIdx.x);
  for (int seg = 0; seg < w.nseg; ++seg) {
    SplitTile s;
    s.first = (w.first_tile + seg) * TR;
    s.A = f.p.A + (int64_t)s.first * f.p.lda;
    s.lda = f.p.lda;
    s.K = f.p.K;
    s.b0 = 2 * (int64_t)w.c0;
    s.blocks = 2 * (w.c1 - w.c0);
    s.count = f.p.count;
    s.out = w.partial ? Part + (int64_t)w.slot * split_stride - (int64_t)sh.whole * TR * ldp : Y;
    s.ldo = w.partial ? ldp : ldy;
    s.ncols = w.partial ? NT * 16 : ncols;
    split_fix<false, NT, MT, WR, WC>(f, s, redo, (uintx4*)lds_raw);
    __syncthreads();
  }
}

template <int NT, int MT, int WR, int WC>
__global__ void __launch_bounds__(WR * WC * 64)
k_split_fix_at(SplitFix f, float* __restrict__ Zpart, int64_t ldz, int64_t split_stride, int blocks_per_sub) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  const int wg = blockIdx.y * gridDim.x + blockIdx.x;
  const int redo = f.redo[wg];
  if (!redo && f.p.flags[wg % kSplitFlags] == 0) return;
  SplitTile s;
  s.A = f.p.A;
  s.lda = f.p.lda;
  s.K = f.p.K;
  s.b0 = (int64_t)blockIdx.y * blocks_per_sub;
  s.blocks = (int)min((int64_t)blocks_per_sub, f.p.blocks - s.b0);
  s.first = blockIdx.x * (WR * MT * 16);
  s.count = f.p.count;
  s.out = Zpart + (int64_t)blockIdx.y * split_stride;
  s.ldo = ldz;
  s.ncols = NT * 16;
  split_fix<true, NT, MT, WR, WC>(f, s, redo, (uintx4*)lds_raw);
}

bool split_fits(bool at, const float* A, int64_t out, int64_t K, int Lp, int64_t lda, uint64_t pack_bytes) {
  // byte offsets of a lane's loads: at most 255 rows and a row length, in 32 bits
  if (K < kSplitMinK || out < kSplitMinOut || Lp < kSplitMinLp || out * K < kSplitMinA || lda > (1 << 21)) return false;
  if (out > INT32_MAX || K > INT32_MAX - 2 * kSplitB) return false;     // block_start
  if (Lp < 48) {                                         // both kernels are near the read of A: see common.h
    const bool vectors = lda % 4 == 0 && (uintptr_t)A % 16 == 0, lines = lda % 32 == 0 && (uintptr_t)A % 128 == 0;
    const bool few = out >= 8000 && K <= (out <= 20480 ? 6000 : 2048), many = out >= 14500 && K >= 20000;
    if (at ? vectors && !few && !many : !lines || K < 14000 || out < 20000) return false;
  }
  return pack_bytes >= pack_layout(out, K, Lp).bytes;
}

SplitPlan split_an_plan(int64_t rows, int64_t K, int Lp, uint64_t scratch_bytes) {
  const NGroups ng = column_groups(Lp, 4);
  SplitPlan p;
  p.nt = ng.nt;
  p.groups = ng.groups;
  p.tile = split_cfg(ng.nt).tile;
  const int T = (int)ceil_div(rows, p.tile), C = (int)split_chunks(K);
  // as many splits as the scratch has room for
  for (int S = kSplitSlots;; S = S * 3 / 4) {
    p.sh = an_shape(T, C, S, 8, 4);
    p.nsplit = p.sh.lt > 0 ? p.sh.f + (p.sh.x > 0 ? 1 : 0) : 0;
    p.partial_rows = p.nsplit > 0 ? rows - (int64_t)p.sh.whole * p.tile : 0;
    if ((uint64_t)p.nsplit * p.partial_rows * Lp * 4 <= scratch_bytes) break;
    if (S <= 1) { p.sh = AnShape{C, T, 0, 1, 0, 0}; p.nsplit = 0; p.partial_rows = 0; break; }
  }
  p.wgs = p.sh.whole + p.sh.lt * p.sh.f + (p.sh.x > 0 ? (int)ceil_div(p.sh.lt, p.sh.j) : 0);
  return p;
}

SplitPlan split_at_plan(int64_t rows, int64_t n, int Lp, uint64_t scratch_bytes) {
  const NGroups ng = column_groups(Lp, 4);
  SplitPlan p;
  p.nt = ng.nt;
  p.groups = ng.groups;
  p.tile = split_cfg(ng.nt).tile;
  p.col_tiles = (int)ceil_div(n, p.tile);
  const int64_t chunks = split_chunks(rows);
  const int64_t room = (int64_t)(scratch_bytes / ((uint64_t)n * Lp * 4));
  const int want = pick_splits(p.col_tiles, kSplitSlots, chunks, (double)Lp / (double)rows, traffic_weight(ng.nt), (int)std::min<int64_t>(room, 4096));
  const int64_t per = ceil_div(chunks, want);
  p.blocks = (int)(2 * chunks);
  p.blocks_per_sub = (int)(2 * per);
  p.nsplit = room < 1 ? 0 : (int)ceil_div(chunks, per);
  return p;
}

// (ten tiles in two columns of waves: the second group of a panel of 21 tiles, whose first group has eleven)
#define BRSVD_SPLIT_SWITCH(nt, tile, CALL)                                                                       \
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
static int split_lds(K kern, int nt, bool* done) {
  if (!*done) {
    BRSVD_HIP_TRY(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 2 * nt * 3 * kFragU * 16));
    *done = true;
  }
  return BRSVD_OK;
}

struct Packed {
  const uintx4* panel;
  int64_t stride;                                        // 16-byte units of one block
  int *flags, *whole;
  SplitRepair repair;
};

static int split_pack(const float* A, int64_t lda, int64_t count, int tile, const float* X, int64_t K, int64_t ldx, int xcols, int Lp,
                      void* pack, Packed* out, hipStream_t stream) {
  const PackLayout lay = pack_layout(count, K, Lp);
  const int64_t blocks = 2 * split_chunks(K), units = blocks * (Lp / 16) * kFragU;
  unsigned* nan = (unsigned*)((char*)pack + lay.nan);
  int *flags = (int*)((char*)pack + lay.flags), *whole = (int*)((char*)pack + lay.whole);
  *out = Packed{(const uintx4*)pack, (Lp / 16) * 3 * kFragU, flags, whole,
                SplitRepair{A, X, lda, ldx, K, xcols, (int)count, tile, Lp / 16, nan, blocks, flags, whole}};
  hipLaunchKernelGGL(k_split_pack, dim3((unsigned)ceil_div(units, 256)), dim3(256), 0, stream, X, K, ldx, xcols, Lp / 16,
                     blocks, (uintx4*)pack, nan, flags, 2 * kSplitFlags + count);
  BRSVD_HIP_TRY(hipGetLastError());
  return BRSVD_OK;
}

// Whether the products of two fp16 numbers each (gemm_half.hip) are taken: `piece` = contraction indices one workgroup adds up, on
// average.  They are where their results are about as accurate or more: what the split loses (7e-8 of a product) has to be less than what
// the additions lose, half as many as here.  Relative error, 3 x bf16 and 2 x fp16 (N(0, 1) entries, K x outputs, pieces; a test holds the
// second to the first):
//   1000 x 300000 1000 1.20e-7 / 1.33e-7    1472 x 60000 1472 1.40e-7 / 1.44e-7   2100 x 30000 1050 1.29e-7 / 1.40e-7
//   1900 x 60000 1900 1.58e-7 / 1.53e-7     6000 x 16000 1500 1.63e-7 / 1.58e-7   12000 x 8192 1500 1.87e-7 / 1.71e-7
//   4000 x 8000 500 1.24e-7 / 1.42e-7       8192 x 1000 256 1.51e-7 / 1.59e-7     12000 x 2000 375 1.72e-7 / 1.72e-7
//   16384 x 1000 512 1.81e-7 / 1.75e-7      33000 x 1000 520 2.27e-7 / 2.01e-7    89083 x 2783 3.86e-7 / 2.98e-7
// Entries uniform in (0, 1): 1472 x 60000 1.41e-7 / 1.40e-7, 16384 x 1000 1.88e-7 / 1.90e-7 (l = 48; 1.75e-7 / 1.73e-7 with l = 110), 89083 x 2783
// 3.42e-7 / 2.68e-7.  A of rank 2 l times orthonormal columns along it, where both are near the rounding of the result: 2783 x 89083
// 1.25e-7 / 9.4e-8, 33000 x 1000 5.06e-8 / 5.07e-8, 200000 x 300 5.3e-8 / 5.6e-8.
constexpr int64_t kHalfMinPiece = 1408, kHalfMinK = 16384;
static bool half_fits(int64_t K, int64_t piece) { return piece >= kHalfMinPiece || K >= kHalfMinK; }
// The place of the packed panel, of the words and of the flags is that of three bf16 numbers; from the flags of rows with small elements
// only on, and through the words of all rows behind them, stands what each workgroup left undone.
static bool half_room(int64_t wgs, int64_t out) { return wgs <= kSplitFlags + out; }
static bool half_fits_an(int64_t out, int64_t K, const SplitPlan& p) {
  const AnShape& sh = p.sh;
  const int64_t tiles = sh.whole + sh.lt, chunks = (int64_t)sh.whole * sh.C + (sh.lt > 0 ? (int64_t)sh.lt * ((sh.C - sh.x) / sh.f) : 0);
  return half_fits(K, 2 * kSplitB * chunks / tiles) && half_room(p.wgs, out);
}
static bool half_fits_at(int64_t out, int64_t K, const SplitPlan& p) {
  return half_fits(K, kSplitB * std::min(p.blocks, p.blocks_per_sub)) && half_room((int64_t)p.col_tiles * p.nsplit, out);
}
int split_parts(bool at, int64_t out, int64_t K, int Lp) {
  if (at) return half_fits_at(out, K, split_at_plan(K, out, Lp, UINT64_MAX)) ? 2 : 3;
  return half_fits_an(out, K, split_an_plan(out, K, Lp, UINT64_MAX)) ? 2 : 3;
}
static int half_prepare(const float* A, int64_t lda, int64_t count, int tile, const float* X, int64_t K, int64_t ldx, int xcols,
                        int Lp, bool at, int64_t wgs, void* pack, Packed* out, HalfPacked* hp, hipStream_t stream) {
  const PackLayout lay = pack_layout(count, K, Lp);
  unsigned* nan = (unsigned*)((char*)pack + lay.nan);
  int* flags = (int*)((char*)pack + lay.flags);
  *out = Packed{(const uintx4*)pack, 0, flags, nullptr,
                SplitRepair{A, X, lda, ldx, K, xcols, (int)count, tile, Lp / 16, nan, 2 * split_chunks(K), flags, nullptr}};
  *hp = HalfPacked{pack, nan, flags, flags + kSplitFlags, kSplitFlags + wgs, X, ldx, xcols};
  return half_pack(A, lda, count, K, Lp, at, *hp, stream);
}
// The column tiles [c0 / 16, c0 / 16 + nt) alone.
static SplitRepair group_repair(SplitRepair p, int c0, int nt) {
  p.X += c0;
  p.xcols = std::min(p.xcols - c0, nt * 16);
  p.nan += c0 / 16 * p.blocks;
  p.nt_total = nt;
  return p;
}

int split_gemm_an(const float* A, int64_t lda, int64_t rows, int64_t K, const float* X, int64_t ldx, int xcols, int Lp,
                  float* Y, int64_t ldy, int ncols, void* scratch, uint64_t scratch_bytes, void* pack,
                  uint64_t pack_bytes, hipStream_t stream, const KernelEvents* ev, bool whole) {
  if (!split_fits(false, A, rows, K, Lp, lda, pack_bytes) || ncols > Lp) return BRSVD_ERR_ARG;
  const SplitPlan p = split_an_plan(rows, K, Lp, scratch_bytes);
  float* part = (float*)scratch;
  const int64_t stride = p.partial_rows * Lp;
  Packed x;
  const bool half = !whole && half_fits_an(rows, K, p);
  HalfPacked hp;
  if (half) BRSVD_TRY(half_prepare(A, lda, rows, p.tile, X, K, ldx, xcols, Lp, false, p.wgs, pack, &x, &hp, stream));
  else BRSVD_TRY(split_pack(A, lda, rows, p.tile, X, K, ldx, xcols, Lp, pack, &x, stream));
  for (int gi = 0; gi < p.groups; ++gi) {
    const int c0 = gi * p.nt * 16, nt = std::min(p.nt, (Lp - c0) / 16);
    if (nt <= 0) break;
    if (half) {
      BRSVD_TRY(half_an(A, lda, rows, K, hp, Lp, c0, nt, p.tile, Y + c0, ldy, std::min(ncols - c0, nt * 16), part ? part + c0 : nullptr,
                        stride, p.sh, p.wgs, stream));
      const SplitFix fix{group_repair(x.repair, c0, nt), PackedPanel{(const uintx4*)hp.panel + (c0 / 16) * 3 * kFragU, (Lp / 16) * 3 * kFragU}, hp.redo};
#define CALL(N, WR, WC)                                                                                              \
  {                                                                                                                  \
    auto kern = k_split_fix_an<N, kSplitMT, WR, WC>;                                                                 \
    static bool done = false;                                                                                        \
    BRSVD_TRY(split_lds(kern, N, &done));                                                                            \
    hipLaunchKernelGGL(kern, dim3(p.wgs), dim3(WR * WC * 64), 2 * N * 3 * kFragU * 16, stream, fix, Y + c0, ldy,      \
                       std::min(ncols - c0, N * 16), part ? part + c0 : nullptr, (int64_t)Lp, stride, p.sh);         \
  }
      BRSVD_SPLIT_SWITCH(nt, p.tile, CALL)
#undef CALL
      BRSVD_HIP_TRY(hipGetLastError());
      continue;
    }
    const uintx4* xp = x.panel + (c0 / 16) * 3 * kFragU;
#define CALL(N, WR, WC)                                                                                              \
  {                                                                                                                  \
    if (p.tile != WR * kSplitMT * 16) return BRSVD_ERR_ARG;                                                          \
    auto kern = k_split_an<N, kSplitMT, WR, WC>;                                                                     \
    static bool done = false;                                                                                        \
    BRSVD_TRY(split_lds(kern, N, &done));                                                                            \
    hipLaunchKernelGGL(kern, dim3(p.wgs), dim3(WR * WC * 64), 2 * N * 3 * kFragU * 16, stream, A, lda, (int)rows, (int)K, \
                       xp, x.stride, Y + c0, ldy, std::min(ncols - c0, N * 16), part ? part + c0 : nullptr, (int64_t)Lp, stride, p.sh, x.flags, x.whole); \
  }
    BRSVD_SPLIT_SWITCH(nt, p.tile, CALL)
#undef CALL
    BRSVD_HIP_TRY(hipGetLastError());
  }
  if (!half) {
    hipLaunchKernelGGL(k_split_repair_an, dim3(p.wgs), dim3(kRepairWaves * 64), 0, stream, x.repair, Y, ldy, ncols, part, (int64_t)Lp,
                       stride, p.sh);
    BRSVD_HIP_TRY(hipGetLastError());
  }
  if (ev) BRSVD_HIP_TRY(hipEventRecord(ev->stop, stream));
  if (p.nsplit > 0) {
    const int64_t r0 = rows - p.partial_rows;
    BRSVD_TRY(reduce_splits_f32(part, p.nsplit, stride, p.partial_rows, ncols, Lp, Y + r0 * ldy, ldy, false, stream));
  }
  if (ev) BRSVD_HIP_TRY(hipEventRecord(ev->sum_stop, stream));
  return BRSVD_OK;
}

int split_gemm_at(const float* A, int64_t lda, int64_t rows, int64_t n, const float* Q, int64_t ldq, int qcols, int Lp,
                  float* Z, int64_t ldz, int ncols, bool accumulate, void* scratch, uint64_t scratch_bytes, void* pack,
                  uint64_t pack_bytes, hipStream_t stream, const KernelEvents* ev, bool whole) {
  if (!split_fits(true, A, n, rows, Lp, lda, pack_bytes) || ncols > Lp) return BRSVD_ERR_ARG;
  const SplitPlan p = split_at_plan(rows, n, Lp, scratch_bytes);
  if (p.nsplit < 1) return BRSVD_ERR_BUDGET;
  if (p.nsplit > 65535) return BRSVD_ERR_ARG;
  float* part = (float*)scratch;
  const int64_t stride = n * Lp;
  Packed x;
  const bool half = !whole && half_fits_at(n, rows, p);
  HalfPacked hp;
  if (half) BRSVD_TRY(half_prepare(A, lda, n, p.tile, Q, rows, ldq, qcols, Lp, true, (int64_t)p.col_tiles * p.nsplit, pack, &x, &hp, stream));
  else BRSVD_TRY(split_pack(A, lda, n, p.tile, Q, rows, ldq, qcols, Lp, pack, &x, stream));
  for (int gi = 0; gi < p.groups; ++gi) {
    const int c0 = gi * p.nt * 16, nt = std::min(p.nt, (Lp - c0) / 16);
    if (nt <= 0) break;
    if (half) {
      BRSVD_TRY(half_at(A, lda, rows, n, hp, Lp, c0, nt, p.tile, part + c0, stride, p.col_tiles, p.nsplit, p.blocks, p.blocks_per_sub,
                        stream));
      const SplitFix fix{group_repair(x.repair, c0, nt), PackedPanel{(const uintx4*)hp.panel + (c0 / 16) * 3 * kFragU, (Lp / 16) * 3 * kFragU}, hp.redo};
#define CALL(N, WR, WC)                                                                                              \
  {                                                                                                                  \
    auto kern = k_split_fix_at<N, kSplitMT, WR, WC>;                                                                 \
    static bool done = false;                                                                                        \
    BRSVD_TRY(split_lds(kern, N, &done));                                                                            \
    hipLaunchKernelGGL(kern, dim3(p.col_tiles, p.nsplit), dim3(WR * WC * 64), 2 * N * 3 * kFragU * 16, stream, fix,   \
                       part + c0, (int64_t)Lp, stride, p.blocks_per_sub);                                            \
  }
      BRSVD_SPLIT_SWITCH(nt, p.tile, CALL)
#undef CALL
      BRSVD_HIP_TRY(hipGetLastError());
      continue;
    }
    const uintx4* qp = x.panel + (c0 / 16) * 3 * kFragU;
#define CALL(N, WR, WC)                                                                                              \
  {                                                                                                                  \
    if (p.tile != WR * kSplitMT * 16) return BRSVD_ERR_ARG;                                                          \
    auto kern = k_split_at<N, kSplitMT, WR, WC>;                                                                     \
    static bool done = false;                                                                                        \
    BRSVD_TRY(split_lds(kern, N, &done));                                                                            \
    hipLaunchKernelGGL(kern, dim3(p.col_tiles, p.nsplit), dim3(WR * WC * 64), 2 * N * 3 * kFragU * 16, stream, A, lda, rows, \
                       (int)n, qp, x.stride, part + c0, (int64_t)Lp, stride, p.blocks, p.blocks_per_sub, x.flags, x.whole);    \
  }
    BRSVD_SPLIT_SWITCH(nt, p.tile, CALL)
#undef CALL
    BRSVD_HIP_TRY(hipGetLastError());
  }
  if (!half) {
    hipLaunchKernelGGL(k_split_repair_at, dim3(p.col_tiles, p.nsplit), dim3(kRepairWaves * 64), 0, stream, x.repair, part, (int64_t)Lp,
                       stride, p.blocks_per_sub);
    BRSVD_HIP_TRY(hipGetLastError());
  }
  if (ev) BRSVD_HIP_TRY(hipEventRecord(ev->stop, stream));
  BRSVD_TRY(reduce_splits_f32(part, p.nsplit, stride, n, ncols, Lp, Z, ldz, accumulate, stream));
  if (ev) BRSVD_HIP_TRY(hipEventRecord(ev->sum_stop, stream));
  return BRSVD_OK;
}

}  // namespace brsvd
