// Small device helpers shared by the MFMA kernels (block form and two-phase) of libvla.
#pragma once

#include "vla_common.h"

namespace vla {

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int C = 16;       // tokens per block
constexpr int LT = C + 4;   // row stride (floats) of the 16-column LDS arrays: conflict-free b128 rows

// Workspace of the two-phase and time-parallel modes, per head and 16-token block (floats):
//   RN  [16]       1 / max(||k_t||, eps) per token, 0 for rows past the end (k^_t = k_t * RN[t])
//   WT  [D][16]    the write directions before their scaling by c_t (w_t; alpha_t with a separate u)
//   SM  [544]      Z [16][16] | -NQ^T [16][16] | -c_t [16] | 1 / max(q_t . zkey_t, eps) [16] (normalised
//                  read-out only)
// each as one array over all blocks of the head.
constexpr int SMB = 2 * C * C + 2 * C;
__host__ __device__ constexpr size_t head_stride(int nblk, int D) {
  return static_cast<size_t>(nblk) * (C + C * D + SMB);
}
__host__ __device__ constexpr size_t off_rn(int /*nblk*/, int /*D*/) { return 0; }
__host__ __device__ constexpr size_t off_wt(int nblk, int /*D*/) { return static_cast<size_t>(nblk) * C; }
__host__ __device__ constexpr size_t off_sm(int nblk, int D) { return static_cast<size_t>(nblk) * (C + C * D); }

__device__ __forceinline__ f4 mfma16(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// ---- FP32 products on the bf16 matrix instruction.  A float32 value is the sum of three bf16 values (3 x 8
// significant bits); a product of two bf16 values is exact in float32, which is what the instruction accumulates
// in.  So a float32 matrix times a matrix of bf16 numbers is three products with nothing left out, and a float32
// matrix times a float32 matrix is the six products of weight 2^-16 and more.  What is left out of a product x y is at
// most 2^-24 |x y| where both factors are split by rounding and 3 x 2^-24 where one is cut off (the state); 0.1 and 0.3
// of 2^-24 in the root mean square, with the sign of the rounded factor's low terms.  Factors are finite: an infinite
// one gives NaN, and so does one that rounds to infinity in bf16 (3.39e38 and more).  Measured on one SIMD: 7.8 ns for
// 16x16x32 in bf16 against 14.2 ns for 16x16x4 in FP32, so three products take 0.21 of the FP32 time and six 0.41; and
// the bf16 instruction leaves the vector ALU free for other waves (32 MFMAs beside 64 FMAs of another wave 0.263 us,
// 0.249 and 0.116 us alone), which the FP32 one does not.
// v_dot2_f32_bf16 would form the residuals below in fewer instructions but excludes the matrix unit (0.428 us for
// the same pair).
//
// v_mfma_f32_16x16x32_bf16 register layout, lane l = 16*g + c, i = 0..7:
//   A operand: A[m = c][k = 8g + i]     B operand: B[k = 8g + i][n = c]     C/D: reg r -> D[m = 4g + r][n = c]
// The order of k is free as long as both operands agree.  Contractions over the head dimension take 32 columns at a
// time in the order of two accumulator tiles: slot i of lane group g is column 4g + i of the first tile for i < 4
// and column 4g + i - 4 of the second one from there (kslot() gives the position of a column).
typedef uint32_t u2 __attribute__((ext_vector_type(2)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f4 mfma_bf16(u4 a, u4 b, f4 c) {
  typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8, a), __builtin_bit_cast(bf8, b), c, 0, 0, 0);
}
// position of column j (a multiple of 4) in a row of operand slots
__host__ __device__ constexpr int kslot(int j) { return (j & ~31) + 8 * ((j >> 2) & 3) + 4 * ((j >> 4) & 1); }

__device__ __forceinline__ float top_half(float x) {
  return __uint_as_float(__float_as_uint(x) & 0xffff0000u);
}
// the upper halves of two float32 values, packed (x0 in the low half)
__device__ __forceinline__ uint32_t pack_tops(float x0, float x1) {
  return __builtin_amdgcn_perm(__float_as_uint(x1), __float_as_uint(x0), 0x07060302u);
}
__device__ __forceinline__ uint32_t pack_rne(float x0, float x1) {
  typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
  typedef float fl2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(fl2{x0, x1}, bf2));
}
// x = h + m + l exactly, each term cut off (never rounded up, so that the largest finite values split as well)
__device__ __forceinline__ void split3_cut(f4 x, u2& h, u2& m, u2& l) {
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const float x0 = x[2 * p], x1 = x[2 * p + 1];
    const float r0 = x0 - top_half(x0), r1 = x1 - top_half(x1);
    const float s0 = r0 - top_half(r0), s1 = r1 - top_half(r1);
    h[p] = pack_tops(x0, x1);
    m[p] = pack_tops(r0, r1);
    l[p] = pack_tops(s0, s1);
  }
}
// The same split with the residuals formed by the matrix unit, which subtracts h times the identity from an accumulator
// tile: operand slot i of a lane is the element in its accumulator register i, so h is used as packed, and x - h has no
// bits below the last place of x, so that it comes out exactly (the same bits as above).  6 vector and 2 matrix instructions
// where the above takes 22 vector ones, at twice the latency: for kernels whose waves cover it (vla_chunk_pipe.hip, 2048
// heads of 128: 2.28 -> 2.00 ms); with two waves per SIMD it gains nothing (vla_chunk.hip: 17.35 and 17.36 ms, 2048 heads
// of 64 6.69 -> 7.07).
__device__ __forceinline__ u2 minus_identity(int c, int g) {
  const int i = c - 4 * g;   // the slot on the diagonal, if 0..3
  return u2{i == 0 ? 0x0000bf80u : i == 1 ? 0xbf800000u : 0u, i == 2 ? 0x0000bf80u : i == 3 ? 0xbf800000u : 0u};
}
// a b over 16 columns, four slots of a lane group
__device__ __forceinline__ f4 mfma_bf16_half(u2 a, u2 b, f4 acc) {
  typedef short s4 __attribute__((ext_vector_type(4)));
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s4, a), __builtin_bit_cast(s4, b), acc, 0, 0, 0);
}
__device__ __forceinline__ f4 residual(f4 x, u2 h, u2 minus_one) { return mfma_bf16_half(minus_one, h, x); }
__device__ __forceinline__ void split3_cut_matrix(f4 x, u2 minus_one, u2& h, u2& m, u2& l) {
  h = u2{pack_tops(x[0], x[1]), pack_tops(x[2], x[3])};
  const f4 r = residual(x, h, minus_one);
  m = u2{pack_tops(r[0], r[1]), pack_tops(r[2], r[3])};
  const f4 s = residual(r, m, minus_one);
  l = u2{pack_tops(s[0], s[1]), pack_tops(s[2], s[3])};
}
// x = h + m + l with h and m rounded to nearest: the terms that a product of two split factors leaves out
// (m l, l m, l l) are then unbiased.
__device__ __forceinline__ void split3_rne(f4 x, u2& h, u2& m, u2& l) {
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const float x0 = x[2 * p], x1 = x[2 * p + 1];
    h[p] = pack_rne(x0, x1);
    const float r0 = x0 - __uint_as_float(h[p] << 16), r1 = x1 - __uint_as_float(h[p] & 0xffff0000u);
    m[p] = pack_rne(r0, r1);
    const float s0 = r0 - __uint_as_float(m[p] << 16), s1 = r1 - __uint_as_float(m[p] & 0xffff0000u);
    l[p] = pack_rne(s0, s1);
  }
}
// Keys that enter the products before they are normalised are staged as k 2^e, and the results multiplied by the rest of
// 1 / max(||k||, eps) = 2^e rest, 1 <= rest < 2: k 2^e is still a bf16 (float32) number and at most 1, so that a product
// with the state stays in range wherever k^ does (||k|| = 1e13 against a state of 1e28).
struct KeyScale { float pow2, rest; };
__device__ __forceinline__ KeyScale key_scale(float rn) {   // rn = 0 (no key): 0 and 0; NaN: rest NaN
  const uint32_t p = __float_as_uint(rn) & 0x7f800000u;
  return KeyScale{__uint_as_float(p), rn * __uint_as_float(0x7f000000u - p)};
}
__device__ __forceinline__ u4 cat(u2 a, u2 b) { return u4{a[0], a[1], b[0], b[1]}; }

// One operand of 32 columns: the NT = 1 (exact bf16 numbers) or 3 (h, m, l) terms.
template <int NT> struct Terms { u4 t[NT]; };

// Operand terms of two accumulator tiles (32 rows of the contraction).
__device__ __forceinline__ Terms<3> split_tiles(f4 x0, f4 x1) {
  u2 h0, m0, l0, h1, m1, l1;
  split3_cut(x0, h0, m0, l0);
  split3_cut(x1, h1, m1, l1);
  return Terms<3>{{cat(h0, h1), cat(m0, m1), cat(l0, l1)}};
}
// with the residuals from the matrix unit (minus_one: minus_identity() of the lane)
__device__ __forceinline__ Terms<3> split_tiles(f4 x0, f4 x1, u2 minus_one) {
  u2 h0, m0, l0, h1, m1, l1;
  split3_cut_matrix(x0, minus_one, h0, m0, l0);
  split3_cut_matrix(x1, minus_one, h1, m1, l1);
  return Terms<3>{{cat(h0, h1), cat(m0, m1), cat(l0, l1)}};
}
// acc += a b over 32 columns.  b holds three terms; a one or three.  Small products first.
template <int NT>
__device__ __forceinline__ f4 mfma_terms(const Terms<NT>& a, const Terms<3>& b, f4 acc) {
  if constexpr (NT == 1) {
    acc = mfma_bf16(a.t[0], b.t[2], acc);
    acc = mfma_bf16(a.t[0], b.t[1], acc);
    return mfma_bf16(a.t[0], b.t[0], acc);
  } else {
    acc = mfma_bf16(a.t[0], b.t[2], acc);
    acc = mfma_bf16(a.t[2], b.t[0], acc);
    acc = mfma_bf16(a.t[1], b.t[1], acc);
    acc = mfma_bf16(a.t[0], b.t[1], acc);
    acc = mfma_bf16(a.t[1], b.t[0], acc);
    return mfma_bf16(a.t[0], b.t[0], acc);
  }
}

// The same over 16 columns (a wave's slab of one tile): half an operand, half the terms to split.
template <int NT> struct HalfTerms { u2 t[NT]; };
__device__ __forceinline__ HalfTerms<3> split_tile(f4 x, u2 minus_one) {
  HalfTerms<3> s;
  split3_cut_matrix(x, minus_one, s.t[0], s.t[1], s.t[2]);
  return s;
}
template <int NT>
__device__ __forceinline__ f4 mfma_terms(const HalfTerms<NT>& a, const HalfTerms<3>& b, f4 acc) {
  if constexpr (NT == 3) {
    acc = mfma_bf16_half(a.t[0], b.t[2], acc);
    acc = mfma_bf16_half(a.t[2], b.t[0], acc);
    acc = mfma_bf16_half(a.t[1], b.t[1], acc);
    acc = mfma_bf16_half(a.t[0], b.t[1], acc);
    acc = mfma_bf16_half(a.t[1], b.t[0], acc);
  } else {
    acc = mfma_bf16_half(a.t[0], b.t[2], acc);
    acc = mfma_bf16_half(a.t[0], b.t[1], acc);
  }
  return mfma_bf16_half(a.t[0], b.t[0], acc);
}
// three terms on the left, one on the right
template <typename T3, typename T1>
__device__ __forceinline__ f4 mfma_terms_left(const T3& a, const T1& b, f4 acc) {
#pragma unroll
  for (int i = 2; i >= 0; --i) {
    if constexpr (sizeof(a.t[0]) == sizeof(u4)) acc = mfma_bf16(a.t[i], b.t[0], acc);
    else acc = mfma_bf16_half(a.t[i], b.t[0], acc);
  }
  return acc;
}

// A contraction over the 16 tokens of a block fills only half of the 32 slots, so one instruction takes two of the
// six products: slots 0-3 of a lane hold one term of its four tokens, slots 4-7 another one.
//   [h m] x [h m] = hh + mm,   [h m] x [m h] = hm + mh,   [l h] x [h l] = lh + hl
// For x = y the sums come out the same with the two factors exchanged (checked bit for bit on the device), so a
// symmetric matrix stays symmetric.
struct TokB { u4 hm, mh, hl; };   // B operand: four tokens per lane
__device__ __forceinline__ TokB tok_b(f4 x) {
  u2 h, m, l;
  split3_rne(x, h, m, l);
  return TokB{cat(h, m), cat(m, h), cat(h, l)};
}
// LDS image of a [rows][16 tokens] A operand: HM holds 16 bytes (h, m of four tokens) and L 8 bytes per row and
// token group; the group index is swizzled by the row so that 16 lanes on 16 rows hit different banks.
__device__ __forceinline__ int tok_chunk(int c, int g) { return g ^ ((c >> 2) & 3); }
__device__ __forceinline__ void tok_store(u4* hm, u2* l, int row, int c, int g, f4 x) {
  u2 h, m, lo;
  split3_rne(x, h, m, lo);
  const int i = 4 * row + tok_chunk(c, g);
  hm[i] = cat(h, m);
  l[i] = lo;
}
struct TokA { u4 hm, lh; };
__device__ __forceinline__ TokA tok_load(const u4* hm, const u2* l, int row, int c, int g) {
  const int i = 4 * row + tok_chunk(c, g);
  TokA a;
  a.hm = hm[i];
  a.lh = cat(l[i], *reinterpret_cast<const u2*>(hm + i));
  return a;
}
__device__ __forceinline__ f4 mfma_tok(const TokA& a, const TokB& b, f4 acc) {
  acc = mfma_bf16(a.lh, b.hl, acc);
  acc = mfma_bf16(a.hm, b.mh, acc);
  return mfma_bf16(a.hm, b.hm, acc);
}
// B operand of X from the LDS image of X (rows = columns of the product), of -X with flip = 0x80008000
__device__ __forceinline__ TokB tok_image_b(const u4* hm, const u2* l, int row, int c, int g, uint32_t flip) {
  const int i = 4 * row + tok_chunk(c, g);
  const u4 x = hm[i] ^ flip;
  const u2 y = l[i] ^ flip;
  return TokB{x, u4{x[2], x[3], x[0], x[1]}, u4{x[0], x[1], y[0], y[1]}};
}

// The products of the block form.  SPLIT: on bf16 terms as above; otherwise on the FP32 matrix instruction, with the
// operands staged as float32 in the same arrays (head size 16 is a single tile: half of the slots of a bf16 product
// would be empty and nothing but the latency of the chain counts; one head of 256 tokens: 51 us with FP32 products,
// 55 us with split ones).  NT: terms of a staged operand.  D: head size (columns of the contraction).
template <bool SPLIT, int NT, int D>
struct BlockOps {
  static_assert(SPLIT || NT == 1, "FP32 products: the values themselves");
  // row stride (in 16 bits) of a term: an odd number of 16-byte pieces
  static constexpr int LDK = SPLIT ? (D + 31) / 32 * 32 + 8 : 2 * D + 8;
  static constexpr int STEP = SPLIT ? 2 : 1;           // accumulator tiles of one step of a contraction over columns
  static constexpr int TERM = C * LDK;                 // one term of 16 tokens
  static constexpr int SIZE = NT * TERM;

  // four elements of a token's row (j0 a multiple of 4)
  static __device__ __forceinline__ void put4(uint16_t* dst, int row, int j0, f4 x) {
    const int at = row * LDK + kslot(j0);
    if constexpr (!SPLIT) {
      *reinterpret_cast<f4*>(&dst[row * LDK + 2 * j0]) = x;
    } else if constexpr (NT == 1) {   // bf16 numbers: the low halves are zero
      *reinterpret_cast<u2*>(&dst[at]) = u2{pack_tops(x[0], x[1]), pack_tops(x[2], x[3])};
    } else {
      u2 h, m, l;
      split3_rne(x, h, m, l);
      *reinterpret_cast<u2*>(&dst[at]) = h;
      *reinterpret_cast<u2*>(&dst[TERM + at]) = m;
      *reinterpret_cast<u2*>(&dst[2 * TERM + at]) = l;
    }
  }
  // the same element of four tokens' rows (column j of rows row0 .. row0 + 3)
  static __device__ __forceinline__ void put_column(uint16_t* dst, int row0, int j, f4 x) {
    if constexpr (!SPLIT) {
#pragma unroll
      for (int r = 0; r < 4; ++r) *reinterpret_cast<float*>(&dst[(row0 + r) * LDK + 2 * j]) = x[r];
    } else {
      static_assert(NT == 3 || !SPLIT, "float32 values");
      u2 t[3];
      split3_rne(x, t[0], t[1], t[2]);
      const int at = row0 * LDK + kslot(j & ~3) + (j & 3);
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          dst[i * TERM + at + r * LDK] = static_cast<uint16_t>(r % 2 ? t[i][r / 2] >> 16 : t[i][r / 2] & 0xffffu);
    }
  }
  // one element back (the terms sum to it exactly)
  static __device__ __forceinline__ float get(const uint16_t* src, int row, int j) {
    if constexpr (!SPLIT) return *reinterpret_cast<const float*>(&src[row * LDK + 2 * j]);
    const int at = row * LDK + kslot(j & ~3) + (j & 3);
    float x = bf16_to_f32(src[at]);
    if constexpr (NT == 3) x = (bf16_to_f32(src[2 * TERM + at]) + bf16_to_f32(src[TERM + at])) + x;
    return x;
  }
  // operand of the 16 tokens (token c on lane c), columns 16 STEP kb onwards (16 bytes at group g either way)
  static __device__ __forceinline__ Terms<NT> operand(const uint16_t* src, int kb, int c, int g) {
    Terms<NT> x;
#pragma unroll
    for (int i = 0; i < NT; ++i) x.t[i] = *reinterpret_cast<const u4*>(&src[i * TERM + c * LDK + 32 * kb + 8 * g]);
    return x;
  }
  // its columns 16 b .. 16 b + 15
  static __device__ __forceinline__ HalfTerms<NT> half_operand(const uint16_t* src, int b, int c, int g) {
    HalfTerms<NT> x;
#pragma unroll
    for (int i = 0; i < NT; ++i)
      x.t[i] = *reinterpret_cast<const u2*>(&src[i * TERM + c * LDK + 32 * (b >> 1) + 8 * g + 4 * (b & 1)]);
    return x;
  }
  // two accumulator tiles (one without the split) as the other operand
  static __device__ __forceinline__ auto tiles(f4 x0, f4 x1) {
    if constexpr (SPLIT) return split_tiles(x0, x1);
    else return x0;
  }
  template <typename X>
  static __device__ __forceinline__ f4 sweep(const Terms<NT>& a, const X& b, f4 acc) {
    if constexpr (SPLIT) {
      return mfma_terms(a, b, acc);
    } else {
      const f4 xa = __builtin_bit_cast(f4, a.t[0]);
      f4 xb;
      if constexpr (sizeof(X) == sizeof(f4)) xb = __builtin_bit_cast(f4, b);
#pragma unroll
      for (int r = 0; r < 4; ++r) acc = mfma16(xa[r], xb[r], acc);
      return acc;
    }
  }
  // The LDS image of a [D][16 tokens] matrix W (hm [4 D], l [4 D]) and updates X += W y, four tokens of y per lane
  static __device__ __forceinline__ void w_store(u4* hm, u2* l, int row, int c, int g, f4 x) {
    if constexpr (SPLIT) tok_store(hm, l, row, c, g, x);
    else hm[4 * row + tok_chunk(c, g)] = __builtin_bit_cast(u4, x);
  }
  static __device__ __forceinline__ auto w_load(const u4* hm, const u2* l, int row, int c, int g) {
    if constexpr (SPLIT) return tok_load(hm, l, row, c, g);
    else return __builtin_bit_cast(f4, hm[4 * row + tok_chunk(c, g)]);
  }
  static __device__ __forceinline__ auto tokens_b(f4 x) {
    if constexpr (SPLIT) return tok_b(x);
    else return x;
  }
  template <typename WA, typename Y>
  static __device__ __forceinline__ f4 update(const WA& wa, const Y& y, f4 acc) {
    if constexpr (SPLIT) {
      return mfma_tok(wa, y, acc);
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) acc = mfma16(wa[r], y[r], acc);
      return acc;
    }
  }
  // A -= W W^T on this wave's columns: a(b, j) is row tile b < N, column tile j < NJ; wrow0 the W row of its column 0.
  //
  // Split: where products are small against the accumulator the bf16 instruction cuts them off some eight bits below
  // its last place, towards minus infinity.  Accumulated into A that is 0.013 to 0.028 units per element and block,
  // always the same way, and A k^ of keys with a common direction (all-positive ones) is small by cancellation and
  // gathers it: heads of 128, mapped keys, T = 2500: error of S against float64 5.0e-6, with FP32 products 1.6e-6.  So
  // the products of an element are summed by themselves and added once (the cut is then 0.009 units of that sum), with
  // the sign of the product alternating from block to block, which cancels it: 0.9e-6.  S has no such small directions
  // and is accumulated into.  Rounding of an update: 0.29 units (root mean square); 0.82 accumulated, 1.15 in FP32.
  // Cost, large batch (2048 heads of 128, T = 8192, bf16): 16.4 -> 17.2 ms.
  template <int N, int NJ, bool TIGHT = false, typename X>
  static __device__ __forceinline__ void downdate(const u4* hm, const u2* l, int wrow0, int c, int g, bool odd_block,
                                                  X&& a) {
    if constexpr (SPLIT) {
      const uint32_t flip = odd_block ? 0u : 0x80008000u;
      const float sign = odd_block ? -1.0f : 1.0f;
      TokB y[NJ];
#pragma unroll
      for (int j = 0; j < NJ; ++j) y[j] = tok_image_b(hm, l, wrow0 + 16 * j, c, g, flip);
      // row tiles at a time in registers; one where two column tiles and three-term operands leave no more
      constexpr int GROUP = ((D >= 128 && NT == 3 && NJ > 1) || TIGHT) ? 1 : 2;
#pragma unroll
      for (int b0 = 0; b0 < N; b0 += GROUP) {
        f4 sum[GROUP][NJ];
#pragma unroll
        for (int i = 0; i < GROUP; ++i) {
          const TokA wa = tok_load(hm, l, 16 * (b0 + i) + c, c, g);
#pragma unroll
          for (int j = 0; j < NJ; ++j) sum[i][j] = mfma_tok(wa, y[j], f4{0, 0, 0, 0});
        }
#pragma unroll
        for (int i = 0; i < GROUP; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j) {
            f4& t = a(b0 + i, j);
#pragma unroll
            for (int r = 0; r < 4; ++r) t[r] = fmaf(sign, sum[i][j][r], t[r]);
            asm volatile("" : "+v"(t));   // in the old value's registers: there are none for a second copy of A
          }
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
      f4 y[NJ];
#pragma unroll
      for (int j = 0; j < NJ; ++j) y[j] = -__builtin_bit_cast(f4, hm[4 * (wrow0 + 16 * j) + tok_chunk(c, g)]);
#pragma unroll
      for (int b = 0; b < N; ++b) {
        const f4 wa = __builtin_bit_cast(f4, hm[4 * (16 * b + c) + tok_chunk(c, g)]);
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          // summed apart as well: one rounding of A instead of four (heads of 64, mapped keys, T = 2500, error of S:
          // 1.67e-6 accumulated); d = 16 is bound by this chain and has few columns to gather it
          if constexpr (D > 16) a(b, j) += update(wa, y[j], f4{0, 0, 0, 0});
          else a(b, j) = update(wa, y[j], a(b, j));
        }
      }
    }
  }
};

__device__ __forceinline__ f4 lds4(const float* p) { return *reinterpret_cast<const f4*>(p); }

// Sum over the 16 lanes of a DPP row; every lane of the row gets the total.
__device__ __forceinline__ float row_sum16(float x) {
  x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xB1, 0xf, 0xf, true));   // quad_perm [1,0,3,2]
  x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x4E, 0xf, 0xf, true));   // quad_perm [2,3,0,1]
  x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x141, 0xf, 0xf, true));  // row_half_mirror
  x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x140, 0xf, 0xf, true));  // row_mirror
  return x;
}

// acc += x[lane L of this 16-lane row] * y   -- one VALU instruction (DPP row broadcast folded into the FMA)
template <int L>
__device__ __forceinline__ void fmac_row_bcast(float& acc, float x, float y) {
  asm volatile("v_fmac_f32_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf bound_ctrl:1"
               : "+v"(acc)
               : "v"(x), "v"(y), "n"(L));
}
// x[lane L of this 16-lane row] * y
template <int L>
__device__ __forceinline__ float mul_row_bcast(float x, float y) {
  float r;
  asm volatile("v_mul_f32_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf bound_ctrl:1"
               : "=v"(r)
               : "v"(x), "v"(y), "n"(L));
  return r;
}

// Forward substitution for Z = (I + N)^{-1}, N strictly lower triangular, columns on lanes:
// on entry nm[s] holds, in lane t of every 16-lane row, -N[t][s]; on exit Z[t] = Z[t][c] in lane c.
// Row t needs N[t][s] in every lane: that is lane t's own register, broadcast by DPP inside the FMA.
template <int T_, int S_>
struct ZRow {
  static __device__ __forceinline__ void run(const float (&nm)[C], const float (&Z)[C], float& acc) {
    if constexpr (S_ < T_) {
      fmac_row_bcast<T_>(acc, nm[S_], Z[S_]);
      ZRow<T_, S_ + 1>::run(nm, Z, acc);
    }
  }
};
template <int T_>
__device__ __forceinline__ void z_rows(const float (&nm)[C], float (&Z)[C], int c) {
  if constexpr (T_ < C) {
    float acc = (c == T_) ? 1.0f : 0.0f;
    ZRow<T_, 0>::run(nm, Z, acc);
    Z[T_] = acc;
    z_rows<T_ + 1>(nm, Z, c);
  }
}
// nm[s] = m[s] * ncs[lane s of the row]  for s = 0..C-1   (ncs = -c_s, lane-distributed)
template <int S_>
__device__ __forceinline__ void scale_cols(const float (&m)[C], float (&nm)[C], float ncs) {
  if constexpr (S_ < C) {
    nm[S_] = mul_row_bcast<S_>(ncs, m[S_]);
    scale_cols<S_ + 1>(m, nm, ncs);
  }
}

// ---- Triangular work on a 16 x 16 tile by one wave, four columns at a time.  The tile sits in the accumulator layout
// (lane l = 16g + c, register r: element [4g + r][c]), so that the rows 4P .. 4P + 3 of a panel are the four registers of the
// 16 lanes g = P: inside the panel every coefficient is a DPP broadcast within those lanes (the other lanes compute values
// that nothing reads), and the rows after it take their rank-4 update from one v_mfma_f32_16x16x4_f32.
//
// Bound by one wave's issue (a vector instruction about every 6 cycles, 8 where it waits for the one before) and the chain
// of 16 pivots.  The factorisation takes some 190 instructions and 1460 cycles; with a column of L and L^{-1} per register
// and v_readlane broadcasts it took 430 and 2220, and scaled only at the end (rcp in the chain) 1630.  Z: 70 instructions
// against 300 with DPP multiply-adds.  Same bits.  256 heads of 64, float32, 2048 tokens 0.402 -> 0.353 ms; 16 heads of 64,
// 4096 tokens 0.147 -> 0.139; 2048 heads of 64, 8192 tokens, bf16 5.78 -> 5.60, of 128 15.72 -> 15.55.
// x[lane L of this row of 16 lanes]
template <int L>
__device__ __forceinline__ float row_bcast(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x150 + L, 0xf, 0xf, true));
}
// x[g] of the lanes 16P + c, on lane 16g + c: the four rows of a panel as one operand register
template <int P>
__device__ __forceinline__ float panel_operand(float x0, float x1, float x2, float x3) {
  auto swap16 = [](float& a, float& b) __attribute__((always_inline)) {   // odd rows of lanes of a, even ones of b
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
  };
  swap16(x0, x1);
  swap16(x2, x3);
  const auto r = P % 2 == 0 ? __builtin_amdgcn_permlane32_swap(__float_as_uint(x0), __float_as_uint(x2), false, false)
                            : __builtin_amdgcn_permlane32_swap(__float_as_uint(x1), __float_as_uint(x3), false, false);
  return __uint_as_float(r[P / 2]);
}
// One panel of cholesky16: m is what the earlier panels left of the matrix, n of the identity.  The panel's rows of L^T
// and L^{-1} go to LDS; m and n take the update (rows up to the panel's last are not read again).
template <int P, bool WITH_L>
__device__ __forceinline__ void cholesky_panel(f4& m, f4& n, float* L, float* Linv, int c, int g) {
  const float r0 = __builtin_amdgcn_rsqf(row_bcast<4 * P>(m[0]));   // 1 ulp; the pivots are delta_t >= 1
  const float l10 = row_bcast<4 * P + 1>(m[0]) * r0, u0 = m[0] * r0;
  float u1 = fmaf(-l10, u0, m[1]);
  const float l20 = row_bcast<4 * P + 2>(m[0]) * r0, l30 = row_bcast<4 * P + 3>(m[0]) * r0;
  const float r1 = __builtin_amdgcn_rsqf(row_bcast<4 * P + 1>(u1));
  const float l21 = row_bcast<4 * P + 2>(u1) * r1, l31 = row_bcast<4 * P + 3>(u1) * r1;
  float u2 = fmaf(-l20, u0, m[2]);
  u1 *= r1;
  u2 = fmaf(-l21, u1, u2);
  const float r2 = __builtin_amdgcn_rsqf(row_bcast<4 * P + 2>(u2));
  const float l32 = row_bcast<4 * P + 3>(u2) * r2;
  float u3 = fmaf(-l31, u1, fmaf(-l30, u0, m[3]));
  u2 *= r2;
  u3 = fmaf(-l32, u2, u3);
  const float r3 = __builtin_amdgcn_rsqf(row_bcast<4 * P + 3>(u3));
  u3 *= r3;
  const float u = panel_operand<P>(u0, u1, u2, u3);   // L[c][4P + g]
  if constexpr (P < 3) m = mfma16(-u, u, m);
  const float v0 = n[0] * r0;
  const float v1 = fmaf(-l10, v0, n[1]) * r1;
  const float v2 = fmaf(-l21, v1, fmaf(-l20, v0, n[2])) * r2;
  const float v3 = fmaf(-l32, v2, fmaf(-l31, v1, fmaf(-l30, v0, n[3]))) * r3;
  const float v = panel_operand<P>(v0, v1, v2, v3);   // L^{-1}[4P + g][c]
  if constexpr (P < 3) n = mfma16(-u, v, n);
  if constexpr (WITH_L) L[c * LT + 4 * P + g] = u;
  Linv[(4 * P + g) * LT + c] = v;
}
// m = I + G -> L [t][s] (row stride LT; only s <= t is meaningful) and L^{-1} [t][s] (zero above the diagonal).  Reads the
// elements [t][s], s <= t, of m's transpose.
template <bool WITH_L = true>
__device__ __forceinline__ void cholesky16(f4 gram, float* L, float* Linv, int c, int g) {
  f4 n;
#pragma unroll
  for (int r = 0; r < 4; ++r) n[r] = 4 * g + r == c ? 1.0f : 0.0f;
  f4 m = gram + n;
  cholesky_panel<0, WITH_L>(m, n, L, Linv, c, g);
  cholesky_panel<1, WITH_L>(m, n, L, Linv, c, g);
  cholesky_panel<2, WITH_L>(m, n, L, Linv, c, g);
  cholesky_panel<3, WITH_L>(m, n, L, Linv, c, g);
}
// Z = (I + N)^{-1}, N = strict_lower(X) diag(c), X [t][s] in LDS (row stride LT), cs: c_t on lane t of every 16 lanes;
// put(t, s, z): z = Z[t][s].  row[r] = -N[c][4g + r], col[p] = -N[c][4p + g]; what they hold on and above the diagonal is not used.
template <int P, typename F>
__device__ __forceinline__ void lower_inverse_panel(f4& x, f4 row, float col, int c, int g, F&& put) {
  const float x0 = x[0];
  const float x1 = fmaf(row_bcast<4 * P + 1>(row[0]), x0, x[1]);
  const float x2 = fmaf(row_bcast<4 * P + 2>(row[1]), x1, fmaf(row_bcast<4 * P + 2>(row[0]), x0, x[2]));
  const float x3 = fmaf(row_bcast<4 * P + 3>(row[2]), x2,
                        fmaf(row_bcast<4 * P + 3>(row[1]), x1, fmaf(row_bcast<4 * P + 3>(row[0]), x0, x[3])));
  const float z = panel_operand<P>(x0, x1, x2, x3);
  if constexpr (P < 3) x = mfma16(col, z, x);
  put(4 * P + g, c, z);
}
template <typename F>
__device__ __forceinline__ void lower_inverse16(const float* X, float cs, int c, int g, F&& put) {
  f4 row = lds4(&X[c * LT + 4 * g]);
  float col[3];
#pragma unroll
  for (int p = 0; p < 3; ++p) col[p] = X[c * LT + 4 * p + g];
#pragma unroll
  for (int r = 0; r < 4; ++r) row[r] *= -__shfl(cs, 4 * g + r);
#pragma unroll
  for (int p = 0; p < 3; ++p) col[p] *= -__shfl(cs, 4 * p + g);
  f4 x;
#pragma unroll
  for (int r = 0; r < 4; ++r) x[r] = 4 * g + r == c ? 1.0f : 0.0f;
  lower_inverse_panel<0>(x, row, col[0], c, g, put);
  lower_inverse_panel<1>(x, row, col[1], c, g, put);
  lower_inverse_panel<2>(x, row, col[2], c, g, put);
  lower_inverse_panel<3>(x, row, 0.0f, c, g, put);
}

// For kernels without registers to spare: the masks and offsets of the two functions above are formed where they are called,
// not kept over the block loop.
struct Lane { int c, g; };
// (With their ranges, so that products with them are shifts and 24-bit ones: v_mul_lo_u32 takes four times as long.)
__device__ __forceinline__ void renew(int& c, int& g) {
  asm volatile("" : "+v"(c), "+v"(g));
  __builtin_assume(c >= 0 && c < 16);
  __builtin_assume(g >= 0 && g < 4);
}
__device__ __forceinline__ Lane fresh_lane(int c, int g) {
  renew(c, g);
  return Lane{c, g};
}

__device__ __forceinline__ void io_store(float* p, float x) { *p = x; }
__device__ __forceinline__ void io_store(uint16_t* p, float x) { *p = f32_to_bf16_rne(x); }
// Two values to two addresses.  For bf16 the pair is rounded (to nearest even) by one packed hardware
// conversion and the halves are stored separately.
__device__ __forceinline__ void io_store2(float* p0, float* p1, float x0, float x1) {
  *p0 = x0;
  *p1 = x1;
}
__device__ __forceinline__ void io_store2(uint16_t* p0, uint16_t* p1, float x0, float x1) {
  typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
  typedef float fl2 __attribute__((ext_vector_type(2)));
  const uint32_t u = __builtin_bit_cast(uint32_t, __builtin_convertvector(fl2{x0, x1}, bf2));
  *p0 = static_cast<uint16_t>(u & 0xffffu);
  *p1 = static_cast<uint16_t>(u >> 16);
}

// A staged row segment of EPT consecutive elements, held in its raw (packed) form until it is used.
template <typename IO, int EPT> struct RawRow;
template <int EPT> struct RawRow<float, EPT> {
  static_assert(EPT % 4 == 0, "whole 16-byte pieces");
  float4 v[EPT / 4];
  __device__ __forceinline__ void load(const float* p) {
#pragma unroll
    for (int e = 0; e < EPT / 4; ++e) v[e] = *reinterpret_cast<const float4*>(p + 4 * e);
  }
  // F = float, or double (every float32 value is a float64 value)
  template <typename F>
  __device__ __forceinline__ void unpack(F (&x)[EPT]) const {
#pragma unroll
    for (int e = 0; e < EPT / 4; ++e) {
      x[4 * e] = v[e].x; x[4 * e + 1] = v[e].y; x[4 * e + 2] = v[e].z; x[4 * e + 3] = v[e].w;
    }
  }
};
template <int EPT> struct RawRow<uint16_t, EPT> {
  static_assert(EPT % 4 == 0, "whole 8-byte pieces");
  static constexpr int PW = EPT % 8 == 0 ? 4 : 2;   // 32-bit words per load: 16-byte pieces, else 8-byte ones
  static constexpr int NP = EPT / (2 * PW);
  typedef uint32_t Piece __attribute__((ext_vector_type(PW)));
  Piece v[NP];
  __device__ __forceinline__ void load(const uint16_t* p) {
#pragma unroll
    for (int e = 0; e < NP; ++e) v[e] = *reinterpret_cast<const Piece*>(p + 2 * PW * e);
  }
  template <typename F>
  __device__ __forceinline__ void unpack(F (&x)[EPT]) const {
#pragma unroll
    for (int e = 0; e < NP; ++e) {
#pragma unroll
      for (int i = 0; i < PW; ++i) {
        const uint32_t u = v[e][i];
        x[2 * (PW * e + i)] = __uint_as_float(u << 16);
        x[2 * (PW * e + i) + 1] = __uint_as_float(u & 0xffff0000u);
      }
    }
  }
};
// ELU(x) + 1, the feature map of Section 3.3
__device__ __forceinline__ float elu_plus_one(float x) { return x > 0.0f ? x + 1.0f : __expf(x); }

__device__ __forceinline__ float widen(float x) { return x; }
__device__ __forceinline__ float widen(uint16_t x) { return bf16_to_f32(x); }
// -x widened to float32: for bf16 the shift and the sign flip are one shift-and-add (adding the top bit is
// flipping it).
__device__ __forceinline__ float neg_widen(float x) { return -x; }
__device__ __forceinline__ float neg_widen(uint16_t x) {
  return __uint_as_float((static_cast<uint32_t>(x) << 16) + 0x80000000u);
}

}  // namespace vla
