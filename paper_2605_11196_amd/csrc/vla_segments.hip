// State at the boundaries of time segments, for the time-parallel mode.
//
// Without the identity refresh the inverse penalty matrix is an explicit inverse (paper Section 3.2 and
// eq. (penalty); eq. (sm) is the Sherman-Morrison form of it):  A_t = (A_0^{-1} + sum_{s<=t} u_s u_s^T)^{-1}, with
// u_s = k^_s by default or the caller's penalty directions, normalised and scaled.  The sum is a plain prefix
// sum, so A at the start of every segment follows from one Gram matrix per segment and one d x d inversion, all
// independent of each other; the segments then run the exact rank-1 recurrence concurrently.  The paper
// treats the A loop as sequential (Section 3.4); this goes beyond it and is not valid with the identity
// refresh.  The directions are the float32 numbers the recurrence kernels work with; their outer products (exact
// in float64) and the sums are float64, or, where that cannot show (fixed_point_gram), fixed point; the inversions are
// float64.  So the boundary matrices are at least as accurate as the float32 chain they replace.
//
// The S recurrence is affine in S (eq. (s-update)): S_end = S_start P + Q per segment.  P and Q come from the waves beside the
// A chain (vla_a_map.hip), with options from the map pass of the S-rows kernel (vla_two_phase.hip); combine_kernel composes them
// from left to right.
#include "vla_mfma_util.h"
#include <math.h>

#include <type_traits>

namespace vla {
namespace {

constexpr int kThreads = 256;

// ------------------------------------------------------------------------------------------ Gram
typedef double d4 __attribute__((ext_vector_type(4)));

// One workgroup (4 waves) per (head, segment); the last segment's matrix is never needed.  Tokens are
// normalised in float32, exactly as the kernels that run the recurrence normalise them (the sum is over the
// directions those kernels use, float32 numbers), and staged through LDS 64 at a time (32 at d = 128); the outer
// products run on the float64 matrix cores (v_mfma_f64_16x16x4_f64: lane l supplies A[i = l % 16][k = l / 16] and
// B[k = l / 16][j = l % 16] and receives D[i = l / 16 + 4 r][j = l % 16] in element r), both operands being the
// same staged tile widened as it is read: a product of two float32 values is exact in float64.  A wave
// holds at most 16 result tiles: up to D = 64 every wave covers the whole matrix and the waves take the
// tokens of a tile in turn (summed through LDS at the end); at D = 128 wave w owns the tile rows w and
// DL/16 - 1 - w from the diagonal on (DL/16 + 1 tiles whatever w: the sum is symmetric, the tiles below the
// diagonal are mirrored at the end).
// DL: the head size of the data; D >= DL: the size the tiles are laid out for.  They differ for d = 96, which
// runs in the d = 128 layout with the columns from 96 on held at zero (the loads, the staging and the final
// stores skip them; three of the four waves then form the products).
template <int D, int DL, typename IO>
__device__ __forceinline__ void gram_sum(const ForwardArgs& a, double* G) {
  static_assert(DL <= D && DL % 16 == 0, "padded layout");
  constexpr int NTI = D / 16;                                // tiles per side
  constexpr int TR = NTI * NTI <= 16 ? NTI : 16 / NTI;       // tile rows per wave
  constexpr int RGW = NTI / TR;                              // waves across the rows
  constexpr int NGW = (kThreads / 64) / RGW;                 // waves across the tokens
  constexpr int TT = D <= 64 ? 64 : 32;                      // tokens per tile
  constexpr int KS = TT / 4;                                 // k-steps (4 tokens) per tile
  constexpr int LDK = D + 16;                                // rows 16 banks apart: conflict-free operand reads
  constexpr int EPT = TT * D / kThreads;                     // elements of the tile each thread stages
  constexpr int TPR = D / EPT;                               // threads per token row
  static_assert(RGW * NGW * 64 == kThreads && KS % NGW == 0 && (TPR == 4 || TPR == 8) && EPT % 4 == 0, "layout");
  // The sum of k^ k^T is symmetric: only the tiles on and above the diagonal are formed (10 of 16 at d = 64,
  // 36 of 64 at d = 128).  Where a wave cannot hold the whole matrix the tile rows are paired so that every
  // wave has the same number of them.
  constexpr bool PAIR = RGW > 1;
  constexpr int NTL = DL / 16;                               // tile rows that hold data
  constexpr int NPT = NTL + 1;                               // tiles of a wave's pair of rows
  static_assert(PAIR ? (NTL % 2 == 0 && NTL / 2 <= RGW && NGW == 1) : (RGW == 1 && D == DL),
                "row w pairs with row NTL - 1 - w; otherwise every wave covers the whole matrix");
  __shared__ __align__(16) float ktb[2][TT * LDK];   // double-buffered: one barrier per tile
  static_assert(NGW == 1 || 2 * TT * LDK * sizeof(float) >= D * D * sizeof(double),
                "the final sum over the waves reuses the tile buffers");
  double* const red = reinterpret_cast<double*>(&ktb[0][0]);

  const int head = blockIdx.x / a.n_seg;
  const int seg = blockIdx.x - head * a.n_seg;
  if (seg == a.n_seg - 1) return;
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int c = lane & 15;
  const int g = lane >> 4;
  const int tgrp = w / RGW;     // which k-steps
  const int tb = seg * a.seg_blocks * C;
  const int te = min(a.T, tb + a.seg_blocks * C);
  // the directions the penalty matrix accumulates: the caller's u (scaled after normalisation), else the keys
  const bool has_u = a.u != nullptr;
  const IO* kh = static_cast<const IO*>(has_u ? a.u : a.k) + static_cast<size_t>(head) * static_cast<size_t>(a.T) * DL;
  const float eps = a.eps;
  const float scale = has_u ? a.u_scale : 1.0f;
  const int srow = tid / TPR;
  const int scol = (tid % TPR) * EPT;

  d4 acc[PAIR ? 1 : TR][PAIR ? 1 : NTI];   // every wave covers the whole matrix, or whole tile rows
  d4 pacc[PAIR ? NPT : 1];                 // paired rows: row w from its diagonal tile on, then row NTL - 1 - w
#pragma unroll
  for (int i = 0; i < (PAIR ? 1 : TR); ++i)
#pragma unroll
    for (int j = 0; j < (PAIR ? 1 : NTI); ++j) acc[i][j] = d4{0, 0, 0, 0};
#pragma unroll
  for (int i = 0; i < (PAIR ? NPT : 1); ++i) pacc[i] = d4{0, 0, 0, 0};

  // Fragments of the next PF tiles are kept in flight in raw form (a few registers each): with a thousand
  // workgroups streaming at once the memory latency is several tiles' worth of work.
  constexpr int PF = 2;   // what the register file allows next to the accumulator registers
  RawRow<IO, EPT> raw[PF];
  auto fetch = [&](int t0, RawRow<IO, EPT>& o) {
    const int t = t0 + srow;
    if (D == DL || scol < DL) o.load(kh + static_cast<size_t>(t < te ? t : te - 1) * DL + scol);
  };
  // stage: k^ = k / max(||k||, eps) as the recurrence kernels form it (float32: hardware reciprocal square
  // root, one Newton step); rows past the end are zero
  auto stage = [&](int t0, const RawRow<IO, EPT>& o, float* kt) {
    const int t = t0 + srow;
    float x[EPT];
    o.unpack(x);
    if (D != DL && scol >= DL) {
#pragma unroll
      for (int e = 0; e < EPT; ++e) x[e] = 0.0f;
    }
    if (a.feature_map && !has_u && (D == DL || scol < DL)) {   // ELU(x) + 1 on keys
#pragma unroll
      for (int e = 0; e < EPT; ++e) x[e] = elu_plus_one(x[e]);
    }
    float ss = 0.0f;
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      x[e] = t < te ? x[e] : 0.0f;
      ss = fmaf(x[e], x[e], ss);
    }
#pragma unroll
    for (int off = TPR / 2; off >= 1; off >>= 1) ss += __shfl_xor(ss, off);
    const float sm = fmaxf(ss, eps * eps);
    float rn = __builtin_amdgcn_rsqf(sm);
    rn = rn * fmaf(-0.5f * sm * rn, rn, 1.5f) * scale;
#pragma unroll
    for (int e = 0; e < EPT; e += 4)
      *reinterpret_cast<f4*>(&kt[srow * LDK + scol + e]) = f4{x[e] * rn, x[e + 1] * rn, x[e + 2] * rn, x[e + 3] * rn};
  };
  // paired rows, for the wave W (a compile-time copy of w): tiles (W, W..NTL-1) then (R1, R1..NTL-1)
  auto pair_products = [&](auto wtag, const float* kt) {
    constexpr int W = decltype(wtag)::value;
    constexpr int R1 = NTL - 1 - W;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      const float* row = &kt[(4 * kk + g) * LDK + c];
      double bv[NTL];
#pragma unroll
      for (int j = W; j < NTL; ++j) bv[j] = static_cast<double>(row[16 * j]);
#pragma unroll
      for (int j = W; j < NTL; ++j)
        pacc[j - W] = __builtin_amdgcn_mfma_f64_16x16x4f64(bv[W], bv[j], pacc[j - W], 0, 0, 0);
#pragma unroll
      for (int j = R1; j < NTL; ++j)
        pacc[NTL - W + j - R1] = __builtin_amdgcn_mfma_f64_16x16x4f64(bv[R1], bv[j], pacc[NTL - W + j - R1], 0, 0, 0);
    }
  };
  // element r of the tile (i, j) is G[16 i + g + 4 r][16 j + c]; its mirror image fills the tile (j, i)
  auto pair_store = [&](auto wtag, double* Gh) {
    constexpr int W = decltype(wtag)::value;
    constexpr int R1 = NTL - 1 - W;
    auto put = [&](int i, int j, const d4& t) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * i + g + 4 * r, col = 16 * j + c;
        Gh[row * DL + col] = t[r];
        if (j > i) Gh[col * DL + row] = t[r];
      }
    };
#pragma unroll
    for (int j = W; j < NTL; ++j) put(W, j, pacc[j - W]);
#pragma unroll
    for (int j = R1; j < NTL; ++j) put(R1, j, pacc[NTL - W + j - R1]);
  };
  // the wave's own copy of the two above (w is uniform over the wave)
  auto for_my_rows = [&](auto&& f) {
    if constexpr (PAIR) {
      if (w == 0) f(std::integral_constant<int, 0>{});
      if (w == 1 && NTL >= 4) f(std::integral_constant<int, (NTL >= 4 ? 1 : 0)>{});
      if (w == 2 && NTL >= 6) f(std::integral_constant<int, (NTL >= 6 ? 2 : 0)>{});
      if (w == 3 && NTL >= 8) f(std::integral_constant<int, (NTL >= 8 ? 3 : 0)>{});
    }
  };
  auto products = [&](const float* kt) {
    if constexpr (PAIR) {
      for_my_rows([&](auto wtag) { pair_products(wtag, kt); });
    } else {
#pragma unroll
      for (int kk = tgrp; kk < KS; kk += NGW) {
        const float* row = &kt[(4 * kk + g) * LDK + c];
        double bv[NTI];
#pragma unroll
        for (int j = 0; j < NTI; ++j) bv[j] = static_cast<double>(row[16 * j]);
#pragma unroll
        for (int i = 0; i < TR; ++i)
#pragma unroll
          for (int j = i; j < NTI; ++j)   // tiles below the diagonal are mirrored at the end
            acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(bv[i], bv[j], acc[i][j], 0, 0, 0);
      }
    }
  };
#pragma unroll
  for (int u = 0; u < PF; ++u)
    if (tb + u * TT < te) fetch(tb + u * TT, raw[u]);
  for (int t0 = tb; t0 < te; t0 += PF * TT) {
#pragma unroll
    for (int u = 0; u < PF; ++u) {
      const int tu = t0 + u * TT;
      if (tu < te) {   // uniform over the workgroup
        float* kt = ktb[u & 1];
        stage(tu, raw[u], kt);
        // the buffer written here was last read two tiles ago, and every wave has passed the barrier of the
        // tile in between since then
        __syncthreads();
        if (tu + PF * TT < te) fetch(tu + PF * TT, raw[u]);
        products(kt);
      }
    }
  }

  double* Gh = G + static_cast<size_t>(blockIdx.x) * DL * DL;
  if constexpr (PAIR) {
    for_my_rows([&](auto wtag) { pair_store(wtag, Gh); });
  } else {
    // element r of tile (i, j) is G[16 i + g + 4 r][16 j + c]; the waves' partial sums meet in LDS
    __syncthreads();   // every wave is done with the tile buffers
    for (int gi = 0; gi < NGW; ++gi) {
      if (tgrp == gi) {
#pragma unroll
        for (int i = 0; i < TR; ++i)
#pragma unroll
          for (int j = i; j < NTI; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int o = (16 * i + g + 4 * r) * D + 16 * j + c;
              red[o] = gi == 0 ? acc[i][j][r] : red[o] + acc[i][j][r];
            }
      }
      __syncthreads();
    }
    for (int o = tid; o < D * D; o += kThreads) {
      const int row = o / D, col = o - row * D;
      Gh[o] = row / 16 > col / 16 ? red[col * D + row] : red[o];   // tile below the diagonal: mirror
    }
  }
}

// ---- The same sums in fixed point on the 8-bit integer matrix instruction.
//
// A direction of length at most 2^E (1 for keys) is rounded to a multiple of 2^(E - 30), an error of at most 2^(E - 31) in an
// element (float32 keeps elements from 2^(E - 7) on exactly so), and written as four signed base-256 digits, X = sum a_i 256^i.  The
// products of digits and their sums over the tokens are exact in 32-bit integers; those of weight 256 and more are formed (15 of
// 16), one sum per weight, and put together in float64 every kChunk tokens, before a sum can overflow.  What is left out, the product
// of the lowest digits, is at most 2^-46 of a token's product of two units, but not a token's alone: the same direction
// over and over leaves out the same each time, off that direction, where lambda0 is all there is.  (Without the two
// products of weight 256 too: one unit key 131072 times, lambda0 = 0.1, A wrong by 8e-6; with them 2e-8, with all 16 1e-10.)
//
// One workgroup per (head, segment).  A thread stages four tokens x four columns: the digits of a column's four
// tokens are transposed in its registers (8 byte permutations) into LDS planes [digit][column][token], from which a lane
// reads the 16 tokens of an operand as 16 bytes.  A plane's rows and their 16-byte pieces are permuted by the column (row()
// and piece()), so that neither the writes nor the reads hit a bank twice.  Tiles on and above the diagonal only, shared out by
// tile rows.
//
// Bound by the staging's vector instructions (about 10 an element) beside 15 matrix ones per tile and 64 tokens.  16 heads of 64,
// 131072 tokens, bf16: 195 us in float64 (v_mfma_f64_16x16x4_f64, 64 cycles each), 119 here (13 products 114, 16 122); 16 heads of
// 128, 32768 tokens 188 and 95 (13 products 89, 16 104).  D = 64 keeps three workgroups per compute unit, though some registers spill:
// with two, 320 heads, 512 tokens, 960 workgroups, the whole call 178 -> 188 us.
typedef int i4 __attribute__((ext_vector_type(4)));

constexpr int fixed_threads(int d) { return d >= 96 ? 512 : 256; }

template <int D, typename IO>
__global__ void __launch_bounds__(fixed_threads(D), D >= 96 ? 2 : 3) gram_fixed_kernel(ForwardArgs a, double* G, int shift) {
  constexpr int NS = D / 16;                        // column strips
  constexpr int KG = D == 32 ? 2 : 1;               // waves across the tokens of a tile
  constexpr int TT = 64 * KG;                       // tokens of a tile
  constexpr int LPR = D == 32 ? 8 : D == 64 ? 16 : 32;   // threads across a token's row
  constexpr int W32 = TT / 4;                       // words of a plane's row
  constexpr int kLowest = 1;                        // weight of the smallest products that are formed
  constexpr int kSums = 7 - kLowest;
  constexpr int kChunk = 16384;                     // tokens whose sums (at most four products of 2^14 each) fit 31 bits
  static_assert(fixed_threads(D) / LPR * 4 == TT && D / 4 <= LPR, "one cell of 4 x 4 per thread");
  __shared__ __align__(16) uint32_t planes[2][4][D * W32];

  const int head = blockIdx.x / a.n_seg;
  const int seg = blockIdx.x - head * a.n_seg;
  if (seg == a.n_seg - 1) return;                   // the last segment's matrix is never needed
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int c = lane & 15;
  const int g = lane >> 4;
  const int tb = seg * a.seg_blocks * C;
  const int te = min(a.T, tb + a.seg_blocks * C);
  const bool has_u = a.u != nullptr;
  const IO* kh = static_cast<const IO*>(has_u ? a.u : a.k) + static_cast<size_t>(head) * static_cast<size_t>(a.T) * D;
  const bool fmap = a.feature_map != 0 && !has_u;
  const float eps = a.eps;
  const float scale = has_u ? a.u_scale : 1.0f;
  const int cg = tid % LPR, tg = tid / LPR;         // column group and token group of this thread
  const bool in_row = D / 4 == LPR || cg < D / 4;
  auto row = [](int col) { return (col & ~3) | ((col ^ (col >> 2)) & 3); };
  auto piece = [](int col, int tq) { return tq ^ ((col >> 2) & 3) ^ ((col >> 4) & 3); };   // tq: 16 tokens

  constexpr int PF = 2;   // tiles in flight
  RawRow<IO, 4> raw[PF][4];
  auto fetch = [&](int t0, RawRow<IO, 4> (&o)[4]) {
    if (!in_row) return;
    const IO* base = kh + static_cast<size_t>(t0) * D + 4 * cg;
    const int lim = te - 1 - t0;
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i].load(base + static_cast<unsigned>((lim >= TT - 1 ? 4 * tg + i : min(4 * tg + i, lim)) * D));
  };
  bool bad = false;   // a direction that is not finite: the matrix is none
  auto stage = [&](int t0, const RawRow<IO, 4> (&o)[4], uint32_t (&pl)[4][D * W32]) {
    uint32_t word[4][4];   // [column][token]
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float x[4];
      if (in_row) {
        o[i].unpack(x);
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] = 0.0f;
      }
      if (fmap && in_row) {
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] = elu_plus_one(x[j]);
      }
      if (t0 + TT > te) {   // uniform: rows past the end are zero
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] = t0 + 4 * tg + i < te ? x[j] : 0.0f;
      }
      float ss = 0.0f;
#pragma unroll
      for (int j = 0; j < 4; ++j) ss = fmaf(x[j], x[j], ss);
      if constexpr (LPR >= 16) ss = row_sum16(ss);
      if constexpr (LPR == 32) ss += __shfl_xor(ss, 16);
      if constexpr (LPR == 8) {
#pragma unroll
        for (int off = 4; off >= 1; off >>= 1) ss += __shfl_xor(ss, off);
      }
      // 1 / max(||k||, eps): hardware reciprocal square root, one Newton step, as the recurrence kernels form it
      const float sm = fmaxf(ss, eps * eps);
      float rn = __builtin_amdgcn_rsqf(sm);
      rn = rn * fmaf(-0.5f * sm * rn, rn, 1.5f) * scale;
      bad = bad || !(ss < __builtin_inff()) || !(fabsf(rn) < __builtin_inff());
      const float fixed = __builtin_ldexpf(rn, shift);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        int X;   // to the nearest integer
        asm("v_cvt_rpi_i32_f32 %0, %1" : "=v"(X) : "v"(x[j] * fixed));
        word[j][i] = static_cast<uint32_t>(X) + 0x00808080u;   // the digits but the highest one plus 128
      }
    }
    if (!in_row) return;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t (&w)[4] = word[j];
      const uint32_t lo01 = __builtin_amdgcn_perm(w[1], w[0], 0x05010400u), hi01 = __builtin_amdgcn_perm(w[1], w[0], 0x07030602u);
      const uint32_t lo23 = __builtin_amdgcn_perm(w[3], w[2], 0x05010400u), hi23 = __builtin_amdgcn_perm(w[3], w[2], 0x07030602u);
      const int col = 4 * cg + j;
      const int at = row(col) * W32 + 16 * (tg >> 4) + 4 * piece(col, (tg >> 2) & 3) + (tg & 3);
      pl[0][at] = __builtin_amdgcn_perm(lo23, lo01, 0x05040100u) ^ 0x80808080u;
      pl[1][at] = __builtin_amdgcn_perm(lo23, lo01, 0x07060302u) ^ 0x80808080u;
      pl[2][at] = __builtin_amdgcn_perm(hi23, hi01, 0x05040100u) ^ 0x80808080u;
      pl[3][at] = __builtin_amdgcn_perm(hi23, hi01, 0x07060302u);
    }
  };

  auto body = [&](auto wtag) {
    constexpr int W = decltype(wtag)::value;
    // the tiles (i, j), i <= j, of wave W: D = 64: first row but its last tile; last column; (1, 1), (1, 2); (2, 2), (3, 3).  From
    // d = 96 the even or the odd columns of the rows W % 4 and NS - 1 - W % 4.  d = 32: the diagonal or (0, 1), for one half of the
    // tokens.
    auto mine = [](int i, int j) constexpr -> bool {
      if (i > j) return false;
      if (D == 32) return (i == j) == (W / 2 == 0);
      if (D == 64) return W == 0 ? i == 0 && j < 3 : W == 1 ? j == 3 && i < 3 : W == 2 ? i == 1 && j < 3 : i == j && i >= 2;
      return W % 4 < NS / 2 && (i == W % 4 || i == NS - 1 - W % 4) && j % 2 == W / 4;
    };
    constexpr int NT = D == 32 ? 2 : D == 64 ? 3 : NS / 2 + 1;   // at most
    i4 acc[NT][kSums];
    auto clear = [&]() {
#pragma unroll
      for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int k = 0; k < kSums; ++k) acc[n][k] = i4{0, 0, 0, 0};
    };
    struct Strip { i4 a[4]; };
    auto strip = [&](const uint32_t (&pl)[4][D * W32], int s) {
      const int col = 16 * s + c;
      const int at = row(col) * W32 + 16 * (KG > 1 ? W % KG : 0) + 4 * piece(col, g);
      Strip x;
#pragma unroll
      for (int l = 0; l < 4; ++l) x.a[l] = *reinterpret_cast<const i4*>(&pl[l][at]);
      return x;
    };
    auto products = [&](const uint32_t (&pl)[4][D * W32]) {
      Strip left[NS];
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        bool used = false;
#pragma unroll
        for (int j = i + 1; j < NS; ++j) used = used || mine(i, j);
        if (used) left[i] = strip(pl, i);
      }
      int n = 0;
#pragma unroll
      for (int j = 0; j < NS; ++j) {
        bool used = false;
#pragma unroll
        for (int i = 0; i <= j; ++i) used = used || mine(i, j);
        if (!used) continue;
        const Strip right = strip(pl, j);
#pragma unroll
        for (int i = 0; i <= j; ++i) {
          if (!mine(i, j)) continue;
          const Strip& x = i == j ? right : left[i];
#pragma unroll
          for (int la = 0; la < 4; ++la)
#pragma unroll
            for (int lb = 0; lb < 4; ++lb)
              if (la + lb >= kLowest)
                acc[n][la + lb - kLowest] = __builtin_amdgcn_mfma_i32_16x16x64_i8(x.a[la], right.a[lb], acc[n][la + lb - kLowest], 0, 0, 0);
          ++n;
        }
        __builtin_amdgcn_sched_barrier(0);   // one strip on the right at a time in registers
      }
    };
    double* Gh = G + static_cast<size_t>(blockIdx.x) * D * D;
    // the sums so far into G (added where an earlier chunk left its own)
    auto flush = [&](bool first, bool none) {
      double* half = reinterpret_cast<double*>(&planes[0][0][0]);   // d = 32: the other half of the tokens
      const double unit = __builtin_ldexp(1.0, 8 * kLowest - 2 * shift);
      int n = 0;
      if constexpr (KG > 1) __syncthreads();   // every wave is done with the planes
#pragma unroll
      for (int pass = 0; pass < KG; ++pass) {
        n = 0;
#pragma unroll
        for (int j = 0; j < NS; ++j)
#pragma unroll
          for (int i = 0; i <= j; ++i) {
            if (!mine(i, j)) continue;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              double v = static_cast<double>(acc[n][kSums - 1][r]);
#pragma unroll
              for (int k = kSums - 2; k >= 0; --k) v = fma(v, 256.0, static_cast<double>(acc[n][k][r]));
              v *= unit;
              const int ri = 16 * i + 4 * g + r, cj = 16 * j + c;
              if constexpr (KG > 1) {
                if (pass == 0 && W % KG == 1) half[ri * D + cj] = v;
                if (pass == 0 || W % KG == 1) continue;
                v += half[ri * D + cj];
              }
              if (!first) v += Gh[ri * D + cj];
              if (none) v = __builtin_nan("");
              Gh[ri * D + cj] = v;
              if (i != j) Gh[cj * D + ri] = v;
            }
            ++n;
          }
        if constexpr (KG > 1) __syncthreads();
      }
    };

    clear();
    bool first = true;
    int since = 0;   // tokens in the sums
#pragma unroll
    for (int u = 0; u < PF; ++u)
      if (tb + u * TT < te) fetch(tb + u * TT, raw[u]);
    for (int t0 = tb; t0 < te; t0 += PF * TT) {
#pragma unroll
      for (int u = 0; u < PF; ++u) {
        const int tu = t0 + u * TT;
        if (tu < te) {   // uniform over the workgroup
          stage(tu, raw[u], planes[u & 1]);
          // the planes written here were last read two tiles ago, and every wave has passed the barrier of the tile in between
          __syncthreads();
          if (tu + PF * TT < te) fetch(tu + PF * TT, raw[u]);
          products(planes[u & 1]);
        }
      }
      since += PF * TT;
      if (since >= kChunk && t0 + PF * TT < te) {
        flush(first, false);
        clear();
        first = false;
        since = 0;
      }
    }
    flush(first, __syncthreads_or(bad) != 0);
  };
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (w == 0) body(std::integral_constant<int, 0>{});
  if (w == 1) body(std::integral_constant<int, 1>{});
  if (w == 2) body(std::integral_constant<int, 2>{});
  if (w == 3) body(std::integral_constant<int, 3>{});
  if constexpr (D >= 96) {
    if (w == 4) body(std::integral_constant<int, 4>{});
    if (w == 5) body(std::integral_constant<int, 5>{});
    if (w == 6) body(std::integral_constant<int, 6>{});
    if (w == 7) body(std::integral_constant<int, 7>{});
  }
}

// Directions are shorter than 2^exponent.
int direction_exponent(const ForwardArgs& a) {
  int exponent = 0;
  if (a.u != nullptr && a.u_scale != 0.0f && isfinite(a.u_scale)) frexpf(a.u_scale, &exponent);
  return exponent;
}
// Calls that take it.  Its errors matter where A is far less certain than float32 can say; relative to the smallest eigenvalue
// of the penalty matrix they are, with r^2 = 4^exponent tokens / lambda0, at most about
//   r 2^-32           the rounding: one direction of length sqrt(lambda0 / tokens), rounded alike every time, or as much of one
//                     across the others
//   r^2 2^-60 5461 D  the lowest digits of one direction, left out alike every time (5461: the mean square of a digit)
// so r^2 is kept to 2^21, 3e-7 and 1e-6 (a matrix as a whole: 1e-7; Gaussian directions: 1e-10).  131072 tokens from the
// default lambda0 of 0.1 are inside, from 0.06 on.  u_scale = 1000, one direction so short that r counts, 65536 tokens, lambda0 = 0.01, was wrong by
// 4e-2 here.  A given A0, whose inverse has eigenvalues that nobody has looked at, keeps float64, and so does lambda0
// below 0.01, where nothing was measured.
bool fixed_point_gram(const ForwardArgs& a) {
  return a.A0 == nullptr && a.lambda0 >= 0.01f && ldexp(static_cast<double>(a.T), 2 * direction_exponent(a)) <= 2097152.0 * a.lambda0;
}

// In-place inclusive prefix sum of the Gram matrices over the segments of a head, one thread per element:
// afterwards G[h][s] = sum over segments 0..s.
__global__ void __launch_bounds__(kThreads) gram_prefix_kernel(double* G, int n_heads, int n_seg, int dd) {
  const long long e = static_cast<long long>(blockIdx.x) * kThreads + threadIdx.x;
  if (e >= static_cast<long long>(n_heads) * dd) return;
  const int head = static_cast<int>(e / dd);
  double* p = G + (static_cast<size_t>(head) * n_seg) * dd + (e - static_cast<long long>(head) * dd);
  double run = 0.0;
  const int n = n_seg - 1;   // the last segment's matrix is never needed
  // sixteen loads in flight at a time: the chain is as long as the memory latency times the trips it makes
  constexpr int U = 16;
  for (int s = 0; s < n; s += U) {
    double x[U];
#pragma unroll
    for (int i = 0; i < U; ++i) x[i] = s + i < n ? p[static_cast<size_t>(s + i) * dd] : 0.0;
#pragma unroll
    for (int i = 0; i < U; ++i) {
      run += x[i];
      if (s + i < n) p[static_cast<size_t>(s + i) * dd] = run;
    }
  }
}

// ------------------------------------------------------------------------------------------ key sums
// Normalised read-out (eq. (output)): zkey_t = zkey_0 + sum_{s<=t} k_s with k_s the key as used before its L2
// normalisation (after the feature map).  Per (head, segment) the sum of its keys, in float64; a thread adds eight
// consecutive columns of every RG-th token, the row groups are summed through LDS.
template <int D, typename IO>
__global__ void __launch_bounds__(kThreads) keysum_kernel(ForwardArgs a, double* part) {
  constexpr int EPT = 8;                 // consecutive columns per thread: one 16- or 32-byte piece of a row
  constexpr int TPR = D / EPT;           // threads per token row
  constexpr int RG = kThreads / TPR;     // rows in flight per pass (the last groups idle when 256 / TPR is no integer)
  __shared__ double red[RG][D];
  const int head = blockIdx.x / a.n_seg;
  const int seg = blockIdx.x - head * a.n_seg;
  const int rg = threadIdx.x / TPR;
  const int j0 = (threadIdx.x % TPR) * EPT;
  const int tb = seg * a.seg_blocks * C;
  const int te = min(a.T, tb + a.seg_blocks * C);
  const IO* kh = static_cast<const IO*>(a.k) + static_cast<size_t>(head) * static_cast<size_t>(a.T) * D;
  double sum[EPT];
#pragma unroll
  for (int e = 0; e < EPT; ++e) sum[e] = 0.0;
  if (rg < RG) {
    for (int t = tb + rg; t < te; t += RG) {
      RawRow<IO, EPT> raw;
      raw.load(kh + static_cast<size_t>(t) * D + j0);
      float x[EPT];
      raw.unpack(x);
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        if (a.feature_map) x[e] = elu_plus_one(x[e]);
        sum[e] += static_cast<double>(x[e]);
      }
    }
#pragma unroll
    for (int e = 0; e < EPT; ++e) red[rg][j0 + e] = sum[e];
  }
  __syncthreads();
  for (int j = threadIdx.x; j < D; j += kThreads) {
    double total = 0.0;
    for (int r = 0; r < RG; ++r) total += red[r][j];
    part[static_cast<size_t>(blockIdx.x) * D + j] = total;
  }
}
// seg_zkey[h][s] = zkey0[h] + the sums of the segments before s, one thread per (head, column)
__global__ void __launch_bounds__(kThreads) keysum_prefix_kernel(const double* part, const float* zkey0,
                                                                 float* seg_zkey, int n_heads, int n_seg, int d) {
  const long long e = static_cast<long long>(blockIdx.x) * kThreads + threadIdx.x;
  if (e >= static_cast<long long>(n_heads) * d) return;
  const int head = static_cast<int>(e / d);
  const int j = static_cast<int>(e - static_cast<long long>(head) * d);
  double run = zkey0 ? static_cast<double>(zkey0[e]) : 0.0;
  const size_t base = static_cast<size_t>(head) * n_seg * d + j;
  constexpr int U = 16;   // loads in flight
  for (int s = 0; s < n_seg; s += U) {
    double x[U];
#pragma unroll
    for (int i = 0; i < U; ++i) x[i] = s + i < n_seg ? part[base + static_cast<size_t>(s + i) * d] : 0.0;
#pragma unroll
    for (int i = 0; i < U; ++i) {
      if (s + i < n_seg) seg_zkey[base + static_cast<size_t>(s + i) * d] = static_cast<float>(run);
      run += x[i];
    }
  }
}

// ------------------------------------------------------------------------------------------ boundary
// Gauss-Jordan inverse, in place, of a symmetric positive definite D x D matrix spread over the workgroup's
// registers (no pivoting needed for such a matrix) in the result layout of the float64 matrix instruction, the tiles on and
// below the diagonal only: wave w holds the tile rows w and NTL - 1 - w, NTL + 1 tiles whatever w; lane (g, c) of it
// M[16 ti + g + 4 r][16 tj + c] of tile (ti, tj), tj <= ti, in element r.
//
// The sweep eliminates KB = 4 pivots at a time.  With P the pivot indices of a step, B = M[P][P], C = M[:, P]
// and R = M[P, :], the in-place step is  M <- M - C' R'  with
//   C'[i] = C[i] (i not in P),  C'[P] = B - I;     R'[:, j] = B^{-1} R[:, j] (j not in P),  R'[:, P] = I + B^{-1}
// which is the usual block sweep (Schur complement off the pivot rows and columns, -C B^{-1} in the pivot
// columns, B^{-1} R in the pivot rows, B^{-1} in the pivot block) written so that every element takes the same
// rank-4 update: one v_mfma_f64_16x16x4_f64 per 16 x 16 tile and step.  After the earlier steps the not yet eliminated part
// of M is a Schur complement (symmetric), the eliminated part is symmetric too, and an eliminated row is minus the transposed
// column: R[a][j] = C[j][a] for j after P and -C[j][a] for j before it, and likewise C[i][a] = -M[P_a][i] for i before P, which is
// where the upper triangle would be read.  The four pivot columns go through LDS: rows from the pivots' tile on out of that
// tile column, the rows before it out of the pivots' tile row (with the sign turned), the identity already subtracted from the
// pivot block; double-buffered, one barrier per step.
// Every lane factors the 4 x 4 block B = L diag(dd) L^T for itself in registers and solves for the one row of
// B^{-1} it needs (row g: a lane supplies R'[g][16 tj + c] as the B operand of column tile tj and C'[16 ti + c][g] as
// the A operand of row tile ti); the pivot columns get theirs from the identity x = e_e - B^{-1} e_e that the stored B - I gives
// them.
// Bound by the issue of a step's float64 instructions (2 x 2 blocks of B with half the reciprocals in the chain but more
// of the others: 41 -> 44 us).  One wave per SIMD and matrix of 128 (two, with the whole
// matrix on a wave per tile row, formed the factor and every x twice as often and twice the products): 234
// matrices of 128 57.6 -> 41.0 us, 39 given ones 54.9 -> 41.7; 256 of 64 14.7 -> 15.2.
// B - I and I + B^{-1} lose the small one of B and B^{-1} against the identity (an element d comes out as 1/d with a
// relative error of 1e-16 d^2), so the sweep runs on the matrix scaled by powers of two, row and column i by the one that
// brings the diagonal element i to [0.5, 2): 0.5 us of 51 (4 heads, 1024 tokens, d = 128).
template <int D>
struct SpdInverse {
  static constexpr int NTL = D / 16;        // tile rows and columns
  static constexpr int NW = NTL / 2;        // waves, two tile rows each
  static constexpr int NT = 64 * NW;        // threads
  static constexpr int NPT = NTL + 1;       // tiles of a wave
  static constexpr int KB = 4;              // pivots per step: the contraction length of the matrix instruction
  static constexpr int STRIDE = D;          // doubles per pivot column
  static constexpr int LDS_DOUBLES = 2 * KB * STRIDE + D / 2;
  static_assert(NTL % 2 == 0, "tile rows in pairs");
  double* colp;                             // LDS [2][KB][STRIDE], then the exponents of the scaling, int [D]
  static __device__ __forceinline__ double recip(double d) {   // hardware estimate refined twice: full precision
    const double y = __builtin_amdgcn_rcp(d);
    const double y1 = y * fma(-d, y, 2.0);
    return y1 * fma(-d, y1, 2.0);
  }
  // f(tile, row tile, column tile) for the tiles of wave W: row NTL - 1 - W first (from its column 0 on), then row W
  template <int W, typename F>
  static __device__ __forceinline__ void tiles(F&& f) {
#pragma unroll
    for (int tj = 0; tj < NTL - W; ++tj) f(tj, NTL - 1 - W, tj);
#pragma unroll
    for (int tj = 0; tj <= W; ++tj) f(NTL - W + tj, W, tj);
  }
  // the wave's own copy of body<W>() (w is uniform over the wave)
  template <typename F>
  static __device__ __forceinline__ void for_my_wave(F&& f) {
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (w == 0) f(std::integral_constant<int, 0>{});
    if (NW > 1 && w == 1) f(std::integral_constant<int, (NW > 1 ? 1 : 0)>{});
    if (NW > 2 && w == 2) f(std::integral_constant<int, (NW > 2 ? 2 : 0)>{});
    if (NW > 3 && w == 3) f(std::integral_constant<int, (NW > 3 ? 3 : 0)>{});
  }
  template <int W>
  __device__ __forceinline__ void run(d4 (&acc)[NPT]) const {
    constexpr int TI[2] = {NTL - 1 - W, W};   // the wave's tile rows
    const int lane = threadIdx.x & 63;
    const int c = lane & 15;
    const int g = lane >> 4;
    int* ex = reinterpret_cast<int*>(colp + 2 * KB * STRIDE);
    tiles<W>([&](int i, int ti, int tj) {
      if (ti != tj) return;
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (c == g + 4 * r) ex[16 * tj + c] = -(__builtin_amdgcn_frexp_exp(acc[i][r]) >> 1);
    });
    __syncthreads();
    // M <- E M E with the powers of two E; on the inverse of that it leaves the inverse of M
    auto scale = [&]() {
      tiles<W>([&](int i, int ti, int tj) {
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[i][r] = __builtin_amdgcn_ldexp(acc[i][r], ex[16 * tj + c] + ex[16 * ti + g + 4 * r]);
      });
    };
    scale();
#pragma unroll
    for (int tp = 0; tp < NTL; ++tp) {       // the tile row and column that hold the pivots
      for (int ps = 0; ps < 4; ++ps) {       // its columns 4 ps .. 4 ps + 3
        const int p0 = 16 * tp + KB * ps;
        double* cp = colp + (ps & 1) * (KB * STRIDE);
        // rows of tile tp and after it: this lane's column of tile (ti, tp) is pivot c & 3 of the step
        if ((c >> 2) == ps) {
          double* mine = cp + (c & 3) * STRIDE + g;
          tiles<W>([&](int i, int ti, int tj) {
            if (tj != tp) return;
#pragma unroll
            for (int r = 0; r < 4; ++r) mine[16 * ti + 4 * r] = acc[i][r] - ((ti == tp && g + 4 * r == c) ? 1.0 : 0.0);
          });
        }
        // rows before it, from the pivots' rows of the tiles (tp, tj): register ps of lane group g is pivot g of the step
        tiles<W>([&](int i, int ti, int tj) {
          if (ti != tp || tj >= tp) return;
          const d4 t = acc[i];
          cp[g * STRIDE + 16 * tj + c] = -(ps == 0 ? t[0] : ps == 1 ? t[1] : ps == 2 ? t[2] : t[3]);
        });
        __syncthreads();
        // B = L diag(dd) L^T (unit lower triangular L, no pivoting: B is symmetric positive definite), every
        // lane for itself in registers; lo[a][c] holds B's lower triangle, then t = L diag(dd) below the diagonal
        double lo[KB][KB], l[KB][KB], inv[KB];
#pragma unroll
        for (int a = 0; a < KB; ++a)
#pragma unroll
          for (int k = 0; k <= a; ++k) {
            const double x = cp[k * STRIDE + p0 + a];
            lo[a][k] = (a == k) ? x + 1.0 : x;
          }
#pragma unroll
        for (int k = 0; k < KB; ++k) {
          // column k: t[a][k] = B[a][k] - sum_{i<k} l[a][i] t[k][i];  dd_k = t[k][k];  l[a][k] = t[a][k] / dd_k
#pragma unroll
          for (int a = k; a < KB; ++a)
#pragma unroll
            for (int i = 0; i < k; ++i) lo[a][k] = fma(-l[a][i], lo[k][i], lo[a][k]);
          inv[k] = recip(lo[k][k]);
#pragma unroll
          for (int a = k + 1; a < KB; ++a) l[a][k] = lo[a][k] * inv[k];
        }
        // y = row g of B^{-1} (= column g: B is symmetric), by the two triangular solves on e_g
        double y[KB];
#pragma unroll
        for (int a = 0; a < KB; ++a) y[a] = (a == g) ? 1.0 : 0.0;
#pragma unroll
        for (int a = 1; a < KB; ++a)
#pragma unroll
          for (int k = 0; k < a; ++k) y[a] = fma(-l[a][k], y[k], y[a]);
#pragma unroll
        for (int a = 0; a < KB; ++a) y[a] *= inv[a];
#pragma unroll
        for (int a = KB - 2; a >= 0; --a)
#pragma unroll
          for (int k = a + 1; k < KB; ++k) y[a] = fma(-l[k][a], y[k], y[a]);
        // C'[16 ti + c][g]
        const double cv[2] = {cp[g * STRIDE + 16 * TI[0] + c], cp[g * STRIDE + 16 * TI[1] + c]};
        // x = (B^{-1} (M[j][P])^T)[g] for the lane's column j of every column tile; then R'[g][j]:
        //   j after the pivots:   R[:, j] = +M[j][P]^T            -> x
        //   j before the pivots:  R[:, j] = -M[j][P]^T            -> -x
        //   j = pivot e:          the column holds (B - I)[:, e]  -> x = (e_e - B^{-1} e_e)[g],  R' = 2 [e = g] - x
#pragma unroll
        for (int tj = 0; tj < NTL - W; ++tj) {
          const int j = 16 * tj + c;
          double x = y[0] * cp[j];
#pragma unroll
          for (int k = 1; k < KB; ++k) x = fma(y[k], cp[k * STRIDE + j], x);
          const double rr = (j >= p0 + KB) ? x : ((j - p0 == g) ? 2.0 - x : -x);
          acc[tj] = __builtin_amdgcn_mfma_f64_16x16x4f64(cv[0], -rr, acc[tj], 0, 0, 0);
          if (tj <= W) acc[NTL - W + tj] = __builtin_amdgcn_mfma_f64_16x16x4f64(cv[1], -rr, acc[NTL - W + tj], 0, 0, 0);
        }
      }
    }
    scale();
  }
};

template <int D, int DL, typename IO>
__global__ void __launch_bounds__(kThreads, D <= 64 ? 3 : 2) gram_kernel(ForwardArgs a, double* G) {
  gram_sum<D, DL, IO>(a, G);
}

// With a caller's A0 the workgroup of a head's last segment, which has no sum to form, inverts A0 into that segment's
// place in G: beside the sums instead of once more in front of every boundary inverse (39 heads of 128, 6 segments, T = 1537,
// float32: the two kernels 140 -> 111 us).  DL < D: bordered with an identity block, whose inverse is itself and which is
// left out of the result.
template <int D, int DL, typename IO>
__global__ void __launch_bounds__(SpdInverse<D>::NT > kThreads ? SpdInverse<D>::NT : kThreads, 2)
gram_given_a0_kernel(ForwardArgs a, double* G) {
  __shared__ __align__(16) double colp[SpdInverse<D>::LDS_DOUBLES];
  const int head = blockIdx.x / a.n_seg;
  if (static_cast<int>(blockIdx.x) - head * a.n_seg != a.n_seg - 1) {   // uniform over the workgroup
    if (threadIdx.x < kThreads) gram_sum<D, DL, IO>(a, G);              // whole waves
    return;
  }
  if (threadIdx.x >= SpdInverse<D>::NT) return;
  const float* A0 = a.A0 + static_cast<size_t>(head) * DL * DL;
  double* out = G + static_cast<size_t>(blockIdx.x) * DL * DL;
  const int c = threadIdx.x & 15;
  const int g = (threadIdx.x & 63) >> 4;
  using Inverse = SpdInverse<D>;
  Inverse::for_my_wave([&](auto wtag) {
    constexpr int W = decltype(wtag)::value;
    d4 acc[Inverse::NPT];
    Inverse::template tiles<W>([&](int n, int ti, int tj) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = 16 * ti + g + 4 * r, j = 16 * tj + c;
        acc[n][r] = D == DL || (i < DL && j < DL)
                        ? 0.5 * (static_cast<double>(A0[i * DL + j]) + static_cast<double>(A0[j * DL + i]))
                        : (i == j ? 1.0 : 0.0);
      }
    });
    Inverse{colp}.template run<W>(acc);
    Inverse::template tiles<W>([&](int n, int ti, int tj) {   // both triangles from the lower one's tiles
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = 16 * ti + g + 4 * r, j = 16 * tj + c;
        if (D != DL && (i >= DL || j >= DL)) continue;
        out[i * DL + j] = acc[n][r];
        if (ti != tj) out[j * DL + i] = acc[n][r];
      }
    });
  });
}

// Never a workgroup of one wave, a second one without work if need be: an odd number of waves leaves the waves of the next kernel's
// workgroups on other SIMDs than those they would share two and two, and the option kernel's A chain, two waves a workgroup, took
// 1670 instead of 1380 us for it (128 heads of 32, 30000 tokens, bf16, u and normalised read-out; whole call 2590 -> 2286).
constexpr int boundary_threads(int d) { return d <= 64 ? 128 : 2 * d; }

// One workgroup per (head, segment): seg_A = inverse(inverse(A0) + sum of the Gram matrices before it),
// G holding the prefix sums (prefixed) or the segments' own, added up here in the same order.
// DL: the head size of the data; D >= DL: the size the inversion is laid out for (d = 96 runs in the d = 128
// layout: the matrix is bordered with an identity block, whose inverse is itself).
template <int D, int DL>
__global__ void __launch_bounds__(boundary_threads(D), D <= 32 ? 4 : D <= 64 ? 3 : 2) boundary_kernel(ForwardArgs a, const double* G, float* seg_A, int prefixed) {
  static_assert(DL <= D, "padded layout");
  constexpr int NT = SpdInverse<D>::NT;
  __shared__ __align__(16) double colp[SpdInverse<D>::LDS_DOUBLES];

  if (NT < boundary_threads(D) && threadIdx.x >= NT) return;   // a whole wave; a barrier counts those that are left
  const int head = blockIdx.x / a.n_seg;
  const int seg = blockIdx.x - head * a.n_seg;
  const int lane = threadIdx.x & 63;
  const int c = lane & 15;
  const int g = lane >> 4;
  const float* A0 = a.A0 ? a.A0 + static_cast<size_t>(head) * DL * DL : nullptr;
  float* out = seg_A + static_cast<size_t>(blockIdx.x) * DL * DL;
  const float diag = 1.0f / a.lambda0;   // the same float32 value the first segment starts from

  // the first segment starts from the caller's A0, bit for bit; an A0 = 0 (infinite lambda0) stays zero
  if (seg == 0 || (!A0 && diag == 0.0f)) {
    for (int e = threadIdx.x; e < DL * DL; e += NT) out[e] = A0 ? A0[e] : (e / DL == e % DL ? diag : 0.0f);
    return;
  }
  // its inverse is in the last segment's place;  as inclusive prefix sums G[head][seg - 1] covers every token before this
  // segment, else G[head][0 .. seg - 1] do
  const double* inv0 = A0 ? G + (static_cast<size_t>(head) * a.n_seg + a.n_seg - 1) * DL * DL : nullptr;
  const int terms = prefixed ? 1 : seg;
  const double* Gh = G + (static_cast<size_t>(blockIdx.x) - terms) * DL * DL;
  const double diag0 = 1.0 / static_cast<double>(diag);
  using Inverse = SpdInverse<D>;
  Inverse::for_my_wave([&](auto wtag) {
    constexpr int W = decltype(wtag)::value;
    d4 acc[Inverse::NPT];
    constexpr int AHEAD = 2;   // segments in flight
    for (int s = 0; s < terms; s += AHEAD) {
      d4 x[AHEAD][Inverse::NPT];
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) {
        const double* Gs = Gh + static_cast<size_t>(min(s + u, terms - 1)) * DL * DL;
        Inverse::template tiles<W>([&](int n, int ti, int tj) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int i = 16 * ti + g + 4 * r, j = 16 * tj + c;
            x[u][n][r] = D == DL || (i < DL && j < DL) ? Gs[i * DL + j] : 0.0;   // inside the DL x DL matrix
          }
        });
      }
#pragma unroll
      for (int u = 0; u < AHEAD; ++u)
        if (s + u < terms) {   // uniform over the workgroup
#pragma unroll
          for (int n = 0; n < Inverse::NPT; ++n) acc[n] = s + u == 0 ? x[u][n] : acc[n] + x[u][n];
        }
    }
    Inverse::template tiles<W>([&](int n, int ti, int tj) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = 16 * ti + g + 4 * r, j = 16 * tj + c;
        if (D == DL || (i < DL && j < DL))
          acc[n][r] = (inv0 ? inv0[i * DL + j] : i == j ? diag0 : 0.0) + acc[n][r];
        else
          acc[n][r] = i == j ? 1.0 : 0.0;
      }
    });
    Inverse{colp}.template run<W>(acc);
    // The inverse of a symmetric matrix is symmetric up to rounding; the lower triangle's values go to both
    // sides so that the float32 matrix the recurrence starts from is exactly symmetric.
    Inverse::template tiles<W>([&](int n, int ti, int tj) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = 16 * ti + g + 4 * r, j = 16 * tj + c;
        if (i < j || (D != DL && (i >= DL || j >= DL))) continue;
        const float v = static_cast<float>(acc[n][r]);
        out[i * DL + j] = v;
        out[j * DL + i] = v;
      }
    });
  });
}

// ------------------------------------------------------------------------------------------ combine
// x <- x P_s + Q_s for s = 0 .. n_seg-2, every intermediate written out as the start state of segment s+1.
// One workgroup per (head, 16-row slab of S), one wave per 16-column slice of the result: each wave keeps the
// whole slab x as accumulator tiles, xt[b][r] = S[row0 + c][16b + 4g + r] (the layout the S-rows kernel loads
// its start state in; the contraction index is taken in the order k = 16b + 4g + r so that a tile feeds
// straight back as the MFMA B operand), computes its own slice of x P + Q and hands it to the other waves
// through LDS.  The chain is sequential in s and short per step, so the operands of the next three
// segments are kept in flight in rotating register sets: every load on a path of its own without a condition, because where a
// path with and one without it meet the compiler cannot count what is in flight and waits for all of it.  One head of 128,
// T = 32768 (90 segments) 443 -> 375 us the whole call, of 64, float32 184 -> 173; 8 heads of 128 in 16 segments 137 -> 128.
// S has a.d_v rows (value heads of another size than the key heads: more or fewer slabs per head, P stays D x D).
template <int D>
__global__ void __launch_bounds__(64 * (D / 16)) combine_kernel(ForwardArgs a, float* seg_S) {
  constexpr int NB = D / 16;
  constexpr int LDX = D + 4;
  constexpr int LA = 3;   // segments of lookahead
  __shared__ __align__(16) float xs[2][16 * LDX];
  const int dv = a.d_v > 0 ? a.d_v : D;
  const int nbv = dv / 16;                       // slabs per head
  const size_t ssz = static_cast<size_t>(dv) * D;            // floats of S and of Q
  const size_t pqsz = static_cast<size_t>(D) * D + ssz;      // floats of one segment's P then Q
  const int head = blockIdx.x / nbv;
  const int row0 = (blockIdx.x - head * nbv) * 16;
  const int jb = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // column slice of this wave
  const int lane = threadIdx.x & 63;
  const int c = lane & 15;
  const int g = lane >> 4;
  const size_t hbase = static_cast<size_t>(head) * a.n_seg;
  const int ro = (row0 + c) * D + 4 * g;   // this lane's float4 inside a d x d matrix, plus 16 b
  const int n = a.n_seg - 1;               // steps

  struct Seg {
    float pa[NB][4];   // P[16b + 4g + r][16 jb + c]
    f4 q;              // Q[row0 + c][16 jb + 4g ..]
  };
  const unsigned po = 4 * g * D + c;
  const unsigned qo = static_cast<unsigned>(c * D + 4 * g);
  auto load = [&](int s, Seg& o) {   // s past the last step: that one's again
    const float* P = a.seg_PQ + (hbase + min(s, n - 1)) * pqsz;
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) o.pa[b][r] = (P + 16 * b * D + 16 * jb)[po + r * D];
    o.q = *reinterpret_cast<const f4*>(P + D * D + row0 * D + 16 * jb + qo);
  };

  f4 xt[NB];
  {
    const float* S0 = a.S0 ? a.S0 + static_cast<size_t>(head) * ssz : nullptr;
#pragma unroll
    for (int b = 0; b < NB; ++b) xt[b] = S0 ? *reinterpret_cast<const f4*>(S0 + ro + 16 * b) : f4{0, 0, 0, 0};
    const f4 mine = S0 ? *reinterpret_cast<const f4*>(S0 + ro + 16 * jb) : f4{0, 0, 0, 0};
    *reinterpret_cast<f4*>(seg_S + hbase * ssz + ro + 16 * jb) = mine;
  }

  auto step = [&](int s, const Seg& o) {
    f4 nx = o.q;
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) nx = mfma16(o.pa[b][r], xt[b][r], nx);
    *reinterpret_cast<f4*>(seg_S + (hbase + s + 1) * ssz + ro + 16 * jb) = nx;
    float* x = xs[s & 1];
    *reinterpret_cast<f4*>(&x[c * LDX + 16 * jb + 4 * g]) = nx;
    __syncthreads();
#pragma unroll
    for (int b = 0; b < NB; ++b) xt[b] = lds4(&x[c * LDX + 16 * b + 4 * g]);
  };

  Seg buf[LA + 1];
  if (n <= LA) {   // all at once, none twice: 1 us of 94 in three segments of 128
#pragma unroll
    for (int u = 0; u < LA; ++u)
      if (u < n) load(u, buf[u]);
#pragma unroll
    for (int u = 0; u < LA; ++u)
      if (u < n) step(u, buf[u]);
    return;
  }
#pragma unroll
  for (int u = 0; u < LA; ++u) {
    load(u, buf[u]);
    __builtin_amdgcn_sched_barrier(0);   // requested in the order of their use, as in the loop
  }
  for (int s = 0;; s += LA + 1) {
#pragma unroll
    for (int u = 0; u <= LA; ++u) {
      if (s + u >= n) return;   // uniform over the workgroup
      load(s + u + LA, buf[(u + LA) % (LA + 1)]);
      step(s + u, buf[u]);
    }
  }
}

// Up to six segments boundary_kernel adds up the Gram matrices before its own by itself (the same sums in the same order), in place
// of a launch of gram_prefix_kernel, which takes 5 us at d = 64 and 10 at 128 and the gap after it; each further two
// cost the last segment a trip to memory, 1 us or more.  Whole calls, prefix kernel / added up, us: 8 heads of 64 in 2, 4, 6, 8, 16
// segments of 4 blocks 44.6 / 42.5, 45.7 / 44.7, 48.4 / 48.0, 50.2 / 51.8, 59.2 / 64.0; 8 heads of 128 90.5 / 88.0, 100.6 /
// 99.5, 110.9 / 109.4, 116.0 / 118.9, 137 / 145; 39 heads of 128 x 64, A0 given, 6 segments 258.0 / 251.3; 96 heads of 128, 5
// segments, T = 4096 934 / 921.
bool boundary_adds_up(int n_seg) { return n_seg <= 6; }

template <int D, int DL = D>
hipError_t launch_boundary_d(const ForwardArgs& a, const double* G, float* seg_A, hipStream_t stream) {
  ForwardArgs args = a;
  int prefixed = boundary_adds_up(a.n_seg) ? 0 : 1;
  void* params[] = {&args, &G, &seg_A, &prefixed};
  return hipLaunchKernel(reinterpret_cast<const void*>(&boundary_kernel<D, DL>), dim3(a.n_heads * a.n_seg),
                         dim3(boundary_threads(D)), params, 0, stream);
}
template <int D, typename IO, int DL = D>
hipError_t launch_gram_d(const ForwardArgs& a, double* G, hipStream_t stream) {
  ForwardArgs args = a;
  int shift = 30 - direction_exponent(a);
  void* params[] = {&args, &G, &shift};
  const bool fixed = fixed_point_gram(a);
  const void* fn = fixed  ? reinterpret_cast<const void*>(&gram_fixed_kernel<DL, IO>)
                   : a.A0 ? reinterpret_cast<const void*>(&gram_given_a0_kernel<D, DL, IO>)
                        : reinterpret_cast<const void*>(&gram_kernel<D, DL, IO>);
  const int threads = fixed ? fixed_threads(DL) : a.A0 && SpdInverse<D>::NT > kThreads ? SpdInverse<D>::NT : kThreads;
  hipError_t err = hipLaunchKernel(fn, dim3(a.n_heads * a.n_seg), dim3(threads), params, 0, stream);
  if (err != hipSuccess || boundary_adds_up(a.n_seg)) return err;
  int nh = a.n_heads, ns = a.n_seg, dd = DL * DL;
  void* p2[] = {&G, &nh, &ns, &dd};
  const long long elems = static_cast<long long>(nh) * dd;
  return hipLaunchKernel(reinterpret_cast<const void*>(&gram_prefix_kernel),
                         dim3(static_cast<unsigned>((elems + kThreads - 1) / kThreads)), dim3(kThreads), p2, 0,
                         stream);
}
template <int D>
hipError_t launch_combine_d(const ForwardArgs& a, float* seg_S, hipStream_t stream) {
  ForwardArgs args = a;
  void* params[] = {&args, &seg_S};
  const int dv = a.d_v > 0 ? a.d_v : D;
  return hipLaunchKernel(reinterpret_cast<const void*>(&combine_kernel<D>), dim3(a.n_heads * (dv / 16)),
                         dim3(64 * (D / 16)), params, 0, stream);
}

}  // namespace

namespace {
template <int D, typename IO>
hipError_t launch_keysum_d(const ForwardArgs& a, double* part, float* seg_zkey, hipStream_t stream) {
  ForwardArgs args = a;
  void* params[] = {&args, &part};
  hipError_t err = hipLaunchKernel(reinterpret_cast<const void*>(&keysum_kernel<D, IO>),
                                   dim3(a.n_heads * a.n_seg), dim3(kThreads), params, 0, stream);
  if (err != hipSuccess) return err;
  const double* cpart = part;
  const float* z0 = a.zkey0;
  int nh = a.n_heads, ns = a.n_seg, d = D;
  void* p2[] = {&cpart, &z0, &seg_zkey, &nh, &ns, &d};
  const long long elems = static_cast<long long>(nh) * d;
  return hipLaunchKernel(reinterpret_cast<const void*>(&keysum_prefix_kernel),
                         dim3(static_cast<unsigned>((elems + kThreads - 1) / kThreads)), dim3(kThreads), p2, 0,
                         stream);
}
}  // namespace

hipError_t launch_keysum(const ForwardArgs& a, int d, int io_dtype, double* part, float* seg_zkey,
                         hipStream_t stream) {
  const bool bf = io_dtype == 1;
  switch (d) {
    case 32: return bf ? launch_keysum_d<32, uint16_t>(a, part, seg_zkey, stream)
                       : launch_keysum_d<32, float>(a, part, seg_zkey, stream);
    case 64: return bf ? launch_keysum_d<64, uint16_t>(a, part, seg_zkey, stream)
                       : launch_keysum_d<64, float>(a, part, seg_zkey, stream);
    case 96: return bf ? launch_keysum_d<96, uint16_t>(a, part, seg_zkey, stream)
                       : launch_keysum_d<96, float>(a, part, seg_zkey, stream);
    case 128: return bf ? launch_keysum_d<128, uint16_t>(a, part, seg_zkey, stream)
                        : launch_keysum_d<128, float>(a, part, seg_zkey, stream);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_gram(const ForwardArgs& a, int d, int io_dtype, double* G, hipStream_t stream) {
  const bool bf = io_dtype == 1;
  switch (d) {
    case 32: return bf ? launch_gram_d<32, uint16_t>(a, G, stream) : launch_gram_d<32, float>(a, G, stream);
    case 64: return bf ? launch_gram_d<64, uint16_t>(a, G, stream) : launch_gram_d<64, float>(a, G, stream);
    case 96: return bf ? launch_gram_d<128, uint16_t, 96>(a, G, stream) : launch_gram_d<128, float, 96>(a, G, stream);
    case 128: return bf ? launch_gram_d<128, uint16_t>(a, G, stream) : launch_gram_d<128, float>(a, G, stream);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_boundary(const ForwardArgs& a, int d, const double* G, float* seg_A, hipStream_t stream) {
  switch (d) {
    case 32: return launch_boundary_d<32>(a, G, seg_A, stream);
    case 64: return launch_boundary_d<64>(a, G, seg_A, stream);
    case 96: return launch_boundary_d<128, 96>(a, G, seg_A, stream);
    case 128: return launch_boundary_d<128>(a, G, seg_A, stream);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_combine(const ForwardArgs& a, int d, float* seg_S, hipStream_t stream) {
  switch (d) {
    case 32: return launch_combine_d<32>(a, seg_S, stream);
    case 64: return launch_combine_d<64>(a, seg_S, stream);
    case 96: return launch_combine_d<96>(a, seg_S, stream);
    case 128: return launch_combine_d<128>(a, seg_S, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace vla
