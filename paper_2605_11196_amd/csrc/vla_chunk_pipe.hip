// Block form of the VLA recurrence (paper Section 3.3; the algebra is at the head of vla_chunk.hip) with the A chain and
// the S chain on waves of their own, the S chain one block behind.
//
// A never reads S, so a block's S side (residuals, read-out, update of S) only needs what the A side left in LDS one block
// earlier: W, Z, NQ, c.  Between two barriers the two sides work at the same time:
//
//   (1)-(2)  A waves: one factorises I + G of block b, one forms c and Z and one NQ of block b - 1
//            S waves: K^ S^T and Q S^T of block b - 1
//   (2)-(3)  A waves: W of block b to LDS          S waves: stage K^ and Q of block b + 1
//   (3)-(1)  A waves: A -= W W^T, Y = K^ A and the Gram matrices of block b + 1
//            S waves: E, o and the update of S of block b - 1
//
// What bounds it.  In the kernel that keeps both states on every wave (vla_chunk.hip) a block takes the sum of these:
// 17000 cycles alone for a head of 128, 20000 with a second head beside it, although its instructions fill half of that.
// Here it takes the longer side of each window: 9500 to 10500 cycles for one head of 128 on its compute unit, 6700
// (from 9400) for one of 64.  With two heads of 128 (four waves per SIMD) it is 16000 for both, vector unit 43 % and matrix
// unit 56 % busy; leaving a part out shortens that by 12 % (splits of A), 10 % (factorisation), 9 % (splits of S), 8 %
// (update of A), 4 % (update of S), and no other part by more than 2 %.  With so many waves the latency of the matrix unit
// is covered, and the residuals of the splits go there (split3_cut_matrix; 2048 heads of 128, 1024 tokens, bf16: 2.28 ->
// 2.00 ms; vla_chunk.hip 2.20).  T = 512, bf16, vla_chunk.hip / here: 16 heads of 64 0.120 / 0.087 ms, 256 heads of 64
// 0.121 / 0.097, 2048 heads of 64 0.413 / 0.365, 256 heads of 128 0.190 / 0.159, 512 heads 0.290 / 0.255.
//
// Vector instructions are what a SIMD has most of: one takes 4.9 cycles, a bf16 matrix instruction 17.7 by itself and 7.7 of
// the vector unit's beside vector work, an FP32 one 32.5 of both.  So rows are addressed as a uniform base with an offset of the
// lane (only the ragged last block clamps and masks), lane indices carry their range (24-bit products), and the partial Gram
// matrices of a wave of 16 columns are formed from half operands: the S waves of d = 64 about 320 -> 270 vector instructions a block.
// 256 heads of 64, float32, 2048 tokens 0.352 -> 0.318 ms; 2048 heads of 64, 8192 tokens, bf16 5.54 -> 5.33, of 128 15.4 ->
// 15.1.  W kept as l, h, m in 24 bytes (two overlapping reads without moves) was 3 % faster with one head per compute unit
// and 3 % slower with four: twice the LDS reads.
//
// Waves of 32 columns (two heads of 128 or four of 64 per compute unit) have to stay within 128 registers: offsets derived
// from the lane are formed anew in each block (the compiler keeps some 60 of them otherwise: 1.27 -> 1.12 ms for 2048 heads
// of 128, 512 tokens), v is fetched beside the pass over S and not a block ahead.  Measured and not kept: staging on the A
// waves (the longer side of that window), a third K^ / Q buffer with staging in the last window (2.02 against 2.03 ms), one
// of the two residuals on the vector unit (2.04), two splits in flight in the pass over S (2.15, registers).
#include "vla_mfma_util.h"

namespace vla {
namespace {

constexpr int group(int n) { return n <= 1 ? 1 : 2 * group((n + 1) / 2); }   // the power of two from n on

// NWA waves own SL = D / NWA columns of A each, NWS waves DV / NWS rows of S each.  WPE: waves per SIMD to compile for.
template <int D, int DV, int NWA, int NWS, typename IO, bool FMAP, int WPE>
__global__ void __launch_bounds__(64 * (NWA + NWS), WPE) chunk_pipe_kernel(ForwardArgs a) {
  constexpr int SL = D / NWA;          // columns of A of one wave
  constexpr int NJ = SL / 16;          // 16-wide tiles among them
  constexpr int NJV = DV / (16 * NWS); // row tiles of S of one wave
  static_assert(NWA >= 2 && SL % 16 == 0 && DV % (16 * NWS) == 0, "whole tiles; two serial sections run at once");
  constexpr int NB = D / 16;
  constexpr int KT = sizeof(IO) == 2 && !FMAP ? 1 : 3;   // operand terms of k and q
  using Ops = BlockOps<true, KT, D>;
  constexpr int NKB = NB / 2;
  constexpr int LDY = SL + 4;
  // Staging (by the S waves): a token row is split over TPR threads of EPT elements each.  Where the threads do not
  // divide into rows of a power of two, or into pieces of four elements, a row takes D / EPT threads of a group of TPR, a
  // power of two up to 16 (whose sum needs no shuffles through LDS), in the smallest pieces of 4, 8 or 16 elements that there
  // are threads for; rows of 96 with one operand term, quick to stage, in pieces of 16.  2048 tokens, pieces of 16 and the
  // smallest, ms: 32 x 64, 16 heads, bf16 with the feature map 0.507 / 0.319, 256 heads, float32 0.414 / 0.341; 64 x 96, 256
  // heads, float32 0.518 / 0.436, bf16 0.451 / 0.409; 128 x 96 0.770 / 0.666 and 0.612 / 0.583; 96 x 96 0.576 / 0.567 and 0.506 /
  // 0.515; 96 x 64 0.552 / 0.552 and 0.493 / 0.524.
  constexpr int NT = 64 * NWS;
  constexpr int TPR0 = NT / C;
  constexpr bool PADDED = (TPR0 & (TPR0 - 1)) != 0 || (C * D / NT) % 4 != 0;
  constexpr int PIECE = D == 96 && KT == 1                                 ? 16
                        : group(D / 4) <= 16 && C * group(D / 4) <= NT ? 4
                        : C * group(D / 8) <= NT                           ? 8
                                                                           : 16;
  constexpr int EPT = PADDED ? PIECE : C * D / NT;
  constexpr int TPR = group(D / EPT);
  static_assert(EPT % 4 == 0 && TPR <= 32 && (TPR & (TPR - 1)) == 0 && C * TPR <= NT && D % EPT == 0 &&
                D / EPT <= TPR, "staging layout");

  __shared__ __align__(16) uint16_t Ksb[2][Ops::SIZE];     // k [t][slot], terms, double-buffered over blocks
  __shared__ __align__(16) uint16_t Qsb[2][Ops::SIZE];     // q
  __shared__ __align__(16) u4 Whm[2][D * 4];               // W [j][t], terms h and m
  __shared__ __align__(16) u2 Wl[2][D * 4];                //           term l
  __shared__ __align__(16) float Yg[NWA][C * (LDY > LT ? LDY : LT)];   // a wave's slab of Y^T, then its partial G [s][t]
  __shared__ __align__(16) float GQp[2][NWA][C * LT];      // partial GQ [t][s]
  __shared__ __align__(16) float Lis[2][C * LT];           // L^{-1} [t][s]
  __shared__ __align__(16) float Lrs[2][C * LT];           // L [t][s]
  __shared__ __align__(16) float Zs[C * LT];               // Z   [t][s]
  __shared__ __align__(16) float NQs[C * LT];              // -NQ^T [t][s]
  __shared__ __align__(16) float wn2p[NWA][C];             // partial ||w_t||^2
  __shared__ __align__(16) float cvec[C];                  // -c_t
  __shared__ __align__(16) float rns[2][C];                // 1 / max(||k_t||, eps) over its power of two (key_scale)

  const int head = blockIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  int c = lane & 15;
  int g = lane >> 4;
  // Once per block: what is derived from the lane (LDS and global offsets) is formed anew, not kept in registers.
  auto fresh = [&]() __attribute__((always_inline)) { renew(c, g); };
  // -1 on the diagonal for the splits: two registers where the waves have them, else formed where it is used
  constexpr bool kKeepIdentity = NB * NJ < 16 && NB * NJV < 16;
  u2 minus_one = minus_identity(c, g);
  asm volatile("" : "+v"(minus_one));
  auto identity = [&]() __attribute__((always_inline)) -> u2 {
    if constexpr (kKeepIdentity) return minus_one;
    else return minus_identity(c, g);
  };
  const int T = a.T;
  const int nblk = (T + C - 1) / C;
  const float eps = a.eps;

  if (wave < NWA) {
    // ================================================================ A chain
    const int w = wave;
    const int col0 = SL * w;
    f4 At[NB][NJ];   // At[b][jn][r] = A[16b + 4g + r][col0 + 16jn + c]
    {
      const float* A0 = a.A0 ? a.A0 + static_cast<size_t>(head) * D * D : nullptr;
      const float diag = 1.0f / a.lambda0;
      const int arc = (4 * g) * D + col0 + c;
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int jn = 0; jn < NJ; ++jn)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            At[b][jn][r] = A0 ? A0[arc + (16 * b + r) * D + 16 * jn]
                              : (16 * b + 4 * g + r == col0 + 16 * jn + c) ? diag : 0.0f;
    }
    f4 yt[NJ];
    // Y^T = K^ A (this wave's columns) and the partial Gram matrices over them
    auto y_and_gram = [&](int blk) __attribute__((always_inline)) {
      const uint16_t* Ks = Ksb[blk & 1];
      const uint16_t* Qs = Qsb[blk & 1];
#pragma unroll
      for (int jn = 0; jn < NJ; ++jn) yt[jn] = f4{0, 0, 0, 0};
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb) {
        const Terms<KT> ka = Ops::operand(Ks, kb, c, g);
#pragma unroll
        for (int jn = 0; jn < NJ; ++jn) yt[jn] = Ops::sweep(ka, split_tiles(At[2 * kb][jn], At[2 * kb + 1][jn], identity()), yt[jn]);
        if (KT > 1 || NB * NJ >= 16) __builtin_amdgcn_sched_barrier(0);
      }
      const f4 rn4 = lds4(&rns[blk & 1][4 * g]);
#pragma unroll
      for (int jn = 0; jn < NJ; ++jn) yt[jn] *= rn4;
      float* Yw = Yg[w];
#pragma unroll
      for (int jn = 0; jn < NJ; ++jn)
#pragma unroll
        for (int r = 0; r < 4; ++r) Yw[(4 * g + r) * LDY + 16 * jn + c] = yt[jn][r];
      // same-wave write -> read: LDS operations of one wave are ordered
      f4 gg = f4{0, 0, 0, 0}, gq = f4{0, 0, 0, 0};
#pragma unroll
      for (int j2 = 0; j2 < NJ / 2; ++j2) {
        const auto ya = split_tiles(lds4(&Yw[c * LDY + 32 * j2 + 4 * g]), lds4(&Yw[c * LDY + 32 * j2 + 16 + 4 * g]), identity());
        gg = Ops::sweep(Ops::operand(Ks, col0 / 32 + j2, c, g), ya, gg);
        gq = Ops::sweep(Ops::operand(Qs, col0 / 32 + j2, c, g), ya, gq);
      }
      if constexpr (NJ == 1) {
        const HalfTerms<3> ya = split_tile(lds4(&Yw[c * LDY + 4 * g]), identity());
        gg = mfma_terms(Ops::half_operand(Ks, w, c, g), ya, gg);
        gq = mfma_terms(Ops::half_operand(Qs, w, c, g), ya, gq);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) Yw[c * LT + 4 * g + r] = gg[r] * rn4[r];
#pragma unroll
      for (int r = 0; r < 4; ++r) GQp[blk & 1][w][(4 * g + r) * LT + c] = gq[r];
    };
    // Cholesky of I + G and L^{-1}; G is stored with its rows on the columns of the tile
    auto factorise = [&](int blk) __attribute__((always_inline)) {
      f4 gram = lds4(&Yg[0][c * LT + 4 * g]);
#pragma unroll
      for (int ww = 1; ww < NWA; ++ww) gram += lds4(&Yg[ww][c * LT + 4 * g]);
      cholesky16(gram, Lrs[blk & 1], Lis[blk & 1], c, g);
    };
    // c_t on lane t of every row of 16
    auto strength = [&](int blk) __attribute__((always_inline)) -> float {
      float wn2 = 0.0f;
#pragma unroll
      for (int ww = 0; ww < NWA; ++ww) wn2 += wn2p[ww][c];
      // hardware reciprocal and square root (1 ulp): c_t only scales the write direction
      const float rdl = __builtin_amdgcn_rcpf(Lrs[blk & 1][c * LT + c]);
      const float an = __builtin_amdgcn_sqrtf(wn2) * rdl;            // ||A_t k^_t|| = ||w_t|| / L_tt
      return rdl * __builtin_amdgcn_rcpf(fmaxf(an, eps));            // alpha^_t = c_t w_t
    };
    // NQ[s][t] = c_s H[s][t] for s <= t, H = L^{-1} GQ (one MFMA tile)
    auto form_nq = [&](int blk) __attribute__((always_inline)) {
      const f4 la = lds4(&Lis[blk & 1][c * LT + 4 * g]);
      f4 gq = f4{0, 0, 0, 0};
#pragma unroll
      for (int ww = 0; ww < NWA; ++ww) gq += lds4(&GQp[blk & 1][ww][c * LT + 4 * g]);
      f4 hq = f4{0, 0, 0, 0};
#pragma unroll
      for (int r = 0; r < 4; ++r) hq = mfma16(la[r], gq[r], hq);
      const float cs = strength(blk);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int s = 4 * g + r;
        const float csr = __shfl(cs, s);
        NQs[c * LT + s] = (s <= c) ? -(csr * hq[r]) : 0.0f;
      }
    };
    // Z = (I + strict_lower(L) diag(c))^{-1}
    auto form_z = [&](int blk) __attribute__((always_inline)) {
      const float cs = strength(blk);
      if (g == 0) cvec[c] = -cs;  // the residual tiles carry -E
      lower_inverse16(Lrs[blk & 1], cs, c, g, [&](int t, int s, float z) { Zs[t * LT + s] = z; });
    };
    // W^T = L^{-1} Y^T, partial ||w_t||^2, W to LDS
    auto form_w = [&](int blk) __attribute__((always_inline)) {
      const f4 la = lds4(&Lis[blk & 1][c * LT + 4 * g]);
      f4 n2 = f4{0, 0, 0, 0};
#pragma unroll
      for (int jn = 0; jn < NJ; ++jn) {
        f4 acc = f4{0, 0, 0, 0};
#pragma unroll
        for (int r = 0; r < 4; ++r) acc = mfma16(la[r], yt[jn][r], acc);
        n2 += acc * acc;
        Ops::w_store(Whm[blk & 1], Wl[blk & 1], col0 + 16 * jn + c, c, g, acc);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) n2[r] = row_sum16(n2[r]);
      if (c == 0) *reinterpret_cast<f4*>(&wn2p[w][4 * g]) = n2;
    };

    __syncthreads();  // block 0 staged
    if (nblk > 0) y_and_gram(0);
    for (int blk = 0; blk < nblk; ++blk) {
      fresh();
      __syncthreads();  // (1) partial Grams of this block visible
      const int sw = (blk + head) % NWA;      // rotates over waves / SIMDs
      const int sw2 = (sw + 1) % NWA, sw3 = (sw + 2) % NWA;
      __builtin_amdgcn_s_setprio(3);
      if (w == sw) factorise(blk);
      else if (w == sw2 && blk > 0) {
        form_z(blk - 1);
        if (NWA < 3) form_nq(blk - 1);
      } else if (NWA > 2 && w == sw3 && blk > 0) {
        form_nq(blk - 1);
      }
      __builtin_amdgcn_s_setprio(2);
      __syncthreads();  // (2) L^{-1} of this block, Z of the one before it visible
      form_w(blk);
      __syncthreads();  // (3) W visible, next block staged
      Ops::template downdate<NB, NJ, (NB * NJ >= 16)>(Whm[blk & 1], Wl[blk & 1], col0 + c, c, g, blk & 1,
                                     [&](int b, int jn) -> f4& { return At[b][jn]; });
      if (blk + 1 < nblk) y_and_gram(blk + 1);
    }
    __syncthreads();  // (1)
    if (w == 0 && nblk > 0) {
      form_z(nblk - 1);
      form_nq(nblk - 1);
    }
    __syncthreads();  // (2) Z of the last block visible
    if (a.A_T) {
      float* AT = a.A_T + static_cast<size_t>(head) * D * D;
      int g2 = g, c2 = c;
      asm volatile("" : "+v"(g2), "+v"(c2));  // recompute the addresses here instead of carrying them over the loop
      const int arc = (4 * g2) * D + col0 + c2;
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int jn = 0; jn < NJ; ++jn)
#pragma unroll
          for (int r = 0; r < 4; ++r) AT[arc + (16 * b + r) * D + 16 * jn] = At[b][jn][r];
    }
  } else {
    // ================================================================ S chain, one block behind; staging
    const int w = wave - NWA;
    const int row0 = 16 * NJV * w;
    f4 St[NB][NJV];   // St[b][jn][r] = S[row0 + 16jn + c][16b + 4g + r]
    {
      const float* S0 = a.S0 ? a.S0 + static_cast<size_t>(head) * DV * D : nullptr;
      const int src = (row0 + c) * D + 4 * g;
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int jn = 0; jn < NJV; ++jn) {
          if (S0) {
            const float4 x = *reinterpret_cast<const float4*>(S0 + src + 16 * jn * D + 16 * b);
            St[b][jn] = f4{x.x, x.y, x.z, x.w};
          } else {
            St[b][jn] = f4{0, 0, 0, 0};
          }
        }
    }
    const size_t slab = static_cast<size_t>(head) * static_cast<size_t>(T) * D;
    const IO* qh = static_cast<const IO*>(a.q) + slab;
    const IO* kh = static_cast<const IO*>(a.k) + slab;
    const bool stage_wave = !PADDED || 64 * w < C * TPR;
    auto tid = [&]() { return 64 * w + 16 * g + c; };
    auto srow = [&]() { return tid() / TPR; };
    auto sseg = [&]() { return (tid() % TPR) * EPT; };
    auto stager = [&]() { return !PADDED || (tid() < C * TPR && sseg() < D); };
    RawRow<IO, EPT> kpre, qpre;
    // Loads never branch or wait: rows past the end are read from the last valid row and replaced by zeros when the
    // registers are consumed.
    auto load_kq = [&](int t0) __attribute__((always_inline)) {
      if (stager()) {
        // uniform base and an offset of the lane; only the ragged last block clamps its rows
        const size_t tok = static_cast<size_t>(t0) * D;
        const int row = t0 + C <= T ? srow() : min(srow(), T - 1 - t0);
        const unsigned koff = static_cast<unsigned>(row * D + sseg());
        kpre.load(kh + tok + koff);
        qpre.load(qh + tok + koff);
      }
    };
    auto stage = [&](int t0, int buf) __attribute__((always_inline)) {
      if (!stage_wave) return;
      float kx[EPT];
      const bool ragged = t0 + C > T;
      const bool live = t0 + srow() < T && stager();
      if (stager()) {
        kpre.unpack(kx);
      } else {
#pragma unroll
        for (int e = 0; e < EPT; ++e) kx[e] = 0.0f;
      }
      if constexpr (FMAP) {
#pragma unroll
        for (int e = 0; e < EPT; ++e) kx[e] = elu_plus_one(kx[e]);
      }
      if (ragged || PADDED) {
#pragma unroll
        for (int e = 0; e < EPT; ++e) kx[e] = live ? kx[e] : 0.0f;
      }
      float ss = 0.0f;
#pragma unroll
      for (int e = 0; e < EPT; ++e) ss = fmaf(kx[e], kx[e], ss);
      // 1 / max(||k||, eps): hardware reciprocal square root refined by one Newton step
      if constexpr (TPR == 16) {
        ss = row_sum16(ss);
      } else {
#pragma unroll
        for (int off = TPR / 2; off >= 1; off >>= 1) ss += __shfl_xor(ss, off);
      }
      const float sm = fmaxf(ss, eps * eps);
      float rn = __builtin_amdgcn_rsqf(sm);
      rn = rn * fmaf(-0.5f * sm * rn, rn, 1.5f);
      if (!stager()) return;
      const KeyScale ks = key_scale(rn);
#pragma unroll
      for (int e = 0; e < EPT; ++e) kx[e] *= ks.pow2;
      if (sseg() == 0) rns[buf][srow()] = ks.rest;
#pragma unroll
      for (int e = 0; e < EPT; e += 4) Ops::put4(Ksb[buf], srow(), sseg() + e, f4{kx[e], kx[e + 1], kx[e + 2], kx[e + 3]});
      float qx[EPT];
      qpre.unpack(qx);
      if constexpr (FMAP) {
#pragma unroll
        for (int e = 0; e < EPT; ++e) qx[e] = elu_plus_one(qx[e]);
      }
      if (ragged) {
#pragma unroll
        for (int e = 0; e < EPT; ++e) qx[e] = live ? qx[e] : 0.0f;
      }
#pragma unroll
      for (int e = 0; e < EPT; e += 4) Ops::put4(Qsb[buf], srow(), sseg() + e, f4{qx[e], qx[e + 1], qx[e + 2], qx[e + 3]});
    };
    const size_t slab_v = static_cast<size_t>(head) * static_cast<size_t>(T) * DV;
    const IO* vh = static_cast<const IO*>(a.v) + slab_v;
    IO* oh = static_cast<IO*>(a.o) + slab_v;
    auto vcol = [&]() { return row0 + c; };
    IO vpre[NJV][4];   // V[t0 + 4g + r][row0 + 16jn + c]
    auto load_v = [&](int t0) __attribute__((always_inline)) {
      const IO* vb = vh + static_cast<size_t>(t0) * DV;
      if (t0 + C <= T) {   // uniform
        const IO* vl = vb + static_cast<unsigned>(4 * g * DV + vcol());
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int jn = 0; jn < NJV; ++jn) vpre[jn][r] = vl[r * DV + 16 * jn];
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const IO* vl = vb + static_cast<unsigned>(min(4 * g + r, T - 1 - t0) * DV + vcol());
#pragma unroll
          for (int jn = 0; jn < NJV; ++jn) vpre[jn][r] = vl[16 * jn];
        }
      }
    };
    f4 ft[NJV], ot[NJV];
    // -F^T = K^ S^T - V^T and R^T = Q S^T: one pass over S, whose split serves both
    auto s_pass = [&](int blk) __attribute__((always_inline)) {
      const uint16_t* Ks = Ksb[blk & 1];
      const uint16_t* Qs = Qsb[blk & 1];
#pragma unroll
      for (int jn = 0; jn < NJV; ++jn) ft[jn] = ot[jn] = f4{0, 0, 0, 0};
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb) {
#pragma unroll
        for (int jn = 0; jn < NJV; ++jn) {
          const auto sb = split_tiles(St[2 * kb][jn], St[2 * kb + 1][jn], identity());
          ft[jn] = Ops::sweep(Ops::operand(Ks, kb, c, g), sb, ft[jn]);
          if constexpr (KT > 1) __builtin_amdgcn_sched_barrier(0);
          ot[jn] = Ops::sweep(Ops::operand(Qs, kb, c, g), sb, ot[jn]);
          __builtin_amdgcn_sched_barrier(0);   // one split at a time in registers
        }
      }
      const f4 rn4 = lds4(&rns[blk & 1][4 * g]);
#pragma unroll
      for (int jn = 0; jn < NJV; ++jn) ft[jn] *= rn4;
    };
    // -E^T = Z (-F^T), O^T = R^T + (-NQ^T)(-E^T), store o
    auto s_update = [&](int blk) __attribute__((always_inline)) {
      const int t0 = C * blk;
      if (t0 + C > T) {  // uniform: rows past the end of the sequence are zero tokens
#pragma unroll
        for (int jn = 0; jn < NJV; ++jn)
#pragma unroll
          for (int r = 0; r < 4; ++r) vpre[jn][r] = (t0 + 4 * g + r < T) ? vpre[jn][r] : IO(0);
      }
#pragma unroll
      for (int jn = 0; jn < NJV; ++jn)
#pragma unroll
        for (int r = 0; r < 4; ++r) ft[jn][r] += neg_widen(vpre[jn][r]);
      const f4 za = lds4(&Zs[c * LT + 4 * g]);
#pragma unroll
      for (int jn = 0; jn < NJV; ++jn) {
        f4 et = f4{0, 0, 0, 0};
#pragma unroll
        for (int r = 0; r < 4; ++r) et = mfma16(za[r], ft[jn][r], et);
        ft[jn] = et;
      }
      const f4 nqa = lds4(&NQs[c * LT + 4 * g]);
      const f4 cg = lds4(&cvec[4 * g]);
#pragma unroll
      for (int jn = 0; jn < NJV; ++jn)
#pragma unroll
        for (int r = 0; r < 4; ++r) ot[jn] = mfma16(nqa[r], ft[jn][r], ot[jn]);
      IO* ol = oh + static_cast<size_t>(t0) * DV + static_cast<unsigned>(4 * g * DV + vcol());
      auto store_row = [&](int r) __attribute__((always_inline)) {
#pragma unroll
        for (int jn = 0; jn + 1 < NJV; jn += 2)
          io_store2(ol + r * DV + 16 * jn, ol + r * DV + 16 * jn + 16, ot[jn][r], ot[jn + 1][r]);
        if (NJV % 2 == 1) io_store(ol + r * DV + 16 * (NJV - 1), ot[NJV - 1][r]);
      };
      if (t0 + C <= T) {   // uniform
#pragma unroll
        for (int r = 0; r < 4; ++r) store_row(r);
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (t0 + 4 * g + r < T) store_row(r);
      }
      __builtin_amdgcn_sched_barrier(0);
      decltype(Ops::tokens_b(f4{})) ce[NJV];
#pragma unroll
      for (int jn = 0; jn < NJV; ++jn) ce[jn] = Ops::tokens_b(ft[jn] * cg);
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const auto wa = Ops::w_load(Whm[blk & 1], Wl[blk & 1], 16 * b + c, c, g);
#pragma unroll
        for (int jn = 0; jn < NJV; ++jn) St[b][jn] = Ops::update(wa, ce[jn], St[b][jn]);
        if (b % 2 == 1) __builtin_amdgcn_sched_barrier(0);
      }
    };

    if (nblk > 0) {
      load_kq(0);
      stage(0, 0);
      if (nblk > 1) load_kq(C);
    }
    __syncthreads();  // block 0 staged
    for (int blk = 0; blk <= nblk; ++blk) {
      fresh();
      __syncthreads();  // (1)
      if (blk > 0) {
        load_v(C * (blk - 1));
        s_pass(blk - 1);
      }
      __syncthreads();  // (2) Z of the block before this one visible; its keys and queries are no longer read
      if (blk < nblk) {
        if (blk + 1 < nblk) stage(C * (blk + 1), (blk + 1) & 1);
        __syncthreads();  // (3) next block staged
      }
      if (blk > 0) s_update(blk - 1);
      if (blk + 2 < nblk) load_kq(C * (blk + 2));
    }
    if (a.S_T) {
      float* ST = a.S_T + static_cast<size_t>(head) * DV * D;
      int g2 = g, c2 = c;
      asm volatile("" : "+v"(g2), "+v"(c2));
      const int src = (row0 + c2) * D + 4 * g2;
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int jn = 0; jn < NJV; ++jn)
          *reinterpret_cast<float4*>(ST + src + 16 * jn * D + 16 * b) =
              make_float4(St[b][jn][0], St[b][jn][1], St[b][jn][2], St[b][jn][3]);
    }
  }
}

template <int D, int DV, int NWA, int NWS, int WPE>
hipError_t launch(const ForwardArgs& a, int io_dtype, hipStream_t stream) {
  ForwardArgs args = a;
  void* params[] = {&args};
  const void* fn;
  if (io_dtype == 1)
    fn = a.feature_map ? reinterpret_cast<const void*>(&chunk_pipe_kernel<D, DV, NWA, NWS, uint16_t, true, WPE>)
                       : reinterpret_cast<const void*>(&chunk_pipe_kernel<D, DV, NWA, NWS, uint16_t, false, WPE>);
  else
    fn = a.feature_map ? reinterpret_cast<const void*>(&chunk_pipe_kernel<D, DV, NWA, NWS, float, true, WPE>)
                       : reinterpret_cast<const void*>(&chunk_pipe_kernel<D, DV, NWA, NWS, float, false, WPE>);
  return hipLaunchKernel(fn, dim3(a.n_heads), dim3(64 * (NWA + NWS)), params, 0, stream);
}

template <int D, int DV, int NWA, int NWS, int WPE>
hipError_t launch_one_term(const ForwardArgs& a, hipStream_t stream) {
  ForwardArgs args = a;
  void* params[] = {&args};
  return hipLaunchKernel(reinterpret_cast<const void*>(&chunk_pipe_kernel<D, DV, NWA, NWS, uint16_t, false, WPE>),
                         dim3(a.n_heads), dim3(64 * (NWA + NWS)), params, 0, stream);
}

}  // namespace

// Waves of 16 columns, every pair of head sizes from d_k = 32 on but 128 x 16.
hipError_t launch_chunk_pipe_narrow(const ForwardArgs& a, int d_k, int d_v, int io_dtype, hipStream_t stream) {
  switch (d_k * 1000 + d_v) {
    case 32016: return launch<32, 16, 2, 1, 4>(a, io_dtype, stream);
    case 32032: return launch<32, 32, 2, 2, 4>(a, io_dtype, stream);
    case 32064: return launch<32, 64, 2, 4, 4>(a, io_dtype, stream);
    case 32096: return launch<32, 96, 2, 6, 4>(a, io_dtype, stream);
    case 32128: return launch<32, 128, 2, 8, 4>(a, io_dtype, stream);
    case 64016: return launch<64, 16, 4, 1, 4>(a, io_dtype, stream);
    case 64032: return launch<64, 32, 4, 2, 4>(a, io_dtype, stream);
    case 64064: return launch<64, 64, 4, 4, 4>(a, io_dtype, stream);
    case 64096: return launch<64, 96, 4, 6, 4>(a, io_dtype, stream);
    case 64128: return launch<64, 128, 4, 8, 4>(a, io_dtype, stream);
    case 96016: return launch<96, 16, 6, 1, 4>(a, io_dtype, stream);
    case 96032: return launch<96, 32, 6, 2, 4>(a, io_dtype, stream);
    case 96064: return launch<96, 64, 6, 4, 4>(a, io_dtype, stream);
    case 96096: return launch<96, 96, 6, 6, 3>(a, io_dtype, stream);
    case 96128: return launch<96, 128, 6, 8, 3>(a, io_dtype, stream);
    case 128032: return launch<128, 32, 8, 2, 4>(a, io_dtype, stream);
    case 128064: return launch<128, 64, 8, 4, 4>(a, io_dtype, stream);
    case 128096: return launch<128, 96, 8, 6, 4>(a, io_dtype, stream);
    case 128128: return launch<128, 128, 8, 8, 4>(a, io_dtype, stream);
    default: return hipErrorInvalidValue;
  }
}

// Waves of 32 columns, bf16 q and k without the feature map.
hipError_t launch_chunk_pipe_wide(const ForwardArgs& a, int d, hipStream_t stream) {
  switch (d) {
    case 64: return launch_one_term<64, 64, 2, 2, 4>(a, stream);
    case 128: return launch_one_term<128, 128, 4, 4, 4>(a, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace vla
