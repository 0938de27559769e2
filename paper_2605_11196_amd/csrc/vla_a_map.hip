// Phase 1 of the time-parallel mode: the A chain of every (head, time segment) and, one block behind on waves of their own,
// the affine map S_end = S_start P + Q of the segment.  Rows of S are independent (eq. (s-update)), so P is what the rows of
// the identity evolve into with v = 0 and Q what a zero state evolves into with the real v: (D + d_v) / 16 slabs of 16 rows,
// dealt out over the map waves.  The work of a block is laid out as in vla_chunk_pipe.hip:
//
//   (1)-(2)  A waves: one factorises I + G of block b, one forms c and Z and one -NQ^T of block b - 1
//            map waves: K^ X^T of block b - 1
//   (2)-(3)  A waves: W of block b to LDS and to the workspace      map waves: stage K^ and Q of block b + 1
//   (3)-(1)  A waves: A -= W W^T, Y = K^ A and the Gram matrices of block b + 1
//            map waves: E and the update of X of block b - 1
//
// What bounds it: the chain of a block (d = 64: 3.0 us alone on its compute unit, the factorisation 0.6 of it), and with two
// workgroups the vector instructions (about 500 a pair of A and map waves, 100 matrix ones beside them: 4.4 us for both).
// The A chain in one kernel (vla_two_phase.hip) and the maps in another, from the records, or on the A chain's own waves took,
// whole calls, bf16, before / with this kernel and its segment plan: 16 heads of 64, T = 4096 0.141 / 0.112 ms, T = 32768
// 0.479 / 0.449, T = 131072 1.565 / 1.576; one head, T = 8192 0.221 / 0.108; 16 heads of 128, T = 32768 1.334 / 1.224; 64 heads
// of 96, T = 2048 0.374 / 0.316; 16 heads of 32, T = 131072 0.881 / 0.783; float32, 16 heads of 64, T = 131072 2.09 / 1.92.
//
// The records that the rows of S read afterwards (1 / ||k_t||, W, Z, -NQ^T, -c; vla_mfma_util.h) go out on the
// way.
#include "vla_mfma_util.h"

namespace vla {
namespace {

constexpr int group(int n) { return n <= 1 ? 1 : 2 * group((n + 1) / 2); }   // the power of two from n on

// NWA waves own SL = D / NWA columns of A each; NWM map waves take the slabs w, w + NWM, ... (SPW slots each).  KT: operand
// terms of k and q (1: bf16 numbers, 3: float32 or mapped ones).  WPE: waves per SIMD to compile for.
template <int D, int NWA, int NWM, int SPW, typename IO, int KT, int WPE>
__global__ void __launch_bounds__(64 * (NWA + NWM), WPE) a_map_kernel(ForwardArgs a) {
  constexpr int SL = D / NWA;          // columns of A of one wave
  constexpr int NJ = SL / 16;          // 16-wide tiles among them
  static_assert(NWA >= 2 && SL % 16 == 0 && NJ <= 2, "whole tiles; two serial sections run at once");
  static_assert(KT == 3 || sizeof(IO) == 2, "one term: bf16 numbers");
  constexpr int NB = D / 16;
  constexpr int PSL = D / 16 / NWM;    // slots of the P run
  static_assert(D / 16 % NWM == 0 && SPW > PSL, "whole slots of the P run");
  constexpr int GRP = SPW > 3 ? 2 : SPW;   // slots whose update is in registers at a time
  using Ops = BlockOps<true, KT, D>;
  constexpr int NKB = NB / 2;
  constexpr int LDY = SL + 4;
  // Staging (by the map waves): a token row is split over TPR threads of EPT elements each, as in vla_chunk_pipe.hip.
  constexpr int NT = 64 * NWM;
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
  __shared__ __align__(16) uint16_t Qs[Ops::SIZE];         // q
  __shared__ __align__(16) u4 Whm[2][D * 4];               // W [j][t], terms h and m
  __shared__ __align__(16) u2 Wl[2][D * 4];                //           term l
  __shared__ __align__(16) float Yg[NWA][C * (LDY > LT ? LDY : LT)];   // a wave's slab of Y^T, then its partial G [s][t]
  __shared__ __align__(16) float GQp[2][NWA][C * LT];      // partial GQ [t][s]
  __shared__ __align__(16) float Lis[2][C * LT];           // L^{-1} [t][s]
  __shared__ __align__(16) float Lrs[2][C * LT];           // L [t][s]
  __shared__ __align__(16) float Zs[C * LT];               // Z   [t][s]
  __shared__ __align__(16) float wn2p[NWA][C];             // partial ||w_t||^2
  __shared__ __align__(16) float cvec[C];                  // -c_t
  __shared__ __align__(16) float rns[2][C];                // 1 / max(||k_t||, eps) over its power of two (key_scale)

  const int hs = blockIdx.x;                     // head * n_seg + seg
  const int head = hs / a.n_seg;
  const int seg = hs - head * a.n_seg;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  int c = lane & 15;
  int g = lane >> 4;
  // Once per block: what is derived from the lane (LDS and global offsets) is formed anew, not kept in registers.
  auto fresh = [&]() __attribute__((always_inline)) { renew(c, g); };
  // -1 on the diagonal for the splits: two registers where the waves have them, else formed where it is used
  constexpr bool kKeepIdentity = NB * NJ < 16 && NB * SPW < 16;
  u2 minus_one = minus_identity(c, g);
  asm volatile("" : "+v"(minus_one));
  auto identity = [&]() __attribute__((always_inline)) -> u2 {
    if constexpr (kKeepIdentity) return minus_one;
    else return minus_identity(c, g);
  };
  const int bb = seg * a.seg_blocks;             // first block of the segment
  const int tb = bb * C;                         // and its first token
  const int T = min(a.T, tb + a.seg_blocks * C); // one past its last token
  const int nblk = T > tb ? (T - tb + C - 1) / C : 0;
  const float eps = a.eps;
  const int nblk_all = (a.T + C - 1) / C;
  float* const wsh = a.ws + static_cast<size_t>(head) * head_stride(nblk_all, D);   // the records of this head

  if (wave < NWA) {
    // ================================================================ A chain
    const int w = wave;
    const int col0 = SL * w;
    f4 At[NB][NJ];   // At[b][jn][r] = A[16b + 4g + r][col0 + 16jn + c]
    {
      const float* A0 = a.seg_A ? a.seg_A + static_cast<size_t>(hs) * D * D
                                : (a.A0 ? a.A0 + static_cast<size_t>(head) * D * D : nullptr);
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
    auto record = [&](int blk) { return wsh + off_sm(nblk_all, D) + static_cast<size_t>(bb + blk) * SMB; };
    // -NQ^T[t][s] = -c_s H[s][t] for s <= t, H = L^{-1} GQ (one MFMA tile)
    auto form_nq = [&](int blk) __attribute__((always_inline)) {
      const f4 la = lds4(&Lis[blk & 1][c * LT + 4 * g]);
      f4 gq = f4{0, 0, 0, 0};
#pragma unroll
      for (int ww = 0; ww < NWA; ++ww) gq += lds4(&GQp[blk & 1][ww][c * LT + 4 * g]);
      f4 hq = f4{0, 0, 0, 0};
#pragma unroll
      for (int r = 0; r < 4; ++r) hq = mfma16(la[r], gq[r], hq);
      const float cs = strength(blk);
      f4 nq;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int s = 4 * g + r;
        const float csr = __shfl(cs, s);
        nq[r] = (s <= c) ? -(csr * hq[r]) : 0.0f;
      }
      *reinterpret_cast<f4*>(record(blk) + C * C + c * C + 4 * g) = nq;
    };
    // Z = (I + strict_lower(L) diag(c))^{-1}
    auto form_z = [&](int blk) __attribute__((always_inline)) {
      float* rec = record(blk);
      const float cs = strength(blk);
      if (g == 0) {
        cvec[c] = -cs;  // the residual tiles carry -E
        rec[2 * C * C + c] = -cs;
      }
      lower_inverse16(Lrs[blk & 1], cs, c, g, [&](int t, int s, float z) {
        Zs[t * LT + s] = z;
        rec[static_cast<unsigned>(t * C + s)] = z;
      });
    };
    // W^T = L^{-1} Y^T, partial ||w_t||^2, W to LDS and to the workspace
    auto form_w = [&](int blk) __attribute__((always_inline)) {
      const f4 la = lds4(&Lis[blk & 1][c * LT + 4 * g]);
      float* wg = wsh + off_wt(nblk_all, D) + static_cast<size_t>(bb + blk) * D * C;
      f4 n2 = f4{0, 0, 0, 0};
#pragma unroll
      for (int jn = 0; jn < NJ; ++jn) {
        f4 acc = f4{0, 0, 0, 0};
#pragma unroll
        for (int r = 0; r < 4; ++r) acc = mfma16(la[r], yt[jn][r], acc);
        n2 += acc * acc;
        Ops::w_store(Whm[blk & 1], Wl[blk & 1], col0 + 16 * jn + c, c, g, acc);
        *reinterpret_cast<f4*>(wg + (col0 + 16 * jn + c) * C + 4 * g) = acc;
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
      const int sw = (blk + hs) % NWA;      // rotates over waves / SIMDs
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
    if (a.A_T && seg == a.n_seg - 1) {
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
    // ================================================================ the map, one block behind; staging
    const int w = wave - NWA;
    const bool do_map = seg != a.n_seg - 1;      // nothing follows the last segment
    const int DV = a.d_v > 0 ? a.d_v : D;        // rows of the Q run
    // slot i: rows row_of(i) .. + 15 of the P run for i < PSL, of the Q run from there on
    auto row_of = [&](int i) { return 16 * (w + NWM * (i < PSL ? i : i - PSL)); };
    auto owns = [&](int i) { return i < PSL || row_of(i) < DV; };
    f4 Xt[NB][SPW];   // Xt[b][i][r] = X[row_of(i) + c][16b + 4g + r]
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int i = 0; i < SPW; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) Xt[b][i][r] = (i < PSL && row_of(i) + c == 16 * b + 4 * g + r) ? 1.0f : 0.0f;
    const size_t slab = static_cast<size_t>(head) * static_cast<size_t>(a.T) * D;
    const IO* qh = static_cast<const IO*>(a.q) + slab;
    const IO* kh = static_cast<const IO*>(a.k) + slab;
    float* const RN = wsh + off_rn(nblk_all, D);
    const bool fmap = a.feature_map != 0;
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
      if (KT == 3 && fmap) {
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
      if (sseg() == 0) RN[t0 + srow()] = live ? rn : 0.0f;   // rows past the end: zero keys
      // one term: k times a power of two, the rest of the norm on the results; else k^ as the rows of S form it again
      const KeyScale ks = KT == 1 ? key_scale(rn) : KeyScale{rn, 1.0f};
#pragma unroll
      for (int e = 0; e < EPT; ++e) kx[e] *= ks.pow2;
      if (sseg() == 0) rns[buf][srow()] = ks.rest;
#pragma unroll
      for (int e = 0; e < EPT; e += 4) Ops::put4(Ksb[buf], srow(), sseg() + e, f4{kx[e], kx[e + 1], kx[e + 2], kx[e + 3]});
      float qx[EPT];
      qpre.unpack(qx);
      if (KT == 3 && fmap) {
#pragma unroll
        for (int e = 0; e < EPT; ++e) qx[e] = elu_plus_one(qx[e]);
      }
      if (ragged) {
#pragma unroll
        for (int e = 0; e < EPT; ++e) qx[e] = live ? qx[e] : 0.0f;
      }
#pragma unroll
      for (int e = 0; e < EPT; e += 4) Ops::put4(Qs, srow(), sseg() + e, f4{qx[e], qx[e + 1], qx[e + 2], qx[e + 3]});
    };
    const IO* vh = static_cast<const IO*>(a.v) + static_cast<size_t>(head) * static_cast<size_t>(a.T) * DV;
    IO vpre[SPW - PSL][4];   // V[t0 + 4g + r][row_of(i) + c] of the Q run
    auto load_v = [&](int t0) __attribute__((always_inline)) {
#pragma unroll
      for (int i = PSL; i < SPW; ++i) {
        if (!owns(i)) continue;   // uniform
        const IO* vb = vh + static_cast<size_t>(t0) * DV + row_of(i);
        if (t0 + C <= T) {   // uniform
          const IO* vl = vb + static_cast<unsigned>(4 * g * DV + c);
#pragma unroll
          for (int r = 0; r < 4; ++r) vpre[i - PSL][r] = vl[r * DV];
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r) vpre[i - PSL][r] = vb[static_cast<unsigned>(min(4 * g + r, T - 1 - t0) * DV + c)];
        }
      }
    };
    f4 ft[SPW];
    // -F^T = K^ X^T - V^T
    auto x_pass = [&](int blk) __attribute__((always_inline)) {
      const uint16_t* Ks = Ksb[blk & 1];
#pragma unroll
      for (int i = 0; i < SPW; ++i) ft[i] = f4{0, 0, 0, 0};
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb) {
        const Terms<KT> ka = Ops::operand(Ks, kb, c, g);
#pragma unroll
        for (int i = 0; i < SPW; ++i) {
          ft[i] = Ops::sweep(ka, split_tiles(Xt[2 * kb][i], Xt[2 * kb + 1][i], identity()), ft[i]);
          __builtin_amdgcn_sched_barrier(0);   // one split at a time in registers
        }
      }
      const f4 rn4 = lds4(&rns[blk & 1][4 * g]);
#pragma unroll
      for (int i = 0; i < SPW; ++i) ft[i] *= rn4;
    };
    // -E^T = Z (-F^T), X^T += W diag(c) E^T
    auto x_update = [&](int blk) __attribute__((always_inline)) {
      const int t0 = tb + C * blk;
      const f4 za = lds4(&Zs[c * LT + 4 * g]);
      const f4 cg = lds4(&cvec[4 * g]);
#pragma unroll
      for (int i = PSL; i < SPW; ++i) {
        if (!owns(i)) continue;
        if (t0 + C > T) {  // uniform: rows past the end of the sequence are zero tokens
#pragma unroll
          for (int r = 0; r < 4; ++r) vpre[i - PSL][r] = (t0 + 4 * g + r < T) ? vpre[i - PSL][r] : IO(0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) ft[i][r] += neg_widen(vpre[i - PSL][r]);
      }
#pragma unroll
      for (int i0 = 0; i0 < SPW; i0 += GRP) {
        decltype(Ops::tokens_b(f4{})) ce[GRP];
#pragma unroll
        for (int i = i0; i < i0 + GRP && i < SPW; ++i) {
          f4 et = f4{0, 0, 0, 0};
#pragma unroll
          for (int r = 0; r < 4; ++r) et = mfma16(za[r], ft[i][r], et);
          ce[i - i0] = Ops::tokens_b(et * cg);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          const auto wa = Ops::w_load(Whm[blk & 1], Wl[blk & 1], 16 * b + c, c, g);
#pragma unroll
          for (int i = i0; i < i0 + GRP && i < SPW; ++i) Xt[b][i] = Ops::update(wa, ce[i - i0], Xt[b][i]);
          if (b % 2 == 1) __builtin_amdgcn_sched_barrier(0);
        }
      }
    };

    if (nblk > 0) {
      load_kq(tb);
      stage(tb, 0);
      if (nblk > 1) load_kq(tb + C);
    }
    __syncthreads();  // block 0 staged
    for (int blk = 0; blk <= nblk; ++blk) {
      fresh();
      __syncthreads();  // (1)
      if (blk > 0 && do_map) {
        load_v(tb + C * (blk - 1));
        x_pass(blk - 1);
      }
      __syncthreads();  // (2) Z of the block before this one visible; its keys are no longer read
      if (blk < nblk) {
        if (blk + 1 < nblk) stage(tb + C * (blk + 1), (blk + 1) & 1);
        __syncthreads();  // (3) next block staged
      }
      if (blk > 0 && do_map) x_update(blk - 1);
      if (blk + 2 < nblk) load_kq(tb + C * (blk + 2));
    }
    if (do_map) {   // per (head, segment): P [D][D], then Q [DV][D]
      float* pq = a.seg_PQ + static_cast<size_t>(hs) * (static_cast<size_t>(D + DV) * D);
#pragma unroll
      for (int i = 0; i < SPW; ++i) {
        if (!owns(i)) continue;
        float* out = pq + (i < PSL ? 0 : D * D) + (row_of(i) + c) * D + 4 * g;
#pragma unroll
        for (int b = 0; b < NB; ++b) *reinterpret_cast<f4*>(out + 16 * b) = Xt[b][i];
      }
    }
  }
}

template <int D, int NWA, int NWM, int SPW, int WPE>
hipError_t launch(const ForwardArgs& a, int io_dtype, hipStream_t stream) {
  ForwardArgs args = a;
  void* params[] = {&args};
  const long long wgs = static_cast<long long>(a.n_heads) * a.n_seg;
  if (wgs > 0x7fffffffLL) return hipErrorInvalidValue;
  const void* fn = io_dtype != 1        ? reinterpret_cast<const void*>(&a_map_kernel<D, NWA, NWM, SPW, float, 3, WPE>)
                   : a.feature_map != 0 ? reinterpret_cast<const void*>(&a_map_kernel<D, NWA, NWM, SPW, uint16_t, 3, WPE>)
                                        : reinterpret_cast<const void*>(&a_map_kernel<D, NWA, NWM, SPW, uint16_t, 1, WPE>);
  return hipLaunchKernel(fn, dim3(static_cast<unsigned>(wgs)), dim3(64 * (NWA + NWM)), params, 0, stream);
}

}  // namespace

// Waves of 16 columns up to d = 96, of 32 at d = 128 (three-term keys leave no registers with 16 waves: 16 heads, T = 32768,
// float32 1.43 against 1.51 ms; bf16 1.22 and 1.25).  d = 64 on two A waves of 32 columns: 16 heads, T = 131072 1.58 -> 1.73 ms.
// Five slots a wave (heads of 32, d_v beyond 96) spill registers where they are compiled for four waves a SIMD.  Up to 256 pairs
// of head and segment, one a compute unit, they are compiled for two: 16 heads, T = 4096, float32 152 -> 141 us, bf16 137 -> 130;
// one head, T = 512, float32 46.1 -> 44.7.  With more pairs than that the workgroups that fit count: 1024 pairs (16 heads,
// T = 16384) on two 289 -> 294, bf16 233 -> 253.
hipError_t launch_a_map(const ForwardArgs& a, int d, int io_dtype, hipStream_t stream) {
  const int dv = a.d_v > 0 ? a.d_v : d;
  const bool few = static_cast<long long>(a.n_heads) * a.n_seg <= 256;
  switch (d) {
    case 32:
      return dv <= 32   ? launch<32, 2, 2, 2, 4>(a, io_dtype, stream)
             : dv == 64 ? launch<32, 2, 2, 3, 4>(a, io_dtype, stream)
             : dv == 96 ? launch<32, 2, 2, 4, 4>(a, io_dtype, stream)
             : few      ? launch<32, 2, 2, 5, 2>(a, io_dtype, stream)
                        : launch<32, 2, 2, 5, 4>(a, io_dtype, stream);
    case 64: return dv <= 64 ? launch<64, 4, 4, 2, 4>(a, io_dtype, stream) : launch<64, 4, 4, 3, 4>(a, io_dtype, stream);
    case 96: return dv <= 96 ? launch<96, 6, 6, 2, 3>(a, io_dtype, stream) : launch<96, 6, 6, 3, 3>(a, io_dtype, stream);
    case 128: return launch<128, 4, 8, 2, 3>(a, io_dtype, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace vla
