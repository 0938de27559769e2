// Block form with the optional lines of Algorithm 1 (the algebra is at the head of vla_chunk_general.hip), the A chain and
// the S chain on waves of their own.  A never reads S, so while the A waves go through a block's chain of dependent steps
// the S waves finish the block before it and begin this one:
//
//   A waves                                              S waves
//   (0)-(1)  Y, X and the partial Gram matrices          -E, o and the update of S of block b - 1
//   (1)-(2)  Cholesky; sums of the Gram matrices;        first half of the pass over S (K^ S^T and Q S^T)
//            read-out denominators
//   (2)-(3)  W, Alpha, P, the key sum                    second half
//   (3)-(0)  A -= W W^T; c, Z; NQ                        stage K^, Q, U of block b + 1
//
// K^, Q, U and Alpha need one buffer each.  The partial Gram matrices of the A waves stay in the accumulator layout (lane l
// keeps what lane l reads) and share their LDS with Y, X and W, so that two workgroups of d = 128 fit a compute unit.
//
// What bounds it: with both states on every wave (vla_chunk_general.hip) a block is the sum of the two chains behind six
// barriers, the matrix unit 31 % and the vector unit 50 % of the cycles.  Here four waves of two heads share a SIMD: in a
// block 418 matrix and some 1320 other vector instructions a head and SIMD; matrix pipes busy 57 % of the cycles, vector issue 42 %
// beside them, LDS 48 %.  2048 heads of 128, 8192 tokens, bf16, every option: 35.9 -> 25.2 ms (16.8 us -> 11.8 us a block of two heads).  Of that: directions in bf16 stay one term
// (three products with A instead of six), the residuals of the splits go to the matrix unit (split3_cut_matrix), the Gram
// matrices are formed from a wave's own columns, without the barrier that a whole Y needs.  k^ is kept once more in float32 for the refresh terms and
// the key sum (256 heads of 128, 512 tokens 0.258 -> 0.231 ms, 2048 heads 1.63 -> 1.59), and the key sum as split terms.
// v is fetched beside the staging: beside the pass over S it cost 100 more spilled registers.
#include "vla_mfma_util.h"

namespace vla {
namespace {

constexpr int group(int n) { return n <= 1 ? 1 : 2 * group((n + 1) / 2); }   // the power of two from n on

enum UKind {
  kUKey = 0,       // u = k^, no refresh: Y = X, two Gram matrices
  kUSeparate,      // a given u: two sweeps of A, five Gram matrices
  kUKeyRefresh,    // u = k^ with a refresh period: one sweep, Y and X differ by the refresh terms
};

// NWA waves own SL = D / NWA columns of A each, NWS waves DV / NWS rows of S each.  WPE: waves per SIMD to compile for.
template <int D, int DV, int NWA, int NWS, typename IO, int UK, int WPE>
__global__ void __launch_bounds__(64 * (NWA + NWS), WPE) chunk_general_pipe_kernel(ForwardArgs a) {
  constexpr int SL = D / NWA;          // columns of A of one wave
  constexpr int NJ = SL / 16;          // 16-wide tiles among them
  constexpr int NJV = DV / (16 * NWS); // row tiles of S of one wave
  static_assert(NWA >= 2 && NJ <= 2 && SL % 16 == 0 && DV % (16 * NWS) == 0 && D % 32 == 0, "whole tiles; serial sections side by side");
  constexpr bool FULL = UK != kUKey;
  constexpr int NB = D / 16;
  constexpr int NKB = NB / 2;
  using Ops = BlockOps<true, 3, D>;    // k^ normalised, q mapped: float32 numbers
  // u: bf16 directions are staged as they come (times a power of two) and their scale goes on the results
  constexpr int UT = UK == kUSeparate && sizeof(IO) == 2 ? 1 : 3;
  using UOps = BlockOps<true, UT, D>;
  constexpr int LDY = SL + 4;
  // Staging (by the S waves): a token row is split over TPR threads of EPT elements each, as in vla_chunk_pipe.hip.
  constexpr int NT = 64 * NWS;
  constexpr int TPR0 = NT / C;
  constexpr bool PADDED = (TPR0 & (TPR0 - 1)) != 0 || (C * D / NT) % 4 != 0;
  constexpr int PIECE = group(D / 4) <= 16 && C * group(D / 4) <= NT ? 4 : C * group(D / 8) <= NT ? 8 : 16;
  constexpr int EPT = PADDED ? PIECE : C * D / NT;
  constexpr int TPR = group(D / EPT);
  static_assert(EPT % 4 == 0 && TPR <= 32 && C * TPR <= NT && D % EPT == 0 && D / EPT <= TPR, "staging layout");

  // Gram matrices, [m][n] = sum_j left[m][j] right[n][j]
  enum { kG = 0, kGK, kGQ, kGX, kXQ };   // Y U^T, Y K^^T, Y Q^T, X K^^T, X Q^T
  // (u = k^: G and Y Q^T stand for all of them)
  // One region: of every wave its slabs of Y and X until their operands are read, then its partial Gram matrices; later W.
  // The sums of GK, GQ, GX and XQ take the last wave's places, behind W; with u = k^ the two have an array of their own.
  constexpr int kSlab = C * LDY;
  constexpr int kXSlab = 3 * 256;        // X's slab: the partial matrices of X go there, those of Y before it
  constexpr int kOwn = !FULL ? (kSlab > 512 ? kSlab : 512) : kXSlab + (kSlab > 512 ? kSlab : 512);   // floats of a wave
  static_assert(kSlab <= kXSlab, "a wave's slabs");
  constexpr int kW = D * 24;
  constexpr int kRegion = NWA * kOwn > kW ? NWA * kOwn : kW;
  static_assert(!FULL || (NWA - 1) * kOwn + 256 >= kW, "the sums lie behind W");

  __shared__ __align__(16) uint16_t Ks[Ops::SIZE];          // K^ [t][slot], terms
  __shared__ __align__(16) uint16_t Qs[Ops::SIZE];          // Q
  __shared__ __align__(16) uint16_t Usb[UK == kUSeparate ? UOps::SIZE : 8];   // U
  // k^ once more as float32, for the steps that need single elements (refresh terms, key sum); recombined from the terms
  // where it would cost a workgroup of the compute unit
  constexpr bool kF32Keys = D != 64;
  constexpr int LDF = D + 4;
  __shared__ __align__(16) float Kf[kF32Keys ? C * LDF : 4];
  __shared__ __align__(16) uint16_t zts[3][D];              // the key sum's terms, in slot order
  __shared__ __align__(16) float region[kRegion];
  __shared__ __align__(16) float sums[FULL ? 4 : 512];
  __shared__ __align__(16) u4 Ahm[D * 4];                   // Alpha [j][t], terms h and m
  __shared__ __align__(16) u2 Al[D * 4];                    //               term l
  __shared__ __align__(16) float Lis[C * LT];               // L^{-1} [t][s]
  __shared__ __align__(16) float Ps[C * LT];                // P transposed: [t][s] = alpha_s . k^_t
  __shared__ __align__(16) float Zs[C * LT];                // Z   [t][s]
  __shared__ __align__(16) float NQs[C * LT];               // -NQ^T [t][s]
  __shared__ __align__(16) float wn2p[NWA][C];              // partial ||alpha_t||^2
  __shared__ __align__(16) float cvec[C];                   // -c_t
  __shared__ __align__(16) float rdens[C];                  // 1 / max(q_t . zkey_t, eps)
  __shared__ __align__(16) float nks[C];                    // max(||k_t||, eps)
  __shared__ __align__(16) float urest[C];                  // scale of u_t over its power of two (UT = 1)
  __shared__ __align__(16) float zks[D];                    // running key sum
  __shared__ __align__(16) float ens[2][C + 4];             // eta n_i, i = 0..C: refresh steps among a block's first i tokens
  u4* const Whm = reinterpret_cast<u4*>(region);            // W [j][t]
  u2* const Wl = reinterpret_cast<u2*>(region + D * 16);
  const uint16_t* const Us = UK == kUSeparate ? Usb : Ks;

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
  const int period = a.refresh_period;
  const bool norm_out = a.normalise_output != 0;

  if (wave < NWA) {
    // ================================================================ A chain
    const int w = wave;
    const int col0 = SL * w;
    const bool key_sum = norm_out || a.zkey_T != nullptr;
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
    // element j of the key sum: the value, and its terms (split3_rne) for the read-out denominators
    auto put_zkey = [&](int j, float z) __attribute__((always_inline)) {
      zks[j] = z;
      u2 h, m, l;
      split3_rne(f4{z, 0, 0, 0}, h, m, l);
      const int at = kslot(j & ~3) + (j & 3);
      zts[0][at] = static_cast<uint16_t>(h[0]);
      zts[1][at] = static_cast<uint16_t>(m[0]);
      zts[2][at] = static_cast<uint16_t>(l[0]);
    };
    if (lane < SL) put_zkey(col0 + lane, a.zkey0 ? a.zkey0[static_cast<size_t>(head) * D + col0 + lane] : 0.0f);
    auto key = [&](int t, int j) __attribute__((always_inline)) -> float {
      if constexpr (kF32Keys) return Kf[t * LDF + j];
      else return Ops::get(Ks, t, j);
    };
    auto part = [&](int i, int ww) __attribute__((always_inline)) -> f4& {
      if constexpr (!FULL) i = i == kGQ || i == kXQ ? 1 : 0;
      return *reinterpret_cast<f4*>(&region[ww * kOwn + i * 256 + (16 * g + c) * 4]);
    };
    // the sum of matrix i over the waves, and where it stands
    auto total = [&](int i) __attribute__((always_inline)) -> f4 {
      f4 x = part(i, 0);
#pragma unroll
      for (int ww = 1; ww < NWA; ++ww) x += part(i, ww);
      return x;
    };
    auto sum = [&](int i) __attribute__((always_inline)) -> f4& {
      if constexpr (FULL) return part(i, NWA - 1);
      else return *reinterpret_cast<f4*>(&sums[(i == kGQ || i == kXQ ? 256 : 0) + (16 * g + c) * 4]);
    };
    f4 yt[NJ], xt[NJ];
    // Y^T = U A, X^T = K^ A (this wave's columns) and the partial Gram matrices over them
    auto y_and_gram = [&](int blk) __attribute__((always_inline)) {
#pragma unroll
      for (int jn = 0; jn < NJ; ++jn) yt[jn] = xt[jn] = f4{0, 0, 0, 0};
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb) {
#pragma unroll
        for (int jn = 0; jn < NJ; ++jn) {
          const auto ab = split_tiles(At[2 * kb][jn], At[2 * kb + 1][jn], identity());
          xt[jn] = Ops::sweep(Ops::operand(Ks, kb, c, g), ab, xt[jn]);
          if constexpr (UK == kUSeparate) yt[jn] = UOps::sweep(UOps::operand(Us, kb, c, g), ab, yt[jn]);
          if (NJ > 1) __builtin_amdgcn_sched_barrier(0);   // one split at a time in registers
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (UK == kUSeparate) {
        if constexpr (UT == 1) {
          const f4 ur = lds4(&urest[4 * g]);
#pragma unroll
          for (int jn = 0; jn < NJ; ++jn) yt[jn] *= ur;
        }
      } else {
#pragma unroll
        for (int jn = 0; jn < NJ; ++jn) yt[jn] = xt[jn];
      }
      if constexpr (FULL) {
        if (period > 0) {  // y'_t = y_t + eta n_t u_t,  x'_t = x_t + eta n'_t k^_t  (n'_t = n_{t+1})
          const float* en = ens[blk & 1];
          f4 e0 = lds4(&en[4 * g]);
          const f4 e1 = f4{e0[1], e0[2], e0[3], en[4 * g + 4]};
          if constexpr (UT == 1) e0 *= lds4(&urest[4 * g]);
#pragma unroll
          for (int jn = 0; jn < NJ; ++jn)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const float kx = key(4 * g + r, col0 + 16 * jn + c);
              const float ux = UK == kUSeparate ? UOps::get(Us, 4 * g + r, col0 + 16 * jn + c) : kx;
              yt[jn][r] = fmaf(e0[r], ux, yt[jn][r]);
              xt[jn][r] = fmaf(e1[r], kx, xt[jn][r]);
            }
        }
      }
      // token rows to operand rows: through LDS, where the partial matrices go afterwards (LDS operations of one wave are ordered)
      float* Yw = &region[w * kOwn];
      auto operand_of = [&](const f4 (&x)[NJ], float* slab) __attribute__((always_inline)) {
#pragma unroll
        for (int jn = 0; jn < NJ; ++jn)
#pragma unroll
          for (int r = 0; r < 4; ++r) slab[(4 * g + r) * LDY + 16 * jn + c] = x[jn][r];
        const f4 x0 = lds4(&slab[c * LDY + 4 * g]);
        if constexpr (NJ > 1) return split_tiles(x0, lds4(&slab[c * LDY + 16 + 4 * g]), identity());
        else return split_tile(x0, identity());
      };
      // this wave's columns of a staged operand
      auto own_columns = [&](auto ops, const uint16_t* src) __attribute__((always_inline)) {
        if constexpr (NJ > 1) return decltype(ops)::operand(src, w, c, g);
        else return decltype(ops)::half_operand(src, w, c, g);
      };
      const f4 zero{0, 0, 0, 0};
      {
        const auto y = operand_of(yt, Yw);
        [[maybe_unused]] f4 gg;
        if constexpr (UK == kUSeparate) {
          const auto u = own_columns(UOps{}, Us);
          if constexpr (UT == 1) gg = mfma_terms_left(y, u, zero) * urest[c];
          else gg = mfma_terms(y, u, zero);
        }
        if constexpr (UK == kUSeparate) part(kG, w) = gg;
        __builtin_amdgcn_sched_barrier(0);
        const f4 gk = mfma_terms(y, own_columns(Ops{}, Ks), zero);
        part(kGK, w) = gk;
        if constexpr (UK == kUKeyRefresh) part(kG, w) = gk;
        __builtin_amdgcn_sched_barrier(0);
        part(kGQ, w) = mfma_terms(y, own_columns(Ops{}, Qs), zero);
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (FULL) {
        const auto x = operand_of(xt, Yw + kXSlab);
        __builtin_amdgcn_sched_barrier(0);
        part(kGX, w) = mfma_terms(x, own_columns(Ops{}, Ks), zero);
        __builtin_amdgcn_sched_barrier(0);
        part(kXQ, w) = mfma_terms(x, own_columns(Ops{}, Qs), zero);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    // read-out denominators: q_t . zkey_t for t = 4g + r, the key sum's part and the block's own, s = c <= t
    auto denominators = [&]() __attribute__((always_inline)) {
      f4 qk = f4{0, 0, 0, 0}, qz = f4{0, 0, 0, 0};
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb) {
        const Terms<3> q = Ops::operand(Qs, kb, c, g);
        qk = Ops::sweep(q, Ops::operand(Ks, kb, c, g), qk);
        Terms<3> z;   // the same column 16 times
#pragma unroll
        for (int i = 0; i < 3; ++i) z.t[i] = *reinterpret_cast<const u4*>(&zts[i][32 * kb + 8 * g]);
        qz = Ops::sweep(q, z, qz);
      }
      const float nk = nks[c];
      f4 den;
#pragma unroll
      for (int r = 0; r < 4; ++r) den[r] = qz[r] + row_sum16((c <= 4 * g + r) ? qk[r] * nk : 0.0f);
#pragma unroll
      for (int r = 0; r < 4; ++r) den[r] = 1.0f / fmaxf(den[r], eps);
      if (c == 0) *reinterpret_cast<f4*>(&rdens[4 * g]) = den;
    };
    // zkey += sum over the block's tokens of ||k_s|| k^_s, this wave's columns
    auto key_sum_pass = [&]() __attribute__((always_inline)) {
      const f4 nk = lds4(&nks[4 * g]);
#pragma unroll
      for (int jn = 0; jn < NJ; ++jn) {
        float z = 0.0f;
#pragma unroll
        for (int r = 0; r < 4; ++r) z = fmaf(nk[r], key(4 * g + r, col0 + 16 * jn + c), z);
        z += __shfl_xor(z, 16);
        z += __shfl_xor(z, 32);
        if (g == 0) put_zkey(col0 + 16 * jn + c, zks[col0 + 16 * jn + c] + z);
      }
    };
    // W^T = L^{-1} Y^T,  Hm = L^{-1} (Y K^^T),  Alpha^T = X^T - M W^T,  ||alpha_t||^2;  P on one wave
    auto form_w = [&](bool with_p) __attribute__((always_inline)) {
      const f4 la = lds4(&Lis[c * LT + 4 * g]);
      const f4 gk = sum(kGK);
      f4 pt = f4{0, 0, 0, 0};
      if (with_p) pt = sum(kGX);
      f4 hm = f4{0, 0, 0, 0}, mop;
#pragma unroll
      for (int r = 0; r < 4; ++r) hm = mfma16(la[r], gk[r], hm);
#pragma unroll
      for (int r = 0; r < 4; ++r) mop[r] = (4 * g + r <= c) ? hm[r] : 0.0f;   // M[t = c][s = 4g + r] = Hm[s][t], s <= t
      f4 n2 = f4{0, 0, 0, 0};
#pragma unroll
      for (int jn = 0; jn < NJ; ++jn) {
        f4 acc = f4{0, 0, 0, 0};
#pragma unroll
        for (int r = 0; r < 4; ++r) acc = mfma16(la[r], yt[jn][r], acc);
        Ops::w_store(Whm, Wl, col0 + 16 * jn + c, c, g, acc);
        f4 at = xt[jn];
#pragma unroll
        for (int r = 0; r < 4; ++r) at = mfma16(mop[r], -acc[r], at);
        n2 += at * at;
        Ops::w_store(Ahm, Al, col0 + 16 * jn + c, c, g, at);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) n2[r] = row_sum16(n2[r]);
      if (c == 0) *reinterpret_cast<f4*>(&wn2p[w][4 * g]) = n2;
      if (with_p) {
#pragma unroll
        for (int r = 0; r < 4; ++r) pt = mfma16(mop[r], -hm[r], pt);   // P[s = 4g + r][t = c]
        *reinterpret_cast<f4*>(&Ps[c * LT + 4 * g]) = pt;
      }
    };
    // c_t on lane t of every row of 16: alpha^_t = c_t alpha_t
    auto strength = [&]() __attribute__((always_inline)) -> float {
      float wn2 = 0.0f;
#pragma unroll
      for (int ww = 0; ww < NWA; ++ww) wn2 += wn2p[ww][c];
      return __builtin_amdgcn_rcpf(fmaxf(__builtin_amdgcn_sqrtf(wn2), eps));
    };
    auto form_z = [&]() __attribute__((always_inline)) {   // N[t][s] = c_s P[s][t]
      const float cs = strength();
      if (g == 0) cvec[c] = -cs;
      lower_inverse16(Ps, cs, c, g, [&](int t, int s, float z) { Zs[t * LT + s] = z; });
    };
    // NQ[s][t] = c_s AQ[s][t] for s <= t, AQ = X Q^T - M (L^{-1} Y Q^T)
    auto form_nq = [&]() __attribute__((always_inline)) {
      const f4 la = lds4(&Lis[c * LT + 4 * g]);
      const f4 gk = sum(kGK), gq = sum(kGQ);
      f4 aq = sum(kXQ);
      f4 hm = f4{0, 0, 0, 0}, nhq = f4{0, 0, 0, 0};
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        hm = mfma16(la[r], gk[r], hm);
        nhq = mfma16(-la[r], gq[r], nhq);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) aq = mfma16((4 * g + r <= c) ? hm[r] : 0.0f, nhq[r], aq);
      const float cs = strength();
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int s = 4 * g + r;
        const float csr = __shfl(cs, s);
        NQs[c * LT + s] = (s <= c) ? -(csr * aq[r]) : 0.0f;
      }
    };
    auto update_a = [&](int blk, int len) __attribute__((always_inline)) {
      Ops::template downdate<NB, NJ, (NB * NJ >= 16)>(Whm, Wl, col0 + c, c, g, blk & 1,
                                                      [&](int b, int jn) -> f4& { return At[b][jn]; });
      if (FULL && period > 0) {   // + eta n on the diagonal, n counted over the live tokens
        const float en_end = ens[blk & 1][len];
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int jn = 0; jn < NJ; ++jn)
            if (b == NJ * w + jn) {
#pragma unroll
              for (int r = 0; r < 4; ++r) At[b][jn][r] += (4 * g + r == c) ? en_end : 0.0f;
            }
      }
    };

    __syncthreads();  // (0) block 0 staged
    for (int blk = 0; blk < nblk; ++blk) {
      fresh();
      const int len = T - C * blk < C ? T - C * blk : C;
      const int sw = (blk + head) % NWA;      // rotates over waves / SIMDs
      const int sw2 = (sw + 1) % NWA, sw3 = (sw + 2) % NWA, sw4 = (sw + 3) % NWA;
      y_and_gram(blk);
      __syncthreads();  // (1) partial Gram matrices visible
      if (w == sw) {
        __builtin_amdgcn_s_setprio(3);
        // u_s . y_t: entries with s < t from their mirror images (with a refresh they are the ones that count)
        cholesky16<false>(total(kG), nullptr, Lis, c, g);
        __builtin_amdgcn_s_setprio(0);
      } else if (w == sw2) {
        const f4 gk = total(kGK), gq = total(kGQ);
        sum(kGK) = gk;
        sum(kGQ) = gq;
        if constexpr (FULL) {
          const f4 gx = total(kGX), xq = total(kXQ);
          sum(kGX) = gx;
          sum(kXQ) = xq;
        }
      }
      if (norm_out && w == (NWA > 2 ? sw3 : sw2)) denominators();
      __syncthreads();  // (2) L^{-1} and the sums visible, the key sum no longer read
      form_w(w == sw4);
      if (key_sum) key_sum_pass();
      __syncthreads();  // (3) W, Alpha, P and the norms visible; K^, Q, U no longer read
      if (w == sw2) {
        __builtin_amdgcn_s_setprio(3);
        form_z();
        __builtin_amdgcn_s_setprio(0);
      } else if (w == (NWA > 2 ? sw3 : sw)) {
        form_nq();
      }
      update_a(blk, len);
      __syncthreads();  // (0) Z, NQ and c visible, next block staged, W no longer read
    }
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
    if (a.zkey_T != nullptr && lane < SL) a.zkey_T[static_cast<size_t>(head) * D + col0 + lane] = zks[col0 + lane];
  } else {
    // ================================================================ S chain; staging
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
    const IO* uh = UK == kUSeparate ? static_cast<const IO*>(a.u) + slab : kh;
    const bool fmap = a.feature_map != 0;
    const bool stage_wave = !PADDED || 64 * w < C * TPR;
    auto tid = [&]() { return 64 * w + 16 * g + c; };
    auto srow = [&]() { return tid() / TPR; };
    auto sseg = [&]() { return (tid() % TPR) * EPT; };
    auto stager = [&]() { return !PADDED || (tid() < C * TPR && sseg() < D); };
    RawRow<IO, EPT> kpre, qpre, upre;
    // Loads never branch on the row: rows past the end read the last valid row and are zeroed when consumed.
    auto load_kqu = [&](int t0) __attribute__((always_inline)) {
      if (stager()) {
        const int tr = t0 + srow();
        const unsigned off = static_cast<unsigned>((tr < T ? tr : T - 1) * D + sseg());
        kpre.load(kh + off);
        qpre.load(qh + off);
        if constexpr (UK == kUSeparate) upre.load(uh + off);
      }
    };
    auto row_total = [&](float x) __attribute__((always_inline)) -> float {
      if constexpr (TPR == 16) return row_sum16(x);
#pragma unroll
      for (int off = TPR / 2; off >= 1; off >>= 1) x += __shfl_xor(x, off);
      return x;
    };
    // 1 / max(sqrt(ss), eps): hardware reciprocal square root refined by one Newton step
    auto inv_norm = [&](float ss, float& clamped) __attribute__((always_inline)) -> float {
      clamped = fmaxf(ss, eps * eps);
      const float rn = __builtin_amdgcn_rsqf(clamped);
      return rn * fmaf(-0.5f * clamped * rn, rn, 1.5f);
    };
    const bool key_elements = kF32Keys && (period > 0 || norm_out || a.zkey_T != nullptr);
    auto unpack = [&](const RawRow<IO, EPT>& raw, float (&x)[EPT], bool ragged, bool live, bool map) __attribute__((always_inline)) {
      if (stager()) {
        raw.unpack(x);
      } else {
#pragma unroll
        for (int e = 0; e < EPT; ++e) x[e] = 0.0f;
      }
      if (map) {
#pragma unroll
        for (int e = 0; e < EPT; ++e) x[e] = elu_plus_one(x[e]);
      }
      if (ragged || PADDED) {
#pragma unroll
        for (int e = 0; e < EPT; ++e) x[e] = live ? x[e] : 0.0f;
      }
    };
    auto stage = [&](int t0, int buf) __attribute__((always_inline)) {
      if constexpr (FULL) {
        if (tid() <= C && period > 0) {  // multiples of the period among the step indices idx0 .. idx0 + tid - 1, 1-based
          const int idx0 = a.step_offset + t0 + 1;
          ens[buf][tid()] = a.refresh_eta * static_cast<float>((idx0 - 1 + tid()) / period - (idx0 - 1) / period);
        }
      }
      if (!stage_wave) return;
      const bool ragged = t0 + C > T;   // uniform
      const bool live = t0 + srow() < T && stager();
      float x[EPT];
      unpack(kpre, x, ragged, live, fmap);
      float ss = 0.0f;
#pragma unroll
      for (int e = 0; e < EPT; ++e) ss = fmaf(x[e], x[e], ss);
      float sm;
      const float rn = inv_norm(row_total(ss), sm);
      if (stager()) {
#pragma unroll
        for (int e = 0; e < EPT; e += 4)
          Ops::put4(Ks, srow(), sseg() + e, f4{x[e] * rn, x[e + 1] * rn, x[e + 2] * rn, x[e + 3] * rn});
        if (key_elements) {
#pragma unroll
          for (int e = 0; e < EPT; e += 4)
            *reinterpret_cast<f4*>(&Kf[kF32Keys ? srow() * LDF + sseg() + e : 0]) = f4{x[e] * rn, x[e + 1] * rn, x[e + 2] * rn, x[e + 3] * rn};
        }
        if (sseg() == 0) nks[srow()] = sm * rn;  // max(||k||, eps)
      }
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (UK == kUSeparate) {
        unpack(upre, x, ragged, live, false);
        float uu = 0.0f;
#pragma unroll
        for (int e = 0; e < EPT; ++e) uu = fmaf(x[e], x[e], uu);
        float um;
        const float su = a.u_scale * inv_norm(row_total(uu), um);
        if (stager()) {
          const KeyScale us = key_scale(su);
          const float f = UT == 1 ? us.pow2 : su;
          if (UT == 1 && sseg() == 0) urest[srow()] = us.rest;
#pragma unroll
          for (int e = 0; e < EPT; e += 4)
            UOps::put4(Usb, srow(), sseg() + e, f4{x[e] * f, x[e + 1] * f, x[e + 2] * f, x[e + 3] * f});
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      unpack(qpre, x, ragged, live, fmap);
      if (stager()) {
#pragma unroll
        for (int e = 0; e < EPT; e += 4) Ops::put4(Qs, srow(), sseg() + e, f4{x[e], x[e + 1], x[e + 2], x[e + 3]});
      }
    };
    const size_t slab_v = static_cast<size_t>(head) * static_cast<size_t>(T) * DV;
    const IO* vh = static_cast<const IO*>(a.v) + slab_v;
    IO* oh = static_cast<IO*>(a.o) + slab_v;
    auto vcol = [&]() { return row0 + c; };
    IO vpre[NJV][4];   // V[t0 + 4g + r][row0 + 16jn + c]
    auto load_v = [&](int t0) __attribute__((always_inline)) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int t = t0 + 4 * g + r;
        const unsigned voff = static_cast<unsigned>((t < T ? t : T - 1) * DV + vcol());
#pragma unroll
        for (int jn = 0; jn < NJV; ++jn) vpre[jn][r] = vh[voff + 16 * jn];
      }
    };
    f4 ft[NJV], ot[NJV];
    // K^ S^T and Q S^T, steps kb0 .. kb1 - 1 of the contraction
    auto s_pass = [&](int kb0, int kb1) __attribute__((always_inline)) {
#pragma unroll
      for (int kb = kb0; kb < kb1; ++kb) {
#pragma unroll
        for (int jn = 0; jn < NJV; ++jn) {
          const auto sb = split_tiles(St[2 * kb][jn], St[2 * kb + 1][jn], identity());
          ft[jn] = Ops::sweep(Ops::operand(Ks, kb, c, g), sb, ft[jn]);
          __builtin_amdgcn_sched_barrier(0);
          ot[jn] = Ops::sweep(Ops::operand(Qs, kb, c, g), sb, ot[jn]);
          __builtin_amdgcn_sched_barrier(0);   // one split at a time in registers
        }
      }
    };
    // -E^T = Z (K^ S^T - V^T), O^T = Q S^T + (-NQ^T)(-E^T), store o, S^T += Alpha diag(c) E^T
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
      if (norm_out) {
        const f4 rd = lds4(&rdens[4 * g]);
#pragma unroll
        for (int jn = 0; jn < NJV; ++jn) ot[jn] *= rd;
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int t = t0 + 4 * g + r;
        if (t < T) {
          const unsigned ooff = static_cast<unsigned>(t * DV + vcol());
#pragma unroll
          for (int jn = 0; jn + 1 < NJV; jn += 2)
            io_store2(oh + ooff + 16 * jn, oh + ooff + 16 * jn + 16, ot[jn][r], ot[jn + 1][r]);
          if (NJV % 2 == 1) io_store(oh + ooff + 16 * (NJV - 1), ot[NJV - 1][r]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      decltype(Ops::tokens_b(f4{})) ce[NJV];
#pragma unroll
      for (int jn = 0; jn < NJV; ++jn) ce[jn] = Ops::tokens_b(ft[jn] * cg);
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const auto aa = Ops::w_load(Ahm, Al, 16 * b + c, c, g);
#pragma unroll
        for (int jn = 0; jn < NJV; ++jn) St[b][jn] = Ops::update(aa, ce[jn], St[b][jn]);
        if (b % 2 == 1) __builtin_amdgcn_sched_barrier(0);
      }
    };

    if (nblk > 0) {
      load_kqu(0);
      stage(0, 0);
      if (nblk > 1) load_kqu(C);
    }
    __syncthreads();  // (0) block 0 staged
    constexpr int kHalf = (NKB + 1) / 2;
    for (int blk = 0; blk < nblk; ++blk) {
      fresh();
      // opaque: the compiler would peel the first block and keep twice the values over the loop (some 60 more registers spilled; 51 are)
      int done = blk;
      asm volatile("" : "+s"(done));
      if (done > 0) s_update(blk - 1);
      __syncthreads();  // (1)
#pragma unroll
      for (int jn = 0; jn < NJV; ++jn) ft[jn] = ot[jn] = f4{0, 0, 0, 0};
      s_pass(0, kHalf);
      __syncthreads();  // (2)
      s_pass(kHalf, NKB);
      __syncthreads();  // (3) K^, Q, U no longer read
      load_v(C * blk);
      if (blk + 1 < nblk) stage(C * (blk + 1), (blk + 1) & 1);
      if (blk + 2 < nblk) load_kqu(C * (blk + 2));
      __syncthreads();  // (0) Z, NQ, c visible; next block staged
    }
    if (nblk > 0) s_update(nblk - 1);
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

template <int D, int DV, int NWA, int NWS, int WPE, typename IO>
hipError_t launch_as(const ForwardArgs& a, hipStream_t stream) {
  ForwardArgs args = a;
  void* params[] = {&args};
  // three-term directions of 64 take the LDS of a fourth workgroup
  constexpr int WPU = D == 64 && NWA == 2 && sizeof(IO) == 4 ? 3 : WPE;
  const void* fn =
      a.u != nullptr         ? reinterpret_cast<const void*>(&chunk_general_pipe_kernel<D, DV, NWA, NWS, IO, kUSeparate, WPU>)
      : a.refresh_period > 0 ? reinterpret_cast<const void*>(&chunk_general_pipe_kernel<D, DV, NWA, NWS, IO, kUKeyRefresh, WPE>)
                             : reinterpret_cast<const void*>(&chunk_general_pipe_kernel<D, DV, NWA, NWS, IO, kUKey, WPE>);
  return hipLaunchKernel(fn, dim3(a.n_heads), dim3(64 * (NWA + NWS)), params, 0, stream);
}
template <int D, int DV, int NWA, int NWS, int WPE>
hipError_t launch(const ForwardArgs& a, int io_dtype, hipStream_t stream) {
  return io_dtype == 1 ? launch_as<D, DV, NWA, NWS, WPE, uint16_t>(a, stream) : launch_as<D, DV, NWA, NWS, WPE, float>(a, stream);
}

}  // namespace

// Waves of 16 columns, every pair of head sizes from d_k = 32 on.
hipError_t launch_chunk_general_pipe_narrow(const ForwardArgs& a, int d_k, int d_v, int io_dtype, hipStream_t stream) {
  switch (d_k * 1000 + d_v) {
    case 32016: return launch<32, 16, 2, 1, 3>(a, io_dtype, stream);
    case 32032: return launch<32, 32, 2, 2, 4>(a, io_dtype, stream);
    case 32064: return launch<32, 64, 2, 4, 4>(a, io_dtype, stream);
    case 32096: return launch<32, 96, 2, 6, 4>(a, io_dtype, stream);
    case 32128: return launch<32, 128, 2, 8, 4>(a, io_dtype, stream);
    case 64016: return launch<64, 16, 4, 1, 4>(a, io_dtype, stream);
    case 64032: return launch<64, 32, 4, 2, 4>(a, io_dtype, stream);
    case 64064: return launch<64, 64, 4, 4, 4>(a, io_dtype, stream);
    case 64096: return launch<64, 96, 4, 6, 4>(a, io_dtype, stream);
    case 64128: return launch<64, 128, 4, 8, 4>(a, io_dtype, stream);
    case 96016: return launch<96, 16, 6, 1, 2>(a, io_dtype, stream);
    case 96032: return launch<96, 32, 6, 2, 2>(a, io_dtype, stream);
    case 96064: return launch<96, 64, 6, 4, 3>(a, io_dtype, stream);
    case 96096: return launch<96, 96, 6, 6, 3>(a, io_dtype, stream);
    case 96128: return launch<96, 128, 6, 8, 3>(a, io_dtype, stream);
    case 128016: return launch<128, 16, 8, 1, 3>(a, io_dtype, stream);
    case 128032: return launch<128, 32, 8, 2, 3>(a, io_dtype, stream);
    case 128064: return launch<128, 64, 8, 4, 3>(a, io_dtype, stream);
    case 128096: return launch<128, 96, 8, 6, 4>(a, io_dtype, stream);
    case 128128: return launch<128, 128, 8, 8, 4>(a, io_dtype, stream);
    default: return hipErrorInvalidValue;
  }
}

// Waves of 32 columns; heads of 128 with a given u in bf16 only.
hipError_t launch_chunk_general_pipe_wide(const ForwardArgs& a, int d_k, int d_v, int io_dtype, hipStream_t stream) {
  switch (d_k * 1000 + d_v) {
    case 64064: return launch<64, 64, 2, 2, 4>(a, io_dtype, stream);
    case 64096: return launch<64, 96, 2, 3, 4>(a, io_dtype, stream);
    case 64128: return launch<64, 128, 2, 4, 4>(a, io_dtype, stream);
    case 128128: {
      ForwardArgs args = a;
      void* params[] = {&args};
      return hipLaunchKernel(reinterpret_cast<const void*>(&chunk_general_pipe_kernel<128, 128, 4, 4, uint16_t, kUSeparate, 4>),
                             dim3(a.n_heads), dim3(512), params, 0, stream);
    }
    default: return hipErrorInvalidValue;
  }
}

}  // namespace vla
