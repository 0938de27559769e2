// Block ("chunked") form of the VLA recurrence on MFMA, 16 tokens per block.
//
// Same recurrence as paper Section 3.3 (eq. (sm), eq. (s-update)) and the read-out numerator of
// eq. (output); within a block of C = 16 tokens the token-by-token matrix-vector work is regrouped
// into dense products, which is exact algebra (results differ only in float32 rounding order).
//
// With A0, S0 the state entering the block, K^ (C x d) the normalised keys, Q, V the queries and
// values of the block (rows = tokens), and u = k^:
//
//   Y^T = K^ A0                                   (C x d)      z before the in-block corrections
//   G   = Y^T K^^T ,  GQ = Y^T Q^T                (C x C)      Gram matrices in the A0 metric
//   I + G = L L^T                                 (Cholesky)   L_tt = sqrt(delta_t), L_ts = w_s . k^_t
//   W^T = L^{-1} Y^T                              (C x d)      w_t = z_t / sqrt(delta_t)
//   A1  = A0 - W W^T                                           C Sherman-Morrison steps at once
//   alpha^_t = c_t w_t ,  c_t = (1/L_tt) / max(||w_t|| / L_tt, eps)       (A_t k^_t = w_t / L_tt)
//   F^T = V - K^ S0^T                             (C x d_v)    residuals against the entering state
//   E^T = Z F^T ,  Z = (I + strict_lower(L) diag(c))^{-1}      residuals e_t of the recurrence
//   O^T = Q S0^T + NQ^T E^T ,  NQ[s][t] = c_s (L^{-1} GQ)[s][t] for s <= t, else 0
//   S1^T = S0^T + W diag(c) E^T
//
// A zero key gives an all-zero row in Y, W and E, so padding the last block with zero tokens is exact.
//
// Work split: NW waves per (batch, head); wave w owns columns [SL*w, SL*w+SL) of A and the same rows of
// S, as 16x16 float32 accumulator tiles that stay in VGPRs for the whole sequence (A is symmetric, so an
// accumulator tile of A can be fed straight back as the B operand).  The C x C factorisations run on
// one wave (rotating with the block index) four columns at a time (cholesky16).
//
// What bounds it: instruction issue -- the matrix unit, the vector instructions that split the state, and the two
// serial sections, of which one head hides the other's.  The five sweeps over A and S are FP32 products formed
// from bf16 terms (vla_mfma_util.h): the state is split into three terms as it is read (11 instructions per two
// elements, once per block: S for both of its products), bf16 keys and queries are one term each, float32 ones
// three; W and E are split once per block.  On FP32 matrix instructions the matrix unit alone took 78 % of the time
// (2048 heads of 128, 512 tokens, float32 1.43 ms now).  Most calls run on the kernel of vla_chunk_pipe.hip; what is left
// here are head sizes of 16, counts that would take that one another round of workgroups, and three-term operands of
// large counts (see pipe_narrow and pipe_wide below).
#include "vla_mfma_util.h"

namespace vla {
namespace {

// Wave priority: LEVELS = 2: the full scheme (level FULL); 1: only the serial chains are raised (level CHAIN at
// their start and end, nothing where CHAIN < 0); 0: every wave stays at the default priority.
template <int LEVELS, int FULL, int CHAIN>
__device__ __forceinline__ void prio() {
  if constexpr (LEVELS == 2) __builtin_amdgcn_s_setprio(FULL);
  else if constexpr (LEVELS == 1 && CHAIN >= 0) __builtin_amdgcn_s_setprio(CHAIN);
}

// SPLIT: products on split bf16 terms, else on the FP32 matrix instruction (d = 16, and where that saves a round of
// workgroups: fp32_products below).
// FMAP: q and k are replaced by ELU(x) + 1 while they are staged (the feature map of Section 3.3).
// DV: head size of v and o (rows of S); the wave that owns columns [SL w, SL w + SL) of A owns rows
// [SLV w, SLV w + SLV) of S.
// LOOP: the workgroups of a launch go through the heads in turn (takes_turns below), else one workgroup per head.
template <int D, int DV, int NW, typename IO, bool FMAP, bool SPLIT, bool LOOP>
__global__ void __launch_bounds__(64 * NW, 2) chunk_kernel(ForwardArgs a) {
  // Measured at 2048 heads, T = 8192: the full scheme gains 5 % with four waves (d = 128), 1 % with three (d = 96),
  // 1-5 % with one (d = 16, 32); two-wave workgroups (d = 64), four of which share a compute unit, lose up to
  // 20 % with any of it (1536 heads: 7.0 -> 8.5 ms) and stay at the default priority.
  constexpr int kLevels = NW == 2 ? 0 : 2;
  constexpr int SL = D / NW;       // columns of A owned by one wave
  constexpr int NJ = SL / 16;      // 16-wide tiles in a slab of A
  // The DV / 16 row tiles of S are shared out over the waves: DV / (16 NW) consecutive tiles each where that
  // divides (kEven), else tile t goes to wave t % NW, and a wave with fewer tiles than the others (or none)
  // runs its spare slots on a copy of the last tile and stores nothing from them.
  constexpr int TV = DV / 16;
  constexpr bool kEven = TV % NW == 0;
  constexpr int NJV = kEven ? TV / NW : (TV + NW - 1) / NW;   // tile slots per wave
  static_assert(DV % 16 == 0 && NJV >= 1, "whole tiles of S");
  constexpr int NB = D / 16;       // 16-row blocks over the whole head dimension
  // operand terms of k and q: bf16 numbers are exact in one, float32 ones (and mapped ones) take three
  constexpr int KT = (sizeof(IO) == 2 && !FMAP) || !SPLIT ? 1 : 3;
  using Ops = BlockOps<SPLIT, KT, D>;
  constexpr int STEP = Ops::STEP;
  constexpr int NKB = NB / STEP;      // steps of a contraction over the head dimension
  static_assert(NB % STEP == 0, "whole steps");
  constexpr int LDY = SL + 4;         // row stride of a wave's slab of Y^T
  constexpr int NT = 64 * NW;
  // Staging: a token row is split over TPR threads of EPT elements each.  For the power-of-two head sizes every
  // thread stages; at d = 96 a row takes 6 threads of 16 elements in a group of 8 (two lanes of each group and
  // the third wave stage nothing), so that a row never straddles a wave and sums with a power-of-two shuffle.
  constexpr int TPR0 = NT / C;                   // thread slots per row when every thread stages
  constexpr bool PADDED = (TPR0 & (TPR0 - 1)) != 0;
  constexpr int EPT = PADDED ? 16 : C * D / NT;  // staged elements per thread per tensor
  constexpr int TPR = PADDED ? 8 : D / EPT;      // thread slots per token row
  static_assert(EPT % 4 == 0 && TPR <= 32 && (TPR & (TPR - 1)) == 0 && C * TPR <= NT && D % EPT == 0 &&
                D / EPT <= TPR, "staging layout");

  __shared__ __align__(16) uint16_t Ksb[2][Ops::SIZE];     // k [t][slot], terms, double-buffered over blocks
  __shared__ __align__(16) uint16_t Qsb[2][Ops::SIZE];     // q
  __shared__ __align__(16) u4 Whm[D * 4];                  // W [j][t], terms h and m
  __shared__ __align__(16) u2 Wl[D * 4];                   //           term l
  __shared__ __align__(16) float Gp[NW][2][C * LT];   // per-wave partial Gram matrices G, GQ  [s][t]; first the
                                                      // wave's slab of Y^T [t][j], which no other wave reads
  __shared__ __align__(16) float Lis[C * LT];         // L^{-1} [t][s]
  __shared__ __align__(16) float Lrs[C * LT];         // L [t][s] (rows), for the wave that forms Z
  __shared__ __align__(16) float Zs[C * LT];          // Z   [t][s]
  __shared__ __align__(16) float NQs[C * LT];         // -NQ^T [t][s]
  __shared__ __align__(16) float wn2p[NW][C];         // per-wave partial ||w_t||^2
  __shared__ __align__(16) float cvec[C];             // -c_t
  __shared__ __align__(16) float rns[2][C];           // 1 / max(||k_t||, eps) over its power of two (key_scale)
  static_assert(C * LDY <= 2 * C * LT, "a slab of Y^T fits the wave's Gram tiles");

  // A head begins with LDS that nothing reads any more: after barrier (5) of its last block a wave reads W, Z, NQ and c, and
  // those are written again only behind the barriers of the next head's first block.
  int head = blockIdx.x;
  do {
  int tid = threadIdx.x;
  if constexpr (LOOP) asm volatile("" : "+v"(tid));   // what is derived from it is formed per head, not kept in registers over all
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave index, known to be uniform
  const int lane = tid & 63;
  const int c = lane & 15;
  const int g = lane >> 4;
  const int T = a.T;
  const float eps = a.eps;
  const int col0 = SL * w;    // first column of this wave's slab of A
  const int row0 = 16 * NJV * w;   // kEven: first row of this wave's slab of S
  // first S row of this wave's tile slot jn, and whether the slot holds a tile of its own
  auto s_row = [&](int jn) -> int {
    if constexpr (kEven) {
      return row0 + 16 * jn;
    } else {
      const int t = w + NW * jn;
      return 16 * (t < TV ? t : TV - 1);
    }
  };
  auto owns = [&](int jn) -> bool { return kEven || w + NW * jn < TV; };
  const bool has_rows = TV >= NW || w < TV;   // uniform in a wave: one without a tile leaves S to the others

  // ---- resident state: accumulator tiles
  // At[b][jn][r] = A[16b + 4g + r][col0 + 16jn + c]
  // St[b][jn][r] = S[row0 + 16jn + c][16b + 4g + r]      (i.e. tiles of S^T)
  f4 At[NB][NJ], St[NB][NJV];
  {
    const float* A0 = a.A0 ? a.A0 + static_cast<size_t>(head) * D * D : nullptr;
    const float* S0 = a.S0 ? a.S0 + static_cast<size_t>(head) * DV * D : nullptr;
    const float diag = 1.0f / a.lambda0;
    const int arc = (4 * g) * D + col0 + c;  // A[4g][col0 + c]
    const int src = c * D + 4 * g;  // S[c][4g]
#pragma unroll
    for (int b = 0; b < NB; ++b) {
#pragma unroll
      for (int jn = 0; jn < NJ; ++jn) {
        if (A0) {
#pragma unroll
          for (int r = 0; r < 4; ++r) At[b][jn][r] = A0[arc + (16 * b + r) * D + 16 * jn];
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            At[b][jn][r] = (16 * b + 4 * g + r == col0 + 16 * jn + c) ? diag : 0.0f;
        }
      }
#pragma unroll
      for (int jn = 0; jn < NJV; ++jn) {
        if (S0) {
          const float4 x = *reinterpret_cast<const float4*>(S0 + src + s_row(jn) * D + 16 * b);
          St[b][jn] = f4{x.x, x.y, x.z, x.w};
        } else {
          St[b][jn] = f4{0, 0, 0, 0};
        }
      }
    }
  }

  const size_t slab = static_cast<size_t>(head) * static_cast<size_t>(T) * D;
  const size_t slab_v = static_cast<size_t>(head) * static_cast<size_t>(T) * DV;
  const IO* qh = static_cast<const IO*>(a.q) + slab;
  const IO* kh = static_cast<const IO*>(a.k) + slab;
  const IO* vh = static_cast<const IO*>(a.v) + slab_v;
  IO* oh = static_cast<IO*>(a.o) + slab_v;

  // staging role of this thread: token row and column segment
  const int srow = tid / TPR;
  const int sseg = (tid % TPR) * EPT;
  const bool stager = !PADDED || (tid < C * TPR && sseg < D);    // this thread holds a row segment
  const bool stage_wave = !PADDED || tid < C * TPR;              // uniform per wave
  const int vcol = s_row(0) + c;  // first element of a v / o row this lane touches in accumulator layout

  RawRow<IO, EPT> kpre, qpre;
  IO vpre[NJV][4];  // V^T in accumulator layout: V[t0 + 4g + r][row0 + 16jn + c]

  // Loads never branch or wait: rows past the end are read from the last valid row and replaced by
  // zeros when the registers are consumed (later).  Offsets are 32-bit from the per-head base pointers.
  auto load_kq = [&](int t0) {
    if (stager) {
      const int tr = t0 + srow;
      const unsigned koff = static_cast<unsigned>((tr < T ? tr : T - 1) * D + sseg);
      kpre.load(kh + koff);
      qpre.load(qh + koff);
    }
  };
  auto load_v = [&](int t0) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int t = t0 + 4 * g + r;
      const unsigned voff = static_cast<unsigned>((t < T ? t : T - 1) * DV + vcol);
#pragma unroll
      for (int jn = 0; jn < NJV; ++jn) vpre[jn][r] = vh[voff + (s_row(jn) - s_row(0))];
    }
  };
  // put this thread's share of the keys and queries of the block starting at t0, and the key norms, into LDS half `buf`
  auto stage = [&](int t0, int buf) __attribute__((always_inline)) {
    if (!stage_wave) return;
    float kx[EPT];
    const bool ragged = t0 + C > T;   // uniform: only the last block can hold rows past the end
    const bool live = t0 + srow < T && stager;  // rows past the end of the sequence become zero tokens
    if (stager) {
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
    // the TPR = 16 threads of a token row are one DPP row; 1 / max(||k||, eps) = rsqrt(max(||k||^2, eps^2)),
    // hardware reciprocal square root refined by one Newton step
    if constexpr (TPR == 16) {
      ss = row_sum16(ss);
    } else {
#pragma unroll
      for (int off = TPR / 2; off >= 1; off >>= 1) ss += __shfl_xor(ss, off);
    }
    const float sm = fmaxf(ss, eps * eps);
    float rn = __builtin_amdgcn_rsqf(sm);
    rn = rn * fmaf(-0.5f * sm * rn, rn, 1.5f);
    if (!stager) return;
    // FP32 products take the normalised keys themselves
    const KeyScale ks = SPLIT ? key_scale(rn) : KeyScale{rn, 1.0f};
#pragma unroll
    for (int e = 0; e < EPT; ++e) kx[e] *= ks.pow2;
    if (sseg == 0) rns[buf][srow] = ks.rest;
#pragma unroll
    for (int e = 0; e < EPT; e += 4) Ops::put4(Ksb[buf], srow, sseg + e, f4{kx[e], kx[e + 1], kx[e + 2], kx[e + 3]});
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
    for (int e = 0; e < EPT; e += 4) Ops::put4(Qsb[buf], srow, sseg + e, f4{qx[e], qx[e + 1], qx[e + 2], qx[e + 3]});
  };
  if (T > 0) {
    load_kq(0);
    load_v(0);
    stage(0, 0);
    if (C < T) load_kq(C);
  }
  __syncthreads();  // block 0 staged

  prio<kLevels, 1, -1>();
  int blk = 0;
  for (int t0 = 0; t0 < T; t0 += C, ++blk) {
    const uint16_t* Ks = Ksb[blk & 1];
    const uint16_t* Qs = Qsb[blk & 1];
    // staging of the next block (this thread's share): done where this wave is not on the critical path
    auto stage_next = [&]() {
      if (t0 + C < T) stage(t0 + C, (blk + 1) & 1);
    };
    auto fetch_next = [&]() {
      if (t0 + 2 * C < T) load_kq(t0 + 2 * C);
    };
    // ================= Y^T = K^ A0 (this wave's columns)
    f4 yt[NJ];
    {
#pragma unroll
      for (int jn = 0; jn < NJ; ++jn) yt[jn] = f4{0, 0, 0, 0};
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb) {
        const Terms<KT> ka = Ops::operand(Ks, kb, c, g);
#pragma unroll
        for (int jn = 0; jn < NJ; ++jn)
          yt[jn] = Ops::sweep(ka, Ops::tiles(At[STEP * kb][jn], At[STEP * kb + STEP - 1][jn]), yt[jn]);
        if (KT > 1) __builtin_amdgcn_sched_barrier(0);
      }
      const f4 rn4 = lds4(&rns[blk & 1][4 * g]);
#pragma unroll
      for (int jn = 0; jn < NJ; ++jn) yt[jn] *= rn4;
    }
    // ================= partial Gram matrices over this wave's columns; Y^T turns through LDS
    {
      float* Yw = Gp[w][0];
#pragma unroll
      for (int jn = 0; jn < NJ; ++jn)
#pragma unroll
        for (int r = 0; r < 4; ++r) Yw[(4 * g + r) * LDY + 16 * jn + c] = yt[jn][r];
      // same-wave write -> read: LDS operations of one wave are ordered
      // G[s][t], GQ[s][t] come out with t on the rows of the accumulator
      f4 gg = f4{0, 0, 0, 0}, gq = f4{0, 0, 0, 0};
      if constexpr (SPLIT) {
        // slots 0-3 hold the first 16 of 32 columns, slots 4-7 the second ones: a slab of 16 columns fills one half
        const f4 zero{0, 0, 0, 0};
        const f4 y0 = lds4(&Yw[c * LDY + 4 * g]);
        const f4 y1 = NJ > 1 ? lds4(&Yw[c * LDY + (NJ > 1 ? 16 : 0) + 4 * g]) : (w & 1) ? y0 : zero;
        const auto ya = Ops::tiles(NJ == 1 && (w & 1) ? zero : y0, y1);
        gg = Ops::sweep(Ops::operand(Ks, col0 / 32, c, g), ya, gg);
        gq = Ops::sweep(Ops::operand(Qs, col0 / 32, c, g), ya, gq);
      } else {
        f4 y[NJ];   // all of the slab before the Gram tiles take its place
#pragma unroll
        for (int jn = 0; jn < NJ; ++jn) y[jn] = lds4(&Yw[c * LDY + 16 * jn + 4 * g]);
#pragma unroll
        for (int jn = 0; jn < NJ; ++jn) {
          gg = Ops::sweep(Ops::operand(Ks, col0 / 16 + jn, c, g), y[jn], gg);
          gq = Ops::sweep(Ops::operand(Qs, col0 / 16 + jn, c, g), y[jn], gq);
        }
      }
      const f4 rn4 = lds4(&rns[blk & 1][4 * g]);
#pragma unroll
      for (int r = 0; r < 4; ++r) Gp[w][0][c * LT + 4 * g + r] = gg[r] * rn4[r];
#pragma unroll
      for (int r = 0; r < 4; ++r) Gp[w][1][c * LT + 4 * g + r] = gq[r];
    }
    __syncthreads();  // (2) partial Grams visible

    // ================= C x C factorisation, phase 1 (one wave): Cholesky of I + G and L^{-1}
    const int sw = (blk + head) % NW;   // wave factorising I + G this block (rotates over waves/SIMDs)
    const int sw2 = (sw + NW / 2) % NW;  // a different wave forms c, Z, NQ
    // ================= -F^T = K^ S0^T - V^T and R^T = Q S0^T: one pass over S, whose split serves both; needed only
    // after barrier (5), so it fills the serial windows
    f4 ft[NJV], ot[NJV];
    auto s_pass = [&]() {
      if (!has_rows) return;
#pragma unroll
      for (int jn = 0; jn < NJV; ++jn) ft[jn] = ot[jn] = f4{0, 0, 0, 0};
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb) {
#pragma unroll
        for (int jn = 0; jn < NJV; ++jn) {
          const auto sb = Ops::tiles(St[STEP * kb][jn], St[STEP * kb + STEP - 1][jn]);
          ft[jn] = Ops::sweep(Ops::operand(Ks, kb, c, g), sb, ft[jn]);
          if constexpr (KT > 1) __builtin_amdgcn_sched_barrier(0);
          ot[jn] = Ops::sweep(Ops::operand(Qs, kb, c, g), sb, ot[jn]);
          if constexpr (SPLIT) __builtin_amdgcn_sched_barrier(0);   // one split at a time in registers
        }
      }
      const f4 rn4 = lds4(&rns[blk & 1][4 * g]);
      if (t0 + C > T) {  // uniform: rows past the end of the sequence are zero tokens
#pragma unroll
        for (int jn = 0; jn < NJV; ++jn)
#pragma unroll
          for (int r = 0; r < 4; ++r) vpre[jn][r] = (t0 + 4 * g + r < T) ? vpre[jn][r] : IO(0);
      }
#pragma unroll
      for (int jn = 0; jn < NJV; ++jn)
#pragma unroll
        for (int r = 0; r < 4; ++r) ft[jn][r] = fmaf(ft[jn][r], rn4[r], neg_widen(vpre[jn][r]));
      if (t0 + C < T) load_v(t0 + C);
    };
    if (w != sw) {  // the other waves work on S while wave sw factorises
      prio<kLevels, 0, -1>();
      stage_next();   // first, so that no staged row is held in registers over the pass
      s_pass();
      fetch_next();
      prio<kLevels, 1, -1>();
    }
    if (w == sw) {
      prio<kLevels, 3, 3>();   // the dependent chain is what the other waves wait for: issue it first
      f4 gram = lds4(&Gp[0][0][c * LT + 4 * g]);
#pragma unroll
      for (int ww = 1; ww < NW; ++ww) gram += lds4(&Gp[ww][0][c * LT + 4 * g]);
      const Lane at = fresh_lane(c, g);
      cholesky16(gram, Lrs, Lis, at.c, at.g);
      prio<kLevels, 1, 0>();
    }
    __syncthreads();  // (3) L^{-1} visible

    // ================= W^T = L^{-1} Y^T, partial ||w_t||^2, W to LDS
    prio<kLevels, 2, -1>();
    const f4 la = lds4(&Lis[c * LT + 4 * g]);
    {
      f4 n2 = f4{0, 0, 0, 0};
#pragma unroll
      for (int jn = 0; jn < NJ; ++jn) {
        f4 acc = f4{0, 0, 0, 0};
#pragma unroll
        for (int r = 0; r < 4; ++r) acc = mfma16(la[r], yt[jn][r], acc);
        n2 += acc * acc;
        Ops::w_store(Whm, Wl, col0 + 16 * jn + c, c, g, acc);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) n2[r] = row_sum16(n2[r]);
      if (c == 0) *reinterpret_cast<f4*>(&wn2p[w][4 * g]) = n2;
    }
    prio<kLevels, 1, -1>();
    __syncthreads();  // (4) W and the norm partials visible

    // ================= phase 2 (wave sw2): c_t, Z, NQ -- the other waves update A meanwhile
    auto update_A = [&]() {
      Ops::template downdate<NB, NJ>(Whm, Wl, col0 + c, c, g, blk & 1, [&](int b, int jn) -> f4& { return At[b][jn]; });
    };
    if (w != sw2) {
      prio<kLevels, 0, -1>();
      update_A();
      prio<kLevels, 1, -1>();
    }
    if (w == sw) {  // (sw != sw2 when NW > 1)
      stage_next();   // first, so that no staged row is held in registers over the pass
      s_pass();
      fetch_next();
    }
    if (w == sw2) {
      prio<kLevels, 3, 3>();
      const float dl = Lrs[c * LT + c];  // L_cc
      float wn2 = 0.0f;
#pragma unroll
      for (int ww = 0; ww < NW; ++ww) wn2 += wn2p[ww][c];
      // hardware reciprocal and square root (1 ulp): c_t only scales the write direction
      const float rdl = __builtin_amdgcn_rcpf(dl);
      const float an = __builtin_amdgcn_sqrtf(wn2) * rdl;                // ||A_t k^_t|| = ||w_t|| / L_tt
      const float cs = rdl * __builtin_amdgcn_rcpf(fmaxf(an, eps));      // alpha^_t = c_t w_t
      if (g == 0) cvec[c] = -cs;  // the residual tiles carry -E, see below
      // Z = (I + strict_lower(L) diag(c))^{-1}
      const Lane at = fresh_lane(c, g);
      lower_inverse16(Lrs, cs, at.c, at.g, [&](int t, int s, float z) { Zs[t * LT + s] = z; });
      // H = L^{-1} GQ (one MFMA tile), NQ[s][t] = c_s H[s][t] for s <= t
      f4 hq = f4{0, 0, 0, 0};
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float gqv = 0.0f;
#pragma unroll
        for (int ww = 0; ww < NW; ++ww) gqv += Gp[ww][1][(4 * g + r) * LT + c];
        hq = mfma16(la[r], gqv, hq);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int s = 4 * g + r;
        const float csr = __shfl(cs, s);
        NQs[c * LT + s] = (s <= c) ? -(csr * hq[r]) : 0.0f;
      }
      prio<kLevels, 1, 0>();
    }
    __syncthreads();  // (5) Z, NQ, c visible

    if (has_rows) {
    // ================= -E^T = Z (-F^T), R^T = Q S0^T, O^T = R^T + (-NQ^T)(-E^T), store o;
    // ce = (-c) (-E^T) = diag(c) E^T
    decltype(Ops::tokens_b(f4{})) ce[NJV];
    {
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
      for (int jn = 0; jn < NJV; ++jn) {
#pragma unroll
        for (int r = 0; r < 4; ++r) ot[jn] = mfma16(nqa[r], ft[jn][r], ot[jn]);
        ce[jn] = Ops::tokens_b(ft[jn] * cg);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int t = t0 + 4 * g + r;
        if (t < T) {
          const unsigned ooff = static_cast<unsigned>(t * DV + vcol);
          if constexpr (kEven) {
#pragma unroll
            for (int jn = 0; jn + 1 < NJV; jn += 2)
              io_store2(oh + ooff + 16 * jn, oh + ooff + 16 * jn + 16, ot[jn][r], ot[jn + 1][r]);
            if (NJV % 2 == 1) io_store(oh + ooff + 16 * (NJV - 1), ot[NJV - 1][r]);
          } else {
#pragma unroll
            for (int jn = 0; jn < NJV; ++jn)
              if (owns(jn)) io_store(oh + ooff + (s_row(jn) - s_row(0)), ot[jn][r]);
          }
        }
      }
    }
    // ================= S^T += W diag(c) E^T  (and A -= W W^T on the wave that formed Z)
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const auto wa = Ops::w_load(Whm, Wl, 16 * b + c, c, g);
#pragma unroll
      for (int jn = 0; jn < NJV; ++jn) St[b][jn] = Ops::update(wa, ce[jn], St[b][jn]);
      if (b % 2 == 1) __builtin_amdgcn_sched_barrier(0);
    }
    }
    if (w == sw2) update_A();
  }

  // ---- final state
  {
    float* AT = a.A_T ? a.A_T + static_cast<size_t>(head) * D * D : nullptr;
    float* ST = a.S_T ? a.S_T + static_cast<size_t>(head) * DV * D : nullptr;
    int g2 = g, c2 = c;
    asm volatile("" : "+v"(g2), "+v"(c2));  // recompute the addresses here instead of carrying them over the loop
    const int arc = (4 * g2) * D + col0 + c2;
    const int src = c2 * D + 4 * g2;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      if (AT) {
#pragma unroll
        for (int jn = 0; jn < NJ; ++jn)
#pragma unroll
          for (int r = 0; r < 4; ++r) AT[arc + (16 * b + r) * D + 16 * jn] = At[b][jn][r];
      }
      if (ST) {
#pragma unroll
        for (int jn = 0; jn < NJV; ++jn)
          if (owns(jn))
            *reinterpret_cast<float4*>(ST + src + s_row(jn) * D + 16 * b) =
                make_float4(St[b][jn][0], St[b][jn][1], St[b][jn][2], St[b][jn][3]);
      }
    }
  }
  head += gridDim.x;
  } while (LOOP && head < a.n_heads);
}

// Which calls go through the heads in turn (LOOP), as many workgroups as the compute units hold together?  A workgroup that
// the hardware starts in another's place comes where room is, and two kinds of last round suffer for it; a workgroup that
// goes on with another head stays where it was.  T = 512, one workgroup per head / in turn, us:
//   A round of workgroups of two waves that is all but full: the free places of some compute units lie on one SIMD, and the
//   last heads wait.  64 x 96, one term: 2000 heads 480 / 480, 2040 538 / 480, 2048 549 / 480, 3000 712 / 717, 3072 772 / 724;
//   64 x 128: 2000 545 / 548, 2048 619 / 548, 3072 897 / 822;  32 x 128, one term 2048 388 / 371, three 517 / 445.  32 x 96 of
//   float32 numbers lets three waves on a SIMD, so that this begins where two rounds of four workgroups would do: 1700 heads 355 / 352,
//   1800 391 / 365, 2048 424 / 370, but 1200 (five together, one round) 240 / 305, 2500 463 / 517.
//   A second round of between a quarter and half of the places: two of its workgroups go where two end together, and none to the
//   next.  64 x 96, one term: 1280 heads 394 / 384, 1536 471 / 447; 32 x 128, one term 1500 355 / 341, three 410 / 392 (one term,
//   1400 heads, T = 1024 648 / 672); 128 x 96, one term: 640 heads 532 / 507, 768 555 / 508, 900 564 / 563;  16 x 128, 256 tokens: 2500
//   heads 232 / 232, 3072 280 / 242, 3500 292 / 293.
// One block does not pay for it: 64 x 128, 3072 heads, 16 tokens 43.8 / 45.8.
enum LastRound { kAny, kFullOrHalf, kThreeQuarters, kHalf };
constexpr LastRound loop_rule(int d, int d_v, int nw, bool f32, bool one_term) {
  if (d == 16) return d_v == 128 ? kHalf : kAny;
  if (nw == 2 && d == 32) return d_v == 128 ? kFullOrHalf : d_v == 96 && f32 ? kThreeQuarters : kAny;
  if (nw == 2 && d == 64) return one_term && d_v > d ? kFullOrHalf : kAny;
  return d == 128 && d_v == 96 && one_term ? kHalf : kAny;
}
// workgroups that the compute units hold together, by registers (two waves per SIMD; 32 x 96 of float32 numbers: as if two)
constexpr int loop_resident(int nw) { return 256 * 8 / nw; }
inline bool takes_turns(LastRound rule, int n_heads, int T, int resident) {
  if (rule == kAny || n_heads <= resident || T < 64) return false;
  const int last = (n_heads - 1) % resident + 1;
  const bool second = n_heads <= 2 * resident;
  const bool half = second && 4 * last >= resident && 2 * last <= resident;
  if (rule == kFullOrHalf) return half || 32 * last >= 31 * resident;
  if (rule == kThreeQuarters) return second && 4 * last > 3 * resident;
  return half;
}

template <int D, int DV, int NW, typename IO, bool FMAP, bool SPLIT>
hipError_t launch_kernel(const ForwardArgs& a, hipStream_t stream) {
  ForwardArgs args = a;
  void* params[] = {&args};
  constexpr LastRound kRule = loop_rule(D, DV, NW, sizeof(IO) == 4, sizeof(IO) == 2 && !FMAP);
  if constexpr (kRule != kAny) {
    if (takes_turns(kRule, a.n_heads, a.T, loop_resident(NW)))
      return hipLaunchKernel(reinterpret_cast<const void*>(&chunk_kernel<D, DV, NW, IO, FMAP, SPLIT, true>),
                             dim3(loop_resident(NW)), dim3(64 * NW), params, 0, stream);
  }
  return hipLaunchKernel(reinterpret_cast<const void*>(&chunk_kernel<D, DV, NW, IO, FMAP, SPLIT, false>), dim3(a.n_heads),
                         dim3(64 * NW), params, 0, stream);
}
template <int D, int DV, int NW, typename IO, bool SPLIT>
hipError_t launch(const ForwardArgs& a, hipStream_t stream) {
  // products on the FP32 instruction are for three-term operands only (d = 16 has no others)
  if constexpr (SPLIT || D == 16 || sizeof(IO) == 4) {
    if (a.feature_map == 0) return launch_kernel<D, DV, NW, IO, false, SPLIT>(a, stream);
  }
  return launch_kernel<D, DV, NW, IO, true, SPLIT>(a, stream);
}
// float32 q and k, or the feature map
template <int D, int DV, int NW>
hipError_t launch_three_terms(const ForwardArgs& a, int io_dtype, hipStream_t stream) {
  return io_dtype == 1        ? launch_kernel<D, DV, NW, uint16_t, true, true>(a, stream)
         : a.feature_map != 0 ? launch_kernel<D, DV, NW, float, true, true>(a, stream)
                              : launch_kernel<D, DV, NW, float, false, true>(a, stream);
}
// bf16 q and k without the feature map
template <int D, int DV, int NW>
hipError_t launch_one_term(const ForwardArgs& a, hipStream_t stream) {
  return launch_kernel<D, DV, NW, uint16_t, false, true>(a, stream);
}
template <int D, int DV, int NW, bool SPLIT = (D > 16)>
hipError_t launch_io(const ForwardArgs& a, int io_dtype, hipStream_t stream) {
  return io_dtype == 1 ? launch<D, DV, NW, uint16_t, SPLIT>(a, stream) : launch<D, DV, NW, float, SPLIT>(a, stream);
}

}  // namespace

bool chunk_supported(int d) { return d == 16 || d == 32 || d == 64 || d == 96 || d == 128; }

// Which kernel a call takes follows from the operand terms of k and q and not from the I/O type: one term for bf16
// numbers, three for float32 ones and for ELU(x) + 1 of either.  Three terms of K^ and Q, double-buffered, decide how
// many workgroups share a compute unit's LDS.  All times below: T = 512, ms.
static int operand_terms(const ForwardArgs& a, int io_dtype) { return io_dtype == 1 && a.feature_map == 0 ? 1 : 3; }
static int rounds(int n_heads, int resident) { return (n_heads + resident - 1) / resident; }

// The kernel with the A chain and the S chain on waves of their own (vla_chunk_pipe.hip)?  It shortens the chain of a block
// and holds twice the waves per head, so it wins as long as its workgroups are resident in one round, and beyond that
// where the other kernel leaves a compute unit with fewer waves than SIMDs' worth of work.  Waves of 16 columns, one term
// and three terms, this file's kernel / that one:
//   d = 128 (three terms): 16 heads 0.286 / 0.154, 256 heads 0.302 / 0.178, 512 heads 0.366 / 0.338, 768 heads 0.655 / 0.523
//     d_v = 96: 256 heads 0.243 / 0.141 and 0.298 / 0.160, 512 heads 0.283 / 0.251 and 0.364 / 0.307, 768 heads 0.515 / 0.376
//     and 0.655 / 0.470; d_v = 64: 256 heads 0.187 / 0.123 and 0.228 / 0.142, 512 heads 0.218 / 0.218 and 0.275 / 0.280, 768
//     heads 0.387 / 0.343 and 0.537 / 0.428; d_v = 32: 256 heads 0.168 / 0.122 and 0.209 / 0.144, 512 heads 0.200 / 0.225 and
//     0.260 / 0.290; d_v = 16 has none (one wave staged every token: 256 heads 0.153 / 0.151 and 0.176 / 0.205)
//   d =  96: 256 heads 0.199 / 0.115 and 0.250 / 0.130, 512 heads 0.231 / 0.211 and 0.296 / 0.254, 768 heads 0.447 / 0.319
//            and 0.561 / 0.386, 2048 heads 0.917 / 0.834 and 1.174 / 1.000
//     d_v = 128, one term: 256 heads 0.273 / 0.130, 512 heads 0.314 / 0.234, 2048 heads 1.247 / 0.920
//     d_v = 64: 256 heads 0.205 / 0.109 and 0.253 / 0.123, 768 heads 0.454 / 0.303 and 0.564 / 0.372, 2048 heads 0.939 / 0.796
//     and 1.188 / 0.974; d_v = 32, three terms: 256 heads 0.196 / 0.114, 512 heads 0.235 / 0.221, 768 heads 0.456 / 0.330, 2048
//     heads 0.932 / 0.865; d_v = 16: 512 heads 0.168 / 0.128 and 0.207 / 0.235, 2048 heads 0.671 / 0.621 and 0.830 / 0.945
//     The first block of each chain stands alone, so where this one has half the rounds of workgroups, two of its heads
//     beside each other win on the shortest sequences.  257 heads, 16 and 32 tokens, in us, before the C x C sections by panels:
//     96 x 96, three terms 16 / 19 and 26 / 28 (48 tokens: 35 / 36); 96 x 64, three terms 16 / 18 and 27 / 27; 96 x 128, one term
//     17 / 19 and 28 / 29.
//   d =  64 (three terms): 16 heads 0.118 / 0.080, 256 heads 0.121 / 0.084, 512 heads 0.147 / 0.122, 640 heads 0.177 / 0.192
//     d_v = 16: 512 heads 0.109 / 0.089 and 0.126 / 0.172; d_v = 32: 512 heads 0.121 / 0.103 and 0.140 / 0.164; d_v = 96: 256 heads
//     0.134 / 0.087 and 0.165 / 0.093, 512 heads 0.168 / 0.129 and 0.199 / 0.184; d_v = 128: 256 heads 0.128 / 0.092 and
//     0.159 / 0.100, 512 heads 0.160 / 0.141 and 0.197 / 0.159, 640 heads 0.191 / 0.206 and 0.237 / 0.238
//   d =  32: 256 heads 0.116 / 0.063 and 0.131 / 0.065, 1024 heads 0.120 / 0.102 and 0.135 / 0.110, 1536 heads 0.158 / 0.161
//            and 0.180 / 0.196
//     d_v = 64: 512 heads 0.126 / 0.086 and 0.141 / 0.092, 768 heads 0.128 / 0.106 and 0.145 / 0.118, 1024 heads 0.135 / 0.126
//     and 0.157 / 0.188; d_v = 96: 512 heads 0.151 / 0.092 and 0.167 / 0.097, 768 heads 0.154 / 0.119 and 0.178 / 0.128;
//     d_v = 128: 256 heads 0.137 / 0.077 and 0.158 / 0.079, 512 heads 0.170 / 0.108 and 0.195 / 0.116, 768 heads 0.175 / 0.166 and
//     0.204 / 0.179, 1024 heads 0.187 / 0.262 and 0.224 / 0.288
// The lines below do not reach every count at which that kernel is ahead, by the times above: beyond 256 heads 128 x 96 and, with
// three terms, 128 x 128 at any count (by 2 to 28 %), 128 x 64 and 128 x 32 from 513 to 768 (3 to 20 %), 96 x 96, 96 x 64 and 96 x 16
// with one term and 96 x 32 with three (6 to 33 %); 512 heads of 64 x 96 and 64 x 128 (8 to 24 %), 513 to 1024 of 32 x 64 and 32 x 96 (7
// to 28 %), 257 to 768 of 32 x 128 (5 to 40 %).
static bool pipe_narrow(int d_k, int d_v, int n_heads, int T, int terms) {
  switch (d_k) {
    case 128: return n_heads <= 256 && d_v > 16;
    case 96: {
      const bool any_length = terms == 1 ? d_v == 32 : d_v == 128;
      const bool blocks = terms == 1 ? d_v == 128 : d_v == 64 || d_v == 96;   // from a few blocks on
      return n_heads <= 256 || any_length ||
             (blocks && (T > (d_v == 96 ? 32 : 16) || rounds(n_heads, 256) < 2 * rounds(n_heads, 512)));
    }
    case 64: return n_heads <= 256 || (n_heads <= 512 && d_v <= 64 && (terms == 1 || d_v == 64));
    case 32: return n_heads <= (d_v <= 32 ? 1024 : d_v <= 96 ? 512 : 256);
    default: return false;
  }
}
// Its waves of 32 columns, one term, where the ones of 16 take more rounds, 16 / 32 columns: 300 heads of 128 0.272 / 0.222, 512
// 0.289 / 0.238, 768 0.439 / 0.386, 2048 1.174 / 0.950 (d_v = 64, against this file's kernel: 0.889 / 1.150, not taken); 257 heads of
// 64 0.102 / 0.099, 1024 0.202 / 0.163, 1280 0.242 / 0.229, 2048 0.391 / 0.336.
static bool pipe_wide(int d_k, int d_v, int n_heads, int terms) {
  return terms == 1 && d_k == d_v && (d_k == 64 || d_k == 128) && n_heads > 256;
}

// What is left for the kernel here: waves of 16 columns instead of 32?  Such a wave has half the splits and products
// between two serial sections but as much of everything else, so it pays while it runs on a SIMD that would be idle: as long
// as the narrow workgroups are resident in one round.  Wide / narrow waves, one term and three terms:
//   d = 128 (4 / 8 waves): d_v = 16: 256 heads 0.156 / 0.150 and 0.191 / 0.172, 512 heads 0.185 / 0.279 and 0.237 / 0.345
//   d =  64 (2 / 4 waves), one term: 768 heads of d_v = 16 0.156 / 0.128, of 96 0.228 / 0.205, of 128 0.267 / 0.200; 1024 heads 0.164 /
//     0.154, 0.245 / 0.355, 0.287 / 0.341; 1536 heads of 16 0.208 / 0.274.  Three terms narrow always (768 heads of d_v = 96 0.280 /
//     0.264, 1024 0.504 / 0.432 before the C x C sections by panels)
//   d =  32 (1 / 2 waves):
//     d_v = 64: 1024 heads 0.156 / 0.135 and 0.176 / 0.158, 1280 heads (three terms) 0.223 / 0.198, 1536: 0.225 / 0.290,
//               3072: 0.447 / 0.479, 2048 heads (one term) 0.205 / 0.287
//     d_v = 128: 1024 heads 0.713 / 0.188 (the wide wave's slab of S does not fit its registers)
static bool narrow_waves(int d_k, int d_v, int n_heads, int terms) {
  switch (d_k) {
    case 128: return n_heads <= 256;
    case 64: return n_heads <= 768 || terms == 3;
    case 32:
      if (d_v >= 96) return true;
      if (d_v == 64) return terms == 3 ? rounds(n_heads, 1280) <= rounds(n_heads, 1536) : n_heads <= 1024;
      return false;
    default: return false;
  }
}

// Three-term operands leave three workgroups of d = 64 and six of d = 32 (wide waves) a compute unit, FP32 products four
// and eight: those win where they save a round.  Square heads then take several heads per workgroup
// (vla_chunk_multihead.hip), others products on the FP32 instruction here.  float32, split / several heads:
//   d = 64: 768 heads 0.188 / 0.282, 1024: 0.329 / 0.278, 1536: 0.400 / 0.577, 2048: 0.567 / 0.569, 3072: 0.767 / 0.841
//   d = 32: 1024 heads 0.135 / 0.156, 1536: 0.180 / 0.216, 2048: 0.312 / 0.221, 3072: 0.364 / 0.426
// and, split / FP32 products here:
//   64 x 16: 768 heads 0.150 / 0.197, 1024: 0.273 / 0.222, 2048: 0.443 / 0.506     64 x 32: 1024 heads 0.311 / 0.246, 2048: 0.493 / 0.571
//   64 x 96: 768 heads 0.252 / 0.358, 1024: 0.427 / 0.360      64 x 128: 768 heads 0.252 / 0.426, 1024: 0.425 / 0.428
//   32 x 16: 1536 heads 0.156 / 0.167, 2048: 0.272 / 0.174    32 x 64: 1536 heads 0.225 / 0.255, 2048: 0.345 / 0.268, 3072: 0.447 / 0.505
static bool fewer_rounds_unsplit(int d_k, int n_heads) {
  if (d_k == 32) return rounds(n_heads, 2048) < rounds(n_heads, 1536);
  if (d_k == 64) return 11 * rounds(n_heads, 1024) < 8 * rounds(n_heads, 768);   // a round of each: 0.28 and 0.20 ms
  return false;
}
static bool fp32_products(int d_k, int d_v, int n_heads) {
  if (d_v == d_k) return false;
  if (d_k == 64) return n_heads > (d_v == 128 ? 896 : 768) && n_heads <= 1024;
  return d_v <= 64 && fewer_rounds_unsplit(d_k, n_heads);
}

// Key heads of 16: the blocks of 256 tokens at once (vla_chunk_d16.hip)?  A span costs a workgroup of 16 waves 8 us with
// four of its blocks there and 16 us with all, a block 3.2 us here; a compute unit holds one such workgroup, here eight
// heads.  Time here / there in us: 64 tokens, 1 head 14.9 / 7.9, 256 heads 15.6 / 8.7; 256 tokens 52.6 / 17.5 and 53.3 / 19.5;
// 2048 tokens 409 / 127 and 414 / 142 (d_v = 64: 534 / 197).  Two rounds, 512 heads: 64 tokens 15.6 / 15.8, 80 tokens 19.0 / 19.4
// (d_v = 64: 24.3 / 26.1), 96 tokens 22.4 / 21.5 (28.7 / 28.2), 272 tokens 57.6 / 47.3 (74.9 / 65.6), 2048 tokens 420 / 276;
// 257 heads are within 0.03 of these ratios.  Three rounds, 768 heads: 0.42 ms either way.  That kernel starts from the inverse of A0, so a given A0 (which need
// not have one) stays here, and so do value heads whose maps do not fit the LDS, lambda0 below 1e-6, where nothing
// was measured, and lambda0 whose reciprocal is zero or subnormal (an infinite one is A0 = 0).  The condition of what it
// inverts, up to (lambda0 + tokens) / lambda0, costs it 1e-16 of it in A k^; block after block loses 6e-8 of it.  Error of o,
// here / there: one key 4096 times, lambda0 = 0.04 6e-2 / 5e-5; four keys, lambda0 = 1e-6, 524288 tokens 38 / 0.3; keys of
// rank 4, lambda0 = 0.1, 16384 tokens 0.17 / 0.02; Gaussian keys, lambda0 = 1e-6, 300 tokens 0.09 / 4e-6.
static bool blocks_at_once(const ForwardArgs& a, int d_v) {
  return d_v <= 64 && a.A0 == nullptr && a.lambda0 >= 1e-6f && a.lambda0 <= 8e37f && a.T >= 64 &&
         (a.n_heads <= 256 || (a.n_heads <= 512 && a.T > 80));
}

// The waves of a head share out the d_v / 16 row tiles of S, evenly where the counts divide and one by one in turn where
// they do not: every pair of head sizes runs.
bool chunk_supported(int d_k, int d_v) { return chunk_supported(d_k) && chunk_supported(d_v); }

hipError_t launch_chunk(const ForwardArgs& a, int d_k, int d_v, int io_dtype, hipStream_t stream) {
  const int terms = operand_terms(a, io_dtype);
  if (d_k == 16 && blocks_at_once(a, d_v)) return launch_chunk_d16(a, d_v, io_dtype, stream);
  if (terms == 3 && d_k == d_v && fewer_rounds_unsplit(d_k, a.n_heads)) return launch_chunk_multihead(a, d_k, io_dtype, stream);
  if (terms == 3 && fp32_products(d_k, d_v, a.n_heads)) {
    switch (d_k * 1000 + d_v) {
      case 32016: return launch_io<32, 16, 1, false>(a, io_dtype, stream);
      case 32064: return launch_io<32, 64, 1, false>(a, io_dtype, stream);
      case 64016: return launch_io<64, 16, 2, false>(a, io_dtype, stream);
      case 64032: return launch_io<64, 32, 2, false>(a, io_dtype, stream);
      case 64096: return launch_io<64, 96, 2, false>(a, io_dtype, stream);
      case 64128: return launch_io<64, 128, 2, false>(a, io_dtype, stream);
      default: break;
    }
  }
  if (pipe_wide(d_k, d_v, a.n_heads, terms)) return launch_chunk_pipe_wide(a, d_k, stream);
  if (pipe_narrow(d_k, d_v, a.n_heads, a.T, terms)) return launch_chunk_pipe_narrow(a, d_k, d_v, io_dtype, stream);
  if (narrow_waves(d_k, d_v, a.n_heads, terms)) {
    switch (d_k * 1000 + d_v) {
      case 64016: return launch_io<64, 16, 4>(a, io_dtype, stream);
      case 64032: return launch_io<64, 32, 4>(a, io_dtype, stream);
      case 64064: return launch_three_terms<64, 64, 4>(a, io_dtype, stream);
      case 64096: return launch_io<64, 96, 4>(a, io_dtype, stream);
      case 64128: return launch_io<64, 128, 4>(a, io_dtype, stream);
      case 128016: return launch_io<128, 16, 8>(a, io_dtype, stream);
      case 32064: return launch_io<32, 64, 2>(a, io_dtype, stream);
      case 32096: return launch_io<32, 96, 2>(a, io_dtype, stream);
      case 32128: return launch_io<32, 128, 2>(a, io_dtype, stream);
      default: break;
    }
  }
  switch (d_k * 1000 + d_v) {   // what pipe_wide and pipe_narrow leave; d_k = 64: one term only, see narrow_waves
    case 16016: return launch_io<16, 16, 1>(a, io_dtype, stream);
    case 32032: return launch_io<32, 32, 1>(a, io_dtype, stream);
    case 96096: return launch_io<96, 96, 3>(a, io_dtype, stream);
    case 128128: return launch_three_terms<128, 128, 4>(a, io_dtype, stream);
    case 16032: return launch_io<16, 32, 1>(a, io_dtype, stream);
    case 32016: return launch_io<32, 16, 1>(a, io_dtype, stream);
    case 32064: return launch_io<32, 64, 1>(a, io_dtype, stream);
    case 64032: return launch_one_term<64, 32, 2>(a, stream);
    case 64128: return launch_one_term<64, 128, 2>(a, stream);
    case 128064: return launch_io<128, 64, 4>(a, io_dtype, stream);
    case 16064: return launch_io<16, 64, 1>(a, io_dtype, stream);
    case 16096: return launch_io<16, 96, 1>(a, io_dtype, stream);
    case 16128: return launch_io<16, 128, 1>(a, io_dtype, stream);
    case 64096: return launch_one_term<64, 96, 2>(a, stream);
    case 64016: return launch_one_term<64, 16, 2>(a, stream);
    case 96016: return launch_io<96, 16, 3>(a, io_dtype, stream);
    case 96032: return launch_three_terms<96, 32, 3>(a, io_dtype, stream);
    case 96064: return launch_io<96, 64, 3>(a, io_dtype, stream);
    case 96128: return launch_one_term<96, 128, 3>(a, stream);
    case 128016: return launch_io<128, 16, 4>(a, io_dtype, stream);
    case 128032: return launch_io<128, 32, 4>(a, io_dtype, stream);
    case 128096: return launch_io<128, 96, 4>(a, io_dtype, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace vla
