// Block form of the VLA recurrence with the optional lines of Algorithm 1 (paper, pseudocode appendix) on
// MFMA: a penalty direction u_t supplied separately from the key (eq. (penalty)), the periodic identity
// refresh A += eta I, the normalised read-out of eq. (output) with its running key sum, and the ELU+1
// feature map on q and k (Section 3.3).
//
// Within a block of at most C = 16 tokens (rows = tokens), entering state A0 (symmetric), S0:
//
//   Y^T = U A0 ,  X^T = K^ A0                        (C x d)   z and A0 k^ before the in-block corrections
//   G = Y^T U^T = L L^T - I                          (C x C)   L_tt^2 = delta_t
//   W^T = L^{-1} Y^T                                 (C x d)   A_t = A0 - sum_{s<=t} w_s w_s^T   (eq. (sm))
//   Hm = L^{-1} (Y^T K^^T)                           (C x C)   Hm[s][t] = w_s . k^_t
//   alpha_t = x_t - sum_{s<=t} Hm[s][t] w_s                    = A_t k^_t          (post-update A)
//   c_t = 1 / max(||alpha_t||, eps)                            alpha^_t = c_t alpha_t
//   P[s][t] = alpha_s . k^_t = (X^T K^^T)[s][t] - sum_{r<=s} Hm[r][s] Hm[r][t]
//   AQ[s][t] = alpha_s . q_t = (X^T Q^T)[s][t] - sum_{r<=s} Hm[r][s] (L^{-1} Y^T Q^T)[r][t]
//   F^T = V - K^ S0^T ,  E^T = Z F^T ,  Z = (I + N)^{-1},  N[t][s] = c_s P[s][t] for s < t    (eq. (s-update))
//   O^T = Q S0^T + NQ^T E^T ,  NQ[s][t] = c_s AQ[s][t] for s <= t, else 0
//   S1^T = S0^T + Alpha diag(c) E^T ,  A1 = A0 - W W^T
//
// With u = k^ and no refresh the rows of X and Y coincide and this reduces to the block form of the plain
// kernel (template flag FULL = false: one sweep of A, two Gram matrices).
//
// Identity refresh: a step whose 1-based index is a multiple of the period adds eta I to A after the
// rank-1 update and before the write direction is formed, anywhere inside a block.  With n_t the number of
// refresh steps among the block's tokens before t and n'_t = n_{t+1} (before or at t), token t updates with
// A0 + eta n_t I - sum_{r<t} w_r w_r^T and writes with A0 + eta n'_t I - sum_{r<=t} w_r w_r^T, so everything
// above holds with
//   y'_t = y_t + eta n_t u_t ,   x'_t = x_t + eta n'_t k^_t
// in place of y_t, x_t (the Gram matrices are formed from Y', X'), with the matrix to factor taken as
// I + u_s . y'_t for t <= s (the upper triangle of Y' U^T, mirrored: the base matrix of the earlier token
// counts), and A1 = A0 + eta n_C I - W W^T.
//
// Normalised read-out: o_t is divided by max(q_t . zkey_t, eps), zkey_t = zkey_0 + sum_{s<=t} k_s with k_s
// the key as used before L2 normalisation, k_s = max(||k_s||, eps) k^_s; inside a block
// q_t . zkey_t = q_t . zkey_start + sum_{s<=t} ||k_s|| (Q K^^T)[t][s].
//
// Work split: D/SL waves per (batch, head); wave w owns columns [SL w, SL w + SL) of A (SL = 16 or 32) and
// the row tiles w, w + D/SL, ... of S as 16x16 MFMA accumulator tiles
// resident in VGPRs for the whole sequence.  The C x C Gram matrices are
// shared out over the waves (each one contracts over the whole head dimension), the C x C factorisations
// run on one wave each, rotating with the block index.
//
// What bounds it: the chain of five barriers of one block, of which a second workgroup on the compute unit hides
// part.  The sweeps over A and S and the Gram matrices are FP32 products on split bf16 terms (vla_mfma_util.h); Y and X
// share their LDS with W and Alpha and the next block is staged at the end of a block, so that two workgroups
// of d = 128 fit a compute unit (80 KB each).  Every option on, 2048 heads of 128, 8192 tokens, bf16: 43.7 ms with FP32
// matrix instructions and one workgroup per compute unit, 35.6 ms so, and 25.2 with the two chains on waves of their own
// (vla_chunk_general_pipe.hip), which takes most calls; pipe_narrow() and pipe_wide() below say which.
#include "vla_mfma_util.h"

namespace vla {
namespace {

// C x C Gram matrices of a block, [m][n] = sum_j left[m][j] right[n][j]
enum GramTile {
  kG = 0,   // Y U^T
  kGK,      // Y K^^T
  kGQ,      // Y Q^T
  kGX,      // X K^^T
  kXQ,      // X Q^T
  kQK,      // Q K^^T      (normalised read-out)
  kQZ,      // Q zkey^T    (normalised read-out; only column 0 is populated)
  kNumGram
};

// Waves per SIMD that the kernel's registers are cut for: as many workgroups as its LDS lets a compute unit hold, but
// no more than its accumulator tiles leave registers for (value heads wider than key heads: two).
constexpr int general_waves_per_simd(int d, int d_v, int sl, bool db) {
  return sl == 32 || d <= 32 || d == 128 || d_v > d || db ? 2 : 3;
}

// FULL: Y and X differ (a separate u, or a refresh period): two sweeps of A and five Gram matrices.
// SCAN: phase 1 of the two-phase and time-parallel modes: one workgroup per (head, time segment) runs the A
//       chain only, from the A the segment starts with, and writes what the S recurrence needs into the
//       workspace (the layout of vla_mfma_util.h: 1 / ||k_t||, the write directions alpha_t in W's place, Z,
//       -NQ^T, -c_t and the reciprocal read-out denominators); S, v and o are not touched.
// DV: head size of v and o (rows of S).  The DV / 16 row tiles of S go to the waves in turn (tile t to wave
//     t % NW: exactly one each for square heads); a wave with fewer tiles than the others, or none, runs its spare
//     slots on a copy of the last tile and stores nothing from them.
// SPLIT: products on split bf16 terms, else on the FP32 matrix instruction.
template <int D, int DV, int SL, typename IO, bool FULL, bool SCAN, bool DB, bool SPLIT>
__global__ void __launch_bounds__(64 * D / SL, general_waves_per_simd(D, DV, SL, DB)) chunk_general_kernel(ForwardArgs a) {
  constexpr int NW = D / SL;       // waves; wave w owns columns SL w .. SL w + SL - 1 of A
  constexpr int NJ = SL / 16;      // 16-wide tiles in a slab of A
  constexpr int TV = DV / 16;      // row tiles of S
  constexpr int NJV = (TV + NW - 1) / NW;   // tile slots per wave
  static_assert(DV % 16 == 0 && (!SCAN || DV == D), "whole tiles of S");
  constexpr int NB = D / 16;       // 16-row blocks over the head dimension
  // Staging: a token row is split over thread slots of EPT elements.  At the power-of-two head sizes every
  // thread stages 4 or 8 elements; at d = 96 a row takes 12 threads of 8 elements in a group of 16 (the other four
  // lanes of the group and the last two waves stage nothing), so that a row sums with a power-of-two shuffle.
  constexpr bool PADDED = (D & (D - 1)) != 0;
  static_assert(!PADDED || NJ == 1, "d = 96: waves of 16 columns");
  constexpr int EPT = PADDED ? 8 : 4 * NJ;      // staged elements per thread per tensor
  constexpr int TPR = PADDED ? 16 : D / EPT;    // thread slots per token row (inside one wave)
  static_assert(D % EPT == 0 && D / EPT <= TPR && C * TPR <= 64 * NW, "staging layout");
  // Y = X: the Gram matrices that differ only in u against k^ coincide
  constexpr int iGK = FULL ? kGK : kG;
  constexpr int iGX = FULL ? kGX : kG;
  constexpr int iXQ = FULL ? kXQ : kGQ;

  // Products over the head dimension and over the tokens on split bf16 terms (vla_mfma_util.h).  Keys are staged
  // normalised and mapped, directions scaled: float32 numbers, three terms each.
  using Ops = BlockOps<SPLIT, SPLIT ? 3 : 1, D>;
  constexpr int STEP = Ops::STEP;
  constexpr int NKB = NB / STEP;      // steps of a contraction over the head dimension
  static_assert(NB % STEP == 0, "whole steps");
  // Y^T and X^T live until the Gram matrices are formed, W and Alpha from then to the end of the block.  DB: regions of
  // their own, and K^ and Q double-buffered, so that the next block is staged beside the serial sections.  Otherwise
  // one region and single buffers, at the price of staging behind one more barrier.
  constexpr int kYX = (FULL ? 2 : 1) * Ops::SIZE * 2;            // bytes
  constexpr int kWA = (SCAN ? 1 : 2) * D * 4 * (16 + 8);
  __shared__ __align__(16) uint16_t Ksb[DB ? 2 : 1][Ops::SIZE]; // K^ [t][j]
  __shared__ __align__(16) uint16_t Qsb[DB ? 2 : 1][Ops::SIZE]; // Q  [t][j]
  __shared__ __align__(16) uint16_t Usb[FULL ? Ops::SIZE : 8];    // U  [t][j]
  __shared__ __align__(16) unsigned char region[DB ? kYX + kWA : (kYX > kWA ? kYX : kWA)];
  uint16_t* Ys = reinterpret_cast<uint16_t*>(region);             // Y^T [t][j]
  uint16_t* Xs = FULL ? Ys + Ops::SIZE : Ys;                      // X^T [t][j]
  unsigned char* const wa_region = region + (DB ? kYX : 0);
  u4* Whm = reinterpret_cast<u4*>(wa_region);                        // W [j][t]
  u2* Wl = reinterpret_cast<u2*>(wa_region + D * 4 * 16);
  u4* Ahm = reinterpret_cast<u4*>(wa_region + D * 4 * 24);           // Alpha [j][t]
  u2* Al = reinterpret_cast<u2*>(wa_region + D * 4 * 40);
  __shared__ __align__(16) float Gs[kNumGram][C * LT];
  __shared__ __align__(16) float Lis[C * LT];         // L^{-1} [t][s]
  __shared__ __align__(16) float Ps[C * LT];          // P transposed: [t][s] = alpha_s . k^_t
  __shared__ __align__(16) float Zs[C * LT];          // Z   [t][s]
  __shared__ __align__(16) float NQs[C * LT];         // -NQ^T [t][s]
  __shared__ __align__(16) float wn2p[NW][C];         // per-wave partial ||alpha_t||^2
  __shared__ __align__(16) float cvec[C];             // -c_t
  __shared__ __align__(16) float rdens[C];            // 1 / max(q_t . zkey_t, eps)
  __shared__ __align__(16) float nks[2][C];           // max(||k_t||, eps), double-buffered over blocks
  __shared__ __align__(16) float zks[D];              // running key sum (each wave touches its own columns)
  __shared__ __align__(16) float ens[2][C + 4];       // eta n_i, i = 0..C: refresh steps among a block's first i tokens

  const int head = SCAN ? blockIdx.x / a.n_seg : blockIdx.x;
  const int seg = SCAN ? blockIdx.x - head * a.n_seg : 0;
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  int c = lane & 15;
  int g = lane >> 4;
  const int tb = SCAN ? seg * a.seg_blocks * C : 0;                 // first token of this workgroup's range
  const int T = SCAN ? min(a.T, tb + a.seg_blocks * C) : a.T;       // one past its last token
  const float eps = a.eps;
  const int col0 = SL * w;
  const int period = a.refresh_period;
  const float eta = a.refresh_eta;
  const bool norm_out = a.normalise_output != 0;
  const bool key_sum = norm_out || a.zkey_T != nullptr;
  const bool fmap = a.feature_map != 0;
  const bool has_u = a.u != nullptr;
  // first S row of this wave's tile slot jn, and whether the slot holds a tile of its own
  auto s_row = [&](int jn) -> int {
    const int t = w + NW * jn;
    return 16 * (t < TV ? t : TV - 1);
  };
  auto owns = [&](int jn) -> bool { return w + NW * jn < TV; };
  // ---- resident state: At[jn][b][r] = A[16b + 4g + r][col0 + 16jn + c],  St[jn][b][r] = S[s_row(jn) + c][16b + 4g + r]
  f4 At[NJ][NB], St[NJV][NB];
  {
    const float* A0 = (SCAN && a.seg_A) ? a.seg_A + static_cast<size_t>(blockIdx.x) * D * D
                                        : (a.A0 ? a.A0 + static_cast<size_t>(head) * D * D : nullptr);
    const float* S0 = (!SCAN && a.S0) ? a.S0 + static_cast<size_t>(head) * DV * D : nullptr;
    const float diag = 1.0f / a.lambda0;
    const int arc = (4 * g) * D + col0 + c;
    const int src = c * D + 4 * g;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
#pragma unroll
      for (int jn = 0; jn < NJ; ++jn) {
        if (A0) {
#pragma unroll
          for (int r = 0; r < 4; ++r) At[jn][b][r] = A0[arc + (16 * b + r) * D + 16 * jn];
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r) At[jn][b][r] = (16 * b + 4 * g + r == col0 + 16 * jn + c) ? diag : 0.0f;
        }
      }
#pragma unroll
      for (int jn = 0; jn < NJV; ++jn) {
        if (S0) {
          const float4 x = *reinterpret_cast<const float4*>(S0 + src + s_row(jn) * D + 16 * b);
          St[jn][b] = f4{x.x, x.y, x.z, x.w};
        } else {
          St[jn][b] = f4{0, 0, 0, 0};
        }
      }
    }
  }
  if (lane < SL) {   // key sum entering this range: the caller's, or the one the segment starts with
    const float* z0 = (SCAN && a.seg_zkey) ? a.seg_zkey + static_cast<size_t>(blockIdx.x) * D
                                           : (a.zkey0 ? a.zkey0 + static_cast<size_t>(head) * D : nullptr);
    zks[col0 + lane] = z0 ? z0[col0 + lane] : 0.0f;
  }
  // workspace records of this head (SCAN)
  const int nblk_all = (a.T + C - 1) / C;
  float* wsh = SCAN ? a.ws + static_cast<size_t>(head) * head_stride(nblk_all, D) : nullptr;
  float* RN = SCAN ? wsh + off_rn(nblk_all, D) : nullptr;
  float* WT = SCAN ? wsh + off_wt(nblk_all, D) : nullptr;
  float* SMp = SCAN ? wsh + off_sm(nblk_all, D) : nullptr;

  const size_t slab = static_cast<size_t>(head) * static_cast<size_t>(a.T) * D;
  const IO* qh = static_cast<const IO*>(a.q) + slab;
  const IO* kh = static_cast<const IO*>(a.k) + slab;
  const size_t slab_v = static_cast<size_t>(head) * static_cast<size_t>(a.T) * DV;
  const IO* vh = static_cast<const IO*>(a.v) + slab_v;
  const IO* uh = has_u ? static_cast<const IO*>(a.u) + slab : kh;
  IO* oh = static_cast<IO*>(a.o) + slab_v;

  // staging role of this thread: token row and 4-element column segment
  const int srow = tid / TPR;
  const int sseg = (tid % TPR) * EPT;
  const bool stager = !PADDED || (tid < C * TPR && sseg < D);   // this thread holds a row segment
  const bool stage_wave = !PADDED || tid < C * TPR;             // uniform per wave

  RawRow<IO, EPT> kpre, qpre, upre;
  IO vpre[NJV][4];  // V in accumulator layout: V[t0 + 4g + r][s_row(jn) + c]

  // Loads never branch on the row: rows past the end read the last valid row and are zeroed when consumed.
  auto load_kqu = [&](int t0) {
    if (stager) {
      const int tr = t0 + srow;
      const unsigned off = static_cast<unsigned>((tr < T ? tr : T - 1) * D + sseg);
      kpre.load(kh + off);
      qpre.load(qh + off);
      if (has_u) upre.load(uh + off);
    }
  };
  auto load_v = [&](int t0) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int t = t0 + 4 * g + r;
      const unsigned voff = static_cast<unsigned>((t < T ? t : T - 1) * DV + c);
#pragma unroll
      for (int jn = 0; jn < NJV; ++jn) vpre[jn][r] = vh[voff + s_row(jn)];
    }
  };
  auto row_total = [&](float x) -> float {
#pragma unroll
    for (int off = TPR / 2; off >= 1; off >>= 1) x += __shfl_xor(x, off);
    return x;
  };
  // 1 / max(sqrt(ss), eps): hardware reciprocal square root refined by one Newton step
  auto inv_norm = [&](float ss, float& clamped) -> float {
    clamped = fmaxf(ss, eps * eps);
    const float rn = __builtin_amdgcn_rsqf(clamped);
    return rn * fmaf(-0.5f * clamped * rn, rn, 1.5f);
  };
  // this thread's share of the block of `len` live tokens that starts at token tfirst (step index idx0, 1-based,
  // counted over the whole sequence): K^, Q (and U) into LDS, key norms and refresh counts into half `buf`
  auto stage = [&](int len, int idx0, int buf, int tfirst) __attribute__((always_inline)) {
    if (!stage_wave) return;
    const bool live = srow < len && stager;
    float x[EPT], kn[EPT];
    if (stager) {
      kpre.unpack(x);
    } else {
#pragma unroll
      for (int e = 0; e < EPT; ++e) x[e] = 0.0f;
    }
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      if (fmap) x[e] = elu_plus_one(x[e]);
      x[e] = live ? x[e] : 0.0f;
    }
    float ss = 0.0f;
#pragma unroll
    for (int e = 0; e < EPT; ++e) ss = fmaf(x[e], x[e], ss);
    float sm;
    const float rn = inv_norm(row_total(ss), sm);
#pragma unroll
    for (int e = 0; e < EPT; ++e) kn[e] = x[e] * rn;
    float us[EPT];
    float su = 0.0f;
    if constexpr (FULL) {
      if (has_u) {
        if (stager) {
          upre.unpack(us);
        } else {
#pragma unroll
          for (int e = 0; e < EPT; ++e) us[e] = 0.0f;
        }
#pragma unroll
        for (int e = 0; e < EPT; ++e) us[e] = live ? us[e] : 0.0f;
        float uu = 0.0f;
#pragma unroll
        for (int e = 0; e < EPT; ++e) uu = fmaf(us[e], us[e], uu);
        float um;
        su = a.u_scale * inv_norm(row_total(uu), um);
      }
      if (tid <= C) {  // multiples of the period among the step indices idx0 .. idx0 + tid - 1
        const int n = period > 0 ? (idx0 - 1 + tid) / period - (idx0 - 1) / period : 0;
        ens[buf][tid] = eta * static_cast<float>(n);
      }
    }
    if (!stager) return;
#pragma unroll
    for (int e = 0; e < EPT; e += 4) {
      Ops::put4(Ksb[DB ? buf : 0], srow, sseg + e, f4{kn[e], kn[e + 1], kn[e + 2], kn[e + 3]});
    }
    if (sseg == 0) {
      nks[buf][srow] = sm * rn;  // max(||k||, eps)
      if constexpr (SCAN) RN[tfirst + srow] = live ? rn : 0.0f;   // rows past the end: zero keys
    }
    qpre.unpack(x);
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      if (fmap) x[e] = elu_plus_one(x[e]);
      x[e] = live ? x[e] : 0.0f;
    }
#pragma unroll
    for (int e = 0; e < EPT; e += 4) {
      Ops::put4(Qsb[DB ? buf : 0], srow, sseg + e, f4{x[e], x[e + 1], x[e + 2], x[e + 3]});
    }
    if constexpr (FULL) {
#pragma unroll
      for (int e = 0; e < EPT; e += 4) {
        Ops::put4(Usb, srow, sseg + e,
                  has_u ? f4{us[e] * su, us[e + 1] * su, us[e + 2] * su, us[e + 3] * su}
                        : f4{kn[e], kn[e + 1], kn[e + 2], kn[e + 3]});   // u = k^ without a separate direction
      }
    }
  };

  if (tb < T) {
    load_kqu(tb);
    if constexpr (!SCAN) load_v(tb);
    stage(T - tb < C ? T - tb : C, a.step_offset + tb + 1, 0, tb);
    if (DB && tb + C < T) load_kqu(tb + C);
  }
  __syncthreads();  // first block staged, zks initialised

  int blk = 0;
  for (int t0 = tb; t0 < T; t0 += C, ++blk) {
    const uint16_t* Ks = Ksb[DB ? blk & 1 : 0];
    const uint16_t* Qs = Qsb[DB ? blk & 1 : 0];
    const uint16_t* Us = FULL ? Usb : Ks;
    const float* en = ens[blk & 1];
    const int len = T - t0 < C ? T - t0 : C;
    const int tn = t0 + C;                           // start of the next block
    auto stage_next = [&]() {
      if (tn < T) stage(T - tn < C ? T - tn : C, a.step_offset + tn + 1, (blk + 1) & 1, tn);
    };
    // keeps addresses from being hoisted out of the loop, where the large heads have no registers for them
    if constexpr (D >= 96) asm volatile("" : "+v"(c), "+v"(g));
    int cc = c;  // opaque copy: keeps lane-dependent masks from being hoisted out of the loop
    asm volatile("" : "+v"(cc));

    // ================= Y^T = U A0, X^T = K^ A0 (this wave's columns) -> LDS
    f4 yt[NJ], xt[NJ];
#pragma unroll
    for (int jn = 0; jn < NJ; ++jn) yt[jn] = xt[jn] = f4{0, 0, 0, 0};
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) {
#pragma unroll
      for (int jn = 0; jn < NJ; ++jn) {
        const auto ab = Ops::tiles(At[jn][STEP * kb], At[jn][STEP * kb + STEP - 1]);
        yt[jn] = Ops::sweep(Ops::operand(Us, kb, c, g), ab, yt[jn]);
        if constexpr (FULL) xt[jn] = Ops::sweep(Ops::operand(Ks, kb, c, g), ab, xt[jn]);
        if (NJ > 1) __builtin_amdgcn_sched_barrier(0);   // one split at a time in registers
      }
    }
    if constexpr (FULL) {
      if (period > 0) {  // y'_t = y_t + eta n_t u_t,  x'_t = x_t + eta n'_t k^_t  (n'_t = n_{t+1})
        const f4 e0 = lds4(&en[4 * g]);
        const f4 e1 = f4{e0[1], e0[2], e0[3], en[4 * g + 4]};
#pragma unroll
        for (int jn = 0; jn < NJ; ++jn)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            yt[jn][r] = fmaf(e0[r], Ops::get(Us, 4 * g + r, col0 + 16 * jn + c), yt[jn][r]);
            xt[jn][r] = fmaf(e1[r], Ops::get(Ks, 4 * g + r, col0 + 16 * jn + c), xt[jn][r]);
          }
      }
    }
#pragma unroll
    for (int jn = 0; jn < NJ; ++jn) {
      if constexpr (!FULL) xt[jn] = yt[jn];
      Ops::put_column(Ys, 4 * g, col0 + 16 * jn + c, yt[jn]);
      if constexpr (FULL) Ops::put_column(Xs, 4 * g, col0 + 16 * jn + c, xt[jn]);
    }
    __syncthreads();  // (1) Y^T, X^T complete

    // ================= Gram matrices, shared out over the waves
    {
      int slot = 0;
#pragma unroll
      for (int i = 0; i < kNumGram; ++i) {
        if (!FULL && (i == kGK || i == kGX || i == kXQ)) continue;
        if ((i == kQK || i == kQZ) && !norm_out) continue;
        const bool mine = (slot % NW) == w;
        ++slot;
        if (!mine) continue;
        const uint16_t* left = (i == kG || i == kGK || i == kGQ) ? Ys : (i == kGX || i == kXQ) ? Xs : Qs;
        const uint16_t* right = (i == kG) ? Us : (i == kGK || i == kGX || i == kQK) ? Ks : Qs;
        f4 acc[2] = {f4{0, 0, 0, 0}, f4{0, 0, 0, 0}};  // two chains: the tile is one wave's whole job here
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
          const auto av = Ops::operand(left, kb, c, g);
          if (i == kQZ) {
            const f4 zero{0, 0, 0, 0};
            const f4 z0 = cc == 0 ? lds4(&zks[16 * STEP * kb + 4 * g]) : zero;
            const f4 z1 = cc == 0 && SPLIT ? lds4(&zks[SPLIT ? 32 * kb + 16 + 4 * g : 0]) : zero;
            acc[kb & 1] = Ops::sweep(av, Ops::tiles(z0, z1), acc[kb & 1]);
          } else {
            acc[kb & 1] = Ops::sweep(av, Ops::operand(right, kb, c, g), acc[kb & 1]);
          }
        }
        acc[0] += acc[1];
#pragma unroll
        for (int r = 0; r < 4; ++r) Gs[i][(4 * g + r) * LT + c] = acc[0][r];
      }
    }
    __syncthreads();  // (2) Gram matrices visible

    // ================= phase 1 (one wave): Cholesky of I + G and L^{-1}
    const int sw = (blk + head) % NW;
    const int sw2 = (sw + (NW > 2 ? NW / 2 + 1 : 1)) % NW;  // another wave, on another SIMD, forms c, Z, NQ
    // -F^T = K^ S0^T - V^T and R^T = Q S0^T in one pass over S; needed only after barrier (5)
    f4 ft[NJV], ot[NJV];
    auto s_pass = [&]() {
#pragma unroll
      for (int jn = 0; jn < NJV; ++jn) {
        ot[jn] = f4{0, 0, 0, 0};
#pragma unroll
        for (int r = 0; r < 4; ++r) ft[jn][r] = (4 * g + r < len) ? neg_widen(vpre[jn][r]) : 0.0f;
      }
      if (tn < T) load_v(tn);
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb) {
#pragma unroll
        for (int jn = 0; jn < NJV; ++jn) {
          const auto sb = Ops::tiles(St[jn][STEP * kb], St[jn][STEP * kb + STEP - 1]);
          ft[jn] = Ops::sweep(Ops::operand(Ks, kb, c, g), sb, ft[jn]);
          ot[jn] = Ops::sweep(Ops::operand(Qs, kb, c, g), sb, ot[jn]);
          if (NJ > 1) __builtin_amdgcn_sched_barrier(0);
        }
      }
    };
    // zkey += sum over the block's tokens of ||k_s|| k^_s, this wave's columns (read by the Gram products only)
    auto key_sum_pass = [&]() {
      if (!key_sum) return;
      const f4 nk = lds4(&nks[blk & 1][4 * g]);
#pragma unroll
      for (int jn = 0; jn < NJ; ++jn) {
        float z = 0.0f;
#pragma unroll
        for (int r = 0; r < 4; ++r) z = fmaf(nk[r], Ops::get(Ks, 4 * g + r, col0 + 16 * jn + c), z);
        z += __shfl_xor(z, 16);
        z += __shfl_xor(z, 32);
        if (lane < 16) zks[col0 + 16 * jn + lane] += z;
      }
    };
    if (w != sw) {
      if constexpr (DB) stage_next();
      if constexpr (!SCAN) s_pass();
      key_sum_pass();
      if (DB && tn + C < T) load_kqu(tn + C);
    } else {
      __builtin_amdgcn_s_setprio(3);   // the dependent chain is what the other waves wait for: issue it first
      f4 gram;
      if (FULL && period > 0) {  // entry (c, s) with s < c from its mirror image (s, c): see the header
#pragma unroll
        for (int r = 0; r < 4; ++r) gram[r] = Gs[kG][(4 * g + r) * LT + c];
      } else {
        gram = lds4(&Gs[kG][c * LT + 4 * g]);
      }
      const Lane at = fresh_lane(c, g);
      cholesky16<false>(gram, nullptr, Lis, at.c, at.g);
      __builtin_amdgcn_s_setprio(0);
    }
    __syncthreads();  // (3) L^{-1} visible

    // ================= W^T = L^{-1} Y^T,  Hm = L^{-1} (Y K^^T),  Alpha^T = X^T - M W^T,  ||alpha_t||^2
    const f4 la = lds4(&Lis[c * LT + 4 * g]);
    f4 mop;   // M as an A operand: M[t = c][s = 4g + r] = Hm[s][t] for s <= t
    f4 nhm;   // -Hm in accumulator layout
    {
      f4 hm = f4{0, 0, 0, 0};
#pragma unroll
      for (int r = 0; r < 4; ++r) hm = mfma16(la[r], Gs[iGK][(4 * g + r) * LT + c], hm);
      nhm = -hm;
#pragma unroll
      for (int r = 0; r < 4; ++r) mop[r] = (4 * g + r <= cc) ? hm[r] : 0.0f;
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
        if constexpr (SCAN) {
          *reinterpret_cast<f4*>(WT + (static_cast<size_t>(t0 / C) * D + col0 + 16 * jn + c) * C + 4 * g) = at;
        } else {
          Ops::w_store(Ahm, Al, col0 + 16 * jn + c, c, g, at);
        }
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) n2[r] = row_sum16(n2[r]);
      if (c == 0) *reinterpret_cast<f4*>(&wn2p[w][4 * g]) = n2;
    }
    __syncthreads();  // (4) W, Alpha and the norm partials visible

    // ================= phase 2 (wave sw2): c_t, Z, NQ, read-out denominators -- the others update A
    auto update_A = [&]() {
      Ops::template downdate<NB, NJ>(Whm, Wl, col0 + c, c, g, blk & 1, [&](int b, int jn) -> f4& { return At[jn][b]; });
      if (FULL && period > 0) {  // + eta n on the diagonal (row 16b + 4g + r against column col0 + 16jn + c), n counted
        const float en_end = en[len];  // over the live tokens
#pragma unroll
        for (int b = 0; b < NB; ++b) {
#pragma unroll
          for (int jn = 0; jn < NJ; ++jn) {
            if (b == NJ * w + jn) {
#pragma unroll
              for (int r = 0; r < 4; ++r) At[jn][b][r] += (4 * g + r == cc) ? en_end : 0.0f;
            }
          }
        }
      }
    };
    if (w != sw2) update_A();
    if (w == sw) {
      if constexpr (DB) stage_next();
      if constexpr (!SCAN) s_pass();
      key_sum_pass();
      if (DB && tn + C < T) load_kqu(tn + C);
    }
    if (w == sw2) {
      __builtin_amdgcn_s_setprio(3);
      float wn2 = 0.0f;
#pragma unroll
      for (int ww = 0; ww < NW; ++ww) wn2 += wn2p[ww][c];
      const float cs = __builtin_amdgcn_rcpf(fmaxf(__builtin_amdgcn_sqrtf(wn2), eps));  // alpha^_t = c_t alpha_t
      float* smb = SCAN ? SMp + static_cast<size_t>(t0 / C) * SMB : nullptr;   // this block's record
      if (g == 0) {
        if constexpr (SCAN) smb[2 * C * C + c] = -cs;
        else cvec[c] = -cs;
      }
      // P and AQ in accumulator layout [s = 4g + r][t = c]
      f4 pt, aq;
      f4 nhq = f4{0, 0, 0, 0};
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        pt[r] = Gs[iGX][(4 * g + r) * LT + c];
        aq[r] = Gs[iXQ][(4 * g + r) * LT + c];
        nhq = mfma16(-la[r], Gs[kGQ][(4 * g + r) * LT + c], nhq);  // -(L^{-1} Y Q^T)
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        pt = mfma16(mop[r], nhm[r], pt);
        aq = mfma16(mop[r], nhq[r], aq);
      }
      // same wave writes and reads: LDS operations of one wave are ordered
      *reinterpret_cast<f4*>(&Ps[c * LT + 4 * g]) = pt;
      const Lane at = fresh_lane(c, g);
      lower_inverse16(Ps, cs, at.c, at.g, [&](int t, int s, float z) {   // N[t][s] = c_s P[s][t]
        if constexpr (SCAN) smb[static_cast<unsigned>(t * C + s)] = z;
        else Zs[t * LT + s] = z;
      });
      f4 nq;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int s = 4 * g + r;
        const float csr = __shfl(cs, s);
        nq[r] = (s <= c) ? -(csr * aq[r]) : 0.0f;
        if constexpr (!SCAN) NQs[c * LT + s] = nq[r];
      }
      if constexpr (SCAN) *reinterpret_cast<f4*>(smb + C * C + c * C + 4 * g) = nq;  // -NQ^T[t = c][s = 4g + r]
      if (norm_out) {  // q_t . zkey_t for t = 4g + r: key-sum part + in-block part over s = c <= t
        const float nk = nks[blk & 1][c];
        f4 den;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float qk = Gs[kQK][(4 * g + r) * LT + c];
          const float qz = Gs[kQZ][(4 * g + r) * LT + c];
          den[r] = row_sum16(qz + ((cc <= 4 * g + r) ? qk * nk : 0.0f));
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) den[r] = 1.0f / fmaxf(den[r], eps);
        if (c == 0) {
          if constexpr (SCAN) *reinterpret_cast<f4*>(smb + 2 * C * C + C + 4 * g) = den;
          else *reinterpret_cast<f4*>(&rdens[4 * g]) = den;
        }
      }
      __builtin_amdgcn_s_setprio(0);
    }
    __syncthreads();  // (5) Z, NQ, c, denominators visible; K^, Q, U no longer needed

    // ================= -E^T = Z (-F^T), O^T = Q S0^T + (-NQ^T)(-E^T), store o;  ce = diag(c) E^T
    if constexpr (!SCAN) {
    decltype(Ops::tokens_b(f4{})) ce[NJV];
    {
      const f4 za = lds4(&Zs[c * LT + 4 * g]);
      f4 et[NJV];
#pragma unroll
      for (int jn = 0; jn < NJV; ++jn) {
        et[jn] = f4{0, 0, 0, 0};
#pragma unroll
        for (int r = 0; r < 4; ++r) et[jn] = mfma16(za[r], ft[jn][r], et[jn]);
      }
      const f4 nqa = lds4(&NQs[c * LT + 4 * g]);
      const f4 cg = lds4(&cvec[4 * g]);
#pragma unroll
      for (int jn = 0; jn < NJV; ++jn) {
#pragma unroll
        for (int r = 0; r < 4; ++r) ot[jn] = mfma16(nqa[r], et[jn][r], ot[jn]);
        ce[jn] = Ops::tokens_b(et[jn] * cg);
        if (norm_out) ot[jn] *= lds4(&rdens[4 * g]);
        if (owns(jn)) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            if (4 * g + r < len)
              io_store(oh + static_cast<unsigned>((t0 + 4 * g + r) * DV + s_row(jn) + c), ot[jn][r]);
          }
        }
      }
    }
    // ================= S^T += Alpha diag(c) E^T  (and A -= W W^T on the wave that formed Z)
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const auto aa = Ops::w_load(Ahm, Al, 16 * b + c, c, g);
#pragma unroll
      for (int jn = 0; jn < NJV; ++jn) St[jn][b] = Ops::update(aa, ce[jn], St[jn][b]);
      if (b % 2 == 1) __builtin_amdgcn_sched_barrier(0);
    }
    }  // !SCAN
    if (!DB && tn < T) load_kqu(tn);   // staged right below; not held in registers before
    if (w == sw2) update_A();
    if constexpr (DB) continue;
    stage_next();
    __syncthreads();  // (6) the next block is staged; W and Alpha no longer needed
  }

  // ---- final state (SCAN: A and the key sum after the last segment; S belongs to phase 2)
  if (!SCAN || seg == a.n_seg - 1) {
    float* AT = a.A_T ? a.A_T + static_cast<size_t>(head) * D * D : nullptr;
    float* ST = (!SCAN && a.S_T) ? a.S_T + static_cast<size_t>(head) * DV * D : nullptr;
    const int arc = (4 * g) * D + col0 + c;
    const int src = c * D + 4 * g;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      if (AT) {
#pragma unroll
        for (int jn = 0; jn < NJ; ++jn)
#pragma unroll
          for (int r = 0; r < 4; ++r) AT[arc + (16 * b + r) * D + 16 * jn] = At[jn][b][r];
      }
      if (ST) {
#pragma unroll
        for (int jn = 0; jn < NJV; ++jn)
          if (owns(jn))
            *reinterpret_cast<float4*>(ST + src + s_row(jn) * D + 16 * b) =
                make_float4(St[jn][b][0], St[jn][b][1], St[jn][b][2], St[jn][b][3]);
      }
    }
    if (a.zkey_T != nullptr && lane < SL) {
      a.zkey_T[static_cast<size_t>(head) * D + col0 + lane] = zks[col0 + lane];
    }
  }
}

template <int D, int DV, int SL, bool DB, bool SPLIT, typename IO>
hipError_t launch(const ForwardArgs& a, hipStream_t stream) {
  ForwardArgs args = a;
  void* params[] = {&args};
  const bool full = a.u != nullptr || a.refresh_period > 0;
  const void* fn = full ? reinterpret_cast<const void*>(&chunk_general_kernel<D, DV, SL, IO, true, false, DB, SPLIT>)
                        : reinterpret_cast<const void*>(&chunk_general_kernel<D, DV, SL, IO, false, false, DB, SPLIT>);
  return hipLaunchKernel(fn, dim3(a.n_heads), dim3(64 * D / SL), params, 0, stream);
}
template <int D, int DV, int SL, bool DB, bool SPLIT>
hipError_t launch_as(const ForwardArgs& a, int io_dtype, hipStream_t stream) {
  return io_dtype == 1 ? launch<D, DV, SL, DB, SPLIT, uint16_t>(a, stream) : launch<D, DV, SL, DB, SPLIT, float>(a, stream);
}
// Which calls the kernel with the A chain and the S chain on waves of their own (vla_chunk_general_pipe.hip) takes.  T = 256,
// this file's kernel (before its C x C sections by panels: 0.95 to 0.98 of the times since) / that one with waves of 16 columns (/ of
// 32), ms; bf16, every option on, unless said otherwise.  Heads of 64 up to 256 and of 32 up to 512 (d_v <= d) were on FP32 products
// there and are on split ones here: error against float64 of o 0.84 to 0.92 of what it was, of S 0.83 to 0.89, of A 0.96 to 1.0 (14 pairs of
// sizes, five sets of options; u = k^ with the feature map, 1000 tokens, A 1.6e-7 -> 2.0e-7, S 4.5e-7 -> 4.7e-7, o 6.0e-7 -> 5.6e-7).
// Heads of 128 x 16 spill (float32, u 205 registers), and win all the same: 256 heads, 64 tokens 0.0430 / 0.0409.
//   d = 128: 64 heads 0.164 / 0.114, 256 heads 0.179 / 0.128, 512 heads 0.307 / 0.238 / 0.201, 2048 heads 1.160 / 0.918 /
//            0.792; float32 256 heads 0.172 / 0.132, 2048 heads 1.253 / 0.993 / 1.006 (three-term u leaves one workgroup of
//            wide waves a compute unit); no u, 2048 heads 0.951 / 0.799 / 0.845 (registers spill)
//     d_v = 96: 2048 heads 1.149 / 0.882;  d_v = 64: 256 heads 0.178 / 0.116, 2048 heads 0.922 / 0.815, 16 tokens 0.080 / 0.084;
//     float32, u, now: 17 to 48 tokens, 2048 heads 0.120 / 0.126 and 0.171 / 0.177, 4096 heads 0.236 / 0.256 and 0.334 / 0.346, 768
//     heads, 32 tokens 0.053 / 0.049;
//     d_v = 32: 256 heads 0.178 / 0.120, 512 heads, float32 0.246 / 0.244, 2048 heads, float32 0.907 / 0.950;
//     d_v = 16: 256 heads 0.168 / 0.139, 512 heads 0.243 / 0.270
//   d =  96: 256 heads 0.147 / 0.105, 2048 heads 1.146 / 0.768, 2048 heads, 16 tokens 0.102 / 0.076; every d_v alike
//   d =  64: 256 heads 0.100 / 0.079, 512 heads 0.132 / 0.109 / 0.114, 768 heads 0.160 / 0.164 / 0.138, 2048 heads 0.408 / 0.388 /
//            0.312; float32 256 heads 0.096 / 0.080, 768 heads 0.161 / 0.174 / 0.159, 2048 heads 0.407 / 0.407 / 0.406
//     d_v = 96: 256 heads 0.118 / 0.082, 512 heads 0.154 / 0.156 / 0.128, 768 heads 0.251 / 0.233 / 0.207, 1024 heads 0.297 /
//     0.304 / 0.324;  d_v = 128 the same within 5 %;  d_v = 32: 512 heads 0.131 / 0.109, 768 heads 0.159 / 0.167 / 0.215
//   d =  32: 512 heads 0.107 / 0.078, 1024 heads 0.112 / 0.106, 2048 heads 0.217 / 0.191, 4096 heads 0.445 / 0.351
//     d_v = 64: 768 heads 0.126 / 0.104, 1024 heads, float32 0.127 / 0.152;  d_v = 128: 256 heads 0.126 / 0.070, 640 heads,
//     float32 0.152 / 0.153, 1024 heads 0.168 / 0.235;  one block, float32, u, 513 heads 0.0132 / 0.0139, 768 heads 0.0143 / 0.0149
//     (with the normalised read-out 0.0148 / 0.0159; two blocks 0.0223 / 0.0225, without u, 513 heads 0.0132 / 0.0127)
bool pipe_narrow(const ForwardArgs& a, int d, int d_v, int io_dtype) {
  switch (d) {
    case 128: {
      const int few_blocks = io_dtype == 0 && a.u != nullptr && a.n_heads > 1024 ? 48 : 16;
      return a.n_heads <= 256 || d_v >= 96 || (d_v == 64 && a.T > few_blocks);
    }
    case 96: return true;
    case 64: return a.n_heads <= 256 || (a.n_heads <= 512 && d_v <= 64);
    case 32: {
      const bool one_block = d_v == 128 && io_dtype == 0 && a.u != nullptr && a.T <= 16;
      return a.n_heads <= (one_block ? 512 : 768) || d_v <= 32;
    }
    default: return false;
  }
}
// Waves of 32 columns: half the waves per head, so twice the heads of a compute unit.
bool pipe_wide(const ForwardArgs& a, int d, int d_v, int io_dtype) {
  if (d == 128) return d_v == 128 && a.n_heads > 256 && io_dtype == 1 && a.u != nullptr;
  if (d == 64) return d_v == 64 ? a.n_heads > 512 : d_v > 64 && a.n_heads > 256 && a.n_heads <= 768;
  return false;
}

// What those leave: d = 128 with narrow value heads beyond one head per compute unit (waves of 32 columns, two workgroups per
// compute unit), small heads beyond the counts above, and d = 16 (T = 512, bf16, every option, heads of 32 on their own
// compute unit: FP32 products, double-buffered 0.175, split 0.188 ms; d = 16 keeps them).
template <int D, int DV>
hipError_t launch_io(const ForwardArgs& a, int io_dtype, hipStream_t stream) {
  if constexpr (D == 128) return launch_as<D, DV, 32, false, true>(a, io_dtype, stream);
  if constexpr (D == 16 && DV == 16) {
    if (a.n_heads <= 512) return launch_as<D, DV, 16, true, false>(a, io_dtype, stream);
  }
  return launch_as<D, DV, 16, false, (D > 16)>(a, io_dtype, stream);
}
// phase 1 of the two-phase and time-parallel modes with options: one workgroup per (head, segment)
template <int D, typename IO, bool FULL>
hipError_t launch_scan_full(const ForwardArgs& a, hipStream_t stream) {
  constexpr int SL = 16;
  const long long wgs = static_cast<long long>(a.n_heads) * a.n_seg;
  if (wgs > 0x7fffffffLL) return hipErrorInvalidValue;
  // Heads of 32 and 64: FP32 products, double-buffered, so that the 768 (d = 64) and 1024 pairs of a segment plan are
  // resident in one round.  Three-term K^ and Q in two buffers would leave two workgroups of d = 64 with u (67 KB), in
  // single ones three at the price of a longer block.  Whole calls, 16 heads, bf16, u and normalised read-out, split
  // double / split single / FP32 double, ms:
  //   d = 64, T = 4096 0.185 / 0.194 / 0.178, T = 16384 0.422 / 0.438 / 0.422, T = 131072 3.33 / 2.67 / 2.66
  //   d = 32, T = 4096 0.136 / 0.149 / 0.134, T = 16384 0.267 / 0.221 / 0.214, T = 65536 0.899 / 0.716 / 0.673
  // From d = 96 the products weigh more: split ones, double-buffered up to one pair per compute unit and, with u, beyond
  // (one workgroup either way); without u two workgroups with single buffers beyond.  T = 32768, 512 pairs, single /
  // double: d = 96 with u 1.73 / 1.69, without 1.28 / 1.51;  d = 128 2.08 / 2.02 and 1.65 / 1.86
  constexpr bool kSplit = D >= 96;
  const void* fn = reinterpret_cast<const void*>(&chunk_general_kernel<D, D, SL, IO, FULL, true, true, kSplit>);
  if constexpr (kSplit && !FULL) {
    if (wgs > 256) fn = reinterpret_cast<const void*>(&chunk_general_kernel<D, D, SL, IO, FULL, true, false, true>);
  }
  ForwardArgs args = a;
  void* params[] = {&args};
  return hipLaunchKernel(fn, dim3(static_cast<unsigned>(wgs)), dim3(64 * D / SL), params, 0, stream);
}
template <int D, typename IO>
hipError_t launch_scan(const ForwardArgs& a, hipStream_t stream) {
  return a.u != nullptr || a.refresh_period > 0 ? launch_scan_full<D, IO, true>(a, stream)
                                                : launch_scan_full<D, IO, false>(a, stream);
}

}  // namespace

hipError_t launch_chunk_general(const ForwardArgs& a, int d, int d_v, int io_dtype, hipStream_t stream) {
  if (pipe_wide(a, d, d_v, io_dtype)) return launch_chunk_general_pipe_wide(a, d, d_v, io_dtype, stream);
  if (pipe_narrow(a, d, d_v, io_dtype)) return launch_chunk_general_pipe_narrow(a, d, d_v, io_dtype, stream);
  switch (d * 1000 + d_v) {
    case 16016: return launch_io<16, 16>(a, io_dtype, stream);
    case 16032: return launch_io<16, 32>(a, io_dtype, stream);
    case 16064: return launch_io<16, 64>(a, io_dtype, stream);
    case 16096: return launch_io<16, 96>(a, io_dtype, stream);
    case 16128: return launch_io<16, 128>(a, io_dtype, stream);
    case 32064: return launch_io<32, 64>(a, io_dtype, stream);
    case 32096: return launch_io<32, 96>(a, io_dtype, stream);
    case 32128: return launch_io<32, 128>(a, io_dtype, stream);
    case 64016: return launch_io<64, 16>(a, io_dtype, stream);
    case 64032: return launch_io<64, 32>(a, io_dtype, stream);
    case 64096: return launch_io<64, 96>(a, io_dtype, stream);
    case 64128: return launch_io<64, 128>(a, io_dtype, stream);
    case 128016: return launch_io<128, 16>(a, io_dtype, stream);
    case 128032: return launch_io<128, 32>(a, io_dtype, stream);
    case 128064: return launch_io<128, 64>(a, io_dtype, stream);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_a_scan_general(const ForwardArgs& a, int d, int io_dtype, hipStream_t stream) {
  const bool bf = io_dtype == 1;
  switch (d) {
    case 32: return bf ? launch_scan<32, uint16_t>(a, stream) : launch_scan<32, float>(a, stream);
    case 64: return bf ? launch_scan<64, uint16_t>(a, stream) : launch_scan<64, float>(a, stream);
    case 96: return bf ? launch_scan<96, uint16_t>(a, stream) : launch_scan<96, float>(a, stream);
    case 128: return bf ? launch_scan<128, uint16_t>(a, stream) : launch_scan<128, float>(a, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace vla
