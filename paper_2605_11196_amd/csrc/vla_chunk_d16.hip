// The recurrence of paper Section 3.3 for key heads of 16 and few heads: the 16-token blocks of a span of 256 tokens run at
// the same time, one on each of the 16 waves of a head's workgroup.
//
// Without the identity refresh A at the start of a block is an explicit inverse, (A_0^{-1} + sum k^ k^T)^{-1} (Section 3.2,
// eq. (penalty); eq. (sm) is its Sherman-Morrison form), and at d = 16 that is one tile: every wave sums the Gram tiles of
// the blocks before its own, inverts the sum and forms K^ A, all in float64 (the k^ are the float32 numbers the recurrence
// uses, and their products are exact in float64).  K^ A has to come from the unrounded inverse: along keys seen often A k^
// is far below the elements of A, and where the recurrence keeps the two consistent step by step, an inverse rounded to
// float32 does not (four keys, 16384 tokens, lambda0 = 0.1: error of o 1.3e-2, now 5e-6; lambda0 = 1e-6, 500 tokens: 6e24, 0.2).
// From there each wave does the C x C work of its block (the algebra is at the head of vla_chunk.hip) and forms what its
// block does to S, which is affine:
//
//   S1^T = S0^T + W diag(c) E^T,  E^T = Z (V - K^ S0^T)    =>    S1^T = S0^T + P' S0^T + Q,
//   P' = -(W diag(c)) (Z K^),  Q = (W diag(c)) (Z V)
//
// One wave per 16 rows of S runs through these maps from left to right (four dependent products a block), and every wave
// reads out its own block from the S it is handed.
//
// What bounds it: the vector instructions of four waves on every SIMD (about 1300 a wave and span).  Block after block on one wave (vla_chunk.hip with one tile, which larger counts of heads keep)
// takes 3.1 us a block, all of it dependent instructions of one wave: one head of 256 tokens 50 us, 16384 tokens 3.25 ms.
// Here a span of 16 blocks takes 14 us: 16.3 us and 0.905 ms (0.925 with each half of a double broadcast by itself and
// lane indices of unknown range; 0.96 with the inverse by four pivots a step on the float64 matrix instruction, 0.94 with the Gram
// tiles read four at a time).  Error against float64 of the first
// 3.9e-7 -> 2.8e-7 (o), 2.8e-7 -> 1.6e-7 (A): every block starts from a float64 inverse.
#include "vla_mfma_util.h"

namespace vla {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

template <int LANE>
__device__ __forceinline__ double row_bcast(double x) {   // x of lane LANE of this 16-lane row
  return __builtin_amdgcn_update_dpp(0.0, x, 0x150 + LANE, 0xf, 0xf, true);
}
__device__ __forceinline__ double readlane(double x, int lane) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(u), lane);
  const uint32_t hi = __builtin_amdgcn_readlane(static_cast<int>(u >> 32), lane);
  return __builtin_bit_cast(double, static_cast<uint64_t>(hi) << 32 | lo);
}

// In-place inverse of a symmetric positive definite 16 x 16 matrix, m[r] = M[g + 4r][c] (the result layout of the float64
// matrix instruction), by Gauss-Jordan.  With 1 + 1/d in the place of the pivot d in its scaled row, every element off that
// row takes the same update m -= column * row; the pivot row is then the scaled row with 1/d itself, which the update could
// not form for a large d (as d - (d - 1)(1 + 1/d) it carries a relative error of 1e-16 d^2).
template <int P>
__device__ __forceinline__ void invert_from(d4& m, int c, int g) {
  if constexpr (P < 16) {
    const double d = readlane(m[P / 4], 16 * (P % 4) + P);
    double x = __shfl(m[P / 4], 16 * (P % 4) + c);   // M[P][c]
    double ri = __builtin_amdgcn_rcp(d);
    ri = fma(fma(-d, ri, 1.0), ri, ri);
    ri = fma(fma(-d, ri, 1.0), ri, ri);
    x = c == P ? 1.0 + ri : x * ri;
#pragma unroll
    for (int r = 0; r < 4; ++r) m[r] = fma(-row_bcast<P>(m[r]), x, m[r]);   // M[g + 4r][P]
    if (g == P % 4) m[P / 4] = c == P ? ri : x;
    invert_from<P + 1>(m, c, g);
  }
}

constexpr int NW = 16;   // waves of a head, blocks of a span

template <int DV, typename IO, bool FMAP>
__global__ void __launch_bounds__(64 * NW, 4) chunk_d16_kernel(ForwardArgs a) {
  constexpr int D = 16;
  constexpr int TV = DV / 16;
  static_assert(TV <= NW, "one wave per row tile of S");
  __shared__ __align__(16) double Gs[NW][D * D];     // Gram tile of each block
  __shared__ __align__(16) double Ms[D * D];         // inverse of A at the start of the span
  __shared__ __align__(16) float Ps[NW][D * LT];     // P' of each block
  __shared__ __align__(16) f4 Qs[NW][TV][64];        // Q of each block, then S^T at its start, in accumulator layout
  __shared__ __align__(16) float T0s[NW][C * LT], T1s[NW][C * LT];   // tiles that turn, each wave's own
  __shared__ __align__(16) float wns[NW][C];

  const int head = blockIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  int c = lane & 15;
  int g = lane >> 4;
  // offsets derived from the lane are formed anew in each part, not kept in registers
  auto fresh = [&]() __attribute__((always_inline)) { renew(c, g); };
  const int T = a.T;
  const float eps = a.eps;
  const int nblk = (T + C - 1) / C;
  float* T0 = T0s[w];
  float* T1 = T1s[w];

  const size_t slab = static_cast<size_t>(head) * static_cast<size_t>(T) * D;
  const size_t slab_v = static_cast<size_t>(head) * static_cast<size_t>(T) * DV;
  const IO* qh = static_cast<const IO*>(a.q) + slab;
  const IO* kh = static_cast<const IO*>(a.k) + slab;
  const IO* vh = static_cast<const IO*>(a.v) + slab_v;
  IO* oh = static_cast<IO*>(a.o) + slab_v;

  // S^T of the chain: X[r] = S[16 w + c][4g + r] on wave w < TV
  f4 X = f4{0, 0, 0, 0};
  if (w < TV && a.S0) {
    const float4 x = *reinterpret_cast<const float4*>(a.S0 + (static_cast<size_t>(head) * DV + 16 * w + c) * D + 4 * g);
    X = f4{x.x, x.y, x.z, x.w};
  }
  const float diag = 1.0f / a.lambda0;
  if (threadIdx.x < D * D) Ms[threadIdx.x] = threadIdx.x % (D + 1) == 0 ? 1.0 / static_cast<double>(diag) : 0.0;

  RawRow<IO, 4> kr, qr;   // token c of the block, columns 4g ..
  IO vr[TV][4];           // V[4g + r][16 jn + c]
  auto load = [&](int blk) {
    const int t0 = C * blk;
    if (t0 >= T) return;   // uniform
    const int t = t0 + c < T ? t0 + c : T - 1;   // rows past the end: the last row, replaced by zeros below
    kr.load(kh + static_cast<unsigned>(t * D + 4 * g));
    qr.load(qh + static_cast<unsigned>(t * D + 4 * g));
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int tv = t0 + 4 * g + r < T ? t0 + 4 * g + r : T - 1;
#pragma unroll
      for (int jn = 0; jn < TV; ++jn) vr[jn][r] = vh[static_cast<unsigned>(tv * DV + 16 * jn + c)];
    }
  };
  load(w);

  for (int b0 = 0; b0 < nblk; b0 += NW) {
    const int blk = b0 + w;
    const int t0 = C * blk;
    const bool live = t0 < T;   // uniform in a wave
    const int here = nblk - b0 < NW ? nblk - b0 : NW;   // blocks of this span
    f4 ka = f4{0, 0, 0, 0}, qa = f4{0, 0, 0, 0}, kt, kc, vt[TV];
    if (live) {
      float kx[4], qx[4];
      kr.unpack(kx);
      qr.unpack(qx);
      const bool row = t0 + c < T;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if constexpr (FMAP) {
          kx[r] = elu_plus_one(kx[r]);
          qx[r] = elu_plus_one(qx[r]);
        }
        ka[r] = row ? kx[r] : 0.0f;
        qa[r] = row ? qx[r] : 0.0f;
#pragma unroll
        for (int jn = 0; jn < TV; ++jn) vt[jn][r] = t0 + 4 * g + r < T ? widen(vr[jn][r]) : 0.0f;
      }
      // 1 / max(||k||, eps): hardware reciprocal square root refined by one Newton step
      float ss = 0.0f;
#pragma unroll
      for (int r = 0; r < 4; ++r) ss = fmaf(ka[r], ka[r], ss);
      ss += __shfl_xor(ss, 16);
      ss += __shfl_xor(ss, 32);
      const float sm = fmaxf(ss, eps * eps);
      float rn = __builtin_amdgcn_rsqf(sm);
      rn = rn * fmaf(-0.5f * sm * rn, rn, 1.5f);
      ka *= rn;
      *reinterpret_cast<f4*>(&T0[c * LT + 4 * g]) = ka;
      // same-wave write -> read: LDS operations of one wave are ordered
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        kt[r] = T0[(4 * g + r) * LT + c];   // K^[4g + r][c]
        kc[r] = T0[c * LT + 4 * r + g];     // K^[c][g + 4r]
      }
      d4 gram = d4{0, 0, 0, 0};
#pragma unroll
      for (int r = 0; r < 4; ++r)
        gram = __builtin_amdgcn_mfma_f64_16x16x4f64(static_cast<double>(kt[r]), static_cast<double>(kt[r]), gram, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) Gs[w][(g + 4 * r) * D + c] = gram[r];
    }
    __syncthreads();  // (1) Gram tiles visible
    fresh();

    f4 za, nqa;
    d4 m;
#pragma unroll
    for (int r = 0; r < 4; ++r) m[r] = Ms[(g + 4 * r) * D + c];
    const int before = w < here ? w : here;
    for (int i = 0; i < before; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) m[r] += Gs[i][(g + 4 * r) * D + c];
    d4 total = m;   // wave 15: after its own block
    if (w == NW - 1 && live) {
#pragma unroll
      for (int r = 0; r < 4; ++r) total[r] += Gs[w][(g + 4 * r) * D + c];
    }
    if (live) {
      // ================= A at the start of the block, m[r] = A[g + 4r][c]
      if (blk == 0) {
#pragma unroll
        for (int r = 0; r < 4; ++r) m[r] = g + 4 * r == c ? static_cast<double>(diag) : 0.0;
      } else {
        invert_from<0>(m, c, g);
      }
      f4 At = f4{0, 0, 0, 0};   // A[4g + r][c], exactly symmetric, for A after the last block
      if (blk == nblk - 1 && a.A_T) {
#pragma unroll
        for (int r = 0; r < 4; ++r) T0[(g + 4 * r) * LT + c] = static_cast<float>(m[r]);
        const f4 across = lds4(&T0[c * LT + 4 * g]);
#pragma unroll
        for (int r = 0; r < 4; ++r) At[r] = 0.5f * (T0[(4 * g + r) * LT + c] + across[r]);
      }
      fresh();
      // ================= Y^T = K^ A, Gram matrices
      f4 yt, gg = f4{0, 0, 0, 0}, gq = f4{0, 0, 0, 0};
      {
        d4 y0 = d4{0, 0, 0, 0}, y1 = d4{0, 0, 0, 0};
#pragma unroll
        for (int r = 0; r < 4; r += 2) {
          y0 = __builtin_amdgcn_mfma_f64_16x16x4f64(static_cast<double>(kc[r]), m[r], y0, 0, 0, 0);
          y1 = __builtin_amdgcn_mfma_f64_16x16x4f64(static_cast<double>(kc[r + 1]), m[r + 1], y1, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) T0[(g + 4 * r) * LT + c] = static_cast<float>(y0[r] + y1[r]);
#pragma unroll
        for (int r = 0; r < 4; ++r) yt[r] = T0[(4 * g + r) * LT + c];
      }
      const f4 y = lds4(&T0[c * LT + 4 * g]);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        gg = mfma16(ka[r], y[r], gg);   // G[s][t], GQ[s][t] with t on the rows of the accumulator
        gq = mfma16(qa[r], y[r], gq);
      }
      *reinterpret_cast<f4*>(&T1[c * LT + 4 * g]) = gq;
#pragma unroll
      for (int r = 0; r < 4; ++r) gq[r] = T1[(4 * g + r) * LT + c];   // GQ[4g + r][c]
      // ================= Cholesky of I + G and L^{-1}
      fresh();
      cholesky16(gg, T0, T1, c, g);
      fresh();
      // ================= W^T = L^{-1} Y^T, ||w_t||^2, H = L^{-1} GQ
      const f4 la = lds4(&T1[c * LT + 4 * g]);
      f4 wt = f4{0, 0, 0, 0}, hq = f4{0, 0, 0, 0};
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        wt = mfma16(la[r], yt[r], wt);
        hq = mfma16(la[r], gq[r], hq);
      }
      f4 n2 = wt * wt;
#pragma unroll
      for (int r = 0; r < 4; ++r) n2[r] = row_sum16(n2[r]);
      if (c == 0) *reinterpret_cast<f4*>(&wns[w][4 * g]) = n2;
      // ================= c_t, Z = (I + strict_lower(L) diag(c))^{-1}, NQ
      const float rdl = __builtin_amdgcn_rcpf(T0[c * LT + c]);
      const float an = __builtin_amdgcn_sqrtf(wns[w][c]) * rdl;          // ||A_t k^_t|| = ||w_t|| / L_tt
      const float cs = rdl * __builtin_amdgcn_rcpf(fmaxf(an, eps));      // alpha^_t = c_t w_t
      lower_inverse16(T0, cs, c, g, [&](int t, int s, float z) { T1[t * LT + s] = z; });
      f4 cg;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        cg[r] = __shfl(cs, 4 * g + r);
        nqa[r] = 4 * g + r <= c ? -(cg[r] * hq[r]) : 0.0f;
      }
      za = lds4(&T1[c * LT + 4 * g]);
      fresh();
      // ================= P' and Q
      f4 zk = f4{0, 0, 0, 0}, pp = f4{0, 0, 0, 0};
#pragma unroll
      for (int r = 0; r < 4; ++r) zk = mfma16(za[r], kt[r], zk);
      zk *= -cg;
#pragma unroll
      for (int r = 0; r < 4; ++r) pp = mfma16(wt[r], zk[r], pp);
#pragma unroll
      for (int r = 0; r < 4; ++r) Ps[w][(4 * g + r) * LT + c] = pp[r];
#pragma unroll
      for (int jn = 0; jn < TV; ++jn) {
        f4 zv = f4{0, 0, 0, 0}, qq = f4{0, 0, 0, 0};
#pragma unroll
        for (int r = 0; r < 4; ++r) zv = mfma16(za[r], vt[jn][r], zv);
        zv *= cg;
#pragma unroll
        for (int r = 0; r < 4; ++r) qq = mfma16(wt[r], zv[r], qq);
        Qs[w][jn][lane] = qq;
      }
      if (blk == nblk - 1 && a.A_T) {   // A1 = A - W W^T
#pragma unroll
        for (int r = 0; r < 4; ++r) At = mfma16(wt[r], -wt[r], At);
#pragma unroll
        for (int r = 0; r < 4; ++r) a.A_T[static_cast<size_t>(head) * D * D + (4 * g + r) * D + c] = At[r];
      }
    }
    __syncthreads();  // (2) maps visible; Gram tiles and Ms read
    fresh();
    if (w == NW - 1) {
#pragma unroll
      for (int r = 0; r < 4; ++r) Ms[(g + 4 * r) * D + c] = total[r];
    }
    if (b0 + NW < nblk) load(blk + NW);
    if (w < TV) {
      f4 q = Qs[0][w][lane], p = lds4(&Ps[0][c * LT + 4 * g]);
#pragma unroll
      for (int i = 0; i < NW; ++i) {
        if (i < here) {
          const int n = i + 1 < here ? i + 1 : i;
          const f4 q1 = Qs[n][w][lane], p1 = lds4(&Ps[n][c * LT + 4 * g]);
          Qs[i][w][lane] = X;
          f4 x0 = X + q, x1 = f4{0, 0, 0, 0};
          x0 = mfma16(p[0], X[0], x0);
          x1 = mfma16(p[1], X[1], x1);
          x0 = mfma16(p[2], X[2], x0);
          x1 = mfma16(p[3], X[3], x1);
          X = x0 + x1;
          q = q1;
          p = p1;
        }
      }
    }
    __syncthreads();  // (3) S at the start of every block visible
    if (live) {
      // -F^T = K^ S^T - V^T, -E^T = Z (-F^T), O^T = Q S^T + (-NQ^T)(-E^T)
#pragma unroll
      for (int jn = 0; jn < TV; ++jn) {
        const f4 s = Qs[w][jn][lane];
        f4 ft = -vt[jn], et = f4{0, 0, 0, 0}, ot = f4{0, 0, 0, 0};
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          ft = mfma16(ka[r], s[r], ft);
          ot = mfma16(qa[r], s[r], ot);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) et = mfma16(za[r], ft[r], et);
#pragma unroll
        for (int r = 0; r < 4; ++r) ot = mfma16(nqa[r], et[r], ot);
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (t0 + 4 * g + r < T) io_store(oh + static_cast<unsigned>((t0 + 4 * g + r) * DV + 16 * jn + c), ot[r]);
      }
    }
  }
  if (w < TV && a.S_T)
    *reinterpret_cast<float4*>(a.S_T + (static_cast<size_t>(head) * DV + 16 * w + c) * D + 4 * g) =
        make_float4(X[0], X[1], X[2], X[3]);
}

template <int DV>
hipError_t launch(const ForwardArgs& a, int io_dtype, hipStream_t stream) {
  ForwardArgs args = a;
  void* params[] = {&args};
  const void* fn;
  if (io_dtype == 1)
    fn = a.feature_map ? reinterpret_cast<const void*>(&chunk_d16_kernel<DV, uint16_t, true>)
                       : reinterpret_cast<const void*>(&chunk_d16_kernel<DV, uint16_t, false>);
  else
    fn = a.feature_map ? reinterpret_cast<const void*>(&chunk_d16_kernel<DV, float, true>)
                       : reinterpret_cast<const void*>(&chunk_d16_kernel<DV, float, false>);
  return hipLaunchKernel(fn, dim3(a.n_heads), dim3(64 * NW), params, 0, stream);
}

}  // namespace

hipError_t launch_chunk_d16(const ForwardArgs& a, int d_v, int io_dtype, hipStream_t stream) {
  switch (d_v) {
    case 16: return launch<16>(a, io_dtype, stream);
    case 32: return launch<32>(a, io_dtype, stream);
    case 64: return launch<64>(a, io_dtype, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace vla
