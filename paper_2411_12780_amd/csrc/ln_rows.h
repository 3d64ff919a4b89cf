// Rows of a bf16 LayerNorm, forward and backward, as a group of lanes holds them: shared by the LayerNorm kernels and by the products
// that end in one, so that both give the same bits.
#pragma once
#include "common.h"

namespace ppll {
namespace {
__device__ __forceinline__ float lo_bf(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi_bf(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ uint32_t pack_bf(float a, float b) { return f32x2_to_bf16x2(a, b); }
__device__ __forceinline__ void unpack8(const uint4& w, float* v) {
  v[0] = lo_bf(w.x); v[1] = hi_bf(w.x); v[2] = lo_bf(w.y); v[3] = hi_bf(w.y);
  v[4] = lo_bf(w.z); v[5] = hi_bf(w.z); v[6] = lo_bf(w.w); v[7] = hi_bf(w.w);
}

// A row of D elements (a multiple of 64) is held by LPR lanes (8 for 64 and 192, 16 up to 384, 32 up to 768, 64 for 1024), 8
// consecutive elements (one 16-byte access) per lane and 8 LPR-column step, so a wave works on 64 / LPR rows at once and the row
// sums are exchanges inside a lane group.
template <int D_> struct LnShape {
  static constexpr int D = D_;
  static constexpr int LPR = D == 64 || D == 192 ? 8 : (D <= 384 ? 16 : (D <= 768 ? 32 : 64));
  static constexpr int NV = D / (8 * LPR);       // 16-byte pieces per lane and row
  static constexpr int RPW = 64 / LPR;           // rows per wave and pass
  static_assert(NV * 8 * LPR == D, "a row is a whole number of pieces per lane");
};
template <int LPR>
__device__ __forceinline__ float group_sum(float v) {
  if constexpr (LPR >= 16) return lanes_sum<LPR>(v);
#pragma unroll
  for (int o = LPR / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Forward: the lane's pieces of a row in, of y out
template <class S>
__device__ __forceinline__ void ln_fwd_row(const uint4 (&w)[S::NV], int lr, const float* g, const float* b, float eps, float& mu, float& rs,
                                           uint4 (&y)[S::NV]) {
  constexpr int LPR = S::LPR, NV = S::NV;
  float v[8 * NV];
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    unpack8(w[j], v + 8 * j);
#pragma unroll
    for (int e = 0; e < 8; ++e) s += v[8 * j + e];
  }
  mu = group_sum<LPR>(s) * (1.0f / S::D);
  float q = 0.f;
#pragma unroll
  for (int j = 0; j < 8 * NV; ++j) { v[j] -= mu; q += v[j] * v[j]; }
  rs = rsqrtf(group_sum<LPR>(q) * (1.0f / S::D) + eps);
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int c = 8 * lr + 8 * LPR * j;
    const float4 g0 = *reinterpret_cast<const float4*>(g + c), g1 = *reinterpret_cast<const float4*>(g + c + 4);
    const float4 b0 = *reinterpret_cast<const float4*>(b + c), b1 = *reinterpret_cast<const float4*>(b + c + 4);
    const float* t = v + 8 * j;
    y[j].x = pack_bf(t[0] * rs * g0.x + b0.x, t[1] * rs * g0.y + b0.y);
    y[j].y = pack_bf(t[2] * rs * g0.z + b0.z, t[3] * rs * g0.w + b0.w);
    y[j].z = pack_bf(t[4] * rs * g1.x + b1.x, t[5] * rs * g1.y + b1.y);
    y[j].w = pack_bf(t[6] * rs * g1.z + b1.z, t[7] * rs * g1.w + b1.w);
  }
}

// Backward.  The rows of a chunk (LNB_WAVES waves x RPW rows a pass) leave one partial row of dg and db, summed pass by pass inside a
// lane group, then across lane groups, then across waves.
constexpr int LNB_WAVES = 8;
template <int DD> constexpr int lnb_rows_per_pass() { return LNB_WAVES * LnShape<DD>::RPW; }

// The lane's pieces of x, dy and (zeros where there is none) the residual gradient in; its terms of dg and db added, of dx out.
// ROUND: dx is rounded to bf16 before the residual gradient is added.
template <class S, bool ROUND>
__device__ __forceinline__ void ln_bwd_row(const uint4 (&wx)[S::NV], const uint4 (&wd)[S::NV], const uint4 (&wr)[S::NV], bool ok, float mu, float rs,
                                           int lr, const float* g, float (&adg)[8 * S::NV], float (&adb)[8 * S::NV], uint4 (&dx)[S::NV]) {
  constexpr int LPR = S::LPR, NV = S::NV;
  float xh[8 * NV], dyh[8 * NV];
  float s1 = 0.f, s2 = 0.f;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int c = 8 * lr + 8 * LPR * j;
    const float4 g0 = *reinterpret_cast<const float4*>(g + c), g1 = *reinterpret_cast<const float4*>(g + c + 4);
    const float gg[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
    float xv[8], dv[8];
    unpack8(wx[j], xv);
    unpack8(wd[j], dv);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int i = 8 * j + e;
      xh[i] = ok ? (xv[e] - mu) * rs : 0.f;
      adg[i] += dv[e] * xh[i];
      adb[i] += dv[e];
      dyh[i] = dv[e] * gg[e];
      s1 += dyh[i];
      s2 += dyh[i] * xh[i];
    }
  }
  s1 = group_sum<LPR>(s1) * (1.0f / S::D);
  s2 = group_sum<LPR>(s2) * (1.0f / S::D);
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    float o[8], rv[8];
    unpack8(wr[j], rv);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      o[e] = rs * (dyh[8 * j + e] - s1 - xh[8 * j + e] * s2);
      if (ROUND) o[e] = bf16_to_f32(f32_to_bf16(o[e]));
      o[e] += rv[e];
    }
    dx[j] = make_uint4(pack_bf(o[0], o[1]), pack_bf(o[2], o[3]), pack_bf(o[4], o[5]), pack_bf(o[6], o[7]));
  }
}

// lane l and lane l ^ 32 (16): after the swap the sum a + b holds a's total on the lanes whose bit 5 (4) is clear and b's
// on the others: one exchange folds two values
__device__ __forceinline__ float fold32(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float fold16(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// Lane groups of a wave hold the same columns: folded (dg to the lower half of the lanes, db to the upper half, then the halves of
// each in turn) into sm[2 D], the wave's piece of LDS
template <class S>
__device__ __forceinline__ void ln_bwd_fold(const float (&adg)[8 * S::NV], const float (&adb)[8 * S::NV], int lane, float* sm) {
  constexpr int D = S::D, LPR = S::LPR, NV = S::NV;
  const int lr = lane % LPR;
  if (LPR <= 32) {
    float f[8 * NV];
#pragma unroll
    for (int i = 0; i < 8 * NV; ++i) f[i] = fold32(adg[i], adb[i]);
    if (LPR <= 16) {
#pragma unroll
      for (int i = 0; i < 4 * NV; ++i) f[i] = fold16(f[i], f[i + 4 * NV]);   // bit 4 of the lane now picks value i or i + 4 NV
      if (LPR == 8) {
#pragma unroll
        for (int i = 0; i < 4 * NV; ++i) f[i] += __shfl_xor(f[i], 8, 64);
      }
      const int half = (lane >> 4) & 1, kind = lane >> 5;
      if ((lane & 15) < LPR) {
#pragma unroll
        for (int i = 0; i < 4 * NV; ++i) {
          const int v = i + half * 4 * NV;
          sm[kind * D + 8 * lr + 8 * LPR * (v >> 3) + (v & 7)] = f[i];
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < 8 * NV; ++i) sm[(lane >> 5) * D + 8 * lr + 8 * LPR * (i >> 3) + (i & 7)] = f[i];
    }
  } else {
#pragma unroll
    for (int i = 0; i < 8 * NV; ++i) {
      const int c = 8 * lr + 8 * LPR * (i >> 3) + (i & 7);
      sm[c] = adg[i];
      sm[D + c] = adb[i];
    }
  }
}
// ... and the waves of a chunk in order, sm[LNB_WAVES][2 D], by `threads` threads
template <int D>
__device__ __forceinline__ void ln_bwd_sum(const float* sm, float* partial, int tid, int threads) {
  for (int i = tid; i < D / 2; i += threads) {   // four of the 2 D columns
    float4 t = *reinterpret_cast<const float4*>(sm + 4 * i);
#pragma unroll
    for (int w = 1; w < LNB_WAVES; ++w) {
      const float4 q = *reinterpret_cast<const float4*>(sm + w * 2 * D + 4 * i);
      t.x += q.x; t.y += q.y; t.z += q.z; t.w += q.w;
    }
    *reinterpret_cast<float4*>(partial + 4 * i) = t;
  }
}
}  // namespace
}  // namespace ppll
