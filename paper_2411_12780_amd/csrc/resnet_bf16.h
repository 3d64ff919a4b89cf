// Device pieces shared by the bf16 ResNet kernels: buffer and transposing LDS reads, half-wave sums, and the finishing of
// BatchNorm sums.
#pragma once
#include "common.h"

namespace ppll {
namespace {
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;

__device__ __forceinline__ float lo_bf(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi_bf(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ uint32_t pack2(float a, float b) { return f32x2_to_bf16x2(a, b); }
__device__ __forceinline__ int out_dim(int in, int stride) { return (in - 1) / stride + 1; }

// Raw buffer access: a load whose byte offset lies beyond the buffer returns 0, so a tap outside the image needs
// no branch, only the offset CONV_OOB (buffers here stay below 2^30 bytes, checked by the launcher).
typedef __attribute__((ext_vector_type(4))) uint32_t conv_u32x4;
constexpr int CONV_OOB = 0x7fffffff;
constexpr int CONV_OOB_BASE = 0x40000000;   // out of range after anything small is added
__device__ __forceinline__ uint4 conv_buf_load16(__amdgpu_buffer_rsrc_t r, int off) {
  const conv_u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
  return make_uint4(v.x, v.y, v.z, v.w);
}

// Transposing LDS read of 16-bit elements: lane r of a 16-lane group hands in the address of 4 elements and receives
// element r % 4 from the addresses of lanes r / 4, r / 4 + 4, r / 4 + 8, r / 4 + 12 of its group.
typedef __attribute__((ext_vector_type(4))) short conv_s16x4;
__device__ __forceinline__ uint2 conv_lds_read_tr(const char* p) {
  const conv_s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) conv_s16x4*)p);
  return __builtin_bit_cast(uint2, v);
}

// One halving step of a butterfly sum over pairs of lanes: of the N values a lane holds, it keeps one half (the upper one if
// `up`), hands the other to its partner and adds what the partner hands over.  CTRL: the DPP control that fetches from the
// partner, a lane whose `up` is the opposite one.
template <int N, int CTRL>
__device__ __forceinline__ void butterfly_halve(float* v, bool up) {
#pragma unroll
  for (int i = 0; i < N / 2; ++i) {
    const float send = up ? v[i] : v[i + N / 2], keep = up ? v[i + N / 2] : v[i];
    v[i] = keep + dpp_f<CTRL>(send);
  }
}
// Sums NV (16 or 32) per-lane values over the 32 lanes of a half-wave in a fixed order: afterwards v[0] of lane li holds
// the total of value index li >> 1 (NV = 16) or li (NV = 32).
template <int NV>
__device__ __forceinline__ void halfwave_sums(float (&v)[NV], int li) {
  static_assert(NV == 16 || NV == 32, "16 or 32 values per lane");
  // lanes 16 apart: one swap hands over two values at once
#pragma unroll
  for (int i = 0; i < NV / 2; ++i) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[i]), __float_as_uint(v[i + NV / 2]), false, false);
    v[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  butterfly_halve<NV / 2, 0x128>(v, (li & 8) != 0);   // row_ror:8: lane ^ 8
  butterfly_halve<NV / 4, 0x141>(v, (li & 4) != 0);   // row_half_mirror: lane ^ 7
  butterfly_halve<NV / 8, 0x4e>(v, (li & 2) != 0);    // quad_perm: lane ^ 2
  if constexpr (NV == 32) butterfly_halve<NV / 16, 0xb1>(v, (li & 1) != 0);   // quad_perm: lane ^ 1
  else v[0] += dpp_f<0xb1>(v[0]);
}
// Per-channel sums over rows with 8 channels per thread.  KIND 0: (sum x, sum x^2) -> mean, rstd,
// running stats.  KIND 1: (sum dyh, sum dyh*xhat), dyh = dy*(y>0) -> dbeta, dgamma.
struct BnSumArgs {
  const uint16_t* x; const uint16_t* dy; const uint16_t* y;
  int rows, C;
  const float* mean; const float* rstd;        // KIND 1 inputs
  float* partial;                              // [blocks][2][C]
  float eps, momentum;
  float* out0; float* out1;                    // KIND 0: mean, rstd; KIND 1: dbeta, dgamma
  float* run_mean; float* run_var;
};

// Channel c's sums (a, b) of x and x^2 -> mean and 1 / sqrt(var + eps); `global`: also the running statistics.
__device__ __forceinline__ void bn_statistics(const BnSumArgs& p, int c, float& a, float& b, bool global) {
  const float n = (float)p.rows, m = a / n, var = fmaxf(b / n - m * m, 0.f);
  if (global) {
    p.run_mean[c] = (1.f - p.momentum) * p.run_mean[c] + p.momentum * m;
    p.run_var[c] = (1.f - p.momentum) * p.run_var[c] + p.momentum * var * (n / (n - 1.f));
  }
  a = m;
  b = 1.0f / sqrtf(var + p.eps);
}

// Adds the workgroup partials [nblocks][2][C] in workgroup order and finishes mean / rstd / running
// statistics (KIND 0) or dbeta / dgamma (KIND 1).  One workgroup of NTHR threads.
// l0 / l1 (LDS, may be null) also receive the two results per channel; `global` says whether this
// workgroup writes them (and the running statistics) to memory.
template <int KIND, int NTHR>
__device__ __forceinline__ void bn_finish(const BnSumArgs& p, unsigned nblocks, float* red, float* l0, float* l1, bool global) {
  const int tid = threadIdx.x;
  // 2C values, four per thread (one 16-byte load per partial row); NTHR/(2C/4) thread groups take the workgroup
  // partials round-robin, eight loads in flight each, then one thread per value adds the groups in order
  // (at most 32 groups: the last stage adds them one after the other)
  const int nv = 2 * p.C, nq = nv / 4, parts = NTHR / nq < 32 ? NTHR / nq : 32;
  if (tid < nq * parts) {
    const int v4 = tid % nq, part = tid / nq;
    float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
    constexpr int U = 16;                                        // partial rows in flight per thread
    for (unsigned bk = part; bk < nblocks; bk += U * parts) {   // summed in workgroup order
      float4 q[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const unsigned bu = bk + u * parts;
        q[u] = bu < nblocks ? *reinterpret_cast<const float4*>(p.partial + (size_t)bu * nv + 4 * v4) : make_float4(0.f, 0.f, 0.f, 0.f);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) { t.x += q[u].x; t.y += q[u].y; t.z += q[u].z; t.w += q[u].w; }
    }
    *reinterpret_cast<float4*>(red + part * nv + 4 * v4) = t;
  }
  __syncthreads();
  if (tid < p.C) {
    float s0 = 0.f, s1 = 0.f;
    for (int part = 0; part < parts; ++part) { s0 += red[part * nv + tid]; s1 += red[part * nv + p.C + tid]; }
    if (KIND == 0) bn_statistics(p, tid, s0, s1, global);
    if (global) { p.out0[tid] = s0; p.out1[tid] = s1; }
    if (l0) { l0[tid] = s0; l1[tid] = s1; }
  }
}


// The normalised value in front of the residual sum and the ReLU; a = rstd * g.  Every kernel that applies a BatchNorm or
// recomputes its ReLU mask takes it from here, so that the mask is the one the forward used.
__device__ __forceinline__ float bn_value(float x, float mean, float a, float b) { return fmaf(x - mean, a, b); }
// ReLU mask of eight stored activations (none negative): bit e is element e > 0
__device__ __forceinline__ uint8_t relu_mask(const uint4& o) {
  const uint32_t w[4] = {o.x, o.y, o.z, o.w};
  uint32_t m = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) m |= ((w[j] & 0x7fffu) ? 1u << (2 * j) : 0u) | ((w[j] & 0x7fff0000u) ? 2u << (2 * j) : 0u);
  return (uint8_t)m;
}
}  // namespace
}  // namespace ppll
