// Attention of one query per (batch, head): the class token's.  In the last encoder layer of an auxiliary network
// only the class-token row of the layer output is read (the head takes LayerNorm -> class token -> Linear), so of
// that layer's attention only the class token's query is needed, against the keys and values of all tokens.
// One workgroup per (batch, head); run-time typed (fp32 or bf16 tensors), fp32 arithmetic.
//   forward:   p = softmax_j(q . k_j / sqrt(dh)),  o = sum_j p_j v_j
//   backward:  dp_j = do . v_j,  ds_j = p_j (dp_j - sum_i p_i dp_i),  dq = sum_j ds_j k_j / sqrt(dh),
//              dk_j = ds_j q / sqrt(dh),  dv_j = p_j do
// Layouts: q, o, dq, do are [B, H*dh]; kv and dkv are [B*T, 2*H*dh] with the keys in the first H*dh columns.
//
// Keys and values are read once and what bounds this is memory, so for bf16 heads of 64 they stay in registers as they were loaded
// (attn_cls64_*): eight lanes hold a row of 64, a workgroup 32 rows a pass, all passes (up to 256 tokens) in flight at once, and LDS
// carries only sums between the waves.  The general kernels stage both as fp32 in LDS: 103 KB at 197 tokens, one workgroup a unit
// whose loads nothing covers, and a thread per row or column then walks it alone.
// Microseconds in a step, general kernel -> this one: 128 images x 197 tokens x 12 heads forward 53.9 -> 15.9 (77 MB), backward
// 67.1 -> 25.2 (155 MB), 64 x 145 x 6 8.8 -> 6.6 and 11.4 -> 7.2, 128 x 65 x 6 7.7 -> 5.8 and 10.0 -> 6.4.
#include "common.h"

namespace ppll {

namespace {
constexpr int CLS_THREADS = 256;
// K and V rows of one head staged in LDS as fp32, one padding float per row (lanes on different rows then hit
// different banks); all threads of the workgroup copy, eight independent loads in flight each
// VEC: bf16 tensors whose rows are multiples of 8 elements at 16-byte aligned addresses: one 16-byte load per 8 elements
template <bool VEC>
__device__ __forceinline__ void stage_head(const void* src, int dt, size_t first, long row_stride, int T, int dh, int tid,
                                           float* dst) {
  if (VEC) {
    const int gpr = dh >> 3, n = T * gpr;     // 16-byte granules per row, in all
    const uint16_t* p = (const uint16_t*)src + first;
#pragma unroll 4
    for (int i = tid; i < n; i += CLS_THREADS) {
      const int j = i / gpr, g = i - j * gpr;
      const uint4 w = *reinterpret_cast<const uint4*>(p + (size_t)j * row_stride + 8 * g);
      float* o = dst + j * (dh + 1) + 8 * g;
      o[0] = __uint_as_float(w.x << 16); o[1] = __uint_as_float(w.x & 0xffff0000u);
      o[2] = __uint_as_float(w.y << 16); o[3] = __uint_as_float(w.y & 0xffff0000u);
      o[4] = __uint_as_float(w.z << 16); o[5] = __uint_as_float(w.z & 0xffff0000u);
      o[6] = __uint_as_float(w.w << 16); o[7] = __uint_as_float(w.w & 0xffff0000u);
    }
    return;
  }
  const int n = T * dh;
#pragma unroll 8
  for (int i = tid; i < n; i += CLS_THREADS) {
    const int j = i / dh, d = i - j * dh;
    dst[j * (dh + 1) + d] = ld_f(src, first + (size_t)j * row_stride + d, dt);
  }
}
// sum / maximum over the workgroup through LDS (red: CLS_THREADS / 64 floats), same order for every thread
__device__ __forceinline__ float block_sum_of(float v, float* red, int tid) {   // v: the wave's sum
  __syncthreads();
  if ((tid & 63) == 0) red[tid >> 6] = v;
  __syncthreads();
  float t = 0.f;
#pragma unroll
  for (int w = 0; w < CLS_THREADS / 64; ++w) t += red[w];
  return t;
}
__device__ __forceinline__ float block_sum(float v, float* red, int tid) { return block_sum_of(wave_sum(v), red, tid); }
// sum of a b, the first exchange (lane ^ 32) taken into a multiply-add with the lane's own product
__device__ __forceinline__ float block_dot(float a, float b, float* red, int tid) {
  const uint32_t ab = __float_as_uint(a * b);
  const auto r = __builtin_amdgcn_permlane32_swap(ab, ab, false, false);
  return block_sum_of(lanes_sum<32>(fmaf(a, b, __uint_as_float((tid & 32) ? r[0] : r[1]))), red, tid);
}
__device__ __forceinline__ float block_max(float v, float* red, int tid) {
  v = wave_max(v);
  __syncthreads();
  if ((tid & 63) == 0) red[tid >> 6] = v;
  __syncthreads();
  float t = red[0];
#pragma unroll
  for (int w = 1; w < CLS_THREADS / 64; ++w) t = fmaxf(t, red[w]);
  return t;
}

// one workgroup per (batch, head): a thread per token for the scores, a thread per feature for the output
template <bool VEC>
__global__ __launch_bounds__(CLS_THREADS) void attn_cls_fwd_kernel(const void* q, const void* kv, int dt, int T, int H, int dh,
                                                                   void* out, float* prob) {
  extern __shared__ float sm[];
  float* Ks = sm;                          // [T][dh + 1]
  float* Vs = Ks + (size_t)T * (dh + 1);   // [T][dh + 1]
  float* qs = Vs + (size_t)T * (dh + 1);   // [dh]
  float* ps = qs + dh;                     // [T]
  float* red = ps + T;                     // [4]
  const int b = blockIdx.x / H, h = blockIdx.x % H, D = H * dh, tid = threadIdx.x;
  const float scale = rsqrtf((float)dh);
  const size_t k0 = (size_t)b * T * 2 * D + (size_t)h * dh;   // key row of token 0; values D further
  stage_head<VEC>(kv, dt, k0, 2L * D, T, dh, tid, Ks);
  stage_head<VEC>(kv, dt, k0 + D, 2L * D, T, dh, tid, Vs);
  for (int d = tid; d < dh; d += CLS_THREADS) qs[d] = ld_f(q, (size_t)b * D + h * dh + d, dt) * scale;
  __syncthreads();
  float sc = -INFINITY;
  if (tid < T) {
    float s = 0.f;
    for (int d = 0; d < dh; ++d) s = fmaf(qs[d], Ks[tid * (dh + 1) + d], s);
    sc = s;
  }
  const float mx = block_max(sc, red, tid);
  const float e = tid < T ? __expf(sc - mx) : 0.f;
  const float sum = block_sum(e, red, tid);
  if (tid < T) { const float p = e / sum; ps[tid] = p; prob[(size_t)blockIdx.x * T + tid] = p; }
  __syncthreads();
  for (int d = tid; d < dh; d += CLS_THREADS) {
    float o = 0.f;
    for (int j = 0; j < T; ++j) o = fmaf(ps[j], Vs[j * (dh + 1) + d], o);
    st_f(out, (size_t)b * D + h * dh + d, o, dt);
  }
}

template <bool VEC>
__global__ __launch_bounds__(CLS_THREADS) void attn_cls_bwd_kernel(const void* q, const void* kv, const float* prob,
                                                                   const void* dout, int dt, int T, int H, int dh, void* dq,
                                                                   void* dkv) {
  extern __shared__ float sm[];
  float* Ks = sm;                          // [T][dh + 1]
  float* Vs = Ks + (size_t)T * (dh + 1);   // [T][dh + 1]
  float* dos = Vs + (size_t)T * (dh + 1);  // [dh]   (the forward's qs)
  float* ps = dos + dh;                    // [T]
  float* red = ps + T;                     // [4]
  float* ds = red + 4;                     // [T]
  float* qs = ds + T;                      // [dh]  scaled query
  const int b = blockIdx.x / H, h = blockIdx.x % H, D = H * dh, tid = threadIdx.x;
  const float scale = rsqrtf((float)dh);
  const size_t k0 = (size_t)b * T * 2 * D + (size_t)h * dh;
  stage_head<VEC>(kv, dt, k0, 2L * D, T, dh, tid, Ks);
  stage_head<VEC>(kv, dt, k0 + D, 2L * D, T, dh, tid, Vs);
  for (int d = tid; d < dh; d += CLS_THREADS) {
    dos[d] = ld_f(dout, (size_t)b * D + h * dh + d, dt);
    qs[d] = ld_f(q, (size_t)b * D + h * dh + d, dt) * scale;
  }
  __syncthreads();
  float p = 0.f, dp = 0.f;
  if (tid < T) {
    for (int d = 0; d < dh; ++d) dp = fmaf(dos[d], Vs[tid * (dh + 1) + d], dp);
    p = prob[(size_t)blockIdx.x * T + tid];
  }
  const float delta = block_dot(p, dp, red, tid);
  if (tid < T) { ps[tid] = p; ds[tid] = p * (dp - delta); }
  __syncthreads();
  for (int d = tid; d < dh; d += CLS_THREADS) {
    float acc = 0.f;
    for (int j = 0; j < T; ++j) acc = fmaf(ds[j], Ks[j * (dh + 1) + d], acc);
    st_f(dq, (size_t)b * D + h * dh + d, acc * scale, dt);
  }
  if (VEC) {
    const int gpr = dh >> 3, n = T * gpr;
    uint16_t* o = (uint16_t*)dkv + k0;
#pragma unroll 2
    for (int i = tid; i < n; i += CLS_THREADS) {
      const int j = i / gpr, d = 8 * (i - j * gpr);
      const float a = ds[j], c = ps[j];
      *reinterpret_cast<uint4*>(o + (size_t)j * 2 * D + d) =
          make_uint4(f32x2_to_bf16x2(a * qs[d], a * qs[d + 1]), f32x2_to_bf16x2(a * qs[d + 2], a * qs[d + 3]),
                     f32x2_to_bf16x2(a * qs[d + 4], a * qs[d + 5]), f32x2_to_bf16x2(a * qs[d + 6], a * qs[d + 7]));
      *reinterpret_cast<uint4*>(o + (size_t)j * 2 * D + D + d) =
          make_uint4(f32x2_to_bf16x2(c * dos[d], c * dos[d + 1]), f32x2_to_bf16x2(c * dos[d + 2], c * dos[d + 3]),
                     f32x2_to_bf16x2(c * dos[d + 4], c * dos[d + 5]), f32x2_to_bf16x2(c * dos[d + 6], c * dos[d + 7]));
    }
    return;
  }
  const int n = T * dh;
  for (int i = tid; i < n; i += CLS_THREADS) {
    const int j = i / dh, d = i - j * dh;
    const size_t kj = k0 + (size_t)j * 2 * D + d;
    st_f(dkv, kj, ds[j] * qs[d], dt);
    st_f(dkv, kj + D, ps[j] * dos[d], dt);
  }
}


// ---- bf16, heads of 64, at most 256 tokens: row j of K and V at pass j / 32, wave j / 8 % 4, lanes 8 (j % 8) .. + 7
__device__ __forceinline__ void unpack8(const uint4& w, float (&v)[8]) {
  const uint32_t u[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) { v[2 * i] = __uint_as_float(u[i] << 16); v[2 * i + 1] = __uint_as_float(u[i] & 0xffff0000u); }
}
__device__ __forceinline__ uint4 scaled8(const float (&v)[8], float a) {
  return make_uint4(f32x2_to_bf16x2(a * v[0], a * v[1]), f32x2_to_bf16x2(a * v[2], a * v[3]), f32x2_to_bf16x2(a * v[4], a * v[5]),
                    f32x2_to_bf16x2(a * v[6], a * v[7]));
}
// <a, row> over the eight lanes of the row
__device__ __forceinline__ float row_dot(const float (&a)[8], const uint4& row) {
  float v[8], s = 0.f;
  unpack8(row, v);
#pragma unroll
  for (int e = 0; e < 8; ++e) s = fmaf(a[e], v[e], s);
#pragma unroll
  for (int o = 4; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  return s;
}
// sum over the eight rows of a wave of a value that the lanes of a row share
__device__ __forceinline__ float rows_sum(float v) {
#pragma unroll
  for (int o = 32; o >= 8; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
// Sums over the eight rows of a wave of the 8 columns a lane holds: a lane gives away half of what it has at each step and ends with
// the column that column_of names.
__device__ __forceinline__ int column_of(int lane) { return 8 * (lane & 7) + 4 * (lane >> 5) + 2 * ((lane >> 4) & 1) + ((lane >> 3) & 1); }
__device__ __forceinline__ float columns_sum(const float (&v)[8], int lane) {
  float a[4], b[2];
  bool up = lane & 32;
#pragma unroll
  for (int e = 0; e < 4; ++e) a[e] = (up ? v[4 + e] : v[e]) + __shfl_xor(up ? v[e] : v[4 + e], 32, 64);
  up = lane & 16;
#pragma unroll
  for (int e = 0; e < 2; ++e) b[e] = (up ? a[2 + e] : a[e]) + __shfl_xor(up ? a[e] : a[2 + e], 16, 64);
  up = lane & 8;
  return (up ? b[1] : b[0]) + __shfl_xor(up ? b[0] : b[1], 8, 64);
}
constexpr int CLS64_TOKENS = 256, CLS64_WAVES = CLS_THREADS / 64;

template <int NP>
__global__ __launch_bounds__(CLS_THREADS) void attn_cls64_fwd_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ kv, int T,
                                                                     int H, uint16_t* __restrict__ out, float* __restrict__ prob) {
  __shared__ float tops[CLS64_WAVES], sums[CLS64_WAVES], part[CLS64_WAVES][64];
  const int b = blockIdx.x / H, h = blockIdx.x % H, D = H * 64, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row0 = tid >> 3, c = 8 * (lane & 7);
  const uint16_t* base = kv + (size_t)b * T * 2 * D + h * 64 + c;
  uint4 k[NP], v[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    const int j = 32 * i + row0;
    k[i] = j < T ? *reinterpret_cast<const uint4*>(base + (size_t)j * 2 * D) : make_uint4(0, 0, 0, 0);
  }
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    const int j = 32 * i + row0;
    v[i] = j < T ? *reinterpret_cast<const uint4*>(base + (size_t)j * 2 * D + D) : make_uint4(0, 0, 0, 0);
  }
  float qv[8];
  unpack8(*reinterpret_cast<const uint4*>(q + (size_t)b * D + h * 64 + c), qv);
#pragma unroll
  for (int e = 0; e < 8; ++e) qv[e] *= 0.125f;   // 1 / sqrt(64)
  float p[NP], mx = -INFINITY;
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    p[i] = row_dot(qv, k[i]);
    if (32 * i + row0 >= T) p[i] = -INFINITY;
    mx = fmaxf(mx, p[i]);
  }
#pragma unroll
  for (int o = 32; o >= 8; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
  if (lane == 0) tops[wave] = mx;
  __syncthreads();
  mx = tops[0];
#pragma unroll
  for (int w = 1; w < CLS64_WAVES; ++w) mx = fmaxf(mx, tops[w]);
  float acc[8] = {}, sum = 0.f;
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    p[i] = 32 * i + row0 < T ? __expf(p[i] - mx) : 0.f;
    sum += p[i];
    float x[8];
    unpack8(v[i], x);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = fmaf(p[i], x[e], acc[e]);
  }
  sum = rows_sum(sum);
  if (lane == 0) sums[wave] = sum;
  part[wave][column_of(lane)] = columns_sum(acc, lane);
  __syncthreads();
  sum = 0.f;
#pragma unroll
  for (int w = 0; w < CLS64_WAVES; ++w) sum += sums[w];
  if ((lane & 7) == 0) {
#pragma unroll
    for (int i = 0; i < NP; ++i)
      if (32 * i + row0 < T) prob[(size_t)blockIdx.x * T + 32 * i + row0] = p[i] / sum;
  }
  if (wave == 0) {
    float o = 0.f;
#pragma unroll
    for (int w = 0; w < CLS64_WAVES; ++w) o += part[w][lane];
    out[(size_t)b * D + h * 64 + lane] = f32_to_bf16(o / sum);
  }
}

template <int NP>
__global__ __launch_bounds__(CLS_THREADS) void attn_cls64_bwd_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ kv,
                                                                     const float* __restrict__ prob, const uint16_t* __restrict__ dout, int T,
                                                                     int H, uint16_t* __restrict__ dq, uint16_t* __restrict__ dkv) {
  __shared__ float sums[CLS64_WAVES], part[CLS64_WAVES][64];
  const int b = blockIdx.x / H, h = blockIdx.x % H, D = H * 64, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row0 = tid >> 3, c = 8 * (lane & 7);
  const size_t first = (size_t)b * T * 2 * D + h * 64 + c, head = (size_t)b * D + h * 64;
  uint4 k[NP], v[NP];
  float p[NP], dp[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    const int j = 32 * i + row0;
    v[i] = j < T ? *reinterpret_cast<const uint4*>(kv + first + (size_t)j * 2 * D + D) : make_uint4(0, 0, 0, 0);
    p[i] = j < T ? prob[(size_t)blockIdx.x * T + j] : 0.f;
  }
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    const int j = 32 * i + row0;
    k[i] = j < T ? *reinterpret_cast<const uint4*>(kv + first + (size_t)j * 2 * D) : make_uint4(0, 0, 0, 0);
  }
  float qv[8], dov[8], delta = 0.f;
  unpack8(*reinterpret_cast<const uint4*>(q + head + c), qv);
  unpack8(*reinterpret_cast<const uint4*>(dout + head + c), dov);
#pragma unroll
  for (int e = 0; e < 8; ++e) qv[e] *= 0.125f;   // 1 / sqrt(64)
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    dp[i] = row_dot(dov, v[i]);
    delta = fmaf(p[i], dp[i], delta);
  }
  delta = rows_sum(delta);
  if (lane == 0) sums[wave] = delta;
  __syncthreads();
  delta = 0.f;
#pragma unroll
  for (int w = 0; w < CLS64_WAVES; ++w) delta += sums[w];
  float acc[8] = {};
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    const int j = 32 * i + row0;
    const float ds = p[i] * (dp[i] - delta);
    float x[8];
    unpack8(k[i], x);
    if (j < T) {
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = fmaf(ds, x[e], acc[e]);
      *reinterpret_cast<uint4*>(dkv + first + (size_t)j * 2 * D) = scaled8(qv, ds);
      *reinterpret_cast<uint4*>(dkv + first + (size_t)j * 2 * D + D) = scaled8(dov, p[i]);
    }
  }
  part[wave][column_of(lane)] = columns_sum(acc, lane);
  __syncthreads();
  if (wave == 0) {
    float o = 0.f;
#pragma unroll
    for (int w = 0; w < CLS64_WAVES; ++w) o += part[w][lane];
    dq[head + lane] = f32_to_bf16(o * 0.125f);
  }
}

// bf16, heads of 64 at 16-byte aligned addresses, all tokens that a block takes (256: 88 registers hold K, V, p and dp)
bool cls64_ok(int dt, int T, int H, int dh, const void* a, const void* b, const void* c, const void* d) {
  return dt == BF16 && dh == 64 && T >= 1 && T <= CLS64_TOKENS && H >= 1 &&
         !((((uintptr_t)a) | ((uintptr_t)b) | ((uintptr_t)c) | ((uintptr_t)d)) & 15);
}
#define CLS64_LAUNCH(KERNEL, ...)                                                                            \
  switch ((T + 31) / 32) {                                                                                   \
    case 1: hipLaunchKernelGGL(KERNEL<1>, dim3(B * H), dim3(CLS_THREADS), 0, s, __VA_ARGS__); break;         \
    case 2: hipLaunchKernelGGL(KERNEL<2>, dim3(B * H), dim3(CLS_THREADS), 0, s, __VA_ARGS__); break;         \
    case 3: hipLaunchKernelGGL(KERNEL<3>, dim3(B * H), dim3(CLS_THREADS), 0, s, __VA_ARGS__); break;         \
    case 4: hipLaunchKernelGGL(KERNEL<4>, dim3(B * H), dim3(CLS_THREADS), 0, s, __VA_ARGS__); break;         \
    case 5: hipLaunchKernelGGL(KERNEL<5>, dim3(B * H), dim3(CLS_THREADS), 0, s, __VA_ARGS__); break;         \
    case 6: hipLaunchKernelGGL(KERNEL<6>, dim3(B * H), dim3(CLS_THREADS), 0, s, __VA_ARGS__); break;         \
    case 7: hipLaunchKernelGGL(KERNEL<7>, dim3(B * H), dim3(CLS_THREADS), 0, s, __VA_ARGS__); break;         \
    default: hipLaunchKernelGGL(KERNEL<8>, dim3(B * H), dim3(CLS_THREADS), 0, s, __VA_ARGS__); break;        \
  }

bool cls_vec_ok(int dt, int H, int dh, const void* a, const void* b) {
  return dt == BF16 && !(dh & 7) && !((((uintptr_t)a) | ((uintptr_t)b)) & 15) && H >= 1;
}
constexpr int CLS_LDS = 160 * 1024;
int allow_lds(const void* fn, size_t bytes, OncePerDevice& once) {
  if (bytes > CLS_LDS) { set_error("class-token attention: %zu bytes of LDS exceed 160 KB", bytes); return PPLL_ERR_CONFIG; }
  return raise_lds(fn, CLS_LDS, once);
}
}  // namespace

size_t attention_cls_lds_bytes(int T, int dh) { return (2 * (size_t)T * (dh + 1) + 2 * (size_t)dh + 2 * (size_t)T + 4) * sizeof(float); }

int launch_attention_cls_fwd(hipStream_t s, const void* q, const void* kv, int dt, int B, int T, int H, int dh, void* out,
                             float* prob) {
  if (cls64_ok(dt, T, H, dh, q, kv, out, nullptr)) {
    CLS64_LAUNCH(attn_cls64_fwd_kernel, (const uint16_t*)q, (const uint16_t*)kv, T, H, (uint16_t*)out, prob);
    PPLL_HIP(hipGetLastError());
    return PPLL_OK;
  }
  const size_t lds = attention_cls_lds_bytes(T, dh);
  static OncePerDevice once[2];
  if (cls_vec_ok(dt, H, dh, kv, nullptr)) {
    PPLL_TRY(allow_lds((const void*)attn_cls_fwd_kernel<true>, lds, once[1]));
    hipLaunchKernelGGL(attn_cls_fwd_kernel<true>, dim3(B * H), dim3(CLS_THREADS), lds, s, q, kv, dt, T, H, dh, out, prob);
  } else {
    PPLL_TRY(allow_lds((const void*)attn_cls_fwd_kernel<false>, lds, once[0]));
    hipLaunchKernelGGL(attn_cls_fwd_kernel<false>, dim3(B * H), dim3(CLS_THREADS), lds, s, q, kv, dt, T, H, dh, out, prob);
  }
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}

int launch_attention_cls_bwd(hipStream_t s, const void* q, const void* kv, const float* prob, const void* dout, int dt, int B,
                             int T, int H, int dh, void* dq, void* dkv) {
  if (cls64_ok(dt, T, H, dh, q, kv, dout, dkv)) {
    CLS64_LAUNCH(attn_cls64_bwd_kernel, (const uint16_t*)q, (const uint16_t*)kv, prob, (const uint16_t*)dout, T, H, (uint16_t*)dq,
                 (uint16_t*)dkv);
    PPLL_HIP(hipGetLastError());
    return PPLL_OK;
  }
  const size_t lds = attention_cls_lds_bytes(T, dh);
  static OncePerDevice once[2];
  if (cls_vec_ok(dt, H, dh, kv, dkv)) {
    PPLL_TRY(allow_lds((const void*)attn_cls_bwd_kernel<true>, lds, once[1]));
    hipLaunchKernelGGL(attn_cls_bwd_kernel<true>, dim3(B * H), dim3(CLS_THREADS), lds, s, q, kv, prob, dout, dt, T, H, dh, dq, dkv);
  } else {
    PPLL_TRY(allow_lds((const void*)attn_cls_bwd_kernel<false>, lds, once[0]));
    hipLaunchKernelGGL(attn_cls_bwd_kernel<false>, dim3(B * H), dim3(CLS_THREADS), lds, s, q, kv, prob, dout, dt, T, H, dh, dq, dkv);
  }
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}

}  // namespace ppll
