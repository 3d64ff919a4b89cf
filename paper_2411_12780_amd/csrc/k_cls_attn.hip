// Attention of one query per (batch, head): the class token's.  In the last encoder layer of an auxiliary network
// only the class-token row of the layer output is read (the head takes LayerNorm -> class token -> Linear), so of
// that layer's attention only the class token's query is needed, against the keys and values of all tokens.
// One workgroup per (batch, head); run-time typed (fp32 or bf16 tensors), fp32 arithmetic.
//   forward:   p = softmax_j(q . k_j / sqrt(dh)),  o = sum_j p_j v_j
//   backward:  dp_j = do . v_j,  ds_j = p_j (dp_j - sum_i p_i dp_i),  dq = sum_j ds_j k_j / sqrt(dh),
//              dk_j = ds_j q / sqrt(dh),  dv_j = p_j do
// Layouts: q, o, dq, do are [B, H*dh]; kv and dkv are [B*T, 2*H*dh] with the keys in the first H*dh columns.
//
// What bounds this is memory: keys and values are read once.  For bf16 heads of 64 (attn_cls64_*) they lie in LDS as bf16, copied
// straight from memory, 50 KB at 197 tokens: with what the kernels declare beside them (2 and 3 KB) three forward workgroups a unit and
// two backward ones, one loading while another multiplies.  The general kernels stage both as fp32 through registers: 103 KB, one
// workgroup a unit whose loads nothing covers.  Sums run in the same order in both.
// Microseconds in a step, general kernel -> this one: 128 images x 197 tokens x 12 heads forward 53.9 -> 21.1 (77 MB), backward
// 67.1 -> 34.3 (155 MB), 64 x 145 x 6 8.8 -> 7.5 and 11.4 -> 8.2, 128 x 65 x 6 7.7 -> 6.0 and 10.0 -> 7.0.  K and V in registers, eight
// lanes a row, sum in another order and take 15.9, 25.2, 6.6, 7.2, 5.8 and 6.4: 1 % of a step at 197 tokens, for gradients that
// differ in single values by their size.
#include "common.h"
#include "gemm_pipe.h"

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


// ---- bf16, heads of 64, at most 256 tokens.  Tiles in LDS: [token][64] bf16, 128-byte rows, the 16-byte granule g of row r at
// g ^ turn(r): lanes on consecutive rows and lanes along a row both spread over all banks.
constexpr int CLS64_TOKENS = CLS_THREADS;   // a thread per token
__device__ __forceinline__ int turn(int r) { return (r >> 1) & 7; }
__host__ __device__ constexpr int cls64_tile(int T) { return (T + 7) / 8 * 1024; }
constexpr int CLS64_LDS = 2 * cls64_tile(CLS64_TOKENS);   // 64 KB, beside what the kernels declare
// K and V of a head, zeros beyond T; there after the next barrier
__device__ __forceinline__ void copy_head(const uint16_t* kv, int b, int h, int T, int D, int tid, char* k, char* v) {
  const __amdgpu_buffer_rsrc_t rs = pipe::make_rsrc(kv + (size_t)b * T * 2 * D, (uint32_t)T * 4u * (uint32_t)D);
  const int lane = tid & 63, g = lane & 7;
  for (int t = __builtin_amdgcn_readfirstlane(tid >> 6); t * 8 < T; t += CLS_THREADS / 64) {
    const int r = t * 8 + (lane >> 3), off = r * 4 * D + h * 128 + ((g ^ turn(r)) << 4);
    pipe::load_to_lds(rs, (pipe::lds_char*)k + t * 1024, r < T ? off : pipe::OOB);
    pipe::load_to_lds(rs, (pipe::lds_char*)v + t * 1024, r < T ? off + 2 * D : pipe::OOB);
  }
}
// <a, row r>, column by column
__device__ __forceinline__ float row_dot(const char* tile, int r, const float* a) {
  float s = 0.f;
#pragma unroll
  for (int g = 0; g < 8; ++g) {
    const uint4 w = *reinterpret_cast<const uint4*>(tile + r * 128 + ((g ^ turn(r)) << 4));
    const uint32_t u[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      s = fmaf(a[8 * g + 2 * e], __uint_as_float(u[e] << 16), s);
      s = fmaf(a[8 * g + 2 * e + 1], __uint_as_float(u[e] & 0xffff0000u), s);
    }
  }
  return s;
}
// sum of w_r row r at column d, row by row
__device__ __forceinline__ float column_sum(const char* tile, int d, const float* w, int T) {
  float s = 0.f;
#pragma unroll 8
  for (int r = 0; r < T; ++r)
    s = fmaf(w[r], bf16_to_f32(*reinterpret_cast<const uint16_t*>(tile + r * 128 + (((d >> 3) ^ turn(r)) << 4) + 2 * (d & 7))), s);
  return s;
}
__device__ __forceinline__ uint4 scaled8(const float* v, float a) {
  return make_uint4(f32x2_to_bf16x2(a * v[0], a * v[1]), f32x2_to_bf16x2(a * v[2], a * v[3]), f32x2_to_bf16x2(a * v[4], a * v[5]),
                    f32x2_to_bf16x2(a * v[6], a * v[7]));
}

__global__ __launch_bounds__(CLS_THREADS) void attn_cls64_fwd_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ kv, int T,
                                                                     int H, uint16_t* __restrict__ out, float* __restrict__ prob) {
  extern __shared__ __align__(1024) char tiles[];      // K, V
  __shared__ __align__(16) float qs[64], ps[CLS64_TOKENS], red[CLS_THREADS / 64];
  const int b = blockIdx.x / H, h = blockIdx.x % H, D = H * 64, tid = threadIdx.x;
  char *K = tiles, *V = tiles + cls64_tile(T);
  copy_head(kv, b, h, T, D, tid, K, V);
  if (tid < 64) qs[tid] = bf16_to_f32(q[(size_t)b * D + h * 64 + tid]) * 0.125f;   // 1 / sqrt(64)
  pipe::wait_vm<0>();
  __syncthreads();
  const float sc = tid < T ? row_dot(K, tid, qs) : -INFINITY;
  const float mx = block_max(sc, red, tid);
  const float e = tid < T ? __expf(sc - mx) : 0.f;
  const float sum = block_sum(e, red, tid);
  if (tid < T) { const float p = e / sum; ps[tid] = p; prob[(size_t)blockIdx.x * T + tid] = p; }
  __syncthreads();
  if (tid < 64) out[(size_t)b * D + h * 64 + tid] = f32_to_bf16(column_sum(V, tid, ps, T));
}

__global__ __launch_bounds__(CLS_THREADS) void attn_cls64_bwd_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ kv,
                                                                     const float* __restrict__ prob, const uint16_t* __restrict__ dout, int T,
                                                                     int H, uint16_t* __restrict__ dq, uint16_t* __restrict__ dkv) {
  extern __shared__ __align__(1024) char tiles[];      // K, V
  __shared__ __align__(16) float qs[64], dos[64], ps[CLS64_TOKENS], ds[CLS64_TOKENS], red[CLS_THREADS / 64];
  const int b = blockIdx.x / H, h = blockIdx.x % H, D = H * 64, tid = threadIdx.x;
  char *K = tiles, *V = tiles + cls64_tile(T);
  copy_head(kv, b, h, T, D, tid, K, V);
  const size_t head = (size_t)b * D + h * 64;
  if (tid < 64) { dos[tid] = bf16_to_f32(dout[head + tid]); qs[tid] = bf16_to_f32(q[head + tid]) * 0.125f; }   // 1 / sqrt(64)
  const float p = tid < T ? prob[(size_t)blockIdx.x * T + tid] : 0.f;
  pipe::wait_vm<0>();
  __syncthreads();
  const float dp = tid < T ? row_dot(V, tid, dos) : 0.f;
  const float delta = block_dot(p, dp, red, tid);
  if (tid < T) { ps[tid] = p; ds[tid] = p * (dp - delta); }
  __syncthreads();
  if (tid < 64) {              // one wave sums up dq while the others store dk and dv
    dq[head + tid] = f32_to_bf16(column_sum(K, tid, ds, T) * 0.125f);
    return;
  }
  const int c = 8 * (tid & 7);
  float qv[8], dov[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) { qv[e] = qs[c + e]; dov[e] = dos[c + e]; }
  uint16_t* o = dkv + (size_t)b * T * 2 * D + h * 64 + c;
#pragma unroll 4
  for (int j = (tid - 64) >> 3; j < T; j += (CLS_THREADS - 64) / 8) {
    *reinterpret_cast<uint4*>(o + (size_t)j * 2 * D) = scaled8(qv, ds[j]);
    *reinterpret_cast<uint4*>(o + (size_t)j * 2 * D + D) = scaled8(dov, ps[j]);
  }
}

// bf16, heads of 64 at 16-byte aligned addresses, all tokens that a block takes
bool cls64_ok(int dt, int T, int H, int dh, const void* a, const void* b) {
  return dt == BF16 && dh == 64 && T >= 1 && T <= CLS64_TOKENS && H >= 1 && (long)T * 256 * H < 0x7fffffffL &&
         !((((uintptr_t)a) | ((uintptr_t)b)) & 15);
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
  if (cls64_ok(dt, T, H, dh, kv, nullptr)) {
    static OncePerDevice once64;
    PPLL_TRY(raise_lds((const void*)attn_cls64_fwd_kernel, CLS64_LDS, once64));
    hipLaunchKernelGGL(attn_cls64_fwd_kernel, dim3(B * H), dim3(CLS_THREADS), 2 * cls64_tile(T), s, (const uint16_t*)q, (const uint16_t*)kv, T,
                       H, (uint16_t*)out, prob);
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
  if (cls64_ok(dt, T, H, dh, kv, dkv)) {
    static OncePerDevice once64;
    PPLL_TRY(raise_lds((const void*)attn_cls64_bwd_kernel, CLS64_LDS, once64));
    hipLaunchKernelGGL(attn_cls64_bwd_kernel, dim3(B * H), dim3(CLS_THREADS), 2 * cls64_tile(T), s, (const uint16_t*)q, (const uint16_t*)kv,
                       prob, (const uint16_t*)dout, T, H, (uint16_t*)dq, (uint16_t*)dkv);
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
