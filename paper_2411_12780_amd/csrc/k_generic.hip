// Straightforward kernels that serve both precisions (element type chosen at
// run time): strided GEMM with fp32 accumulation, LayerNorm, column sums,
// cross-entropy, the ViT embedding pieces, a per-(batch, head) attention and
// the optimizers.  They carry the fp32 path and every shape the MFMA kernels do
// not take.  All reductions are ordered (no float atomics), so results are
// reproducible run to run.
#include "common.h"
#include "plan.h"
#include "ln_rows.h"

namespace ppll {

// ===================================================================== GEMM
namespace {
constexpr int GT = 64;   // tile edge in M and N
constexpr int GK = 16;   // tile depth

__device__ __forceinline__ float gelu_f(float h) { return 0.5f * h * (1.0f + erff(h * 0.70710678118654752f)); }
__device__ __forceinline__ float dgelu_f(float h) {
  float cdf = 0.5f * (1.0f + erff(h * 0.70710678118654752f));
  float pdf = 0.39894228040143268f * __expf(-0.5f * h * h);
  return cdf + h * pdf;
}

__global__ __launch_bounds__(256) void gemm_generic_kernel(GemmArgs g) {
  __shared__ float As[GK][GT + 4];
  __shared__ float Bs[GK][GT + 4];
  const int tid = threadIdx.x;
  const int m0 = blockIdx.y * GT, n0 = blockIdx.x * GT;
  const int tm = (tid / 16) * 4, tn = (tid % 16) * 4;
  float acc[4][4] = {};
  for (int k0 = 0; k0 < g.K; k0 += GK) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      int idx = tid + r * 256;
      int m, k;
      if (g.a_sk == 1) { m = idx / GK; k = idx % GK; } else { k = idx / GT; m = idx % GT; }
      float v = 0.f;
      if (m0 + m < g.M && k0 + k < g.K) v = ld_f(g.A, (size_t)((long)(m0 + m) * g.a_sm + (long)(k0 + k) * g.a_sk), g.a_dt);
      As[k][m] = v;
      int n;
      if (g.b_sk == 1) { n = idx / GK; k = idx % GK; } else { k = idx / GT; n = idx % GT; }
      v = 0.f;
      if (n0 + n < g.N && k0 + k < g.K) v = ld_f(g.B, (size_t)((long)(k0 + k) * g.b_sk + (long)(n0 + n) * g.b_sn), g.b_dt);
      Bs[k][n] = v;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < GK; ++k) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) { a[i] = As[k][tm + i]; b[i] = Bs[k][tn + i]; }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    int m = m0 + tm + i;
    if (m >= g.M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int n = n0 + tn + j;
      if (n >= g.N) continue;
      float v = acc[i][j];
      if (g.bias) v += g.bias[n];
      if (g.residual) v += ld_f(g.residual, (size_t)((long)m * g.ldr + n), g.r_dt);
      size_t o = (size_t)((long)m * g.ldc + n);
      if (g.epilogue == EPI_GELU) {
        st_f(g.C, o, dgelu_f(v), g.c_dt);
        st_f(g.C2, o, gelu_f(v), g.c_dt);
      } else if (g.epilogue == EPI_DGELU) {
        st_f(g.C, o, v * ld_f(g.aux, (size_t)((long)m * g.ldaux + n), g.aux_dt), g.c_dt);
      } else {
        st_f(g.C, o, v, g.c_dt);
      }
    }
  }
}
}  // namespace

namespace {
// Few outputs (classifier head): one wave per output element, lanes stride over k.
__global__ __launch_bounds__(256) void gemm_wave_per_output_kernel(GemmArgs g) {
  const long o = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (o >= (long)g.M * g.N) return;
  const int m = (int)(o / g.N), n = (int)(o % g.N), lane = threadIdx.x & 63;
  float acc = 0.f;
  for (int k = lane; k < g.K; k += 64)
    acc = fmaf(ld_f(g.A, (size_t)((long)m * g.a_sm + (long)k * g.a_sk), g.a_dt),
               ld_f(g.B, (size_t)((long)k * g.b_sk + (long)n * g.b_sn), g.b_dt), acc);
  acc = wave_sum(acc);
  if (lane == 0) st_f(g.C, (size_t)((long)m * g.ldc + n), acc + (g.bias ? g.bias[n] : 0.f), g.c_dt);
}
// Short reductions: one thread per output element.
__global__ __launch_bounds__(256) void gemm_thread_per_output_kernel(GemmArgs g) {
  const long o = (long)blockIdx.x * 256 + threadIdx.x;
  if (o >= (long)g.M * g.N) return;
  const int m = (int)(o / g.N), n = (int)(o % g.N);
  float acc = 0.f;
  for (int k = 0; k < g.K; ++k)
    acc = fmaf(ld_f(g.A, (size_t)((long)m * g.a_sm + (long)k * g.a_sk), g.a_dt),
               ld_f(g.B, (size_t)((long)k * g.b_sk + (long)n * g.b_sn), g.b_dt), acc);
  st_f(g.C, (size_t)((long)m * g.ldc + n), acc + (g.bias ? g.bias[n] : 0.f), g.c_dt);
}
}  // namespace

int launch_gemm_generic(hipStream_t s, const GemmArgs& g) {
  if (g.M <= 0 || g.N <= 0 || g.K <= 0) { set_error("gemm: empty shape %d x %d x %d", g.M, g.N, g.K); return PPLL_ERR_SHAPE; }
  const long outputs = (long)g.M * g.N;
  if (g.epilogue == EPI_NONE && !g.residual && outputs <= 65536) {
    if (g.K <= 32) hipLaunchKernelGGL(gemm_thread_per_output_kernel, dim3((outputs + 255) / 256), dim3(256), 0, s, g);
    else if (outputs <= 16384) hipLaunchKernelGGL(gemm_wave_per_output_kernel, dim3((outputs + 3) / 4), dim3(256), 0, s, g);
    else goto tiled;
    PPLL_HIP(hipGetLastError());
    return PPLL_OK;
  }
tiled:
  dim3 grid((g.N + GT - 1) / GT, (g.M + GT - 1) / GT);
  hipLaunchKernelGGL(gemm_generic_kernel, grid, dim3(256), 0, s, g);
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}

// ===================================================================== reductions over rows
namespace {
constexpr int RED_ROWS = 64;   // rows per partial

// partial[c][n] = sum_{r in chunk c} f(x[r,n]);  mode 0: x, mode 1: (x - shift[n])^2
__global__ __launch_bounds__(256) void colsum_partial_kernel(const void* x, int dt, int rows, int N, int mode,
                                                             const float* shift, float* partial) {
  int n = blockIdx.x * 256 + threadIdx.x;
  if (n >= N) return;
  int r0 = blockIdx.y * RED_ROWS, r1 = min(rows, r0 + RED_ROWS);
  float sh = mode == 1 ? shift[n] : 0.f, acc = 0.f;
  for (int r = r0; r < r1; ++r) {
    float v = ld_f(x, (size_t)r * N + n, dt);
    if (mode == 1) { v -= sh; v *= v; }
    acc += v;
  }
  partial[(size_t)blockIdx.y * N + n] = acc;
}

// out[n] = scale * sum_c partial[c*stride + n].  A workgroup owns 16 columns; 16 thread groups
// take the chunks round-robin and are combined through LDS in a fixed order.
__global__ __launch_bounds__(256) void reduce_partials_kernel(const float* partial, int chunks, int N, long stride,
                                                              float scale, float* out) {
  __shared__ float red[16][17];
  const int col = threadIdx.x & 15, grp = threadIdx.x >> 4;
  const int n = blockIdx.x * 16 + col;
  float acc = 0.f;
  if (n < N)
    for (int c = grp; c < chunks; c += 16) acc += partial[(size_t)c * stride + n];
  red[grp][col] = acc;
  __syncthreads();
  if (grp == 0 && n < N) {
    float t = 0.f;
#pragma unroll
    for (int g = 0; g < 16; ++g) t += red[g][col];
    out[n] = t * scale;
  }
}

// the same for up to RED_BATCH reductions in one launch: workgroups first[j] .. first[j+1]-1 belong to job j.
// A job whose rows are 16-byte aligned with a length that is a multiple of 4 takes four columns per
// thread (64 columns per workgroup, 256-byte row segments); the 16 thread groups take the partial
// rows round-robin, eight loads in flight, and are added in group order.
constexpr int RED_BATCH = 40;   // the table stays below the 4 KB of a kernel's arguments
struct ReduceBatch { int n; int first[RED_BATCH + 1]; int vec4[RED_BATCH]; ReduceJob job[RED_BATCH]; };
__global__ __launch_bounds__(256) void reduce_batch_kernel(ReduceBatch a) {
  __shared__ float red[16][65];
  __shared__ float outer_red[64][4 * OUTER_MAX + 1];
  int j = 0;
  while (j + 1 < a.n && (int)blockIdx.x >= a.first[j + 1]) ++j;
  const float* partial = a.job[j].src;
  const int chunks = a.job[j].chunks, N = a.job[j].N;
  const long stride = a.job[j].stride;
  const int col = threadIdx.x & 15, grp = threadIdx.x >> 4;
  if (a.job[j].outer) {
    // four columns n and all c: a thread takes 4 n x 4 c of a row, the 64 groups of four threads take the rows round-robin,
    // four in flight, and are added in group order.  (16 n a workgroup, a thread one n and 16 c of every 16th row: a
    // load for every product, 20 us at 1024 rows; so the whole launch takes 10.)
    static_assert(OUTER_MAX == 16, "four threads of four c");
    const float* dl = a.job[j].outer;
    const int C = a.job[j].outer_n, n0 = ((int)blockIdx.x - a.first[j]) * 4, c0 = 4 * (threadIdx.x & 3), g4 = threadIdx.x >> 2;
    float acc[4][4] = {};
    constexpr int U = 4;
    for (int r0 = g4; r0 < chunks; r0 += 64 * U) {
      float z[U][4], d[U][4];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool in = r0 + 64 * u < chunks;
        const float* zp = partial + (size_t)(r0 + 64 * u) * stride;
        const float* dp = dl + (size_t)(r0 + 64 * u) * C;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          z[u][e] = in ? zp[min(n0 + e, N - 1)] : 0.f;
          d[u][e] = in ? dp[min(c0 + e, C - 1)] : 0.f;
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int c = 0; c < 4; ++c) acc[e][c] = fmaf(z[u][e], d[u][c], acc[e][c]);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int c = 0; c < 4; ++c) outer_red[g4][e * OUTER_MAX + c0 + c] = acc[e][c];
    __syncthreads();
    const int o = threadIdx.x & 63, quarter = threadIdx.x >> 6;
    float t = 0.f;
#pragma unroll
    for (int g = 0; g < 16; ++g) t += outer_red[16 * quarter + g][o];
    red[quarter][o] = t;
    __syncthreads();
    const int c = o % OUTER_MAX, m = n0 + o / OUTER_MAX;
    if (quarter == 0 && c < C && m < N)
      a.job[j].dst[(size_t)m * C + c] = (red[0][o] + red[1][o] + red[2][o] + red[3][o]) * a.job[j].scale;
    return;
  }
  if (a.vec4[j]) {
    const int n = ((int)blockIdx.x - a.first[j]) * 64 + 4 * col;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    if (n < N)
      for (int c = grp; c < chunks; c += 16 * 8) {
        float4 q[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int cu = c + 16 * u;
          q[u] = cu < chunks ? *reinterpret_cast<const float4*>(partial + (size_t)cu * stride + n) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) { acc.x += q[u].x; acc.y += q[u].y; acc.z += q[u].z; acc.w += q[u].w; }
      }
    red[grp][4 * col] = acc.x; red[grp][4 * col + 1] = acc.y; red[grp][4 * col + 2] = acc.z; red[grp][4 * col + 3] = acc.w;
    __syncthreads();
    if (threadIdx.x < 64) {
      const int m = ((int)blockIdx.x - a.first[j]) * 64 + threadIdx.x;
      if (m < N) {
        float t = 0.f;
#pragma unroll
        for (int g = 0; g < 16; ++g) t += red[g][threadIdx.x];
        a.job[j].dst[m] = t * a.job[j].scale;
      }
    }
    return;
  }
  const int n = ((int)blockIdx.x - a.first[j]) * 16 + col;
  float acc = 0.f;
  if (n < N)
    for (int c = grp; c < chunks; c += 16 * 8) {
      float q[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) q[u] = c + 16 * u < chunks ? partial[(size_t)(c + 16 * u) * stride + n] : 0.f;
#pragma unroll
      for (int u = 0; u < 8; ++u) acc += q[u];
    }
  red[grp][col] = acc;
  __syncthreads();
  if (grp == 0 && n < N) {
    float t = 0.f;
#pragma unroll
    for (int g = 0; g < 16; ++g) t += red[g][col];
    a.job[j].dst[n] = t * a.job[j].scale;
  }
}
}  // namespace

float* ReduceQueue::space(size_t floats, bool* queued) {
  const size_t need = (floats + 63) & ~(size_t)63;
  if (arena && used + need <= arena_floats) {
    float* p = arena + used;
    used += need;
    *queued = true;
    return p;
  }
  *queued = false;
  return scratch;
}

int ReduceQueue::reduce(hipStream_t s, bool queued, const float* src, int chunks, int N, long stride, float scale,
                        float* out) {
  if (!queued) return reduce_partials(s, src, chunks, N, stride, scale, out);
  jobs.push_back(ReduceJob{src, out, chunks, N, stride, scale, nullptr, 0});
  return PPLL_OK;
}

int ReduceQueue::reduce_outer(hipStream_t s, bool queued, const float* src, int rows, int N, const float* outer, int outer_n, float* out) {
  const ReduceJob job{src, out, rows, N, N, 1.0f, outer, outer_n};
  if (queued) { jobs.push_back(job); return PPLL_OK; }
  ReduceBatch b{};
  b.n = 1; b.job[0] = job; b.first[1] = (N + 3) / 4;
  hipLaunchKernelGGL(reduce_batch_kernel, dim3(b.first[1]), dim3(256), 0, s, b);
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}

int ReduceQueue::flush(hipStream_t s) {
  for (size_t j0 = 0; j0 < jobs.size(); j0 += RED_BATCH) {
    ReduceBatch b{};
    b.n = (int)(jobs.size() - j0 < (size_t)RED_BATCH ? jobs.size() - j0 : (size_t)RED_BATCH);
    int blocks = 0;
    for (int j = 0; j < b.n; ++j) {
      b.job[j] = jobs[j0 + j];
      b.first[j] = blocks;
      const ReduceJob& q = b.job[j];
      b.vec4[j] = !q.outer && q.N >= 64 && (q.N % 4) == 0 && (q.stride % 4) == 0 && !(((uintptr_t)q.src) & 15);
      blocks += q.outer ? (q.N + 3) / 4 : b.vec4[j] ? (q.N + 63) / 64 : (q.N + 15) / 16;
    }
    b.first[b.n] = blocks;
    if (blocks > 0) {
      hipLaunchKernelGGL(reduce_batch_kernel, dim3(blocks), dim3(256), 0, s, b);
      PPLL_HIP(hipGetLastError());
    }
  }
  jobs.clear();
  return PPLL_OK;
}

int reduce_partials(hipStream_t s, const float* partial, int chunks, int N, long stride, float scale, float* out) {
  hipLaunchKernelGGL(reduce_partials_kernel, dim3((N + 15) / 16), dim3(256), 0, s, partial, chunks, N, stride, scale,
                     out);
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}

int colsum_partial_floats(int rows, int N) { return ((rows + RED_ROWS - 1) / RED_ROWS) * N; }

int colsum_mode(hipStream_t s, const void* x, int dt, int rows, int N, int mode, const float* shift, float scale,
                ReduceQueue& rq, float* out) {
  int chunks = (rows + RED_ROWS - 1) / RED_ROWS;
  bool queued;
  float* partials = rq.space((size_t)chunks * N, &queued);
  hipLaunchKernelGGL(colsum_partial_kernel, dim3((N + 255) / 256, chunks), dim3(256), 0, s, x, dt, rows, N, mode,
                     shift, partials);
  PPLL_HIP(hipGetLastError());
  return rq.reduce(s, queued, partials, chunks, N, N, scale, out);
}

int launch_colsum(hipStream_t s, const void* x, int dt, int rows, int N, ReduceQueue& rq, float* out) {
  return colsum_mode(s, x, dt, rows, N, 0, nullptr, 1.0f, rq, out);
}

// ===================================================================== LayerNorm
namespace {
constexpr int LN_ROWS = 8;    // rows per workgroup in the run-time-typed backward (4 waves x 2: a row is a latency chain)

__global__ __launch_bounds__(256) void layernorm_fwd_kernel(const void* x, int dt, long xs, int rows, int D,
                                                            const float* g, const float* b, float eps, void* y,
                                                            float* mean, float* rstd) {
  int row = blockIdx.x * 4 + threadIdx.x / 64, lane = threadIdx.x % 64;
  if (row >= rows) return;
  size_t base = (size_t)row * xs;
  float s = 0.f;
  for (int d = lane; d < D; d += 64) s += ld_f(x, base + d, dt);
  float mu = wave_sum(s) / D;
  float q = 0.f;
  for (int d = lane; d < D; d += 64) { float c = ld_f(x, base + d, dt) - mu; q += c * c; }
  float rs = rsqrtf(wave_sum(q) / D + eps);
  for (int d = lane; d < D; d += 64)
    st_f(y, (size_t)row * D + d, (ld_f(x, base + d, dt) - mu) * rs * g[d] + b[d], dt);
  if (lane == 0) { mean[row] = mu; rstd[row] = rs; }
}

// One wave per row.  dx = dres + rstd * (dyh - mean(dyh) - xhat * mean(dyh*xhat)), dyh = dy*g.
// Each workgroup owns LN_ROWS consecutive rows and emits one partial of dg and db.
__global__ __launch_bounds__(256) void layernorm_bwd_kernel(const void* dy, const void* x, int dt, long xs, int rows,
                                                            int D, const float* g, const float* mean,
                                                            const float* rstd, const void* dres, int dres_every, void* dx,
                                                            float* partial) {
  extern __shared__ float sm[];          // [4][2][D]
  int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  float* my_dg = sm + (size_t)wave * 2 * D;
  float* my_db = my_dg + D;
  for (int d = lane; d < D; d += 64) { my_dg[d] = 0.f; my_db[d] = 0.f; }
  int r0 = blockIdx.x * LN_ROWS;
  for (int rr = wave; rr < LN_ROWS; rr += 4) {
    int row = r0 + rr;
    if (row >= rows) break;
    float mu = mean[row], rs = rstd[row];
    size_t xb = (size_t)row * xs, yb = (size_t)row * D;
    float s1 = 0.f, s2 = 0.f;
    for (int d = lane; d < D; d += 64) {
      float xh = (ld_f(x, xb + d, dt) - mu) * rs;
      float dyv = ld_f(dy, yb + d, dt);
      float dyh = dyv * g[d];
      s1 += dyh; s2 += dyh * xh;
      my_dg[d] += dyv * xh; my_db[d] += dyv;
    }
    s1 = wave_sum(s1) / D; s2 = wave_sum(s2) / D;
    if (dx) {
      for (int d = lane; d < D; d += 64) {
        float xh = (ld_f(x, xb + d, dt) - mu) * rs;
        float dyh = ld_f(dy, yb + d, dt) * g[d];
        float v = rs * (dyh - s1 - xh * s2);
        if (dres_every > 1 && dt == BF16) v = bf16_to_f32(f32_to_bf16(v));
        if (dres && row % dres_every == 0) v += ld_f(dres, (size_t)(row / dres_every) * D + d, dt);
        st_f(dx, yb + d, v, dt);
      }
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < 2 * D; i += 256)
    partial[(size_t)blockIdx.x * 2 * D + i] = sm[i] + sm[2 * D + i] + sm[4 * D + i] + sm[6 * D + i];
}
}  // namespace

// ---- bf16 fast path: the row in registers, one pass (ln_rows.h)
namespace {
template <int DD>
__global__ __launch_bounds__(256) void layernorm_fwd_bf16_kernel(const uint16_t* x, long xs, int rows,
                                                                 const float* g, const float* b, float eps,
                                                                 uint16_t* y, float* mean, float* rstd) {
  using S = LnShape<DD>;
  constexpr int D = S::D, LPR = S::LPR, NV = S::NV, RPW = S::RPW;
  const int lane = threadIdx.x & 63, lr = lane % LPR;
  const int row = (blockIdx.x * 4 + (threadIdx.x >> 6)) * RPW + lane / LPR;
  const bool ok = row < rows;
  uint4 w[NV], o[NV];
#pragma unroll
  for (int j = 0; j < NV; ++j) w[j] = make_uint4(0, 0, 0, 0);
  if (ok)
#pragma unroll
    for (int j = 0; j < NV; ++j) w[j] = *reinterpret_cast<const uint4*>(x + (size_t)row * xs + 8 * lr + 8 * LPR * j);
  float mu, rs;
  ln_fwd_row<S>(w, lr, g, b, eps, mu, rs, o);
  if (!ok) return;
#pragma unroll
  for (int j = 0; j < NV; ++j) *reinterpret_cast<uint4*>(y + (size_t)row * D + 8 * lr + 8 * LPR * j) = o[j];
  if (lr == 0) { mean[row] = mu; rstd[row] = rs; }
}

// Backward.  What bounds it at training sizes (8320 rows of width 384: 26 MB, 3.6 us at the rate the last-level cache
// delivers) is the latency of one row's chain - loads, two row sums, the write - so the rows are spread over as many waves
// as there are: eight waves per workgroup, one pass over 64 / LPR rows each up to just under 1024 workgroups (four per unit on
// 256 units), 512 to 1024 workgroups of more passes beyond (each leaves one partial row of dg, db, which a later kernel adds up).
// dres_every: rows r with r % dres_every == 0 take row r / dres_every of dres, the others none (1: every row its own)
template <int DD, bool ONE, bool SPARSE>
__global__ __launch_bounds__(64 * LNB_WAVES, 2) void layernorm_bwd_bf16_kernel(const uint16_t* dy, const uint16_t* x, long xs,
                                                                 int rows, const float* g, const float* mean,
                                                                 const float* rstd, const uint16_t* dres, int dres_every,
                                                                 uint16_t* dx, float* partial, int passes) {
  using S = LnShape<DD>;
  constexpr int D = S::D, LPR = S::LPR, NV = S::NV, RPW = S::RPW;
  __shared__ __align__(16) float sm[LNB_WAVES][2 * D];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, lr = lane % LPR, sub = lane / LPR;
  float adg[8 * NV], adb[8 * NV];
#pragma unroll
  for (int j = 0; j < 8 * NV; ++j) { adg[j] = 0.f; adb[j] = 0.f; }
  const int r0 = blockIdx.x * (ONE ? 1 : passes) * (LNB_WAVES * RPW);
  for (int pass = 0; pass < (ONE ? 1 : passes); ++pass) {
    const int row = r0 + pass * (LNB_WAVES * RPW) + wave * RPW + sub;
    const bool ok = row < rows;
    uint4 wx[NV], wd[NV], wr[NV], o[NV];
    long rrow = row;
    bool has_res = dres != nullptr && ok;
    if (SPARSE) { rrow = row / dres_every; has_res = has_res && row % dres_every == 0; }
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const int c = 8 * lr + 8 * LPR * j;
      wx[j] = wd[j] = wr[j] = make_uint4(0, 0, 0, 0);
      if (ok) {
        wx[j] = *reinterpret_cast<const uint4*>(x + (size_t)row * xs + c);
        wd[j] = *reinterpret_cast<const uint4*>(dy + (size_t)row * D + c);
      }
      if (has_res) wr[j] = *reinterpret_cast<const uint4*>(dres + (size_t)rrow * D + c);
    }
    const float mu = ok ? mean[row] : 0.f, rs = ok ? rstd[row] : 0.f;
    // a compact dres is added to the stored gradient: rounded to the activation type before and after
    ln_bwd_row<S, SPARSE>(wx, wd, wr, ok, mu, rs, lr, g, adg, adb, o);
    if (dx && ok)
#pragma unroll
      for (int j = 0; j < NV; ++j) *reinterpret_cast<uint4*>(dx + (size_t)row * D + 8 * lr + 8 * LPR * j) = o[j];
  }
  ln_bwd_fold<S>(adg, adb, lane, sm[wave]);
  __syncthreads();
  ln_bwd_sum<D>(&sm[0][0], partial + (size_t)blockIdx.x * 2 * D, threadIdx.x, 64 * LNB_WAVES);
}

bool ln_fast_dim(int D) {
  return D == 64 || D == 128 || D == 192 || D == 256 || D == 384 || D == 512 || D == 768 || D == 1024;
}
bool ln_fast_ok(int dt, int D, long xs, const void* a, const void* b, const void* c, const void* d) {
  if (dt != BF16 || (xs & 1)) return false;
  if (!ln_fast_dim(D)) return false;
  return !(xs & 7) && !((((uintptr_t)a) | ((uintptr_t)b) | ((uintptr_t)c) | ((uintptr_t)d)) & 15);
}
}  // namespace

#define LN_DISPATCH(D_EXPR, CALL)                      \
  switch (D_EXPR) {                                    \
    case 64: { constexpr int DD = 64; CALL; break; }   \
    case 128: { constexpr int DD = 128; CALL; break; } \
    case 192: { constexpr int DD = 192; CALL; break; } \
    case 256: { constexpr int DD = 256; CALL; break; } \
    case 384: { constexpr int DD = 384; CALL; break; } \
    case 512: { constexpr int DD = 512; CALL; break; } \
    case 768: { constexpr int DD = 768; CALL; break; } \
    default: { constexpr int DD = 1024; CALL; break; } \
  }

int launch_layernorm_fwd(hipStream_t s, const void* x, int dt, long xs, int rows, int D, const float* g,
                         const float* b, float eps, void* y, float* mean, float* rstd) {
  if (ln_fast_ok(dt, D, xs, x, y, g, b)) {
    LN_DISPATCH(D, hipLaunchKernelGGL((layernorm_fwd_bf16_kernel<DD>),
                                      dim3((rows + 4 * LnShape<DD>::RPW - 1) / (4 * LnShape<DD>::RPW)), dim3(256), 0, s,
                                      (const uint16_t*)x, xs, rows, g, b, eps, (uint16_t*)y, mean, rstd));
  } else {
    hipLaunchKernelGGL(layernorm_fwd_kernel, dim3((rows + 3) / 4), dim3(256), 0, s, x, dt, xs, rows, D, g, b, eps, y,
                       mean, rstd);
  }
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}

// rows per pass of a workgroup of the fast backward, and its passes at a given row count (see the kernel)
static int lnb_pass_rows(int D) {
  int v = 1;
  LN_DISPATCH(D, v = lnb_rows_per_pass<DD>());
  return v;
}
static int lnb_passes(int rows, int D) {
  const int p = rows / (lnb_pass_rows(D) * 512);
  return p < 1 ? 1 : p;
}
int layernorm_bwd_rows(int rows, int D) { return lnb_pass_rows(D) * lnb_passes(rows, D); }
static size_t ln_floats(int rows, int D, int per) { return (size_t)((rows + per - 1) / per) * 2 * D; }
size_t layernorm_bwd_partial_floats(int rows, int D, int dt) {
  return ln_floats(rows, D, dt == BF16 && ln_fast_dim(D) ? layernorm_bwd_rows(rows, D) : LN_ROWS);
}
size_t layernorm_bwd_most_floats(int rows, int D, int dt) {
  const size_t usual = layernorm_bwd_partial_floats(rows, D, dt), stand_in = ln_floats(rows, D, LN_ROWS);
  return usual > stand_in ? usual : stand_in;
}

int launch_layernorm_bwd(hipStream_t s, const void* dy, const void* x, int dt, long xs, int rows, int D,
                         const float* g, const float* mean, const float* rstd, const void* dres, int dres_every,
                         void* dx_out, ReduceQueue& rq, float* dg, float* db) {
  int chunks;
  const bool fast = ln_fast_ok(dt, D, xs, x, dy, dres, dx_out) && !(((uintptr_t)g) & 15);
  bool queued;
  float* partials = rq.space(fast ? layernorm_bwd_partial_floats(rows, D, dt) : ln_floats(rows, D, LN_ROWS), &queued);
  if (fast) {
    const int passes = lnb_passes(rows, D), per = layernorm_bwd_rows(rows, D);
    chunks = (rows + per - 1) / per;
#define LNB_LAUNCH(ONE, SPARSE)                                                                                            \
  LN_DISPATCH(D, hipLaunchKernelGGL((layernorm_bwd_bf16_kernel<DD, ONE, SPARSE>), dim3(chunks), dim3(64 * LNB_WAVES), 0, s, \
                                    (const uint16_t*)dy, (const uint16_t*)x, xs, rows, g, mean, rstd,                      \
                                    (const uint16_t*)dres, dres_every, (uint16_t*)dx_out, partials, passes))
    if (dres_every > 1) { LNB_LAUNCH(false, true); }   // one layer of a step
    else if (passes == 1) { LNB_LAUNCH(true, false); }
    else { LNB_LAUNCH(false, false); }
#undef LNB_LAUNCH
  } else {
    chunks = (rows + LN_ROWS - 1) / LN_ROWS;
    size_t lds = (size_t)8 * D * sizeof(float);
    if (lds > 48 * 1024) { set_error("layernorm_bwd: dim %d too large", D); return PPLL_ERR_CONFIG; }
    hipLaunchKernelGGL(layernorm_bwd_kernel, dim3(chunks), dim3(256), lds, s, dy, x, dt, xs, rows, D, g, mean, rstd,
                       dres, dres_every, dx_out, partials);
  }
  PPLL_HIP(hipGetLastError());
  return layernorm_bwd_reduce(s, rq, queued, partials, chunks, D, dg, db);
}

int layernorm_bwd_reduce(hipStream_t s, ReduceQueue& rq, bool queued, const float* partials, int chunks, int D, float* dg, float* db) {
  // each partial row is [dg | db]; the two gradients are neighbours in the parameter table
  if (db == dg + D) return rq.reduce(s, queued, partials, chunks, 2 * D, 2L * D, 1.0f, dg);
  PPLL_TRY(rq.reduce(s, queued, partials, chunks, D, 2L * D, 1.0f, dg));
  return rq.reduce(s, queued, partials + D, chunks, D, 2L * D, 1.0f, db);
}

// ===================================================================== cross-entropy
namespace {
constexpr size_t CE_LDS_FLOATS = 12288;   // 48 KiB: batch 1024 x 10 classes fits
// One workgroup: mean loss (also copied to loss2 when given), dlogits, and the head's bias gradient
// db[c] = sum over the batch of dlogits[b][c], added in batch order.
__global__ __launch_bounds__(256) void cross_entropy_kernel(const float* logits, const int32_t* labels, int B, int C,
                                                            float* loss, float* loss2, float* dlogits, float* dbias,
                                                            int* flag) {
  __shared__ float red[256];
  extern __shared__ float dl[];             // a copy of dlogits when the launcher gave it room (CE_LDS_FLOATS)
  const bool in_lds = (size_t)B * C <= CE_LDS_FLOATS;
  float acc = 0.f;
  for (int b = threadIdx.x; b < B; b += 256) {
    const float* z = logits + (size_t)b * C;
    float mx = z[0];
    for (int c = 1; c < C; ++c) mx = fmaxf(mx, z[c]);
    float se = 0.f;
    for (int c = 0; c < C; ++c) se += expf(z[c] - mx);
    float lse = mx + logf(se);
    int y = labels[b];
    bool ok = y >= 0 && y < C;
    if (!ok) *flag = 1;
    for (int c = 0; c < C; ++c) {
      const float d = (expf(z[c] - lse) - ((ok && c == y) ? 1.f : 0.f)) / B;
      dlogits[(size_t)b * C + c] = d;
      if (in_lds) dl[b * C + c] = d;
    }
    if (ok) acc += lse - z[y];
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    *loss = red[0] / B;
    if (loss2) *loss2 = red[0] / B;
  }
  if (dbias) {   // dlogits were written by this workgroup before the barriers above
    // 256 / C thread groups take the batch rows round-robin, then one thread per class adds the groups in order
    const int parts = C <= 256 ? 256 / C : 1;
    __syncthreads();   // red is reused
    if (C <= 256) {
      const int c = threadIdx.x % C, part = threadIdx.x / C;
      float t = 0.f;
      if (part < parts)
        for (int b = part; b < B; b += parts) t += in_lds ? dl[b * C + c] : dlogits[(size_t)b * C + c];
      red[threadIdx.x] = t;
      __syncthreads();
      if (threadIdx.x < C) {
        float u = 0.f;
        for (int k = 0; k < parts; ++k) u += red[k * C + threadIdx.x];
        dbias[threadIdx.x] = u;
      }
    } else {
      for (int c = threadIdx.x; c < C; c += 256) {
        float t = 0.f;
        for (int b = 0; b < B; b += 8) {    // eight loads in flight, added in batch order
          float q[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) q[u] = b + u < B ? (in_lds ? dl[(b + u) * C + c] : dlogits[(size_t)(b + u) * C + c]) : 0.f;
#pragma unroll
          for (int u = 0; u < 8; ++u) t += q[u];
        }
        dbias[c] = t;
      }
    }
  }
}
}  // namespace

int launch_cross_entropy(hipStream_t s, const float* logits, const int32_t* labels, int B, int C, float* loss,
                         float* loss2, float* dlogits, float* dbias, int* flag) {
  const size_t lds = (size_t)B * C <= CE_LDS_FLOATS ? (size_t)B * C * sizeof(float) : 0;
  hipLaunchKernelGGL(cross_entropy_kernel, dim3(1), dim3(256), lds, s, logits, labels, B, C, loss, loss2, dlogits, dbias,
                     flag);
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}

// ===================================================================== auxiliary head, fused
namespace {
// LayerNorm of the class token, Linear to the classes, mean softmax cross-entropy, and everything
// back to the gradient of the class token, for 4 batch rows per workgroup (one wave each).  Without
// LayerNorm parameters (ln_g null) the rows go to the Linear layer as they are: the ResNet head on
// the pooled features.  Values
// that the unfused kernels keep in the activation type (z = LN output, dz) are rounded to it here as
// well.  What has to be summed over the batch (loss, head weight / bias gradient, LayerNorm scale /
// shift gradient) leaves as one partial row per workgroup: [D*C | C | D | D | 1] floats.
constexpr int HEAD_ROWS = 4, HEAD_THREADS = 64 * HEAD_ROWS;   // 1 and 2 rows per workgroup measured slower (more partial rows)
__device__ __forceinline__ float round_to(float v, int dt) { return dt == BF16 ? bf16_to_f32(f32_to_bf16(v)) : v; }
__global__ __launch_bounds__(HEAD_THREADS) void vit_head_kernel(const void* x, int dt, long xs, int B, int D, int C,
                                                       const float* ln_g, const float* ln_b, float eps,
                                                       const float* W, const float* bias, const int32_t* labels,
                                                       void* dcls, float* partial, int* flag, int w_in_lds) {
  extern __shared__ float sm[];
  float* xh = sm;                               // [4][D] normalised input
  float* zs = xh + HEAD_ROWS * D;               // [4][D] LayerNorm output
  float* dzs = zs + HEAD_ROWS * D;              // [4][D] gradient at the LayerNorm output
  float* dl = dzs + HEAD_ROWS * D;              // [4][C] logits, then dlogits
  float* lossw = dl + HEAD_ROWS * C;            // [4]
  // Everything that is read once per class or per column inside the dependent chains below comes from LDS: a global
  // load in such a chain (the bias of class c behind the c-th dot product, the LayerNorm scale behind a column of
  // dz) stalls its wave for a full memory latency each time (measured: 24.9 -> 21.3 us at 128 rows of width 384).
  const bool ln = ln_g != nullptr;
  float* bs = lossw + HEAD_ROWS;                // [C] head bias
  float* lng = bs + C;                          // [D] LayerNorm scale, [D] shift (unused without LayerNorm)
  float* lnb = lng + D;
  // copies with eight loads in flight per thread
  auto stage_in = [&](float* dst, const float* src, int n) {
    for (int i0 = threadIdx.x; i0 < n; i0 += 8 * HEAD_THREADS) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) { const int i = i0 + u * HEAD_THREADS; v[u] = i < n ? src[i] : 0.f; }
#pragma unroll
      for (int u = 0; u < 8; ++u) { const int i = i0 + u * HEAD_THREADS; if (i < n) dst[i] = v[u]; }
    }
  };
  stage_in(bs, bias, C);
  if (ln) { stage_in(lng, ln_g, D); stage_in(lnb, ln_b, D); }
  // the head weight, read 2 C times per row, comes from LDS when there is room for it
  if (w_in_lds) {
    float* wl = lnb + D;
    stage_in(wl, W, D * C);
    W = wl;
  }
  __syncthreads();
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int b = blockIdx.x * HEAD_ROWS + wave;
  const bool live = b < B;
  const int y = live ? labels[b] : 0;           // asked for early, used after the logits
  float* xr = xh + wave * D; float* zr = zs + wave * D; float* dzr = dzs + wave * D; float* lr = dl + wave * C;
  float rs = 0.f;
  if (live) {
    const size_t base = (size_t)b * xs;
    // the row comes in with up to eight loads in flight per lane
    for (int d0 = lane; d0 < D; d0 += 8 * 64) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) { const int d = d0 + 64 * u; v[u] = d < D ? ld_f(x, base + d, dt) : 0.f; }
#pragma unroll
      for (int u = 0; u < 8; ++u) { const int d = d0 + 64 * u; if (d < D) xr[d] = v[u]; }
    }
    if (ln) {
      float s = 0.f;
      for (int d = lane; d < D; d += 64) s += xr[d];
      const float mu = wave_sum(s) / D;
      float q = 0.f;
      for (int d = lane; d < D; d += 64) { const float c = xr[d] - mu; q += c * c; }
      rs = rsqrtf(wave_sum(q) / D + eps);
      for (int d = lane; d < D; d += 64) {
        const float h = (xr[d] - mu) * rs;
        xr[d] = h;
        zr[d] = round_to(h * lng[d] + lnb[d], dt);
      }
    } else {
      for (int d = lane; d < D; d += 64) { zr[d] = xr[d]; xr[d] = 0.f; }
    }
    wave_sync();
    // five classes per pass over the row: a wave alone on its SIMD has nothing to hide an LDS read behind, so the
    // reads of a pass are independent of each other and the five sums are exchanged side by side
    for (int c0 = 0; c0 < C; c0 += 5) {
      float a[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
      for (int d = lane; d < D; d += 64) {
        const float zv = zr[d];
        const float* wr = W + d * C + c0;
#pragma unroll
        for (int u = 0; u < 5; ++u) a[u] += zv * (c0 + u < C ? wr[u] : 0.f);
      }
#pragma unroll
      for (int u = 0; u < 5; ++u) a[u] = wave_sum(a[u]);
      if (lane == 0) {
#pragma unroll
        for (int u = 0; u < 5; ++u) if (c0 + u < C) lr[c0 + u] = a[u] + bs[c0 + u];
      }
    }
    wave_sync();
    float mx = -INFINITY;
    for (int c = lane; c < C; c += 64) mx = fmaxf(mx, lr[c]);
    mx = wave_max(mx);
    float se = 0.f;
    for (int c = lane; c < C; c += 64) se += expf(lr[c] - mx);
    const float lse = mx + logf(wave_sum(se));
    const bool ok = y >= 0 && y < C;
    if (!ok && lane == 0) *flag = 1;
    const float mine = ok ? lse - lr[y] : 0.f;
    wave_sync();
    for (int c = lane; c < C; c += 64) lr[c] = (expf(lr[c] - lse) - ((ok && c == y) ? 1.f : 0.f)) / B;
    if (lane == 0) lossw[wave] = mine;
    wave_sync();
    float s1 = 0.f, s2 = 0.f;
    for (int d = lane; d < D; d += 64) {
      float a = 0.f;
      const float* wr = W + d * C;
#pragma unroll 5
      for (int c = 0; c < C; ++c) a += lr[c] * wr[c];
      a = round_to(a, dt);
      dzr[d] = a;
      if (ln) {
        const float dyh = a * lng[d];
        s1 += dyh; s2 += dyh * xr[d];
      } else {
        st_f(dcls, (size_t)b * D + d, a, dt);
      }
    }
    if (ln) {
      s1 = wave_sum(s1) / D; s2 = wave_sum(s2) / D;
      for (int d = lane; d < D; d += 64)
        st_f(dcls, (size_t)b * D + d, rs * (dzr[d] * lng[d] - s1 - xr[d] * s2), dt);
    }
  } else {
    for (int d = lane; d < D; d += 64) { xr[d] = 0.f; zr[d] = 0.f; dzr[d] = 0.f; }
    for (int c = lane; c < C; c += 64) lr[c] = 0.f;
    if (lane == 0) lossw[wave] = 0.f;
  }
  __syncthreads();
  float* out = partial + (size_t)blockIdx.x * ((size_t)D * C + C + 2 * D + 1);
  {
    // (d, c) of element i = d C + c, stepped along with i instead of divided out every time
    const int dstep = HEAD_THREADS / C, cstep = HEAD_THREADS % C;
    int d = (int)threadIdx.x / C, c = (int)threadIdx.x % C;
    for (int i = threadIdx.x; i < D * C; i += HEAD_THREADS) {
      float t = 0.f;
#pragma unroll
      for (int w = 0; w < HEAD_ROWS; ++w) t += zs[w * D + d] * dl[w * C + c];
      out[i] = t;
      d += dstep; c += cstep;
      if (c >= C) { c -= C; ++d; }
    }
  }
  float* o2 = out + (size_t)D * C;
  for (int c = threadIdx.x; c < C; c += HEAD_THREADS) {
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < HEAD_ROWS; ++w) t += dl[w * C + c];
    o2[c] = t;
  }
  float* o3 = o2 + C;
  for (int d = threadIdx.x; d < D; d += HEAD_THREADS) {
    float tg = 0.f, tb = 0.f;
#pragma unroll
    for (int w = 0; w < HEAD_ROWS; ++w) { tg += dzs[w * D + d] * xh[w * D + d]; tb += dzs[w * D + d]; }
    o3[d] = tg; o3[D + d] = tb;
  }
  if (threadIdx.x == 0) {
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < HEAD_ROWS; ++w) t += lossw[w];
    o3[2 * D] = t;
  }
}
}  // namespace


namespace {
// The same for few classes (C <= OUTER_MAX) and D <= 64 HEAD_NV: one row per workgroup.  The kernel is one dependent chain -
// row, LayerNorm sums, logits, softmax, gradient, LayerNorm's sums, row - so everything it reads is asked for up front, the
// four waves share the classes and the columns where there is something to share (each holds the whole row otherwise), and
// the batch sums are left to the reduction launch: z, dz o xhat, dz, dlogits and loss of every row go out as they are, the
// weight gradient z^T dlogits is formed there.  18.8 us at 128 rows of width 384 with four rows per workgroup and the weight
// gradient formed here.  The sums run over the columns in the order of the kernel above.
constexpr int HEAD_NV = 16;
__host__ __device__ inline size_t head_row_floats(int D, int C) { return (size_t)3 * D + C + 1; }
template <int NV>
__global__ __launch_bounds__(256) void head_row_kernel(const void* x, int dt, long xs, int B, int D, int C, const float* ln_g,
                                                       const float* ln_b, float eps, const float* W, const float* bias,
                                                       const int32_t* labels, void* dcls, float* out_z, float* out_dzx,
                                                       float* out_dz, float* out_dl, float* out_loss, int* flag) {
  extern __shared__ __align__(16) float sm[];
  float* wl = sm;                               // [D][C]
  float* dzs = wl + ((D * C + 3) & ~3);         // [D]
  float* lr = dzs + D;                          // [C] logits
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, b = blockIdx.x;
  const bool ln = ln_g != nullptr;
  // the row and the LayerNorm parameters in registers, column lane + 64 i in element i
  float xv[NV], gv[NV], bv[NV];
  const size_t base = (size_t)b * xs;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int d = lane + 64 * i;
    xv[i] = d < D ? ld_f(x, base + d, dt) : 0.f;
    gv[i] = ln && d < D ? ln_g[d] : 0.f;
    bv[i] = ln && d < D ? ln_b[d] : 0.f;
  }
  const int y = labels[b];
  const float my_bias = lane < C ? bias[lane] : 0.f;
  {
    const int n4 = (D * C) >> 2;
    for (int i0 = tid; i0 < n4; i0 += 8 * 256) {
      float4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = i0 + 256 * u < n4 ? reinterpret_cast<const float4*>(W)[i0 + 256 * u] : make_float4(0, 0, 0, 0);
#pragma unroll
      for (int u = 0; u < 8; ++u) if (i0 + 256 * u < n4) reinterpret_cast<float4*>(wl)[i0 + 256 * u] = v[u];
    }
    for (int i = 4 * n4 + tid; i < D * C; i += 256) wl[i] = W[i];
  }
  float zv[NV], rs = 0.f;
  if (ln) {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i) s += xv[i];
    const float mu = wave_sum(s) / D;
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i) { const float c = lane + 64 * i < D ? xv[i] - mu : 0.f; q += c * c; }
    rs = rsqrtf(wave_sum(q) / D + eps);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      xv[i] = lane + 64 * i < D ? (xv[i] - mu) * rs : 0.f;
      zv[i] = lane + 64 * i < D ? round_to(xv[i] * gv[i] + bv[i], dt) : 0.f;
    }
  } else {
#pragma unroll
    for (int i = 0; i < NV; ++i) { zv[i] = xv[i]; xv[i] = 0.f; }
  }
  __syncthreads();
  float a[OUTER_MAX / 4];
#pragma unroll
  for (int u = 0; u < OUTER_MAX / 4; ++u) a[u] = 0.f;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int d = lane + 64 * i;
    if (d < D) {
#pragma unroll
      for (int u = 0; u < OUTER_MAX / 4; ++u) if (wave + 4 * u < C) a[u] += zv[i] * wl[d * C + wave + 4 * u];
    }
  }
#pragma unroll
  for (int u = 0; u < OUTER_MAX / 4; ++u) a[u] = wave_sum(a[u]);
#pragma unroll
  for (int u = 0; u < OUTER_MAX / 4; ++u) if (lane == 0 && wave + 4 * u < C) lr[wave + 4 * u] = a[u];
  __syncthreads();
  const float logit = lane < C ? lr[lane] + my_bias : -INFINITY;
  const float mx = wave_max(logit);
  const float lse = mx + logf(wave_sum(lane < C ? expf(logit - mx) : 0.f));
  const bool ok = y >= 0 && y < C;
  const float dl = lane < C ? (expf(logit - lse) - ((ok && lane == y) ? 1.f : 0.f)) / B : 0.f;
  if (wave == 0) {
    const float ly = __shfl(logit, ok ? y : 0, 64);
    if (lane < C) out_dl[(size_t)b * C + lane] = dl;
    if (lane == 0) { out_loss[b] = ok ? lse - ly : 0.f; if (!ok) *flag = 1; }
  }
  float dlc[OUTER_MAX];
#pragma unroll
  for (int c = 0; c < OUTER_MAX; ++c) dlc[c] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(dl), c));
  for (int d = tid; d < D; d += 256) {
    float v = 0.f;
#pragma unroll
    for (int c = 0; c < OUTER_MAX; ++c) if (c < C) v += dlc[c] * wl[d * C + c];
    v = round_to(v, dt);
    dzs[d] = v;
    if (!ln) st_f(dcls, (size_t)b * D + d, v, dt);
  }
  __syncthreads();
  float dz[NV], s1 = 0.f, s2 = 0.f;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int d = lane + 64 * i;
    dz[i] = d < D ? dzs[d] : 0.f;
    const float dyh = dz[i] * gv[i];
    s1 += dyh; s2 += dyh * xv[i];
  }
  if (ln) { s1 = wave_sum(s1) / D; s2 = wave_sum(s2) / D; }
#pragma unroll
  for (int i = 0; i < NV; ++i) {          // the waves share the columns to write
    const int d = lane + 64 * i;
    if ((i & 3) == wave && d < D) {
      const size_t o = (size_t)b * D + d;
      out_z[o] = zv[i];
      if (ln) {
        st_f(dcls, o, rs * fmaf(-xv[i], s2, fmaf(dz[i], gv[i], -s1)), dt);
        out_dzx[o] = dz[i] * xv[i];
        out_dz[o] = dz[i];
      }
    }
  }
}
size_t head_row_lds(int D, int C) { return ((((size_t)D * C + 3) & ~(size_t)3) + D + C) * sizeof(float); }
bool head_rows_ok(int D, int C, const float* W) {
  return C <= OUTER_MAX && D <= 64 * HEAD_NV && head_row_lds(D, C) <= 64 * 1024 && !(((uintptr_t)W) & 15);
}
}  // namespace

size_t vit_head_partial_floats(int B, int D, int C) {
  const size_t few = (size_t)((B + HEAD_ROWS - 1) / HEAD_ROWS) * ((size_t)D * C + C + 2 * D + 1), rows = (size_t)B * head_row_floats(D, C);
  return few > rows ? few : rows;
}
static size_t vit_head_lds(int D, int C, bool with_w) {
  return ((size_t)3 * HEAD_ROWS * D + HEAD_ROWS * C + HEAD_ROWS + C + 2 * D + (with_w ? (size_t)D * C : 0)) * sizeof(float);
}
bool vit_head_fused_ok(int D, int C) { return vit_head_lds(D, C, false) <= 64 * 1024; }

int launch_vit_head(hipStream_t s, const void* x, int dt, long xs, int B, int D, int C, const float* ln_g,
                    const float* ln_b, float eps, const float* W, const float* bias, const int32_t* labels, void* dcls,
                    ReduceQueue& rq, float* d_ln_g, float* d_ln_b, float* dW, float* dbias, float* loss, float* loss2,
                    int* flag) {
  bool queued;
  float* partials = rq.space(vit_head_partial_floats(B, D, C), &queued);
  if (head_rows_ok(D, C, W)) {
    float *z = partials, *dzx = z + (size_t)B * D, *dz = dzx + (size_t)B * D, *dl = dz + (size_t)B * D, *ls = dl + (size_t)B * C;
#define HEAD_LAUNCH(NV)                                                                                                        \
  hipLaunchKernelGGL(head_row_kernel<NV>, dim3(B), dim3(256), head_row_lds(D, C), s, x, dt, xs, B, D, C, ln_g, ln_b, eps, W, bias, \
                     labels, dcls, z, dzx, dz, dl, ls, flag)
    if (D <= 64) HEAD_LAUNCH(1);
    else if (D <= 192) HEAD_LAUNCH(3);
    else if (D <= 384) HEAD_LAUNCH(6);
    else if (D <= 768) HEAD_LAUNCH(12);
    else HEAD_LAUNCH(16);
#undef HEAD_LAUNCH
    PPLL_HIP(hipGetLastError());
    PPLL_TRY(rq.reduce_outer(s, queued, z, B, D, dl, C, dW));
    PPLL_TRY(rq.reduce(s, queued, dl, B, C, C, 1.0f, dbias));
    if (ln_g) {
      PPLL_TRY(rq.reduce(s, queued, dzx, B, D, D, 1.0f, d_ln_g));
      PPLL_TRY(rq.reduce(s, queued, dz, B, D, D, 1.0f, d_ln_b));
    }
    PPLL_TRY(rq.reduce(s, queued, ls, B, 1, 1, 1.0f / B, loss));
    if (loss2) PPLL_TRY(rq.reduce(s, queued, ls, B, 1, 1, 1.0f / B, loss2));
    return PPLL_OK;
  }
  const int chunks = (B + HEAD_ROWS - 1) / HEAD_ROWS;
  const long P = (long)D * C + C + 2 * D + 1;
  const bool with_w = vit_head_lds(D, C, true) <= 64 * 1024;
  hipLaunchKernelGGL(vit_head_kernel, dim3(chunks), dim3(HEAD_THREADS), vit_head_lds(D, C, with_w), s, x, dt, xs, B, D, C, ln_g, ln_b,
                     eps, W, bias, labels, dcls, partials, flag, (int)with_w);
  PPLL_HIP(hipGetLastError());
  PPLL_TRY(rq.reduce(s, queued, partials, chunks, D * C, P, 1.0f, dW));
  PPLL_TRY(rq.reduce(s, queued, partials + (size_t)D * C, chunks, C, P, 1.0f, dbias));
  if (ln_g) {
    PPLL_TRY(rq.reduce(s, queued, partials + (size_t)D * C + C, chunks, D, P, 1.0f, d_ln_g));
    PPLL_TRY(rq.reduce(s, queued, partials + (size_t)D * C + C + D, chunks, D, P, 1.0f, d_ln_b));
  }
  PPLL_TRY(rq.reduce(s, queued, partials + (size_t)D * C + C + 2 * D, chunks, 1, P, 1.0f / B, loss));
  if (loss2) PPLL_TRY(rq.reduce(s, queued, partials + (size_t)D * C + C + 2 * D, chunks, 1, P, 1.0f / B, loss2));
  return PPLL_OK;
}

// ===================================================================== ViT embedding pieces
namespace {
__global__ __launch_bounds__(256) void patchify_kernel(const void* img, int dt, int B, int H, int W, int C, int P,
                                                       void* out) {
  size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  int gw = W / P, gh = H / P, ppc = P * P * C;
  size_t total = (size_t)B * gh * gw * ppc;
  if (i >= total) return;
  int e = i % ppc; size_t pidx = i / ppc;
  int ch = e % C, c = (e / C) % P, r = e / (C * P);
  int gx = pidx % gw, gy = (pidx / gw) % gh; int b = pidx / ((size_t)gw * gh);
  size_t src = (((size_t)b * H + gy * P + r) * W + gx * P + c) * C + ch;
  if (dt == BF16) ((uint16_t*)out)[i] = ((const uint16_t*)img)[src];
  else ((float*)out)[i] = ((const float*)img)[src];
}

// bf16, P*C and W*C multiples of 8: a patch row (P*C contiguous elements in the image and in the patch vector) moves as
// 16-byte pieces, one per thread; 32-bit index arithmetic
__global__ __launch_bounds__(256) void patchify_bf16_kernel(const uint16_t* img, int B, int H, int W, int C, int P,
                                                            uint16_t* out) {
  const uint32_t row8 = (uint32_t)(P * C) >> 3, gw = W / P, gh = H / P;
  const uint32_t total = (uint32_t)B * gh * gw * P * row8;
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  if (i >= total) return;
  const uint32_t v = i % row8, t = i / row8;      // piece within the patch row; (patch, row)
  const uint32_t r = t % P, pidx = t / P;
  const uint32_t gx = pidx % gw, q = pidx / gw, gy = q % gh, b = q / gh;
  const size_t src = (((size_t)b * H + gy * P + r) * W + gx * P) * C + 8 * v;
  *reinterpret_cast<uint4*>(out + (size_t)i * 8) = *reinterpret_cast<const uint4*>(img + src);
}

__global__ __launch_bounds__(256) void assemble_tokens_kernel(const void* E, int dt, const float* cls,
                                                              const float* pos, int B, int T, int D, void* x0) {
  size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (size_t)B * T * D) return;
  int d = i % D, t = (i / D) % T; int b = i / ((size_t)D * T);
  float v = t == 0 ? cls[d] : ld_f(E, ((size_t)b * (T - 1) + (t - 1)) * D + d, dt);
  st_f(x0, i, v + pos[(size_t)t * D + d], dt);
}

// bf16, D a multiple of 8: 8 elements per thread
__global__ __launch_bounds__(256) void assemble_tokens_bf16_kernel(const uint16_t* E, const float* cls, const float* pos,
                                                                   int B, int T, int D, uint16_t* x0) {
  const size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 8;
  if (i >= (size_t)B * T * D) return;
  const int d = i % D, t = (i / D) % T;
  const int b = i / ((size_t)D * T);
  float v[8];
  if (t == 0) {
    const float4 c0 = *reinterpret_cast<const float4*>(cls + d), c1 = *reinterpret_cast<const float4*>(cls + d + 4);
    v[0] = c0.x; v[1] = c0.y; v[2] = c0.z; v[3] = c0.w; v[4] = c1.x; v[5] = c1.y; v[6] = c1.z; v[7] = c1.w;
  } else {
    const uint4 w = *reinterpret_cast<const uint4*>(E + ((size_t)b * (T - 1) + (t - 1)) * D + d);
    v[0] = __uint_as_float(w.x << 16); v[1] = __uint_as_float(w.x & 0xffff0000u);
    v[2] = __uint_as_float(w.y << 16); v[3] = __uint_as_float(w.y & 0xffff0000u);
    v[4] = __uint_as_float(w.z << 16); v[5] = __uint_as_float(w.z & 0xffff0000u);
    v[6] = __uint_as_float(w.w << 16); v[7] = __uint_as_float(w.w & 0xffff0000u);
  }
  const float4 p0 = *reinterpret_cast<const float4*>(pos + (size_t)t * D + d);
  const float4 p1 = *reinterpret_cast<const float4*>(pos + (size_t)t * D + d + 4);
  *reinterpret_cast<uint4*>(x0 + i) =
      make_uint4(f32x2_to_bf16x2(v[0] + p0.x, v[1] + p0.y), f32x2_to_bf16x2(v[2] + p0.z, v[3] + p0.w),
                 f32x2_to_bf16x2(v[4] + p1.x, v[5] + p1.y), f32x2_to_bf16x2(v[6] + p1.z, v[7] + p1.w));
}
__global__ __launch_bounds__(256) void scatter_cls_bf16_kernel(const uint16_t* dcls, int B, int T, int D, uint16_t* dx) {
  const size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 8;
  if (i >= (size_t)B * T * D) return;
  const int d = i % D, t = (i / D) % T;
  const int b = i / ((size_t)D * T);
  uint4 w = make_uint4(0, 0, 0, 0);
  if (t == 0) w = *reinterpret_cast<const uint4*>(dcls + (size_t)b * D + d);
  *reinterpret_cast<uint4*>(dx + i) = w;
}

constexpr int EMB_ROWS = 8;   // batch entries per partial
// partial[c][t,d] = sum over the chunk's batch entries of dx[b,t,d]; dE = dx[:,1:,:] gathered
__global__ __launch_bounds__(256) void embed_bwd_kernel(const void* dx, int dt, int B, int T, int D, float* partial,
                                                        void* dE) {
  size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;   // over [T, D]
  if (i >= (size_t)T * D) return;
  int d = i % D, t = i / D;
  const int b0 = blockIdx.y * EMB_ROWS, b1 = min(B, b0 + EMB_ROWS);
  float acc = 0.f;
  for (int b = b0; b < b1; ++b) {
    size_t src = ((size_t)b * T + t) * D + d;
    acc += ld_f(dx, src, dt);
    if (t > 0) {
      size_t dst = ((size_t)b * (T - 1) + (t - 1)) * D + d;
      if (dt == BF16) ((uint16_t*)dE)[dst] = ((const uint16_t*)dx)[src];
      else ((float*)dE)[dst] = ((const float*)dx)[src];
    }
  }
  partial[(size_t)blockIdx.y * T * D + i] = acc;
}

// bf16, D a multiple of 8: a thread takes 8 consecutive d of one token and the chunk's 8 batch entries,
// whose loads are issued together; the sum still runs in batch order
__global__ __launch_bounds__(256) void embed_bwd_bf16_kernel(const uint16_t* dx, int B, int T, int D, float* partial,
                                                             uint16_t* dE) {
  const size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 8;   // over [T, D]
  if (i >= (size_t)T * D) return;
  const int d = i % D, t = i / D;
  const int b0 = blockIdx.y * EMB_ROWS;
  uint4 v[EMB_ROWS];
#pragma unroll
  for (int u = 0; u < EMB_ROWS; ++u) {
    v[u] = make_uint4(0, 0, 0, 0);
    if (b0 + u < B) v[u] = *reinterpret_cast<const uint4*>(dx + ((size_t)(b0 + u) * T + t) * D + d);
  }
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int u = 0; u < EMB_ROWS; ++u) {
    if (b0 + u >= B) break;
    const uint32_t* w = reinterpret_cast<const uint32_t*>(&v[u]);
#pragma unroll
    for (int e = 0; e < 4; ++e) { acc[2 * e] += __uint_as_float(w[e] << 16); acc[2 * e + 1] += __uint_as_float(w[e] & 0xffff0000u); }
    if (t > 0) *reinterpret_cast<uint4*>(dE + ((size_t)(b0 + u) * (T - 1) + (t - 1)) * D + d) = v[u];
  }
  float* out = partial + (size_t)blockIdx.y * T * D + i;
  *reinterpret_cast<float4*>(out) = make_float4(acc[0], acc[1], acc[2], acc[3]);
  *reinterpret_cast<float4*>(out + 4) = make_float4(acc[4], acc[5], acc[6], acc[7]);
}

__global__ __launch_bounds__(256) void scatter_cls_kernel(const void* dcls, int dt, int B, int T, int D, void* dx) {
  size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (size_t)B * T * D) return;
  int d = i % D, t = (i / D) % T; int b = i / ((size_t)D * T);
  st_f(dx, i, t == 0 ? ld_f(dcls, (size_t)b * D + d, dt) : 0.f, dt);
}
}  // namespace

int launch_patchify(hipStream_t s, const void* img, int dt, int B, int H, int W, int C, int P, void* patches) {
  size_t total = (size_t)B * H * W * C;
  const size_t used = (size_t)B * (H / P) * (W / P) * P * P * C;   // pixels of whole patches
  if (dt == BF16 && !((P * C) & 7) && !((W * C) & 7) && !((((uintptr_t)img) | ((uintptr_t)patches)) & 15) &&
      used / 8 < ((size_t)1 << 31)) {
    hipLaunchKernelGGL(patchify_bf16_kernel, dim3((unsigned)((used / 8 + 255) / 256)), dim3(256), 0, s, (const uint16_t*)img, B,
                       H, W, C, P, (uint16_t*)patches);
    PPLL_HIP(hipGetLastError());
    return PPLL_OK;
  }
  hipLaunchKernelGGL(patchify_kernel, dim3((total + 255) / 256), dim3(256), 0, s, img, dt, B, H, W, C, P, patches);
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}
int launch_assemble_tokens(hipStream_t s, const void* E, int dt, const float* cls, const float* pos, int B, int T,
                           int D, void* x0) {
  size_t total = (size_t)B * T * D;
  const bool vec = dt == BF16 && !(D & 7) &&
                   !((((uintptr_t)E) | ((uintptr_t)cls) | ((uintptr_t)pos) | ((uintptr_t)x0)) & 15);
  if (vec)
    hipLaunchKernelGGL(assemble_tokens_bf16_kernel, dim3((total / 8 + 255) / 256), dim3(256), 0, s, (const uint16_t*)E,
                       cls, pos, B, T, D, (uint16_t*)x0);
  else
    hipLaunchKernelGGL(assemble_tokens_kernel, dim3((total + 255) / 256), dim3(256), 0, s, E, dt, cls, pos, B, T, D, x0);
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}
int embed_bwd_partial_floats(int B, int T, int D) { return ((B + EMB_ROWS - 1) / EMB_ROWS) * T * D; }
int launch_embed_bwd(hipStream_t s, const void* dx, int dt, int B, int T, int D, ReduceQueue& rq, float* dpos,
                     float* dcls, void* dE) {
  const int total = T * D, chunks = (B + EMB_ROWS - 1) / EMB_ROWS;
  bool queued;
  float* partials = rq.space((size_t)chunks * total, &queued);
  if (dt == BF16 && !(D & 7) && !((((uintptr_t)dx) | ((uintptr_t)dE) | ((uintptr_t)partials)) & 15))
    hipLaunchKernelGGL(embed_bwd_bf16_kernel, dim3((total / 8 + 255) / 256, chunks), dim3(256), 0, s, (const uint16_t*)dx, B,
                       T, D, partials, (uint16_t*)dE);
  else
    hipLaunchKernelGGL(embed_bwd_kernel, dim3((total + 255) / 256, chunks), dim3(256), 0, s, dx, dt, B, T, D, partials, dE);
  PPLL_HIP(hipGetLastError());
  PPLL_TRY(rq.reduce(s, queued, partials, chunks, total, total, 1.0f, dpos));
  return rq.reduce(s, queued, partials, chunks, D, total, 1.0f, dcls);   // the cls row is token 0
}
int launch_scatter_cls(hipStream_t s, const void* dcls, int dt, int B, int T, int D, void* dx) {
  size_t total = (size_t)B * T * D;
  if (dt == BF16 && !(D & 7) && !((((uintptr_t)dcls) | ((uintptr_t)dx)) & 15))
    hipLaunchKernelGGL(scatter_cls_bf16_kernel, dim3((total / 8 + 255) / 256), dim3(256), 0, s, (const uint16_t*)dcls, B,
                       T, D, (uint16_t*)dx);
  else
    hipLaunchKernelGGL(scatter_cls_kernel, dim3((total + 255) / 256), dim3(256), 0, s, dcls, dt, B, T, D, dx);
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}

// ===================================================================== attention (per batch, head)
namespace {
// One workgroup per (batch, head); K and V of the head live in LDS as fp32 with
// a padded row so that lanes reading different keys hit different banks.  Each
// wave takes query rows round-robin: scores with lanes over keys, softmax by
// wave reductions, then the weighted sum with lanes over the head dimension.
constexpr int ATT_MAX_T = 256;

__global__ __launch_bounds__(256) void attention_fwd_kernel(const void* qkv, int dt, int T, int H, int dh, void* out,
                                                            float* lse) {
  extern __shared__ float sm[];
  const int ld = dh + 1;
  float* Ks = sm;                       // [T][ld]
  float* Vs = Ks + (size_t)T * ld;      // [T][ld]
  float* qs = Vs + (size_t)T * ld;      // [4][dh]
  float* ps = qs + 4 * dh;              // [4][T]
  const int b = blockIdx.x / H, h = blockIdx.x % H, D = H * dh;
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  const float scale = rsqrtf((float)dh);
  for (int i = threadIdx.x; i < T * dh; i += 256) {
    int t = i / dh, d = i % dh;
    size_t base = ((size_t)b * T + t) * 3 * D + h * dh + d;
    Ks[t * ld + d] = ld_f(qkv, base + D, dt);
    Vs[t * ld + d] = ld_f(qkv, base + 2 * D, dt);
  }
  __syncthreads();
  float* q = qs + wave * dh;
  float* p = ps + wave * T;
  for (int i = wave; i < T; i += 4) {
    size_t qb = ((size_t)b * T + i) * 3 * D + h * dh;
    for (int d = lane; d < dh; d += 64) q[d] = ld_f(qkv, qb + d, dt);
    wave_sync();
    float sc[ATT_MAX_T / 64];
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < ATT_MAX_T / 64; ++r) {
      int j = lane + r * 64;
      float a = -INFINITY;
      if (j < T) {
        a = 0.f;
        for (int d = 0; d < dh; ++d) a = fmaf(q[d], Ks[j * ld + d], a);
        a *= scale;
      }
      sc[r] = a;
      mx = fmaxf(mx, a);
    }
    mx = wave_max(mx);
    float se = 0.f;
#pragma unroll
    for (int r = 0; r < ATT_MAX_T / 64; ++r) {
      int j = lane + r * 64;
      float e = j < T ? __expf(sc[r] - mx) : 0.f;
      sc[r] = e;
      se += e;
    }
    se = wave_sum(se);
    float inv = 1.0f / se;
#pragma unroll
    for (int r = 0; r < ATT_MAX_T / 64; ++r) {
      int j = lane + r * 64;
      if (j < T) p[j] = sc[r] * inv;
    }
    wave_sync();
    for (int d = lane; d < dh; d += 64) {
      float o = 0.f;
      for (int j = 0; j < T; ++j) o = fmaf(p[j], Vs[j * ld + d], o);
      st_f(out, ((size_t)b * T + i) * D + h * dh + d, o, dt);
    }
    if (lane == 0) lse[((size_t)b * H + h) * T + i] = mx + __logf(se);
    wave_sync();
  }
}

// Backward in two ordered passes.  Pass A (wave per query row i): D_i =
// <dO_i, O_i>, P_i recomputed from the saved log-sum-exp, dS_i = P_i o (dO_i V^T
// - D_i), dQ_i = scale dS_i K.  Pass B (wave per key j) recomputes column j of P
// and dS from Q and dO (now in LDS) and accumulates dV_j = sum_i P_ij dO_i and
// dK_j = scale sum_i dS_ij Q_i in a fixed order.
__global__ __launch_bounds__(256) void attention_bwd_kernel(const void* qkv, const void* out, const void* dout,
                                                            const float* lse, int dt, int T, int H, int dh,
                                                            void* dqkv) {
  extern __shared__ float sm[];
  const int ld = dh + 1;
  float* As = sm;                        // pass A: K, pass B: Q     [T][ld]
  float* Bs = As + (size_t)T * ld;       // pass A: V, pass B: dO    [T][ld]
  float* vec = Bs + (size_t)T * ld;      // [4][2][dh] per-wave row vectors
  float* ps = vec + 8 * dh;              // [4][2][T]  per-wave p and ds
  float* Dr = ps + 8 * T;                // [T] row dots
  float* Ls = Dr + T;                    // [T] lse
  const int b = blockIdx.x / H, h = blockIdx.x % H, D = H * dh;
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  const float scale = rsqrtf((float)dh);
  for (int i = threadIdx.x; i < T * dh; i += 256) {
    int t = i / dh, d = i % dh;
    size_t base = ((size_t)b * T + t) * 3 * D + h * dh + d;
    As[t * ld + d] = ld_f(qkv, base + D, dt);
    Bs[t * ld + d] = ld_f(qkv, base + 2 * D, dt);
  }
  for (int i = threadIdx.x; i < T; i += 256) Ls[i] = lse[((size_t)b * H + h) * T + i];
  __syncthreads();
  float* v0 = vec + wave * 2 * dh;       // q_i  / k_j
  float* v1 = v0 + dh;                   // dO_i / v_j
  float* p0 = ps + wave * 2 * T;         // p
  float* p1 = p0 + T;                    // ds
  // ---- pass A
  for (int i = wave; i < T; i += 4) {
    size_t qb = ((size_t)b * T + i) * 3 * D + h * dh, ob = ((size_t)b * T + i) * D + h * dh;
    float dd = 0.f;
    for (int d = lane; d < dh; d += 64) {
      v0[d] = ld_f(qkv, qb + d, dt);
      float g = ld_f(dout, ob + d, dt);
      v1[d] = g;
      dd += g * ld_f(out, ob + d, dt);
    }
    dd = wave_sum(dd);
    if (lane == 0) Dr[i] = dd;
    wave_sync();
    for (int j = lane; j < T; j += 64) {
      float s = 0.f, dp = 0.f;
      for (int d = 0; d < dh; ++d) { s = fmaf(v0[d], As[j * ld + d], s); dp = fmaf(v1[d], Bs[j * ld + d], dp); }
      float pj = __expf(s * scale - Ls[i]);
      p1[j] = pj * (dp - dd);
    }
    wave_sync();
    for (int d = lane; d < dh; d += 64) {
      float a = 0.f;
      for (int j = 0; j < T; ++j) a = fmaf(p1[j], As[j * ld + d], a);
      st_f(dqkv, qb + d, a * scale, dt);
    }
    wave_sync();
  }
  __syncthreads();
  // ---- reload: Q and dO
  for (int i = threadIdx.x; i < T * dh; i += 256) {
    int t = i / dh, d = i % dh;
    As[t * ld + d] = ld_f(qkv, ((size_t)b * T + t) * 3 * D + h * dh + d, dt);
    Bs[t * ld + d] = ld_f(dout, ((size_t)b * T + t) * D + h * dh + d, dt);
  }
  __syncthreads();
  // ---- pass B
  for (int j = wave; j < T; j += 4) {
    size_t kb = ((size_t)b * T + j) * 3 * D + h * dh;
    for (int d = lane; d < dh; d += 64) { v0[d] = ld_f(qkv, kb + D + d, dt); v1[d] = ld_f(qkv, kb + 2 * D + d, dt); }
    wave_sync();
    for (int i = lane; i < T; i += 64) {
      float s = 0.f, dp = 0.f;
      for (int d = 0; d < dh; ++d) { s = fmaf(As[i * ld + d], v0[d], s); dp = fmaf(Bs[i * ld + d], v1[d], dp); }
      float pij = __expf(s * scale - Ls[i]);
      p0[i] = pij;
      p1[i] = pij * (dp - Dr[i]);
    }
    wave_sync();
    for (int d = lane; d < dh; d += 64) {
      float dv = 0.f, dk = 0.f;
      for (int i = 0; i < T; ++i) { dv = fmaf(p0[i], Bs[i * ld + d], dv); dk = fmaf(p1[i], As[i * ld + d], dk); }
      st_f(dqkv, kb + D + d, dk * scale, dt);
      st_f(dqkv, kb + 2 * D + d, dv, dt);
    }
    wave_sync();
  }
}

int allow_lds(const void* fn, size_t bytes, OncePerDevice& once) {
  if (bytes > UNIT_LDS) { set_error("attention: %zu bytes of LDS exceed 160 KB", bytes); return PPLL_ERR_CONFIG; }
  return raise_lds(fn, UNIT_LDS, once);
}
}  // namespace

int launch_attention_fwd_generic(hipStream_t s, const void* qkv, int dt, int B, int T, int H, int dh, void* out,
                                 float* lse) {
  if (T > ATT_MAX_T || T < 1) { set_error("attention: tokens %d outside 1..%d", T, ATT_MAX_T); return PPLL_ERR_CONFIG; }
  const size_t lds = att_heads_lds(T, dh, false);
  static OncePerDevice once;
  PPLL_TRY(allow_lds((const void*)attention_fwd_kernel, lds, once));
  hipLaunchKernelGGL(attention_fwd_kernel, dim3(B * H), dim3(256), lds, s, qkv, dt, T, H, dh, out, lse);
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}

int launch_attention_bwd_generic(hipStream_t s, const void* qkv, const void* out, const void* dout, const float* lse,
                                 int dt, int B, int T, int H, int dh, void* dqkv) {
  if (T > ATT_MAX_T || T < 1) { set_error("attention: tokens %d outside 1..%d", T, ATT_MAX_T); return PPLL_ERR_CONFIG; }
  const size_t lds = att_heads_lds(T, dh, true);
  static OncePerDevice once;
  PPLL_TRY(allow_lds((const void*)attention_bwd_kernel, lds, once));
  hipLaunchKernelGGL(attention_bwd_kernel, dim3(B * H), dim3(256), lds, s, qkv, out, dout, lse, dt, T, H, dh, dqkv);
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}

// ===================================================================== optimizers
namespace {
// Algorithm 1, update line, over the flat parameter blob.  Bound by memory (SGD 22 bytes a parameter, AdamW 30); four
// parameters per thread, 16 bytes per access.
// Coupled L2 decay, momentum buffer (first step: buffer = gradient), plain or Nesterov step.
struct SgdArgs { float lr, momentum, wd; int nesterov, first; };
__device__ __forceinline__ float sgd_one(float w, float g, float& buf, const SgdArgs& a) {
  float gr = g + a.wd * w;
  if (a.momentum != 0.f) {
    const float bv = a.first ? gr : a.momentum * buf + gr;
    buf = bv;
    gr = a.nesterov ? gr + a.momentum * bv : bv;
  }
  return w - a.lr * gr;
}
__global__ __launch_bounds__(256) void sgd_kernel(float* p, const float* g, float* buf, uint16_t* shadow, size_t n, SgdArgs a) {
  const size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4;
  const bool use_buf = a.momentum != 0.f;
  if (i + 4 <= n) {
    const float4 w = *reinterpret_cast<const float4*>(p + i), gr = *reinterpret_cast<const float4*>(g + i);
    float4 b = use_buf && !a.first ? *reinterpret_cast<const float4*>(buf + i) : make_float4(0.f, 0.f, 0.f, 0.f);
    const float4 o = make_float4(sgd_one(w.x, gr.x, b.x, a), sgd_one(w.y, gr.y, b.y, a), sgd_one(w.z, gr.z, b.z, a), sgd_one(w.w, gr.w, b.w, a));
    if (use_buf) *reinterpret_cast<float4*>(buf + i) = b;
    *reinterpret_cast<float4*>(p + i) = o;
    if (shadow) *reinterpret_cast<uint2*>(shadow + i) = make_uint2(f32x2_to_bf16x2(o.x, o.y), f32x2_to_bf16x2(o.z, o.w));
    return;
  }
  for (size_t j = i; j < n; ++j) {
    float b = use_buf ? buf[j] : 0.f;
    const float o = sgd_one(p[j], g[j], b, a);
    if (use_buf) buf[j] = b;
    p[j] = o;
    if (shadow) shadow[j] = f32_to_bf16(o);
  }
}

// AdamW: decoupled decay, bias-corrected moments (corrections computed on the host).
struct AdamArgs { float lr, b1, b2, eps, wd, bc1, bc2; };
__device__ __forceinline__ float adamw_one(float p, float gr, float& m, float& v, const AdamArgs& a) {
  const float w = p * (1.0f - a.lr * a.wd);
  m = a.b1 * m + (1.0f - a.b1) * gr;
  v = a.b2 * v + (1.0f - a.b2) * gr * gr;
  return w - a.lr * (m / a.bc1) / (sqrtf(v / a.bc2) + a.eps);
}
__global__ __launch_bounds__(256) void adamw_kernel(float* p, const float* g, float* m, float* v, uint16_t* shadow, size_t n, AdamArgs a) {
  const size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i + 4 <= n) {
    const float4 w = *reinterpret_cast<const float4*>(p + i), gr = *reinterpret_cast<const float4*>(g + i);
    float4 mi = *reinterpret_cast<const float4*>(m + i), vi = *reinterpret_cast<const float4*>(v + i);
    const float4 o = make_float4(adamw_one(w.x, gr.x, mi.x, vi.x, a), adamw_one(w.y, gr.y, mi.y, vi.y, a),
                                 adamw_one(w.z, gr.z, mi.z, vi.z, a), adamw_one(w.w, gr.w, mi.w, vi.w, a));
    *reinterpret_cast<float4*>(m + i) = mi;
    *reinterpret_cast<float4*>(v + i) = vi;
    *reinterpret_cast<float4*>(p + i) = o;
    if (shadow) *reinterpret_cast<uint2*>(shadow + i) = make_uint2(f32x2_to_bf16x2(o.x, o.y), f32x2_to_bf16x2(o.z, o.w));
    return;
  }
  for (size_t j = i; j < n; ++j) {
    float mi = m[j], vi = v[j];
    const float o = adamw_one(p[j], g[j], mi, vi, a);
    m[j] = mi; v[j] = vi; p[j] = o;
    if (shadow) shadow[j] = f32_to_bf16(o);
  }
}

__global__ __launch_bounds__(256) void refresh_shadow_kernel(const float* p, uint16_t* shadow, size_t n) {
  size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) shadow[i] = f32_to_bf16(p[i]);
}

__global__ __launch_bounds__(256) void fill_zero_kernel(uint32_t* p, size_t words) {
  size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < words) p[i] = 0u;
}
}  // namespace

int launch_sgd(hipStream_t s, float* p, const float* g, float* buf, uint16_t* shadow, size_t n, float lr, float momentum,
               int nesterov, float wd, int first) {
  hipLaunchKernelGGL(sgd_kernel, dim3((n + 1023) / 1024), dim3(256), 0, s, p, g, buf, shadow, n, SgdArgs{lr, momentum, wd, nesterov, first});
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}
int launch_adamw(hipStream_t s, float* p, const float* g, float* m, float* v, uint16_t* shadow, size_t n, float lr,
                 float b1, float b2, float eps, float wd, float bc1, float bc2) {
  hipLaunchKernelGGL(adamw_kernel, dim3((n + 1023) / 1024), dim3(256), 0, s, p, g, m, v, shadow, n, AdamArgs{lr, b1, b2, eps, wd, bc1, bc2});
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}
int launch_refresh_shadow(hipStream_t s, const float* p, uint16_t* shadow, size_t n) {
  hipLaunchKernelGGL(refresh_shadow_kernel, dim3((n + 255) / 256), dim3(256), 0, s, p, shadow, n);
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}
namespace {
__global__ __launch_bounds__(256) void copy_probe_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, size_t n16) {
  size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n16) dst[i] = src[i];
}
}  // namespace
// Plain copy of known size: the reference that hardware byte counters are scaled against.
int launch_copy_probe(hipStream_t s, const void* src, void* dst, size_t bytes) {
  size_t n16 = bytes / 16;
  hipLaunchKernelGGL(copy_probe_kernel, dim3((unsigned)((n16 + 255) / 256)), dim3(256), 0, s, (const uint4*)src, (uint4*)dst, n16);
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}
int launch_fill_zero(hipStream_t s, void* p, size_t bytes) {
  size_t words = (bytes + 3) / 4;
  hipLaunchKernelGGL(fill_zero_kernel, dim3((words + 255) / 256), dim3(256), 0, s, (uint32_t*)p, words);
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}

}  // namespace ppll
