// fp32 Linear-layer products on the matrix cores (v_mfma_f32_32x32x2_f32: 32-bit products, 32-bit sums) and the attention
// of shapes that the bf16 matrix-core attention does not take.
//
// Products.  C[M,N] = A(M,k) B(k,N).  At the sizes the fp32 path is used at (some hundred rows, widths of 64 to 384) a
// product has 0.01 to 0.5 GFLOP: latency decides, so a workgroup owns a 32 x 32 (64 x 64 for large outputs) tile, its four
// waves split k between them (a contiguous quarter each) and every wave reads its fragments straight from memory in the
// MFMA's register layout, two groups of loads in flight: a k-contiguous operand 16 bytes per lane (lane half h holds k =
// 8 g + 4 h .. + 3 of its row, MFMA e of a group takes element e of every lane), any other operand 4 bytes per lane and k
// (32 neighbouring rows: a full 128-byte line).  The four partial tiles meet in LDS and are added in wave order.  The
// run-time-typed kernel took 22.6 us per product (and 21.6 us for a weight gradient) at 520 rows of width 64.
// Weight gradients of a step go out as one launch over a table of products, bias gradients (column sums of B) included.
#include "common.h"
#include "plan.h"

namespace ppll {

namespace {
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

constexpr int OOB = 0x7fffffff;        // beyond every buffer here (all below 2^30 bytes, checked on the host)
constexpr int OOB_BASE = 0x40000000;   // stays out of range after a k offset (< 2^30) is added
constexpr int U = 4;                   // groups of 8 k per register set

struct F32Args {
  const float* A; const float* B; float* C; float* colsum;   // colsum: column sums of B (or null)
  int lda, ldb, ldc, M, N, K;
  const float* bias;
  const float* residual; int ldr;
  int epilogue;
  float* C2;
  const float* aux; int ldaux;
  uint32_t a_bytes, b_bytes;
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_of(const void* ptr, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(ptr), 0, (int)bytes, 0x00020000);
}

template <int R> struct F32Frags { float a[U][R][4], b[U][R][4]; };
template <int R> constexpr int part_ld() { return 32 * R + 4; }
template <int R> constexpr int f32_lds_bytes() { return 4 * 32 * R * part_ld<R>() * 4 + 4 * 32 * R * 4; }

// AT: A stored [K][M], else [M][K]; BT: B stored [K][N], else [N][K].  R x R MFMA tiles of 32 x 32 per workgroup.
template <bool AT, bool BT, int R>
__device__ __forceinline__ void gemm_f32_tile(const F32Args& p, const int m0, const int n0) {
  extern __shared__ __align__(16) float f32_smem[];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, row = lane & 31, h = lane >> 5;
  const __amdgpu_buffer_rsrc_t rsA = rsrc_of(p.A, p.a_bytes), rsB = rsrc_of(p.B, p.b_bytes);
  const int per_wave = ((p.K + 31) / 32) * 8;                     // k of a wave, a multiple of 8
  const int k_beg = wave * per_wave, k_end = min(p.K, k_beg + per_wave);
  int a_base[R], b_base[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int m = m0 + 32 * r + row, n = n0 + 32 * r + row;
    a_base[r] = m < p.M ? (AT ? m * 4 : (int)((long)m * p.lda * 4)) : OOB_BASE;
    b_base[r] = n < p.N ? (BT ? n * 4 : (int)((long)n * p.ldb * 4)) : OOB_BASE;
  }
  auto load_one = [&](__amdgpu_buffer_rsrc_t rs, bool tr, int base, int ld, int k, float (&v)[4]) {
    if (tr) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        v[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, k + e < k_end ? base + (k + e) * ld * 4 : OOB, 0, 0));
    } else {   // K is a multiple of 4 here
      const u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(rs, k < k_end ? base + 4 * k : OOB, 0, 0);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = __uint_as_float(w[e]);
    }
  };
  auto load_set = [&](int k0, F32Frags<R>& f) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = k0 + 8 * u + 4 * h;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        load_one(rsA, AT, a_base[r], p.lda, k, f.a[u][r]);
        load_one(rsB, BT, b_base[r], p.ldb, k, f.b[u][r]);
      }
    }
  };
  f32x16 acc[R][R];
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int j = 0; j < R; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
  const bool do_colsum = BT && p.colsum != nullptr && m0 == 0;
  float csum[R] = {};
  auto multiply = [&](const F32Frags<R>& f) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
          for (int j = 0; j < R; ++j)   // B first: a lane then holds 4 consecutive columns of one row of C
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(f.b[u][j][e], f.a[u][i][e], acc[i][j], 0, 0, 0);
        if (do_colsum) {
#pragma unroll
          for (int j = 0; j < R; ++j) csum[j] += f.b[u][j][e];
        }
      }
  };
  F32Frags<R> f0, f1;
  load_set(k_beg, f0);
  for (int k = k_beg; k < k_end; k += 16 * U) {   // sets past the wave's range read as zeros
    load_set(k + 8 * U, f1);
    multiply(f0);
    load_set(k + 16 * U, f0);
    multiply(f1);
  }
  constexpr int LD = part_ld<R>(), T = 32 * R;
  float* part = f32_smem;                          // [4][T][LD]
  float* cs = part + 4 * T * LD;                   // [4][T]
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int j = 0; j < R; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<float4*>(part + (wave * T + 32 * i + row) * LD + 32 * j + 8 * q + 4 * h) =
            make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
  if (do_colsum) {
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const float t = csum[j] + __shfl_xor(csum[j], 32, 64);
      if (h == 0) cs[wave * T + 32 * j + row] = t;
    }
  }
  __syncthreads();
  if (do_colsum && tid < T && n0 + tid < p.N) p.colsum[n0 + tid] = (cs[tid] + cs[T + tid]) + (cs[2 * T + tid] + cs[3 * T + tid]);
  constexpr int TPR = T / 4;                       // threads per row of the tile, four columns each
  const int nn = (tid % TPR) * 4, n = n0 + nn;
  if (n >= p.N) return;                            // N is a multiple of 4
#pragma unroll
  for (int pass = 0; pass < T / (256 / TPR); ++pass) {
    const int mm = pass * (256 / TPR) + tid / TPR, m = m0 + mm;
    if (m >= p.M) break;
    float4 t = *reinterpret_cast<const float4*>(part + mm * LD + nn);
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      const float4 x = *reinterpret_cast<const float4*>(part + (w * T + mm) * LD + nn);
      t.x += x.x; t.y += x.y; t.z += x.z; t.w += x.w;
    }
    if (p.bias) {
      const float4 b = *reinterpret_cast<const float4*>(p.bias + n);
      t.x += b.x; t.y += b.y; t.z += b.z; t.w += b.w;
    }
    if (p.residual) {
      const float4 b = *reinterpret_cast<const float4*>(p.residual + (size_t)m * p.ldr + n);
      t.x += b.x; t.y += b.y; t.z += b.z; t.w += b.w;
    }
    float4* c = reinterpret_cast<float4*>(p.C + (size_t)m * p.ldc + n);
    if (p.epilogue == EPI_GELU) {                  // C2 = gelu(h), C = gelu'(h)
      const float hv[4] = {t.x, t.y, t.z, t.w};
      float g[4], d[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float cdf = 0.5f * (1.0f + erff(hv[e] * 0.70710678118654752f));
        g[e] = hv[e] * cdf;
        d[e] = cdf + hv[e] * (0.39894228040143268f * __expf(-0.5f * hv[e] * hv[e]));
      }
      *c = make_float4(d[0], d[1], d[2], d[3]);
      *reinterpret_cast<float4*>(p.C2 + (size_t)m * p.ldc + n) = make_float4(g[0], g[1], g[2], g[3]);
    } else if (p.epilogue == EPI_DGELU) {
      const float4 x = *reinterpret_cast<const float4*>(p.aux + (size_t)m * p.ldaux + n);
      *c = make_float4(t.x * x.x, t.y * x.y, t.z * x.z, t.w * x.w);
    } else {
      *c = t;
    }
  }
}

template <bool BT, int R>
__global__ __launch_bounds__(256) void gemm_f32_kernel(F32Args p) {
  gemm_f32_tile<false, BT, R>(p, (int)blockIdx.y * 32 * R, (int)blockIdx.x * 32 * R);
}

// Weight and bias gradients of several layers: C_j = A_j^T B_j with both operands stored [K][.].
struct F32Problem { const float* A; const float* B; float* C; float* colsum; int lda, ldb, ldc, M, N, K, tiles_n, first_tile; uint32_t a_bytes, b_bytes; };
constexpr int F32_GROUP_MAX = 40;
struct F32Group { int n; F32Problem prob[F32_GROUP_MAX]; };
template <int R>
__global__ __launch_bounds__(256) void gemm_f32_grouped_kernel(F32Group a) {
  const int t = blockIdx.x;
  int j = 0;
  while (j + 1 < a.n && t >= a.prob[j + 1].first_tile) ++j;
  const F32Problem& q = a.prob[j];
  F32Args p{};
  p.A = q.A; p.B = q.B; p.C = q.C; p.colsum = q.colsum; p.lda = q.lda; p.ldb = q.ldb; p.ldc = q.ldc;
  p.M = q.M; p.N = q.N; p.K = q.K; p.a_bytes = q.a_bytes; p.b_bytes = q.b_bytes;
  const int local = t - q.first_tile;
  gemm_f32_tile<true, true, R>(p, (local / q.tiles_n) * 32 * R, (local % q.tiles_n) * 32 * R);
}

bool al16(const void* p) { return (((uintptr_t)p) & 15) == 0; }
long f32_bytes(bool tr, int rows, int K, long ld) { return 4 * (tr ? (long)(K - 1) * ld + rows : (long)(rows - 1) * ld + K); }
long tiles_of(int M, int N, int edge) { return (long)((M + edge - 1) / edge) * ((N + edge - 1) / edge); }
}  // namespace

bool gemm_f32_supported(const GemmArgs& g) {
  if (g.a_dt != F32 || g.b_dt != F32 || g.c_dt != F32 || g.M < 1 || g.N < 1 || g.K < 1) return false;
  const bool at = g.a_sm == 1 && g.a_sk != 1, bt = g.b_sn == 1 && g.b_sk != 1;
  if ((!at && g.a_sk != 1) || (!bt && g.b_sk != 1)) return false;
  const long lda = at ? g.a_sk : g.a_sm, ldb = bt ? g.b_sk : g.b_sn;
  // 16-byte accesses: along k where k is contiguous, along the rows of C always
  if (!at && ((lda & 3) || (g.K & 3) || !al16(g.A))) return false;
  if (!bt && ((ldb & 3) || (g.K & 3) || !al16(g.B))) return false;
  if ((g.N & 3) || (g.ldc & 3) || !al16(g.C)) return false;
  if (g.bias && !al16(g.bias)) return false;
  if (g.residual && (g.r_dt != F32 || (g.ldr & 3) || !al16(g.residual))) return false;
  if (g.epilogue == EPI_GELU && (!g.C2 || !al16(g.C2))) return false;
  if (g.epilogue == EPI_DGELU && (g.aux_dt != F32 || (g.ldaux & 3) || !al16(g.aux))) return false;
  const long lim = (1L << 30) - 64;
  return f32_bytes(at, g.M, g.K, lda) <= lim && f32_bytes(bt, g.N, g.K, ldb) <= lim && g.ldc < (1L << 31) && g.ldr < (1L << 31) && g.ldaux < (1L << 31);
}
bool gemm_f32_groupable(const GemmArgs& g) {
  if (!gemm_f32_supported(g)) return false;
  const bool at = g.a_sm == 1 && g.a_sk != 1, bt = g.b_sn == 1 && g.b_sk != 1;
  return at && bt && !g.bias && !g.residual && g.epilogue == EPI_NONE;
}

// 64 x 64 tiles (half the operand traffic) once they give every compute unit a workgroup
static long f32_units() { const int units = compute_units(); return units > 0 ? units : 256; }

template <bool BT, int R>
static int f32_launch(hipStream_t s, const F32Args& p) {
  static OncePerDevice once;
  PPLL_TRY(raise_lds((const void*)gemm_f32_kernel<BT, R>, f32_lds_bytes<R>(), once));
  hipLaunchKernelGGL((gemm_f32_kernel<BT, R>), dim3((p.N + 32 * R - 1) / (32 * R), (p.M + 32 * R - 1) / (32 * R)), dim3(256), f32_lds_bytes<R>(), s, p);
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}
int launch_gemm_f32(hipStream_t s, const GemmArgs& g) {
  if (g.a_sk != 1 || g.colsum) { set_error("launch_gemm_f32: A stored [K][M] and column sums are for sets of weight gradients"); return PPLL_ERR_CONFIG; }
  const bool bt = g.b_sn == 1 && g.b_sk != 1;
  F32Args p{};
  p.A = (const float*)g.A; p.B = (const float*)g.B; p.C = (float*)g.C;
  p.lda = (int)g.a_sm; p.ldb = (int)(bt ? g.b_sk : g.b_sn); p.ldc = (int)g.ldc;
  p.M = g.M; p.N = g.N; p.K = g.K; p.bias = g.bias; p.residual = (const float*)g.residual; p.ldr = (int)g.ldr;
  p.epilogue = g.epilogue; p.C2 = (float*)g.C2; p.aux = (const float*)g.aux; p.ldaux = (int)g.ldaux;
  p.a_bytes = (uint32_t)f32_bytes(false, g.M, g.K, p.lda); p.b_bytes = (uint32_t)f32_bytes(bt, g.N, g.K, p.ldb);
  if (tiles_of(g.M, g.N, 64) >= f32_units()) return bt ? f32_launch<true, 2>(s, p) : f32_launch<false, 2>(s, p);
  return bt ? f32_launch<true, 1>(s, p) : f32_launch<false, 1>(s, p);
}

int launch_gemm_f32_grouped(hipStream_t s, const GemmArgs* gs, int n) {
  static OncePerDevice once;
  PPLL_TRY(raise_lds((const void*)gemm_f32_grouped_kernel<2>, f32_lds_bytes<2>(), once));
  for (int j0 = 0; j0 < n; j0 += F32_GROUP_MAX) {
    F32Group a{};
    a.n = n - j0 < F32_GROUP_MAX ? n - j0 : F32_GROUP_MAX;
    long wide_tiles = 0;
    for (int j = 0; j < a.n; ++j) wide_tiles += tiles_of(gs[j0 + j].M, gs[j0 + j].N, 64);
    const bool wide = wide_tiles >= 2 * f32_units();   // the reduction is the long side here: more waves first
    const int edge = wide ? 64 : 32;
    int tiles = 0;
    for (int j = 0; j < a.n; ++j) {
      const GemmArgs& g = gs[j0 + j];
      F32Problem& q = a.prob[j];
      q.A = (const float*)g.A; q.B = (const float*)g.B; q.C = (float*)g.C; q.colsum = g.colsum;
      q.lda = (int)g.a_sk; q.ldb = (int)g.b_sk; q.ldc = (int)g.ldc; q.M = g.M; q.N = g.N; q.K = g.K;
      q.a_bytes = (uint32_t)f32_bytes(true, g.M, g.K, q.lda); q.b_bytes = (uint32_t)f32_bytes(true, g.N, g.K, q.ldb);
      q.tiles_n = (g.N + edge - 1) / edge; q.first_tile = tiles;
      tiles += (int)tiles_of(g.M, g.N, edge);
    }
    if (wide) hipLaunchKernelGGL(gemm_f32_grouped_kernel<2>, dim3(tiles), dim3(256), f32_lds_bytes<2>(), s, a);
    else hipLaunchKernelGGL(gemm_f32_grouped_kernel<1>, dim3(tiles), dim3(256), f32_lds_bytes<1>(), s, a);
    PPLL_HIP(hipGetLastError());
  }
  return PPLL_OK;
}

// ===================================================================== attention
// Any head size and element type, T up to 256.  A workgroup takes ATT_ROWS query rows (keys in the second half of the
// backward) of one (batch, head), 16 lanes each; the rows they are compared with lie in LDS as fp32, 4 floats apart from a
// multiple of 16 so that 16 lanes reading 16 rows hit different banks.  One workgroup per (batch, head) walking all its
// rows is 32 workgroups at batch 8: 73 us forward and 190 us backward at 65 tokens, 16-wide heads.  That kernel keeps the shapes
// with many heads whose rows leave one of these workgroups a unit, see att_by_rows.
namespace {
__device__ __forceinline__ float4 ld4(const void* p, size_t i, int dt, int left) {   // elements i .. i+3, zero beyond `left`
  if (left >= 4) {
    if (dt == F32 && !((i | ((uintptr_t)p >> 2)) & 3)) return *reinterpret_cast<const float4*>((const float*)p + i);
    return make_float4(ld_f(p, i, dt), ld_f(p, i + 1, dt), ld_f(p, i + 2, dt), ld_f(p, i + 3, dt));
  }
  return make_float4(ld_f(p, i, dt), left > 1 ? ld_f(p, i + 1, dt) : 0.f, left > 2 ? ld_f(p, i + 2, dt) : 0.f, 0.f);
}
__device__ __forceinline__ float sum16(float v) {
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float max16(float v) {
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ float dot4(const float* a, const float* b, int q4) {
  float s = 0.f;
  for (int q = 0; q < q4; ++q) {
    const float4 x = *reinterpret_cast<const float4*>(a + 4 * q), y = *reinterpret_cast<const float4*>(b + 4 * q);
    s = fmaf(x.x, y.x, s); s = fmaf(x.y, y.y, s); s = fmaf(x.z, y.z, s); s = fmaf(x.w, y.w, s);
  }
  return s;
}
// rows 0 .. n-1 of a matrix with row stride ld, starting at element `base`, into LDS
__device__ __forceinline__ void stage_rows(float* dst, const void* src, size_t base, long ld, int dt, int n, const AttShape& a) {
  for (int i = threadIdx.x; i < n * a.q4; i += 256) {
    const int t = i / a.q4, q = i - t * a.q4;
    *reinterpret_cast<float4*>(dst + t * a.pitch + 4 * q) = ld4(src, base + (size_t)t * ld + 4 * q, dt, a.dh - 4 * q);
  }
}

__global__ __launch_bounds__(256) void attn_rows_fwd_kernel(const void* qkv, int dt, int T, int H, int dh, void* out, float* lse) {
  extern __shared__ __align__(16) float f32_smem[];
  const AttShape a = att_shape(T, H, dh);
  float* Ks = f32_smem;
  float* Vs = Ks + T * a.pitch;
  float* Qs = Vs + T * a.pitch;             // [ATT_ROWS]
  float* ps = Qs + ATT_ROWS * a.pitch;      // [ATT_ROWS][tp]
  const int b = blockIdx.x / H, h = blockIdx.x % H, D = H * dh, i0 = blockIdx.y * ATT_ROWS;
  const int g = threadIdx.x >> 4, l = threadIdx.x & 15, i = i0 + g;
  const size_t base = (size_t)b * T * 3 * D + h * dh;
  stage_rows(Ks, qkv, base + D, 3 * D, dt, T, a);
  stage_rows(Vs, qkv, base + 2 * D, 3 * D, dt, T, a);
  stage_rows(Qs, qkv, base + (size_t)i0 * 3 * D, 3 * D, dt, min(ATT_ROWS, T - i0), a);
  __syncthreads();
  if (i >= T) return;                       // a row's 16 lanes leave together; no barrier follows
  const float scale = rsqrtf((float)dh);
  float* p = ps + g * a.tp;
  float mx = -INFINITY;
  for (int j = l; j < T; j += 16) {
    const float s = dot4(Qs + g * a.pitch, Ks + j * a.pitch, a.q4) * scale;
    p[j] = s;
    mx = fmaxf(mx, s);
  }
  mx = max16(mx);
  float se = 0.f;
  for (int j = l; j < T; j += 16) { const float e = __expf(p[j] - mx); p[j] = e; se += e; }
  se = sum16(se);
  const float inv = 1.0f / se;
  wave_sync();
  for (int d = l; d < dh; d += 16) {
    float o = 0.f;
    int j = 0;
    for (; j + 4 <= T; j += 4) {
      const float4 w = *reinterpret_cast<const float4*>(p + j);
      const float* v = Vs + j * a.pitch + d;
      o = fmaf(w.x, v[0], o); o = fmaf(w.y, v[a.pitch], o); o = fmaf(w.z, v[2 * a.pitch], o); o = fmaf(w.w, v[3 * a.pitch], o);
    }
    for (; j < T; ++j) o = fmaf(p[j], Vs[j * a.pitch + d], o);
    st_f(out, ((size_t)b * T + i) * D + h * dh + d, o * inv, dt);
  }
  if (l == 0) lse[((size_t)b * H + h) * T + i] = mx + __logf(se);
}

// blockIdx.y even: query rows (dQ = scale dS K), odd: keys (dV = P^T dO, dK = scale dS^T Q); P from the saved
// log-sum-exp, dS = P o (dO V^T - <dO, O>).
__global__ __launch_bounds__(256) void attn_rows_bwd_kernel(const void* qkv, const void* out, const void* dout, const float* lse,
                                                            int dt, int T, int H, int dh, void* dqkv) {
  extern __shared__ __align__(16) float f32_smem[];
  const AttShape a = att_shape(T, H, dh);
  float* As = f32_smem;                     // queries: K, keys: Q
  float* Bs = As + T * a.pitch;             // queries: V, keys: dO
  float* own0 = Bs + T * a.pitch;           // q_i / k_j
  float* own1 = own0 + ATT_ROWS * a.pitch;  // dO_i / v_j
  float* ps = own1 + ATT_ROWS * a.pitch;    // [ATT_ROWS][tp] P (keys only)
  float* ds = ps + ATT_ROWS * a.tp;         // [ATT_ROWS][tp] dS
  float* Ls = ds + ATT_ROWS * a.tp;         // [T] log-sum-exp
  float* Dr = Ls + T;                       // [T] <dO, O>
  const int b = blockIdx.x / H, h = blockIdx.x % H, D = H * dh, i0 = (blockIdx.y >> 1) * ATT_ROWS;
  const bool keys = blockIdx.y & 1;
  const int g = threadIdx.x >> 4, l = threadIdx.x & 15, i = i0 + g, rows = min(ATT_ROWS, T - i0);
  const size_t base = (size_t)b * T * 3 * D + h * dh, obase = (size_t)b * T * D + h * dh;
  const float scale = rsqrtf((float)dh);
  stage_rows(As, qkv, base + (keys ? 0 : D), 3 * D, dt, T, a);
  if (keys) stage_rows(Bs, dout, obase, D, dt, T, a);
  else stage_rows(Bs, qkv, base + 2 * D, 3 * D, dt, T, a);
  stage_rows(own0, qkv, base + (size_t)i0 * 3 * D + (keys ? D : 0), 3 * D, dt, rows, a);
  if (keys) stage_rows(own1, qkv, base + (size_t)i0 * 3 * D + 2 * D, 3 * D, dt, rows, a);
  else stage_rows(own1, dout, obase + (size_t)i0 * D, D, dt, rows, a);
  for (int t = threadIdx.x; t < T; t += 256) Ls[t] = lse[((size_t)b * H + h) * T + t];
  // row dots: of the workgroup's own queries, or of all queries
  for (int t = keys ? g : i; t < T; t += keys ? 16 : T) {
    float s = 0.f;
    for (int d = l; d < dh; d += 16) s += ld_f(dout, obase + (size_t)t * D + d, dt) * ld_f(out, obase + (size_t)t * D + d, dt);
    s = sum16(s);
    if (l == 0) Dr[t] = s;
  }
  __syncthreads();
  if (i >= T) return;                       // as above
  const float* o0 = own0 + g * a.pitch;
  const float* o1 = own1 + g * a.pitch;
  float *p = ps + g * a.tp, *e = ds + g * a.tp;
  for (int j = l; j < T; j += 16) {
    const float s = dot4(o0, As + j * a.pitch, a.q4), dp = dot4(o1, Bs + j * a.pitch, a.q4);
    const float pj = __expf(s * scale - (keys ? Ls[j] : Ls[i]));
    if (keys) p[j] = pj;
    e[j] = pj * (dp - (keys ? Dr[j] : Dr[i]));
  }
  wave_sync();
  const size_t ob = base + (size_t)i * 3 * D;
  for (int d = l; d < dh; d += 16) {
    float x = 0.f, y = 0.f;
    if (keys) {
      for (int j = 0; j < T; ++j) { y = fmaf(p[j], Bs[j * a.pitch + d], y); x = fmaf(e[j], As[j * a.pitch + d], x); }
      st_f(dqkv, ob + D + d, x * scale, dt);
      st_f(dqkv, ob + 2 * D + d, y, dt);
    } else {
      for (int j = 0; j < T; ++j) x = fmaf(e[j], As[j * a.pitch + d], x);
      st_f(dqkv, ob + d, x * scale, dt);
    }
  }
}

}  // namespace

int launch_attention_rows_fwd(hipStream_t s, const void* qkv, int dt, int B, int T, int H, int dh, void* out, float* lse) {
  const size_t lds = att_rows_lds(att_shape(T, H, dh), false);
  static OncePerDevice once;
  PPLL_TRY(raise_lds((const void*)attn_rows_fwd_kernel, UNIT_LDS, once));
  hipLaunchKernelGGL(attn_rows_fwd_kernel, dim3(B * H, (T + ATT_ROWS - 1) / ATT_ROWS), dim3(256), lds, s, qkv, dt, T, H, dh, out, lse);
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}
int launch_attention_rows_bwd(hipStream_t s, const void* qkv, const void* out, const void* dout, const float* lse, int dt, int B,
                              int T, int H, int dh, void* dqkv) {
  const size_t lds = att_rows_lds(att_shape(T, H, dh), true);
  static OncePerDevice once;
  PPLL_TRY(raise_lds((const void*)attn_rows_bwd_kernel, UNIT_LDS, once));
  hipLaunchKernelGGL(attn_rows_bwd_kernel, dim3(B * H, 2 * ((T + ATT_ROWS - 1) / ATT_ROWS)), dim3(256), lds, s, qkv, out, dout, lse,
                     dt, T, H, dh, dqkv);
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}

}  // namespace ppll
