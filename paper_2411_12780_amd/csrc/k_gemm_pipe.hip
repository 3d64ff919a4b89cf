// Linear-layer products with many output tiles: C[M,N] = A[M,K] B, bf16 operands, fp32 accumulation, the epilogues of the
// tiled kernel, bit-identical results (the same order of k).
//
// The tiled kernel is held by the data movement of a 128 x 128 tile: 32 KB into LDS and 96 KB of LDS traffic per 64 k, through
// registers, a wave reading 64 x 64.  Here operands go straight to LDS, and the fragment reads of a k step run under the products of the
// one before.  Three forms (the rules are in plan.h), a wave owning 128 x 64 or 160 x 64 in the first two:
//  128 x 256 or 160 x 256 tiles of four waves, three stages of 32 k, two workgroups a unit (72 or 78 KB of LDS each), so that one
//    stores its tile under the other's products: where the epilogue is long or tiles are few;
//  256 x 256 or 320 x 256 tiles of eight waves, two stages of 64 k, a unit to themselves (128 or 144 KB): a third less to bring into LDS,
//    and rows of 128 bytes of an operand with k contiguous.  Rows of 64 bytes come from L2 at 26 bytes a clock and unit, whole cache
//    lines at 52; brought 64 bytes a row, the copies of 25216 x 768 x 3072 alone took 76 us, whole lines 72 from HBM and 47 from L2.
//  128 x 128 tiles of four waves that multiply, 64 x 64 each, and four that copy, four stages of 64 k, a unit to themselves (128 KB): where
//    every tile finds a unit.  Units left over bring rows of A, columns of B and what the epilogue takes into L2 ahead of the tiles.
//    Tiled kernel -> without that -> with it, B [K][N], bias and residual, us a launch behind others on other operands, from memory (in
//    brackets: from the last-level cache): 8320 x 384 x 1536 21.2 -> 21.2 -> 18.2 (18.6 -> 14.2 -> 13.7), x 384 10.6 -> 10.1 -> 9.7 (9.0 ->
//    8.0 -> 7.6), 5200 x 384 x 1536 19.6 -> 19.8 -> 14.5 (17.9 -> 13.5 -> 12.6), 4160 x 768 x 3072 34.3 -> 32.8 -> 26.1 (30.9 -> 22.7 -> 23.0);
//    B [N][K], neither: 8320 x 384 x 1536 21.4 -> 19.9 -> 17.2 (18.3 -> 13.7 -> 13.3), x 1152 16.8 -> 15.8 -> 13.9 (14.6 -> 11.2 -> 11.0).
// Microseconds, tiled kernel -> first form -> second: 25216 x 768 x 3072 138 -> 117 -> 100 (1192 TFLOP/s), 25216 x 2304 x 768 132 -> 105 ->
// 93, 25216 x 3072 x 768 with GELU 198 -> 172 -> 162 and with its derivative 182 -> 165 -> 151 (310 MB of epilogue traffic each),
// 8320 x 1152 x 384 16.8 -> 16.4 -> 14.8, 8320 x 1536 x 384 with GELU 27.9 -> 24.8 -> 24.0.  What bounds it: in the main loop LDS reads and
// products, which take 85 of those 100 us without any copies and 68 without the reads as well; the epilogue where K is short.
#include "common.h"
#include "gemm_pipe.h"
#include "plan.h"

namespace ppll {

namespace {
using namespace pipe;

struct PipeArgs {
  const uint16_t* A; long lda;      // A[m*lda + k]
  const uint16_t* B; long ldb;      // BT ? B[k*ldb + n] : B[n*ldb + k]
  uint16_t* C; long ldc;
  int M, N, K;
  TileMap map;
  int helpers;                      // workgroups an XCD that have no tile
  const float* bias;
  const uint16_t* residual; long ldr;
  int epilogue;
  uint16_t* C2;
  const uint16_t* aux; long ldaux;
  uint32_t a_bytes, b_bytes, c_bytes, r_bytes, aux_bytes;
};

__device__ __forceinline__ u32x4 pipe_load16(__amdgpu_buffer_rsrc_t r, int off) { return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0); }
__device__ __forceinline__ u32x4 pack8(const float (&v)[8]) {
  return (u32x4){f32x2_to_bf16x2(v[0], v[1]), f32x2_to_bf16x2(v[2], v[3]), f32x2_to_bf16x2(v[4], v[5]), f32x2_to_bf16x2(v[6], v[7])};
}

template <bool BT, int WGM, int WGN, int IM, int NS, int KT>
__global__ __launch_bounds__((Shape<false, BT, WGM, WGN, IM, NS, KT>::THREADS), 2) void gemm_pipe_kernel(PipeArgs p) {
  PPLL_CODE_TO_L2(4);
  using S = Shape<false, BT, WGM, WGN, IM, NS, KT>;
  constexpr int JN = 2;
  extern __shared__ __align__(1024) char smem[];
  const int slot = blockIdx.x >> 3;
  int tm, tn;
  if (S::COPY_WAVES && slot >= p.map.per_xcd) {
    const Bring b{p.A, p.B, p.residual, p.a_bytes, p.b_bytes, p.r_bytes, (int)(p.lda * 2), (int)(p.ldb * 2), (int)(p.ldr * 2), p.M, p.N, p.K, S::BM, S::BN, p.helpers};
    bring_operands<BT, S::THREADS>(b, p.map, blockIdx.x & 7, slot - p.map.per_xcd, (lds_char*)code_words__);
    return;
  }
  if (S::COPY_WAVES) {
    if (!tile_at(p.map, blockIdx.x & 7, slot, tm, tn)) return;
  } else {
    // XCD x (workgroup id % 8) takes a contiguous range of the tiles, row by row: they share operand panels in its L2
    const int t = (blockIdx.x & 7) * p.map.per_xcd + slot;
    tm = t / p.map.tiles_n;
    tn = t % p.map.tiles_n;
    if (slot >= p.map.per_xcd || tm >= p.map.tiles_m) return;
  }
  const int m0 = tm * S::BM, n0 = tn * S::BN;
  f32x16 acc[JN][IM];
  float none[JN][8];
#pragma unroll
  for (int j = 0; j < JN; ++j)
#pragma unroll
    for (int i = 0; i < IM; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[j][i][e] = 0.f;
  multiply<S, false, BT, false>(make_rsrc(p.A, p.a_bytes), make_rsrc(p.B, p.b_bytes), p.lda, p.ldb, m0, n0, p.M, p.N, p.K,
                                (lds_char*)smem, acc, none, false);
  if (S::COPY_WAVES && threadIdx.x >= 64 * S::W) return;

  // Epilogue: a wave passes its accumulators (lane = one row, 4 consecutive columns a group) through its own piece of LDS, 32 rows
  // at a time, and takes them out 8 consecutive columns a lane; what a piece needs from memory is asked for one piece ahead.
  constexpr int COLS = JN * 32, PITCH = COLS + 4, LPR = COLS / 8, RPP = 64 / LPR, NP = 32 / RPP;
  static_assert(S::W * 32 * PITCH * 4 <= S::LDS, "");
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float* st = reinterpret_cast<float*>(smem) + wave * 32 * PITCH;
  const int mw = m0 + wave / WGN * IM * 32, c8 = lane % LPR * 8, n = n0 + wave % WGN * COLS + c8, r0 = lane / LPR;
  const int col2 = n < p.N ? 2 * n : OOB_BASE;
  float bias[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (p.bias) {
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(p.bias, (uint32_t)p.N * 4u);
    const u32x4 lo = pipe_load16(rs, 2 * col2), hi = pipe_load16(rs, 2 * col2 + 16);
#pragma unroll
    for (int e = 0; e < 4; ++e) { bias[e] = __uint_as_float(lo[e]); bias[4 + e] = __uint_as_float(hi[e]); }
  }
  const bool has_res = p.residual != nullptr, has_aux = p.epilogue == EPI_DGELU;
  const __amdgpu_buffer_rsrc_t rsR = make_rsrc(p.residual, p.r_bytes), rsX = make_rsrc(p.aux, p.aux_bytes);
  const __amdgpu_buffer_rsrc_t rsC = make_rsrc(p.C, p.c_bytes), rsC2 = make_rsrc(p.C2, p.C2 ? p.c_bytes : 0u);
  u32x4 res[2][NP], aux[2][NP];
  auto ask = [&](int im, u32x4 (&r)[NP], u32x4 (&x)[NP]) {
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      const int m = mw + im * 32 + q * RPP + r0;
      if (has_res) r[q] = pipe_load16(rsR, m < p.M ? (int)(m * p.ldr * 2) + col2 : OOB);
      if (has_aux) x[q] = pipe_load16(rsX, m < p.M ? (int)(m * p.ldaux * 2) + col2 : OOB);
    }
  };
  ask(0, res[0], aux[0]);
#pragma unroll
  for (int im = 0; im < IM; ++im) {
    if (im + 1 < IM) ask(im + 1, res[(im + 1) & 1], aux[(im + 1) & 1]);
#pragma unroll
    for (int jn = 0; jn < JN; ++jn)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<float4*>(st + (lane & 31) * PITCH + jn * 32 + 8 * q + 4 * (lane >> 5)) =
            make_float4(acc[jn][im][4 * q], acc[jn][im][4 * q + 1], acc[jn][im][4 * q + 2], acc[jn][im][4 * q + 3]);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      const int m = mw + im * 32 + q * RPP + r0;
      const float4 lo = *reinterpret_cast<const float4*>(st + (q * RPP + r0) * PITCH + c8);
      const float4 hi = *reinterpret_cast<const float4*>(st + (q * RPP + r0) * PITCH + c8 + 4);
      float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] += bias[e];
      if (has_res) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t w = res[im & 1][q][e];
          v[2 * e] += __uint_as_float(w << 16); v[2 * e + 1] += __uint_as_float(w & 0xffff0000u);
        }
      }
      if (has_aux) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {   // the saved GELU derivative
          const uint32_t w = aux[im & 1][q][e];
          v[2 * e] *= __uint_as_float(w << 16); v[2 * e + 1] *= __uint_as_float(w & 0xffff0000u);
        }
      }
      const int off = m < p.M ? (int)(m * p.ldc * 2) + col2 : OOB;
      if (p.epilogue == EPI_GELU) {   // C2 = gelu(h), C = gelu'(h) from one evaluation of the normal CDF and density
        float dg[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          float cdf, pdf;
          cdf_pdf(v[e], cdf, pdf);
          dg[e] = cdf + v[e] * pdf; v[e] *= cdf;
        }
        __builtin_amdgcn_raw_buffer_store_b128(pack8(dg), rsC, off, 0, THROUGH);
        __builtin_amdgcn_raw_buffer_store_b128(pack8(v), rsC2, off, 0, THROUGH);
      } else {
        __builtin_amdgcn_raw_buffer_store_b128(pack8(v), rsC, off, 0, THROUGH);
      }
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
  }
}

template <bool BT, int WGM, int IM, int STAGES, int KT, int WAVES_N = 4>
int pipe_launch(hipStream_t s, PipeArgs& p, int units = 0) {
  using S = Shape<false, BT, WGM, WAVES_N, IM, STAGES, KT>;
  if (S::COPY_WAVES) {
    p.map = tile_map(p.M, p.N, S::BM, S::BN, units);
    p.helpers = helper_workgroups(p.map.per_xcd, units);
  } else {
    const int tiles_m = (p.M + S::BM - 1) / S::BM, tiles_n = (p.N + S::BN - 1) / S::BN;
    p.map = TileMap{tiles_m, tiles_n, (int)(((long)tiles_m * tiles_n + 7) / 8), 0, 0, 0, false};
  }
  static OncePerDevice once;
  PPLL_TRY(raise_lds((const void*)gemm_pipe_kernel<BT, WGM, WAVES_N, IM, STAGES, KT>, S::LDS, once));
  hipLaunchKernelGGL((gemm_pipe_kernel<BT, WGM, WAVES_N, IM, STAGES, KT>), dim3(8 * (p.map.per_xcd + p.helpers)), dim3(S::THREADS), S::LDS, s, p);
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}

}  // namespace

bool gemm_pipe_supported(const GemmArgs& g) {
  if (!gemm_mfma_supported(g) || g.a_sk != 1 || g.colsum || g.c_dt != BF16 || g.K < PIPE_MIN_K) return false;
  const bool bt = g.b_sn == 1 && g.b_sk != 1;
  // 32-bit byte offsets also for the rows (k rows) of the last tile that do not exist
  return g.a_sm <= (1 << 20) && (bt ? g.b_sk : g.b_sn) <= (1 << 20);
}
int gemm_pipe_choice(const GemmArgs& g) {
  if (!gemm_pipe_supported(g)) return 0;
  const ProductEnd end = g.epilogue == EPI_GELU ? END_GELU : g.epilogue == EPI_DGELU ? END_DGELU : g.residual ? END_RESIDUAL : g.bias ? END_BIAS : END_PLAIN;
  const int units = product_units(g);
  if (!g.shared && copy_wave_tiles(g.M, g.N, g.K, units)) return 3;
  const int wide = wide_tile_rows(g.M, g.N, g.K, end, units), alone = unit_tile_rows(g.M, g.N, g.K, end, wide, units);
  return alone ? alone : wide;
}

int launch_gemm_pipe(hipStream_t s, const GemmArgs& g, int im) {
  const bool bt = g.b_sn == 1 && g.b_sk != 1;
  PipeArgs p{};
  p.A = (const uint16_t*)g.A; p.lda = g.a_sm;
  p.B = (const uint16_t*)g.B; p.ldb = bt ? g.b_sk : g.b_sn;
  p.C = (uint16_t*)g.C; p.ldc = g.ldc;
  p.M = g.M; p.N = g.N; p.K = g.K;
  p.bias = g.bias; p.residual = (const uint16_t*)g.residual; p.ldr = g.ldr;
  p.epilogue = g.epilogue; p.C2 = (uint16_t*)g.C2; p.aux = (const uint16_t*)g.aux; p.ldaux = g.ldaux;
  p.a_bytes = (uint32_t)(((long)(g.M - 1) * p.lda + g.K) * 2);
  p.b_bytes = (uint32_t)((bt ? (long)(g.K - 1) * p.ldb + g.N : (long)(g.N - 1) * p.ldb + g.K) * 2);
  p.c_bytes = (uint32_t)(((long)(g.M - 1) * g.ldc + g.N) * 2);
  p.r_bytes = g.residual ? (uint32_t)(((long)(g.M - 1) * g.ldr + g.N) * 2) : 0u;
  p.aux_bytes = g.epilogue == EPI_DGELU ? (uint32_t)(((long)(g.M - 1) * g.ldaux + g.N) * 2) : 0u;
  void* prof = nullptr;
  PPLL_TRY(profile_begin(s, 2.0 * g.M * g.N * g.K, &prof));
  if (im == 3) PPLL_TRY((bt ? pipe_launch<true, 2, 2, 4, 64, 2>(s, p, product_units(g)) : pipe_launch<false, 2, 2, 4, 64, 2>(s, p, product_units(g))));
  else if (im == 4) PPLL_TRY((bt ? pipe_launch<true, 1, 4, 3, 32>(s, p) : pipe_launch<false, 1, 4, 3, 32>(s, p)));
  else if (im == 5) PPLL_TRY((bt ? pipe_launch<true, 1, 5, 3, 32>(s, p) : pipe_launch<false, 1, 5, 3, 32>(s, p)));
  else if (im == 8) PPLL_TRY((bt ? pipe_launch<true, 2, 4, 2, 64>(s, p) : pipe_launch<false, 2, 4, 2, 64>(s, p)));
  else PPLL_TRY((bt ? pipe_launch<true, 2, 5, 2, 64>(s, p) : pipe_launch<false, 2, 5, 2, 64>(s, p)));
  return profile_end(s, prof);
}

}  // namespace ppll
