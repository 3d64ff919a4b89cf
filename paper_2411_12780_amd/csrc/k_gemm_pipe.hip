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
//    every tile finds a unit.  Units left over bring A into L2 ahead of the tiles.  Operands from beyond L2, tiled kernel -> without that
//    -> with it: 8320 x 384 x 1536 21.4 -> 19.3 -> 15.8, x 1152 17.0 -> 15.2 -> 12.7, 8320 x 384 x 384 with a residual 10.5 -> 10.0 -> 9.6;
//    5200 x 384 x 1536 20.1 -> 14.2, 4160 x 768 x 3072 36.5 -> 26 us.
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
  int M, N, K, tiles_n, tiles, per_xcd;
  int tiles_m;                      // 0, or tiles are numbered column by column
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

// A workgroup beyond those that have tiles brings a share of what its XCD's tiles read into the L2 there, rows of A and columns of B k by k
// ahead of them, then the residual, a word of every cache line (the words go to LDS that nothing reads, as in CodeToL2).  Tiles of a row of
// them read the same rows at the same time, and a unit has about 25 GB/s of lines on their way from beyond L2: three tiles to a row get
// through A at 1.6 TB/s.
template <bool BT, int BM, int BN, int THREADS> __device__ __forceinline__ void bring_operands(const PipeArgs& p, int helper, lds_char* to) {
  const int t0 = (blockIdx.x & 7) * p.per_xcd, t1 = min(t0 + p.per_xcd, p.tiles);
  if (t0 >= t1) return;
  const int row0 = p.tiles_m ? 0 : t0 / p.tiles_n * BM, rows = (p.tiles_m ? p.M : min(((t1 - 1) / p.tiles_n + 1) * BM, p.M)) - row0;
  const int col0 = p.tiles_m ? t0 / p.tiles_m * BN : 0, cols = (p.tiles_m ? min(((t1 - 1) / p.tiles_m + 1) * BN, p.N) : p.N) - col0;
  const int nl = (cols + 63) / 64, chunk = rows + (BT ? 64 * nl : cols), lines = chunk * ((p.K + 63) / 64);    // of 64 k, and in all
  const int lda2 = (int)(p.lda * 2), ldb2 = (int)(p.ldb * 2), ldr2 = (int)(p.ldr * 2);
  const __amdgpu_buffer_rsrc_t rsA = make_rsrc(p.A, p.a_bytes), rsB = make_rsrc(p.B, p.b_bytes), rsR = make_rsrc(p.residual, p.r_bytes);
  const int lane = threadIdx.x & 63, first = helper * THREADS + (int)(threadIdx.x & ~63), step = p.helpers * THREADS;
  for (int i0 = first; i0 < lines; i0 += step) {
    const int i = i0 + lane, c = i / chunk, r = i - c * chunk, q = r - rows;
    const int k = BT ? c * 64 + q / nl : 0;
    const int offB = BT ? k < p.K ? k * ldb2 + col0 * 2 + q % nl * 128 : OOB : (col0 + q) * ldb2 + c * 128;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsA, to, 4, i < lines && q < 0 ? (row0 + r) * lda2 + c * 128 : OOB, 0, 0, 0);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsB, to, 4, i < lines && q >= 0 ? offB : OOB, 0, 0, 0);
    wait_vm<2>();      // not so far ahead that L2 has lost it again (4160 x 768 x 3072: 26.8 us without this, 25.4)
  }
  if (p.residual)
    for (int i0 = first; i0 < rows * nl; i0 += step) {
      const int i = i0 + lane, r = i / nl;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsR, to, 4, r < rows ? (row0 + r) * ldr2 + col0 * 2 + (i - r * nl) * 128 : OOB, 0, 0, 0);
    }
  wait_vm<0>();
}

template <bool BT, int WGM, int WGN, int IM, int NS, int KT>
__global__ __launch_bounds__((Shape<false, BT, WGM, WGN, IM, NS, KT>::THREADS), 2) void gemm_pipe_kernel(PipeArgs p) {
  PPLL_CODE_TO_L2(4);
  using S = Shape<false, BT, WGM, WGN, IM, NS, KT>;
  constexpr int JN = 2;
  extern __shared__ __align__(1024) char smem[];
  // XCD x (workgroup id % 8) takes a contiguous range of the tiles, row by row, or column by column where rows are the longer: they share
  // operand panels in its L2
  const int slot = blockIdx.x >> 3, t = (blockIdx.x & 7) * p.per_xcd + slot;
  if (S::COPY_WAVES && slot >= p.per_xcd) {   // a unit without a tile
    bring_operands<BT, S::BM, S::BN, S::THREADS>(p, slot - p.per_xcd, (lds_char*)code_words__);
    return;
  }
  if (slot >= p.per_xcd || t >= p.tiles) return;
  const int m0 = (S::COPY_WAVES && p.tiles_m ? t % p.tiles_m : t / p.tiles_n) * S::BM, n0 = (S::COPY_WAVES && p.tiles_m ? t / p.tiles_m : t % p.tiles_n) * S::BN;
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
int pipe_launch(hipStream_t s, PipeArgs& p) {
  using S = Shape<false, BT, WGM, WAVES_N, IM, STAGES, KT>;
  p.tiles_n = (p.N + S::BN - 1) / S::BN;
  const int tiles_m = (p.M + S::BM - 1) / S::BM;
  p.tiles = tiles_m * p.tiles_n;
  p.tiles_m = S::COPY_WAVES && tiles_m < p.tiles_n ? tiles_m : 0;
  p.per_xcd = (p.tiles + 7) / 8;
  p.helpers = S::COPY_WAVES ? helper_workgroups(p.per_xcd, compute_units()) : 0;
  static OncePerDevice once;
  PPLL_TRY(raise_lds((const void*)gemm_pipe_kernel<BT, WGM, WAVES_N, IM, STAGES, KT>, S::LDS, once));
  hipLaunchKernelGGL((gemm_pipe_kernel<BT, WGM, WAVES_N, IM, STAGES, KT>), dim3(8 * (p.per_xcd + p.helpers)), dim3(S::THREADS), S::LDS, s, p);
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
  const int units = compute_units();
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
  if (im == 3) PPLL_TRY((bt ? pipe_launch<true, 2, 2, 4, 64, 2>(s, p) : pipe_launch<false, 2, 2, 4, 64, 2>(s, p)));
  else if (im == 4) PPLL_TRY((bt ? pipe_launch<true, 1, 4, 3, 32>(s, p) : pipe_launch<false, 1, 4, 3, 32>(s, p)));
  else if (im == 5) PPLL_TRY((bt ? pipe_launch<true, 1, 5, 3, 32>(s, p) : pipe_launch<false, 1, 5, 3, 32>(s, p)));
  else if (im == 8) PPLL_TRY((bt ? pipe_launch<true, 2, 4, 2, 64>(s, p) : pipe_launch<false, 2, 4, 2, 64>(s, p)));
  else PPLL_TRY((bt ? pipe_launch<true, 2, 5, 2, 64>(s, p) : pipe_launch<false, 2, 5, 2, 64>(s, p)));
  return profile_end(s, prof);
}

}  // namespace ppll
