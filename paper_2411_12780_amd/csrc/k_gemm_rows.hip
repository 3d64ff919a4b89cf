// Linear-layer products with few output tiles: C[M,N] = A[M,K] B[K,N], bf16 operands, fp32 accumulation (v_mfma_f32_32x32x16_bf16), the epilogues of the tiled kernel.
//
// These are the products of the last auxiliary encoder layer when only its class-token rows are computed (one row per image: M = batch)
// and all products of small batches.  They have almost no arithmetic (0.04 - 0.15 GFLOP) and a reduction index of 384 to 3072, so what
// they cost is the way of their operands: 64- or 128-row tiles give a few dozen workgroups that walk K one 64-wide step after the other.
// Here a workgroup owns a 32 x 32 (32 x 64) output tile and its four waves split K between them, each a contiguous quarter; the four
// partial tiles meet in LDS, are added in wave order (results do not depend on timing) and pass through the epilogue.
//  A wave copies its part of both operands straight into stages of its own in LDS, 64 k each and in whole cache lines, up to four stages
// on their way, and waits for nobody.  (Fragments read from memory in the MFMA's layout, 32 bytes of a line at a time, filled the L1 with
// lines that were gone before the next 32 bytes were asked for: more loads in flight made it slower.)  Units without a tile bring the
// operands into the L2s (Bring, in gemm_pipe.h), an XCD's tiles share what they read (tile_map), and what the epilogue takes is asked for
// before the products.  Two stages (64 KB a workgroup, 96 with tiles of 32 x 64) where the range of a wave is no longer, where there are more
// tiles than units, with tiles of 32 x 64, and in a pipeline, whose other streams want LDS.  There one stage, 32 and 48 KB, is no better: four
// blocks of width 768, 85 rows 1627 us a batch with one and 1593 with two, 240 rows 1779 and 1818, of width 384, 204 and 240 rows, 923 and
// 921, 943 and 943; and fragments from memory, 20 and 37 KB, in the library of that time took 1543 where these take 1326 (768, 85 rows), 1851 and 1550 (240 rows), 1039 and
// 946 (384, 240 rows).  Microseconds, fragments from memory -> this, operands from beyond L2 (in brackets: from L2):
//   128 x 768 x 3072  [K][N] 14.1 -> 8.6 (9.1 -> 6.4)   [N][K] 16.1 -> 7.6 (12.6 -> 6.0)      128 x 3072 x 768  GELU 9.0 -> 6.4   its derivative 10.2 -> 5.9
//   128 x 384 x 1536          7.3 -> 5.4 (5.7 -> 4.8)           8.6 -> 5.0 (7.4 -> 4.7)       256 x 1536 x 384  GELU 5.5 -> 5.4   its derivative  6.2 -> 4.9
//   128 x 768 x 768           5.4 -> 4.6                        5.9 -> 4.5                    256 x 3072 x 768  GELU 11.8 -> 11.0  its derivative 14.3 -> 9.6
// A step of 3 + 1 layers of width 768, 640 rows, 611 -> 590 us, of width 384, 8320 rows, 847 -> 839, its evaluation 320 -> 317.
//
// Operand layouts: A is [M][K] with k contiguous (row stride lda: the class-token rows of a token matrix are T*D apart).  B is either
// [N][K] with k contiguous (input gradients: W stored [in,out] read as B(k = out, n = in)) or [K][N] with n contiguous (forward: W
// [in,out]), taken out of LDS with the transposing read.
#include "common.h"
#include "gemm_pipe.h"
#include "plan.h"

namespace ppll {

namespace {
using namespace pipe;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;

constexpr int KT = 64;                 // k of a stage: 128 bytes, one cache line, of a row of an operand with k contiguous
struct RowsArgs {
  const uint16_t* A; long lda;
  const uint16_t* B; long ldb;
  void* C; int c_f32; long ldc;
  int M, N, K;
  const float* bias;
  const uint16_t* residual; long ldr;
  int epilogue;
  uint16_t* C2;
  const uint16_t* aux; long ldaux;
  const void* side; int lds2;          // what the epilogue takes, the residual or the saved GELU derivative, for the helpers; bytes from row to row
  uint32_t a_bytes, b_bytes, s_bytes;
  int steps_per_wave;                  // 16-wide k-steps of each of the four waves
  TileMap map;
  int helpers;                         // workgroups an XCD that have no tile
};

// A wave's stages in LDS: 32 rows of A and 32 JN of B, 64 k each.
//  k contiguous in memory: [row][64 k], the 16-byte granule g of row r at g ^ ((r / 2) % 8).
//  B with n contiguous: [64 k][32 JN n] as in memory; 64-byte windows (JN = 2) w of k row k at w ^ (k / 2 % 2).
// The fragment reads then spread over all banks.  A copy instruction fills 1 KB in lane order: the lanes fetch in that order.
constexpr int A_BYTES = 32 * KT * 2;
template <int JN> constexpr int copies() { return 4 + 4 * JN; }
template <int JN> constexpr int stage_bytes() { return copies<JN>() * 1024; }

// The fragments of a stage, all there when the block ends (the compiler would order LDS reads that it knows of behind the copies into LDS)
template <bool BT, int JN> __device__ __forceinline__ void read_stage(u32x4 (&a)[4], u32x4 (&b)[4][JN], int addrA, int addrB) {
  asm volatile("ds_read_b128 %0, %4\n ds_read_b128 %1, %5\n ds_read_b128 %2, %6\n ds_read_b128 %3, %7\n s_waitcnt lgkmcnt(0)"
               : "=&v"(a[0]), "=&v"(a[1]), "=&v"(a[2]), "=&v"(a[3])
               : "v"(addrA), "v"(addrA ^ 32), "v"(addrA ^ 64), "v"(addrA ^ 96)
               : "memory");
#pragma unroll
  for (int j = 0; j < JN; ++j) {
    if constexpr (BT) {
      constexpr int P = 64 * JN;       // bytes of a k row
      const int at = addrB ^ (64 * j);
      u32x2 lo[4], hi[4];
      asm volatile("ds_read_b64_tr_b16 %0, %8\n ds_read_b64_tr_b16 %1, %8 offset:%9\n ds_read_b64_tr_b16 %2, %8 offset:%10\n "
                   "ds_read_b64_tr_b16 %3, %8 offset:%11\n ds_read_b64_tr_b16 %4, %8 offset:%12\n ds_read_b64_tr_b16 %5, %8 offset:%13\n "
                   "ds_read_b64_tr_b16 %6, %8 offset:%14\n ds_read_b64_tr_b16 %7, %8 offset:%15\n s_waitcnt lgkmcnt(0)"
                   : "=&v"(lo[0]), "=&v"(hi[0]), "=&v"(lo[1]), "=&v"(hi[1]), "=&v"(lo[2]), "=&v"(hi[2]), "=&v"(lo[3]), "=&v"(hi[3])
                   : "v"(at), "n"(4 * P), "n"(16 * P), "n"(20 * P), "n"(32 * P), "n"(36 * P), "n"(48 * P), "n"(52 * P)
                   : "memory");
#pragma unroll
      for (int u = 0; u < 4; ++u) b[u][j] = (u32x4){lo[u].x, lo[u].y, hi[u].x, hi[u].y};
    } else {
      const int at = addrB + 32 * KT * 2 * j;
      asm volatile("ds_read_b128 %0, %4\n ds_read_b128 %1, %5\n ds_read_b128 %2, %6\n ds_read_b128 %3, %7\n s_waitcnt lgkmcnt(0)"
                   : "=&v"(b[0][j]), "=&v"(b[1][j]), "=&v"(b[2][j]), "=&v"(b[3][j])
                   : "v"(at), "v"(at ^ 32), "v"(at ^ 64), "v"(at ^ 96)
                   : "memory");
    }
  }
}

// NS stages a wave
template <bool BT, int JN, int NS>
__global__ __launch_bounds__(256) void gemm_rows_kernel(RowsArgs p) {
  constexpr int TN = 32 * JN, PART_LD = TN + 4, STAGE = stage_bytes<JN>(), COPIES = copies<JN>();
  // the waves' stages, then (behind a barrier) their partial tiles
  extern __shared__ __align__(1024) char lds[];
  float (*part)[32][PART_LD] = reinterpret_cast<float (*)[32][PART_LD]>(lds);
  static_assert(4 * 32 * PART_LD * 4 <= 4 * NS * STAGE, "");
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int r = lane & 31, half = lane >> 5;
  const int slot = blockIdx.x >> 3;
  if (slot >= p.map.per_xcd) {
    const Bring b{p.A, p.B, p.side, p.a_bytes, p.b_bytes, p.s_bytes, (int)(p.lda * 2), (int)(p.ldb * 2), p.lds2, p.M, p.N, p.K, 32, TN, p.helpers};
    bring_operands<BT, 256>(b, p.map, blockIdx.x & 7, slot - p.map.per_xcd, (lds_char*)lds);
    return;
  }
  int tm, tn;
  if (!tile_at(p.map, blockIdx.x & 7, slot, tm, tn)) return;
  const int m0 = tm * 32, n0 = tn * TN;
  const __amdgpu_buffer_rsrc_t rsA = make_rsrc(p.A, p.a_bytes), rsB = make_rsrc(p.B, p.b_bytes);
  const int k_wave = wave * p.steps_per_wave * 16, k_end = min(p.K, k_wave + p.steps_per_wave * 16), lda2 = (int)(p.lda * 2), ldb2 = (int)(p.ldb * 2);
  // what the lane fetches: byte offsets at the wave's first k, and that k
  int va[4], vb[4 * JN], ka[2], kb = 0;
#pragma unroll
  for (int c = 0; c < 4 * JN; ++c) {
    const int row = 8 * c + (lane >> 3), gran = (lane & 7) ^ ((lane >> 4) + 4 * (c & 1));
    if (c < 2) ka[c] = k_wave + 8 * gran;
    if (c < 4) va[c] = m0 + row < p.M ? (m0 + row) * lda2 + (k_wave + 8 * gran) * 2 : OOB_BASE;
    if (!BT) {
      vb[c] = n0 + row < p.N ? (n0 + row) * ldb2 + (k_wave + 8 * gran) * 2 : OOB_BASE;
    } else {
      constexpr int SL = 4 * JN, ROWS = 64 / SL;         // 16-byte slots of a k row, k rows of a copy
      const int kr = ROWS * c + lane / SL, slot16 = JN == 1 ? lane & 3 : ((((lane & 7) >> 2) ^ ((kr >> 1) & 1)) * 4 + (lane & 3)), col = n0 + 8 * slot16;
      if (c == 0) kb = k_wave + kr;
      vb[c] = col < p.N && k_wave + kr < k_end ? (k_wave + kr) * ldb2 + col * 2 : OOB_BASE;
    }
  }
  lds_char* to = (lds_char*)lds + wave * (NS * STAGE);
  auto bring = [&](int s, int at) {    // stage s of the wave; what lies past its range of k reads as zeros
#pragma unroll
    for (int c = 0; c < 4; ++c) load_to_lds(rsA, to + at + c * 1024, ka[c & 1] + KT * s < k_end ? va[c] + 2 * KT * s : OOB);
#pragma unroll
    for (int c = 0; c < 4 * JN; ++c) {
      const int k = BT ? kb + 16 / JN * c : ka[c & 1];
      load_to_lds(rsB, to + at + A_BYTES + c * 1024, k + KT * s < k_end ? vb[c] + (BT ? KT * s * ldb2 : 2 * KT * s) : OOB);
    }
  };
  const int base = wave * (NS * STAGE) + (int)(uintptr_t)(lds_char*)lds;
  const int addrA = base + r * 128 + ((half ^ ((r >> 1) & 7)) << 4);
  const int kr = 8 * half + ((lane & 15) >> 2);
  const int addrB = base + A_BYTES + (BT ? kr * (64 * JN) + (JN == 2 ? ((kr >> 1) & 1) << 6 : 0) + (16 * ((lane >> 4) & 1) + 4 * (lane & 3)) * 2
                                         : r * 128 + ((half ^ ((r >> 1) & 7)) << 4));
#pragma unroll
  for (int s = 0; s < NS; ++s) bring(s, s * STAGE);
  f32x16 acc[JN];
#pragma unroll
  for (int j = 0; j < JN; ++j)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[j][i] = 0.f;
  // what the epilogue takes is on its way before the products
  constexpr int TPR = TN / 4;
  const int n = n0 + tid % TPR * 4;                      // N is a multiple of 8: four columns from a multiple of 4 below N are all inside
  float4 bias = make_float4(0.f, 0.f, 0.f, 0.f);
  uint2 side[JN][2];                                     // residual, factor
  if (n < p.N && p.bias) bias = *reinterpret_cast<const float4*>(p.bias + n);
#pragma unroll
  for (int pass = 0; pass < JN; ++pass) {
    const int m = m0 + pass * (256 / TPR) + tid / TPR;
    if (m < p.M && n < p.N) {
      if (p.residual) side[pass][0] = *reinterpret_cast<const uint2*>(p.residual + (size_t)m * p.ldr + n);
      if (p.epilogue == EPI_DGELU) side[pass][1] = *reinterpret_cast<const uint2*>(p.aux + (size_t)m * p.ldaux + n);
    }
  }
  const int stages = (p.steps_per_wave + KT / 16 - 1) / (KT / 16);
  for (int s = 0, at = 0; s < stages; ++s) {
    wait_vm<(NS - 1) * COPIES>();      // the oldest stage is there
    u32x4 a[4], b[4][JN];
    read_stage<BT, JN>(a, b, addrA + at, addrB + at);
    bring(s + NS, at);
    // the MFMA takes the B fragment first: a lane then holds 4 consecutive columns (n) of one output row (m)
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int j = 0; j < JN; ++j)
        acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, b[u][j]), __builtin_bit_cast(bf16x8, a[u]), acc[j], 0, 0, 0);
    at = at + STAGE == NS * STAGE ? 0 : at + STAGE;
  }
  wait_vm<0>();                        // no copy lands in a partial tile
  __syncthreads();
  // acc[j][4 q + e] = C[m0 + r][n0 + 32 j + 8 q + 4 half + e] summed over this wave's k
#pragma unroll
  for (int j = 0; j < JN; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<float4*>(&part[wave][r][32 * j + 8 * q + 4 * half]) =
          make_float4(acc[j][4 * q], acc[j][4 * q + 1], acc[j][4 * q + 2], acc[j][4 * q + 3]);
  __syncthreads();
#pragma unroll
  for (int pass = 0; pass < JN; ++pass) {
    const int mm = pass * (256 / TPR) + tid / TPR, nn = (tid % TPR) * 4, m = m0 + mm;
    if (m >= p.M || n >= p.N) continue;
    float v[4];
    {
      float4 t = *reinterpret_cast<const float4*>(&part[0][mm][nn]);
  #pragma unroll
      for (int w = 1; w < 4; ++w) {
        const float4 x = *reinterpret_cast<const float4*>(&part[w][mm][nn]);
        t.x += x.x; t.y += x.y; t.z += x.z; t.w += x.w;
      }
      v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    }
    if (p.bias) { v[0] += bias.x; v[1] += bias.y; v[2] += bias.z; v[3] += bias.w; }
    if (p.residual) {
      const uint2 w = side[pass][0];
      v[0] += __uint_as_float(w.x << 16); v[1] += __uint_as_float(w.x & 0xffff0000u);
      v[2] += __uint_as_float(w.y << 16); v[3] += __uint_as_float(w.y & 0xffff0000u);
    }
    if (p.epilogue == EPI_DGELU) {
      const uint2 w = side[pass][1];
      v[0] *= __uint_as_float(w.x << 16); v[1] *= __uint_as_float(w.x & 0xffff0000u);
      v[2] *= __uint_as_float(w.y << 16); v[3] *= __uint_as_float(w.y & 0xffff0000u);
    }
    if (p.c_f32) {
      *reinterpret_cast<float4*>((float*)p.C + (size_t)m * p.ldc + n) = make_float4(v[0], v[1], v[2], v[3]);
      continue;
    }
    uint16_t* c = (uint16_t*)p.C + (size_t)m * p.ldc + n;
    if (p.epilogue == EPI_GELU) {   // C2 = gelu(h), C = gelu'(h): one evaluation of the normal CDF and density
      float gl[4], dg[4];
  #pragma unroll
      for (int e = 0; e < 4; ++e) {
        float cdf, pdf;
        cdf_pdf(v[e], cdf, pdf);
        gl[e] = v[e] * cdf; dg[e] = cdf + v[e] * pdf;
      }
      *reinterpret_cast<uint2*>(c) = make_uint2(f32x2_to_bf16x2(dg[0], dg[1]), f32x2_to_bf16x2(dg[2], dg[3]));
      *reinterpret_cast<uint2*>(p.C2 + (size_t)m * p.ldc + n) = make_uint2(f32x2_to_bf16x2(gl[0], gl[1]), f32x2_to_bf16x2(gl[2], gl[3]));
    } else {
      *reinterpret_cast<uint2*>(c) = make_uint2(f32x2_to_bf16x2(v[0], v[1]), f32x2_to_bf16x2(v[2], v[3]));
    }
  }
}

template <bool BT, int JN, int NS> int rows_launch(hipStream_t s, dim3 grid, const RowsArgs& p) {
  constexpr int LDS = 4 * NS * stage_bytes<JN>();
  static OncePerDevice once;
  if (LDS > 64 * 1024) PPLL_TRY(raise_lds((const void*)gemm_rows_kernel<BT, JN, NS>, LDS, once));
  hipLaunchKernelGGL((gemm_rows_kernel<BT, JN, NS>), grid, dim3(256), LDS, s, p);
  return PPLL_OK;
}
bool aligned_to(const void* p, uintptr_t a) { return (((uintptr_t)p) & (a - 1)) == 0; }
}  // namespace

bool gemm_rows_supported(const GemmArgs& g) {
  if (g.a_dt != BF16 || g.b_dt != BF16 || g.colsum) return false;
  if (g.M < 1 || !few_tiles(g.M, g.N, g.K, product_units(g)) || g.N < 1 || g.K < 1 || (g.N & 7) || (g.K & 7)) return false;
  if (g.a_sk != 1 || (g.a_sm & 7) || !aligned_to(g.A, 16)) return false;
  const bool bt = g.b_sn == 1 && g.b_sk != 1;
  if (bt) {
    if ((g.b_sk & 7) || !aligned_to(g.B, 16)) return false;
  } else {
    if (g.b_sk != 1 || (g.b_sn & 7) || !aligned_to(g.B, 16)) return false;
  }
  if (g.c_dt == BF16 ? ((g.ldc & 3) || !aligned_to(g.C, 8)) : ((g.ldc & 3) || !aligned_to(g.C, 16))) return false;
  if (g.bias && !aligned_to(g.bias, 16)) return false;
  if (g.residual && (g.r_dt != BF16 || (g.ldr & 3) || !aligned_to(g.residual, 8))) return false;
  if (g.epilogue == EPI_GELU && (g.c_dt != BF16 || !g.C2 || !aligned_to(g.C2, 8))) return false;
  if (g.epilogue == EPI_DGELU && (g.aux_dt != BF16 || (g.ldaux & 3) || !aligned_to(g.aux, 8))) return false;
  // operands are addressed with 32-bit byte offsets
  const long lim = (1L << 30) - 64;
  const long a_bytes = ((long)(g.M - 1) * g.a_sm + g.K) * 2;
  const long b_bytes = bt ? ((long)(g.K - 1) * g.b_sk + g.N) * 2 : ((long)(g.N - 1) * g.b_sn + g.K) * 2;
  return a_bytes <= lim && b_bytes <= lim;
}

int launch_gemm_rows(hipStream_t s, const GemmArgs& g) {
  if (!gemm_rows_supported(g)) { set_error("launch_gemm_rows: unsupported product"); return PPLL_ERR_CONFIG; }
  const bool bt = g.b_sn == 1 && g.b_sk != 1;
  RowsArgs p{};
  p.A = (const uint16_t*)g.A; p.lda = g.a_sm;
  p.B = (const uint16_t*)g.B; p.ldb = bt ? g.b_sk : g.b_sn;
  p.C = g.C; p.c_f32 = g.c_dt == F32; p.ldc = g.ldc;
  p.M = g.M; p.N = g.N; p.K = g.K;
  p.bias = g.bias; p.residual = (const uint16_t*)g.residual; p.ldr = g.ldr;
  p.epilogue = g.epilogue; p.C2 = (uint16_t*)g.C2; p.aux = (const uint16_t*)g.aux; p.ldaux = g.ldaux;
  p.a_bytes = (uint32_t)(((long)(g.M - 1) * g.a_sm + g.K) * 2);
  p.b_bytes = (uint32_t)(bt ? ((long)(g.K - 1) * g.b_sk + g.N) * 2 : ((long)(g.N - 1) * g.b_sn + g.K) * 2);
  const int steps = (g.K + 15) / 16;
  p.steps_per_wave = (steps + 3) / 4;
  const int units = product_units(g);
  const bool wide = few_tiles_wide(g.M, g.N, units);
  p.map = tile_map(g.M, g.N, 32, wide ? 64 : 32, units);
  p.helpers = g.shared ? 0 : helper_workgroups(p.map.per_xcd, units);
  const long lds = g.epilogue == EPI_DGELU ? g.ldaux : g.ldr, s_bytes = ((long)(g.M - 1) * lds + g.N) * 2;
  if (s_bytes < (1L << 30)) {
    p.side = g.epilogue == EPI_DGELU ? g.aux : g.residual;
    p.lds2 = (int)(lds * 2); p.s_bytes = (uint32_t)s_bytes;
  }
  const dim3 grid(8 * (p.map.per_xcd + p.helpers));
  void* prof = nullptr;
  PPLL_TRY(profile_begin(s, 2.0 * g.M * g.N * g.K, &prof, g.M <= FEW_ROWS ? 2 : 0));
  const bool two = p.steps_per_wave <= 2 * KT / 16 || g.shared || 8 * p.map.per_xcd > units;
  if (wide) PPLL_TRY(bt ? (rows_launch<true, 2, 2>(s, grid, p)) : (rows_launch<false, 2, 2>(s, grid, p)));
  else if (two) PPLL_TRY(bt ? (rows_launch<true, 1, 2>(s, grid, p)) : (rows_launch<false, 1, 2>(s, grid, p)));
  else PPLL_TRY(bt ? (rows_launch<true, 1, 4>(s, grid, p)) : (rows_launch<false, 1, 4>(s, grid, p)));
  PPLL_HIP(hipGetLastError());
  return profile_end(s, prof);
}

}  // namespace ppll
