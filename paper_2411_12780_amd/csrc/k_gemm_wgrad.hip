// Sets of weight-gradient products C_j[M,N] = A_j^T B_j (both operands [k][.], fp32 output, bias gradients as column sums of B_j) on
// tiles of 384 x 192, some divided along k so that every compute unit has about the same to do.
//
// What bounds such a launch is bringing operands to LDS and out of it again.  A tile of 384 x 192 brings 36 KB per 32 k, half of what
// 128 x 128 tiles bring for as many products, and a wave's 96 x 96 part reads a third less of them than 64 x 64.  384 and 192 because
// widths of 192, 384 and 768 are whole numbers of tiles.  Eight waves, one workgroup a unit (147 KB of LDS, 144 accumulators of 256
// registers): operands go straight to LDS, four stages of 32 k; the fragment reads of a k step run under the products of the one before.
// There are fewer tiles than units, or the last round is far from full: the tiles beyond the last full round are divided along k into
// parts that fill one (`big_grad_tiles` in plan.h).  A part leaves its fp32 sums in a slot of the workspace and a second kernel adds them in
// ascending k: results do not depend on timing.
// Microseconds of a set, 128 x 128 or 128 x 256 tiles -> these: 3 + 1 layers of width 384, 8320 rows 131.6 -> 122.7, 16640 rows 261.9 ->
// 206.7 (820 TFLOP/s); 3 + 1 of width 768, 5800 rows 343 -> 271; 1 + 1 of width 768, 6304 rows 198 -> 135; 3 + 1 of width 192, 25216 rows 221 ->
// 144.  Two workgroups a unit with 192 x 192 tiles, three stages, were 1 % (of a step) behind; a barrier every 64 k instead of 32, level.
#include "common.h"
#include "gemm_pipe.h"
#include "plan.h"

namespace ppll {

namespace {
using namespace pipe;

constexpr int EDGE_M = BIG_EDGE_M, EDGE = BIG_EDGE, WAVE_EDGE = 96, TILES = 3;       // a wave's part of a tile, 32 x 32 products along its edge
constexpr int WAVES = EDGE_M / WAVE_EDGE * 2, STAGES = 4;
constexpr int OPER_A = EDGE_M * KS * 2, OPER_B = EDGE * KS * 2, STAGE = OPER_A + OPER_B, LDS_BYTES = STAGES * STAGE;
constexpr int COPIES_A = OPER_A / 1024 / WAVES, COPIES_B = (OPER_B / 1024 + WAVES - 1) / WAVES;    // of an operand, a wave and stage
constexpr int COPIES_LEAST = COPIES_A + OPER_B / 1024 / WAVES;
constexpr int SLOT_FLOATS = EDGE_M * EDGE + EDGE;                // a part's sums, then its column sums
static_assert(EDGE == 2 * WAVE_EDGE && OPER_A % (1024 * WAVES) == 0, "");

struct BigProblem {
  const uint16_t* A; const uint16_t* B; float* C; float* colsum;
  int lda, ldb, ldc, M, N, K, tiles_m, tiles_n, first_tile;
};
struct BigArgs {
  // products with a long reduction come first: their tiles [0, whole_tiles) run whole, [whole_tiles, long_tiles) in `cuts` parts; the
  // tiles of the others, [long_tiles, total_tiles), whole at the end
  int n, total_tiles, long_tiles, whole_tiles, cuts;
  float* ws;                                                   // [divided tile][part] slots
  BigProblem prob[BIG_PRODUCTS];
};

// Tile t -> its product and its place there.  Across the shorter side first, so that a stretch of tiles shares the panels of that side.
__device__ __forceinline__ int big_locate(const BigArgs& a, int t, int& tm, int& tn) {
  int j = 0;
  while (j + 1 < a.n && t >= a.prob[j + 1].first_tile) ++j;
  const int local = t - a.prob[j].first_tile, m = a.prob[j].tiles_m, n = a.prob[j].tiles_n;
  if (m >= n) { tm = local / n; tn = local % n; } else { tm = local % m; tn = local / m; }
  return j;
}
__device__ __forceinline__ int steps_per_part(int K, int cuts) { return ((K + KS - 1) / KS + cuts - 1) / cuts; }

// LDS: [32 k][384] and [32 k][192] as in memory.  The 64-byte window w of k row k sits at w ^ (k % 4) where rows are 768 bytes apart, at
// w ^ (k / 2 % 2) where 384: a transposing read, one window of 8 k rows, then takes every bank twice.
template <int E> __device__ __forceinline__ int window_turn(int k) { return E % 128 ? (k >> 1) & 1 : k & 3; }
template <int E> __device__ __forceinline__ int frag_at(int tile, int lane) {   // lane address of the fragment of rows 32 tile .. + 31, k step 0
  const int k = 8 * (lane >> 5) + ((lane & 15) >> 2);
  return k * (2 * E) + ((tile ^ window_turn<E>(k)) << 6) + (16 * ((lane >> 4) & 1) + 4 * (lane & 3)) * 2;
}

// Byte offset, at k = 0 of a stage, of what lies at byte l of an operand's stage: a copy fills 1 KB of LDS in lane order, so the turn is
// applied to what a lane fetches
template <int E> __device__ __forceinline__ int fetch_from(int l, int ld2, int row0, int rows) {
  const int k = l / (2 * E), at = l % (2 * E), col = row0 + (((at >> 6) ^ window_turn<E>(k)) << 5) + ((at & 63) >> 1);
  return col < rows ? k * ld2 + col * 2 : OOB_BASE;
}

// One k step: the products of the fragments at hand, and under them the reads of the next ones, which are there when the block ends
// (one block, because the compiler would order LDS reads that it knows of behind the copies into LDS).
template <int KK>
__device__ __forceinline__ void big_step(f32x16 (&acc)[TILES][TILES], const Frags<true, TILES>& a, const Frags<true, TILES>& b,
                                            Frags<true, TILES>& na, Frags<true, TILES>& nb, const int (&fa)[TILES], const int (&fb)[TILES], int at) {
#define PPLL_MMA(J, I) "v_mfma_f32_32x32x16_bf16 %[c" #J #I "], %[q" #J "], %[p" #I "], %[c" #J #I "]\n"
#define PPLL_READ(L, H, R) "ds_read_b64_tr_b16 %[" #L "], %[" #R "] offset:%[lo]\n ds_read_b64_tr_b16 %[" #H "], %[" #R "] offset:%[hi]\n"
#define PPLL_READ_A(L, H, R) "ds_read_b64_tr_b16 %[" #L "], %[" #R "] offset:%[al]\n ds_read_b64_tr_b16 %[" #H "], %[" #R "] offset:%[ah]\n"
  asm volatile("s_nop 1\n" PPLL_MMA(0, 0) PPLL_READ(m0, n0, rb0) PPLL_READ_A(l0, h0, ra0) PPLL_MMA(0, 1) PPLL_READ_A(l1, h1, ra1) PPLL_MMA(0, 2)
               PPLL_READ_A(l2, h2, ra2) PPLL_MMA(1, 0) PPLL_READ(m1, n1, rb1) PPLL_MMA(1, 1) PPLL_READ(m2, n2, rb2) PPLL_MMA(1, 2)
               PPLL_MMA(2, 0) PPLL_MMA(2, 1) PPLL_MMA(2, 2) "s_waitcnt lgkmcnt(0)"
               : [c00] "+v"(acc[0][0]), [c01] "+v"(acc[0][1]), [c02] "+v"(acc[0][2]), [c10] "+v"(acc[1][0]), [c11] "+v"(acc[1][1]),
                 [c12] "+v"(acc[1][2]), [c20] "+v"(acc[2][0]), [c21] "+v"(acc[2][1]), [c22] "+v"(acc[2][2]),
                 [l0] "=&v"(na.lo[0]), [h0] "=&v"(na.hi[0]), [l1] "=&v"(na.lo[1]), [h1] "=&v"(na.hi[1]), [l2] "=&v"(na.lo[2]), [h2] "=&v"(na.hi[2]),
                 [m0] "=&v"(nb.lo[0]), [n0] "=&v"(nb.hi[0]), [m1] "=&v"(nb.lo[1]), [n1] "=&v"(nb.hi[1]), [m2] "=&v"(nb.lo[2]), [n2] "=&v"(nb.hi[2])
               : [p0] "v"(a.get(0)), [p1] "v"(a.get(1)), [p2] "v"(a.get(2)), [q0] "v"(b.get(0)), [q1] "v"(b.get(1)), [q2] "v"(b.get(2)),
                 [ra0] "v"(fa[0] + at), [ra1] "v"(fa[1] + at), [ra2] "v"(fa[2] + at), [rb0] "v"(fb[0] + at), [rb1] "v"(fb[1] + at),
                 [rb2] "v"(fb[2] + at), [lo] "n"(KK * 32 * EDGE), [hi] "n"(KK * 32 * EDGE + 8 * EDGE), [al] "n"(KK * 32 * EDGE_M), [ah] "n"(KK * 32 * EDGE_M + 8 * EDGE_M)
               : "memory");
#undef PPLL_MMA
#undef PPLL_READ
#undef PPLL_READ_A
}

__global__ __launch_bounds__(64 * WAVES, 2) void gemm_big_grads_kernel(BigArgs a) {
  PPLL_CODE_TO_L2(1);
  extern __shared__ __align__(1024) char smem[];
  // workgroup id -> item: the whole tiles first, then the parts, then the short tiles; within each kind XCD x (id % 8) takes a
  // contiguous stretch, parts of one k range next to each other: neighbours share operand panels, and they share an L2
  const int xcd = blockIdx.x & 7, rest = a.long_tiles - a.whole_tiles, parts = rest * a.cuts;
  int slot = blockIdx.x >> 3, t, c = -1;
  const int per1 = (a.whole_tiles + 7) >> 3, per2 = (parts + 7) >> 3, per3 = (a.total_tiles - a.long_tiles + 7) >> 3;
  if (slot < per1) {
    t = xcd * per1 + slot;
    if (t >= a.whole_tiles) return;
  } else if ((slot -= per1) < per2) {
    const int i = xcd * per2 + slot;
    if (i >= parts) return;
    t = a.whole_tiles + i % rest; c = i / rest;
  } else {
    slot -= per2;
    t = a.long_tiles + xcd * per3 + slot;
    if (slot >= per3 || t >= a.total_tiles) return;
  }
  int tm, tn;
  const BigProblem& p = a.prob[big_locate(a, t, tm, tn)];
  const int m0 = tm * EDGE_M, n0 = tn * EDGE, M = p.M, N = p.N;
  int k0 = 0, K = p.K;
  if (c >= 0) {
    const int per = steps_per_part(p.K, a.cuts) * KS;
    k0 = min(c * per, p.K); K = min(per, p.K - k0);          // a trailing part may have none
  }
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wm = wave >> 1, wn = wave & 1;
  const int lda2 = p.lda * 2, ldb2 = p.ldb * 2;
  // k rows past the last one of the range lie past the end of the buffer and read as zeros
  const __amdgpu_buffer_rsrc_t rsA = make_rsrc(p.A + (size_t)k0 * p.lda, K > 0 ? (uint32_t)((K - 1) * lda2 + M * 2) : 0u);
  const __amdgpu_buffer_rsrc_t rsB = make_rsrc(p.B + (size_t)k0 * p.ldb, K > 0 ? (uint32_t)((K - 1) * ldb2 + N * 2) : 0u);
  int va[COPIES_A], vb[COPIES_B];
#pragma unroll
  for (int q = 0; q < COPIES_A; ++q) va[q] = fetch_from<EDGE_M>((q * WAVES + wave) * 1024 + lane * 16, lda2, m0, M);
#pragma unroll
  for (int q = 0; q < COPIES_B; ++q) vb[q] = fetch_from<EDGE>((q * WAVES + wave) * 1024 + lane * 16, ldb2, n0, N);
  lds_char* lds = (lds_char*)smem;
  const int nk = (K + KS - 1) / KS;
  auto issue = [&](int i) {                // copies of stage i (zeros past the last one)
    const bool live = i < nk;
    const int ka = i * KS * lda2, kb = i * KS * ldb2;
    lds_char* st = lds + (i % STAGES) * STAGE + wave * 1024;
#pragma unroll
    for (int q = 0; q < COPIES_A; ++q) load_to_lds(rsA, st + q * (1024 * WAVES), live ? va[q] + ka : OOB_BASE);
#pragma unroll
    for (int q = 0; q < COPIES_B; ++q)
      if ((q + 1) * WAVES * 1024 <= OPER_B || (q * WAVES + wave) * 1024 < OPER_B) load_to_lds(rsB, st + OPER_A + q * (1024 * WAVES), live ? vb[q] + kb : OOB_BASE);
  };
  const int base = (int)(uintptr_t)lds;
  int fa[TILES], fb[TILES];
#pragma unroll
  for (int i = 0; i < TILES; ++i) {
    fa[i] = base + frag_at<EDGE_M>(wm * TILES + i, lane);
    fb[i] = base + OPER_A + frag_at<EDGE>(wn * TILES + i, lane);
  }
  f32x16 acc[TILES][TILES];                // [n][m]: C^T tiles, lane l holds row l % 32, columns 8 q + 4 (l / 32) + e in element 4 q + e
#pragma unroll
  for (int j = 0; j < TILES; ++j)
#pragma unroll
    for (int i = 0; i < TILES; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[j][i][e] = 0.f;
  const bool do_colsum = p.colsum && m0 == 0 && wm == 0;
  // sixteen chains a column, as on the other tiles: k % 8 in each half of a k step.  (With two, 25216 rows around 1 gave sums 3.1e-7 off,
  // with these 3.8e-8; around 0 1.1e-7 and 6.2e-8.)
  float csum[TILES][8] = {};
  Frags<true, TILES> a0, b0, a1, b1;
  auto column_sums = [&](const Frags<true, TILES>& b) {
    if (!do_colsum) return;
#pragma unroll
    for (int j = 0; j < TILES; ++j) {
      const u32x4 v = b.get(j);
#pragma unroll
      for (int e = 0; e < 4; ++e) { csum[j][2 * e] += __uint_as_float(v[e] << 16); csum[j][2 * e + 1] += __uint_as_float(v[e] & 0xffff0000u); }
    }
  };
#pragma unroll
  for (int i = 0; i < STAGES - 1; ++i) issue(i);
  wait_vm<(STAGES - 2) * COPIES_LEAST>();
  barrier();
#pragma unroll
  for (int i = 0; i < TILES; ++i) { set_zero(a1, i); set_zero(b1, i); }
  big_step<0>(acc, a1, b1, a0, b0, fa, fb, 0);     // the first fragments: products with zeros under the reads
  int st = 0;
  for (int i = 0; i < nk; ++i) {
    const int nx = st + STAGE == LDS_BYTES ? 0 : st + STAGE;
    wait_vm<(STAGES - 3) * COPIES_LEAST>();          // this wave's part of stage i + 1 is in LDS
    barrier();             // and everyone's; nobody reads stage i - 1 any more
    issue(i + STAGES - 1);
    column_sums(b0);
    big_step<1>(acc, a0, b0, a1, b1, fa, fb, st);
    column_sums(b1);
    big_step<0>(acc, a1, b1, a0, b0, fa, fb, nx);
    st = nx;
  }
  asm volatile("s_nop 15\n s_nop 3" ::: "memory");    // the last products are through
#pragma unroll
  for (int j = 0; j < TILES; ++j)
#pragma unroll
    for (int i = 0; i < TILES; ++i) asm volatile("" : "+v"(acc[j][i]));
  wait_vm<0>();
  barrier();               // the stages are free for the epilogue

  float* out = c >= 0 ? a.ws + ((size_t)(t - a.whole_tiles) * a.cuts + c) * SLOT_FLOATS : p.C + (size_t)m0 * p.ldc + n0;
  const int ld = c >= 0 ? EDGE : p.ldc, rows = c >= 0 ? EDGE_M : M - m0, cols = c >= 0 ? EDGE : N - n0;
  if (do_colsum) {
    float* sums = c >= 0 ? out + EDGE_M * EDGE : p.colsum + n0;
#pragma unroll
    for (int j = 0; j < TILES; ++j) {
      float sum = ((csum[j][0] + csum[j][1]) + (csum[j][2] + csum[j][3])) + ((csum[j][4] + csum[j][5]) + (csum[j][6] + csum[j][7]));
      sum += __shfl_xor(sum, 32, 64);       // the other half of every k step
      const int n = wn * WAVE_EDGE + j * 32 + lane;
      if (lane < 32 && n < cols) sums[n] = sum;
    }
  }
  // a wave passes 32 rows at a time through its own piece of LDS and stores them 384 bytes a row
  constexpr int SP = WAVE_EDGE + 4, Q = WAVE_EDGE / 4;
  static_assert(WAVES * 32 * SP * 4 <= LDS_BYTES && 32 * Q % 64 == 0, "");
  float* piece = reinterpret_cast<float*>(smem) + wave * 32 * SP;
#pragma unroll
  for (int im = 0; im < TILES; ++im) {
#pragma unroll
    for (int jn = 0; jn < TILES; ++jn)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<float4*>(piece + (lane & 31) * SP + jn * 32 + 8 * q + 4 * (lane >> 5)) =
            make_float4(acc[jn][im][4 * q], acc[jn][im][4 * q + 1], acc[jn][im][4 * q + 2], acc[jn][im][4 * q + 3]);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int q = 0; q < 32 * Q / 64; ++q) {
      const int l = q * 64 + lane, r = l / Q, c4 = l % Q * 4, m = wm * WAVE_EDGE + im * 32 + r, n = wn * WAVE_EDGE + c4;
      const float4 v = *reinterpret_cast<const float4*>(piece + r * SP + c4);
      if (m < rows && n < cols) *reinterpret_cast<float4*>(out + (size_t)m * ld + n) = v;   // N is a multiple of 8
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
  }
}

// Eight rows of a divided tile per workgroup: the sum of its parts, added in ascending k
constexpr int SUM_ROWS = 8, SUM_THREADS = EDGE / 4 * SUM_ROWS;
__global__ __launch_bounds__(SUM_THREADS) void gemm_big_grads_sum_kernel(BigArgs a) {
  const int d = blockIdx.x / (EDGE_M / SUM_ROWS), strip = blockIdx.x % (EDGE_M / SUM_ROWS), tid = threadIdx.x;
  int tm, tn;
  const BigProblem& p = a.prob[big_locate(a, a.whole_tiles + d, tm, tn)];
  const int m0 = tm * EDGE_M, n0 = tn * EDGE, row = strip * SUM_ROWS + tid / (EDGE / 4), c4 = tid % (EDGE / 4) * 4;
  const float* slot = a.ws + (size_t)d * a.cuts * SLOT_FLOATS;
  auto sum = [&](int at) {
    constexpr int U = 8;
    float4 s = *reinterpret_cast<const float4*>(slot + at);
    for (int c = 1; c < a.cuts; c += U) {
      float4 v[U];
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (c + u < a.cuts) v[u] = *reinterpret_cast<const float4*>(slot + (size_t)(c + u) * SLOT_FLOATS + at);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (c + u < a.cuts) { s.x += v[u].x; s.y += v[u].y; s.z += v[u].z; s.w += v[u].w; }
    }
    return s;
  };
  if (m0 + row < p.M && n0 + c4 < p.N) *reinterpret_cast<float4*>(p.C + (size_t)(m0 + row) * p.ldc + n0 + c4) = sum(row * EDGE + c4);
  if (strip == 0 && p.colsum && m0 == 0 && tid < EDGE / 4 && n0 + c4 < p.N) {
    const float4 s = sum(EDGE_M * EDGE + c4);
    float* o = p.colsum + n0 + c4;
    o[0] = s.x; o[1] = s.y; o[2] = s.z; o[3] = s.w;
  }
}
}  // namespace

size_t gemm_big_grads_floats(int parts) { return (size_t)parts * SLOT_FLOATS; }

int launch_gemm_big_grads(hipStream_t s, const GemmArgs* gs, int n, float* ws, const BigGradPlan& plan) {
  static OncePerDevice once;
  PPLL_TRY(raise_lds((const void*)gemm_big_grads_kernel, LDS_BYTES, once));
  BigArgs a{};
  a.n = n; a.ws = ws;
  a.total_tiles = plan.tiles; a.long_tiles = plan.long_tiles; a.whole_tiles = plan.whole_tiles; a.cuts = plan.cuts;
  int tiles = 0, filled = 0;
  double flops = 0.0;
  for (int pass = 0; pass < 2; ++pass) {               // long reductions first, then the short ones
    for (int j = 0; j < n; ++j) {
      const GemmArgs& g = gs[j];
      if ((wg_steps(g.K) >= plan.long_steps) != (pass == 0)) continue;
      BigProblem& q = a.prob[filled++];
      q.A = (const uint16_t*)g.A; q.lda = (int)g.a_sk; q.B = (const uint16_t*)g.B; q.ldb = (int)g.b_sk;
      q.C = (float*)g.C; q.ldc = (int)g.ldc; q.colsum = g.colsum; q.M = g.M; q.N = g.N; q.K = g.K;
      q.tiles_m = (g.M + EDGE_M - 1) / EDGE_M; q.tiles_n = (g.N + EDGE - 1) / EDGE;
      q.first_tile = tiles;
      tiles += q.tiles_m * q.tiles_n;
      flops += 2.0 * g.M * g.N * g.K;
    }
  }
  const int rest = plan.long_tiles - plan.whole_tiles;
  void* prof = nullptr;
  PPLL_TRY(profile_begin(s, flops, &prof));
  const int grid = 8 * ((plan.whole_tiles + 7) / 8 + (rest * plan.cuts + 7) / 8 + (tiles - plan.long_tiles + 7) / 8);
  hipLaunchKernelGGL(gemm_big_grads_kernel, dim3(grid), dim3(64 * WAVES), LDS_BYTES, s, a);
  PPLL_HIP(hipGetLastError());
  if (rest > 0) {
    hipLaunchKernelGGL(gemm_big_grads_sum_kernel, dim3(EDGE_M / SUM_ROWS * rest), dim3(SUM_THREADS), 0, s, a);
    PPLL_HIP(hipGetLastError());
  }
  return profile_end(s, prof);
}

}  // namespace ppll
