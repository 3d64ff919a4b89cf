// Linear-layer products whose 64 x 64 output tiles find a compute unit each: C[M,N] = A[M,K] B, bf16 operands, fp32 accumulation,
// the epilogues of the tiled kernel.
//
// With so few tiles a product takes as long as one tile does, and what bounds that is the chain along k.  A 64 x 128 tile whose four
// waves copy through registers, multiply and meet at a barrier spends 0.37 us per 64 k (640 x 768 x 3072: 22 us on 60 of 256
// units), because the phases follow one another.  Here they run beside one another, 0.23 us per 64 k: four waves do nothing but copy,
// straight from memory to LDS, three stages ahead of four waves that multiply, a 32 x 32 quarter of the tile each.  A quarter walks
// along all of k in order, so the results are the tiled kernel's bit for bit.  (Eight multiplying waves that share out the k steps of
// a stage and add up at the end were no faster, 14.5 us at 640 x 768 x 3072, and their sums run in an order of their own: through
// four pipelined blocks of width 768 results moved by 1.4 %.)  A copy takes rows of 128 bytes, whole cache lines: with 64 bytes a row
// the loop took half as long again, the lines being fetched twice from beyond L2.  Smaller tiles find more units and copy more per
// product; beyond one a unit the tiled kernel catches up (`split_tiles`).  64 KB of LDS and 118 registers a wave leave room for a workgroup of
// another stream (with stages twice as deep a pipeline of three blocks of width 192, 4160 rows, took 570 us a batch instead of 520).
// Operands from beyond L2, as in a step, took the loop half as long again; units without a tile bring them into L2 ahead of the tiles (Bring,
// in gemm_pipe.h), and an XCD takes a block of the tiles where that shares more of them (tile_map): 640 x 768 x 3072 19.2 -> 11.9 us, x 2304
// 15.3 -> 9.6, x 768 6.5 -> 5.5, 1105 x 768 x 3072 20.1 -> 17.0, 2176 x 384 x 1536 11.7 -> 9.3.
// Microseconds, tiled kernel -> this one: 640 x 768 x 768 8.6 -> 5.8, 640 x 768 x 2304 17.7 -> 11.3, 640 x 768 x 3072 22.4 -> 14.2,
// 1500 x 384 x 384 6.2 -> 4.3, 1500 x 384 x 1536 13.0 -> 8.3; a step of 3 + 1 layers of width 768, 640 rows, 776 -> 680.
#include "common.h"
#include "gemm_pipe.h"
#include "plan.h"

namespace ppll {

namespace {
using namespace pipe;

struct SplitArgs {
  const uint16_t* A; long lda;      // A[m*lda + k]
  const uint16_t* B; long ldb;      // BT ? B[k*ldb + n] : B[n*ldb + k]
  uint16_t* C; long ldc;
  int M, N, K;
  TileMap map;
  int helpers;                      // workgroups an XCD that have no tile
  const float* bias;
  const uint16_t* side; long lds;   // residual, or the saved GELU derivative (EPI_DGELU)
  int epilogue;
  uint16_t* C2;
  uint32_t a_bytes, b_bytes, c_bytes, s_bytes;
};

constexpr int EDGE = 64, KT = 64;    // tile, k of a stage: 128 bytes, one cache line, of a row of an operand with k contiguous
constexpr int WAVES = 4, COPY_WAVES = 4, STAGES = 4;   // multiplying waves have 32 x 32 of the tile each
constexpr int OPER = EDGE * KT * 2, STAGE = 2 * OPER;

__device__ __forceinline__ u32x4 split_load16(__amdgpu_buffer_rsrc_t r, int off) { return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0); }
__device__ __forceinline__ u32x4 pack8(const float (&v)[8]) {
  return (u32x4){f32x2_to_bf16x2(v[0], v[1]), f32x2_to_bf16x2(v[2], v[3]), f32x2_to_bf16x2(v[4], v[5]), f32x2_to_bf16x2(v[6], v[7])};
}
__device__ __forceinline__ void swap_halves(float& a, float& b) {   // the upper 32 lanes of a for the lower 32 of b
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(r[0]); b = __uint_as_float(r[1]);
}

// One operand of a stage in LDS, 64 rows x 64 k, 128 bytes a (k) row.
//  TR = false: k contiguous in memory, [row][64 k]: the 16-byte granule g of row r at g ^ ((r / 2) % 8).
//  TR = true: row index contiguous, [64 k][64 rows] as in memory: the 64-byte window w of k row k at w ^ (k / 2 % 2).
// The fragment reads then spread over all banks.
__device__ __forceinline__ int window(int k) { return (k >> 1) & 1; }
// lane address of the fragment of rows row0 .. row0 + 31 at the first k step; TR = false: at k step kk with 32 kk flipped in it, else
// 2048 kk further on
template <bool TR> __device__ __forceinline__ int frag(int row0, int lane) {
  const int half = lane >> 5, r = lane & 31;
  if (!TR) return (row0 + r) * 128 + ((half ^ ((r >> 1) & 7)) << 4);
  const int k = 8 * half + ((lane & 15) >> 2);
  return k * 128 + (((row0 >> 5) ^ window(k)) << 6) + (16 * ((lane >> 4) & 1) + 4 * (lane & 3)) * 2;
}

// What a copying wave brings of one operand, N copies a stage.  From stage to stage only a scalar offset changes.  The range check
// compares a lane's offset with the length less that scalar, so the scalar stays below the length: stages past the last have a length
// of 0.
template <bool TR, int N> struct Copies {
  int v[N], gk[2], step, first;         // byte offsets of the lane in stage 0; first k of its granules, by parity of the copy
  const void* p; uint32_t bytes;
  __device__ __forceinline__ void init(const void* ptr, uint32_t n, long ld, int row0, int nrows, int lane, int first_) {
    p = ptr; bytes = n; first = first_;
    const int ld2 = (int)(ld * 2);
    step = TR ? KT * ld2 : KT * 2;
#pragma unroll
    for (int c = 0; c < N; ++c) {
      const int q = first + c;
      if (TR) {
        const int kr = q * 8 + (lane >> 3), slot = lane & 7, col = row0 + (((slot >> 2) ^ window(kr)) * 4 + (slot & 3)) * 8;
        v[c] = col < nrows ? kr * ld2 + col * 2 : OOB_BASE;
      } else {
        const int g = (lane & 7) ^ ((lane >> 4) + 4 * (q & 1));
        v[c] = (row0 + q * 8 + (lane >> 3)) * ld2 + g * 16;   // rows past the last one lie past the end of the buffer
        gk[q & 1] = g * 8;
      }
    }
  }
  __device__ __forceinline__ void issue(lds_char* to, int i, int stages, int K) const {
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(p, i < stages ? bytes : 0u);
    const int off = i < stages ? i * step : 0;
    to += first * 1024;
    if (!TR && i == stages - 1 && K % KT) {
      const int left = K - i * KT;
#pragma unroll
      for (int c = 0; c < N; ++c) load_to_lds(rs, to + c * 1024, gk[(first + c) & 1] < left ? v[c] : OOB_BASE, off);
    } else {
#pragma unroll
      for (int c = 0; c < N; ++c) load_to_lds(rs, to + c * 1024, v[c], off);
    }
  }
};

// A copying wave, from the first stage to the last.  Barriers: one with stage 0 in LDS, one per stage.
template <bool TR>
__device__ __forceinline__ void copy_stages(const void* ptr, uint32_t bytes, long ld, int row0, int nrows, int lane, int w, lds_char* to, int stages, int K) {
  constexpr int N = OPER / 1024 / (COPY_WAVES / 2), AHEAD = STAGES - 1;
  Copies<TR, N> c;
  c.init(ptr, bytes, ld, row0, nrows, lane, w * N);
#pragma unroll 1
  for (int i = 0; i < AHEAD; ++i) c.issue(to + i * STAGE, i, stages, K);
  wait_vm<N * (AHEAD - 1)>();
  barrier();
  int wr = AHEAD * STAGE;
  for (int i = 0; i < stages; ++i) {
    wait_vm<N * (AHEAD - 2)>();          // this wave's part of stage i + 1 is there
    barrier();        // and everyone's; nobody reads stage i - 1 any more
    c.issue(to + wr, i + AHEAD, stages, K);
    wr += STAGE;
    if (wr == STAGES * STAGE) wr = 0;
  }
  wait_vm<0>();                          // no copy outlives the workgroup, whose LDS others get
}

// The four k steps of a stage in a wave, in order: the products of the fragments at hand, and under them the reads of the next stage's,
// which are there when the block ends (one block, because the compiler would order LDS reads that it knows of behind the copies into
// LDS).  The reads come first, so a vector instruction before the block is two and more away from the first product.
template <bool BT>
__device__ __forceinline__ void split_stage(f32x16& acc, const Frags<false, 4>& a, const Frags<BT, 4>& b, Frags<false, 4>& na, Frags<BT, 4>& nb,
                                            int addrA, int addrB) {
#define PPLL_MMA "v_mfma_f32_32x32x16_bf16 %[c], %[q0], %[p0], %[c]\n v_mfma_f32_32x32x16_bf16 %[c], %[q1], %[p1], %[c]\n" \
                 "v_mfma_f32_32x32x16_bf16 %[c], %[q2], %[p2], %[c]\n v_mfma_f32_32x32x16_bf16 %[c], %[q3], %[p3], %[c]\n s_waitcnt lgkmcnt(0)"
#define PPLL_NEXT_A [x0] "=&v"(na.v[0]), [x1] "=&v"(na.v[1]), [x2] "=&v"(na.v[2]), [x3] "=&v"(na.v[3])
#define PPLL_CUR [p0] "v"(a.get(0)), [p1] "v"(a.get(1)), [p2] "v"(a.get(2)), [p3] "v"(a.get(3)), [q0] "v"(b.get(0)), [q1] "v"(b.get(1)), \
                 [q2] "v"(b.get(2)), [q3] "v"(b.get(3)), [ra0] "v"(addrA), [ra1] "v"(addrA ^ 32), [ra2] "v"(addrA ^ 64), [ra3] "v"(addrA ^ 96)
  if constexpr (BT) {   // the upper half of a fragment is k + 4: the same window, 512 bytes on
    asm volatile("ds_read_b128 %[x0], %[ra0]\n ds_read_b64_tr_b16 %[l0], %[rb]\n ds_read_b64_tr_b16 %[h0], %[rb] offset:512\n"
                 "ds_read_b128 %[x1], %[ra1]\n ds_read_b64_tr_b16 %[l1], %[rb] offset:2048\n ds_read_b64_tr_b16 %[h1], %[rb] offset:2560\n"
                 "ds_read_b128 %[x2], %[ra2]\n ds_read_b64_tr_b16 %[l2], %[rb] offset:4096\n ds_read_b64_tr_b16 %[h2], %[rb] offset:4608\n"
                 "ds_read_b128 %[x3], %[ra3]\n ds_read_b64_tr_b16 %[l3], %[rb] offset:6144\n ds_read_b64_tr_b16 %[h3], %[rb] offset:6656\n" PPLL_MMA
                 : [c] "+v"(acc), PPLL_NEXT_A, [l0] "=&v"(nb.lo[0]), [h0] "=&v"(nb.hi[0]), [l1] "=&v"(nb.lo[1]), [h1] "=&v"(nb.hi[1]),
                   [l2] "=&v"(nb.lo[2]), [h2] "=&v"(nb.hi[2]), [l3] "=&v"(nb.lo[3]), [h3] "=&v"(nb.hi[3])
                 : PPLL_CUR, [rb] "v"(addrB)
                 : "memory");
  } else {
    asm volatile("ds_read_b128 %[x0], %[ra0]\n ds_read_b128 %[y0], %[rb0]\n ds_read_b128 %[x1], %[ra1]\n ds_read_b128 %[y1], %[rb1]\n"
                 "ds_read_b128 %[x2], %[ra2]\n ds_read_b128 %[y2], %[rb2]\n ds_read_b128 %[x3], %[ra3]\n ds_read_b128 %[y3], %[rb3]\n" PPLL_MMA
                 : [c] "+v"(acc), PPLL_NEXT_A, [y0] "=&v"(nb.v[0]), [y1] "=&v"(nb.v[1]), [y2] "=&v"(nb.v[2]), [y3] "=&v"(nb.v[3])
                 : PPLL_CUR, [rb0] "v"(addrB), [rb1] "v"(addrB ^ 32), [rb2] "v"(addrB ^ 64), [rb3] "v"(addrB ^ 96)
                 : "memory");
  }
#undef PPLL_MMA
#undef PPLL_NEXT_A
#undef PPLL_CUR
}

template <bool BT>
__global__ __launch_bounds__(64 * (WAVES + COPY_WAVES), 4) void gemm_split_kernel(SplitArgs p) {
  PPLL_CODE_TO_L2(1);
  __shared__ __align__(1024) char smem[STAGES * STAGE];
  const int slot = blockIdx.x >> 3;
  if (slot >= p.map.per_xcd) {
    const Bring b{p.A, p.B, p.side, p.a_bytes, p.b_bytes, p.s_bytes, (int)(p.lda * 2), (int)(p.ldb * 2), (int)(p.lds * 2), p.M, p.N, p.K, EDGE, EDGE, p.helpers};
    bring_operands<BT, 64 * (WAVES + COPY_WAVES)>(b, p.map, blockIdx.x & 7, slot - p.map.per_xcd, (lds_char*)code_words__);
    return;
  }
  int tm, tn;
  if (!tile_at(p.map, blockIdx.x & 7, slot, tm, tn)) return;
  const int m0 = tm * EDGE, n0 = tn * EDGE;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int K = p.K, stages = (K + KT - 1) / KT;
  lds_char* lds = (lds_char*)smem;
  if (wave >= WAVES) {
    const int w = wave - WAVES;
    if (w & 1) copy_stages<BT>(p.B, p.b_bytes, p.ldb, n0, p.N, lane, w >> 1, lds + OPER, stages, K);
    else copy_stages<false>(p.A, p.a_bytes, p.lda, m0, p.M, lane, w >> 1, lds, stages, K);
    return;
  }
  const int mw = (wave >> 1) * 32, nw = (wave & 1) * 32;
  const int base = (int)(uintptr_t)lds, fa = base + frag<false>(mw, lane), fb = base + OPER + frag<BT>(nw, lane);
  // What the epilogue takes from memory, asked for ahead of the loop.  It has a row a lane, columns n .. n + 7 and n + 16 .. n + 23
  const bool has_aux = p.epilogue == EPI_DGELU, has_res = p.side && !has_aux;
  const int m = m0 + mw + (lane & 31), n = n0 + nw + 8 * (lane >> 5);
  u32x4 bias[2][2], side[2];
  {
    const __amdgpu_buffer_rsrc_t rsB = make_rsrc(p.bias, p.bias ? (uint32_t)p.N * 4u : 0u), rsS = make_rsrc(p.side, p.s_bytes);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      bias[u][0] = split_load16(rsB, 4 * (n + 16 * u));
      bias[u][1] = split_load16(rsB, 4 * (n + 16 * u) + 16);
      side[u] = split_load16(rsS, m < p.M && n + 16 * u < p.N ? (int)((m * p.lds + n + 16 * u) * 2) : OOB);
    }
  }
  f32x16 acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;
  Frags<false, 4> a0, a1;
  Frags<BT, 4> b0, b1;
  barrier();
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) { set_zero(a1, kk); set_zero(b1, kk); }
  split_stage<BT>(acc, a1, b1, a0, b0, fa, fb);         // the first fragments: products with zeros under the reads
  int rd = 0, i = 0;
  auto next = [&] { rd += STAGE; if (rd == STAGES * STAGE) rd = 0; };
  for (; i + 1 < stages; i += 2) {
    barrier();                                          // stage i + 1 is there, nobody reads stage i - 1 any more
    next();
    split_stage<BT>(acc, a0, b0, a1, b1, fa + rd, fb + rd);
    barrier();
    next();
    split_stage<BT>(acc, a1, b1, a0, b0, fa + rd, fb + rd);
  }
  if (i < stages) {
    barrier();
    split_stage<BT>(acc, a0, b0, a1, b1, fa + rd, fb + rd);
  }
  asm volatile("s_nop 15\n s_nop 3" : "+v"(acc)::"memory");     // the last products are through

  const __amdgpu_buffer_rsrc_t rsC = make_rsrc(p.C, p.c_bytes), rsC2 = make_rsrc(p.C2, p.C2 ? p.c_bytes : 0u);
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = acc[8 * u + e];
    // a lane has columns 4 (lane / 32) .. + 3 of two groups of 8: lanes 0 .. 31 get the first group, lanes 32 .. 63 the second
#pragma unroll
    for (int e = 0; e < 4; ++e) swap_halves(x[e], x[4 + e]);
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] += __uint_as_float(bias[u][e >> 2][e & 3]);
    if (has_res) {
#pragma unroll
      for (int e = 0; e < 4; ++e) { x[2 * e] += __uint_as_float(side[u][e] << 16); x[2 * e + 1] += __uint_as_float(side[u][e] & 0xffff0000u); }
    }
    if (has_aux) {   // the saved GELU derivative
#pragma unroll
      for (int e = 0; e < 4; ++e) { x[2 * e] *= __uint_as_float(side[u][e] << 16); x[2 * e + 1] *= __uint_as_float(side[u][e] & 0xffff0000u); }
    }
    const int off = m < p.M && n + 16 * u < p.N ? (int)((m * p.ldc + n + 16 * u) * 2) : OOB;   // N is a multiple of 8
    if (p.epilogue == EPI_GELU) {   // C2 = gelu(h), C = gelu'(h) from one evaluation of the normal CDF and density
      float dg[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float cdf, pdf;
        cdf_pdf(x[e], cdf, pdf);
        dg[e] = cdf + x[e] * pdf; x[e] *= cdf;
      }
      __builtin_amdgcn_raw_buffer_store_b128(pack8(dg), rsC, off, 0, 0);
      __builtin_amdgcn_raw_buffer_store_b128(pack8(x), rsC2, off, 0, 0);
    } else {
      __builtin_amdgcn_raw_buffer_store_b128(pack8(x), rsC, off, 0, 0);
    }
  }
}

}  // namespace

bool gemm_split_choice(const GemmArgs& g) { return gemm_split_supported(g) && split_tiles(g.M, g.N, g.K, product_units(g)); }
bool gemm_split_supported(const GemmArgs& g) { return gemm_pipe_supported(g) && !(g.residual && g.epilogue == EPI_DGELU); }

int launch_gemm_split(hipStream_t s, const GemmArgs& g) {
  const bool bt = g.b_sn == 1 && g.b_sk != 1;
  SplitArgs p{};
  p.A = (const uint16_t*)g.A; p.lda = g.a_sm;
  p.B = (const uint16_t*)g.B; p.ldb = bt ? g.b_sk : g.b_sn;
  p.C = (uint16_t*)g.C; p.ldc = g.ldc;
  p.M = g.M; p.N = g.N; p.K = g.K;
  p.bias = g.bias; p.epilogue = g.epilogue; p.C2 = (uint16_t*)g.C2;
  const bool dgelu = g.epilogue == EPI_DGELU;
  p.side = (const uint16_t*)(dgelu ? g.aux : g.residual); p.lds = dgelu ? g.ldaux : g.ldr;
  p.a_bytes = (uint32_t)(((long)(g.M - 1) * p.lda + g.K) * 2);
  p.b_bytes = (uint32_t)((bt ? (long)(g.K - 1) * p.ldb + g.N : (long)(g.N - 1) * p.ldb + g.K) * 2);
  p.c_bytes = (uint32_t)(((long)(g.M - 1) * g.ldc + g.N) * 2);
  p.s_bytes = p.side ? (uint32_t)(((long)(g.M - 1) * p.lds + g.N) * 2) : 0u;
  const int units = product_units(g);
  p.map = tile_map(g.M, g.N, EDGE, EDGE, units);
  p.helpers = g.shared ? 0 : helper_workgroups(p.map.per_xcd, units);
  const dim3 grid(8 * (p.map.per_xcd + p.helpers)), block(64 * (WAVES + COPY_WAVES));
  void* prof = nullptr;
  PPLL_TRY(profile_begin(s, 2.0 * g.M * g.N * g.K, &prof));
  if (bt) hipLaunchKernelGGL(gemm_split_kernel<true>, grid, block, 0, s, p);
  else hipLaunchKernelGGL(gemm_split_kernel<false>, grid, block, 0, s, p);
  PPLL_HIP(hipGetLastError());
  return profile_end(s, prof);
}

}  // namespace ppll
