// Linear-layer products whose 64 x 64 output tiles find a compute unit each: C[M,N] = A[M,K] B, bf16 operands, fp32 accumulation,
// the epilogues of the tiled kernel.
//
// With so few tiles a product takes as long as one tile does, and what bounds that is the chain along k.  A 64 x 128 tile whose four
// waves copy through registers, multiply and meet at a barrier spends 0.4 us per 64 k (640 x 768 x 3072: 22 us on 60 of 256
// units), four times what its products take, because the phases follow one another.  Here they run beside one another: four waves
// do nothing but copy, straight from memory to LDS, three stages ahead of eight waves that multiply; those share out the four
// k steps of a stage of 64 k, so that each barrier has two products a wave behind it, and add up at the end.  A copy takes rows of
// 128 bytes, whole cache lines: with 64 bytes a row the loop took half as long again, the lines being fetched twice from beyond L2.
// Smaller tiles find more units and copy more per product; beyond one a unit the tiled kernel is ahead.  64 KB of LDS and 62
// registers a wave leave room for a workgroup of another stream (with stages twice as deep and no more waves a pipeline of three
// blocks of width 192, 4160 rows, took 570 us a batch instead of 520).
// Microseconds, tiled kernel -> this one: 640 x 768 x 768 8.6 -> 6.2, 640 x 768 x 2304 18.2 -> 12.0, 640 x 768 x 3072 22.2 -> 14.8,
// 1500 x 384 x 384 6.1 -> 4.5, 1500 x 384 x 1536 13.2 -> 9.0; a step of 3 + 1 layers of width 768, 640 rows, 756 -> 678.
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
  int M, N, K, tiles_n, tiles, per_xcd;
  const float* bias;
  const uint16_t* side; long lds;   // residual, or the saved GELU derivative (EPI_DGELU)
  int epilogue;
  uint16_t* C2;
  uint32_t a_bytes, b_bytes, c_bytes, s_bytes;
};

constexpr int EDGE = 64, KT = 64;    // tile, k of a stage: 128 bytes, one cache line, of a row of an operand with k contiguous
constexpr int WAVES = 8, COPY_WAVES = 4, STAGES = 4;
constexpr int GROUPS = WAVES / 2;     // of two waves, side by side, each 64 x 32 of the tile; group g takes k step g of a stage
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
// lane address of the fragment of rows row0 .. row0 + 31 at k step kk
template <bool TR> __device__ __forceinline__ int frag(int row0, int kk, int lane) {
  const int half = lane >> 5, r = lane & 31;
  if (!TR) return (row0 + r) * 128 + (((2 * kk + half) ^ ((r >> 1) & 7)) << 4);
  const int k = 16 * kk + 8 * half + ((lane & 15) >> 2);
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

// A copying wave, from the first stage to the last.  Barriers: one with stage 0 in LDS, one per stage, two behind the loop.
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
  wait_vm<0>();
  barrier();
  barrier();
}

// One k step of a wave, 64 rows x 32 columns: the products of the fragments at hand, and under them the reads of the next ones, which
// are there when the block ends (one block, because the compiler would order LDS reads that it knows of behind the copies into LDS).
template <bool BT>
__device__ __forceinline__ void split_step(f32x16 (&acc)[2], const Frags<false, 2>& a, const Frags<BT, 1>& b, Frags<false, 2>& na, Frags<BT, 1>& nb,
                                           int addrA, int addrB) {
#define PPLL_MMA "v_mfma_f32_32x32x16_bf16 %[c0], %[q], %[p0], %[c0]\n v_mfma_f32_32x32x16_bf16 %[c1], %[q], %[p1], %[c1]\n s_waitcnt lgkmcnt(0)"
  if constexpr (BT) {
    asm volatile("ds_read_b128 %[x0], %[ra]\n ds_read_b64_tr_b16 %[lo], %[rb]\n ds_read_b64_tr_b16 %[hi], %[rb] offset:512\n"   // k + 4: the same window
                 "ds_read_b128 %[x1], %[ra] offset:4096\n" PPLL_MMA
                 : [c0] "+v"(acc[0]), [c1] "+v"(acc[1]), [x0] "=&v"(na.v[0]), [x1] "=&v"(na.v[1]), [lo] "=&v"(nb.lo[0]), [hi] "=&v"(nb.hi[0])
                 : [p0] "v"(a.get(0)), [p1] "v"(a.get(1)), [q] "v"(b.get(0)), [ra] "v"(addrA), [rb] "v"(addrB)
                 : "memory");
  } else {
    asm volatile("ds_read_b128 %[x0], %[ra]\n ds_read_b128 %[y], %[rb]\n ds_read_b128 %[x1], %[ra] offset:4096\n" PPLL_MMA
                 : [c0] "+v"(acc[0]), [c1] "+v"(acc[1]), [x0] "=&v"(na.v[0]), [x1] "=&v"(na.v[1]), [y] "=&v"(nb.v[0])
                 : [p0] "v"(a.get(0)), [p1] "v"(a.get(1)), [q] "v"(b.get(0)), [ra] "v"(addrA), [rb] "v"(addrB)
                 : "memory");
  }
#undef PPLL_MMA
}

template <bool BT>
__global__ __launch_bounds__(64 * (WAVES + COPY_WAVES), 3) void gemm_split_kernel(SplitArgs p) {
  __shared__ __align__(1024) char smem[STAGES * STAGE];
  // XCD x (workgroup id % 8) takes a contiguous range of the tiles, row by row: they share operand panels in its L2
  const int slot = blockIdx.x >> 3, t = (blockIdx.x & 7) * p.per_xcd + slot;
  if (slot >= p.per_xcd || t >= p.tiles) return;
  const int m0 = t / p.tiles_n * EDGE, n0 = t % p.tiles_n * EDGE;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int K = p.K, stages = (K + KT - 1) / KT;
  lds_char* lds = (lds_char*)smem;
  if (wave >= WAVES) {
    const int w = wave - WAVES;
    if (w & 1) copy_stages<BT>(p.B, p.b_bytes, p.ldb, n0, p.N, lane, w >> 1, lds + OPER, stages, K);
    else copy_stages<false>(p.A, p.a_bytes, p.lda, m0, p.M, lane, w >> 1, lds, stages, K);
    return;
  }
  const int grp = wave >> 1, nw = n0 + (wave & 1) * 32;
  f32x16 acc[2];
  {   // the accumulators of the first group start from the bias: a lane holds columns 8 q + 4 (lane / 32) .. + 3
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(p.bias, p.bias && grp == 0 ? (uint32_t)p.N * 4u : 0u);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const u32x4 b = split_load16(rs, 4 * (nw + 8 * q + 4 * (lane >> 5)));
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[0][4 * q + e] = acc[1][4 * q + e] = __uint_as_float(b[e]);
    }
  }
  const int base = (int)(uintptr_t)lds, fa = base + frag<false>(0, grp, lane), fb = base + OPER + frag<BT>((wave & 1) * 32, grp, lane);
  Frags<false, 2> a0, a1;
  Frags<BT, 1> b0, b1;
  barrier();
  set_zero(a1, 0); set_zero(a1, 1); set_zero(b1, 0);
  split_step<BT>(acc, a1, b1, a0, b0, fa, fb);          // the first fragments: products with zeros under the reads
  int rd = 0, i = 0;
  auto next = [&] { rd += STAGE; if (rd == STAGES * STAGE) rd = 0; };
  for (; i + 1 < stages; i += 2) {
    barrier();                       // stage i + 1 is there, nobody reads stage i - 1 any more
    next();
    split_step<BT>(acc, a0, b0, a1, b1, fa + rd, fb + rd);
    barrier();
    next();
    split_step<BT>(acc, a1, b1, a0, b0, fa + rd, fb + rd);
  }
  if (i < stages) {
    barrier();
    split_step<BT>(acc, a0, b0, a1, b1, fa + rd, fb + rd);
  }
  asm volatile("s_nop 15\n s_nop 3" : "+v"(acc[0]), "+v"(acc[1])::"memory");     // the last products are through

  // Epilogue.  The four units of a wave's tile, 32 rows x 16 columns each, go to the four groups: a wave gives the others' to LDS, lane
  // for lane, and adds up its own in the order of the groups.
  const bool has_aux = p.epilogue == EPI_DGELU, has_res = p.side && !has_aux;
  const int m = m0 + 32 * (grp >> 1) + (lane & 31), n = nw + 16 * (grp & 1) + 8 * (lane >> 5);
  const bool ok = m < p.M && n < p.N;      // N is a multiple of 8
  u32x4 side = {0, 0, 0, 0};
  if (p.side) side = split_load16(make_rsrc(p.side, p.s_bytes), ok ? (int)((m * p.lds + n) * 2) : OOB);
  barrier();            // no copy is under way and nobody reads a stage any more
  float4* units = reinterpret_cast<float4*>(smem) + (wave & 1) * (GROUPS * 4 * 128) + lane;   // [group][unit][2][64 lanes]
  static_assert(WAVES * 4 * 128 * 16 <= STAGES * STAGE, "");
  float own[8], x[8];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int i2 = u >> 1, b = 8 * (u & 1);
    if (u != grp) {
      units[(grp * 4 + u) * 128] = make_float4(acc[i2][b], acc[i2][b + 1], acc[i2][b + 2], acc[i2][b + 3]);
      units[(grp * 4 + u) * 128 + 64] = make_float4(acc[i2][b + 4], acc[i2][b + 5], acc[i2][b + 6], acc[i2][b + 7]);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) own[e] = acc[i2][b + e];
    }
  }
  __syncthreads();
#pragma unroll
  for (int g = 0; g < GROUPS; ++g) {
    float4 lo = make_float4(own[0], own[1], own[2], own[3]), hi = make_float4(own[4], own[5], own[6], own[7]);
    if (g != grp) { lo = units[(g * 4 + grp) * 128]; hi = units[(g * 4 + grp) * 128 + 64]; }
    const float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = g ? x[e] + v[e] : v[e];
  }
  // lanes 0..31 get columns 0..7, lanes 32..63 columns 8..15 of the unit
#pragma unroll
  for (int e = 0; e < 4; ++e) swap_halves(x[e], x[4 + e]);
  if (has_res) {
#pragma unroll
    for (int e = 0; e < 4; ++e) { x[2 * e] += __uint_as_float(side[e] << 16); x[2 * e + 1] += __uint_as_float(side[e] & 0xffff0000u); }
  }
  if (has_aux) {   // the saved GELU derivative
#pragma unroll
    for (int e = 0; e < 4; ++e) { x[2 * e] *= __uint_as_float(side[e] << 16); x[2 * e + 1] *= __uint_as_float(side[e] & 0xffff0000u); }
  }
  const __amdgpu_buffer_rsrc_t rsC = make_rsrc(p.C, p.c_bytes);
  const int off = ok ? (int)((m * p.ldc + n) * 2) : OOB;
  if (p.epilogue == EPI_GELU) {   // C2 = gelu(h), C = gelu'(h) from one evaluation of the normal CDF and density
    float dg[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float cdf, pdf;
      cdf_pdf(x[e], cdf, pdf);
      dg[e] = cdf + x[e] * pdf; x[e] *= cdf;
    }
    __builtin_amdgcn_raw_buffer_store_b128(pack8(dg), rsC, off, 0, 0);
    __builtin_amdgcn_raw_buffer_store_b128(pack8(x), make_rsrc(p.C2, p.c_bytes), off, 0, 0);
  } else {
    __builtin_amdgcn_raw_buffer_store_b128(pack8(x), rsC, off, 0, 0);
  }
}

}  // namespace

bool gemm_split_choice(const GemmArgs& g) { return gemm_split_supported(g) && split_tiles(g.M, g.N, g.K, compute_units()); }
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
  p.tiles_n = (g.N + EDGE - 1) / EDGE;
  p.tiles = (g.M + EDGE - 1) / EDGE * p.tiles_n;
  p.per_xcd = (p.tiles + 7) / 8;
  const dim3 grid(8 * p.per_xcd), block(64 * (WAVES + COPY_WAVES));
  void* prof = nullptr;
  PPLL_TRY(profile_begin(s, 2.0 * g.M * g.N * g.K, &prof, g.M < 256 ? 2 : 0));   // few output rows: a class of its own
  if (bt) hipLaunchKernelGGL(gemm_split_kernel<true>, grid, block, 0, s, p);
  else hipLaunchKernelGGL(gemm_split_kernel<false>, grid, block, 0, s, p);
  PPLL_HIP(hipGetLastError());
  return profile_end(s, prof);
}

}  // namespace ppll
