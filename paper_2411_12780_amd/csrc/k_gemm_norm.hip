// Linear-layer products whose result goes through a LayerNorm next, both in one launch: bf16 operands, fp32 accumulation, results bit for
// bit those of the product kernels and the LayerNorm kernels (the same order of k, the same row code: ln_rows.h).
//  forward: x = A B + bias + residual is stored, and y = LayerNorm(x) with its means and deviations;
//  backward: dy = A B, rounded as it would be stored, goes through the LayerNorm's backward pass and is stored nowhere.
//
// What bounds a LayerNorm launch is its start and its rows' way from and to memory; what the product leaves in registers it has to fetch again.
// A workgroup owns 64 whole rows, 192 or 384 columns: four or eight waves of 32 rows x 96 columns, operands through registers into two
// stages of 64 k in LDS (more of them do not fit beside 384 columns), the finished tile as fp32 in LDS, from which lane groups take whole
// rows as the LayerNorm kernels hold them.  At width 192 two workgroups share a unit, so that one multiplies while the other copies.
// Microseconds as two launches and here, 8320 rows of width 192: K = 192 forward 11.4 -> 7.5, K = 768 16.1 -> 12.1, backward 20.9 -> 18.0;
// steps of 3 + 1 layers of width 192, 8320 rows, 543 -> 507, 2 + 1 layers of 25216 rows 778 -> 744.  The rule and its figures: norm_tiles() and
// norm_with_product().
#include "common.h"
#include "ln_rows.h"
#include "plan.h"

namespace ppll {

namespace {
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;

constexpr int OOB = 0x7fffffff;        // no buffer here reaches 2^30 bytes (checked on the host)
constexpr int OOB_BASE = 0x40000000;   // stays out of range after anything below 2^30 is added
constexpr int BM = 64, BK = 64;

struct NormArgs {
  const uint16_t* A; long lda;      // A[m*lda + k]
  const uint16_t* B; long ldb;      // BT ? B[k*ldb + n] : B[n*ldb + k]
  int M, K;
  uint32_t a_bytes, b_bytes;
  const float* g;                   // the LayerNorm's scale
  // forward
  const float* bias; const uint16_t* residual;
  uint16_t* x_out;
  const float* b; float eps;
  uint16_t* y; float *mean_out, *rstd_out;
  // backward
  const uint16_t* x; const float *mean, *rstd;
  const uint16_t* dres; uint16_t* dx;       // dx may be null
  float* partial;
};

template <bool BT, int N_> struct NormShape {
  static constexpr int N = N_, WN = N / 96, W = 2 * WN, TH = 64 * W;
  // [64 k][N] rows of B: the next row's banks 64 bytes on (or back), as in the tiled kernel
  static constexpr int PITCH = 2 * N + 64;
  static constexpr int A_BYTES = BM * 128, B_BYTES = BT ? BK * PITCH : N * 128, SLOT = A_BYTES + B_BYTES;
  static constexpr int NA = BM * 8 / TH, NB = N * 8 / TH;      // 16-byte pieces of a stage a thread
  static constexpr int FP = N + 4;                             // floats of a row of the finished tile
  static constexpr int TILE = BM * FP * 4, SUMS = LNB_WAVES * 2 * N * 4;
  static constexpr int LDS = 2 * SLOT > TILE + SUMS ? 2 * SLOT : TILE + SUMS;
  static_assert(NB == 6 && WN * 96 == N, "");
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t norm_rsrc(const void* ptr, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(ptr), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ uint4 norm_load16(__amdgpu_buffer_rsrc_t r, int off) {
  const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
  return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ uint2 norm_read_tr(const char* p) {   // see the tiled kernel
  const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p);
  return __builtin_bit_cast(uint2, v);
}
// [row][64 k]: rows of 128 bytes, the 16-byte granule of a row turned by its row
__device__ __forceinline__ int granule(int row, int g) { return row * 128 + ((g ^ ((row >> 1) & 7)) << 4); }

template <bool BT, int N, bool BWD>
__global__ __launch_bounds__((NormShape<BT, N>::TH), 2) void gemm_norm_kernel(NormArgs p) {
  PPLL_CODE_TO_L2(2);
  using S = NormShape<BT, N>;
  using L = LnShape<N>;
  constexpr int NA = S::NA, NB = S::NB, TH = S::TH;
  extern __shared__ __align__(16) char smem[];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int wm = wave / S::WN, wn = wave % S::WN, m0 = blockIdx.x * BM;
  const int nk = (p.K + BK - 1) / BK;

  f32x16 acc[3];
#pragma unroll
  for (int j = 0; j < 3; ++j)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[j][e] = 0.f;

  // ---- operands: memory -> registers -> LDS, a stage of 64 k at a time
  const __amdgpu_buffer_rsrc_t rsA = norm_rsrc(p.A, p.a_bytes), rsB = norm_rsrc(p.B, p.b_bytes);
  const int lda2 = (int)(p.lda * 2), ldb2 = (int)(p.ldb * 2);
  const int gk = (tid & 7) * 8;                       // first k of this thread's granules of an operand with k contiguous
  int offA[NA], offB[BT ? 3 : 1];
#pragma unroll
  for (int q = 0; q < NA; ++q) {
    const int row = m0 + (tid >> 3) + q * (TH / 8);
    offA[q] = row < p.M ? row * lda2 + gk * 2 : OOB_BASE;
  }
  // BT: a wave brings 64 / W k rows, 3 pieces a lane for every BK rows / 2: piece q of lane l is granule (l + 64 q) % (N / 8) of k row
  // (l + 64 q) / (N / 8), and pieces q and q + 3 are 24 * 8 / N rows apart
  constexpr int G = N / 8, KROWS = BK / S::W, HALF = 3 * 64 / G;
  int krow[BT ? 3 : 1];
  if (BT) {
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const int i = lane + 64 * q, kr = wave * KROWS + i / G;
      krow[BT ? q : 0] = kr;
      offB[BT ? q : 0] = kr * ldb2 + (i % G) * 16;
    }
  } else {
    offB[0] = (tid >> 3) * ldb2 + gk * 2;
  }
  static_assert(2 * HALF == KROWS && HALF * G == 192, "");
  struct Regs { uint4 a[NA], b[NB]; };
  auto gload = [&](int i, Regs& r) {
    const int k0 = i * BK;
    const bool kin = k0 + gk < p.K;
#pragma unroll
    for (int q = 0; q < NA; ++q) r.a[q] = norm_load16(rsA, kin ? offA[q] + 2 * k0 : OOB);
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      if (BT) {
        const int h = q / 3 * HALF, j = BT ? q % 3 : 0;
        r.b[q] = norm_load16(rsB, k0 + krow[j] + h < p.K ? offB[j] + (k0 + h) * ldb2 : OOB);
      } else {
        r.b[q] = norm_load16(rsB, kin ? offB[0] + q * (TH / 8) * ldb2 + 2 * k0 : OOB);
      }
    }
  };
  // part u (0 .. 3) of the thread's writes of a stage
  auto lstore = [&](int slot, const Regs& r, int u) {
    char* la = smem + slot * S::SLOT;
    char* lb = la + S::A_BYTES;
    if (u == 3) {
#pragma unroll
      for (int q = 0; q < NA; ++q) *reinterpret_cast<uint4*>(la + granule((tid >> 3) + q * (TH / 8), tid & 7)) = r.a[q];
      return;
    }
#pragma unroll
    for (int q = 2 * u; q < 2 * u + 2; ++q) {
      if (BT) {
        const int i = lane + 64 * (q % 3), kr = wave * KROWS + i / G + q / 3 * HALF;
        *reinterpret_cast<uint4*>(lb + kr * S::PITCH + (i % G) * 16) = r.b[q];
      } else {
        *reinterpret_cast<uint4*>(lb + granule((tid >> 3) + q * (TH / 8), tid & 7)) = r.b[q];
      }
    }
  };
  const int fr = lane & 31, fh = lane >> 5;
  const int tr_lane = (8 * fh + ((lane & 15) >> 2)) * S::PITCH + (16 * ((lane >> 4) & 1) + 4 * (lane & 3)) * 2;
  auto load_frags = [&](int slot, int kk, bf16x8& fa, bf16x8 (&fb)[3]) {
    const char* la = smem + slot * S::SLOT;
    const char* lb = la + S::A_BYTES;
    fa = *reinterpret_cast<const bf16x8*>(la + granule(wm * 32 + fr, 2 * kk + fh));
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const int n0 = wn * 96 + j * 32;
      if (BT) {
        const char* q = lb + tr_lane + kk * 16 * S::PITCH + n0 * 2;
        const uint2 lo = norm_read_tr(q), hi = norm_read_tr(q + 4 * S::PITCH);
        fb[j] = __builtin_bit_cast(bf16x8, make_uint4(lo.x, lo.y, hi.x, hi.y));
      } else {
        fb[j] = *reinterpret_cast<const bf16x8*>(lb + granule(n0 + fr, 2 * kk + fh));
      }
    }
  };
  bf16x8 fa[2], fb[2][3];
  auto multiply = [&](int slot, const Regs& rn, bool next) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      if (kk < 3) load_frags(slot, kk + 1, fa[(kk + 1) & 1], fb[(kk + 1) & 1]);
#pragma unroll
      for (int j = 0; j < 3; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[kk & 1][j], fa[kk & 1], acc[j], 0, 0, 0);
      if (next) lstore(slot ^ 1, rn, kk);
    }
  };
  // Two stages in LDS and two in registers: stage t travels in register set t % 2 and slot t % 2; while stage i is multiplied, i + 1
  // moves from registers to LDS and i + 2 and i + 3 are on their way from memory.
  Regs r[2];
  gload(0, r[0]);
  gload(1, r[1]);
#pragma unroll
  for (int u = 0; u < 4; ++u) lstore(0, r[0], u);
  __syncthreads();
  gload(2, r[0]);
  load_frags(0, 0, fa[0], fb[0]);
  auto step = [&](int u, Regs& rn, int i) {
    multiply(u, rn, true);
    __syncthreads();
    load_frags(u ^ 1, 0, fa[0], fb[0]);
    gload(i + 3, rn);
  };
  int i = 0;
  for (; i + 2 < nk; i += 2) {
    step(0, r[1], i);
    step(1, r[0], i + 1);
  }
  if (nk - i == 2) {
    step(0, r[1], i);
    multiply(1, r[0], false);
  } else {
    multiply(0, r[1], false);
  }

  // ---- whole rows: lane groups of LPR lanes, wave w of pass q has the rows of wave q W + w of the LayerNorm kernels
  constexpr int LPR = L::LPR, NV = L::NV, RPW = L::RPW;
  static_assert(2 * S::W * RPW == BM && (2 * S::W) % LNB_WAVES == 0, "two passes");
  const int lr = lane % LPR;
  auto row_of = [&](int pass) { return (pass * S::W + wave) * RPW + lane / LPR; };
  uint4 e0[2][NV], e1[2][NV];      // residual; x and the residual gradient
  float mu[2], rs[2];
  auto ask = [&](int pass) {
    const int m = m0 + row_of(pass);
    const bool ok = m < p.M;
    mu[pass] = rs[pass] = 0.f;
    if (BWD && ok) { mu[pass] = p.mean[m]; rs[pass] = p.rstd[m]; }
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const size_t at = (size_t)m * N + 8 * lr + 8 * LPR * j;
      e0[pass][j] = e1[pass][j] = make_uint4(0, 0, 0, 0);
      if (ok) {
        e0[pass][j] = *reinterpret_cast<const uint4*>((BWD ? p.x : p.residual) + at);
        if (BWD && p.dres) e1[pass][j] = *reinterpret_cast<const uint4*>(p.dres + at);
      }
    }
  };
  ask(0);
  __syncthreads();                 // every wave is done with the operand stages
  float* tile = reinterpret_cast<float*>(smem);
#pragma unroll
  for (int j = 0; j < 3; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<float4*>(tile + (wm * 32 + fr) * S::FP + wn * 96 + j * 32 + 8 * q + 4 * fh) =
          make_float4(acc[j][4 * q], acc[j][4 * q + 1], acc[j][4 * q + 2], acc[j][4 * q + 3]);
  ask(1);
  __syncthreads();
  float* sums = reinterpret_cast<float*>(smem + S::TILE);
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    const int row = row_of(pass), m = m0 + row;
    const bool ok = m < p.M;
    float v[8 * NV];
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const float* t = tile + row * S::FP + 8 * lr + 8 * LPR * j;
      const float4 lo = *reinterpret_cast<const float4*>(t), hi = *reinterpret_cast<const float4*>(t + 4);
      const float f[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
      for (int e = 0; e < 8; ++e) v[8 * j + e] = f[e];
    }
    uint4 w[NV], o[NV];
    if (!BWD) {
#pragma unroll
      for (int j = 0; j < NV; ++j) {
        const int c = 8 * lr + 8 * LPR * j;
        const float4 lo = *reinterpret_cast<const float4*>(p.bias + c), hi = *reinterpret_cast<const float4*>(p.bias + c + 4);
        const float bias[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
        float res[8];
        unpack8(e0[pass][j], res);
#pragma unroll
        for (int e = 0; e < 8; ++e) { v[8 * j + e] += bias[e]; v[8 * j + e] += res[e]; }
      }
    }
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      w[j] = make_uint4(pack_bf(v[8 * j], v[8 * j + 1]), pack_bf(v[8 * j + 2], v[8 * j + 3]), pack_bf(v[8 * j + 4], v[8 * j + 5]),
                        pack_bf(v[8 * j + 6], v[8 * j + 7]));
      if (!ok) w[j] = make_uint4(0, 0, 0, 0);      // a row that is not there is 0 times B, whatever B holds
    }
    if (!BWD) {
      float mean, rstd;
      if (ok)
#pragma unroll
        for (int j = 0; j < NV; ++j) store_through(p.x_out + (size_t)m * N + 8 * lr + 8 * LPR * j, w[j]);
      ln_fwd_row<L>(w, lr, p.g, p.b, p.eps, mean, rstd, o);
      if (ok) {
#pragma unroll
        for (int j = 0; j < NV; ++j) store_through(p.y + (size_t)m * N + 8 * lr + 8 * LPR * j, o[j]);
        if (lr == 0) { p.mean_out[m] = mean; p.rstd_out[m] = rstd; }
      }
    } else {
      float adg[8 * NV], adb[8 * NV];
#pragma unroll
      for (int c = 0; c < 8 * NV; ++c) adg[c] = adb[c] = 0.f;
      ln_bwd_row<L, false>(e0[pass], w, e1[pass], ok, mu[pass], rs[pass], lr, p.g, adg, adb, o);
      if (ok && p.dx)
#pragma unroll
        for (int j = 0; j < NV; ++j) store_through(p.dx + (size_t)m * N + 8 * lr + 8 * LPR * j, o[j]);
      ln_bwd_fold<L>(adg, adb, lane, sums + (pass * S::W + wave) % LNB_WAVES * 2 * N);
      // LNB_WAVES of the LayerNorm kernel's waves make a chunk: one of them a pass, or both passes together
      if ((pass + 1) * S::W % LNB_WAVES == 0) {
        constexpr int CHUNK = LNB_WAVES * RPW;
        const int chunk = ((pass + 1) * S::W / LNB_WAVES - 1) + blockIdx.x * (BM / CHUNK);
        __syncthreads();
        if (chunk * CHUNK < p.M) ln_bwd_sum<N>(sums, p.partial + (size_t)chunk * 2 * N, tid, TH);
        __syncthreads();
      }
    }
  }
}

template <bool BT, int N, bool BWD>
int norm_launch(hipStream_t s, const NormArgs& p) {
  using S = NormShape<BT, N>;
  static OncePerDevice once;
  PPLL_TRY(raise_lds((const void*)gemm_norm_kernel<BT, N, BWD>, S::LDS, once));
  hipLaunchKernelGGL((gemm_norm_kernel<BT, N, BWD>), dim3((p.M + BM - 1) / BM), dim3(S::TH), S::LDS, s, p);
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}
template <bool BWD>
int norm_dispatch(hipStream_t s, const GemmArgs& g, NormArgs& p) {
  const bool bt = g.b_sn == 1 && g.b_sk != 1;
  p.A = (const uint16_t*)g.A; p.lda = g.a_sm;
  p.B = (const uint16_t*)g.B; p.ldb = bt ? g.b_sk : g.b_sn;
  p.M = g.M; p.K = g.K;
  p.a_bytes = (uint32_t)(((long)(g.M - 1) * p.lda + g.K) * 2);
  p.b_bytes = (uint32_t)((bt ? (long)(g.K - 1) * p.ldb + g.N : (long)(g.N - 1) * p.ldb + g.K) * 2);
  void* prof = nullptr;
  PPLL_TRY(profile_begin(s, 2.0 * g.M * g.N * g.K, &prof));
  // a block has its forward products with B [K][N] and its input gradients with [N][K]; the other two forms serve the test of the kernel
  if (g.N == 384) PPLL_TRY((bt ? norm_launch<true, 384, BWD>(s, p) : norm_launch<false, 384, BWD>(s, p)));
  else PPLL_TRY((bt ? norm_launch<true, 192, BWD>(s, p) : norm_launch<false, 192, BWD>(s, p)));
  return profile_end(s, prof);
}
bool al16(const void* q) { return !(((uintptr_t)q) & 15); }
bool product_ok(const GemmArgs& g) {
  return (g.N == 192 || g.N == 384) && g.a_sk == 1 && !g.colsum && g.c_dt == BF16 && g.epilogue == EPI_NONE && g.K >= 8 && gemm_mfma_supported(g) &&
         g.a_sm <= (1 << 20) && (g.b_sn == 1 && g.b_sk != 1 ? g.b_sk : g.b_sn) <= (1 << 20);
}
}  // namespace

bool gemm_norm_fwd_supported(const GemmArgs& g, const NormOut& n) {
  return product_ok(g) && g.bias && g.residual && g.ldc == g.N && g.ldr == g.N && al16(n.g) && al16(n.b) && al16(n.y);
}
bool gemm_norm_bwd_supported(const GemmArgs& g, const NormGrad& n) {
  return product_ok(g) && !g.bias && !g.residual && layernorm_bwd_rows(g.M, g.N) == LNB_WAVES * (g.N == 384 ? LnShape<384>::RPW : LnShape<192>::RPW) &&
         al16(n.x) && al16(n.g) && al16(n.dres) && al16(n.dx);
}

int launch_gemm_norm_fwd(hipStream_t s, const GemmArgs& g, const NormOut& n) {
  NormArgs p{};
  p.bias = g.bias; p.residual = (const uint16_t*)g.residual; p.x_out = (uint16_t*)g.C;
  p.g = n.g; p.b = n.b; p.eps = n.eps; p.y = (uint16_t*)n.y; p.mean_out = n.mean; p.rstd_out = n.rstd;
  return norm_dispatch<false>(s, g, p);
}

int launch_gemm_norm_bwd(hipStream_t s, const GemmArgs& g, const NormGrad& n, ReduceQueue& rq) {
  NormArgs p{};
  bool queued;
  p.partial = rq.space(layernorm_bwd_partial_floats(g.M, g.N, BF16), &queued);
  p.x = (const uint16_t*)n.x; p.mean = n.mean; p.rstd = n.rstd; p.g = n.g; p.dres = (const uint16_t*)n.dres; p.dx = (uint16_t*)n.dx;
  PPLL_TRY(norm_dispatch<true>(s, g, p));
  const int per = layernorm_bwd_rows(g.M, g.N);
  return layernorm_bwd_reduce(s, rq, queued, p.partial, (g.M + per - 1) / per, g.N, n.dg, n.db);
}

}  // namespace ppll
