// Shared declarations of the HIP implementation: element types, error plumbing
// and the launcher interface between the block engine and the kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <functional>
#include <vector>
#include <stddef.h>
#include <stdint.h>

#include "../../include/ppll.h"
#include "device.h"

namespace ppll {

// Element type of a buffer as seen by a kernel.
enum DType : int { F32 = 0, BF16 = 1 };
inline size_t dtype_size(int dt) { return dt == BF16 ? 2 : 4; }

void set_error(const char* fmt, ...);

#define PPLL_HIP(expr)                                                              \
  do {                                                                              \
    hipError_t e__ = (expr);                                                        \
    if (e__ != hipSuccess) {                                                        \
      ::ppll::set_error("%s failed: %s (%s:%d)", #expr, hipGetErrorString(e__),     \
                        __FILE__, __LINE__);                                        \
      return PPLL_ERR_HIP;                                                          \
    }                                                                               \
  } while (0)

#define PPLL_TRY(expr)                \
  do {                                \
    int s__ = (expr);                 \
    if (s__ != PPLL_OK) return s__;   \
  } while (0)

// More than 64 KB of dynamic LDS needs an opt-in per kernel, and the attribute belongs to a device's copy of the kernel: raises
// it on the current device.  `bytes` is the most that any launch of the kernel asks for, never the size at hand: a thread with a
// smaller one would lower what another has just raised.
int raise_lds(const void* kernel, int bytes, OncePerDevice& once);
// Compute units of the current device, 0 where there is none.  The rules of most launches ask, so the runtime is asked once per
// device: its query takes 117 ns, and a batch of a four-block pipeline of small blocks, bound by the host, asked some 130 times.
int compute_units();

#ifdef __HIPCC__
// bf16 <-> fp32 by bit manipulation, round to nearest even.
__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float(((uint32_t)h) << 16); }
// float -> bf16, round to nearest even: gfx950's v_cvt_pk_bf16_f32 (one instruction for two values)
__device__ __forceinline__ uint16_t f32_to_bf16(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ __forceinline__ uint32_t f32x2_to_bf16x2(float lo, float hi) {
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
  const bf16x2_t v = {(__bf16)lo, (__bf16)hi};
  return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ float ld_f(const void* p, size_t i, int dt) {
  return dt == BF16 ? bf16_to_f32(((const uint16_t*)p)[i]) : ((const float*)p)[i];
}
__device__ __forceinline__ void st_f(void* p, size_t i, float v, int dt) {
  if (dt == BF16) ((uint16_t*)p)[i] = f32_to_bf16(v);
  else ((float*)p)[i] = v;
}
// Reductions over the lanes of a wave (LANES = 64) or of each group of 32 / 16 lanes, every lane receiving the result: the
// butterfly lane ^ 32, ^ 16, ^ 8, ^ 4, ^ 2, ^ 1 without the LDS crossbar.  Once the lanes that differ in the higher bits hold
// the same value, a rotation inside a row of 16 by 8, 4, 2, 1 fetches from a lane that holds what lane ^ 8, 4, 2, 1 holds.
// (__shfl_xor goes through LDS: some 60 clocks per exchange against 8.)
template <int CTRL> __device__ __forceinline__ float dpp_f(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int LANES, class OP> __device__ __forceinline__ float lanes_reduce(float v, OP op) {
  if (LANES > 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = op(__uint_as_float(r[0]), __uint_as_float(r[1]));
  }
  if (LANES > 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = op(__uint_as_float(r[0]), __uint_as_float(r[1]));
  }
  v = op(v, dpp_f<0x128>(v));   // row_ror:8
  v = op(v, dpp_f<0x124>(v));
  v = op(v, dpp_f<0x122>(v));
  return op(v, dpp_f<0x121>(v));
}
template <int LANES> __device__ __forceinline__ float lanes_sum(float v) {
  return lanes_reduce<LANES>(v, [](float a, float b) { return a + b; });
}
__device__ __forceinline__ float wave_sum(float v) { return lanes_sum<64>(v); }
__device__ __forceinline__ float wave_max(float v) {
  return lanes_reduce<64>(v, [](float a, float b) { return fmaxf(a, b); });
}
// Orders LDS traffic between the lanes of one wave (writes before, reads after).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// Stores that go through L2 to memory at once (sc1).  An ordinary store leaves its line dirty in the XCD's L2, and what the last ones
// have left there, up to 4 MB in each of the 8, is written back when the kernel ends, with nothing else running (an evaluation forward
// of 3 + 1 layers of width 384: 359 us with ordinary stores in the products, 343 with these).  For results that other kernels read, where
// the stores of one instruction fill cache lines: pieces of lines, which L2 puts together otherwise, go out one by one (attention,
// 32 bytes of a row at a time: that forward 3 us longer; few-tile products likewise: 497 -> 504 us for a step of 585 rows of width
// 384; fp32 products, every other 16 bytes: 452 -> 481 us for a step of 148 rows of
// width 768; convolution results, 8 bytes: steps a tenth longer).  Nor for maps so small that the next kernel finds them in L2: see
// k_resnet_fused.hip.
constexpr int THROUGH = 16;     // as the cache policy of a buffer store
__device__ __forceinline__ void store_through(void* p, uint4 v) {
  typedef __attribute__((ext_vector_type(4))) unsigned int u32x4_t;
  __builtin_amdgcn_global_store_b128((__attribute__((address_space(1))) u32x4_t*)p, (u32x4_t){v.x, v.y, v.z, v.w}, "agent");
}
// End of the code object's instructions, defined by the linker.
extern "C" __attribute__((visibility("hidden"))) __device__ const char _etext[];
// Brings a kernel's own code into the L2 of its XCD at once.  A step goes through more code than the instruction cache holds and
// through so much data that the code has left L2 as well by the time a kernel comes round again; its waves then wait for one line
// after another from beyond L2.  So the first wave of the first workgroup on each XCD (workgroups go to the 8 XCDs in turn) asks for a
// word of every line of the first CHUNKS x 8 KB: CHUNKS instructions of 64 lines of 128 bytes.  The words go to 256 bytes of LDS that
// nothing else uses, so that no register waits for them, and the wave does not end before they are there.
// Eight product kernels in turn, on operands that do not stay in L2, take 2.2 us a launch more than each of them over and over; with
// this 0.7 (8320 x 384 x 384).  A step of 3 + 1 layers of width 384, 8320 rows: 938 -> 923 us.  For the product kernels of full tiles and
// the convolutions of 64 channels, of which 16 to 32 of up to 34 KB are brought, and for the kernel with copying waves (640 rows of
// width 768 672 -> 666 us a step).  Not for the few-tile kernel of rows: its launches of some 4 us and of few data find their code in L2,
// and the wave that waits for it ends last (evaluation of 155 rows of width 384 162.8 -> 164.9 us, a step of 210 rows of width 192
// 339.4 -> 341.9); nor for attention, where steps of every size are level.
typedef __attribute__((address_space(3))) char lds_byte;
template <int CHUNKS> class CodeToL2 {
  const bool on_;

 public:
  __device__ __forceinline__ explicit CodeToL2(lds_byte* to)
      : on_(CHUNKS > 0 && blockIdx.x < 8 && blockIdx.y == 0 && blockIdx.z == 0 && __builtin_amdgcn_readfirstlane(threadIdx.x) < 64) {
    if (!on_) return;
    uint64_t pc;
    asm volatile("s_getpc_b64 %0" : "=s"(pc));
    const uint64_t left = (uint64_t)(uintptr_t)_etext - pc, most = CHUNKS * 8192;
    const __amdgpu_buffer_rsrc_t code = __builtin_amdgcn_make_buffer_rsrc((void*)pc, 0, (int)(left < most ? left : most), 0x00020000);
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) __builtin_amdgcn_raw_ptr_buffer_load_lds(code, to, 4, (int)(threadIdx.x & 63) * 128 + c * 8192, 0, 0, 0);
  }
  __device__ __forceinline__ ~CodeToL2() {
    if (on_) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
};
#define PPLL_CODE_TO_L2(CHUNKS)                    \
  __shared__ __align__(16) char code_words__[256]; \
  const ::ppll::CodeToL2<CHUNKS> code_to_l2__((::ppll::lds_byte*)code_words__)
// Exact-form GELU through the rational erf approximation of Abramowitz & Stegun 7.1.26
// (|error| < 1.5e-7, far below bf16 resolution); erf(h/sqrt 2) and the normal density share
// one exponential: e^{-z^2} with z = h/sqrt 2 is e^{-h^2/2}.
__device__ __forceinline__ void cdf_pdf(float h, float& cdf, float& pdf) {
  const float z = fabsf(h) * 0.70710678118654752f;
  const float t = __builtin_amdgcn_rcpf(1.0f + 0.3275911f * z);
  const float ex = __expf(-z * z);
  const float poly = ((((1.061405429f * t - 1.453152027f) * t + 1.421413741f) * t - 0.284496736f) * t + 0.254829592f) * t;
  const float erf_abs = 1.0f - poly * ex;
  cdf = 0.5f * (1.0f + copysignf(erf_abs, h));
  pdf = 0.39894228040143268f * ex;
}
#endif

// ---------------------------------------------------------------- GEMM
// C[m,n] = sum_k A(m,k) B(k,n), fp32 accumulation, element strides for both
// operands so that one routine covers Y = X W, dX = dY W^T and dW = X^T dY.
enum Epilogue : int {
  EPI_NONE = 0,   // C = acc (+bias) (+residual)
  // GELU of h = acc + bias: C2 = gelu(h) and C = gelu'(h), the factor the backward pass multiplies by (h itself is
  // needed nowhere else, and the forward has the normal CDF and density at hand anyway)
  EPI_GELU = 1,
  EPI_DGELU = 2   // C = acc * aux   (aux = the gelu'(h) saved by EPI_GELU)
};
struct GemmArgs {
  const void* A; int a_dt; long a_sm, a_sk;   // A(m,k) = A[m*a_sm + k*a_sk]
  const void* B; int b_dt; long b_sk, b_sn;   // B(k,n) = B[k*b_sk + n*b_sn]
  void* C; int c_dt; long ldc;                // row-major output
  int M, N, K;
  const float* bias;                          // [N] fp32 or null
  const void* residual; int r_dt; long ldr;   // [M,N] or null
  int epilogue;
  void* C2;                                   // EPI_GELU second output (c_dt, ldc)
  const void* aux; int aux_dt; long ldaux;    // EPI_DGELU: the saved GELU derivative
  float* colsum;                              // optional: out[n] = sum_k B(k,n) (bias gradient of a dW product);
                                              // honoured only by the matrix-core kernels
  bool shared;                                // launches of other blocks want the device's units at the same time (a pipeline)
  int units;                                  // compute units of the device, 0: whoever needs them asks (product_units)
};
inline int product_units(const GemmArgs& g) { return g.units ? g.units : compute_units(); }
int launch_gemm(hipStream_t s, const GemmArgs& g);          // picks the MFMA kernel when the shape allows
int launch_gemm_generic(hipStream_t s, const GemmArgs& g);
// Products with few output rows (the class-token rows of a pruned auxiliary layer): see k_gemm_rows.hip
bool gemm_rows_supported(const GemmArgs& g);
int launch_gemm_rows(hipStream_t s, const GemmArgs& g);
// Products with many output tiles, bf16 output: see k_gemm_pipe.hip.  The choice (0: not this kernel, 3: 128 x 128 tiles with copying waves,
// else rows of a tile / 32) goes to the launch.
int gemm_pipe_choice(const GemmArgs& g);
bool gemm_pipe_supported(const GemmArgs& g);
int launch_gemm_pipe(hipStream_t s, const GemmArgs& g, int choice);
// Products whose 64 x 64 tiles find a compute unit each, bf16 output: see k_gemm_split.hip
bool gemm_split_choice(const GemmArgs& g);
bool gemm_split_supported(const GemmArgs& g);
int launch_gemm_split(hipStream_t s, const GemmArgs& g);
// fp32 products on the matrix cores: see k_f32.hip
bool gemm_f32_supported(const GemmArgs& g);
bool gemm_f32_groupable(const GemmArgs& g);
int launch_gemm_f32(hipStream_t s, const GemmArgs& g);
int launch_gemm_f32_grouped(hipStream_t s, const GemmArgs* gs, int n);
bool gemm_mfma_supported(const GemmArgs& g);
int launch_gemm_mfma(hipStream_t s, const GemmArgs& g);   // A stored [M][K]
bool gemm_mfma_groupable(const GemmArgs& g);
// every product must be groupable; ws (gemm_mfma_balanced_floats() floats or more), when given, lets the launch deal
// the k-steps out evenly over the compute units (parts of divided tiles pass through it)
int launch_gemm_mfma_grouped(hipStream_t s, const GemmArgs* gs, int n, float* ws = nullptr, size_t ws_floats = 0, bool any_order = false);
size_t gemm_mfma_balanced_floats();
// The same on tiles of 384 x 192: see k_gemm_wgrad.hip.  ws: gemm_big_grads_floats(parts of the divided tiles) floats.
struct BigGradPlan;
size_t gemm_big_grads_floats(int parts);
int launch_gemm_big_grads(hipStream_t s, const GemmArgs* gs, int n, float* ws, const BigGradPlan& plan);
// whether this set goes there, and the workspace that it then needs
bool gemm_big_grads_choice(const GemmArgs* gs, int n, size_t* ws_floats);
// A set of independent products of one element type, each a weight gradient that gemm_weight_grad_groupable() accepts, in
// one launch.  ws: room of gemm_mfma_balanced_floats() for the parts of divided tiles, for a launch that is the sole user of it
// while it runs (null: tiles stay whole).
inline bool gemm_weight_grad_groupable(const GemmArgs& g) { return gemm_mfma_groupable(g) || gemm_f32_groupable(g); }
// any_order: the sums over k may be divided elsewhere than by the 128 x 128 tiles (ws then has the room that gemm_big_grads_choice() says).
int launch_gemm_group(hipStream_t s, const GemmArgs* gs, int n, float* ws = nullptr, size_t ws_floats = 0, bool any_order = false);
// Per-launch timing of the contraction kernels (a measurement aid, off unless a block asks for it).  A block that
// times its launches binds its record to the calling thread for the duration of a step; the launch functions
// below the block engine then bracket each contraction launch with a pair of events on its stream.
// kind 0: GEMM over a token matrix (units = flops), 1: convolution (units = bytes), 2: GEMM with fewer than 256 output rows
// (the class-token products of the pruned auxiliary layer; units = flops)
struct TimedLaunch { hipEvent_t a, b; double units; int kind; };
struct LaunchTimes {
  std::vector<TimedLaunch> timed;
  std::vector<hipEvent_t> pool;
  double ms[3] = {0, 0, 0}, units[3] = {0, 0, 0};
  long long launches[3] = {0, 0, 0};
};
void profile_bind(LaunchTimes* t);     // null: launches of this thread are not timed
bool profile_enabled();                // a record is bound to this thread
int profile_begin(hipStream_t s, double units, void** token, int kind = 0);
int profile_end(hipStream_t s, void* token);
int profile_drain(LaunchTimes& t);     // waits for the recorded events and adds them to t.ms / t.units / t.launches
void profile_destroy(LaunchTimes& t);
int reduce_partials(hipStream_t s, const float* partial, int chunks, int N, long stride, float scale, float* out);

// Second stage of the two-stage (ordered, atomic-free) reductions.  A first-stage kernel asks for
// room for its partial sums: from the arena, if there is one with space left, and then the second
// stage is only queued and all queued ones run as one launch in flush() (parameter gradients are
// not needed before the optimizer update); otherwise from the shared scratch buffer, and the
// second stage runs at once.  The summation order is the same either way.
// outer != null: dst[n * outer_n + c] = sum over rows r of src[r][n] * outer[r][c] (outer [chunks][outer_n], outer_n <=
// OUTER_MAX), a weight gradient with few output columns
constexpr int OUTER_MAX = 16;
struct ReduceJob { const float* src; float* dst; int chunks, N; long stride; float scale; const float* outer; int outer_n; };
struct ReduceQueue {
  float* scratch = nullptr;            // shared by all reductions that finish at once
  float* arena = nullptr;              // private room for the queued ones, handed out front to back
  size_t arena_floats = 0, used = 0;
  std::vector<ReduceJob> jobs;
  float* space(size_t floats, bool* queued);
  int reduce(hipStream_t s, bool queued, const float* src, int chunks, int N, long stride, float scale, float* out);
  int reduce_outer(hipStream_t s, bool queued, const float* src, int rows, int N, const float* outer, int outer_n, float* out);
  int flush(hipStream_t s);
  void reset() { used = 0; jobs.clear(); }
};
int colsum_mode(hipStream_t s, const void* x, int dt, int rows, int N, int mode, const float* shift, float scale,
                ReduceQueue& rq, float* out);

// ---------------------------------------------------------------- row-wise ops
int launch_layernorm_fwd(hipStream_t s, const void* x, int dt, long x_row_stride, int rows, int D,
                         const float* g, const float* b, float eps, void* y, float* mean, float* rstd);
// dx_out = dres + LN'(dy) (either may be null); partial sums of dg/db ([nchunks][2][D]) are
// reduced into dg, db through the queue.  dres_every > 1: dres [rows / dres_every, D] belongs to rows 0, dres_every, ...
int launch_layernorm_bwd(hipStream_t s, const void* dy, const void* x, int dt, long x_row_stride, int rows,
                         int D, const float* g, const float* mean, const float* rstd, const void* dres, int dres_every,
                         void* dx_out, ReduceQueue& rq, float* dg, float* db);
// Partial sums of dg and db: what the kernel of this width leaves (a block holds as much for each of its LayerNorms), and the most
// there can be (the shared scratch): where parameters lie off 16 bytes the run-time-typed kernel stands in, which leaves up to six
// times as many rows (3152 instead of 526 at 25216 x 768); what then finds no room of its own is finished at once.
size_t layernorm_bwd_partial_floats(int rows, int D, int dt);
size_t layernorm_bwd_most_floats(int rows, int D, int dt);
int layernorm_bwd_rows(int rows, int D);       // rows that leave one partial row, on the bf16 path
// the second stage of those sums
int layernorm_bwd_reduce(hipStream_t s, ReduceQueue& rq, bool queued, const float* partials, int chunks, int D, float* dg, float* db);

// A Linear product and the LayerNorm behind it, in one launch where that is ahead (k_gemm_norm.hip), else in two.
// forward: C = product, y = LayerNorm(C); `stored` (may be empty) is called behind the launch that stores C
struct NormOut { const float *g, *b; float eps; void* y; float *mean, *rstd; };
int launch_gemm_then_norm(hipStream_t s, const GemmArgs& g, const NormOut& n, const std::function<int()>& stored);
// backward: the product is the gradient dy at the output of the LayerNorm of x, dx = dres + LN'(dy) (dres, dx may be null).  C is where
// dy goes if it goes anywhere: nothing else may read it.
struct NormGrad { const void* x; const float *mean, *rstd, *g; const void* dres; void* dx; float *dg, *db; };
int launch_gemm_then_norm_bwd(hipStream_t s, const GemmArgs& g, const NormGrad& n, ReduceQueue& rq);
bool gemm_norm_fwd_supported(const GemmArgs& g, const NormOut& n);
bool gemm_norm_bwd_supported(const GemmArgs& g, const NormGrad& n);
int launch_gemm_norm_fwd(hipStream_t s, const GemmArgs& g, const NormOut& n);
int launch_gemm_norm_bwd(hipStream_t s, const GemmArgs& g, const NormGrad& n, ReduceQueue& rq);

// out[n] = sum over rows of x[r, n]  (two-stage, deterministic)
int launch_colsum(hipStream_t s, const void* x, int dt, int rows, int N, ReduceQueue& rq, float* out);
int colsum_partial_floats(int rows, int N);

// mean softmax cross-entropy and its gradient; loss2 (optional) receives a copy of the loss, dbias (optional)
// the column sums of dlogits
int launch_cross_entropy(hipStream_t s, const float* logits, const int32_t* labels, int B, int C,
                         float* loss, float* loss2, float* dlogits, float* dbias, int* flag);

// ViT auxiliary head in one launch: z = LN(x[:, 0, :]), logits = z W + b, mean cross-entropy, and back to
// dcls = dL/dx[:, 0, :]; the batch sums (loss, dW, db, LayerNorm dg / db) go through the reduction queue.
size_t vit_head_partial_floats(int B, int D, int C);
bool vit_head_fused_ok(int D, int C);
int launch_vit_head(hipStream_t s, const void* x, int dt, long x_row_stride, int B, int D, int C, const float* ln_g,
                    const float* ln_b, float eps, const float* W, const float* bias, const int32_t* labels, void* dcls,
                    ReduceQueue& rq, float* d_ln_g, float* d_ln_b, float* dW, float* dbias, float* loss, float* loss2,
                    int* flag);

// ---------------------------------------------------------------- ViT pieces
int launch_patchify(hipStream_t s, const void* img, int dt, int B, int H, int W, int C, int P, void* patches);
int launch_assemble_tokens(hipStream_t s, const void* E, int dt, const float* cls, const float* pos, int B,
                           int T, int D, void* x0);
// dpos[t,d] = sum_b dx[b,t,d]; dcls[d] = dpos[0,d]; dE = dx[:,1:,:] gathered
int launch_embed_bwd(hipStream_t s, const void* dx, int dt, int B, int T, int D, ReduceQueue& rq, float* dpos,
                     float* dcls, void* dE);
int embed_bwd_partial_floats(int B, int T, int D);
// dx[b,0,:] = dcls[b,:], every other row 0
int launch_scatter_cls(hipStream_t s, const void* dcls, int dt, int B, int T, int D, void* dx);

int launch_attention_fwd(hipStream_t s, const void* qkv, int dt, int B, int T, int H, int dh, void* out,
                         float* lse);
int launch_attention_bwd(hipStream_t s, const void* qkv, const void* out, const void* dout, const float* lse,
                         int dt, int B, int T, int H, int dh, void* dqkv);
bool attention_mfma_supported(int dt, int T, int H, int dh, const void* a, const void* b, const void* c,
                              const void* d);
int launch_attention_fwd_mfma(hipStream_t s, const void* qkv, int B, int T, int H, void* out, float* lse);
int launch_attention_bwd_mfma(hipStream_t s, const void* qkv, const void* out, const void* dout, const float* lse,
                              int B, int T, int H, void* dqkv);
int launch_attention_rows_fwd(hipStream_t s, const void* qkv, int dt, int B, int T, int H, int dh, void* out, float* lse);
int launch_attention_rows_bwd(hipStream_t s, const void* qkv, const void* out, const void* dout, const float* lse, int dt,
                              int B, int T, int H, int dh, void* dqkv);
int launch_attention_fwd_generic(hipStream_t s, const void* qkv, int dt, int B, int T, int H, int dh, void* out,
                                 float* lse);
int launch_attention_bwd_generic(hipStream_t s, const void* qkv, const void* out, const void* dout,
                                 const float* lse, int dt, int B, int T, int H, int dh, void* dqkv);

// Attention of the class token's query alone against all keys and values of its (batch, head): q, out, dq, dout are
// [B, H*dh], kv and dkv [B*T, 2*H*dh] (keys then values), prob [B, H, T] fp32 (saved by the forward).
size_t attention_cls_lds_bytes(int T, int dh);
int launch_attention_cls_fwd(hipStream_t s, const void* q, const void* kv, int dt, int B, int T, int H, int dh, void* out,
                             float* prob);
int launch_attention_cls_bwd(hipStream_t s, const void* q, const void* kv, const float* prob, const void* dout, int dt, int B,
                             int T, int H, int dh, void* dq, void* dkv);

// ---------------------------------------------------------------- optimizers
// `shadow` (nullable): bf16 copy of the updated parameters, same offsets
int launch_sgd(hipStream_t s, float* p, const float* g, float* buf, uint16_t* shadow, size_t n, float lr,
               float momentum, int nesterov, float wd, int first);
int launch_adamw(hipStream_t s, float* p, const float* g, float* m, float* v, uint16_t* shadow, size_t n, float lr,
                 float b1, float b2, float eps, float wd, float bias_corr1, float bias_corr2);
int launch_refresh_shadow(hipStream_t s, const float* p, uint16_t* shadow, size_t n);
int launch_fill_zero(hipStream_t s, void* p, size_t bytes);
int launch_copy_probe(hipStream_t s, const void* src, void* dst, size_t bytes);

// ---------------------------------------------------------------- ResNet pieces
// stat / stat_blocks (nullable): room for the sums a BatchNorm over y needs (bn_partial_floats of y's shape); on
// return *stat_blocks is the number of partial rows the convolution wrote there itself (0: none, the BatchNorm
// has to make its own pass)
int launch_conv3x3_fwd(hipStream_t s, const void* x, const void* w, int wdt, int dt, int B, int H, int W, int Ci,
                       int Co, int stride, void* y, float* stat = nullptr, int* stat_blocks = nullptr);
// dx = dgrad(dy, w) (+ dres * (ymask > 0) when dres != null)
// The BatchNorm whose output gradient a convolution's input gradient dx is: output y (ReLU mask), input x, saved
// statistics, and room for the partial sums of its backward pass (bn_partial_floats of its shape).
// mask: what launch_conv_bn_bwd takes in place of y
struct BnBwdSums {
  const void* y; const void* x; const float* mean; const float* rstd; float* partials;
  const uint8_t* mask;
};
// bn / stat_blocks (nullable): on return *stat_blocks is the number of partial rows of that BatchNorm's two backward
// sums that the convolution wrote to bn->partials itself (0: none, launch_bn_bwd has to make its own pass)
int launch_conv3x3_dgrad(hipStream_t s, const void* dy, const void* w, int wdt, int dt, int B, int H, int W, int Ci,
                         int Co, int stride, const void* dres, const void* ymask, void* dx, const BnBwdSums* bn = nullptr,
                         int* stat_blocks = nullptr);
// Convolution (stride 1, C -> C) that applies the BatchNorm in front of it on the way in (k_resnet_fused.hip).
// The BatchNorm: input x, `blocks` partial rows of its sums, where statistics go, parameters, residual, output y.
struct BnInput {
  const void* x; float* partials; int blocks;
  float eps, momentum; float *mean, *rstd, *run_mean, *run_var;
  const float *g, *b; const void* res; void* y; uint8_t* mask;   // mask (nullable): receives the ReLU mask of y, a bit an element; y
                                                                 // may be null with 16 channels where nothing else reads it
};
// Backward: gradient dy at the BatchNorm's output, the output's ReLU mask, partial rows of its two sums, saved statistics,
// where dgamma and dbeta go.
struct BnGrad {
  const void *dy, *x; const uint8_t* mask; float* partials; int blocks;
  const float *mean, *rstd, *g, *b; float *dg, *db;
};
bool conv_bn_ok(int dt, int B, int H, int W, int C);
int conv_bn_stat_blocks(int B, int H, int W, int C);   // partial rows it leaves
// dst = conv(y) with y = relu(bn(bn->x) + bn->res), stored in bn->y; without bn, dst = conv(x).  stat: sums of dst.  units (here and
// below): compute units of the device, 0: asked for.
int launch_conv_bn_fwd(hipStream_t s, const BnInput* bn, const void* x, const void* w, int B, int H, int W, int C, void* dst,
                       float* stat, int* stat_blocks, int units = 0);
// d = gradient at the BatchNorm's input, dst = conv^T(d) (+ dres where dmask is set); next (nullable): the BatchNorm whose
// output gradient dst is, its sums go to stat
// fg (nullable, where conv_bn_filter_floats() says so): the convolution's weight gradient dw as well, in place of d, which is not stored.
// in: its input, or null: that is relu(bn) of next->x with these g and b.
struct ConvFilterGrad { float* dw; const void* in; const float *g, *b; };
size_t conv_bn_filter_floats(int B, int H, int W, int C, int units = 0);      // room for the partial sums, 0: not from this kernel
int launch_conv_bn_bwd(hipStream_t s, const BnGrad& bn, const void* w, int B, int H, int W, int C, void* d, const void* dres,
                       const uint8_t* dmask, void* dst, const BnBwdSums* next, float* stat, int* stat_blocks,
                       const ConvFilterGrad* fg = nullptr, ReduceQueue* rq = nullptr, int units = 0);
// the sums alone ([*blocks][2][C] partial rows, at most 256)
int launch_bn_sums_fwd_bf16(hipStream_t s, const void* x, int rows, int C, float* partials, int* blocks);
int launch_bn_sums_bwd_bf16(hipStream_t s, const void* dy, const void* y, const void* x, int rows, int C, const float* mean,
                            const float* rstd, float* partials, int* blocks);
// dw [9][ci_keep][Co]: the gradient for the first ci_keep input channels (all of them by default; fewer when
// the caller padded x with zero channels)
int launch_conv3x3_wgrad(hipStream_t s, const void* x, const void* dy, int dt, int B, int H, int W, int Ci,
                         int Co, int stride, ReduceQueue& rq, float* dw, int ci_keep = -1);
// weight gradients of n convolutions of one shape (x [B,H,W,Ci], dy [B,Ho,Wo,Co] each): one launch where the
// matrix-core kernel takes the shape, else one launch per convolution
struct ConvWgradJob { const void* x; const void* dy; float* dw; };
int launch_conv3x3_wgrad_group(hipStream_t s, const ConvWgradJob* jobs, int n, int dt, int B, int H, int W, int Ci, int Co,
                               int stride, ReduceQueue& rq);
int launch_conv3x3_wgrad_group_bf16(hipStream_t s, const ConvWgradJob* jobs, int n, int B, int H, int W, int Ci, int Co,
                                    int stride, ReduceQueue& rq, bool* done);
// second stage of a convolution weight gradient: adds `rows` partial filters [9][Ci][Co], `stride` floats apart, into
// dw [9][keep][Co]
int reduce_conv_filters(hipStream_t s, ReduceQueue& rq, bool queued, const float* partials, int rows, long stride,
                        int Ci, int Co, int keep, float* dw);
// x [P, c] -> y [P, 16] with zero channels appended (c < 16); w [9][c][Co] (fp32 master) -> wp [9][16][Co] bf16
int launch_pad_channels16(hipStream_t s, const void* x, size_t P, int c, void* y);
int launch_pad_filter16(hipStream_t s, const float* w, int c, int Co, void* wp);
int conv3x3_wgrad_partial_floats(int B, int H, int W, int Ci, int Co, int stride);
// shortcut of a downsampling basic block: y = every stride-th pixel of x [B,H,W,Ci] with Co - Ci zero channels
// appended; its transpose adds dy * (ymask > 0) into dx
int launch_shortcut_fwd(hipStream_t s, const void* x, int dt, int B, int H, int W, int Ci, int Co, int stride, void* y);
int launch_shortcut_bwd(hipStream_t s, const void* dy, const void* ymask, int dt, int B, int H, int W, int Ci, int Co,
                        int stride, void* dx);
// training-mode statistics over rows of x [rows, C]; also updates running stats
int launch_bn_stats(hipStream_t s, const void* x, int dt, int rows, int C, float eps, float momentum,
                    float* partials, float* mean, float* rstd, float* run_mean, float* run_var);
// statistics of x, running-statistics update and y = relu(bn(x) (+ res)): the BatchNorm of a training step
// ready_blocks: rows of `partials` the producing convolution has already filled (see launch_conv3x3_fwd), else 0
// mask (nullable, bf16 only): receives the ReLU mask of y, one bit an element
int launch_bn_train_fwd(hipStream_t s, const void* x, int dt, int rows, int C, float eps, float momentum, float* partials,
                        float* mean, float* rstd, float* run_mean, float* run_var, const float* g, const float* b,
                        const void* res, void* y, int ready_blocks = 0, uint8_t* mask = nullptr);
// y = relu(bn(x) (+ res)); units: compute units of the device, 0: asked for
int launch_bn_running_stats(hipStream_t s, const float* run_mean, const float* run_var, int C, float eps, float* mean,
                            float* rstd);
int launch_bn_apply(hipStream_t s, const void* x, int dt, int rows, int C, const float* mean, const float* rstd,
                    const float* g, const float* b, const void* res, void* y, int units = 0);
// dyh = dy * (y > 0); dx = bn'(dyh); dg = sum dyh*xhat; db = sum dyh
// ready_blocks: rows of `partials` the convolution that produced dy has already filled (see launch_conv3x3_dgrad), else 0
int launch_bn_bwd(hipStream_t s, const void* dy, const void* y, const void* x, int dt, int rows, int C,
                  const float* mean, const float* rstd, const float* g, float* partials, float* dg,
                  float* db, void* dx, int ready_blocks = 0);
int bn_partial_floats(int rows, int C);
// bf16 fast path (k_resnet_bf16.hip)
bool conv_bf16_supported(int dt, int wdt, int Ci, int Co, const void* a, const void* b, const void* c);
bool conv_pixels_fit(int B, int H, int W);
bool conv_fwd_bf16_ok(int Ci, int Co);
bool conv_dgrad_bf16_ok(int Ci, int Co);
bool conv_wgrad_bf16_ok(int H, int W, int Ci, int Co, int stride);
// stat (nullable): the kernel also writes per-workgroup per-channel sums of its stored outputs there
// ([*stat_blocks][2][Co] floats: what the BatchNorm behind the convolution reduces)
int launch_conv3x3_fwd_bf16(hipStream_t s, const void* x, const void* w, int B, int H, int W, int Ci, int Co,
                            int stride, void* y, float* stat = nullptr, int* stat_blocks = nullptr);
int launch_conv3x3_dgrad_bf16(hipStream_t s, const void* dy, const void* w, int B, int H, int W, int Ci, int Co,
                              int stride, const void* dres, const void* ymask, void* dx, const BnBwdSums* bn = nullptr,
                              int* stat_blocks = nullptr);
int launch_conv3x3_wgrad_bf16(hipStream_t s, const void* x, const void* dy, int B, int H, int W, int Ci, int Co,
                              int stride, ReduceQueue& rq, float* dw, int ci_keep);
size_t conv3x3_wgrad_bf16_partial_floats(int B, int H, int W, int Ci, int Co, int stride);
bool eltwise_bf16_ok(int dt, size_t elems, int C0, int C1, const void* a, const void* b, const void* c);
int launch_gap_bwd_bf16(hipStream_t s, const void* dpooled, int B, int HW, int C, void* dx);
bool gap_fwd_bf16_ok(int dt, int C, const void* x, const void* pooled);
int launch_gap_fwd_bf16(hipStream_t s, const void* x, int B, int HW, int C, void* pooled);
int launch_shortcut_fwd_bf16(hipStream_t s, const void* x, int B, int H, int W, int Ci, int Co, int stride, void* y);
int launch_shortcut_bwd_bf16(hipStream_t s, const void* dy, const void* ymask, int B, int H, int W, int Ci, int Co, int stride,
                             void* dx);
bool bn_bf16_supported(int dt, int rows, int C, const void* a, const void* b, const void* c, const void* d);
size_t bn_bf16_partial_floats(int rows, int C);
int launch_bn_stats_bf16(hipStream_t s, const void* x, int rows, int C, float eps, float momentum, float* partials,
                         float* mean, float* rstd, float* run_mean, float* run_var);
int launch_bn_train_fwd_bf16(hipStream_t s, const void* x, int rows, int C, float eps, float momentum, float* partials,
                             float* mean, float* rstd, float* run_mean, float* run_var, const float* g, const float* b,
                             const void* res, void* y, int ready_blocks = 0, uint8_t* mask = nullptr);
int launch_bn_apply_bf16(hipStream_t s, const void* x, int rows, int C, const float* mean, const float* rstd,
                         const float* g, const float* b, const void* res, void* y, uint8_t* mask = nullptr, int units = 0);
int launch_bn_bwd_bf16(hipStream_t s, const void* dy, const void* y, const void* x, int rows, int C, const float* mean,
                       const float* rstd, const float* g, float* partials, float* dg, float* db, void* dx, int ready_blocks = 0);
int launch_gap_fwd(hipStream_t s, const void* x, int dt, int B, int HW, int C, void* pooled);
int launch_gap_bwd(hipStream_t s, const void* dpooled, int dt, int B, int HW, int C, void* dx);

}  // namespace ppll
