// Kernel selection: the MFMA kernels take the bf16 shapes they are built for,
// everything else goes to the run-time-typed kernels.  Also holds the optional
// per-launch timing of a block's contraction kernels used by the benchmark.
#include <vector>

#include "common.h"
#include "plan.h"

namespace ppll {

namespace {
thread_local LaunchTimes* t_times = nullptr;

hipEvent_t pooled_event(LaunchTimes& t) {
  if (!t.pool.empty()) { hipEvent_t e = t.pool.back(); t.pool.pop_back(); return e; }
  hipEvent_t e = nullptr;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  return e;
}
}  // namespace

void profile_bind(LaunchTimes* t) { t_times = t; }
bool profile_enabled() { return t_times != nullptr; }

// Adds the elapsed time of every bracketed launch since the last drain, per kind (0: GEMM, 1: convolution).
int profile_drain(LaunchTimes& t) {
  for (TimedLaunch& l : t.timed) {
    PPLL_HIP(hipEventSynchronize(l.b));
    float dt = 0.f;
    PPLL_HIP(hipEventElapsedTime(&dt, l.a, l.b));
    t.ms[l.kind] += dt; t.units[l.kind] += l.units; ++t.launches[l.kind];
    t.pool.push_back(l.a); t.pool.push_back(l.b);
  }
  t.timed.clear();
  return PPLL_OK;
}

void profile_destroy(LaunchTimes& t) {
  for (TimedLaunch& l : t.timed) { (void)hipEventDestroy(l.a); (void)hipEventDestroy(l.b); }
  for (hipEvent_t e : t.pool) (void)hipEventDestroy(e);
  t.timed.clear(); t.pool.clear();
}

// Brackets one kernel launch with a pair of events when the calling thread has a record bound.
int profile_begin(hipStream_t s, double units, void** token, int kind) {
  *token = nullptr;
  if (!t_times) return PPLL_OK;
  TimedLaunch tl{pooled_event(*t_times), pooled_event(*t_times), units, kind};
  if (!tl.a || !tl.b) { set_error("hipEventCreate failed"); return PPLL_ERR_HIP; }
  PPLL_HIP(hipEventRecord(tl.a, s));
  t_times->timed.push_back(tl);
  *token = (void*)(uintptr_t)t_times->timed.size();
  return PPLL_OK;
}
int profile_end(hipStream_t s, void* token) {
  if (!token || !t_times) return PPLL_OK;
  PPLL_HIP(hipEventRecord(t_times->timed[(size_t)(uintptr_t)token - 1].b, s));
  return PPLL_OK;
}

int raise_lds(const void* kernel, int bytes, OncePerDevice& once) {
  int dev = 0;
  PPLL_HIP(hipGetDevice(&dev));
  return once(dev, [&]() -> int {
    PPLL_HIP(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes));
    return PPLL_OK;
  });
}

int compute_units() {
  static PerDevice units;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  return units(dev, [&] {
    int n = 0;
    return hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess ? n : 0;
  });
}

int launch_gemm(hipStream_t s, const GemmArgs& g) {
  if (gemm_rows_supported(g)) return launch_gemm_rows(s, g);   // few output rows: latency, not throughput
  if (gemm_split_choice(g)) return launch_gemm_split(s, g);   // a tile a unit at most: the chain along k
  if (const int im = gemm_pipe_choice(g)) return launch_gemm_pipe(s, g, im);                // many tiles: throughput
  if (gemm_mfma_supported(g) && g.a_sk == 1) return launch_gemm_mfma(s, g);
  return gemm_f32_supported(g) && g.a_sk == 1 ? launch_gemm_f32(s, g) : launch_gemm_generic(s, g);
}

int launch_gemm_then_norm(hipStream_t s, const GemmArgs& g, const NormOut& n, const std::function<int()>& stored) {
  if (gemm_norm_fwd_supported(g, n) && norm_with_product(g.M, g.N, g.K, g.shared, product_units(g))) {
    PPLL_TRY(launch_gemm_norm_fwd(s, g, n));
    return stored ? stored() : PPLL_OK;
  }
  PPLL_TRY(launch_gemm(s, g));
  if (stored) PPLL_TRY(stored());
  return launch_layernorm_fwd(s, g.C, g.c_dt, g.ldc, g.M, g.N, n.g, n.b, n.eps, n.y, n.mean, n.rstd);
}
int launch_gemm_then_norm_bwd(hipStream_t s, const GemmArgs& g, const NormGrad& n, ReduceQueue& rq) {
  if (gemm_norm_bwd_supported(g, n) && norm_with_product(g.M, g.N, g.K, g.shared, product_units(g))) return launch_gemm_norm_bwd(s, g, n, rq);
  PPLL_TRY(launch_gemm(s, g));
  return launch_layernorm_bwd(s, g.C, n.x, g.c_dt, g.N, g.M, g.N, n.g, n.mean, n.rstd, n.dres, 1, n.dx, rq, n.dg, n.db);
}

int launch_gemm_group(hipStream_t s, const GemmArgs* gs, int n, float* ws, size_t ws_floats, bool any_order) {
  if (n <= 0) return PPLL_OK;
  return gs[0].a_dt == F32 ? launch_gemm_f32_grouped(s, gs, n) : launch_gemm_mfma_grouped(s, gs, n, ws, ws_floats, any_order);
}

int launch_attention_fwd(hipStream_t s, const void* qkv, int dt, int B, int T, int H, int dh, void* out, float* lse) {
  if (attention_mfma_supported(dt, T, H, dh, qkv, out, nullptr, nullptr)) return launch_attention_fwd_mfma(s, qkv, B, T, H, out, lse);
  if (att_by_rows(T, H, dh, false, (long)B * H, compute_units())) return launch_attention_rows_fwd(s, qkv, dt, B, T, H, dh, out, lse);
  return launch_attention_fwd_generic(s, qkv, dt, B, T, H, dh, out, lse);
}

int launch_attention_bwd(hipStream_t s, const void* qkv, const void* out, const void* dout, const float* lse, int dt,
                         int B, int T, int H, int dh, void* dqkv) {
  if (attention_mfma_supported(dt, T, H, dh, qkv, out, dout, dqkv))
    return launch_attention_bwd_mfma(s, qkv, out, dout, lse, B, T, H, dqkv);
  if (att_by_rows(T, H, dh, true, (long)B * H, compute_units())) return launch_attention_rows_bwd(s, qkv, out, dout, lse, dt, B, T, H, dh, dqkv);
  return launch_attention_bwd_generic(s, qkv, out, dout, lse, dt, B, T, H, dh, dqkv);
}

}  // namespace ppll

// One product on one kernel, for tests of a kernel against another (no part of the public interface): 1 few tiles, 2 tiled, 3 tiles of 128 x 128 with copying waves, 4 / 5 /
// 8 / 10 tiles of 128 / 160 / 256 / 320 rows of 256 columns, 6 tiles of 64 x 64.  C[M,N] = A[M][K] B, B [K][N] (bt) or [N][K], bf16 throughout.
extern "C" int ppll_internal_product(int kernel, int M, int N, int K, const void* A, long lda, const void* B, long ldb, int bt,
                                     void* C, long ldc, const float* bias, const void* residual, int epilogue, void* C2,
                                     const void* aux, void* stream) {
  using namespace ppll;
  GemmArgs g{};
  g.A = A; g.a_dt = BF16; g.a_sm = lda; g.a_sk = 1;
  g.B = B; g.b_dt = BF16; g.b_sk = bt ? ldb : 1; g.b_sn = bt ? 1 : ldb;
  g.C = C; g.c_dt = BF16; g.ldc = ldc; g.M = M; g.N = N; g.K = K;
  g.bias = bias; g.residual = residual; g.r_dt = BF16; g.ldr = ldc;
  g.epilogue = epilogue; g.C2 = C2; g.aux = aux; g.aux_dt = BF16; g.ldaux = ldc;
  hipStream_t s = (hipStream_t)stream;
  if (kernel == 1 && gemm_rows_supported(g)) return launch_gemm_rows(s, g);
  if (kernel == 2 && gemm_mfma_supported(g)) return launch_gemm_mfma(s, g);
  if ((kernel == 3 || kernel == 4 || kernel == 5 || kernel == 8 || kernel == 10) && gemm_pipe_supported(g)) return launch_gemm_pipe(s, g, kernel);
  if (kernel == 6 && gemm_split_supported(g)) return launch_gemm_split(s, g);
  set_error("kernel %d does not take this product", kernel);
  return PPLL_ERR_CONFIG;
}

// Attention on the matrix cores alone, bf16, head size 64, for tests (no part of the public interface): forward, then backward if dqkv
// is given.  Refuses what that kernel does not take.
extern "C" int ppll_internal_attention(int B, int T, int H, const void* qkv, void* out, float* lse, const void* dout, void* dqkv, void* stream) {
  using namespace ppll;
  if (!attention_mfma_supported(BF16, T, H, 64, qkv, out, dout, dqkv)) {
    set_error("the matrix-core attention does not take %d tokens", T);
    return PPLL_ERR_CONFIG;
  }
  PPLL_TRY(launch_attention_fwd_mfma((hipStream_t)stream, qkv, B, T, H, out, lse));
  return dqkv ? launch_attention_bwd_mfma((hipStream_t)stream, qkv, out, dout, lse, B, T, H, dqkv) : PPLL_OK;
}

// Attention of the class token's query, as the dispatch takes it, bf16, for tests (no part of the public interface)
extern "C" int ppll_internal_attention_cls(int B, int T, int H, int dh, const void* q, const void* kv, void* out, float* prob, const void* dout,
                                           void* dq, void* dkv, void* stream) {
  using namespace ppll;
  PPLL_TRY(launch_attention_cls_fwd((hipStream_t)stream, q, kv, BF16, B, T, H, dh, out, prob));
  return launch_attention_cls_bwd((hipStream_t)stream, q, kv, prob, dout, BF16, B, T, H, dh, dq, dkv);
}

// A set of weight-gradient products C[M,N] = A^T B on tiles of 384 x 192, divided as asked for, for tests of that kernel (no part of the
// public interface).  shape: M, N, K, row strides of A [K][M], B [K][N] and C of each product; column sums of B where asked for.  The
// tiles of reductions over more than 448 rows but the first `whole` run in `cuts` parts; ws_floats: room in ws.
extern "C" int ppll_internal_weight_grads(int n, const int* shape, const void* const* A, const void* const* B, float* const* C,
                                          float* const* colsum, float* ws, size_t ws_floats, int cuts, int whole, void* stream) {
  using namespace ppll;
  if (n < 1 || n > BIG_PRODUCTS || cuts < 1) { set_error("a set of %d products in %d parts", n, cuts); return PPLL_ERR_CONFIG; }
  std::vector<GemmArgs> gs(n);
  BigGradPlan plan{true, cuts, 0, 0, 0, 8};
  for (int j = 0; j < n; ++j) {
    const int* q = shape + 6 * j;
    GemmArgs g{};
    g.A = A[j]; g.a_dt = BF16; g.a_sm = 1; g.a_sk = q[3];
    g.B = B[j]; g.b_dt = BF16; g.b_sk = q[4]; g.b_sn = 1;
    g.C = C[j]; g.c_dt = F32; g.ldc = q[5]; g.M = q[0]; g.N = q[1]; g.K = q[2];
    g.colsum = colsum[j];
    if (!gemm_mfma_groupable(g)) { set_error("product %d is no weight gradient that the matrix-core kernels take", j); return PPLL_ERR_CONFIG; }
    gs[j] = g;
    const int tiles = (int)big_tiles({g.M, g.N, g.K});
    plan.tiles += tiles;
    if (wg_steps(g.K) >= plan.long_steps) plan.long_tiles += tiles;
  }
  plan.whole_tiles = cuts > 1 ? whole : plan.long_tiles;
  const int rest = plan.long_tiles - plan.whole_tiles;
  if (rest < 0 || (rest > 0 && (size_t)rest * cuts > ws_floats / gemm_big_grads_floats(1))) { set_error("the workspace is too small"); return PPLL_ERR_WORKSPACE; }
  return launch_gemm_big_grads((hipStream_t)stream, gs.data(), n, ws, plan);
}

// A Linear product C[M,N] = A[M][K] B (+ bias + residual) and the LayerNorm behind it, in one launch (fused) or in two (the
// tiled kernel first), for tests (no part of
// the public interface).  Forward (x null): y, mean, rstd of C.  Backward (x given): dx = dres + LN'(product) and [dg | db] in dgb, with
// room for the partial sums in scratch (layernorm_bwd_most_floats).
extern "C" int ppll_internal_product_norm(int fused, int M, int N, int K, const void* A, long lda, const void* B, long ldb, int bt, void* C,
                                          const float* bias, const void* residual, const float* gamma, const float* beta, float eps, void* y,
                                          float* mean, float* rstd, const void* x, const void* dres, void* dx, float* dgb, float* scratch, void* stream) {
  using namespace ppll;
  GemmArgs g{};
  g.A = A; g.a_dt = BF16; g.a_sm = lda; g.a_sk = 1;
  g.B = B; g.b_dt = BF16; g.b_sk = bt ? ldb : 1; g.b_sn = bt ? 1 : ldb;
  g.C = C; g.c_dt = BF16; g.ldc = N; g.M = M; g.N = N; g.K = K;
  g.bias = bias; g.residual = residual; g.r_dt = BF16; g.ldr = N;
  hipStream_t s = (hipStream_t)stream;
  if (x) {
    const NormGrad n{x, mean, rstd, gamma, dres, dx, dgb, dgb + N};
    ReduceQueue rq;
    rq.scratch = scratch;
    if (fused && gemm_norm_bwd_supported(g, n)) return launch_gemm_norm_bwd(s, g, n, rq);
    if (!fused) {
      PPLL_TRY(launch_gemm_mfma(s, g));
      return launch_layernorm_bwd(s, C, x, BF16, N, M, N, gamma, mean, rstd, dres, 1, dx, rq, dgb, dgb + N);
    }
  } else {
    const NormOut n{gamma, beta, eps, y, mean, rstd};
    if (fused && gemm_norm_fwd_supported(g, n)) return launch_gemm_norm_fwd(s, g, n);
    if (!fused) {
      PPLL_TRY(launch_gemm_mfma(s, g));
      return launch_layernorm_fwd(s, C, BF16, N, M, N, gamma, beta, eps, y, mean, rstd);
    }
  }
  set_error("no fused kernel takes this product");
  return PPLL_ERR_CONFIG;
}
