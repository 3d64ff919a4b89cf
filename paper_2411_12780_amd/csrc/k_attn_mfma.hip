// Multi-head self-attention core for head dimension 64 in bf16 on the matrix
// cores, forward and backward, one workgroup per (batch, head) (of the backward
// also two), a wave per tile of 32 tokens or per two (T <= 256).
//
// Layout trick.  v_mfma_f32_32x32x16_bf16 gives lane l column l%32 of the
// 32 x 32 result and 16 of its rows (8*(e/4) + 4*(l/32) + e%4).  Scores are
// therefore produced transposed, S^T = K Q^T: a lane owns one query and holds
// its scores against 16 of the 32 keys of a tile, so the row softmax is a
// reduction over the lane's own registers plus one exchange with lane l^32.
// The same registers, packed to bf16, are directly the second operand of the
// next product (O^T = V^T P^T, dQ^T = K^T dS^T): the k index of an MFMA may be
// assigned to (lane half, element) in any order as long as both operands agree,
// so the first operand is fetched with the matching key order.  P and dS never
// pass through memory.
//
// Operands whose reduction index is the token (V^T, K^T, Q^T, dO^T) come out of the [token][64] tiles by transposing reads.  All sums run
// in a fixed order.  16 keys (queries) and more beyond the last token are left out of a last tile.
//
// Forward: K and V, 57 KB at 197 tokens, straight from memory to LDS.  What bounds it is memory and, above 160 tokens, the scores held
// in registers: 7 waves of 160 are all of a unit.  Microseconds with both copied through registers and V transposed there -> now:
// 128 images x 197 tokens x 12 heads 62 -> 45.5, 60 x 145 x 6 13.8 -> 8.9, 128 x 65 x 6 8.3 -> 6.4; with two tiles a wave, one after the
// other, and two workgroups a unit 62, 8.8 and 6.5.
//
// Backward: one part (wave = query tile) forms P and dS with a lane per query and accumulates dQ; another (wave = key tile) forms them
// again with a lane per key (scores recomputed in the other orientation instead of transposing registers) and accumulates dK and dV.
// The first needs K and V of the head in LDS, the second Q and dO.
// What bounds it is memory, each part waiting for its tiles and then storing them: 57 us of 143 at 128 x 197 tokens x 12 heads are
// loads, 40 stores.  So the tiles, half of what they were with transposed copies beside them, leave room for two or three workgroups a
// unit; up to 128 tokens one workgroup does both parts behind one barrier, all loads asked for at once, beyond that each part is a
// workgroup of its own (four tiles of 197 tokens would leave room for one).  Results leave 16 bytes a lane (8 bytes: 152 us; whole rows
// through LDS: 143).
// Microseconds with transposed copies, one workgroup a head at every size -> now: 128 images x 197 tokens x 12 heads 171 -> 143,
// 60 x 145 x 6 36.5 -> 29, 128 x 65 x 6 20.6 -> 16.8, 20 x 65 x 6 10.9 -> 7.9, 64 x 100 x 12 35.6 -> 28.
#include <type_traits>

#include "common.h"
#include "gemm_pipe.h"
#include "plan.h"

namespace ppll {

namespace {
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;

__device__ __forceinline__ bf16x8 ld_frag(const uint16_t* p, bool ok) {
  uint4 v = make_uint4(0, 0, 0, 0);
  if (ok) v = *reinterpret_cast<const uint4*>(p);
  return __builtin_bit_cast(bf16x8, v);
}
__device__ __forceinline__ uint32_t pack2(float a, float b) { return f32x2_to_bf16x2(a, b); }
__device__ __forceinline__ bf16x8 pack8(const float* v) {
  uint4 u = make_uint4(pack2(v[0], v[1]), pack2(v[2], v[3]), pack2(v[4], v[5]), pack2(v[6], v[7]));
  return __builtin_bit_cast(bf16x8, u);
}
constexpr float kScale = 0.125f;   // 1/sqrt(64)

// ---- Tiles in LDS: [token][64] bf16, 128-byte rows, the 16-byte granule g of row r at g ^ turn(r).  The fragment reads (16 rows x one
// granule at a time) and the transposing reads (4 rows x 64 bytes, rows r and r + 2 in different halves of the banks) both spread
// over all banks.
__device__ __forceinline__ int turn(int r) { return ((r & 2) << 1) | ((r >> 2) & 3); }
// Copies rows of 64 bf16 to a tile of TP rows, straight from memory to LDS, zeros beyond T.  off: byte offset of row 0 in the buffer
template <int TP, int W>
__device__ __forceinline__ void copy_rows(__amdgpu_buffer_rsrc_t rs, int off, int ld2, int T, pipe::lds_char* tile, int wave, int lane) {
#pragma unroll
  for (int i = 0; i < (TP / 8 + W - 1) / W; ++i) {
    const int q = i * W + wave, r = q * 8 + (lane >> 3);
    if (TP / 8 % W == 0 || q < TP / 8) pipe::load_to_lds(rs, tile + q * 1024, r < T ? off + r * ld2 + (((lane & 7) ^ turn(r)) << 4) : pipe::OOB);
  }
}
// lane part of the address of rows 0 .. 31 of a tile at k step kk (16 columns), and of their transpose: columns 32 dt .. + 31 as rows,
// tokens 0 .. 3 and 8 .. 11 (upper lanes: + 4) as k
__device__ __forceinline__ int row_addr(int lane, int kk) { return (lane & 31) * 128 + (((2 * kk + (lane >> 5)) ^ turn(lane & 31)) << 4); }
__device__ __forceinline__ int col_addr(int lane, int dt, int hi) {
  const int r = 8 * hi + 4 * (lane >> 5) + ((lane & 15) >> 2), g = 4 * dt + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
  return r * 128 + ((g ^ turn(r)) << 4) + 8 * (lane & 1);
}
typedef __attribute__((ext_vector_type(4))) short s16x4;
__device__ __forceinline__ bf16x8 tr_frag(const char* lo, const char* hi) {
  const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)lo);
  const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)hi);
  const uint2 u = __builtin_bit_cast(uint2, a), v = __builtin_bit_cast(uint2, b);
  return __builtin_bit_cast(bf16x8, make_uint4(u.x, u.y, v.x, v.y));
}
__device__ __forceinline__ float dot8(uint4 a, uint4 b) {
  const uint32_t x[4] = {a.x, a.y, a.z, a.w}, y[4] = {b.x, b.y, b.z, b.w};
  float d = 0.f;
#pragma unroll
  for (int w = 0; w < 4; ++w)
    d += __uint_as_float(x[w] << 16) * __uint_as_float(y[w] << 16) + __uint_as_float(x[w] & 0xffff0000u) * __uint_as_float(y[w] & 0xffff0000u);
  return d;
}

// A lane holds 4 consecutive columns of a row of results, its partner in the other half of the wave the next 4: they trade, and store
// 16 bytes each.
__device__ __forceinline__ void store_row(uint16_t* row, const f32x16 (&v)[2], float scale, int hh) {
#pragma unroll
  for (int dt = 0; dt < 2; ++dt)
#pragma unroll
    for (int q = 0; q < 4; q += 2) {
      const auto lo = __builtin_amdgcn_permlane32_swap(pack2(v[dt][4 * q] * scale, v[dt][4 * q + 1] * scale),
                                                       pack2(v[dt][4 * q + 4] * scale, v[dt][4 * q + 5] * scale), false, false);
      const auto hi = __builtin_amdgcn_permlane32_swap(pack2(v[dt][4 * q + 2] * scale, v[dt][4 * q + 3] * scale),
                                                       pack2(v[dt][4 * q + 6] * scale, v[dt][4 * q + 7] * scale), false, false);
      *reinterpret_cast<uint4*>(row + 32 * dt + 8 * (q + hh)) = make_uint4(lo[0], hi[0], lo[1], hi[1]);
    }
}

// Waves a SIMD: as many as the scores of a query, 16 registers a tile, let in beside the rest
constexpr int fwd_waves_per_simd(int nkt) { return nkt <= 3 ? 4 : nkt <= 5 ? 3 : 2; }

template <int NKT>
__global__ __launch_bounds__(64 * NKT, fwd_waves_per_simd(NKT)) void attn_fwd_mfma_kernel(const uint16_t* __restrict__ qkv, int T, int H,
                                                                            uint16_t* __restrict__ out, float* __restrict__ lse_out) {
  constexpr int TP = 32 * NKT, TILE = TP * 128;
  extern __shared__ __align__(1024) char smem[];      // K, V
  const int b = blockIdx.x / H, h = blockIdx.x % H, D = 64 * H;
  const long ld = 3L * D;
  const int lane = threadIdx.x & 63, li = lane & 31, hh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint16_t* base = qkv + (size_t)b * T * ld + h * 64;
  const __amdgpu_buffer_rsrc_t rs = pipe::make_rsrc(qkv + (size_t)b * T * ld, (uint32_t)(T * ld * 2));
  pipe::lds_char* lds = (pipe::lds_char*)smem;
  copy_rows<TP, NKT>(rs, (h * 64 + D) * 2, (int)ld * 2, T, lds, wave, lane);
  copy_rows<TP, NKT>(rs, (h * 64 + 2 * D) * 2, (int)ld * 2, T, lds + TILE, wave, lane);
  int ra[4], ca[2][2];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) ra[kk] = row_addr(lane, kk);
#pragma unroll
  for (int dt = 0; dt < 2; ++dt)
#pragma unroll
    for (int hi = 0; hi < 2; ++hi) ca[dt][hi] = col_addr(lane, dt, hi);
  const int qi = 32 * wave + li;
  bf16x8 qf[4];   // a wave's own queries: read once, straight from memory, in flight with the copies
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) qf[kk] = ld_frag(base + (long)qi * ld + 16 * kk + 8 * hh, qi < T);
  pipe::wait_vm<0>();
  __syncthreads();
  const bool padded = T < TP, last_half = T > TP - 16;   // of the last tile: 16 keys and more beyond the last token are left out
  f32x16 s[NKT];
#pragma unroll
  for (int jt = 0; jt < NKT; ++jt) {
#pragma unroll
    for (int e = 0; e < 16; ++e) s[jt][e] = 0.f;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
      s[jt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(smem + ra[kk] + 4096 * jt), qf[kk], s[jt], 0, 0, 0);
  }
  // softmax over the keys of query qi: s[jt][e] belongs to key 32 jt + 8 (e / 4) + 4 hh + e % 4
  if (padded) {
#pragma unroll
    for (int e = 0; e < 16; ++e)
      if (32 * (NKT - 1) + 8 * (e >> 2) + 4 * hh + (e & 3) >= T) s[NKT - 1][e] = -INFINITY;
  }
  float mx = -INFINITY;
#pragma unroll
  for (int jt = 0; jt < NKT; ++jt)
#pragma unroll
    for (int e = 0; e < 16; ++e) mx = fmaxf(mx, s[jt][e]);
  mx = fmaxf(mx, __shfl_xor(mx, 32, 64)) * kScale;
  float sum = 0.f;
#pragma unroll
  for (int jt = 0; jt < NKT; ++jt)
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      if (jt == NKT - 1 && half && !last_half) continue;
#pragma unroll
      for (int e = 8 * half; e < 8 * half + 8; ++e) {
        const float p = __expf(s[jt][e] * kScale - mx);
        s[jt][e] = p;
        sum += p;
      }
    }
  sum += __shfl_xor(sum, 32, 64);
  const float inv = 1.0f / sum;

  f32x16 o[2];
#pragma unroll
  for (int dt = 0; dt < 2; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) o[dt][e] = 0.f;
#pragma unroll
  for (int jt = 0; jt < NKT; ++jt)
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      if (jt == NKT - 1 && half && !last_half) continue;
      float pv[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) pv[e] = s[jt][8 * half + e] * inv;
      const bf16x8 pf = pack8(pv);
#pragma unroll
      for (int dt = 0; dt < 2; ++dt) {
        const int at = TILE + 4096 * jt + 2048 * half;
        o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tr_frag(smem + ca[dt][0] + at, smem + ca[dt][1] + at), pf, o[dt], 0, 0, 0);
      }
    }
  if (qi < T) {
    store_row(out + ((size_t)b * T + qi) * D + h * 64, o, 1.f, hh);
    if (hh == 0) lse_out[((size_t)b * H + h) * T + qi] = mx + __logf(sum);
  }
}

// Waves of a backward workgroup, each with one tile of 32 tokens, from five tiles on with two: 60 images x 145 tokens x 6 heads 29 us,
// 32 with five waves.  Three waves a SIMD leave 168 registers; with two tiles a wave those spilled (52 us).
constexpr int bwd_waves(int nkt) { return nkt <= 4 ? nkt : (nkt + 1) / 2; }
constexpr int bwd_waves_per_simd(int nkt) { return nkt <= 4 ? 3 : 2; }
// Both parts in one workgroup, us, one / two: 128 images x 65 tokens x 6 heads 16.7 / 21.1, 128 x 17 x 12 8.3 / 10.4, 20 x 100 x 12
// 11.1 / 12.7; few heads alone are a little ahead in two (20 x 65 x 6 7.9 / 7.3).  Beyond four tiles there is no room.
constexpr bool bwd_both(int nkt) { return nkt <= 4; }
constexpr int bwd_lds(int nkt) { return (bwd_both(nkt) ? 4 : 2) * nkt * 4096 + 2 * 32 * nkt * (int)sizeof(float); }

template <int NKT>
__global__ __launch_bounds__(64 * bwd_waves(NKT), bwd_waves_per_simd(NKT)) void attn_bwd_mfma_kernel(
    const uint16_t* __restrict__ qkv, const uint16_t* __restrict__ out, const uint16_t* __restrict__ dout, const float* __restrict__ lse,
    int T, int H, int heads, uint16_t* __restrict__ dqkv) {
  constexpr int TP = 32 * NKT, W = bwd_waves(NKT), TILE = TP * 128;
  constexpr bool BOTH = bwd_both(NKT);
  constexpr int QO = BOTH ? 2 * TILE : 0;      // tiles: K, V at 0, Q, dO at QO
  extern __shared__ __align__(1024) char smem[];
  // the two workgroups of a head are 8 apart: the same XCD, whose L2 holds what both read
  const int id = BOTH ? blockIdx.x : (blockIdx.x >> 4) * 8 + (blockIdx.x & 7);
  const bool do_queries = BOTH || !(blockIdx.x & 8), do_keys = BOTH || (blockIdx.x & 8);
  if (id >= heads) return;
  const int b = id / H, h = id % H, D = 64 * H;
  const long ld = 3L * D;
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, hh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint16_t* base = qkv + (size_t)b * T * ld + h * 64;
  const uint16_t* obase = out + (size_t)b * T * D + h * 64;
  const uint16_t* dobase = dout + (size_t)b * T * D + h * 64;
  uint16_t* gbase = dqkv + (size_t)b * T * ld + h * 64;
  const float* lbase = lse + (size_t)id * T;
  const __amdgpu_buffer_rsrc_t rs = pipe::make_rsrc(qkv + (size_t)b * T * ld, (uint32_t)(T * ld * 2));
  pipe::lds_char* lds = (pipe::lds_char*)smem;
  float* Dsh = reinterpret_cast<float*>(smem + QO + 2 * TILE);   // [TP] <dO_i, O_i>
  float* Lsh = Dsh + TP;                                         // [TP] log-sum-exp
  int ra[4], ca[2][2];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) ra[kk] = row_addr(lane, kk);
#pragma unroll
  for (int dt = 0; dt < 2; ++dt)
#pragma unroll
    for (int hi = 0; hi < 2; ++hi) ca[dt][hi] = col_addr(lane, dt, hi);
  auto rows = [&](int at, int tile) { return *reinterpret_cast<const bf16x8*>(smem + at + tile); };
  const int whole = T >> 5;   // tiles without padding

  if (do_queries) {
    copy_rows<TP, W>(rs, (h * 64 + D) * 2, (int)ld * 2, T, lds, wave, lane);
    copy_rows<TP, W>(rs, (h * 64 + 2 * D) * 2, (int)ld * 2, T, lds + TILE, wave, lane);
  }
  if (do_keys) {
    copy_rows<TP, W>(rs, h * 128, (int)ld * 2, T, lds + QO, wave, lane);
    // dO -> LDS; D_i = <dO_i, O_i> from the same pass: 8 lanes per token, then a 3-step exchange
#pragma unroll
    for (int i = 0; i < (TP / 8 + W - 1) / W; ++i) {
      const int q = i * W + wave, r = q * 8 + (lane >> 3), g = lane & 7;
      if (TP / 8 % W != 0 && q >= TP / 8) break;
      uint4 dov = make_uint4(0, 0, 0, 0), ov = dov;
      if (r < T) {
        dov = *reinterpret_cast<const uint4*>(dobase + (long)r * D + 8 * g);
        ov = *reinterpret_cast<const uint4*>(obase + (long)r * D + 8 * g);
      }
      *reinterpret_cast<uint4*>(smem + QO + TILE + r * 128 + ((g ^ turn(r)) << 4)) = dov;
      float dd = dot8(dov, ov);
      dd += __shfl_xor(dd, 1, 64);
      dd += __shfl_xor(dd, 2, 64);
      dd += __shfl_xor(dd, 4, 64);
      if (g == 0) {
        Dsh[r] = dd;
        Lsh[r] = r < T ? lbase[r] : 0.f;
      }
    }
  }
  if (BOTH) {
    pipe::wait_vm<0>();
    __syncthreads();
  }

  if (do_queries) {   // wave = query tile, lane = query: dQ
#pragma unroll 1
    for (int t = wave; t < NKT; t += W) {
      const int qi = 32 * t + li;
      const bool ok = qi < T;
      bf16x8 qf[4], dof[4];
      float d_i = 0.f, lse_i = 0.f;
      if (BOTH) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) { qf[kk] = rows(t * 4096 + ra[kk], QO); dof[kk] = rows(t * 4096 + ra[kk], QO + TILE); }
        d_i = Dsh[qi]; lse_i = Lsh[qi];
      } else {
        float d[4];
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          qf[kk] = ld_frag(base + (long)qi * ld + 16 * kk + 8 * hh, ok);
          dof[kk] = ld_frag(dobase + (long)qi * D + 16 * kk + 8 * hh, ok);
          d[kk] = dot8(__builtin_bit_cast(uint4, dof[kk]), __builtin_bit_cast(uint4, ld_frag(obase + (long)qi * D + 16 * kk + 8 * hh, ok)));
          d[kk] += __shfl_xor(d[kk], 32, 64);
        }
        d_i = (d[0] + d[1]) + (d[2] + d[3]);     // the order of the keys' workgroup
        if (ok) lse_i = lbase[qi];
        if (t == wave) {                // the first tile of every wave
          pipe::wait_vm<0>();
          __syncthreads();
        }
      }
      f32x16 dq[2];
#pragma unroll
      for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) dq[dt][e] = 0.f;
      auto keys = [&](int jt, auto padded) {
        f32x16 s, dp;
#pragma unroll
        for (int e = 0; e < 16; ++e) { s[e] = 0.f; dp[e] = 0.f; }
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          const int at = jt * 4096 + ra[kk];
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rows(at, 0), qf[kk], s, 0, 0, 0);
          dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rows(at, TILE), dof[kk], dp, 0, 0, 0);
        }
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          __builtin_amdgcn_sched_barrier(0);
          if (padded && 32 * jt + 16 * half >= T) continue;
          float ds[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const int i = 8 * half + e;
            float p = __expf(s[i] * kScale - lse_i);
            if (padded && 32 * jt + 8 * (i >> 2) + 4 * hh + (i & 3) >= T) p = 0.f;
            ds[e] = p * (dp[i] - d_i);
          }
          const bf16x8 dsf = pack8(ds);
#pragma unroll
          for (int dt = 0; dt < 2; ++dt) {
            const char *lo = smem + (jt * 4096 + ca[dt][0]), *hi = smem + (jt * 4096 + ca[dt][1]);
            dq[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tr_frag(lo + 2048 * half, hi + 2048 * half), dsf, dq[dt], 0, 0, 0);
          }
        }
      };
#pragma unroll 1
      for (int jt = 0; jt < whole; ++jt) keys(jt, std::false_type{});
      if (whole < NKT) keys(whole, std::true_type{});
      if (ok) store_row(gbase + (long)qi * ld, dq, kScale, hh);
    }
  }

  if (do_keys) {   // wave = key tile, lane = key: dK, dV
#pragma unroll 1
    for (int t = wave; t < NKT; t += W) {
      const int kj = 32 * t + li;
      bf16x8 kf[4], vf[4];
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        if (BOTH) { kf[kk] = rows(t * 4096 + ra[kk], 0); vf[kk] = rows(t * 4096 + ra[kk], TILE); continue; }
        kf[kk] = ld_frag(base + (long)kj * ld + D + 16 * kk + 8 * hh, kj < T);
        vf[kk] = ld_frag(base + (long)kj * ld + 2 * D + 16 * kk + 8 * hh, kj < T);
      }
      if (!BOTH && t == wave) {
        pipe::wait_vm<0>();
        __syncthreads();
      }
      f32x16 dk[2], dv[2];
#pragma unroll
      for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) { dk[dt][e] = 0.f; dv[dt][e] = 0.f; }
      auto queries = [&](int it, auto padded) {
        f32x16 s, dp;
#pragma unroll
        for (int e = 0; e < 16; ++e) { s[e] = 0.f; dp[e] = 0.f; }
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          const int at = it * 4096 + ra[kk];
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rows(at, QO), kf[kk], s, 0, 0, 0);     // rows = queries, lane = key
          dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rows(at, QO + TILE), vf[kk], dp, 0, 0, 0);
        }
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          __builtin_amdgcn_sched_barrier(0);
          if (padded && 32 * it + 16 * half >= T) continue;
          float p[8], ds[8];
#pragma unroll
          for (int q4 = 0; q4 < 2; ++q4) {
            const int q0 = 32 * it + 16 * half + 8 * q4 + 4 * hh;
            const float4 l4 = *reinterpret_cast<const float4*>(Lsh + q0);
            const float4 d4 = *reinterpret_cast<const float4*>(Dsh + q0);
            const float lv[4] = {l4.x, l4.y, l4.z, l4.w}, dvv[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int i = 8 * half + 4 * q4 + e;
              float pe = __expf(s[i] * kScale - lv[e]);
              if (padded && q0 + e >= T) pe = 0.f;
              p[4 * q4 + e] = pe;
              ds[4 * q4 + e] = pe * (dp[i] - dvv[e]);
            }
          }
          const bf16x8 pf = pack8(p), dsf = pack8(ds);
#pragma unroll
          for (int dt = 0; dt < 2; ++dt) {
            const char *lo = smem + (it * 4096 + ca[dt][0]), *hi = smem + (it * 4096 + ca[dt][1]);
            dv[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tr_frag(lo + QO + TILE + 2048 * half, hi + QO + TILE + 2048 * half), pf, dv[dt], 0, 0, 0);
            dk[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tr_frag(lo + QO + 2048 * half, hi + QO + 2048 * half), dsf, dk[dt], 0, 0, 0);
          }
        }
      };
#pragma unroll 1
      for (int it = 0; it < whole; ++it) queries(it, std::false_type{});
      if (whole < NKT) queries(whole, std::true_type{});
      if (kj < T) {
        store_row(gbase + (long)kj * ld + D, dk, kScale, hh);
        store_row(gbase + (long)kj * ld + 2 * D, dv, 1.f, hh);
      }
    }
  }
}

#define ATTN_DISPATCH(NKT_VALUE, CALL)                \
  switch (NKT_VALUE) {                                \
    case 1: { constexpr int NKT = 1; CALL; break; }   \
    case 2: { constexpr int NKT = 2; CALL; break; }   \
    case 3: { constexpr int NKT = 3; CALL; break; }   \
    case 4: { constexpr int NKT = 4; CALL; break; }   \
    case 5: { constexpr int NKT = 5; CALL; break; }   \
    case 6: { constexpr int NKT = 6; CALL; break; }   \
    case 7: { constexpr int NKT = 7; CALL; break; }   \
    default: { constexpr int NKT = 8; CALL; break; }  \
  }

template <int NKT>
int launch_fwd(hipStream_t s, const uint16_t* qkv, int B, int T, int H, uint16_t* out, float* lse) {
  constexpr int lds = 2 * 4096 * NKT;   // 64 KB at T = 256
  hipLaunchKernelGGL((attn_fwd_mfma_kernel<NKT>), dim3(B * H), dim3(64 * NKT), lds, s, qkv, T, H, out, lse);
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}

template <int NKT>
int launch_bwd(hipStream_t s, const uint16_t* qkv, const uint16_t* out, const uint16_t* dout, const float* lse, int B,
               int T, int H, uint16_t* dqkv) {
  constexpr int lds = bwd_lds(NKT);
  const int heads = B * H, grid = bwd_both(NKT) ? heads : 16 * ((heads + 7) / 8);
  static OncePerDevice once;
  if (lds > 64 * 1024) PPLL_TRY(raise_lds((const void*)attn_bwd_mfma_kernel<NKT>, lds, once));
  hipLaunchKernelGGL((attn_bwd_mfma_kernel<NKT>), dim3(grid), dim3(64 * bwd_waves(NKT)), lds, s, qkv, out, dout, lse, T, H, heads, dqkv);
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}
}  // namespace

bool attention_mfma_supported(int dt, int T, int H, int dh, const void* a, const void* b, const void* c, const void* d) {
  if (dt != BF16 || dh != 64 || T < 1 || T > 256 || H < 1 || !att_offsets_fit(T, H)) return false;
  return !((((uintptr_t)a) | ((uintptr_t)b) | ((uintptr_t)c) | ((uintptr_t)d)) & 15);
}

int launch_attention_fwd_mfma(hipStream_t s, const void* qkv, int B, int T, int H, void* out, float* lse) {
  int st = PPLL_OK;
  ATTN_DISPATCH((T + 31) / 32, st = launch_fwd<NKT>(s, (const uint16_t*)qkv, B, T, H, (uint16_t*)out, lse));
  return st;
}

int launch_attention_bwd_mfma(hipStream_t s, const void* qkv, const void* out, const void* dout, const float* lse,
                              int B, int T, int H, void* dqkv) {
  int st = PPLL_OK;
  ATTN_DISPATCH((T + 31) / 32, st = launch_bwd<NKT>(s, (const uint16_t*)qkv, (const uint16_t*)out,
                                                     (const uint16_t*)dout, lse, B, T, H, (uint16_t*)dqkv));
  return st;
}

}  // namespace ppll
