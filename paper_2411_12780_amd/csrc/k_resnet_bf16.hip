// bf16 fast path of the ResNet blocks (channel counts 16, 32, 48, 64):
//  * 3x3 convolution forward and input gradient as an implicit GEMM on the
//    matrix cores: a lane owns one output pixel, reads its 3x3 neighbourhood
//    straight from the NHWC tensor in MFMA fragment order (8 consecutive
//    channels = 16 bytes), the filter sits in LDS (forward: as in memory, read
//    with transposing LDS reads; input gradient: [in channel][tap, out channel]);
//    the product is issued filter-first so that a lane ends up with 4 consecutive
//    output channels of its pixel (8-byte stores).
//  * BatchNorm statistics / backward sums: 8 channels per thread (16-byte loads),
//    per-workgroup partials, added in workgroup order either by a one-workgroup launch
//    or, on small tensors, by every workgroup of the kernel that applies them (a
//    last-arrival scheme in one launch was slower: device-scope fences cost more).
//  * the elementwise pieces: shortcut of a downsampling block, global average pooling.
#include "resnet_bf16.h"
#include "plan.h"

namespace ppll {

namespace {
struct ConvArgs {
  const uint16_t* src;     // forward: x [B,H,W,Ci]; input gradient: dy [B,Ho,Wo,Co]
  const uint16_t* w;       // [9][Ci][Co]
  uint16_t* dst;           // forward: y [B,Ho,Wo,Co]; input gradient: dx [B,H,W,Ci]
  int B, H, W, Ci, Co, stride;
  const uint16_t* dres;    // input gradient only: dx += dres * (ymask > 0)
  const uint16_t* ymask;
  float* stat;             // STAT: [workgroups][2][channels produced] partial sums for the BatchNorm next in line:
                           //  forward: sum and sum of squares of the stored outputs;
                           //  input gradient: the two backward sums of the BatchNorm whose output gradient dx is
                           //  (sum dyh, sum dyh * xhat with dyh = dx * (bn_y > 0), xhat = (bn_x - bn_mean) * bn_rstd)
  const uint16_t* bn_y; const uint16_t* bn_x; const float* bn_mean; const float* bn_rstd;
};

// the forward convolution sums its outputs for the BatchNorm behind it up to this many workgroups; the input gradient
// the backward sums of the BatchNorm before it up to fewer (at 512, 1024 x 8 x 8 x 64, it measured 5 % of the step slower)
constexpr long CONV_STAT_MAX_BLOCKS = 512, CONV_BWD_STAT_MAX_BLOCKS = 256;
constexpr int CONV_STAT_LDS = 4 * 2 * 2 * 32 * 4;   // [wave][sum kind][lane half][32] floats behind the filter

// MODE 0: forward.  MODE 1: input gradient.  NO = channels produced, KC = 16 * K16 channels reduced.
// GRP: how many of a pixel's nine tap loads are issued before the first product waits for one
// (0: one, 1: the three of a filter row, 3: all nine; a filter row measured best).
// LIN (forward, and input gradient at stride 1): a tap's source is the centre pixel's plus a constant,
// so a tap costs one offset addition and one select between that offset and "out of range".
// STAT (forward): the workgroup also writes the per-channel sum and sum of squares of the values it stored (as
// stored: after rounding to bf16), which is what the BatchNorm behind the convolution needs of its input; the sums
// run per lane over the workgroup's tiles, then over the lanes of a half-wave, then over the four waves.
template <int MODE, int K16, int NT, int GRP, bool LIN, bool STAT>
__global__ __launch_bounds__(256) void conv3x3_mfma_kernel(ConvArgs p) {
  // The filter in LDS.  Input gradient: [produced channel ci][tap, co] with rows RSW bytes apart (co, the reduced
  // index, is the contiguous one in memory: a fragment is one 16-byte read).  Forward: as in memory, [tap, ci][co]
  // with rows of PB bytes (the produced channels rounded up to 32); a fragment, 8 consecutive (tap, ci) of one co,
  // comes out of two transposing LDS reads.
  extern __shared__ __align__(16) char wl[];
  constexpr int KC = 16 * K16;
  const int NO = MODE == 0 ? p.Co : p.Ci;
  constexpr int RSW = 18 * KC + 16;
  const int PB = (NO + 31) / 32 * 64;
  const int Ho = out_dim(p.H, p.stride), Wo = out_dim(p.W, p.stride);
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, li = lane & 31, hh = lane >> 5;
  // filter -> LDS; 8 output channels per 16-byte load, four loads in flight per thread
  {
    const int nvec = 9 * p.Ci * p.Co / 8;
    for (int v0 = tid; v0 < nvec; v0 += 4 * 256) {
      uint4 wv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int v = v0 + 256 * u;
        wv[u] = make_uint4(0, 0, 0, 0);
        if (v < nvec) wv[u] = *reinterpret_cast<const uint4*>(p.w + (size_t)v * 8);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int v = v0 + 256 * u;
        if (v >= nvec) break;
        const int e = v * 8, co = e % p.Co, ci = (e / p.Co) % p.Ci, tap = e / (p.Co * p.Ci);
        if (MODE == 0) {       // row (tap, ci), 8 consecutive co: a plain copy
          *reinterpret_cast<uint4*>(wl + (tap * KC + ci) * PB + 2 * co) = wv[u];
        } else {               // one row (ci), 8 consecutive k
          *reinterpret_cast<uint4*>(wl + ci * RSW + 2 * (tap * KC + co)) = wv[u];
        }
      }
    }
  }
  __syncthreads();
  // forward: lane part of a fragment address: (tap, ci) row 8 (lane/32) + (lane%16)/4, co 16 ((lane/16)%2) + 4 (lane%4)
  const int tr_lane = (8 * hh + ((lane & 15) >> 2)) * PB + (16 * ((lane >> 4) & 1) + 4 * (lane & 3)) * 2;
  const int OH = MODE == 0 ? Ho : p.H, OW = MODE == 0 ? Wo : p.W;      // output spatial size
  const int SH = MODE == 0 ? p.H : Ho, SW = MODE == 0 ? p.W : Wo;      // source spatial size
  const long P = (long)p.B * OH * OW, ntiles = (P + 127) / 128;
  // NT = tiles of 32 produced channels (NO = 16: the upper half of the one tile is never stored)
  const __amdgpu_buffer_rsrc_t rsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p.src), 0, (int)((long)p.B * SH * SW * KC * 2), 0x00020000);
  constexpr int NV = NT * 16;
  float st0[STAT ? NV : 1], st1[STAT ? NV : 1];
  if (STAT) {
#pragma unroll
    for (int j = 0; j < NV; ++j) { st0[j] = 0.f; st1[j] = 0.f; }
  }
  // the workgroup keeps its filter for several tiles of 128 pixels
  for (long tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    // 32-bit index arithmetic (the launcher checks that the pixel count fits): 64-bit division costs more than the tile
    const uint32_t pix = (uint32_t)tile * 128 + wave * 32 + li;
    const bool live = pix < (uint32_t)P;
    const uint32_t prow = pix / (uint32_t)OW;
    const int ox = (int)(pix - prow * (uint32_t)OW), oy = (int)(prow % (uint32_t)OH), b = (int)(prow / (uint32_t)OH);
    f32x16 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;
    constexpr int NG = GRP == 0 ? 9 : (GRP == 1 ? 3 : 1), TG = 9 / NG;   // groups of taps whose loads are in flight together
    // LIN: centre source pixel (cy, cx); tap (ky, kx) reads (cy + sg (ky-1), cx + sg (kx-1)), sg = +1 forward, -1 gradient
    const int sg = MODE == 0 ? 1 : -1;
    const int cy = MODE == 0 ? oy * p.stride : oy, cx = MODE == 0 ? ox * p.stride : ox;
    const int base = (((b * SH + cy) * SW + cx) * KC + 8 * hh) * 2;
    bool rowok[3], colok[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      rowok[d] = live && (unsigned)(cy + sg * (d - 1)) < (unsigned)SH;
      colok[d] = (unsigned)(cx + sg * (d - 1)) < (unsigned)SW;
    }
    auto tap_load = [&](const int grp, uint4 (&xv)[TG][K16]) {
#pragma unroll
      for (int j = 0; j < TG; ++j) {
        const int tap = grp * TG + j, ky = tap / 3, kx = tap % 3;
        if (LIN) {
          // ky is uniform (GRP = 1: ky = grp, kx = j): the row test is picked with scalar selects
          const bool ok = (ky == 0 ? rowok[0] : (ky == 1 ? rowok[1] : rowok[2])) && (kx == 0 ? colok[0] : (kx == 1 ? colok[1] : colok[2]));
          const int off = base + sg * (((ky - 1) * SW + (kx - 1)) * KC * 2);
#pragma unroll
          for (int c16 = 0; c16 < K16; ++c16) xv[j][c16] = conv_buf_load16(rsrc, ok ? off + 32 * c16 : CONV_OOB);
        } else {
          int sy, sx;
          bool ok = live;
          if (MODE == 0) {
            sy = oy * p.stride + ky - 1; sx = ox * p.stride + kx - 1;
          } else {
            // stride is 1 or 2 (checked by the launcher): mask and shift instead of a division per tap
            const int ty = oy + 1 - ky, tx = ox + 1 - kx, sm1 = p.stride - 1;
            ok = ok && ty >= 0 && tx >= 0 && !((ty | tx) & sm1);
            sy = ty >> sm1; sx = tx >> sm1;
          }
          ok = ok && sy >= 0 && sy < SH && sx >= 0 && sx < SW;
          const uint16_t* sp = p.src + (((long)b * SH + sy) * SW + sx) * KC + 8 * hh;
#pragma unroll
          for (int c16 = 0; c16 < K16; ++c16) {
            xv[j][c16] = make_uint4(0, 0, 0, 0);
            if (ok) xv[j][c16] = *reinterpret_cast<const uint4*>(sp + 16 * c16);
          }
        }
      }
    };
    auto tap_mma = [&](const int grp, const uint4 (&xv)[TG][K16]) {
#pragma unroll
      for (int j = 0; j < TG; ++j) {
        const int tap = grp * TG + j;
        const char* wrow = wl + 2 * (tap * KC + 8 * hh);
#pragma unroll
        for (int c16 = 0; c16 < K16; ++c16) {
          const bf16x8 xf = __builtin_bit_cast(bf16x8, xv[j][c16]);
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            bf16x8 wf;
            if (MODE == 0) {
              const char* fp = wl + tr_lane + (tap * KC + 16 * c16) * PB + 64 * t;
              const uint2 lo = conv_lds_read_tr(fp), hi = conv_lds_read_tr(fp + 4 * PB);
              wf = __builtin_bit_cast(bf16x8, make_uint4(lo.x, lo.y, hi.x, hi.y));
            } else {
              wf = *reinterpret_cast<const bf16x8*>(wrow + (t * 32 + li) * RSW + 32 * c16);
            }
            acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf, xf, acc[t], 0, 0, 0);
          }
        }
      }
    };
    // Up to 32 reduced channels: the loads of a tap group are in flight while the group before it is multiplied (two
    // register sets); with three groups of three taps (GRP = 1) that leaves one load latency per tile exposed instead
    // of three (7.1 -> 6.4 us for the 32 -> 32 forward at 128 x 16 x 16).  With 48 or 64 reduced channels the second
    // register set (96 registers at 64 channels) spills, and the rolled loop over the groups measured faster
    // (0.92 against 0.97 ms per step at the 8 x 8 stage of ResNet-32).
    if constexpr (NG == 3 && K16 <= 2) {
      uint4 xa[TG][K16], xb[TG][K16];
      tap_load(0, xa);
      tap_load(1, xb);
      tap_mma(0, xa);
      tap_load(2, xa);
      tap_mma(1, xb);
      tap_mma(2, xa);
    } else {
#pragma unroll 1
      for (int grp = 0; grp < NG; ++grp) {
        uint4 xv[TG][K16];
        tap_load(grp, xv);
        tap_mma(grp, xv);
      }
    }
    if (!live) continue;
    // acc[t][4q+e] = out[pix][32t + 8q + 4hh + e]
    uint16_t* drow = p.dst + (size_t)pix * NO;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int c = 32 * t + 8 * q + 4 * hh;
          if (c >= NO) continue;
          float v[4] = {acc[t][4 * q], acc[t][4 * q + 1], acc[t][4 * q + 2], acc[t][4 * q + 3]};
          if (MODE == 1 && p.dres) {
            const uint2 m = *reinterpret_cast<const uint2*>(p.ymask + (size_t)pix * NO + c);
            const uint2 r = *reinterpret_cast<const uint2*>(p.dres + (size_t)pix * NO + c);
            if (lo_bf(m.x) > 0.f) v[0] += lo_bf(r.x);
            if (hi_bf(m.x) > 0.f) v[1] += hi_bf(r.x);
            if (lo_bf(m.y) > 0.f) v[2] += lo_bf(r.y);
            if (hi_bf(m.y) > 0.f) v[3] += hi_bf(r.y);
          }
          const uint2 o = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
          *reinterpret_cast<uint2*>(drow + c) = o;
          if (STAT) {
            const float r[4] = {lo_bf(o.x), hi_bf(o.x), lo_bf(o.y), hi_bf(o.y)};
            if (MODE == 0) {
#pragma unroll
              for (int e = 0; e < 4; ++e) { st0[16 * t + 4 * q + e] += r[e]; st1[16 * t + 4 * q + e] += r[e] * r[e]; }
            } else {
              const uint2 by = *reinterpret_cast<const uint2*>(p.bn_y + (size_t)pix * NO + c);
              const uint2 bx = *reinterpret_cast<const uint2*>(p.bn_x + (size_t)pix * NO + c);
              const float4 mu = *reinterpret_cast<const float4*>(p.bn_mean + c), rs = *reinterpret_cast<const float4*>(p.bn_rstd + c);
              const float yv[4] = {lo_bf(by.x), hi_bf(by.x), lo_bf(by.y), hi_bf(by.y)};
              const float xv[4] = {lo_bf(bx.x), hi_bf(bx.x), lo_bf(bx.y), hi_bf(bx.y)};
              const float mv[4] = {mu.x, mu.y, mu.z, mu.w}, rv[4] = {rs.x, rs.y, rs.z, rs.w};
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const float d = yv[e] > 0.f ? r[e] : 0.f;
                st0[16 * t + 4 * q + e] += d;
                st1[16 * t + 4 * q + e] += d * (xv[e] - mv[e]) * rv[e];
              }
            }
          }
        }
      }
  }
  if constexpr (STAT) {
    // value index j = 16 t + 4 q + e of lane half hh is channel 32 t + 8 q + 4 hh + e
    float* red = reinterpret_cast<float*>(wl + (size_t)((NO + 31) / 32 * 32) * RSW);
    halfwave_sums<NV>(st0, li);
    halfwave_sums<NV>(st1, li);
    if (NV == 32 || !(li & 1)) {
      const int j = NV == 32 ? li : li >> 1;
      red[((wave * 2 + 0) * 2 + hh) * 32 + j] = st0[0];
      red[((wave * 2 + 1) * 2 + hh) * 32 + j] = st1[0];
    }
    __syncthreads();
    if (tid < 2 * NO) {
      const int which = tid / NO, c = tid % NO, j = 16 * (c >> 5) + 4 * ((c & 31) >> 3) + (c & 3), h2 = (c & 7) >> 2;
      float tot = 0.f;
#pragma unroll
      for (int w = 0; w < 4; ++w) tot += red[((w * 2 + which) * 2 + h2) * 32 + j];
      p.stat[(size_t)blockIdx.x * 2 * NO + tid] = tot;
    }
  }
}

// Input gradient at stride 2 (H and W even, no fused shortcut gradient).  An input pixel (y, x) receives from the taps ky with
// (y + 1 - ky) even only: one tap per axis for even y (ky = 1), two for odd y (ky = 0, 2).  A tile is 128 gradient pixels in a row: those
// pixels, the one behind them and as many a row of the image further on are laid in LDS, with 16-byte loads while the tile before is
// multiplied, and a wave forms both input rows of its 32 pixels, the taps of (y, 2 hx) and (y, 2 hx + 1) together.
// What bounds it is the maps' way through memory.  Pixels of one parity of both axes at a time, and their operands from memory 32 bytes of
// a line at a time, as this was before, wrote every line of the result in two or four visits that were far apart and read the
// gradient nine times.  Microseconds before and now: 1024 x 32 x 32 x 16 from 64 channels 45 -> 20.5 (67 MB: 11 us at a copy's rate; both
// rows together but operands from memory 35), 1024 x 32 x 32 x 16 from 32 21 -> 14.4, 848 x 16 x 16 x 64 from 64 12.5 -> 11.1, 128 x 16 x 16
// x 32 from 64 6.0 -> 5.7.
constexpr int DG_PX = 128;             // gradient pixels of a tile
template <int K16> constexpr int dgrad_s2_pitch() { return 32 * K16 + 16; }
template <int K16> constexpr int dgrad_s2_tile_bytes() { return 2 * (DG_PX + 1) * dgrad_s2_pitch<K16>(); }
template <int K16, int NT>
__global__ __launch_bounds__(256) void conv3x3_dgrad_s2_kernel(ConvArgs p, int parts) {
  constexpr int KC = 16 * K16, RSW = 18 * KC + 16, PX = dgrad_s2_pitch<K16>(), ROW = (DG_PX + 1) * 2 * K16, NP = (2 * ROW + 255) / 256;
  extern __shared__ __align__(16) char xt[];        // [this row, next row][DG_PX + 1] pixels, then the filter
  char* wl = xt + dgrad_s2_tile_bytes<K16>();       // [Ci rounded up to 32][9*Co] bf16, row stride RSW bytes
  const int NO = p.Ci;
  const int Ho = p.H / 2, Wo = p.W / 2;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, li = lane & 31, hh = lane >> 5;
  const uint32_t Pc = (uint32_t)p.B * Ho * Wo, tiles = (Pc + DG_PX - 1) / DG_PX;
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p.src), 0, (int)(Pc * KC * 2), 0x00020000);
  uint4 next[NP];
  auto load = [&](uint32_t tile) {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int v = tid + 256 * i, row = v >= ROW, u = v - row * ROW;
      const uint32_t q = tile * DG_PX + u / (2 * K16) + row * Wo;
      next[i] = conv_buf_load16(rsrc, v < 2 * ROW && q < Pc ? (int)(q * (KC * 2)) + 16 * (u % (2 * K16)) : CONV_OOB);
    }
  };
  // parts = 2: workgroups 2 t and 2 t + 1 form the even and the odd rows of tile t
  const uint32_t first = blockIdx.x / parts, step = gridDim.x / parts;
  load(first);
  {
    const int nvec = 9 * p.Ci * p.Co / 8;           // the filter row of an input channel: 8 consecutive output channels per copy
    for (int v = tid; v < nvec; v += 256) {
      const int e = v * 8, co = e % p.Co, ci = (e / p.Co) % p.Ci, tap = e / (p.Co * p.Ci);
      *reinterpret_cast<uint4*>(wl + ci * RSW + 2 * (tap * KC + co)) = *reinterpret_cast<const uint4*>(p.w + (size_t)v * 8);
    }
  }
  for (uint32_t tile = first; tile < tiles; tile += step) {
    __syncthreads();                                // the tile before has been read
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int v = tid + 256 * i;
      if (v < 2 * ROW) *reinterpret_cast<uint4*>(xt + v / (2 * K16) * PX + 16 * (v % (2 * K16))) = next[i];
    }
    __syncthreads();
    if (tile + step < tiles) load(tile + step);
    const uint32_t q = tile * DG_PX + wave * 32 + li;
    const bool live = q < Pc;
    const uint32_t qrow = q / (uint32_t)Wo;
    const int hx = (int)(q - qrow * (uint32_t)Wo), hy = (int)(qrow % (uint32_t)Ho), b = (int)(qrow / (uint32_t)Ho);
#pragma unroll
    for (int cy = 0; cy < 2; ++cy) {
      if (parts == 2 && cy != (int)(blockIdx.x & 1)) continue;
      f32x16 acc[2][NT];
#pragma unroll
      for (int cx = 0; cx < 2; ++cx)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int e = 0; e < 16; ++e) acc[cx][t][e] = 0.f;
      // axis parity 0: tap 1 reads the pixel itself; parity 1: tap 0 reads the next one, tap 2 the pixel itself
#pragma unroll
      for (int dy = cy; dy >= 0; --dy)
#pragma unroll
        for (int dx = 1; dx >= 0; --dx) {
          const bool in = live && hy + dy < Ho && hx + dx < Wo;
          const char* px = xt + (dy * (DG_PX + 1) + wave * 32 + li + dx) * PX + 16 * hh;
          bf16x8 xf[K16];
#pragma unroll
          for (int c16 = 0; c16 < K16; ++c16) {
            const uint4 v = *reinterpret_cast<const uint4*>(px + 32 * c16);
            xf[c16] = __builtin_bit_cast(bf16x8, in ? v : make_uint4(0, 0, 0, 0));
          }
#pragma unroll
          for (int cx = dx; cx < 2; ++cx) {
            const char* wrow = wl + 2 * (((cy ? 2 - 2 * dy : 1) * 3 + (cx ? 2 - 2 * dx : 1)) * KC + 8 * hh);
#pragma unroll
            for (int c16 = 0; c16 < K16; ++c16)
#pragma unroll
              for (int t = 0; t < NT; ++t)
                acc[cx][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(wrow + (t * 32 + li) * RSW + 32 * c16), xf[c16],
                                                                     acc[cx][t], 0, 0, 0);
          }
        }
      // a lane has channels 8 qq + 4 hh .. of qq = 0 .. 3; exchanged with the other half of the wave, 8 of one qq
      uint16_t* drow = p.dst + ((size_t)(b * p.H + 2 * hy + cy) * p.W + 2 * hx) * NO;
#pragma unroll
      for (int cx = 0; cx < 2; ++cx)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int qq = 0; qq < 4; qq += 2) {
            const f32x16& v = acc[cx][t];
            const auto lo = __builtin_amdgcn_permlane32_swap(pack2(v[4 * qq], v[4 * qq + 1]), pack2(v[4 * qq + 4], v[4 * qq + 5]), false, false);
            const auto hi = __builtin_amdgcn_permlane32_swap(pack2(v[4 * qq + 2], v[4 * qq + 3]), pack2(v[4 * qq + 6], v[4 * qq + 7]), false, false);
            if (live && 32 * t + 8 * qq < NO)       // NO is a multiple of 16
              *reinterpret_cast<uint4*>(drow + cx * NO + 32 * t + 8 * (qq + hh)) = make_uint4(lo[0], hi[0], lo[1], hi[1]);
          }
    }
  }
}

// ---------------------------------------------------------------- BatchNorm
template <int KIND>
__global__ __launch_bounds__(256) void bn_sums_kernel(BnSumArgs p) {
  __shared__ float red[256][17];
  const int groups = p.C / 8;                   // channel groups of 8
  const int lanes = 256 / groups;               // row lanes per workgroup
  const int tid = threadIdx.x, cg = tid % groups, rl = tid / groups;
  float a0[8], a1[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) { a0[j] = 0.f; a1[j] = 0.f; }
  float mu[8], rs[8];
  if (KIND == 1) {
#pragma unroll
    for (int j = 0; j < 8; ++j) { mu[j] = p.mean[8 * cg + j]; rs[j] = p.rstd[8 * cg + j]; }
  }
  if (rl < lanes) {
    // four rows per trip, their loads issued together; the sums of a lane still run in row order
    const int stride = gridDim.x * lanes;
    for (int r = blockIdx.x * lanes + rl; r < p.rows; r += 4 * stride) {
      uint4 xv[4], dv[4], yv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int ru = r + u * stride;
        xv[u] = dv[u] = yv[u] = make_uint4(0, 0, 0, 0);
        if (ru < p.rows) {
          const size_t off = (size_t)ru * p.C + 8 * cg;
          xv[u] = *reinterpret_cast<const uint4*>(p.x + off);
          if (KIND == 1) {
            dv[u] = *reinterpret_cast<const uint4*>(p.dy + off);
            yv[u] = *reinterpret_cast<const uint4*>(p.y + off);
          }
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (r + u * stride >= p.rows) break;
        const uint32_t* xw = reinterpret_cast<const uint32_t*>(&xv[u]);
        if (KIND == 0) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float a = lo_bf(xw[j]), b = hi_bf(xw[j]);
            a0[2 * j] += a; a0[2 * j + 1] += b; a1[2 * j] += a * a; a1[2 * j + 1] += b * b;
          }
        } else {
          const uint32_t* dw = reinterpret_cast<const uint32_t*>(&dv[u]);
          const uint32_t* yw = reinterpret_cast<const uint32_t*>(&yv[u]);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float d0 = lo_bf(yw[j]) > 0.f ? lo_bf(dw[j]) : 0.f, d1 = hi_bf(yw[j]) > 0.f ? hi_bf(dw[j]) : 0.f;
            a0[2 * j] += d0; a0[2 * j + 1] += d1;
            a1[2 * j] += d0 * (lo_bf(xw[j]) - mu[2 * j]) * rs[2 * j];
            a1[2 * j + 1] += d1 * (hi_bf(xw[j]) - mu[2 * j + 1]) * rs[2 * j + 1];
          }
        }
      }
    }
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) { red[tid][j] = a0[j]; red[tid][8 + j] = a1[j]; }
  __syncthreads();
  // thread c < 2C adds the row lanes of its (sum kind, channel) in order
  if (tid < 2 * p.C) {
    const int which = tid / p.C, c = tid % p.C, g = c / 8, j = c % 8;
    float t = 0.f;
#pragma unroll 8
    for (int l = 0; l < lanes; ++l) t += red[l * groups + g][8 * which + j];
    p.partial[(size_t)blockIdx.x * 2 * p.C + tid] = t;
  }
}

template <int KIND>
__global__ __launch_bounds__(1024) void bn_finish_kernel(BnSumArgs p, unsigned nblocks) {
  __shared__ __align__(16) float red[4096];
  bn_finish<KIND, 1024>(p, nblocks, red, nullptr, nullptr, true);
}

// Pieces of 8 channels a thread, 256 apart, so of the same channels (256 % (C / 8) = 0).  One piece a thread spends eight loads of parameters and
// in the backward pass eight divisions on each of it: with AP_PIECES of them, 1024 x 32 x 32 x 16 forward 17.3 -> 15.7 us, backward 21.0 ->
// 20.4; beside other blocks of a pipeline 19.6 -> 17.0 and 25.1 -> 23.4.  Small maps, which only an evaluation has here, take one
// (bn_apply_pieces): five basic blocks on 24 x 8 x 8 x 64 evaluated 170.0 us, with four 172.0.
// y = relu(bn(x) (+ res))
template <int PIECES>
__global__ __launch_bounds__(256) void bn_apply_bf16_kernel(const uint16_t* x, size_t chunks, int C, const float* mean,
                                                            const float* rstd, const float* g, const float* b,
                                                            const uint16_t* res, uint16_t* y, uint8_t* mask) {
  const size_t i0 = (size_t)blockIdx.x * (256 * PIECES) + threadIdx.x;
  uint4 xv[PIECES], rv[PIECES];
#pragma unroll
  for (int u = 0; u < PIECES; ++u) {
    const size_t i = i0 + 256 * u;
    xv[u] = rv[u] = make_uint4(0, 0, 0, 0);
    if (i < chunks) {
      xv[u] = *reinterpret_cast<const uint4*>(x + i * 8);
      if (res) rv[u] = *reinterpret_cast<const uint4*>(res + i * 8);
    }
  }
  const int c0 = 8 * (threadIdx.x % (C / 8));
  float mu[8], k[8], sh[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) { mu[c] = mean[c0 + c]; k[c] = rstd[c0 + c] * g[c0 + c]; sh[c] = b[c0 + c]; }
#pragma unroll
  for (int u = 0; u < PIECES; ++u) {
    const size_t i = i0 + 256 * u;
    if (i >= chunks) return;
    const uint32_t* xw = reinterpret_cast<const uint32_t*>(&xv[u]);
    const uint32_t* rw = reinterpret_cast<const uint32_t*>(&rv[u]);
    uint32_t o[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int c = 2 * j;
      const float p = bn_value(lo_bf(xw[j]), mu[c], k[c], sh[c]) + lo_bf(rw[j]);
      const float q = bn_value(hi_bf(xw[j]), mu[c + 1], k[c + 1], sh[c + 1]) + hi_bf(rw[j]);
      o[j] = pack2(fmaxf(p, 0.f), fmaxf(q, 0.f));
    }
    const uint4 ov = make_uint4(o[0], o[1], o[2], o[3]);
    store_through(y + i * 8, ov);
    if (mask) mask[i] = relu_mask(ov);
  }
}

// dx = (g rstd / N) (N dyh - dbeta - xhat dgamma)
__global__ __launch_bounds__(256) void bn_bwd_apply_bf16_kernel(const uint16_t* dy, const uint16_t* y,
                                                                const uint16_t* x, size_t chunks, int C, int rows,
                                                                const float* mean, const float* rstd, const float* g,
                                                                const float* dg, const float* db, uint16_t* dx) {
  const size_t i0 = (size_t)blockIdx.x * (256 * AP_PIECES) + threadIdx.x;
  uint4 xv[AP_PIECES], dv[AP_PIECES], yv[AP_PIECES];
#pragma unroll
  for (int u = 0; u < AP_PIECES; ++u) {
    const size_t i = i0 + 256 * u;
    xv[u] = dv[u] = yv[u] = make_uint4(0, 0, 0, 0);
    if (i < chunks) {
      xv[u] = *reinterpret_cast<const uint4*>(x + i * 8);
      dv[u] = *reinterpret_cast<const uint4*>(dy + i * 8);
      yv[u] = *reinterpret_cast<const uint4*>(y + i * 8);
    }
  }
  const int c0 = 8 * (threadIdx.x % (C / 8));
  const float n = (float)rows;
  float mu[8], rs[8], k[8], sb[8], sg[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    mu[c] = mean[c0 + c]; rs[c] = rstd[c0 + c]; sb[c] = db[c0 + c]; sg[c] = dg[c0 + c];
    k[c] = g[c0 + c] * rs[c] / n;
  }
#pragma unroll
  for (int u = 0; u < AP_PIECES; ++u) {
    const size_t i = i0 + 256 * u;
    if (i >= chunks) return;
    const uint32_t* xw = reinterpret_cast<const uint32_t*>(&xv[u]);
    const uint32_t* dw = reinterpret_cast<const uint32_t*>(&dv[u]);
    const uint32_t* yw = reinterpret_cast<const uint32_t*>(&yv[u]);
    uint32_t o[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float r[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int c = 2 * j + h;
        const float yy = h ? hi_bf(yw[j]) : lo_bf(yw[j]), dd = h ? hi_bf(dw[j]) : lo_bf(dw[j]);
        const float xx = h ? hi_bf(xw[j]) : lo_bf(xw[j]);
        const float d = yy > 0.f ? dd : 0.f, xh = (xx - mu[c]) * rs[c];
        r[h] = k[c] * (n * d - sb[c] - xh * sg[c]);
      }
      o[j] = pack2(r[0], r[1]);
    }
    store_through(dx + i * 8, make_uint4(o[0], o[1], o[2], o[3]));
  }
}

// Small tensors: the apply kernels add up the partial sums themselves (every workgroup, in the same order;
// workgroup 0 writes the results to memory), which saves the finishing launch.
__global__ __launch_bounds__(256) void bn_apply_fused_kernel(BnSumArgs p, unsigned nblocks, size_t chunks, const float* g,
                                                             const float* b, const uint16_t* res, uint16_t* y, uint8_t* mask) {
  __shared__ __align__(16) float red[1024];
  __shared__ float s_mean[128], s_rstd[128];
  bn_finish<0, 256>(p, nblocks, red, s_mean, s_rstd, blockIdx.x == 0);
  __syncthreads();
  const uint32_t i32 = blockIdx.x * 256 + threadIdx.x;
  if (i32 >= chunks) return;
  const size_t i = i32;
  const int c0 = (int)(8 * (i32 % (uint32_t)(p.C / 8)));
  const uint4 xv = *reinterpret_cast<const uint4*>(p.x + i * 8);
  const uint32_t* xw = reinterpret_cast<const uint32_t*>(&xv);
  uint4 rv = make_uint4(0, 0, 0, 0);
  if (res) rv = *reinterpret_cast<const uint4*>(res + i * 8);
  const uint32_t* rw = reinterpret_cast<const uint32_t*>(&rv);
  uint32_t o[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int c = c0 + 2 * j;
    const float u = bn_value(lo_bf(xw[j]), s_mean[c], s_rstd[c] * g[c], b[c]) + lo_bf(rw[j]);
    const float v = bn_value(hi_bf(xw[j]), s_mean[c + 1], s_rstd[c + 1] * g[c + 1], b[c + 1]) + hi_bf(rw[j]);
    o[j] = pack2(fmaxf(u, 0.f), fmaxf(v, 0.f));
  }
  const uint4 ov = make_uint4(o[0], o[1], o[2], o[3]);
  store_through(y + i * 8, ov);
  if (mask) mask[i] = relu_mask(ov);
}
__global__ __launch_bounds__(256) void bn_bwd_apply_fused_kernel(BnSumArgs p, unsigned nblocks, size_t chunks, const float* g,
                                                                 uint16_t* dx) {
  __shared__ __align__(16) float red[1024];
  __shared__ float s_db[128], s_dg[128];
  bn_finish<1, 256>(p, nblocks, red, s_db, s_dg, blockIdx.x == 0);
  __syncthreads();
  const uint32_t i32 = blockIdx.x * 256 + threadIdx.x;
  if (i32 >= chunks) return;
  const size_t i = i32;
  const int c0 = (int)(8 * (i32 % (uint32_t)(p.C / 8)));
  const uint4 xv = *reinterpret_cast<const uint4*>(p.x + i * 8);
  const uint4 dv = *reinterpret_cast<const uint4*>(p.dy + i * 8);
  const uint4 yv = *reinterpret_cast<const uint4*>(p.y + i * 8);
  const uint32_t* xw = reinterpret_cast<const uint32_t*>(&xv);
  const uint32_t* dw = reinterpret_cast<const uint32_t*>(&dv);
  const uint32_t* yw = reinterpret_cast<const uint32_t*>(&yv);
  const float n = (float)p.rows;
  uint32_t o[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float r[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int c = c0 + 2 * j + h;
      const float yy = h ? hi_bf(yw[j]) : lo_bf(yw[j]), dd = h ? hi_bf(dw[j]) : lo_bf(dw[j]);
      const float xx = h ? hi_bf(xw[j]) : lo_bf(xw[j]);
      const float d = yy > 0.f ? dd : 0.f, xh = (xx - p.mean[c]) * p.rstd[c];
      r[h] = g[c] * p.rstd[c] / n * (n * d - s_db[c] - xh * s_dg[c]);
    }
    o[j] = pack2(r[0], r[1]);
  }
  store_through(dx + i * 8, make_uint4(o[0], o[1], o[2], o[3]));
}

// Elementwise helpers of the stage, 8 channels (16 bytes) per thread, 32-bit index arithmetic.
// dx[b, p, c] = dpooled[b, c] / HW
__global__ __launch_bounds__(256) void gap_bwd_bf16_kernel(const uint16_t* dpooled, uint32_t HW, uint32_t C, uint32_t chunks,
                                                           uint16_t* dx) {
  const uint32_t i = blockIdx.x * 256 + threadIdx.x;
  if (i >= chunks) return;
  const uint32_t cpr = C / 8, cg = i % cpr, b = (i / cpr) / HW;
  const uint4 v = *reinterpret_cast<const uint4*>(dpooled + (size_t)b * C + 8 * cg);
  const uint32_t* w = reinterpret_cast<const uint32_t*>(&v);
  const float hw = (float)HW;
  uint32_t o[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) o[j] = pack2(lo_bf(w[j]) / hw, hi_bf(w[j]) / hw);
  store_through(dx + (size_t)i * 8, make_uint4(o[0], o[1], o[2], o[3]));
}

// pooled[b, c] = mean over the HW pixels of x[b, p, c]: one workgroup per image, thread (channel group of 8, pixel
// lane); the pixel lanes are added in order
__global__ __launch_bounds__(256) void gap_fwd_bf16_kernel(const uint16_t* x, int HW, int C, uint16_t* pooled) {
  __shared__ float red[256][9];
  const int groups = C / 8, lanes = 256 / groups, cg = threadIdx.x % groups, pl = threadIdx.x / groups;
  const uint16_t* xb = x + (size_t)blockIdx.x * HW * C + 8 * cg;
  float a[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (pl < lanes)
    for (int p0 = pl; p0 < HW; p0 += 4 * lanes) {     // four loads in flight
      uint4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int pp = p0 + u * lanes;
        v[u] = pp < HW ? *reinterpret_cast<const uint4*>(xb + (size_t)pp * C) : make_uint4(0, 0, 0, 0);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t* w = reinterpret_cast<const uint32_t*>(&v[u]);
#pragma unroll
        for (int j = 0; j < 4; ++j) { a[2 * j] += lo_bf(w[j]); a[2 * j + 1] += hi_bf(w[j]); }
      }
    }
#pragma unroll
  for (int j = 0; j < 8; ++j) red[threadIdx.x][j] = a[j];
  __syncthreads();
  if (threadIdx.x < C) {
    const int g = threadIdx.x / 8, j = threadIdx.x % 8;
    float t = 0.f;
    for (int l = 0; l < lanes; ++l) t += red[l * groups + g][j];
    pooled[(size_t)blockIdx.x * C + threadIdx.x] = f32_to_bf16(t / HW);
  }
}

// y[b,oy,ox,c] = x[b, oy*stride, ox*stride, c] for c < Ci, 0 above
__global__ __launch_bounds__(256) void shortcut_fwd_bf16_kernel(const uint16_t* x, uint32_t H, uint32_t W, uint32_t Ci,
                                                                uint32_t Co, uint32_t stride, uint32_t Ho, uint32_t Wo,
                                                                uint32_t chunks, uint16_t* y) {
  const uint32_t i = blockIdx.x * 256 + threadIdx.x;
  if (i >= chunks) return;
  const uint32_t cpr = Co / 8, cg = i % cpr, pix = i / cpr, ox = pix % Wo, oy = (pix / Wo) % Ho, b = pix / (Wo * Ho);
  uint4 v = make_uint4(0, 0, 0, 0);
  if (8 * cg < Ci) v = *reinterpret_cast<const uint4*>(x + ((size_t)(b * H + oy * stride) * W + ox * stride) * Ci + 8 * cg);
  store_through(y + (size_t)i * 8, v);
}

// dx[b, oy*stride, ox*stride, c] += dy[b,oy,ox,c] * (ymask[b,oy,ox,c] > 0) for c < Ci
__global__ __launch_bounds__(256) void shortcut_bwd_bf16_kernel(const uint16_t* dy, const uint16_t* ymask, uint32_t H,
                                                                uint32_t W, uint32_t Ci, uint32_t Co, uint32_t stride,
                                                                uint32_t Ho, uint32_t Wo, uint32_t chunks, uint16_t* dx) {
  const uint32_t i = blockIdx.x * 256 + threadIdx.x;
  if (i >= chunks) return;
  const uint32_t cpr = Ci / 8, cg = i % cpr, pix = i / cpr, ox = pix % Wo, oy = (pix / Wo) % Ho, b = pix / (Wo * Ho);
  const size_t yi = (size_t)pix * Co + 8 * cg, xi = ((size_t)(b * H + oy * stride) * W + ox * stride) * Ci + 8 * cg;
  const uint4 dv = *reinterpret_cast<const uint4*>(dy + yi), mv = *reinterpret_cast<const uint4*>(ymask + yi);
  const uint4 xv = *reinterpret_cast<const uint4*>(dx + xi);
  const uint32_t* dw = reinterpret_cast<const uint32_t*>(&dv);
  const uint32_t* mw = reinterpret_cast<const uint32_t*>(&mv);
  const uint32_t* xw = reinterpret_cast<const uint32_t*>(&xv);
  uint32_t o[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float lo = lo_bf(xw[j]) + (lo_bf(mw[j]) > 0.f ? lo_bf(dw[j]) : 0.f);
    const float hi = hi_bf(xw[j]) + (hi_bf(mw[j]) > 0.f ? hi_bf(dw[j]) : 0.f);
    o[j] = pack2(lo, hi);
  }
  *reinterpret_cast<uint4*>(dx + xi) = make_uint4(o[0], o[1], o[2], o[3]);
}

bool al16(const void* p) { return !(((uintptr_t)p) & 15); }

// LDS of the implicit-GEMM convolution: the filter as [produced channels rounded up to 32][9 * reduced + 8] bf16
size_t conv_mfma_lds(int produced, int reduced) { return (size_t)((produced + 31) / 32 * 32) * (18 * reduced + 16); }
constexpr size_t CONV_MFMA_LDS_MAX = 96 * 1024;
// workgroups of the forward / stride-1 kernel for P output pixels: a workgroup keeps its filter for up to 4 tiles of
// 128 pixels once there are more than 2048 of them
long conv_mfma_blocks(long P) {
  const long ntiles = (P + 127) / 128;
  const long tpw = ntiles >= 8192 ? 4 : (ntiles >= 4096 ? 2 : 1);
  return (ntiles + tpw - 1) / tpw;
}
template <int MODE, int K16, int NT, int GRP, bool LIN, bool STAT>
int conv_mfma_launch_g(hipStream_t s, const ConvArgs& p, long P, size_t lds) {
  lds += STAT ? CONV_STAT_LDS : 0;
  static OncePerDevice once;
  PPLL_TRY(raise_lds((const void*)conv3x3_mfma_kernel<MODE, K16, NT, GRP, LIN, STAT>, (int)(CONV_MFMA_LDS_MAX + CONV_STAT_LDS), once));
  hipLaunchKernelGGL((conv3x3_mfma_kernel<MODE, K16, NT, GRP, LIN, STAT>), dim3((unsigned)conv_mfma_blocks(P)), dim3(256), lds, s, p);
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}
template <int MODE, int K16>
int conv_mfma_launch_k(hipStream_t s, const ConvArgs& p, long P, size_t lds) {
  const int produced = MODE == 0 ? p.Co : p.Ci;
  // GRP = 1: the three taps of a filter row in flight together
  // linear tap addressing through a buffer descriptor: forward always, input gradient at stride 1; the source
  // tensor has to stay below 2^30 bytes
  const bool lin = (MODE == 0 || p.stride == 1) && (long)p.B * p.H * p.W * (16 * K16) * 2 < ((long)1 << 30);
  if (p.stat) {
    if (produced <= 32)
      return lin ? conv_mfma_launch_g<MODE, K16, 1, 1, true, true>(s, p, P, lds) : conv_mfma_launch_g<MODE, K16, 1, 1, false, true>(s, p, P, lds);
    return lin ? conv_mfma_launch_g<MODE, K16, 2, 1, true, true>(s, p, P, lds) : conv_mfma_launch_g<MODE, K16, 2, 1, false, true>(s, p, P, lds);
  }
  if (produced <= 32)
    return lin ? conv_mfma_launch_g<MODE, K16, 1, 1, true, false>(s, p, P, lds) : conv_mfma_launch_g<MODE, K16, 1, 1, false, false>(s, p, P, lds);
  return lin ? conv_mfma_launch_g<MODE, K16, 2, 1, true, false>(s, p, P, lds) : conv_mfma_launch_g<MODE, K16, 2, 1, false, false>(s, p, P, lds);
}
// k16 = reduced channels / 16: 1, 2, 3 or 4
template <int MODE>
int conv_mfma_launch(hipStream_t s, const ConvArgs& p, long P, int k16, size_t lds) {
  switch (k16) {
    case 1: return conv_mfma_launch_k<MODE, 1>(s, p, P, lds);
    case 2: return conv_mfma_launch_k<MODE, 2>(s, p, P, lds);
    case 3: return conv_mfma_launch_k<MODE, 3>(s, p, P, lds);
    case 4: return conv_mfma_launch_k<MODE, 4>(s, p, P, lds);
  }
  set_error("conv3x3: %d reduced channels have no matrix-core kernel", 16 * k16);
  return PPLL_ERR_CONFIG;
}
}  // namespace

// the convolution kernels index pixels with 32 bits
bool conv_pixels_fit(int B, int H, int W) { return (size_t)B * H * W < ((size_t)1 << 31) - 128; }
bool conv_bf16_supported(int dt, int wdt, int Ci, int Co, const void* a, const void* b, const void* c) {
  if (dt != BF16 || wdt != BF16) return false;
  if ((Ci % 16) || (Co % 16) || Ci > 128 || Co > 128) return false;
  return al16(a) && al16(b) && al16(c);
}

template <int K16, int NT>
static int conv_dgrad_s2_launch_k(hipStream_t s, const ConvArgs& p, size_t lds) {
  static OncePerDevice once;
  PPLL_TRY(raise_lds((const void*)conv3x3_dgrad_s2_kernel<K16, NT>, 160 * 1024, once));
  const long pc = (long)p.B * (p.H / 2) * (p.W / 2);
  // One round of what the units hold.  Up to half of that, two workgroups a tile (a row parity each).
  const uint32_t tiles = (uint32_t)((pc + DG_PX - 1) / DG_PX);
  lds += dgrad_s2_tile_bytes<K16>();
  const uint32_t places = std::max(1, compute_units()) * (uint32_t)(160 * 1024 / lds);
  const int parts = 2 * tiles <= places ? 2 : 1;
  hipLaunchKernelGGL((conv3x3_dgrad_s2_kernel<K16, NT>), dim3(std::min(parts * tiles, places)), dim3(256), lds, s, p, parts);
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}
static int conv_dgrad_s2_launch(hipStream_t s, const ConvArgs& p, int k16, size_t lds) {
  const bool two = p.Ci > 32;
  switch (k16) {
    case 1: return two ? conv_dgrad_s2_launch_k<1, 2>(s, p, lds) : conv_dgrad_s2_launch_k<1, 1>(s, p, lds);
    case 2: return two ? conv_dgrad_s2_launch_k<2, 2>(s, p, lds) : conv_dgrad_s2_launch_k<2, 1>(s, p, lds);
    case 3: return two ? conv_dgrad_s2_launch_k<3, 2>(s, p, lds) : conv_dgrad_s2_launch_k<3, 1>(s, p, lds);
    case 4: return two ? conv_dgrad_s2_launch_k<4, 2>(s, p, lds) : conv_dgrad_s2_launch_k<4, 1>(s, p, lds);
  }
  set_error("conv3x3: %d reduced channels have no matrix-core kernel", 16 * k16);
  return PPLL_ERR_CONFIG;
}

int launch_conv3x3_fwd_bf16(hipStream_t s, const void* x, const void* w, int B, int H, int W, int Ci, int Co,
                            int stride, void* y, float* stat, int* stat_blocks) {
  const long P = (long)B * ((H - 1) / stride + 1) * ((W - 1) / stride + 1);
  // The sums cost the kernel registers and ~25 % of its time at 16 channels; they pay where the BatchNorm's own pass
  // over the tensor is mostly launch and ramp, i.e. on small tensors (measured: 9 % of the step at 128 x 16 x 16 x 32,
  // 3 % at 1024 x 8 x 8 x 64, a loss at 1024 x 16 x 16 x 32 and above, where also 2048 partial rows have to be added up)
  if (conv_mfma_blocks(P) > CONV_STAT_MAX_BLOCKS) stat = nullptr;
  ConvArgs p{(const uint16_t*)x, (const uint16_t*)w, (uint16_t*)y, B, H, W, Ci, Co, stride, nullptr, nullptr, stat,
             nullptr, nullptr, nullptr, nullptr};
  if (stat_blocks) *stat_blocks = stat ? (int)conv_mfma_blocks(P) : 0;
  const size_t lds = conv_mfma_lds(Co, Ci);
  void* prof = nullptr;   // algorithmic bytes: input, output and filter once
  PPLL_TRY(profile_begin(s, 2.0 * ((double)B * H * W * Ci + (double)P * Co + 9.0 * Ci * Co), &prof, 1));
  PPLL_TRY((conv_mfma_launch<0>(s, p, P, Ci / 16, lds)));
  return profile_end(s, prof);
}

int launch_conv3x3_dgrad_bf16(hipStream_t s, const void* dy, const void* w, int B, int H, int W, int Ci, int Co,
                              int stride, const void* dres, const void* ymask, void* dx, const BnBwdSums* bn,
                              int* stat_blocks) {
  const long P = (long)B * H * W;
  // sums for the BatchNorm that dx is the output gradient of: stride 1 only, small tensors only (as in the forward)
  const bool sums = bn && bn->partials && stride == 1 && conv_mfma_blocks(P) <= CONV_BWD_STAT_MAX_BLOCKS && al16(bn->y) &&
                    al16(bn->x) && al16(bn->mean) && al16(bn->rstd);
  if (stat_blocks) *stat_blocks = sums ? (int)conv_mfma_blocks(P) : 0;
  ConvArgs p{(const uint16_t*)dy, (const uint16_t*)w, (uint16_t*)dx, B, H, W, Ci, Co, stride, (const uint16_t*)dres,
             (const uint16_t*)ymask, sums ? bn->partials : nullptr, sums ? (const uint16_t*)bn->y : nullptr,
             sums ? (const uint16_t*)bn->x : nullptr, sums ? bn->mean : nullptr, sums ? bn->rstd : nullptr};
  const size_t lds = conv_mfma_lds(Ci, Co);
  const double Po = (double)B * ((H - 1) / stride + 1) * ((W - 1) / stride + 1);
  void* prof = nullptr;   // algorithmic bytes: dy, dx and filter once, plus the shortcut gradient and its mask
  PPLL_TRY(profile_begin(s, 2.0 * (Po * Co + (double)P * Ci * (dres ? 3.0 : 1.0) + 9.0 * Ci * Co), &prof, 1));
  if (stride == 2 && !(H & 1) && !(W & 1) && !dres && Po * Co * 2 < (double)(1 << 30))
    PPLL_TRY(conv_dgrad_s2_launch(s, p, Co / 16, lds));
  else
    PPLL_TRY((conv_mfma_launch<1>(s, p, P, Co / 16, lds)));
  return profile_end(s, prof);
}

// forward and input gradient produce up to 64 channels (two MFMA tiles of 32; 16 and 48 leave half a tile idle)
bool conv_fwd_bf16_ok(int Ci, int Co) { return Co % 16 == 0 && Co <= 64 && Ci <= 64 && conv_mfma_lds(Co, Ci) <= CONV_MFMA_LDS_MAX; }
bool conv_dgrad_bf16_ok(int Ci, int Co) { return Ci % 16 == 0 && Ci <= 64 && Co <= 64 && conv_mfma_lds(Ci, Co) <= CONV_MFMA_LDS_MAX; }
bool bn_bf16_supported(int dt, int rows, int C, const void* a, const void* b, const void* c, const void* d) {
  if (dt != BF16 || (C % 8) || C < 8 || C > 128 || (256 % (C / 8))) return false;
  if ((size_t)rows * C / 8 >= ((size_t)1 << 32)) return false;   // the kernels index 16-byte chunks with 32 bits
  return al16(a) && al16(b) && al16(c) && al16(d);
}
static int bn_blocks(int rows, int C) {
  const int lanes = 256 / (C / 8);
  int blocks = (rows + lanes * 8 - 1) / (lanes * 8);     // about eight rows per thread
  return blocks < 1 ? 1 : (blocks > 256 ? 256 : blocks);
}
template <int KIND>
static int bn_sums_launch(hipStream_t s, const BnSumArgs& p, int blocks, bool finish) {
  hipLaunchKernelGGL(bn_sums_kernel<KIND>, dim3(blocks), dim3(256), 0, s, p);
  PPLL_HIP(hipGetLastError());
  if (finish) {
    hipLaunchKernelGGL(bn_finish_kernel<KIND>, dim3(1), dim3(1024), 0, s, p, (unsigned)blocks);
    PPLL_HIP(hipGetLastError());
  }
  return PPLL_OK;
}
// the apply kernel of a small tensor (at most 1024 workgroups) finishes the sums itself
static bool bn_fused_finish(size_t chunks) { return (chunks + 255) / 256 <= 1024; }
// room for the partials of the BatchNorm's own sums kernels or of the convolution that produced its input (one row of
// pixels per BatchNorm row), whichever are more
size_t bn_bf16_partial_floats(int rows, int C) {
  const long a = bn_blocks(rows, C), b = conv_mfma_blocks(rows);
  return (size_t)(a > b ? a : b) * 2 * C;
}

// The three helpers need channel counts that are multiples of 8, 16-byte aligned tensors and fewer than 2^31 elements.
bool eltwise_bf16_ok(int dt, size_t elems, int C0, int C1, const void* a, const void* b, const void* c) {
  return dt == BF16 && (C0 % 8) == 0 && (C1 % 8) == 0 && elems < ((size_t)1 << 31) && al16(a) && al16(b) && al16(c);
}
// C a multiple of 8 that divides 256 * 8 into whole pixel lanes, at most 256 channels
bool gap_fwd_bf16_ok(int dt, int C, const void* x, const void* pooled) {
  return dt == BF16 && (C % 8) == 0 && C >= 8 && C <= 256 && (256 % (C / 8)) == 0 && al16(x) && !(((uintptr_t)pooled) & 1);
}
int launch_gap_fwd_bf16(hipStream_t s, const void* x, int B, int HW, int C, void* pooled) {
  hipLaunchKernelGGL(gap_fwd_bf16_kernel, dim3(B), dim3(256), 0, s, (const uint16_t*)x, HW, C, (uint16_t*)pooled);
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}
int launch_gap_bwd_bf16(hipStream_t s, const void* dpooled, int B, int HW, int C, void* dx) {
  const uint32_t chunks = (uint32_t)((size_t)B * HW * C / 8);
  hipLaunchKernelGGL(gap_bwd_bf16_kernel, dim3((chunks + 255) / 256), dim3(256), 0, s, (const uint16_t*)dpooled, (uint32_t)HW,
                     (uint32_t)C, chunks, (uint16_t*)dx);
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}
int launch_shortcut_fwd_bf16(hipStream_t s, const void* x, int B, int H, int W, int Ci, int Co, int stride, void* y) {
  const uint32_t Ho = (H - 1) / stride + 1, Wo = (W - 1) / stride + 1;
  const uint32_t chunks = (uint32_t)((size_t)B * Ho * Wo * Co / 8);
  hipLaunchKernelGGL(shortcut_fwd_bf16_kernel, dim3((chunks + 255) / 256), dim3(256), 0, s, (const uint16_t*)x, (uint32_t)H,
                     (uint32_t)W, (uint32_t)Ci, (uint32_t)Co, (uint32_t)stride, Ho, Wo, chunks, (uint16_t*)y);
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}
int launch_shortcut_bwd_bf16(hipStream_t s, const void* dy, const void* ymask, int B, int H, int W, int Ci, int Co, int stride,
                             void* dx) {
  const uint32_t Ho = (H - 1) / stride + 1, Wo = (W - 1) / stride + 1;
  const uint32_t chunks = (uint32_t)((size_t)B * Ho * Wo * Ci / 8);
  hipLaunchKernelGGL(shortcut_bwd_bf16_kernel, dim3((chunks + 255) / 256), dim3(256), 0, s, (const uint16_t*)dy,
                     (const uint16_t*)ymask, (uint32_t)H, (uint32_t)W, (uint32_t)Ci, (uint32_t)Co, (uint32_t)stride, Ho, Wo, chunks,
                     (uint16_t*)dx);
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}

int launch_bn_stats_bf16(hipStream_t s, const void* x, int rows, int C, float eps, float momentum, float* partials,
                         float* mean, float* rstd, float* run_mean, float* run_var) {
  BnSumArgs p{};
  p.x = (const uint16_t*)x; p.rows = rows; p.C = C; p.partial = partials; p.eps = eps;
  p.momentum = momentum; p.out0 = mean; p.out1 = rstd; p.run_mean = run_mean; p.run_var = run_var;
  PPLL_TRY(bn_sums_launch<0>(s, p, bn_blocks(rows, C), true));
  return PPLL_OK;
}

// statistics and y = relu(bn(x) (+ res)) of a training step
// ready_blocks > 0: `partials` already holds that many rows of sums, written by the convolution that produced x
int launch_bn_train_fwd_bf16(hipStream_t s, const void* x, int rows, int C, float eps, float momentum, float* partials,
                             float* mean, float* rstd, float* run_mean, float* run_var, const float* g, const float* b,
                             const void* res, void* y, int ready_blocks, uint8_t* mask) {
  BnSumArgs p{};
  p.x = (const uint16_t*)x; p.rows = rows; p.C = C; p.partial = partials; p.eps = eps;
  p.momentum = momentum; p.out0 = mean; p.out1 = rstd; p.run_mean = run_mean; p.run_var = run_var;
  const size_t chunks = (size_t)rows * C / 8;
  const int blocks = ready_blocks > 0 ? ready_blocks : bn_blocks(rows, C);
  // every workgroup of the fused kernel adds up all partial rows itself: only worth it for few of both
  if (!bn_fused_finish(chunks) || blocks > 256) {
    if (ready_blocks > 0) {
      hipLaunchKernelGGL(bn_finish_kernel<0>, dim3(1), dim3(1024), 0, s, p, (unsigned)blocks);
      PPLL_HIP(hipGetLastError());
    } else {
      PPLL_TRY(bn_sums_launch<0>(s, p, blocks, true));
    }
    return launch_bn_apply_bf16(s, x, rows, C, mean, rstd, g, b, res, y, mask);
  }
  if (ready_blocks <= 0) PPLL_TRY(bn_sums_launch<0>(s, p, blocks, false));
  hipLaunchKernelGGL(bn_apply_fused_kernel, dim3((unsigned)((chunks + 255) / 256)), dim3(256), 0, s, p, (unsigned)blocks, chunks,
                     g, b, (const uint16_t*)res, (uint16_t*)y, mask);
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}

static int bn_apply_launch(hipStream_t s, int pieces, const void* x, size_t chunks, int C, const float* mean, const float* rstd,
                           const float* g, const float* b, const void* res, void* y, uint8_t* mask) {
  const dim3 grid((unsigned)((chunks + 256 * pieces - 1) / (256 * pieces)));
  auto kernel = pieces == 1 ? bn_apply_bf16_kernel<1> : bn_apply_bf16_kernel<AP_PIECES>;
  hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, (const uint16_t*)x, chunks, C, mean, rstd, g, b, (const uint16_t*)res, (uint16_t*)y, mask);
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}
int launch_bn_apply_bf16(hipStream_t s, const void* x, int rows, int C, const float* mean, const float* rstd,
                         const float* g, const float* b, const void* res, void* y, uint8_t* mask, int units) {
  const size_t chunks = (size_t)rows * C / 8;
  return bn_apply_launch(s, bn_apply_pieces(chunks, units ? units : compute_units()), x, chunks, C, mean, rstd, g, b, res, y, mask);
}

// ready_blocks > 0: `partials` already holds that many rows of the two sums, written by the convolution that produced dy
int launch_bn_bwd_bf16(hipStream_t s, const void* dy, const void* y, const void* x, int rows, int C, const float* mean,
                       const float* rstd, const float* g, float* partials, float* dg, float* db, void* dx, int ready_blocks) {
  BnSumArgs p{};
  p.x = (const uint16_t*)x; p.dy = (const uint16_t*)dy; p.y = (const uint16_t*)y; p.rows = rows; p.C = C;
  p.mean = mean; p.rstd = rstd; p.partial = partials; p.out0 = db; p.out1 = dg;
  const size_t chunks = (size_t)rows * C / 8;
  const int blocks = ready_blocks > 0 ? ready_blocks : bn_blocks(rows, C);
  if (bn_fused_finish(chunks) && blocks <= 256) {
    if (ready_blocks <= 0) PPLL_TRY(bn_sums_launch<1>(s, p, blocks, false));
    hipLaunchKernelGGL(bn_bwd_apply_fused_kernel, dim3((unsigned)((chunks + 255) / 256)), dim3(256), 0, s, p, (unsigned)blocks,
                       chunks, g, (uint16_t*)dx);
    PPLL_HIP(hipGetLastError());
    return PPLL_OK;
  }
  if (ready_blocks > 0) {
    hipLaunchKernelGGL(bn_finish_kernel<1>, dim3(1), dim3(1024), 0, s, p, (unsigned)blocks);
    PPLL_HIP(hipGetLastError());
  } else {
    PPLL_TRY(bn_sums_launch<1>(s, p, blocks, true));
  }
  hipLaunchKernelGGL(bn_bwd_apply_bf16_kernel, dim3((unsigned)((chunks + 256 * AP_PIECES - 1) / (256 * AP_PIECES))), dim3(256), 0, s,
                     (const uint16_t*)dy, (const uint16_t*)y, (const uint16_t*)x, chunks, C, rows, mean, rstd, g, dg, db,
                     (uint16_t*)dx);
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}

int launch_bn_sums_fwd_bf16(hipStream_t s, const void* x, int rows, int C, float* partials, int* blocks) {
  BnSumArgs p{};
  p.x = (const uint16_t*)x; p.rows = rows; p.C = C; p.partial = partials;
  *blocks = bn_blocks(rows, C);
  return bn_sums_launch<0>(s, p, *blocks, false);
}
int launch_bn_sums_bwd_bf16(hipStream_t s, const void* dy, const void* y, const void* x, int rows, int C, const float* mean,
                            const float* rstd, float* partials, int* blocks) {
  BnSumArgs p{};
  p.x = (const uint16_t*)x; p.dy = (const uint16_t*)dy; p.y = (const uint16_t*)y; p.rows = rows; p.C = C;
  p.mean = mean; p.rstd = rstd; p.partial = partials;
  *blocks = bn_blocks(rows, C);
  return bn_sums_launch<1>(s, p, *blocks, false);
}

}  // namespace ppll

// Input gradient of a 3x3 convolution of stride 2, bf16, for tests (no part of the public interface)
extern "C" int ppll_internal_conv_dgrad_s2(int B, int H, int W, int Ci, int Co, const void* dy, const void* w, void* dx, void* stream) {
  using namespace ppll;
  if ((H & 1) || (W & 1) || !conv_dgrad_bf16_ok(Ci, Co) || !conv_bf16_supported(BF16, BF16, Ci, Co, dy, w, dx)) {
    set_error("no such launch");
    return PPLL_ERR_CONFIG;
  }
  return launch_conv3x3_dgrad_bf16((hipStream_t)stream, dy, w, B, H, W, Ci, Co, 2, nullptr, nullptr, dx, nullptr, nullptr);
}

// y = relu(bn(x) (+ res)) and its mask, bf16, 1 or AP_PIECES pieces a thread, for tests (no part of the public interface)
extern "C" int ppll_internal_bn_apply(int pieces, int rows, int C, const void* x, const float* mean, const float* rstd, const float* g,
                                      const float* b, const void* res, void* y, void* mask, void* stream) {
  using namespace ppll;
  if ((pieces != 1 && pieces != AP_PIECES) || !bn_bf16_supported(BF16, rows, C, x, y, res, nullptr)) { set_error("no such launch"); return PPLL_ERR_CONFIG; }
  return bn_apply_launch((hipStream_t)stream, pieces, x, (size_t)rows * C / 8, C, mean, rstd, g, b, res, y, (uint8_t*)mask);
}
