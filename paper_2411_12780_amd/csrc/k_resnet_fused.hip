// 3x3 convolution, stride 1, C -> C channels (16, 32 or 64), with the BatchNorm in front of it applied on the way in:
//  forward: y = relu(bn(x) (+ residual)) is formed once per pixel, stored (the backward pass and the shortcut read it) and
//    laid in LDS with a one-pixel border, the convolution reads it there and leaves the sums that the BatchNorm behind it
//    needs of the stored outputs;
//  backward: the input gradient d of the BatchNorm behind the convolution (from dy, the ReLU mask and the two finished sums)
//    is formed once per pixel, stored (the weight gradient reads it) and laid in LDS, the transposed convolution reads it
//    there, adds the shortcut's gradient and leaves the backward sums of the BatchNorm in front.
//
// What bounds these layers is the number of times a feature map crosses the memory (large maps) and the number of dependent
// launches (small ones).  A BatchNorm and its convolution, microseconds on an MI355X, as separate kernels (sums, finish,
// apply, convolution gathering its nine taps from memory) and here:
//                        1024 x 32 x 32 x 16    848 x 8 x 8 x 64    128 x 16 x 16 x 32
//   forward                    51 -> 29.5           29.5 -> 16          11.5 -> 7.1
//   backward                   76 -> 47             36 -> 20            13.6 -> 8.6
// (at the first of them the maps alone take 20 - 27 and 34 - 41 us at a copy's rate).  A tile of 256 (128) pixels is loaded
// with 16-byte loads while the tile before it is multiplied, pixels lie 2 C + 16 bytes apart in LDS (16 lanes reading 16
// bytes of neighbouring pixels hit every bank once), a workgroup keeps its filter for all its tiles.  One workgroup of eight
// waves per compute unit, two with 16 channels and of four waves: few enough partial sums for every workgroup of the next
// kernel to add them up itself.
// ReLU masks travel as one bit an element.  Partial sums, parameters, first tile and filter are asked for together: waiting for them in
// turn, a small forward launch took 10.8 instead of 7.1 us.
//
// With 16 channels and several tiles a workgroup the backward form leaves the convolution's weight gradient as well: d is in LDS with its
// border, the convolution's input comes along at the tile's own pixels, and neither d nor, where it is the output of a block's first
// BatchNorm, that input is stored (it is formed again from the input of the BatchNorm, which is read for its sums).  Ten convolutions of
// 1024 x 32 x 32 x 16: 47 us each and 151 for the ten weight gradients, now 46.5 each.
//
// What bounds the large maps is the vector unit, 70 - 76 % busy.  So the places of a thread's pieces are kept from tile to tile, what lies
// beyond the last image is out of range of a buffer and not behind a branch, a mask's bit is spread over a word and combined with AND
// (with the weight gradients, a stage of ResNet-32 at batch 1024: 1207 -> 1045 us; five blocks of 848 x 8 x 8 x 64: 511 -> 500).
#include "resnet_bf16.h"

namespace ppll {

namespace {
struct ConvBnArgs {
  const uint16_t* x;      // BatchNorm input [B,H,W,C] (forward with bn = 0: the convolution's input as it is)
  const uint16_t* aux;    // forward: residual (or null); backward: dy, the gradient at the BatchNorm's output
  const uint8_t* mask;    // backward: ReLU mask of the BatchNorm's output
  uint16_t* mid;          // forward: y out (or null); backward: d out (unless the weight gradient is formed here)
  uint8_t* mask_out;      // forward: ReLU mask of y (or null), bit e of byte i: element 8 i + e is positive
  const uint16_t* w;      // [9][C][C]
  uint16_t* dst;          // the convolution's result
  float* stat;            // [workgroups][2][C] sums for the next BatchNorm (backward: may be null)
  const uint16_t* dres; const uint8_t* dmask;    // backward: dst += dres where the mask is set
  // backward: the BatchNorm that dst is the output gradient of
  const uint8_t* nmask; const uint16_t* nx; const float *nmean, *nrstd;
  // weight gradient of the convolution: its input, or the parameters of the next BatchNorm, whose output it is; a partial filter a workgroup
  const uint16_t* in; const float *ng, *nb; float* filters;
  BnSumArgs sums; unsigned nblocks;              // partial sums of the BatchNorm in front, finished by every workgroup
  const float *g, *b;
  int bn;                 // forward: 0 = the input is taken as it is
  int H, wl;              // rows of an image, log2 of the pixels of a row
  int rows;               // B * H
  int sr, srl, seg;       // a tile: seg stretches of sr rows (log2 in srl), each inside one image
  int inv;                // 65536 / (sr + 2), rounded up
  int tiles;
  uint32_t bytes;         // of a [B,H,W,C] tensor
};

template <int C, bool BWD> constexpr int filter_bytes() {
  return BWD ? (C + 31) / 32 * 32 * (18 * C + 16) : 9 * C * ((C + 31) / 32 * 64);
}
constexpr int pixel_pitch(int C) { return 2 * C + 16; }
// rows of an image that a tile of 32 `waves` pixels takes, and its bytes in LDS
constexpr int tile_rows(int waves, int H, int W) { return 32 * waves / W < H ? 32 * waves / W : H; }
constexpr int tile_bytes(int waves, int H, int W, int C) {
  return 32 * waves / W / tile_rows(waves, H, W) * (tile_rows(waves, H, W) + 2) * (W + 2) * pixel_pitch(C);
}
constexpr int most_tile_bytes(int C, int waves) {   // of any map that conv_bn_ok accepts
  int most = 0;
  for (int H = 8; H <= 32; H *= 2)
    for (int W = 8; W <= 32; W *= 2) most = tile_bytes(waves, H, W, C) > most ? tile_bytes(waves, H, W, C) : most;
  return most;
}
// Floats from one partial filter to the next: not a multiple of 9 KB, see wgt_row() of the weight-gradient kernel
constexpr int filter_row(int C) { return 9 * C * C + 64; }
// From this size of a map on, what the convolution stages is stored through L2: the kernels that follow find a smaller one in L2.
// Microseconds of a step of four basic blocks, ordinary stores / through L2: 32 channels, 0.125 MB 167 / 170, 0.5 MB 175 / 177,
// 1.5 MB 190 / 191, 2 MB 198 / 198, 4 MB 256 / 249; 16 channels, 0.125 MB 144 / 147, 1 MB 161 / 162, 2 MB 180 / 179, 4 MB 256 / 250.  With 64
// channels the two are level up to 1.5 MB, and the choice in the kernel costs 1 %: always through.
constexpr uint32_t THROUGH_BYTES = 2 << 20;

// Whether the weight gradient is formed on the way back as well, and from what: the convolution's input y as it lies in memory, or formed
// again, relu(bn(nx)), from the input of the next BatchNorm, which is read for its sums anyway (the forward pass then does not store y)
enum FilterGrad { NO_FILTER, INPUT_STORED, INPUT_AGAIN };

// v where bit e of m is set, else 0
__device__ __forceinline__ float where_bit(uint32_t m, int e, float v) {
  uint32_t all;      // the builtin ends up as a comparison and a choice
  asm("v_bfe_i32 %0, %1, %2, 1" : "=v"(all) : "v"(m), "n"(e));
  return __uint_as_float(__float_as_uint(v) & all);
}

template <int C, int WAVES, bool BWD, FilterGrad FG>
__global__ __launch_bounds__(64 * WAVES, C == 16 ? 4 : 1) void conv_bn_kernel(ConvBnArgs p) {
  static_assert(FG == NO_FILTER || (BWD && C == 16 && WAVES == 8), "");
  PPLL_CODE_TO_L2(C == 64 ? 2 : 0);    // narrower filters: no difference
  constexpr int TH = 64 * WAVES, NT = (C + 31) / 32, K16 = C / 16, CG = C / 8, PITCH = pixel_pitch(C);
  constexpr int PB = (C + 31) / 32 * 64, RSW = 18 * C + 16, FILTER = filter_bytes<C, BWD>();
  // staged pieces per thread: C/16 x (sr + 2) / sr; sr is 4 or more, with eight waves 8 or more
  constexpr int NIT = WAVES == 4 ? (3 * K16 + 1) / 2 : (5 * K16 + 3) / 4;
  constexpr int PSTEP = TH / CG;                       // pixels between a thread's pieces
  constexpr int NV = NT * 16, NQ = C < 32 ? 2 : 4;     // 16 channels: half a tile
  constexpr bool FOLD = NV == 32;                      // output sums folded over the lanes tile by tile (64 registers less)
  extern __shared__ __align__(16) char lds[];
  __shared__ __align__(16) float red[2048];            // partial sums being added up; output sums of the waves
  __shared__ __align__(16) float s0[C], s1[C], nbn[FG == INPUT_AGAIN ? 4 : 2][C];
  char* wl = lds;
  char* xt = lds + FILTER;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, li = lane & 31, hh = lane >> 5;
  const int W = 1 << p.wl, WP = W + 2, srp = p.sr + 2;
  const int cg = tid % CG, pi0 = tid / CG, npx = p.seg * srp * W;
  const bool bn = BWD || p.bn;

  // Everything a workgroup waits for at its start is asked for at once, in the order in which it is needed.
  // (1) the partial sums: 2 C values, four per thread; groups of threads take the rows round-robin
  constexpr int NQ4 = C / 2, PARTS = TH / NQ4 < 32 ? TH / NQ4 : 32, U = C == 32 ? 16 : C == 16 ? 4 : 8;
  const int v4 = tid % NQ4, part = tid / NQ4;
  float4 ps[U];
  if (bn && part < PARTS) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const unsigned bu = part + u * PARTS;
      ps[u] = bu < p.nblocks ? *reinterpret_cast<const float4*>(p.sums.partial + (size_t)bu * 2 * C + 4 * v4) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }
  // (2) the BatchNorm's parameters for this thread's eight channels
  float pg[8], pb[8], mean[8], prs[8];
  if (bn) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      pg[j] = p.g[8 * cg + j];
      if (!BWD) pb[j] = p.b[8 * cg + j];
      if (BWD) { mean[j] = p.sums.mean[8 * cg + j]; prs[j] = p.sums.rstd[8 * cg + j]; }
    }
  }
  // (3) the first tile
  const __amdgpu_buffer_rsrc_t rsx = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p.x), 0, (int)p.bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsa = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p.aux), 0, p.aux ? (int)p.bytes : 0, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsm = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p.mask), 0, (int)(p.bytes >> 4), 0x00020000);
  auto tensor = [&](const void* q, uint32_t bytes) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(q), 0, q ? (int)bytes : 0, 0x00020000); };
  const __amdgpu_buffer_rsrc_t rsd = tensor(p.dst, p.bytes), rsdr = tensor(p.dres, p.bytes), rsnx = tensor(p.stat ? p.nx : nullptr, p.bytes), rsin = tensor(p.in, p.bytes);
  const __amdgpu_buffer_rsrc_t rsdm = tensor(p.dres ? p.dmask : nullptr, p.bytes >> 4), rsnm = tensor(p.stat ? p.nmask : nullptr, p.bytes >> 4);
  uint4 rx[NIT], ra[NIT];
  uint32_t rm[BWD ? NIT : 1];
  // A piece of this thread in a tile, of pixel pi: its byte offset (out of range: nothing to load), place in LDS, and whether it lies in
  // the tile proper (not in the border).  What does not change from tile to tile is kept in registers up to 32 channels.
  constexpr bool KEEP = C <= 32;
  int rel[KEEP ? NIT : 1], dy[KEEP ? NIT : 1], at[KEEP ? NIT : 1];      // offset from the tile's first row, row of the image likewise, place
  auto within = [&](int pi, int& rel, int& dy, int& place) {
    const int prow = pi >> p.wl, col = pi & (W - 1);
    const int sg = p.seg > 1 ? __mul24(prow, p.inv) >> 16 : 0, lr = prow - __mul24(sg, srp);
    rel = ((((sg << p.srl) + lr - 1) << p.wl) + col) * (C * 2) + 16 * cg;
    dy = pi < npx ? lr - 1 : 1 << 20;
    place = pi < npx ? (__mul24(prow, WP) + col + 1) * PITCH + 16 * cg : -1;
  };
  if constexpr (KEEP)
#pragma unroll
    for (int it = 0; it < NIT; ++it) within(pi0 + it * PSTEP, rel[it], dy[it], at[it]);
  auto locate = [&](int tile, int p0, int it, int& off, int& place, bool& core) {
    const int row0 = tile * (p.sr * p.seg), y0 = p.seg > 1 ? 0 : row0 & (p.H - 1);
    int r, d;
    if constexpr (KEEP) { r = rel[it]; d = dy[it]; place = at[it]; }
    else within(p0 + it * PSTEP, r, d, place);
    const uint32_t o = (uint32_t)((row0 << p.wl) * (C * 2) + r);
    const bool in = (unsigned)(y0 + d) < (unsigned)p.H && o < p.bytes;
    off = in ? (int)o : CONV_OOB;
    core = in && (unsigned)d < (unsigned)p.sr;
  };
  auto load = [&](int tile, int p0) {
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      int off, place;
      bool core;
      locate(tile, p0, it, off, place, core);
      rx[it] = conv_buf_load16(rsx, off);
      ra[it] = conv_buf_load16(rsa, off);
      if (BWD) rm[it] = __builtin_amdgcn_raw_buffer_load_b8(rsm, off == CONV_OOB ? CONV_OOB : off >> 4, 0, 0);
    }
  };
  load(blockIdx.x, pi0);
  // (4) the filter
  constexpr int NVEC = 9 * C * C / 8, FV = (NVEC + TH - 1) / TH;
  constexpr int FB = FV < 6 ? FV : (FV + 1) / 2;       // 16-byte pieces in flight per thread
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  u32x4 wv[FB];
  auto filter_load = [&](int f0) {
#pragma unroll
    for (int u = 0; u < FB; ++u) wv[u] = *reinterpret_cast<const u32x4*>(p.w + (size_t)min(tid + TH * (f0 + u), NVEC - 1) * 8);
  };
  auto filter_store = [&](int f0) {
#pragma unroll
    for (int u = 0; u < FB; ++u) {
      const int v = tid + TH * (f0 + u);
      const int e = v * 8, co = e % C, ci = (e / C) % C, tap = e / (C * C);
      if (v < NVEC) *reinterpret_cast<u32x4*>(wl + (BWD ? ci * RSW + 2 * (tap * C + co) : (tap * C + ci) * PB + 2 * co)) = wv[u];
    }
  };
  filter_load(0);
  // the border columns stay zero
  for (int i = tid; i < p.seg * srp * 2 * CG; i += TH) {
    const int c = i % CG, q = i / CG, row = q >> 1;
    *reinterpret_cast<uint4*>(xt + (row * WP + (q & 1) * (W + 1)) * PITCH + 16 * c) = make_uint4(0, 0, 0, 0);
  }
  if (bn) {   // sums added in row order within a group of threads, then group by group
    if (part < PARTS) {
      float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
      for (unsigned bk = part;; ) {
#pragma unroll
        for (int u = 0; u < U; ++u) { t.x += ps[u].x; t.y += ps[u].y; t.z += ps[u].z; t.w += ps[u].w; }
        bk += U * PARTS;
        if (bk >= p.nblocks) break;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const unsigned bu = bk + u * PARTS;
          ps[u] = bu < p.nblocks ? *reinterpret_cast<const float4*>(p.sums.partial + (size_t)bu * 2 * C + 4 * v4) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
      }
      *reinterpret_cast<float4*>(red + part * 2 * C + 4 * v4) = t;
    }
    __syncthreads();
    if (tid < C) {
      float a = 0.f, c = 0.f;
#pragma unroll 8
      for (int q = 0; q < PARTS; ++q) { a += red[q * 2 * C + tid]; c += red[q * 2 * C + C + tid]; }
      if (!BWD) bn_statistics(p.sums, tid, a, c, blockIdx.x == 0);
      s0[tid] = a; s1[tid] = c;
      if (blockIdx.x == 0) { p.sums.out0[tid] = a; p.sums.out1[tid] = c; }
    }
  }
  filter_store(0);
  if constexpr (FB < FV) { filter_load(FB); filter_store(FB); }
  if (BWD) {
    for (int c = tid; c < C; c += TH) {
      nbn[0][c] = p.stat ? p.nmean[c] : 0.f; nbn[1][c] = p.stat ? p.nrstd[c] : 0.f;
      if constexpr (FG == INPUT_AGAIN) { nbn[2][c] = p.nrstd[c] * p.ng[c]; nbn[3][c] = p.nb[c]; }
    }
  }
  __syncthreads();
  // this thread's eight channels: mean, scale a = rstd g, shift b; backward: d = a (dyh - k0) - (x - mean) k1
  float a[8], k0[BWD ? 8 : 1], k1[BWD ? 8 : 1];
  if (bn) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int c = 8 * cg + j;
      if (!BWD) mean[j] = s0[c];
      a[j] = (BWD ? prs[j] : s1[c]) * pg[j];
      if (BWD) {
        const float n = (float)p.sums.rows;
        k0[j] = s0[c] / n;
        k1[j] = s1[c] / n * prs[j] * a[j];
      }
    }
  }
  // With a weight gradient to keep they wait in LDS for the next tile
  __shared__ __align__(16) float terms[FG ? 4 : 1][C];
  if constexpr (FG != NO_FILTER) {
    if (pi0 == 0)
#pragma unroll
      for (int j = 0; j < 8; ++j) { terms[0][8 * cg + j] = mean[j]; terms[1][8 * cg + j] = a[j]; terms[2][8 * cg + j] = k0[j]; terms[3][8 * cg + j] = k1[j]; }
    __syncthreads();
  }
  // forward: lane part of a filter fragment address (see conv3x3_mfma_kernel)
  const int tr_lane = (8 * hh + ((lane & 15) >> 2)) * PB + (16 * ((lane >> 4) & 1) + 4 * (lane & 3)) * 2;
  // this lane's pixel of a tile
  const int prow = (wave * 32 + li) >> p.wl, pcol = (wave * 32 + li) & (W - 1);
  const int psg = prow >> p.srl, plr = prow & (p.sr - 1);
  const char* xpix = xt + ((psg * srp + plr + 1) * WP + pcol + 1) * PITCH + 16 * hh;
  float st0[NV], st1[NV], f0 = 0.f, f1 = 0.f;
#pragma unroll
  for (int j = 0; j < NV; ++j) { st0[j] = 0.f; st1[j] = 0.f; }

  // Weight gradient: dw[tap][ci][co] is the sum over the pixels q of y[q][ci] d[q - tap][co]: the convolution's input at the tile's own
  // pixels, which the output phase leaves in LDS, and d with its border as it is staged.  A fragment is 8 pixels of a channel, out of
  // transposing reads of [pixel][channel].  Wave w has tap w over all pixels of the tile, and of tap 8 its own 32: 8 registers, where all
  // taps over its own pixels are 36 and do not fit beside the rest.
  char* yt = xt + p.seg * srp * WP * PITCH;
  typedef __attribute__((ext_vector_type(4))) float f32x4;
  f32x4 dw[FG ? 2 : 1];
  int dl0 = 0, dl1 = 0;       // this lane's pixels of the first 32 of a tile, and 4 on
  if constexpr (FG != NO_FILTER) {
    dw[0] = dw[1] = (f32x4){0.f, 0.f, 0.f, 0.f};
    auto at = [&](int px) { return (((px >> p.wl) + 1) * WP + (px & (W - 1)) + 1) * PITCH + 8 * (lane & 3); };
    const int px = 8 * (lane >> 4) + ((lane & 15) >> 2);
    dl0 = at(px);
    dl1 = at(px + 4);
  }

  for (int tile = blockIdx.x; tile < p.tiles; tile += gridDim.x) {
    // backward: what is formed from it is formed again in every tile; kept in registers it spills, and a reload waits for
    // the next tile's loads (62 instead of 47 us at 1024 x 32 x 32 x 16)
    int p0 = pi0;
    if (BWD && !KEEP) asm volatile("" : "+v"(p0));
    if constexpr (FG != NO_FILTER) {
      int c = 8 * cg;
      asm volatile("" : "+v"(c));      // read here, in every tile
      auto eight = [&](const float* from, float (&to)[8]) {
        const float4 lo = *reinterpret_cast<const float4*>(from + c), hi = *reinterpret_cast<const float4*>(from + c + 4);
        to[0] = lo.x; to[1] = lo.y; to[2] = lo.z; to[3] = lo.w; to[4] = hi.x; to[5] = hi.y; to[6] = hi.z; to[7] = hi.w;
      };
      eight(terms[0], mean); eight(terms[1], a); eight(terms[2], k0); eight(terms[3], k1);
    }
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      int off, place;
      bool core;
      locate(tile, p0, it, off, place, core);
      const uint32_t* xw = reinterpret_cast<const uint32_t*>(&rx[it]);
      const uint32_t* aw = reinterpret_cast<const uint32_t*>(&ra[it]);
      uint4 o = rx[it];
      uint32_t* ow = reinterpret_cast<uint32_t*>(&o);
      if (bn) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float v[2];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int e = 2 * j + h;
            const float xv = h ? hi_bf(xw[j]) : lo_bf(xw[j]), av = h ? hi_bf(aw[j]) : lo_bf(aw[j]);
            if (BWD) {
              const float dyh = where_bit(rm[BWD ? it : 0], e, av);
              v[h] = fmaf(a[e], dyh - k0[e], -(xv - mean[e]) * k1[e]);
            } else {
              v[h] = fmaxf(bn_value(xv, mean[e], a[e], pb[e]) + av, 0.f);
            }
          }
          ow[j] = pack2(v[0], v[1]);
        }
        if (off == CONV_OOB) o = make_uint4(0, 0, 0, 0);      // rows outside the image
        if (core && FG == NO_FILTER) {
          if (C > 16 || BWD || p.mid) {
            if (C == 64 || p.bytes >= THROUGH_BYTES) store_through((char*)p.mid + off, o);
            else *reinterpret_cast<uint4*>((char*)p.mid + off) = o;
          }
          if (!BWD && p.mask_out) p.mask_out[off >> 4] = relu_mask(o);
        }
      }
      if (place >= 0) *reinterpret_cast<uint4*>(xt + place) = o;
    }
    __syncthreads();
    const int grow = tile * (p.sr * p.seg) + psg * p.sr + plr;
    const uint32_t pix = ((uint32_t)grow << p.wl) + pcol;   // a tensor has fewer than 2^29 elements
    // Pixels beyond the last image: out of range, loads give 0 and stores are dropped (they are whole images, whose staged pixels are 0, and
    // so are their results)
    const int byte0 = grow < p.rows ? (int)(pix * C * 2) + 8 * hh : CONV_OOB_BASE, bits0 = grow < p.rows ? (int)(pix * C >> 3) : CONV_OOB_BASE;
    // backward: what the outputs of the tile are combined with, asked for ahead of the next tile (64 channels: registers only
    // for half of it at a time, asked for at the end)
    uint2 dr[NT][NQ], nx[NT][NQ], yin[FG == INPUT_STORED ? NQ : 1];
    uint32_t dm[NT], nm[NT];                               // a mask's bits of 16 or 32 channels
    auto bits = [&](__amdgpu_buffer_rsrc_t rs, int off) -> uint32_t {
      if constexpr (C == 16) return (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rs, off, 0, 0);
      else return __builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0);
    };
    auto four = [&](__amdgpu_buffer_rsrc_t rs, int off) {
      const auto v = __builtin_amdgcn_raw_buffer_load_b64(rs, off, 0, 0);
      return make_uint2(v[0], v[1]);
    };
    auto outer_load = [&](int t) {
      dm[t] = bits(rsdm, bits0 + 4 * t);
      nm[t] = bits(rsnm, bits0 + 4 * t);
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        dr[t][q] = four(rsdr, byte0 + 64 * t + 16 * q);
        nx[t][q] = four(rsnx, byte0 + 64 * t + 16 * q);
        if constexpr (FG == INPUT_STORED) yin[q] = four(rsin, byte0 + 64 * t + 16 * q);
      }
    };
    if (BWD && NT == 1) outer_load(0);
    if (tile + (int)gridDim.x < p.tiles) load(tile + gridDim.x, p0);
    f32x16 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      const int ky = tap / 3 - 1, kx = tap % 3 - 1;
      const char* xp = xpix + (BWD ? -1 : 1) * (ky * WP + kx) * PITCH;
#pragma unroll
      for (int c16 = 0; c16 < K16; ++c16) {
        const bf16x8 xf = *reinterpret_cast<const bf16x8*>(xp + 32 * c16);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          bf16x8 wf;
          if (BWD) {
            wf = *reinterpret_cast<const bf16x8*>(wl + 2 * (tap * C + 8 * hh) + (t * 32 + li) * RSW + 32 * c16);
          } else {
            const char* fp = wl + tr_lane + (tap * C + 16 * c16) * PB + 64 * t;
            const uint2 lo = conv_lds_read_tr(fp), hi = conv_lds_read_tr(fp + 4 * PB);
            wf = __builtin_bit_cast(bf16x8, make_uint4(lo.x, lo.y, hi.x, hi.y));
          }
          acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf, xf, acc[t], 0, 0, 0);
        }
      }
    }
    // 64 channels forward: four waves 10.75 us a launch at 154 x 8 x 8, 11.4 without the branch; eight at 848 x 8 x 8, ten launches a step, 503
    // us a step with it, 498 without
    if (C != 64 || WAVES == 8 || BWD || grow < p.rows) {
      // acc[t][4q+e] = out[pix][32t + 8q + 4hh + e]
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        if (BWD && NT > 1) outer_load(t);
        uint32_t first_x, first_y, dmh = 0, nmh = 0;       // masks from this half's first channel on
        if (BWD) { dmh = dm[t] >> (4 * hh); nmh = nm[t] >> (4 * hh); }
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          const int c = 32 * t + 8 * q + 4 * hh;
          float v[4] = {acc[t][4 * q], acc[t][4 * q + 1], acc[t][4 * q + 2], acc[t][4 * q + 3]};
          if (BWD) {
            const float rv[4] = {lo_bf(dr[t][q].x), hi_bf(dr[t][q].x), lo_bf(dr[t][q].y), hi_bf(dr[t][q].y)};
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] += where_bit(dmh, 8 * q + e, rv[e]);
          }
          const uint2 o = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
          // lanes l and l + 32 have channels 0 - 3, 8 - 11 and 4 - 7, 12 - 15 of every 16: exchanged, 0 - 7 and 8 - 15, a 16-byte store
          // instead of two of 8 (848 x 8 x 8 x 64, a stage of ten: 520 -> 514 us a step; ResNet-32 in eight modules 2579 -> 2550).  With
          // 16 channels an instruction fills whole lines
          if (q % 2 == 0) {
            first_x = o.x; first_y = o.y;
          } else {
            const auto x = __builtin_amdgcn_permlane32_swap(first_x, o.x, false, false), y = __builtin_amdgcn_permlane32_swap(first_y, o.y, false, false);
            __builtin_amdgcn_raw_buffer_store_b128((conv_u32x4){x[0], y[0], x[1], y[1]}, rsd, byte0 + 8 * hh + 64 * t + 16 * (q - 1), 0, C == 16 ? THROUGH : 0);
          }
          const float r[4] = {lo_bf(o.x), hi_bf(o.x), lo_bf(o.y), hi_bf(o.y)};
          if (!BWD) {
#pragma unroll
            for (int e = 0; e < 4; ++e) { st0[16 * t + 4 * q + e] += r[e]; st1[16 * t + 4 * q + e] += r[e] * r[e]; }
          } else if (p.stat) {
            const float xv[4] = {lo_bf(nx[t][q].x), hi_bf(nx[t][q].x), lo_bf(nx[t][q].y), hi_bf(nx[t][q].y)};
            const float4 mu = *reinterpret_cast<const float4*>(&nbn[0][c]), rs = *reinterpret_cast<const float4*>(&nbn[1][c]);
            const float mv[4] = {mu.x, mu.y, mu.z, mu.w}, rv[4] = {rs.x, rs.y, rs.z, rs.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float d = where_bit(nmh, 8 * q + e, r[e]);
              st0[16 * t + 4 * q + e] += d;
              st1[16 * t + 4 * q + e] += d * (xv[e] - mv[e]) * rv[e];
            }
          }
          if constexpr (FG != NO_FILTER) {
            uint2 y;
            if constexpr (FG == INPUT_AGAIN) {
              const float xv[4] = {lo_bf(nx[t][q].x), hi_bf(nx[t][q].x), lo_bf(nx[t][q].y), hi_bf(nx[t][q].y)};
              const float4 mu = *reinterpret_cast<const float4*>(&nbn[0][c]), sc = *reinterpret_cast<const float4*>(&nbn[2][c]);
              const float4 sh = *reinterpret_cast<const float4*>(&nbn[3][c]);
              const float mv[4] = {mu.x, mu.y, mu.z, mu.w}, av[4] = {sc.x, sc.y, sc.z, sc.w}, bv[4] = {sh.x, sh.y, sh.z, sh.w};
              float yv[4];
#pragma unroll
              for (int e = 0; e < 4; ++e) yv[e] = fmaxf(bn_value(xv[e], mv[e], av[e], bv[e]), 0.f);
              y = make_uint2(pack2(yv[0], yv[1]), pack2(yv[2], yv[3]));
            } else {
              y = yin[q];
            }
            *reinterpret_cast<uint2*>(yt + (wave * 32 + li) * PITCH + 2 * c) = y;
          }
        }
      }
    }
    if (FOLD && (!BWD || p.stat)) {
      halfwave_sums<NV>(st0, li);
      halfwave_sums<NV>(st1, li);
      f0 += st0[0]; f1 += st1[0];
#pragma unroll
      for (int j = 0; j < NV; ++j) { st0[j] = 0.f; st1[j] = 0.f; }
    }
    if constexpr (FG != NO_FILTER) {
      __syncthreads();
      int yl = (8 * (lane >> 4) + ((lane & 15) >> 2)) * PITCH + 8 * (lane & 3), d0 = dl0, d1 = dl1;
      asm volatile("" : "+v"(yl), "+v"(d0), "+v"(d1));     // the taps' addresses are not kept from tile to tile
      auto frag = [](const char* a, const char* b) {
        const uint2 lo = conv_lds_read_tr(a), hi = conv_lds_read_tr(b);
        return __builtin_bit_cast(bf16x8, make_uint4(lo.x, lo.y, hi.x, hi.y));
      };
      const int w = __builtin_amdgcn_readfirstlane(wave);
      auto tap_at = [&](int t) { return -((t / 3 - 1) * WP + t % 3 - 1) * PITCH; };
      auto pixels = [&](int ks, bf16x8& yf) {       // the tile's pixels from 32 ks on: whole rows of one image
        const int row = ks << (5 - p.wl);
        yf = frag(yt + yl + 32 * ks * PITCH, yt + yl + (32 * ks + 4) * PITCH);
        return ((row >> p.srl) * srp + (row & (p.sr - 1))) * WP * PITCH;
      };
      f32x4 sum = {0.f, 0.f, 0.f, 0.f};             // of the tile: sums of tiles make shorter chains than one over all steps
#pragma unroll 2
      for (int ks = 0; ks < WAVES; ++ks) {
        bf16x8 yf;
        const int off = pixels(ks, yf) + tap_at(w);
        sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(yf, frag(xt + d0 + off, xt + d1 + off), sum, 0, 0, 0);
      }
      dw[0] += sum;
      bf16x8 yf;
      const int off = pixels(w, yf) + tap_at(8);
      dw[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(yf, frag(xt + d0 + off, xt + d1 + off), dw[1], 0, 0, 0);
    }
    __syncthreads();
  }
  if constexpr (FG != NO_FILTER) {
    // dw[t][e] = dw[tap][4 (lane / 16) + e][lane % 16]; the waves' shares of tap 8 are added in order
    float* fold = reinterpret_cast<float*>(xt);
    const int place = 4 * (lane >> 4) * C + (lane & 15);
    float* out = p.filters + (size_t)blockIdx.x * filter_row(C);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      out[(wave * C + e) * C + place] = dw[0][e];
      fold[wave * C * C + e * C + place] = dw[1][e];
    }
    __syncthreads();
    if (tid < C * C) {
      float sum = 0.f;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) sum += fold[w * C * C + tid];
      out[8 * C * C + tid] = sum;
    }
  }
  if (!BWD || p.stat) {
    // value index j = 16 t + 4 q + e of lane half hh is channel 32 t + 8 q + 4 hh + e
    if (!FOLD) {
      halfwave_sums<NV>(st0, li);
      halfwave_sums<NV>(st1, li);
      f0 = st0[0]; f1 = st1[0];
    }
    if (NV == 32 || !(li & 1)) {
      const int j = NV == 32 ? li : li >> 1;
      red[((wave * 2 + 0) * 2 + hh) * 32 + j] = f0;
      red[((wave * 2 + 1) * 2 + hh) * 32 + j] = f1;
    }
    __syncthreads();
    if (tid < 2 * C) {
      const int which = tid / C, c = tid % C, j = 16 * (c >> 5) + 4 * ((c & 31) >> 3) + (c & 3), h2 = (c & 7) >> 2;
      float tot = 0.f;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) tot += red[((w * 2 + which) * 2 + h2) * 32 + j];
      p.stat[(size_t)blockIdx.x * 2 * C + tid] = tot;
    }
  }
}

bool cb_al16(const void* p) { return !(((uintptr_t)p) & 15); }
int log2_of(int v) { int l = 0; while ((1 << l) < v) ++l; return l; }
template <int C, int WAVES, bool BWD, FilterGrad FG>
int conv_bn_launch(hipStream_t s, const ConvBnArgs& p, int grid, int in_lds) {
  constexpr int Y = FG ? 32 * WAVES * pixel_pitch(C) : 0;       // the convolution's input at a tile's own pixels
  const int lds = filter_bytes<C, BWD>() + in_lds + Y;
  static OncePerDevice once;
  PPLL_TRY(raise_lds((const void*)conv_bn_kernel<C, WAVES, BWD, FG>, filter_bytes<C, BWD>() + most_tile_bytes(C, WAVES) + Y, once));
  hipLaunchKernelGGL((conv_bn_kernel<C, WAVES, BWD, FG>), dim3(grid), dim3(64 * WAVES), lds, s, p);
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}
// Eight waves (256 pixels) a tile once those give most compute units one (at least 200 tiles), else four: with fewer, half the
// compute units would stand idle, with more, the smaller tile loads its two border rows for half as many pixels.
struct TileShape { int waves, sr, seg, tiles, grid; };
TileShape tile_shape(int B, int H, int W, int C, int units) {
  TileShape t{};
  const long px = (long)B * H * W;
  const int asked = units ? units : compute_units(), cus = asked > 0 ? asked : 256;
  t.waves = px >= 200L * 256 ? 8 : 4;
  const int rt = 32 * t.waves / W;
  t.sr = tile_rows(t.waves, H, W);
  t.seg = rt / t.sr;
  t.tiles = (int)(((long)B * H + rt - 1) / rt);
  const int most = t.waves == 8 && C > 16 ? cus : 2 * cus, per = (t.tiles + most - 1) / most;
  t.grid = (t.tiles + per - 1) / per;
  return t;
}
template <bool BWD>
int conv_bn_dispatch(hipStream_t s, ConvBnArgs& p, const TileShape& t, int B, int H, int W, int C, int* stat_blocks) {
  p.H = H; p.wl = log2_of(W); p.rows = B * H; p.sr = t.sr; p.srl = log2_of(t.sr); p.seg = t.seg;
  p.inv = (65536 + t.sr + 1) / (t.sr + 2); p.tiles = t.tiles; p.bytes = (uint32_t)((long)B * H * W * C * 2);
  const int in_lds = tile_bytes(t.waves, H, W, C);
  if (stat_blocks) *stat_blocks = p.stat ? t.grid : 0;
  if constexpr (BWD) {
    if (p.filters && p.in) return conv_bn_launch<16, 8, true, INPUT_STORED>(s, p, t.grid, in_lds);
    if (p.filters) return conv_bn_launch<16, 8, true, INPUT_AGAIN>(s, p, t.grid, in_lds);
  }
  if (C == 16) return t.waves == 8 ? conv_bn_launch<16, 8, BWD, NO_FILTER>(s, p, t.grid, in_lds) : conv_bn_launch<16, 4, BWD, NO_FILTER>(s, p, t.grid, in_lds);
  if (C == 32) return t.waves == 8 ? conv_bn_launch<32, 8, BWD, NO_FILTER>(s, p, t.grid, in_lds) : conv_bn_launch<32, 4, BWD, NO_FILTER>(s, p, t.grid, in_lds);
  return t.waves == 8 ? conv_bn_launch<64, 8, BWD, NO_FILTER>(s, p, t.grid, in_lds) : conv_bn_launch<64, 4, BWD, NO_FILTER>(s, p, t.grid, in_lds);
}
}  // namespace

// Square-ish power-of-two maps of 8 to 32 pixels a side: a tile is then whole rows of one image or whole images.
bool conv_bn_ok(int dt, int B, int H, int W, int C) {
  auto side = [](int v) { return v == 8 || v == 16 || v == 32; };
  return dt == BF16 && (C == 16 || C == 32 || C == 64) && side(H) && side(W) && (long)B * H * W * C * 2 < (1L << 30) - 64;
}
int conv_bn_stat_blocks(int B, int H, int W, int C) { return tile_shape(B, H, W, C, 0).grid; }
// Where a workgroup has several tiles (above 512 of them, always of eight waves): a partial filter, 9 KB, is written and read again for
// every workgroup, against 32 KB of maps a tile that need not be.  With 32 and 64 channels a filter is 37 and 147 KB.
static size_t filter_floats(const TileShape& t, int C) { return C == 16 && t.waves == 8 && t.tiles > t.grid ? (size_t)t.grid * filter_row(C) : 0; }
size_t conv_bn_filter_floats(int B, int H, int W, int C, int units) { return C == 16 ? filter_floats(tile_shape(B, H, W, C, units), C) : 0; }

int launch_conv_bn_fwd(hipStream_t s, const BnInput* bn, const void* x, const void* w, int B, int H, int W, int C, void* dst,
                       float* stat, int* stat_blocks, int units) {
  ConvBnArgs p{};
  p.x = (const uint16_t*)(bn ? bn->x : x); p.w = (const uint16_t*)w; p.dst = (uint16_t*)dst; p.stat = stat;
  if (bn) {
    p.bn = 1; p.aux = (const uint16_t*)bn->res; p.mid = (uint16_t*)bn->y; p.mask_out = bn->mask; p.g = bn->g; p.b = bn->b; p.nblocks = (unsigned)bn->blocks;
    p.sums.rows = B * H * W; p.sums.C = C; p.sums.partial = bn->partials; p.sums.eps = bn->eps; p.sums.momentum = bn->momentum;
    p.sums.out0 = bn->mean; p.sums.out1 = bn->rstd; p.sums.run_mean = bn->run_mean; p.sums.run_var = bn->run_var;
    if (!cb_al16(bn->res) || !cb_al16(bn->y)) { set_error("conv_bn: unaligned tensors"); return PPLL_ERR_CONFIG; }
  }
  if (!cb_al16(p.x) || !cb_al16(w) || !cb_al16(dst)) { set_error("conv_bn: unaligned tensors"); return PPLL_ERR_CONFIG; }
  void* prof = nullptr;   // the bytes of the convolution alone: input, output and filter once
  PPLL_TRY(profile_begin(s, 2.0 * (2.0 * B * H * W * C + 9.0 * C * C), &prof, 1));
  PPLL_TRY(conv_bn_dispatch<false>(s, p, tile_shape(B, H, W, C, units), B, H, W, C, stat_blocks));
  return profile_end(s, prof);
}

int launch_conv_bn_bwd(hipStream_t s, const BnGrad& bn, const void* w, int B, int H, int W, int C, void* d, const void* dres,
                       const uint8_t* dmask, void* dst, const BnBwdSums* next, float* stat,
                       int* stat_blocks, const ConvFilterGrad* fg, ReduceQueue* rq, int units) {
  ConvBnArgs p{};
  const TileShape t = tile_shape(B, H, W, C, units);
  bool queued = false;
  if (fg) {
    const size_t room = filter_floats(t, C);
    if (!room || (!fg->in && (!next || !fg->g || !fg->b))) { set_error("conv_bn: no weight gradient from this launch"); return PPLL_ERR_CONFIG; }
    p.filters = rq->space(room, &queued);
    if (!queued) { set_error("conv_bn: no room for partial filters"); return PPLL_ERR_WORKSPACE; }   // what is shared holds the sums of a BatchNorm
    p.in = (const uint16_t*)fg->in; p.ng = fg->g; p.nb = fg->b;
    if (!cb_al16(fg->in)) { set_error("conv_bn: unaligned tensors"); return PPLL_ERR_CONFIG; }
  }
  p.x = (const uint16_t*)bn.x; p.aux = (const uint16_t*)bn.dy; p.mask = bn.mask; p.mid = (uint16_t*)d;
  p.w = (const uint16_t*)w; p.dst = (uint16_t*)dst; p.dres = (const uint16_t*)dres; p.dmask = dmask;
  p.g = bn.g; p.b = bn.b; p.nblocks = (unsigned)bn.blocks;
  p.sums.rows = B * H * W; p.sums.C = C; p.sums.partial = bn.partials; p.sums.mean = bn.mean; p.sums.rstd = bn.rstd;
  p.sums.out0 = bn.db; p.sums.out1 = bn.dg;
  if (next) {
    p.stat = stat; p.nmask = next->mask; p.nx = (const uint16_t*)next->x; p.nmean = next->mean; p.nrstd = next->rstd;
  }
  for (const void* q : {(const void*)p.x, (const void*)p.aux, (const void*)d, w, (const void*)dst, dres, (const void*)p.nx})
    if (!cb_al16(q)) { set_error("conv_bn: unaligned tensors"); return PPLL_ERR_CONFIG; }
  void* prof = nullptr;   // the bytes of the convolution alone: its two maps and the filter once, the shortcut gradient where present
  PPLL_TRY(profile_begin(s, 2.0 * ((double)B * H * W * C * (dres ? 3.0 : 2.0) + 9.0 * C * C), &prof, 1));
  PPLL_TRY(conv_bn_dispatch<true>(s, p, t, B, H, W, C, stat_blocks));
  PPLL_TRY(profile_end(s, prof));
  if (!fg) return PPLL_OK;
  return reduce_conv_filters(s, *rq, queued, p.filters, t.grid, filter_row(C), C, C, C, fg->dw);
}

}  // namespace ppll

// Backward of a BatchNorm and the convolution in front of it, 16 channels, with its weight gradient, for tests (no part of the public
// interface): in one launch (filters), or with d stored and the weight gradient from a launch of its own.  The convolution's input is `in`,
// or, where that is null, relu(bn(nx)), formed in y in the second case.  sums: one row of the BatchNorm's two sums; stat: room for those
// of the next, whose rows are reported; arena: room for partial filters.
extern "C" int ppll_internal_conv_bn_bwd(int filters, int B, int H, int W, const void* x, const void* dy, const void* mask, float* sums, const float* mean,
                                         const float* rstd, const float* g, float* dgb, const void* w, void* d, const void* dres, const void* dmask,
                                         void* dst, const void* nx, const void* nmask, const float* nmean, const float* nrstd, const float* ng,
                                         const float* nb, float* stat, int* stat_rows, const void* in, void* y, float* dw, float* arena,
                                         size_t arena_floats, void* stream) {
  using namespace ppll;
  hipStream_t s = (hipStream_t)stream;
  constexpr int C = 16;
  if (!conv_bn_ok(BF16, B, H, W, C) || (filters && !conv_bn_filter_floats(B, H, W, C))) { set_error("no such launch"); return PPLL_ERR_CONFIG; }
  ReduceQueue rq;
  rq.arena = rq.scratch = arena; rq.arena_floats = arena_floats;
  const BnGrad bn{dy, x, (const uint8_t*)mask, sums, 1, mean, rstd, g, g, dgb, dgb + C};
  const BnBwdSums next{nullptr, nx, nmean, nrstd, nullptr, (const uint8_t*)nmask};
  const ConvFilterGrad fg{dw, in, ng, nb};
  PPLL_TRY(launch_conv_bn_bwd(s, bn, w, B, H, W, C, d, dres, (const uint8_t*)dmask, dst, &next, stat, stat_rows, filters ? &fg : nullptr, &rq));
  if (!filters) {
    if (!in) PPLL_TRY(launch_bn_apply(s, nx, BF16, B * H * W, C, nmean, nrstd, ng, nb, nullptr, y));
    PPLL_TRY(launch_conv3x3_wgrad(s, in ? in : y, d, BF16, B, H, W, C, C, 1, rq, dw));
  }
  return rq.flush(s);
}
