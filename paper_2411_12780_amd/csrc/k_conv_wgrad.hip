// Weight gradient of a 3x3 convolution (padding 1, stride 1 or 2) on the matrix cores, bf16 in, fp32 sums out, 16 / 32 / 48 /
// 64 input and 32 / 64 output channels or 16 -> 16.
//
// The reduction index of a 16x16x32 MFMA is the output pixel.  A tile is a stretch of output rows (whole images where they
// are small, a piece of a row where that is wide): its pixels of x, with the border the taps reach into, and of dy are laid in
// LDS as they are in memory, [pixel][channel], and the transposing LDS read forms fragments of 4 pixels x 16 channels from
// them.  Its 16 addresses are free, so any tap of any pixel is an address, whatever the row length and the stride: no pixel
// has to be aligned, shifted or masked.  A wave owns 16 input x 32 output channels for all nine taps (72 accumulators, which
// leaves room for two workgroups on a compute unit); where that takes fewer than eight waves, the others take other
// pixels, and the sums are folded in LDS in a fixed order.  One partial filter per workgroup; the ordered second-stage
// reduction adds them.  The next tile's loads are in flight while a tile is multiplied.
//
// Bound by memory at 16 channels (ten convolutions of 1024 x 32 x 32: 670 MB in 151 us), by the LDS reads of the fragments
// (11 KB for 18 products) at 64.  Images transposed to [channel][pixel] on their way into LDS instead, with products over 8
// consecutive pixels of a row, took 95 us where this takes 51 (nine of 848 x 8 x 8, 64 -> 64), and rows of 4 pixels needed a
// vector kernel, 58 us where this takes 13 (848 x 8 x 8, 64 -> 64, stride 2).
#include <algorithm>
#include "resnet_bf16.h"

namespace ppll {

namespace {
typedef __attribute__((ext_vector_type(4))) float wg_f32x4;

// up to 16 convolutions of one shape in a launch: blockIdx.y picks the convolution
constexpr int WGT_GROUP = 16;
struct WgtGroup { const uint16_t* x[WGT_GROUP]; const uint16_t* dy[WGT_GROUP]; float* partial[WGT_GROUP]; };
// A tile: seg images, or (seg = 1) sr rows x sc columns of one; chunks of rows and columns per image; rows and columns of x
// in LDS; pixels of the tile, and rounded up to 32
struct WgtShape { int B, H, W, Ho, Wo, seg, sr, sc, nrc, ncc, xr, xc, px, px32, tiles; };

// Floats from one partial filter to the next.  A filter is a multiple of 9 KB: without the 256 bytes more, the rows that a
// thread of the second stage adds up lie on a few memory channels.
constexpr int wgt_row(int Ci, int Co) { return 9 * Ci * Co + 64; }

template <int CIT, int COT, int S> struct Wgt {
  static constexpr int CI = 16 * CIT, CO = 16 * COT, COW = COT >= 2 ? 2 : 1, POS = CIT * (COT / COW);
  static constexpr int WAVES = 8 % POS == 0 ? 8 : 6, WK = WAVES / POS, TH = 64 * WAVES, NW = 9 * CI * CO;
  static constexpr int PER = CIT * COT == 16 ? 1 : 2;         // workgroups per compute unit
  // most pixels of a tile
  static constexpr int NPX = S == 1 ? (CIT * COT == 1 ? 512 : CIT * COT >= 8 && PER == 2 ? 128 : 256) : (CIT > 1 && PER == 2 ? 64 : 128);
  static constexpr int PX = 2 * CI + 16, PD = 2 * CO + 16;    // bytes from pixel to pixel in LDS: 4 pixels on different banks
  // 16-byte pieces of a tile per thread that are loaded ahead (what a wider border needs is loaded when it is stored)
  static constexpr int NIX_ = ((S == 1 ? NPX * 2 * CIT * 16 : NPX * 8 * CIT * 13) / 10 + TH - 1) / TH, MOST = PER == 2 ? 5 : 10, NIX = NIX_ < MOST ? NIX_ : MOST;
  static constexpr int NID = (NPX * 2 * COT + TH - 1) / TH;
  static size_t lds(const WgtShape& g) {
    const size_t tile = (size_t)g.seg * g.xr * g.xc * PX + (size_t)g.px32 * (PD + 8) + (size_t)g.seg * g.xr * g.xc * 4, fold = (size_t)(WK / 2) * NW * 4;
    return tile > fold ? tile : fold;
  }
};

template <int CIT, int COT, int S>
__global__ __launch_bounds__((Wgt<CIT, COT, S>::TH), (2 * Wgt<CIT, COT, S>::PER)) void conv3x3_wgrad_mfma_kernel(WgtGroup grp, WgtShape g) {
  using K = Wgt<CIT, COT, S>;
  constexpr int CI = K::CI, CO = K::CO, TH = K::TH, PX = K::PX, PD = K::PD, NIX = K::NIX, NID = K::NID, WK = K::WK, COW = K::COW;
  extern __shared__ __align__(16) char sm[];
  const uint16_t* __restrict__ x = grp.x[blockIdx.y];
  const uint16_t* __restrict__ dy = grp.dy[blockIdx.y];
  const int nx = g.seg * g.xr * g.xc, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, r = lane & 15, q = lane >> 4;
  const int pos = wave % K::POS, kq = wave / K::POS, ci0 = 16 * (pos % CIT), co0 = 16 * COW * (pos / CIT);
  char* xt = sm;
  char* dt = sm + (size_t)nx * PX;
  // tables: pixel of the tile -> byte offset of its first tap; pixel of x or dy -> image, row and column within the tile, ten
  // bits each (in LDS: kept in registers, they spill, and the reloads wait for the loads in flight)
  int* table = reinterpret_cast<int*>(dt + g.px32 * PD);
  int* dtab = table + g.px32;
  int* xtab = dtab + g.px32;
  for (int p = tid; p < g.px32; p += TH) {
    const int row = p / g.sc, lc = p - row * g.sc, sg = row / g.sr, lr = row - sg * g.sr;
    table[p] = p < g.px ? ((sg * g.xr + S * lr) * g.xc + S * lc) * PX : 0;
    dtab[p] = p < g.px ? sg << 20 | lr << 10 | lc : 1023 << 20;
  }
  for (int p = tid; p < nx; p += TH) {
    const int row = p / g.xc, sg = row / g.xr;
    xtab[p] = sg << 20 | (row - sg * g.xr) << 10 | (p - row * g.xc);
  }
  __syncthreads();
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  u32x4 rx[NIX], rd[NID];
  int b0 = 0, row0 = 0, col0 = 0, images = 0;
  auto place = [&](int tile) {
    const int ct = tile % g.ncc, rest = tile / g.ncc;
    b0 = rest / g.nrc * g.seg;
    row0 = rest % g.nrc * g.sr;
    col0 = ct * g.sc;
    images = min(g.seg, g.B - b0);
  };
  // 16-byte piece v of the tile's x or dy
  auto x_load = [&](__amdgpu_buffer_rsrc_t rs, int v) {
    const int at = xtab[min(v / (2 * CIT), nx - 1)], sg = at >> 20, yy = S * row0 + (at >> 10 & 1023) - 1, xx = S * col0 + (at & 1023) - 1;
    const bool in = sg < images && (unsigned)yy < (unsigned)g.H && (unsigned)xx < (unsigned)g.W;
    return __builtin_amdgcn_raw_buffer_load_b128(rs, in ? (((sg * g.H + yy) * g.W + xx) * CI + 8 * (v % (2 * CIT))) * 2 : CONV_OOB, 0, 0);
  };
  auto d_load = [&](__amdgpu_buffer_rsrc_t rs, int v) {
    const int at = dtab[min(v / (2 * COT), g.px32 - 1)], sg = at >> 20, oy = row0 + (at >> 10 & 1023), ox = col0 + (at & 1023);
    const bool in = sg < images && oy < g.Ho && ox < g.Wo;
    return __builtin_amdgcn_raw_buffer_load_b128(rs, in ? (((sg * g.Ho + oy) * g.Wo + ox) * CO + 8 * (v % (2 * COT))) * 2 : CONV_OOB, 0, 0);
  };
  auto x_rsrc = [&]() {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(x + (size_t)b0 * g.H * g.W * CI), 0, images * g.H * g.W * CI * 2, 0x00020000);
  };
  auto load = [&](int t) {
    const __amdgpu_buffer_rsrc_t rsx = x_rsrc();
    const __amdgpu_buffer_rsrc_t rsd = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(dy + (size_t)b0 * g.Ho * g.Wo * CO), 0, images * g.Ho * g.Wo * CO * 2, 0x00020000);
#pragma unroll
    for (int i = 0; i < NIX; ++i) rx[i] = x_load(rsx, t + i * TH);
#pragma unroll
    for (int i = 0; i < NID; ++i) rd[i] = d_load(rsd, t + i * TH);
  };
  wg_f32x4 acc[9][COW];
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int u = 0; u < COW; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[t][u][e] = 0.f;
  // this lane's part of a fragment: pixel (lane & 15) / 4 of four, channels 4 (lane & 3) .. + 3
  const char* xl = xt + 2 * (ci0 + 4 * (lane & 3));
  const char* dl = dt + 2 * (co0 + 4 * (lane & 3));
  const int pl = 8 * q + ((lane & 15) >> 2);
  const int rowb = g.xc * PX;
  place(blockIdx.x);
  load(tid);
  for (int tile = blockIdx.x; tile < g.tiles; tile += gridDim.x) {
    int t = tid;
    asm volatile("" : "+v"(t));      // addresses formed from it are not kept in registers over the products
#pragma unroll
    for (int i = 0; i < NIX; ++i) {
      const int v = t + i * TH;
      if (v < nx * 2 * CIT) *reinterpret_cast<u32x4*>(xt + v / (2 * CIT) * PX + 16 * (v % (2 * CIT))) = rx[i];
    }
    for (int v = t + NIX * TH; v < nx * 2 * CIT; v += TH)
      *reinterpret_cast<u32x4*>(xt + v / (2 * CIT) * PX + 16 * (v % (2 * CIT))) = x_load(x_rsrc(), v);
#pragma unroll
    for (int i = 0; i < NID; ++i) {
      const int v = t + i * TH;
      if (v < g.px32 * 2 * COT) *reinterpret_cast<u32x4*>(dt + v / (2 * COT) * PD + 16 * (v % (2 * COT))) = rd[i];
    }
    __syncthreads();
    if (tile + (int)gridDim.x < g.tiles) {
      place(tile + gridDim.x);
      load(t);
    }
    for (int ks = kq; ks < g.px32 / 32; ks += WK) {
      const int p = 32 * ks + pl;
      const char* x0 = xl + table[p];
      const char* x1 = xl + table[p + 4];
      bf16x8 df[COW];
#pragma unroll
      for (int u = 0; u < COW; ++u) {
        const uint2 lo = conv_lds_read_tr(dl + p * PD + 32 * u), hi = conv_lds_read_tr(dl + (p + 4) * PD + 32 * u);
        df[u] = __builtin_bit_cast(bf16x8, make_uint4(lo.x, lo.y, hi.x, hi.y));
      }
#pragma unroll
      for (int ky = 0; ky < 3; ++ky)
#pragma unroll
        for (int kx = 0; kx < 3; ++kx) {
          const uint2 lo = conv_lds_read_tr(x0 + ky * rowb + kx * PX), hi = conv_lds_read_tr(x1 + ky * rowb + kx * PX);
          const bf16x8 xf = __builtin_bit_cast(bf16x8, make_uint4(lo.x, lo.y, hi.x, hi.y));
#pragma unroll
          for (int u = 0; u < COW; ++u) acc[3 * ky + kx][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf, df[u], acc[3 * ky + kx][u], 0, 0, 0);
        }
    }
    __syncthreads();
  }
  // acc[tap][u][e] = dw[tap][ci0 + 4 q + e][co0 + 16 u + r] of this wave's pixels; the upper half of the waves that share
  // those hands its sums over, until one is left
  float* fold = reinterpret_cast<float*>(sm);
#pragma unroll
  for (int h = WK / 2; h >= 1; h /= 2) {
    if (kq >= h && kq < 2 * h)
#pragma unroll
      for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int u = 0; u < COW; ++u)
#pragma unroll
          for (int e = 0; e < 4; ++e) fold[(kq - h) * K::NW + (t * CI + ci0 + 4 * q + e) * CO + co0 + 16 * u + r] = acc[t][u][e];
    __syncthreads();
    if (kq < h)
#pragma unroll
      for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int u = 0; u < COW; ++u)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[t][u][e] += fold[kq * K::NW + (t * CI + ci0 + 4 * q + e) * CO + co0 + 16 * u + r];
    __syncthreads();
  }
  if (kq == 0) {
    float* out = grp.partial[blockIdx.y] + (size_t)blockIdx.x * wgt_row(CI, CO);
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
      for (int u = 0; u < COW; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) out[(t * CI + ci0 + 4 * q + e) * CO + co0 + 16 * u + r] = acc[t][u][e];
  }
}

// The largest tile of up to NPX pixels whose LDS lets two workgroups share a compute unit.
constexpr size_t WGT_LDS = 160 * 1024;
template <class K>
WgtShape wgt_shape(int B, int H, int W, int stride) {
  WgtShape g{};
  g.B = B; g.H = H; g.W = W; g.Ho = (H - 1) / stride + 1; g.Wo = (W - 1) / stride + 1;
  for (int px = K::NPX;; px = px * 3 / 4) {
    g.ncc = (g.Wo + px - 1) / px;
    g.sc = (g.Wo + g.ncc - 1) / g.ncc;
    const int rows = px / g.sc;
    if (g.ncc == 1 && rows >= g.Ho) {
      g.sr = g.Ho;
      g.seg = rows / g.Ho < B ? rows / g.Ho : B;
    } else {
      g.sr = rows < g.Ho ? rows : g.Ho;
      g.seg = 1;
    }
    g.nrc = (g.Ho + g.sr - 1) / g.sr;
    g.sr = (g.Ho + g.nrc - 1) / g.nrc;
    g.xr = stride * (g.sr - 1) + 3; g.xc = stride * (g.sc - 1) + 3;
    g.px = g.seg * g.sr * g.sc; g.px32 = (g.px + 31) / 32 * 32;
    const size_t tile = (size_t)g.seg * g.xr * g.xc * K::PX + (size_t)g.px32 * (K::PD + 8) + (size_t)g.seg * g.xr * g.xc * 4;
    if (tile <= WGT_LDS / K::PER || px <= 1) break;
  }
  g.tiles = (B + g.seg - 1) / g.seg * g.nrc * g.ncc;
  return g;
}
// Workgroups per convolution: the n of a launch share one round of the places on the device.  A partial filter is written and
// read once more (8 bytes a weight at about 4 bytes a picosecond), a tile takes a workgroup about 3 us: in r rounds of tiles,
// 3 us x r + 2 ps x workgroups x n x weights.
int wgt_blocks(const WgtShape& g, int per, int weights, int n) {
  const int cus = compute_units(), units = cus > 0 ? cus : 256, places = std::max(1, per * units / n);
  int best = 1;
  double least = 1e30;
  for (int r = (g.tiles + places - 1) / places; 3.0 * r < least; ++r) {
    const int b = (g.tiles + r - 1) / r;
    const double us = 3.0 * r + 2e-6 * b * n * weights;
    if (us < least) { least = us; best = b; }
  }
  return best;
}
// what one shape needs: `run` with n = 0 only reports the workgroups of a launch of `of` convolutions
template <int CIT, int COT, int S>
int wgt_run(hipStream_t s, const WgtGroup* grp, int n, int of, int B, int H, int W, int* blocks) {
  using K = Wgt<CIT, COT, S>;
  const WgtShape g = wgt_shape<K>(B, H, W, S);
  *blocks = wgt_blocks(g, K::PER, K::NW, of);
  if (!n) return PPLL_OK;
  const size_t lds = K::lds(g);
  static OncePerDevice once;
  PPLL_TRY(raise_lds((const void*)conv3x3_wgrad_mfma_kernel<CIT, COT, S>, (int)WGT_LDS, once));
  hipLaunchKernelGGL((conv3x3_wgrad_mfma_kernel<CIT, COT, S>), dim3(*blocks, n), dim3(K::TH), lds, s, *grp, g);
  PPLL_HIP(hipGetLastError());
  return PPLL_OK;
}
template <int S>
int wgt_stride(hipStream_t s, const WgtGroup* grp, int n, int of, int B, int H, int W, int Ci, int Co, int* blocks) {
  if (Co == 16) return wgt_run<1, 1, S>(s, grp, n, of, B, H, W, blocks);
  if (Co == 32) {
    if (Ci == 16) return wgt_run<1, 2, S>(s, grp, n, of, B, H, W, blocks);
    if (Ci == 32) return wgt_run<2, 2, S>(s, grp, n, of, B, H, W, blocks);
    if (Ci == 48) return wgt_run<3, 2, S>(s, grp, n, of, B, H, W, blocks);
    return wgt_run<4, 2, S>(s, grp, n, of, B, H, W, blocks);
  }
  if (Ci == 16) return wgt_run<1, 4, S>(s, grp, n, of, B, H, W, blocks);
  if (Ci == 32) return wgt_run<2, 4, S>(s, grp, n, of, B, H, W, blocks);
  if (Ci == 48) return wgt_run<3, 4, S>(s, grp, n, of, B, H, W, blocks);
  return wgt_run<4, 4, S>(s, grp, n, of, B, H, W, blocks);
}
int wgt_dispatch(hipStream_t s, const WgtGroup* grp, int n, int of, int B, int H, int W, int Ci, int Co, int stride, int* blocks) {
  return stride == 1 ? wgt_stride<1>(s, grp, n, of, B, H, W, Ci, Co, blocks) : wgt_stride<2>(s, grp, n, of, B, H, W, Ci, Co, blocks);
}
}  // namespace

bool conv_wgrad_bf16_ok(int H, int W, int Ci, int Co, int stride) {
  if ((stride != 1 && stride != 2) || (long)H * W * 64 * 2 >= (1L << 30)) return false;   // byte offsets of an image in 32 bits
  if (Co == 16) return Ci == 16;
  return (Co == 32 || Co == 64) && Ci % 16 == 0 && Ci >= 16 && Ci <= 64;
}

// the most there can be: one convolution in a launch
size_t conv3x3_wgrad_bf16_partial_floats(int B, int H, int W, int Ci, int Co, int stride) {
  if (!conv_wgrad_bf16_ok(H, W, Ci, Co, stride)) return 0;
  int blocks = 0;
  wgt_dispatch(nullptr, nullptr, 0, 1, B, H, W, Ci, Co, stride, &blocks);
  return (size_t)blocks * wgt_row(Ci, Co);
}

int launch_conv3x3_wgrad_bf16(hipStream_t s, const void* x, const void* dy, int B, int H, int W, int Ci, int Co,
                              int stride, ReduceQueue& rq, float* dw, int ci_keep) {
  bool queued;
  int blocks = 0;
  PPLL_TRY(wgt_dispatch(s, nullptr, 0, 1, B, H, W, Ci, Co, stride, &blocks));
  WgtGroup g{};
  g.x[0] = (const uint16_t*)x; g.dy[0] = (const uint16_t*)dy; g.partial[0] = rq.space((size_t)blocks * wgt_row(Ci, Co), &queued);
  PPLL_TRY(wgt_dispatch(s, &g, 1, 1, B, H, W, Ci, Co, stride, &blocks));
  return reduce_conv_filters(s, rq, queued, g.partial[0], blocks, wgt_row(Ci, Co), Ci, Co, ci_keep, dw);
}

// Weight gradients of n convolutions of one shape in as few launches as possible (16 per launch).  Returns
// PPLL_OK with *done = false, having launched nothing, when the queue has no private room left for all partial sums
// (the caller then launches them one by one).
int launch_conv3x3_wgrad_group_bf16(hipStream_t s, const ConvWgradJob* jobs, int n, int B, int H, int W, int Ci, int Co,
                                    int stride, ReduceQueue& rq, bool* done) {
  *done = false;
  const int of = n < WGT_GROUP ? n : WGT_GROUP;
  int blocks = 0;
  PPLL_TRY(wgt_dispatch(s, nullptr, 0, of, B, H, W, Ci, Co, stride, &blocks));
  const int nw = wgt_row(Ci, Co);
  const size_t need = ((size_t)blocks * nw + 63) & ~(size_t)63;
  if (!rq.arena || rq.used + need * n > rq.arena_floats) return PPLL_OK;
  for (int j0 = 0; j0 < n; j0 += WGT_GROUP) {
    const int m = n - j0 < WGT_GROUP ? n - j0 : WGT_GROUP;
    WgtGroup g{};
    for (int j = 0; j < m; ++j) {
      bool queued;
      g.x[j] = (const uint16_t*)jobs[j0 + j].x; g.dy[j] = (const uint16_t*)jobs[j0 + j].dy;
      g.partial[j] = rq.space((size_t)blocks * nw, &queued);     // queued: room was checked above
    }
    PPLL_TRY(wgt_dispatch(s, &g, m, of, B, H, W, Ci, Co, stride, &blocks));
    for (int j = 0; j < m; ++j) PPLL_TRY(reduce_conv_filters(s, rq, true, g.partial[j], blocks, nw, Ci, Co, Ci, jobs[j0 + j].dw));
  }
  *done = true;
  return PPLL_OK;
}

}  // namespace ppll
