// Main loop of the bf16 matrix-core products: C tile += A(m, k) B(k, n) over a range of k, fp32 accumulation in
// v_mfma_f32_32x32x16_bf16, operands copied from memory straight into LDS (buffer loads with an LDS destination).
#pragma once
#include "common.h"
#include "plan.h"

namespace ppll {
namespace pipe {

typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

constexpr int OOB = 0x7fffffff;        // no buffer here reaches 2^30 bytes (checked on the host)
constexpr int OOB_BASE = 0x40000000;   // a base offset that stays out of range after anything below 2^30 is added
constexpr int KS = 32;                 // k of a stage

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* ptr, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(ptr), 0, (int)bytes, 0x00020000);
}
typedef __attribute__((address_space(3))) char lds_char;
__device__ __forceinline__ void load_to_lds(__amdgpu_buffer_rsrc_t r, lds_char* dst, int voff, int soff = 0) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, dst, 16, voff, soff, 0, 0);
}

template <int N> __device__ __forceinline__ void wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
// A workgroup barrier without the waits of __syncthreads: a wave has waited for its copies itself, its reads are over where split_stage
// and k_step end.  The builtin promises nothing about memory, so the compiler is told that no access moves across it: the epilogues
// write with ordinary stores to stages that other waves have just read.
__device__ __forceinline__ void barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Helpers: workgroups beyond those that have tiles, on units that have none.  Each brings a share of what its XCD's tiles read into the L2
// there, rows of A and columns of B k by k ahead of them, then what the epilogue takes, a word of every cache line (the words go to LDS that
// nothing reads, as in CodeToL2).  Tiles of a row of them read the same rows at the same time, and a unit has about 25 GB/s of lines on
// their way from beyond L2: three tiles to a row get through A at 1.6 TB/s.
struct Bring {
  const void *A, *B, *side;            // side: [M][N], read by the epilogue, or null
  uint32_t a_bytes, b_bytes, s_bytes;
  int lda2, ldb2, lds2;                // bytes from row to row
  int M, N, K, bm, bn, helpers;        // helpers: of an XCD
};
template <bool BT, int THREADS> __device__ __forceinline__ void bring_operands(const Bring& p, const TileMap& t, int xcd, int helper, lds_char* to) {
  const TileRange x = tiles_of(t, xcd);
  if (x.m0 >= x.m1 || x.n0 >= x.n1) return;
  const int row0 = x.m0 * p.bm, rows = min(x.m1 * p.bm, p.M) - row0, col0 = x.n0 * p.bn, cols = min(x.n1 * p.bn, p.N) - col0;
  const int nl = (cols + 63) / 64, chunk = rows + (BT ? 64 * nl : cols), lines = chunk * ((p.K + 63) / 64);    // of 64 k, and in all
  const __amdgpu_buffer_rsrc_t rsA = make_rsrc(p.A, p.a_bytes), rsB = make_rsrc(p.B, p.b_bytes), rsS = make_rsrc(p.side, p.s_bytes);
  const int lane = threadIdx.x & 63, first = helper * THREADS + (int)(threadIdx.x & ~63), step = p.helpers * THREADS;
  for (int i0 = first; i0 < lines; i0 += step) {
    const int i = i0 + lane, c = i / chunk, r = i - c * chunk, q = r - rows;
    const int k = BT ? c * 64 + q / nl : 0;
    const int offB = BT ? k < p.K ? k * p.ldb2 + col0 * 2 + q % nl * 128 : OOB : (col0 + q) * p.ldb2 + c * 128;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsA, to, 4, i < lines && q < 0 ? (row0 + r) * p.lda2 + c * 128 : OOB, 0, 0, 0);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsB, to, 4, i < lines && q >= 0 ? offB : OOB, 0, 0, 0);
    wait_vm<2>();      // not so far ahead that L2 has lost it again (4160 x 768 x 3072: 26.8 us without this, 25.4)
  }
  if (p.side)
    for (int i0 = first; i0 < rows * nl; i0 += step) {
      const int i = i0 + lane, r = i / nl;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsS, to, 4, r < rows ? (row0 + r) * p.lds2 + col0 * 2 + (i - r * nl) * 128 : OOB, 0, 0, 0);
    }
  wait_vm<0>();
}

// One operand: ROWS rows (m or n) x KS k per stage.
//  TR = false: k contiguous in memory.  LDS [row][32 k], 64 bytes a row; the 16-byte granule g of row r sits at
//    g ^ ((r / 4) % 4): 16 lanes reading one granule of 16 rows hit every bank once.  (64 k a stage: 128 bytes a row, a whole cache
//    line, g at g ^ ((r / 2) % 8).)
//  TR = true: row index contiguous.  LDS [32 k][ROWS] as in memory; the 64-byte window w of k row k sits at w ^ (k % 4):
//    the transposing read (16 lanes hand in 4 k rows x 32 bytes) of 8 k rows then spreads over all banks.
// A copy instruction of a wave fills 1 KB of LDS in lane order, so the permutations are applied to the addresses that the
// lanes fetch from; they stay inside one row segment, i.e. inside one cache line.
template <bool TR, int ROWS, int KT = KS> struct Operand {
  static_assert((!TR || ROWS == 128 || ROWS == 256) && (KT == 32 || KT == 64), "");
  static constexpr int BYTES = ROWS * KT * 2;
  static constexpr int COPIES = BYTES / 1024;            // wave instructions per stage
  static constexpr int PITCH = TR ? ROWS * 2 : KT * 2;
  static constexpr int STEP_ROWS = 1024 / PITCH;         // k rows (rows) per copy instruction
  int vbase;      // byte offset this lane fetches from at k = 0, copy 0
  int gk;         // TR = false: first k (within the stage) of the lane's granule
  int ld2;        // bytes between rows (TR: between k rows)
  // wave: the k rows of a wave's copies differ from those of its first by a multiple of 4 (an even number of waves of 2 rows,
  // or 4 rows a copy), so the window permutation is the same in all of them
  __device__ __forceinline__ void init(long ld, int row0, int nrows, int lane, int wave) {
    ld2 = (int)(ld * 2);
    if (TR) {
      constexpr int SL = PITCH / 16;                     // 16-byte slots of a k row
      const int kr = lane / SL, slot = lane % SL, win = (slot >> 2) ^ ((kr + STEP_ROWS * wave) & 3);   // STEP_ROWS is 2 or 4
      const int col = row0 + (win * 4 + (slot & 3)) * 8;
      vbase = col < nrows ? kr * ld2 + col * 2 : OOB_BASE;
      gk = kr;
    } else {                                             // rows past the last one lie past the end of the buffer
      const int g = KT == 32 ? (lane & 3) ^ ((lane >> 4) & 3) : (lane & 7) ^ ((lane >> 4) + 4 * (wave & 1));
      gk = g * 8;
      vbase = (row0 + lane / (PITCH / 16)) * ld2 + g * 16;
    }
  }
};

// A workgroup of WGM_ x WGN_ waves, each 32 IM_ x 64 of the output tile, and NS_ stages in LDS.  Four stages of 64 k: as many waves again
// that do nothing but copy.
template <bool AT, bool BT, int WGM_, int WGN_, int IM_, int NS_, int KT_ = KS> struct Shape {
  static constexpr int KT = KT_, WGN = WGN_, IM = IM_, NS = NS_, W = WGM_ * WGN_, BM = WGM_ * IM * 32, BN = WGN_ * 64;
  static constexpr bool COPY_WAVES = KT == 64 && NS == 4;
  static constexpr int THREADS = 64 * W * (COPY_WAVES ? 2 : 1);
  using OA = Operand<AT, BM, KT>;
  using OB = Operand<BT, BN, KT>;
  static constexpr int STAGE = OA::BYTES + OB::BYTES, LDS = NS * STAGE;
  static constexpr int COPIES = OA::COPIES / W + OB::COPIES / W;   // per wave and stage, of some waves one more
  static_assert(OB::COPIES % W == 0 && (!AT || OA::COPIES % W == 0) && W % 2 == 0 && (KT == 32 ? NS >= 3 : (NS == 2 && W == 8) || COPY_WAVES), "");
};

// The fragments (8 consecutive k of one row per lane) of a wave's tile, 32 IM rows of A and 64 of B, at one k step of 16.  A
// transposing read gives half of one.
template <bool TR, int N> struct Frags {
  u32x4 v[N];
  __device__ __forceinline__ u32x4 get(int i) const { return v[i]; }
};
template <int N> struct Frags<true, N> {
  u32x2 lo[N], hi[N];
  __device__ __forceinline__ u32x4 get(int i) const { return (u32x4){lo[i].x, lo[i].y, hi[i].x, hi[i].y}; }
};
template <int N> __device__ __forceinline__ void set_zero(Frags<false, N>& f, int i) { f.v[i] = (u32x4){0, 0, 0, 0}; }
template <int N> __device__ __forceinline__ void set_zero(Frags<true, N>& f, int i) { f.lo[i] = f.hi[i] = (u32x2){0, 0}; }
// Lane address of MFMA tile 0 of a wave (rows row0 .. row0 + 31, row0 a multiple of 32 x tiles of the wave), k step 0, stage 0
template <bool TR, int ROWS, int KT = KS> __device__ __forceinline__ int frag_base(int region, int row0, int lane) {
  if (TR) {
    const int kr = 8 * (lane >> 5) + ((lane & 15) >> 2);
    return region + kr * (ROWS * 2) + (((row0 >> 5) ^ (kr & 3)) << 6) + (16 * ((lane >> 4) & 1) + 4 * (lane & 3)) * 2;
  }
  const int r = lane & 31;
  if (KT == 64) return region + (row0 + r) * 128 + (((lane >> 5) ^ ((r >> 1) & 7)) << 4);
  return region + (row0 + r) * 64 + (((lane >> 5) ^ ((r >> 2) & 3)) << 4);
}

// One k step of a wave: the products of the fragments at hand, and under them the reads of the next fragments (k step KK
// of the stage that addrA, addrB point into), which have arrived when the block ends.  It is one assembly block because the
// compiler would order LDS reads that it knows of behind all outstanding copies into LDS; the wait is inside, so every output
// is there when the compiler thinks it is.  The s_nop covers a register of the products written by a vector instruction before.
#define PPLL_MMA(J, I) "v_mfma_f32_32x32x16_bf16 %[c" #J #I "], %[q" #J "], %[p" #I "], %[c" #J #I "]\n"
#define PPLL_ACC [c00] "+v"(acc[0][0]), [c01] "+v"(acc[0][1]), [c02] "+v"(acc[0][2]), [c03] "+v"(acc[0][3]), \
                 [c10] "+v"(acc[1][0]), [c11] "+v"(acc[1][1]), [c12] "+v"(acc[1][2]), [c13] "+v"(acc[1][3])
#define PPLL_CUR [p0] "v"(a.get(0)), [p1] "v"(a.get(1)), [p2] "v"(a.get(2)), [p3] "v"(a.get(3)), [q0] "v"(b.get(0)), [q1] "v"(b.get(1))
#define PPLL_ROWS [r1] "n"(R32), [r2] "n"(2 * R32), [r3] "n"(3 * R32), [r4] "n"(4 * R32)
template <bool AT, bool BT, int ROWS_A, int ROWS_B, int KK, int IM, int KT = KS>
__device__ __forceinline__ void k_step(f32x16 (&acc)[2][IM], const Frags<AT, IM>& a, const Frags<BT, 2>& b, Frags<AT, IM>& na, Frags<BT, 2>& nb,
                                       int addrA, int addrB) {
  static_assert(IM == 4 || (IM == 5 && !AT), "");
  constexpr int PA = ROWS_A * 2, PB = ROWS_B * 2, R32 = 64 * KT;     // bytes of 32 rows with k contiguous
  if constexpr (IM == 5 && BT) {
    asm volatile("s_nop 1\n" PPLL_MMA(0, 0)
                 "ds_read_b64_tr_b16 %[l0], %[rb0] offset:%[ol]\n ds_read_b64_tr_b16 %[h0], %[rb0] offset:%[oh]\n" PPLL_MMA(0, 1)
                 "ds_read_b128 %[x0], %[ra]\n ds_read_b128 %[x1], %[ra] offset:%[r1]\n" PPLL_MMA(0, 2)
                 "ds_read_b128 %[x2], %[ra] offset:%[r2]\n ds_read_b128 %[x3], %[ra] offset:%[r3]\n" PPLL_MMA(0, 3)
                 "ds_read_b128 %[x4], %[ra] offset:%[r4]\n ds_read_b64_tr_b16 %[l1], %[rb1] offset:%[ol]\n" PPLL_MMA(0, 4)
                 "ds_read_b64_tr_b16 %[h1], %[rb1] offset:%[oh]\n"
                 PPLL_MMA(1, 0) PPLL_MMA(1, 1) PPLL_MMA(1, 2) PPLL_MMA(1, 3) PPLL_MMA(1, 4) "s_waitcnt lgkmcnt(0)"
                 : PPLL_ACC, [c04] "+v"(acc[0][4]), [c14] "+v"(acc[1][4]), [x0] "=&v"(na.v[0]), [x1] "=&v"(na.v[1]), [x2] "=&v"(na.v[2]),
                   [x3] "=&v"(na.v[3]), [x4] "=&v"(na.v[4]), [l0] "=&v"(nb.lo[0]), [h0] "=&v"(nb.hi[0]), [l1] "=&v"(nb.lo[1]), [h1] "=&v"(nb.hi[1])
                 : PPLL_CUR, [p4] "v"(a.get(4)), [ra] "v"(KK ? addrA ^ (32 * KK) : addrA), [rb0] "v"(addrB), [rb1] "v"(addrB ^ 64),
                   [ol] "n"(KK * 16 * PB), [oh] "n"(KK * 16 * PB + 4 * PB), PPLL_ROWS
                 : "memory");
  } else if constexpr (IM == 5) {
    asm volatile("s_nop 1\n" PPLL_MMA(0, 0) "ds_read_b128 %[y0], %[rb]\n ds_read_b128 %[x0], %[ra]\n" PPLL_MMA(0, 1)
                 "ds_read_b128 %[x1], %[ra] offset:%[r1]\n ds_read_b128 %[x2], %[ra] offset:%[r2]\n" PPLL_MMA(0, 2)
                 "ds_read_b128 %[x3], %[ra] offset:%[r3]\n ds_read_b128 %[x4], %[ra] offset:%[r4]\n" PPLL_MMA(0, 3)
                 "ds_read_b128 %[y1], %[rb] offset:%[r1]\n" PPLL_MMA(0, 4)
                 PPLL_MMA(1, 0) PPLL_MMA(1, 1) PPLL_MMA(1, 2) PPLL_MMA(1, 3) PPLL_MMA(1, 4) "s_waitcnt lgkmcnt(0)"
                 : PPLL_ACC, [c04] "+v"(acc[0][4]), [c14] "+v"(acc[1][4]), [x0] "=&v"(na.v[0]), [x1] "=&v"(na.v[1]), [x2] "=&v"(na.v[2]),
                   [x3] "=&v"(na.v[3]), [x4] "=&v"(na.v[4]), [y0] "=&v"(nb.v[0]), [y1] "=&v"(nb.v[1])
                 : PPLL_CUR, [p4] "v"(a.get(4)), [ra] "v"(KK ? addrA ^ (32 * KK) : addrA), [rb] "v"(KK ? addrB ^ (32 * KK) : addrB), PPLL_ROWS
                 : "memory");
  } else if constexpr (!AT && BT) {
    asm volatile("s_nop 1\n" PPLL_MMA(0, 0)
                 "ds_read_b64_tr_b16 %[l0], %[rb0] offset:%[ol]\n ds_read_b64_tr_b16 %[h0], %[rb0] offset:%[oh]\n" PPLL_MMA(0, 1)
                 "ds_read_b128 %[x0], %[ra]\n ds_read_b128 %[x1], %[ra] offset:%[r1]\n" PPLL_MMA(0, 2)
                 "ds_read_b128 %[x2], %[ra] offset:%[r2]\n ds_read_b128 %[x3], %[ra] offset:%[r3]\n" PPLL_MMA(0, 3)
                 "ds_read_b64_tr_b16 %[l1], %[rb1] offset:%[ol]\n ds_read_b64_tr_b16 %[h1], %[rb1] offset:%[oh]\n"
                 PPLL_MMA(1, 0) PPLL_MMA(1, 1) PPLL_MMA(1, 2) PPLL_MMA(1, 3) "s_waitcnt lgkmcnt(0)"
                 : PPLL_ACC, [x0] "=&v"(na.v[0]), [x1] "=&v"(na.v[1]), [x2] "=&v"(na.v[2]), [x3] "=&v"(na.v[3]),
                   [l0] "=&v"(nb.lo[0]), [h0] "=&v"(nb.hi[0]), [l1] "=&v"(nb.lo[1]), [h1] "=&v"(nb.hi[1])
                 : PPLL_CUR, [ra] "v"(KK ? addrA ^ (32 * KK) : addrA), [rb0] "v"(addrB), [rb1] "v"(addrB ^ 64), [ol] "n"(KK * 16 * PB),
                   [oh] "n"(KK * 16 * PB + 4 * PB), PPLL_ROWS
                 : "memory");
  } else if constexpr (!AT && !BT) {
    asm volatile("s_nop 1\n" PPLL_MMA(0, 0) "ds_read_b128 %[y0], %[rb]\n ds_read_b128 %[x0], %[ra]\n" PPLL_MMA(0, 1)
                 "ds_read_b128 %[x1], %[ra] offset:%[r1]\n ds_read_b128 %[x2], %[ra] offset:%[r2]\n" PPLL_MMA(0, 2)
                 "ds_read_b128 %[x3], %[ra] offset:%[r3]\n ds_read_b128 %[y1], %[rb] offset:%[r1]\n" PPLL_MMA(0, 3)
                 PPLL_MMA(1, 0) PPLL_MMA(1, 1) PPLL_MMA(1, 2) PPLL_MMA(1, 3) "s_waitcnt lgkmcnt(0)"
                 : PPLL_ACC, [x0] "=&v"(na.v[0]), [x1] "=&v"(na.v[1]), [x2] "=&v"(na.v[2]), [x3] "=&v"(na.v[3]), [y0] "=&v"(nb.v[0]),
                   [y1] "=&v"(nb.v[1])
                 : PPLL_CUR, [ra] "v"(KK ? addrA ^ (32 * KK) : addrA), [rb] "v"(KK ? addrB ^ (32 * KK) : addrB), PPLL_ROWS
                 : "memory");
  } else {
    static_assert(AT && BT, "");
    asm volatile("s_nop 1\n" PPLL_MMA(0, 0)
                 "ds_read_b64_tr_b16 %[m0], %[rb0] offset:%[ol]\n ds_read_b64_tr_b16 %[n0], %[rb0] offset:%[oh]\n"
                 "ds_read_b64_tr_b16 %[l0], %[ra0] offset:%[al]\n ds_read_b64_tr_b16 %[h0], %[ra0] offset:%[ah]\n" PPLL_MMA(0, 1)
                 "ds_read_b64_tr_b16 %[l1], %[ra1] offset:%[al]\n ds_read_b64_tr_b16 %[h1], %[ra1] offset:%[ah]\n"
                 "ds_read_b64_tr_b16 %[l2], %[ra2] offset:%[al]\n ds_read_b64_tr_b16 %[h2], %[ra2] offset:%[ah]\n" PPLL_MMA(0, 2)
                 "ds_read_b64_tr_b16 %[l3], %[ra3] offset:%[al]\n ds_read_b64_tr_b16 %[h3], %[ra3] offset:%[ah]\n" PPLL_MMA(0, 3)
                 "ds_read_b64_tr_b16 %[m1], %[rb1] offset:%[ol]\n ds_read_b64_tr_b16 %[n1], %[rb1] offset:%[oh]\n"
                 PPLL_MMA(1, 0) PPLL_MMA(1, 1) PPLL_MMA(1, 2) PPLL_MMA(1, 3) "s_waitcnt lgkmcnt(0)"
                 : PPLL_ACC, [l0] "=&v"(na.lo[0]), [h0] "=&v"(na.hi[0]), [l1] "=&v"(na.lo[1]), [h1] "=&v"(na.hi[1]),
                   [l2] "=&v"(na.lo[2]), [h2] "=&v"(na.hi[2]), [l3] "=&v"(na.lo[3]), [h3] "=&v"(na.hi[3]), [m0] "=&v"(nb.lo[0]),
                   [n0] "=&v"(nb.hi[0]), [m1] "=&v"(nb.lo[1]), [n1] "=&v"(nb.hi[1])
                 : PPLL_CUR, [ra0] "v"(addrA), [ra1] "v"(addrA ^ 64), [ra2] "v"(addrA ^ 128), [ra3] "v"(addrA ^ 192), [rb0] "v"(addrB),
                   [rb1] "v"(addrB ^ 64), [al] "n"(KK * 16 * PA), [ah] "n"(KK * 16 * PA + 4 * PA), [ol] "n"(KK * 16 * PB),
                   [oh] "n"(KK * 16 * PB + 4 * PB)
                 : "memory");
  }
}
#undef PPLL_MMA
#undef PPLL_ACC
#undef PPLL_CUR
#undef PPLL_ROWS

// The four k steps of a stage of 64 k in a wave that has 64 x 64 of a 128 x 128 tile, in order, and under them the reads of all
// fragments of the next stage, which are there when the block ends.  (Read a k step ahead instead, 4 products do not cover the reads'
// way: a stage of 8320 x 384 x 1536 took 0.49 us, 0.38 in one block.)
template <bool BT> struct StageFrags {
  Frags<false, 8> a;      // fragment 2 kk + i: k step kk, 32-row tile i
  Frags<BT, 8> b;
};
template <bool BT>
__device__ __forceinline__ void stage_step(f32x16 (&acc)[2][2], const StageFrags<BT>& f, StageFrags<BT>& n, int addrA, int addrB) {
  if constexpr (BT) {
    asm volatile("ds_read_b128 %[x0], %[ra0]\n ds_read_b128 %[x1], %[ra0] offset:4096\n ds_read_b64_tr_b16 %[l0], %[rb0] offset:0\n "
                 "v_mfma_f32_32x32x16_bf16 %[c00], %[q0], %[p0], %[c00]\n ds_read_b64_tr_b16 %[h0], %[rb0] offset:1024\n "
                 "ds_read_b64_tr_b16 %[l1], %[rb1] offset:0\n ds_read_b64_tr_b16 %[h1], %[rb1] offset:1024\n "
                 "v_mfma_f32_32x32x16_bf16 %[c01], %[q0], %[p1], %[c01]\n ds_read_b128 %[x2], %[ra1]\n "
                 "ds_read_b128 %[x3], %[ra1] offset:4096\n ds_read_b64_tr_b16 %[l2], %[rb0] offset:4096\n "
                 "v_mfma_f32_32x32x16_bf16 %[c10], %[q1], %[p0], %[c10]\n ds_read_b64_tr_b16 %[h2], %[rb0] offset:5120\n "
                 "ds_read_b64_tr_b16 %[l3], %[rb1] offset:4096\n ds_read_b64_tr_b16 %[h3], %[rb1] offset:5120\n "
                 "v_mfma_f32_32x32x16_bf16 %[c11], %[q1], %[p1], %[c11]\n ds_read_b128 %[x4], %[ra2]\n "
                 "ds_read_b128 %[x5], %[ra2] offset:4096\n ds_read_b64_tr_b16 %[l4], %[rb0] offset:8192\n "
                 "v_mfma_f32_32x32x16_bf16 %[c00], %[q2], %[p2], %[c00]\n ds_read_b64_tr_b16 %[h4], %[rb0] offset:9216\n "
                 "ds_read_b64_tr_b16 %[l5], %[rb1] offset:8192\n ds_read_b64_tr_b16 %[h5], %[rb1] offset:9216\n "
                 "v_mfma_f32_32x32x16_bf16 %[c01], %[q2], %[p3], %[c01]\n ds_read_b128 %[x6], %[ra3]\n "
                 "ds_read_b128 %[x7], %[ra3] offset:4096\n ds_read_b64_tr_b16 %[l6], %[rb0] offset:12288\n "
                 "v_mfma_f32_32x32x16_bf16 %[c10], %[q3], %[p2], %[c10]\n ds_read_b64_tr_b16 %[h6], %[rb0] offset:13312\n "
                 "ds_read_b64_tr_b16 %[l7], %[rb1] offset:12288\n ds_read_b64_tr_b16 %[h7], %[rb1] offset:13312\n "
                 "v_mfma_f32_32x32x16_bf16 %[c11], %[q3], %[p3], %[c11]\n v_mfma_f32_32x32x16_bf16 %[c00], %[q4], %[p4], %[c00]\n "
                 "v_mfma_f32_32x32x16_bf16 %[c01], %[q4], %[p5], %[c01]\n v_mfma_f32_32x32x16_bf16 %[c10], %[q5], %[p4], %[c10]\n "
                 "v_mfma_f32_32x32x16_bf16 %[c11], %[q5], %[p5], %[c11]\n v_mfma_f32_32x32x16_bf16 %[c00], %[q6], %[p6], %[c00]\n "
                 "v_mfma_f32_32x32x16_bf16 %[c01], %[q6], %[p7], %[c01]\n v_mfma_f32_32x32x16_bf16 %[c10], %[q7], %[p6], %[c10]\n "
                 "v_mfma_f32_32x32x16_bf16 %[c11], %[q7], %[p7], %[c11]\n s_waitcnt lgkmcnt(0)"
                 : [c00] "+v"(acc[0][0]), [c01] "+v"(acc[0][1]), [c10] "+v"(acc[1][0]), [c11] "+v"(acc[1][1]), [x0] "=&v"(n.a.v[0]),
                   [x1] "=&v"(n.a.v[1]), [x2] "=&v"(n.a.v[2]), [x3] "=&v"(n.a.v[3]), [x4] "=&v"(n.a.v[4]), [x5] "=&v"(n.a.v[5]),
                   [x6] "=&v"(n.a.v[6]), [x7] "=&v"(n.a.v[7]), [l0] "=&v"(n.b.lo[0]), [h0] "=&v"(n.b.hi[0]),
                   [l1] "=&v"(n.b.lo[1]), [h1] "=&v"(n.b.hi[1]), [l2] "=&v"(n.b.lo[2]), [h2] "=&v"(n.b.hi[2]),
                   [l3] "=&v"(n.b.lo[3]), [h3] "=&v"(n.b.hi[3]), [l4] "=&v"(n.b.lo[4]), [h4] "=&v"(n.b.hi[4]),
                   [l5] "=&v"(n.b.lo[5]), [h5] "=&v"(n.b.hi[5]), [l6] "=&v"(n.b.lo[6]), [h6] "=&v"(n.b.hi[6]),
                   [l7] "=&v"(n.b.lo[7]), [h7] "=&v"(n.b.hi[7])
                 : [p0] "v"(f.a.get(0)), [q0] "v"(f.b.get(0)), [p1] "v"(f.a.get(1)), [q1] "v"(f.b.get(1)),
                   [p2] "v"(f.a.get(2)), [q2] "v"(f.b.get(2)), [p3] "v"(f.a.get(3)), [q3] "v"(f.b.get(3)),
                   [p4] "v"(f.a.get(4)), [q4] "v"(f.b.get(4)), [p5] "v"(f.a.get(5)), [q5] "v"(f.b.get(5)),
                   [p6] "v"(f.a.get(6)), [q6] "v"(f.b.get(6)), [p7] "v"(f.a.get(7)), [q7] "v"(f.b.get(7)), [ra0] "v"(addrA),
                   [ra1] "v"(addrA ^ 32), [ra2] "v"(addrA ^ 64), [ra3] "v"(addrA ^ 96), [rb0] "v"(addrB), [rb1] "v"(addrB ^ 64)
                 : "memory");
  } else {
    asm volatile("ds_read_b128 %[x0], %[ra0]\n ds_read_b128 %[x1], %[ra0] offset:4096\n "
                 "v_mfma_f32_32x32x16_bf16 %[c00], %[q0], %[p0], %[c00]\n ds_read_b128 %[y0], %[rb0]\n "
                 "ds_read_b128 %[y1], %[rb0] offset:4096\n v_mfma_f32_32x32x16_bf16 %[c01], %[q0], %[p1], %[c01]\n "
                 "ds_read_b128 %[x2], %[ra1]\n ds_read_b128 %[x3], %[ra1] offset:4096\n "
                 "v_mfma_f32_32x32x16_bf16 %[c10], %[q1], %[p0], %[c10]\n ds_read_b128 %[y2], %[rb1]\n "
                 "ds_read_b128 %[y3], %[rb1] offset:4096\n v_mfma_f32_32x32x16_bf16 %[c11], %[q1], %[p1], %[c11]\n "
                 "ds_read_b128 %[x4], %[ra2]\n ds_read_b128 %[x5], %[ra2] offset:4096\n "
                 "v_mfma_f32_32x32x16_bf16 %[c00], %[q2], %[p2], %[c00]\n ds_read_b128 %[y4], %[rb2]\n "
                 "ds_read_b128 %[y5], %[rb2] offset:4096\n v_mfma_f32_32x32x16_bf16 %[c01], %[q2], %[p3], %[c01]\n "
                 "ds_read_b128 %[x6], %[ra3]\n ds_read_b128 %[x7], %[ra3] offset:4096\n "
                 "v_mfma_f32_32x32x16_bf16 %[c10], %[q3], %[p2], %[c10]\n ds_read_b128 %[y6], %[rb3]\n "
                 "ds_read_b128 %[y7], %[rb3] offset:4096\n v_mfma_f32_32x32x16_bf16 %[c11], %[q3], %[p3], %[c11]\n "
                 "v_mfma_f32_32x32x16_bf16 %[c00], %[q4], %[p4], %[c00]\n v_mfma_f32_32x32x16_bf16 %[c01], %[q4], %[p5], %[c01]\n "
                 "v_mfma_f32_32x32x16_bf16 %[c10], %[q5], %[p4], %[c10]\n v_mfma_f32_32x32x16_bf16 %[c11], %[q5], %[p5], %[c11]\n "
                 "v_mfma_f32_32x32x16_bf16 %[c00], %[q6], %[p6], %[c00]\n v_mfma_f32_32x32x16_bf16 %[c01], %[q6], %[p7], %[c01]\n "
                 "v_mfma_f32_32x32x16_bf16 %[c10], %[q7], %[p6], %[c10]\n v_mfma_f32_32x32x16_bf16 %[c11], %[q7], %[p7], %[c11]\n "
                 "s_waitcnt lgkmcnt(0)"
                 : [c00] "+v"(acc[0][0]), [c01] "+v"(acc[0][1]), [c10] "+v"(acc[1][0]), [c11] "+v"(acc[1][1]), [x0] "=&v"(n.a.v[0]),
                   [x1] "=&v"(n.a.v[1]), [x2] "=&v"(n.a.v[2]), [x3] "=&v"(n.a.v[3]), [x4] "=&v"(n.a.v[4]), [x5] "=&v"(n.a.v[5]),
                   [x6] "=&v"(n.a.v[6]), [x7] "=&v"(n.a.v[7]), [y0] "=&v"(n.b.v[0]), [y1] "=&v"(n.b.v[1]), [y2] "=&v"(n.b.v[2]),
                   [y3] "=&v"(n.b.v[3]), [y4] "=&v"(n.b.v[4]), [y5] "=&v"(n.b.v[5]), [y6] "=&v"(n.b.v[6]), [y7] "=&v"(n.b.v[7])
                 : [p0] "v"(f.a.get(0)), [q0] "v"(f.b.get(0)), [p1] "v"(f.a.get(1)), [q1] "v"(f.b.get(1)),
                   [p2] "v"(f.a.get(2)), [q2] "v"(f.b.get(2)), [p3] "v"(f.a.get(3)), [q3] "v"(f.b.get(3)),
                   [p4] "v"(f.a.get(4)), [q4] "v"(f.b.get(4)), [p5] "v"(f.a.get(5)), [q5] "v"(f.b.get(5)),
                   [p6] "v"(f.a.get(6)), [q6] "v"(f.b.get(6)), [p7] "v"(f.a.get(7)), [q7] "v"(f.b.get(7)), [ra0] "v"(addrA),
                   [ra1] "v"(addrA ^ 32), [ra2] "v"(addrA ^ 64), [ra3] "v"(addrA ^ 96), [rb0] "v"(addrB), [rb1] "v"(addrB ^ 32),
                   [rb2] "v"(addrB ^ 64), [rb3] "v"(addrB ^ 96)
                 : "memory");
  }
}

// acc[jn][im] (of a wave that multiplies): C^T tiles (the B fragment goes first into the MFMA): lane l holds row im*32 + l%32, columns jn*32 + 8 q +
// 4 (l/32) + e in element 4 q + e.  csum[jn] (COLSUM, wave-uniform do_colsum): this lane's share, k % 8 = e of its half of every
// k step in element e, of the sum over k of B's row jn*32 + l%32.
template <class S, bool AT, bool BT, bool COLSUM>
__device__ __forceinline__ void multiply(const __amdgpu_buffer_rsrc_t rsA, const __amdgpu_buffer_rsrc_t rsB, long lda, long ldb,
                                         int m0, int n0, int M, int N, int K, lds_char* lds, f32x16 (&acc)[2][S::IM],
                                         float (&csum)[2][8], bool do_colsum) {
  constexpr int NS = S::NS, IM = S::IM, KT = S::KT;
  const int nk = (K + KT - 1) / KT;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) % S::W;
  const int wm = wave / S::WGN, wn = wave % S::WGN;
  using OA = typename S::OA;
  using OB = typename S::OB;
  OA oa;
  OB ob;
  oa.init(lda, m0, M, lane, wave);
  ob.init(ldb, n0, N, lane, wave);
  auto issue = [&](int i) {       // copies of stage i (all zeros past the last one)
    const int k0 = i * KT;
    const bool live = i < nk;
    lds_char* st = lds + (i % NS) * S::STAGE;
    int va, vb;                   // k rows past the last one of an operand stored by k lie past the end of its buffer
    if (AT) va = live ? oa.vbase + k0 * oa.ld2 : OOB_BASE;
    else va = live && k0 + oa.gk < K ? oa.vbase + k0 * 2 : OOB_BASE;
    if (BT) vb = live ? ob.vbase + k0 * ob.ld2 : OOB_BASE;
    else vb = live && k0 + ob.gk < K ? ob.vbase + k0 * 2 : OOB_BASE;
#pragma unroll
    for (int c = 0; c < (OA::COPIES + S::W - 1) / S::W; ++c) {
      const int q = c * S::W + wave;
      if (c < OA::COPIES / S::W || q < OA::COPIES) load_to_lds(rsA, st + q * 1024, va + q * OA::STEP_ROWS * oa.ld2);
    }
#pragma unroll
    for (int c = 0; c < OB::COPIES / S::W; ++c) {
      const int q = c * S::W + wave;
      load_to_lds(rsB, st + OA::BYTES + q * 1024, vb + q * OB::STEP_ROWS * ob.ld2);
    }
  };
  const int base = (int)(uintptr_t)lds;
  const int fa0 = frag_base<AT, S::BM, KT>(base, wm * IM * 32, lane), fb0 = frag_base<BT, S::BN, KT>(base + OA::BYTES, wn * 64, lane);
  Frags<AT, IM> a0, a1;
  Frags<BT, 2> b0, b1;
  auto column_sums = [&](const Frags<BT, 2>& b) {
    if (!COLSUM || !do_colsum) return;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const u32x4 v = b.get(j);
#pragma unroll
      for (int e = 0; e < 4; ++e) { csum[j][2 * e] += __uint_as_float(v[e] << 16); csum[j][2 * e + 1] += __uint_as_float(v[e] & 0xffff0000u); }
    }
  };
  if constexpr (KT == 32) {
#pragma unroll
    for (int i = 0; i < NS - 1; ++i) issue(i);
    wait_vm<(NS - 2) * S::COPIES>();
    barrier();
    // the first fragments: products with zeros under the reads (the accumulators stay zero)
#pragma unroll
    for (int i = 0; i < IM; ++i) set_zero(a1, i);
#pragma unroll
    for (int j = 0; j < 2; ++j) set_zero(b1, j);
    k_step<AT, BT, S::BM, S::BN, 0, IM>(acc, a1, b1, a0, b0, fa0, fb0);
    for (int i = 0; i < nk; ++i) {
      const int st = (i % NS) * S::STAGE, nx = ((i + 1) % NS) * S::STAGE;
      wait_vm<(NS - 3) * S::COPIES>();       // this wave's part of stage i + 1 is in LDS
      barrier();          // and everyone's; nobody reads stage i - 1 any more
      issue(i + NS - 1);
      column_sums(b0);
      k_step<AT, BT, S::BM, S::BN, 1, IM>(acc, a0, b0, a1, b1, fa0 + st, fb0 + st);
      column_sums(b1);
      k_step<AT, BT, S::BM, S::BN, 0, IM>(acc, a1, b1, a0, b0, fa0 + nx, fb0 + nx);
    }
  } else if constexpr (S::COPY_WAVES) {
    // All fragments of a stage are in registers before it is multiplied, so its place in LDS is filled again meanwhile: NS - 1 stages are on
    // their way.  Issuing 32 copies takes a unit about as long as a stage's products take (0.35 us and 0.29, each without the other), and a
    // wave that does both waits for them in turn (0.45): so four waves copy and four multiply (0.37).
    static_assert(!AT && IM == 2 && S::BM == 128 && S::BN == 128, "");
    if (tid >= 64 * S::W) {
      for (int i = 0; i < NS; ++i) issue(i);
      wait_vm<(NS - 1) * S::COPIES>();
      barrier();
      for (int i = 0; i < nk; ++i) {
        wait_vm<(NS - 2) * S::COPIES>();     // this wave's part of stage i + 1 is in LDS
        barrier();                           // and everyone's; nobody reads stage i any more
        issue(i + NS);
      }
      wait_vm<0>();
      barrier();
      return;
    }
    StageFrags<BT> f0, f1;
#pragma unroll
    for (int i = 0; i < 8; ++i) { set_zero(f1.a, i); set_zero(f1.b, i); }
    barrier();
    stage_step<BT>(acc, f1, f0, fa0, fb0);   // the first fragments: products with zeros under the reads
    int st = 0;
    auto next = [&] {
      barrier();
      st = st + S::STAGE == NS * S::STAGE ? 0 : st + S::STAGE;
    };
    for (int i = 0; i < nk; i += 2) {
      next();
      stage_step<BT>(acc, f0, f1, fa0 + st, fb0 + st);
      if (i + 1 >= nk) break;
      next();
      stage_step<BT>(acc, f1, f0, fa0 + st, fb0 + st);
    }
  } else {
    // two stages of 64 k: one is filled from the moment that everyone has read it until the same point a stage later
    issue(0);
    issue(1);
    wait_vm<S::COPIES>();
    barrier();
#pragma unroll
    for (int i = 0; i < IM; ++i) set_zero(a1, i);
#pragma unroll
    for (int j = 0; j < 2; ++j) set_zero(b1, j);
    k_step<AT, BT, S::BM, S::BN, 0, IM, KT>(acc, a1, b1, a0, b0, fa0, fb0);
    for (int i = 0; i < nk; ++i) {
      const int st = (i & 1) * S::STAGE, nx = S::STAGE - st;
      k_step<AT, BT, S::BM, S::BN, 1, IM, KT>(acc, a0, b0, a1, b1, fa0 + st, fb0 + st);
      k_step<AT, BT, S::BM, S::BN, 2, IM, KT>(acc, a1, b1, a0, b0, fa0 + st, fb0 + st);
      k_step<AT, BT, S::BM, S::BN, 3, IM, KT>(acc, a0, b0, a1, b1, fa0 + st, fb0 + st);
      wait_vm<0>();         // this wave's part of stage i + 1 is in LDS
      barrier();            // and everyone's; nobody reads stage i any more
      issue(i + 2);
      k_step<AT, BT, S::BM, S::BN, 0, IM, KT>(acc, a1, b1, a0, b0, fa0 + nx, fb0 + nx);
    }
  }
  // the last products are through before a vector instruction reads the accumulators
  asm volatile("s_nop 15\n s_nop 3" ::: "memory");
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int i = 0; i < IM; ++i) asm volatile("" : "+v"(acc[j][i]));
  wait_vm<0>();
  barrier();            // the stages are free for the epilogue
}

}  // namespace pipe
}  // namespace ppll
