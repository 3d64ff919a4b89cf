// Main loop of the bf16 matrix-core products: C tile += A(m, k) B(k, n) over a range of k, fp32 accumulation in
// v_mfma_f32_32x32x16_bf16, operands copied from memory straight into LDS (buffer loads with an LDS destination).
#pragma once
#include "common.h"

namespace ppll {
namespace pipe {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
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
__device__ __forceinline__ void load_to_lds(__amdgpu_buffer_rsrc_t r, lds_char* dst, int voff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, dst, 16, voff, 0, 0, 0);
}

// Fragment reads are inline assembly: the compiler would order every LDS read it knows of behind all outstanding copies into
// LDS.  Their results count as ready at once for the compiler, so every use sits behind a wait that names the registers.
template <int OFF> __device__ __forceinline__ void lds_read16(u32x4& d, int addr) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(d) : "v"(addr), "n"(OFF));
}
template <int OFF> __device__ __forceinline__ void lds_read_tr(u32x2& d, int addr) {
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(d) : "v"(addr), "n"(OFF));
}
template <int N> __device__ __forceinline__ void wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// One operand: ROWS rows (m or n) x KS k per stage.
//  TR = false: k contiguous in memory.  LDS [row][32 k], 64 bytes a row; the 16-byte granule g of row r sits at
//    g ^ ((r / 4) % 4): 16 lanes reading one granule of 16 rows hit every bank once.
//  TR = true: row index contiguous.  LDS [32 k][ROWS] as in memory; the 64-byte window w of k row k sits at w ^ (k % 4):
//    the transposing read (16 lanes hand in 4 k rows x 32 bytes) of 8 k rows then spreads over all banks.
// A copy instruction of a wave fills 1 KB of LDS in lane order, so the permutations are applied to the addresses that the
// lanes fetch from; they stay inside one row segment, i.e. inside one cache line.
template <bool TR, int ROWS> struct Operand {
  static_assert(!TR || ROWS == 128 || ROWS == 256, "");
  static constexpr int BYTES = ROWS * KS * 2;
  static constexpr int COPIES = BYTES / 1024;            // wave instructions per stage
  static constexpr int PITCH = TR ? ROWS * 2 : 64;
  static constexpr int STEP_ROWS = TR ? 1024 / PITCH : 16;   // k rows (rows) per copy instruction
  int vbase;      // byte offset this lane fetches from at k = 0, copy 0
  int gk;         // TR = false: first k (within the stage) of the lane's granule
  int ld2;        // bytes between rows (TR: between k rows)
  __device__ __forceinline__ void init(long ld, int row0, int nrows, int lane) {
    ld2 = (int)(ld * 2);
    if (TR) {
      constexpr int SL = PITCH / 16;                     // 16-byte slots of a k row
      const int kr = lane / SL, slot = lane % SL, win = (slot >> 2) ^ (kr & 3);   // STEP_ROWS is 2 or 4
      const int col = row0 + (win * 4 + (slot & 3)) * 8;
      vbase = col < nrows ? kr * ld2 + col * 2 : OOB_BASE;
      gk = kr;
    } else {
      const int g = (lane & 3) ^ ((lane >> 4) & 3);
      gk = g * 8;
      vbase = (row0 + (lane >> 2)) * ld2 + g * 16;       // rows past the last one lie past the end of the buffer
    }
  }
};

template <bool AT, bool BT, int WGM, int WGN, int IM, int JN, int NS> struct Shape {
  static constexpr int W = WGM * WGN, THREADS = 64 * W, BM = WGM * IM * 32, BN = WGN * JN * 32;
  using OA = Operand<AT, BM>;
  using OB = Operand<BT, BN>;
  static constexpr int STAGE = OA::BYTES + OB::BYTES, LDS = NS * STAGE;
  static constexpr int COPIES = (OA::COPIES + OB::COPIES) / W;   // per wave and stage
  static_assert((OA::COPIES + OB::COPIES) % W == 0, "");
};


// 8 consecutive k of one row per lane (an MFMA operand)
template <bool TR> struct Frag;
template <> struct Frag<false> {
  u32x4 v;
  __device__ __forceinline__ void tie() { asm volatile("" : "+v"(v)); }
  __device__ __forceinline__ bf16x8 get() const { return __builtin_bit_cast(bf16x8, v); }
};
template <> struct Frag<true> {
  u32x2 lo, hi;   // put together only behind the wait
  __device__ __forceinline__ void tie() { asm volatile("" : "+v"(lo), "+v"(hi)); }
  __device__ __forceinline__ bf16x8 get() const { return __builtin_bit_cast(bf16x8, (u32x4){lo.x, lo.y, hi.x, hi.y}); }
};
// Lane address of MFMA tile 0 of a wave (rows row0 .. row0 + 31, row0 a multiple of 32 x tiles of the wave), k step 0, stage 0
template <bool TR, int ROWS> __device__ __forceinline__ int frag_base(int region, int row0, int lane) {
  if (TR) {
    const int kr = 8 * (lane >> 5) + ((lane & 15) >> 2);
    return region + kr * (ROWS * 2) + (((row0 >> 5) ^ (kr & 3)) << 6) + (16 * ((lane >> 4) & 1) + 4 * (lane & 3)) * 2;
  }
  const int r = lane & 31;
  return region + (row0 + r) * 64 + (((lane >> 5) ^ ((r >> 2) & 3)) << 4);
}
// fragments of N tiles, 32 rows apart, at k step KK (16 k) of a stage; addr = frag_base + stage offset
template <bool TR, int ROWS, int N, int KK, int I = 0> __device__ __forceinline__ void read_frags(Frag<TR> (&f)[N], int addr) {
  if constexpr (I < N) {
    if constexpr (TR) {
      constexpr int P = ROWS * 2;
      const int a = addr ^ (I << 6);
      lds_read_tr<KK * 16 * P>(f[I].lo, a);
      lds_read_tr<KK * 16 * P + 4 * P>(f[I].hi, a);
    } else {
      lds_read16<I * 2048>(f[I].v, KK ? addr ^ 32 : addr);
    }
    read_frags<TR, ROWS, N, KK, I + 1>(f, addr);
  }
}
template <int N> __device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N < 15 ? N : 15) : "memory"); }

// What one call multiplies: k from k_beg (a multiple of KS) on, nk stages, k >= k_end reads as zero (k_end beyond the operand
// when its k index is the outer one: the buffer ends there).
struct Range { int k_beg, nk, k_end; };

// acc[jn][im]: C^T tiles (the B fragment goes first into the MFMA): lane l holds row im*32 + l%32, columns jn*32 + 8 q +
// 4 (l/32) + e in element 4 q + e.  csum (COLSUM): per-lane sums over k of B's rows, in the same layout.
template <class S, bool AT, bool BT, int WGM, int WGN, int IM, int JN, int NS, bool COLSUM>
__device__ __forceinline__ void multiply(const __amdgpu_buffer_rsrc_t rsA, const __amdgpu_buffer_rsrc_t rsB, long lda, long ldb,
                                         int m0, int n0, int M, int N, const Range rg, lds_char* lds, f32x16 (&acc)[JN][IM],
                                         f32x16 (&csum)[JN], bool do_colsum) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  using OA = typename S::OA;
  using OB = typename S::OB;
  OA oa;
  OB ob;
  oa.init(lda, m0, M, lane);
  ob.init(ldb, n0, N, lane);
  auto issue = [&](int i) {       // copies of stage i (all zeros past the last one)
    const int k0 = rg.k_beg + i * KS;
    const bool live = i < rg.nk;
    lds_char* st = lds + (i % NS) * S::STAGE;
    int va, vb;
    if (AT) va = live ? oa.vbase + k0 * oa.ld2 : OOB_BASE;
    else va = live && k0 + oa.gk < rg.k_end ? oa.vbase + k0 * 2 : OOB_BASE;
    if (BT) vb = live ? ob.vbase + k0 * ob.ld2 : OOB_BASE;
    else vb = live && k0 + ob.gk < rg.k_end ? ob.vbase + k0 * 2 : OOB_BASE;
#pragma unroll
    for (int c = 0; c < OA::COPIES / S::W; ++c) {
      const int q = c * S::W + wave;
      load_to_lds(rsA, st + q * 1024, va + q * OA::STEP_ROWS * oa.ld2);
    }
#pragma unroll
    for (int c = 0; c < OB::COPIES / S::W; ++c) {
      const int q = c * S::W + wave;
      load_to_lds(rsB, st + OA::BYTES + q * 1024, vb + q * OB::STEP_ROWS * ob.ld2);
    }
  };
  const int base = (int)(uintptr_t)lds;
  const int fa0 = frag_base<AT, S::BM>(base, wm * IM * 32, lane), fb0 = frag_base<BT, S::BN>(base + OA::BYTES, wn * JN * 32, lane);
  Frag<AT> a0[IM], a1[IM];
  Frag<BT> b0[JN], b1[JN];
  constexpr int READS = IM * (AT ? 2 : 1) + JN * (BT ? 2 : 1);
  const bf16x8 ones = {(__bf16)1.f, (__bf16)1.f, (__bf16)1.f, (__bf16)1.f, (__bf16)1.f, (__bf16)1.f, (__bf16)1.f, (__bf16)1.f};
  auto mma = [&](Frag<AT> (&a)[IM], Frag<BT> (&b)[JN]) {
#pragma unroll
    for (int i = 0; i < IM; ++i) a[i].tie();
#pragma unroll
    for (int j = 0; j < JN; ++j) b[j].tie();
#pragma unroll
    for (int j = 0; j < JN; ++j) {
      const bf16x8 fb = b[j].get();
#pragma unroll
      for (int i = 0; i < IM; ++i) acc[j][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb, a[i].get(), acc[j][i], 0, 0, 0);
      if (COLSUM && do_colsum) csum[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb, ones, csum[j], 0, 0, 0);
    }
  };
#pragma unroll
  for (int i = 0; i < NS - 1; ++i) issue(i);
  wait_vm<(NS - 2) * S::COPIES>();
  __builtin_amdgcn_s_barrier();
  read_frags<AT, S::BM, IM, 0>(a0, fa0);
  read_frags<BT, S::BN, JN, 0>(b0, fb0);
  for (int i = 0; i < rg.nk; ++i) {
    const int st = (i % NS) * S::STAGE, nx = ((i + 1) % NS) * S::STAGE;
    wait_vm<(NS - 3) * S::COPIES>();       // this wave's part of stage i + 1 is in LDS
    __builtin_amdgcn_s_barrier();          // and everyone's; nobody reads stage i - 1 any more
    issue(i + NS - 1);
    read_frags<AT, S::BM, IM, 1>(a1, fa0 + st);
    read_frags<BT, S::BN, JN, 1>(b1, fb0 + st);
    wait_lds<READS>();
    mma(a0, b0);
    __builtin_amdgcn_sched_barrier(0);
    read_frags<AT, S::BM, IM, 0>(a0, fa0 + nx);
    read_frags<BT, S::BN, JN, 0>(b0, fb0 + nx);
    wait_lds<READS>();
    mma(a1, b1);
    __builtin_amdgcn_sched_barrier(0);
  }
  wait_lds<0>();
#pragma unroll
  for (int i = 0; i < IM; ++i) a0[i].tie();
#pragma unroll
  for (int j = 0; j < JN; ++j) b0[j].tie();
  wait_vm<0>();
  __builtin_amdgcn_s_barrier();            // the stages are free for the epilogue
}

}  // namespace pipe
}  // namespace ppll
