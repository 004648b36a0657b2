// Real GEMM tile engine with FP32-level accuracy on the F16 matrix cores
// (v_mfma_f32_32x32x16_f16).
//
// Every operand value is split into two halves, x = hi + lo with hi = f16(x) and
// lo = f16(x - hi) (22 bits and a sign), and a product is hi hi + hi lo + lo hi summed in
// FP32.  The f16 matrix instruction adds 16 products per rounding of the accumulator, the
// FP32 one (v_mfma_f32_32x32x2_f32) two, so the split product is the more exact of the two:
// rel-L2 error against FP64 at K = 256 (normal x cosine values) 1.86e-7 against 2.86e-7,
// at 5.3 times the matrix rate (three products of 32 cycles for K = 16 against eight of
// 64).  Operands are scaled by powers of two, exactly, so that their halves stay in the
// f16 range (65504 down to 2^-14, 2^-24 for subnormal halves).
//
// Panel format of a split operand, in memory and in LDS: [k / 16][piece][row][8 halves]
// with pieces hi k 0-7, hi k 8-15, lo k 0-7, lo k 8-15.  A stage of LDS is a plain copy of
// the panel; 32 lanes read 32 consecutive 16-byte pieces (no bank conflicts, no padding)
// and each lane gets the eight consecutive k of its row that the instruction wants.
//
// A workgroup computes a BM x BN tile with BM/WM x BN/WN waves, each owning a WM x WN tile
// of 32 x 32 blocks.  Two LDS stages; the loaders return the staged data by value, so that
// it stays in registers.
//
// 32x32x16 lane layout (wave64): A operand lane l holds A[l%32][8(l/32) + 0..7], B operand
// lane l holds B[8(l/32) + 0..7][l%32]; accumulator register r of lane l holds
// C[8(r/4) + 4(l/32) + r%4][l%32].
#pragma once

#include <hip/hip_runtime.h>

namespace rw {

typedef _Float16 hg8 __attribute__((ext_vector_type(8)));
typedef _Float16 hg2 __attribute__((ext_vector_type(2)));
typedef float hg16 __attribute__((ext_vector_type(16)));

constexpr int kHgPieceBytes = 16;
// bytes of one operand row's share of a panel: 64 per 16 k
__host__ __device__ constexpr size_t hg_panel_bytes(size_t k, size_t rows) { return k * rows * 4; }

template <int BM_, int BN_, int BK_, int WM_, int WN_>
struct HgCfg {
  static constexpr int BM = BM_, BN = BN_, BK = BK_, WM = WM_, WN = WN_;
  static constexpr int WAVES_M = BM / WM, WAVES_N = BN / WN;
  static constexpr int NT = WAVES_M * WAVES_N * 64;
  static constexpr int TM = WM / 32, TN = WN / 32;
  static constexpr int KS = BK / 16;
  static constexpr int A_BYTES = KS * 4 * BM * kHgPieceBytes;
  static constexpr int B_BYTES = KS * 4 * BN * kHgPieceBytes;
  static constexpr int STAGE_BYTES = A_BYTES + B_BYTES;
  static constexpr int LDS_BYTES = 2 * STAGE_BYTES;
  static_assert(BM % WM == 0 && BN % WN == 0 && WM % 32 == 0 && WN % 32 == 0, "tile shape");
  static_assert(BK % 16 == 0, "k-steps of 16");
};

// hi and lo halves of two values, packed.  lo = f16(x - hi) is one mixed-precision fused
// multiply-add (hi * -1 + x, exact before its rounding); the factor is opaque so that it is
// not turned back into a subtraction between two conversions.
__device__ __forceinline__ void hg_split2(float a, float b, unsigned* hi, unsigned* lo) {
  float m1 = -1.f;
  asm("" : "+s"(m1));
  asm("" : "+v"(a));
  asm("" : "+v"(b));
  unsigned hb = __builtin_bit_cast(unsigned, hg2{(_Float16)a, (_Float16)b});
  asm("" : "+v"(hb));   // keeps the two conversions one packed instruction
  const hg2 h = __builtin_bit_cast(hg2, hb);
  const hg2 l = {(_Float16)__builtin_fmaf((float)h[0], m1, a), (_Float16)__builtin_fmaf((float)h[1], m1, b)};
  *hi = hb;
  *lo = __builtin_bit_cast(unsigned, l);
}

// LDS position of tile row r: the plain one.
struct HgPlainRows {
  static __device__ __forceinline__ int pos(int r) { return r; }
};

// Loader of an operand stored as a panel of ld rows: a stage is copied as it is.
template <class Cfg, int ROWS>
struct HgPanelLoader {
  using Rows = HgPlainRows;
  static constexpr int TOTAL = Cfg::KS * 4 * ROWS;
  static constexpr int PER_THREAD = (TOTAL + Cfg::NT - 1) / Cfg::NT;   // the last round may be partial
  const uint4* src;   // panel, already offset to the tile's first row
  int ld;
  struct Regs {
    uint4 v[PER_THREAD];
  };

  __device__ Regs load(int k0, int tid) const {
    Regs r;
#pragma unroll
    for (int i = 0; i < PER_THREAD; ++i) {
      const int idx = tid + i * Cfg::NT;
      if (TOTAL % Cfg::NT != 0 && idx >= TOTAL) break;
      r.v[i] = src[(size_t)(k0 / 4 + idx / ROWS) * ld + idx % ROWS];
    }
    return r;
  }
  __device__ void store(char* dst, int tid, const Regs& r) const {
#pragma unroll
    for (int i = 0; i < PER_THREAD; ++i) {
      const int idx = tid + i * Cfg::NT;
      if (TOTAL % Cfg::NT != 0 && idx >= TOTAL) break;
      reinterpret_cast<uint4*>(dst)[idx] = r.v[i];
    }
  }
};

template <class Cfg>
struct HgAcc {
  hg16 c[Cfg::TM][Cfg::TN];
  __device__ void zero() {
#pragma unroll
    for (int i = 0; i < Cfg::TM; ++i)
#pragma unroll
      for (int j = 0; j < Cfg::TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) c[i][j][r] = 0.f;
  }
};

template <class Cfg, class ARows, class BRows>
__device__ __forceinline__ void hg_stage_mma(HgAcc<Cfg>& acc, const char* a, const char* b, int wrow, int wcol,
                                             int lane) {
  const int h = lane >> 5, l32 = lane & 31;
  const hg8* ap = reinterpret_cast<const hg8*>(a) + wrow + ARows::pos(l32);
  const hg8* bp = reinterpret_cast<const hg8*>(b) + wcol + BRows::pos(l32);
#pragma unroll
  for (int u = 0; u < Cfg::KS; ++u) {
    hg8 ah[Cfg::TM], al[Cfg::TM], bh[Cfg::TN], bl[Cfg::TN];
#pragma unroll
    for (int i = 0; i < Cfg::TM; ++i) {
      ah[i] = ap[(4 * u + h) * Cfg::BM + 32 * i];
      al[i] = ap[(4 * u + 2 + h) * Cfg::BM + 32 * i];
    }
#pragma unroll
    for (int j = 0; j < Cfg::TN; ++j) {
      bh[j] = bp[(4 * u + h) * Cfg::BN + 32 * j];
      bl[j] = bp[(4 * u + 2 + h) * Cfg::BN + 32 * j];
    }
    // the small products first; each pass runs over all blocks, so that dependent MFMAs
    // are TM TN issues apart
#pragma unroll
    for (int i = 0; i < Cfg::TM; ++i)
#pragma unroll
      for (int j = 0; j < Cfg::TN; ++j)
        acc.c[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah[i], bl[j], acc.c[i][j], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < Cfg::TM; ++i)
#pragma unroll
      for (int j = 0; j < Cfg::TN; ++j)
        acc.c[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al[i], bh[j], acc.c[i][j], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < Cfg::TM; ++i)
#pragma unroll
      for (int j = 0; j < Cfg::TN; ++j)
        acc.c[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah[i], bh[j], acc.c[i][j], 0, 0, 0);
  }
}

// K loop over [k_begin, k_end) (multiples of BK, k_end > k_begin) whose first stage the
// caller has already loaded into registers (ra0, rb0).  Two stages of global loads are in
// flight: stage k+2 is requested while stage k is multiplied and stage k+1 (already in
// registers) is prepared and written to the other LDS buffer (one stage in flight left a
// wave waiting for it behind a third of its MFMAs: the pupil GEMM of 16 stacks 345 -> 323
// us).  The last stages are peeled, so that no branch surrounds the loads and stores.  The
// caller's barrier must separate an earlier use of the LDS from this call; on return every
// wave has left it.
template <class Cfg, class ALoader, class BLoader>
__device__ __forceinline__ void hg_mainloop_pre(HgAcc<Cfg>& acc, const ALoader& la, const BLoader& lb,
                                                const typename ALoader::Regs& ra0,
                                                const typename BLoader::Regs& rb0, int k_begin, int k_end,
                                                char* lds, int tid, int wrow, int wcol, int lane) {
  using AR = typename ALoader::Rows;
  using BR = typename BLoader::Rows;
  const int KT = (k_end - k_begin) / Cfg::BK;
  const int k1 = min(k_begin + Cfg::BK, k_end - Cfg::BK);
  auto ra1 = la.load(k1, tid);
  auto rb1 = lb.load(k1, tid);
  la.store(lds, tid, ra0);
  lb.store(lds + Cfg::A_BYTES, tid, rb0);
  __syncthreads();
#pragma unroll 2
  for (int kt = 0; kt < KT - 2; ++kt) {
    char* cur = lds + (kt & 1) * Cfg::STAGE_BYTES;
    char* nxt = lds + ((kt + 1) & 1) * Cfg::STAGE_BYTES;
    const auto ra2 = la.load(k_begin + (kt + 2) * Cfg::BK, tid);
    const auto rb2 = lb.load(k_begin + (kt + 2) * Cfg::BK, tid);
    __builtin_amdgcn_sched_barrier(0);
    hg_stage_mma<Cfg, AR, BR>(acc, cur, cur + Cfg::A_BYTES, wrow, wcol, lane);
    la.store(nxt, tid, ra1);
    lb.store(nxt + Cfg::A_BYTES, tid, rb1);
    __syncthreads();
    ra1 = ra2;
    rb1 = rb2;
  }
  if (KT > 1) {
    char* cur = lds + (KT & 1) * Cfg::STAGE_BYTES;
    char* nxt = lds + ((KT - 1) & 1) * Cfg::STAGE_BYTES;
    hg_stage_mma<Cfg, AR, BR>(acc, cur, cur + Cfg::A_BYTES, wrow, wcol, lane);
    la.store(nxt, tid, ra1);
    lb.store(nxt + Cfg::A_BYTES, tid, rb1);
    __syncthreads();
  }
  char* last = lds + ((KT - 1) & 1) * Cfg::STAGE_BYTES;
  hg_stage_mma<Cfg, AR, BR>(acc, last, last + Cfg::A_BYTES, wrow, wcol, lane);
  __syncthreads();
}

template <class Cfg, class ALoader, class BLoader>
__device__ __forceinline__ void hg_mainloop(HgAcc<Cfg>& acc, const ALoader& la, const BLoader& lb, int k_begin,
                                            int k_end, char* lds, int tid, int wrow, int wcol, int lane) {
  const auto ra = la.load(k_begin, tid);
  const auto rb = lb.load(k_begin, tid);
  hg_mainloop_pre<Cfg>(acc, la, lb, ra, rb, k_begin, k_end, lds, tid, wrow, wcol, lane);
}

// Sixteen consecutive k of one row as its four 16-byte pieces (hi 0-7, hi 8-15, lo 0-7, lo 8-15)
__device__ __forceinline__ void hg_split16(const float* v, uint4 out[4]) {
  unsigned h[8], l[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) hg_split2(v[2 * i], v[2 * i + 1], &h[i], &l[i]);
  out[0] = make_uint4(h[0], h[1], h[2], h[3]);
  out[1] = make_uint4(h[4], h[5], h[6], h[7]);
  out[2] = make_uint4(l[0], l[1], l[2], l[3]);
  out[3] = make_uint4(l[4], l[5], l[6], l[7]);
}

// Workgroup ids are dealt round-robin over the 8 XCDs of the chip; renumber them
// so that consecutive logical ids run on the same XCD (and share its L2).
__device__ __forceinline__ int xcd_remap(int bid, int nblocks) {
  const int per = nblocks / 8;
  const int xcd = bid % 8, slot = bid / 8;
  if (slot >= per) return bid;   // the ragged last round keeps its id (ids >= 8 * per)
  return xcd * per + slot;
}

}  // namespace rw
