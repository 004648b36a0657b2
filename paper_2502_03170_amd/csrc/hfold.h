// Loader of the folded pupil for the split-f16 GEMMs: used by the plain Fourier form and by
// the batched emitters (both store folded pupils as [q = 2 jf + pj][kk = 2 lf + pl], complex).
#pragma once

#include "hgemm.h"
#include "rw_common.h"

namespace rw {

// A operand of the pupil GEMMs: the folded pupil with the defocus factor exp(i k s_z z)
// applied and split into f16 halves on the way into LDS.  Contraction index kk = 2 lf + pl;
// 32-row blocks hold 16 folded rows q = 2 jf + pj as rows 8 (q/4) + 4 ri + q%4 (ri = re / im),
// so that an accumulator lane holds 16 consecutive q of one part.  One thread takes a folded
// cell (jf, lf) with its four parities: its eight values share one defocus factor, whose
// phase is formed and reduced in FP64 (in revolutions) before the FP32 hardware sine and
// cosine.
// LDS position of a row within its 32-row block.  The row bits are (pj, jf0, ri, jf1, jf2);
// position (jf0, jf1 ^ pj, jf2 ^ ri, pj, ri) puts both the eight rows that a read phase
// covers (all pj, jf0, ri) and the eight that a write phase covers (all jf0, jf1, jf2) in
// distinct 16-byte columns of the banks.
struct HgFoldRows {
  static __device__ __forceinline__ int make(int pj, int ri, int j8) {
    return (j8 ^ (pj << 1) ^ (ri << 2)) | (pj << 3) | (ri << 4);
  }
  static __device__ __forceinline__ int pos(int r) {
    return make(r & 1, (r >> 2) & 1, ((r >> 1) & 1) | ((r >> 2) & 6));
  }
};

// PZ planes share a tile: its BM rows are PZ runs of BM / PZ rows of the same folded pupil
// rows, each with its own defocus, so that the pupil is read once for all of them.
template <class Cfg, int PZ>
struct FoldDefocusLoader {
  using Rows = HgFoldRows;
  static constexpr int JF = Cfg::BM / PZ / 4, CELLS = Cfg::BK / 2;
  static constexpr int TOTAL = JF * CELLS;
  static constexpr int PER_THREAD = (TOTAL + Cfg::NT - 1) / Cfg::NT;
  static_assert(JF % 8 == 0, "whole 32-row blocks per plane");
  const float2* Pf;    // [2 nhp][2 nhp] of this stack and component, from folded row jf0
  const double* kszf;  // [nhp][nhp], from row jf0
  double zrev[PZ];     // z / 2 pi, so that k s_z zrev is the phase in revolutions
  int w, nhp;          // w = 2 nhp
  struct Regs {
    float4 v[PER_THREAD][2];   // [pj]: (pl = 0, 1)
    double kz[PER_THREAD];
  };
  // folded row and cell of task idx: the four cells of a 16-byte piece side by side, then
  // eight folded rows, then the pieces, then the 32-row blocks
  static __device__ __forceinline__ void task(int idx, int* jl, int* lc) {
    *jl = ((idx >> 2) & 7) | (idx / (4 * Cfg::BK) << 3);
    *lc = (idx & 3) | (((idx >> 5) % (Cfg::BK / 8)) << 2);
  }

  __device__ Regs load(int k0, int tid) const {
    Regs r;
#pragma unroll
    for (int i = 0; i < PER_THREAD; ++i) {
      const int idx = tid + i * Cfg::NT;
      if (TOTAL % Cfg::NT != 0 && idx >= TOTAL) break;
      int jl, lc;
      task(idx, &jl, &lc);
      const float2* p = Pf + (size_t)(2 * jl) * w + k0 + 2 * lc;
      r.v[i][0] = *reinterpret_cast<const float4*>(p);
      r.v[i][1] = *reinterpret_cast<const float4*>(p + w);
      r.kz[i] = kszf[(size_t)jl * nhp + k0 / 2 + lc];
    }
    return r;
  }
  __device__ void store(char* dst, int tid, const Regs& r) const {
#pragma unroll
    for (int i = 0; i < PER_THREAD; ++i) {
      const int idx = tid + i * Cfg::NT;
      if (TOTAL % Cfg::NT != 0 && idx >= TOTAL) break;
      int jl, lc;
      task(idx, &jl, &lc);
      const int piece = 4 * (lc >> 3) + ((lc >> 2) & 1);
      char* d = dst + (size_t)(piece * Cfg::BM + 32 * (jl >> 3)) * 16 + 4 * (lc & 3);
#pragma unroll
      for (int z = 0; z < PZ; ++z) {
        float sn, cs;
        sincos_rev(r.kz[i] * zrev[z], &sn, &cs);
#pragma unroll
        for (int pj = 0; pj < 2; ++pj)
#pragma unroll
          for (int ri = 0; ri < 2; ++ri) {
            const float4 v = r.v[i][pj];
            const float x0 = ri ? v.x * sn + v.y * cs : v.x * cs - v.y * sn;
            const float x1 = ri ? v.z * sn + v.w * cs : v.z * cs - v.w * sn;
            unsigned hi, lo;
            hg_split2(x0, x1, &hi, &lo);
            char* o = d + (z * (Cfg::BM / PZ) + HgFoldRows::make(pj, ri, jl & 7)) * 16;
            *reinterpret_cast<unsigned*>(o) = hi;
            *reinterpret_cast<unsigned*>(o + 2 * Cfg::BM * 16) = lo;
          }
      }
    }
  }
};

}  // namespace rw
