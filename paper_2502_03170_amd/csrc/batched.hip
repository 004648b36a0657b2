// Batched emitters: the Fourier form (Sec. 3.3 eq. "cartesian vectorial" with the
// Sec. 3.4 correction factors) for thousands of emitters with individual sub-pixel
// position, axial position, Zernike vector (Sec. 3.4.2), crop size and plane count,
// in one persistent launch per tile class.
//
// Per emitter b the pupil phase is
//   Phi_b[j,l] = 2 pi sum_q c_bq Z_q(s) - k (s_x x0_b + s_y y0_b)
// a sum over 23 tables, basis = (2 pi Z_1..Z_21, s_x, s_y), which a thread keeps in registers
// for its pupil cells and applies to several emitters.  The cell-centred grids are
// mirror-symmetric, so each emitter's pupil is folded in the same pass (four parities per
// folded cell, written to the emitter's HBM slot) and each plane d of each field component c
// are two real-coefficient GEMMs on the matrix cores,
//   T  = (D o Pf_c) B1_S    (N x S; D = exp(i k s_z z) of each folded cell)
//   E' = A2_S T             (S x S, T kept in LDS),  E = -i E'
// and I = sum_c |E_c|^2.  A2_S / B1_S are the rows of one 96-row table that cover the
// crop (pixel i of an S-crop is table row i - S/2 + 32).  Crops are evaluated on 32- or
// 64-wide tiles, the two tile classes; the (emitter, plane) items of each class are dealt,
// emitter by emitter and longest first, to eight queues, one per XCD, and the class's
// persistent kernel takes items from the queues' atomic counters until they are exhausted.
#include <algorithm>
#include <cmath>
#include <complex>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <new>
#include <string>
#include <numeric>
#include <vector>

#include "hfold.h"
#include "rw_common.h"
#include "rw_fourier.h"
#include "rw_plan.h"

namespace rw {

constexpr int kTabRows = 96;    // DFT table rows: x_r = (r - 32) * pixel
constexpr int kBasisRows = 23;  // 21 Zernike + s_x + s_y
constexpr int kMaxWgPerCu = 4;  // workgroups per CU of the persistent launch (configuration bound)
constexpr int kTileClasses = 2;  // crops on 32- and on 64-row tiles
constexpr int kQueues = 8 * kTileClasses;   // one queue per XCD for each class

struct BatchParam {
  double zoff;      // -z_e
  double ts;        // emitter depth below the coverslip (Gibson-Lanni)
  long long off;    // voxel offset of the emitter's output
  int S, D, SP, pad;
};

struct BatchArgs {
  const BatchParam* params;  // [n] cost-sorted (slot order)
  const float2* Q;           // [3][N][N]
  const double* ksz;         // [N][N]
  const float* coef;         // [n][23] coefficients of the phase, slot order
  const float* basis;        // [23][N*N]
  const double4* gl;         // [N*N] Gibson-Lanni phase W = t_s (g1.x + i g1.y) + (g0.x + i g0.y) as
                             // (g0.x, g0.y, g1.x, g1.y), or null without the layer
  const uint4* tab;          // split-f16 panel of 96 rows r, k = 2f + p: 2^kTabExp cos / sin (k s[f] x_r)
  float tscale;              // power of two on T
  unsigned escale;           // packed powers of two: fields per unit of the image product
  float2* Pf;                // [n][3][N][N] folded pupils, slot order
  const int* list;           // [n] slots grouped by XCD queue
  const long long* pre;      // [n + 1] plane prefix sums over list
  const int* qoff;           // [17] queue q owns list[qoff[q] .. qoff[q+1]); queues 8 t + x of tile class t
  unsigned long long* counter;   // [16] next item of each queue
  float* I;
  float2* E;
  int n, N;
  int group;                 // emitters per workgroup of the fold kernel
  double pitch;
};

// Folded pupil of every emitter.  The pupil and pixel grids are mirror-symmetric
// (s[N-1-j] = -s[j]); with P = Q_c exp(i Phi) at the four mirror cells of (jf, lf),
//   Pf_{pj,pl}[jf][lf] = i^(pj+pl) sum_{a,b} (-1)^(a pj + b pl) P[mir_a(jf)][mir_b(lf)],
// stored at Pf[c][2jf + pj][2lf + pl].  A thread owns one folded cell: the 23 basis values and
// the base pupil of its four mirror cells stay in registers while it goes through `group`
// emitters, whose coefficients come over the scalar path.  The phase is reduced in FP64 and
// goes through sincospif, which has no path for large arguments (the hardware sine and cosine
// left the intensities at 1.5e-7 of their norm in place of 1.0e-7 and saved 20 us of 289).
// Bound by the writes (393 KB an emitter at N = 128).  4096 emitters: 289 us; the phases as a
// matrix product of their own (80 us), written and read back by a workgroup per emitter (531
// us), took 611.
// Workgroup 0 also sets each queue's counter to its first item (a kernel, not a memset, so
// that the launch sequence can be captured in a graph; one launch less than a kernel of its
// own).
__global__ void __launch_bounds__(256) batch_fold_kernel(BatchArgs a) {
  const int N = a.N, nh = N / 2;
  const size_t NN = (size_t)N * N;
  const int tid = threadIdx.x;
  if (blockIdx.x == 0 && tid < kQueues) a.counter[tid] = (unsigned long long)a.pre[a.qoff[tid]];
  const int cells = nh * nh / 256;   // whole workgroups at every pupil size
  const int cell = blockIdx.x % cells * 256 + tid;
  const int jf = cell / nh, lf = cell % nh, j1 = N - 1 - jf, l1 = N - 1 - lf;
  const int idx[4] = {jf * N + lf, jf * N + l1, j1 * N + lf, j1 * N + l1};
  float basis[4][kBasisRows];
  float2 Q[3][4];
  double4 g[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
#pragma unroll
    for (int k = 0; k < kBasisRows; ++k) basis[q][k] = a.basis[(size_t)k * NN + idx[q]];
#pragma unroll
    for (int c = 0; c < 3; ++c) Q[c][q] = a.Q[(size_t)c * NN + idx[q]];
    g[q] = a.gl ? a.gl[idx[q]] : make_double4(0.0, 0.0, 0.0, 0.0);
  }
  const int s0 = blockIdx.x / cells * a.group, s1 = min(s0 + a.group, a.n);
#pragma unroll 1
  for (int slot = s0; slot < s1; ++slot) {
    const float* cf = a.coef + (size_t)slot * kBasisRows;
    float phi[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < kBasisRows; ++k)
#pragma unroll
      for (int q = 0; q < 4; ++q) phi[q] = fmaf(cf[k], basis[q][k], phi[q]);
    float er[4], ei[4];
    if (a.gl) {
      // the layer's phase is formed in FP64 and joins phi before the reduction; its imaginary
      // part is the evanescent decay
      const double ts = a.params[slot].ts;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const double wr = ts * g[q].z + g[q].x, wi = ts * g[q].w + g[q].y;
        const float amp = (float)exp(-wi);
        float sn, cs;
        sincospif(half_turns(wr + (double)phi[q]), &sn, &cs);
        er[q] = amp * cs;
        ei[q] = amp * sn;
      }
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) sincospif(half_turns((double)phi[q]), &ei[q], &er[q]);
    }
    float2* Pf = a.Pf + (size_t)slot * 3 * NN;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      float pr[4], pi[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float2 v = Q[c][q];
        pr[q] = v.x * er[q] - v.y * ei[q];
        pi[q] = v.x * ei[q] + v.y * er[q];
      }
      float4* o = reinterpret_cast<float4*>(Pf + (size_t)c * NN + (size_t)(2 * jf) * N + 2 * lf);
      // (pj, pl) = (0,0): +,+,+,+   (0,1): i(+,-,+,-)   (1,0): i(+,+,-,-)   (1,1): -(+,-,-,+)
      o[0] = make_float4(pr[0] + pr[1] + pr[2] + pr[3], pi[0] + pi[1] + pi[2] + pi[3],
                         -(pi[0] - pi[1] + pi[2] - pi[3]), pr[0] - pr[1] + pr[2] - pr[3]);
      o[N / 2] = make_float4(-(pi[0] + pi[1] - pi[2] - pi[3]), pr[0] + pr[1] - pr[2] - pr[3],
                             -(pr[0] - pr[1] - pr[2] + pr[3]), -(pi[0] - pi[1] - pi[2] + pi[3]));
    }
  }
}

// Plane kernel.  Plane d of emitter `slot`, per field component c, with the operands split in
// f16 halves (hgemm.h):
//   T[q][n]  = sum_kk (D o Pf_c)[q][kk] B1[kk][n]     2N x SP, K = N: the defocused pupil staged
//              as in the plain form (D = exp(i k s_z z) of each folded cell, FP64 phase in
//              revolutions, hardware sine and cosine), all rows (q, re / im) in one workgroup
//   E'[m][n] = sum_q A2[m][q] T[q][n]                 SP x SP, K = N, real and imaginary part
//   E = -i E',  I = sum_c |E_c|^2
// T never leaves the CU: it is written to LDS as a split panel (rows ri SP + n, k = q) in the
// place of the stage buffers and is the second product's operand as it lies there; the table
// rows of the other operand come from global memory (one table serves both products).  SP =
// 64: a wave per 32 x 32 block of the image; SP = 32: K split over the waves, the partial sums
// joined through LDS.  Waves own 64 pupil rows (N = 128) or 32.
// Bound by the matrix cores and by what stands between their products (staging, the split of
// T).  Measured on 4096 emitters (crops 24-64, 1-41 planes, N = 128), a whole call: 16.7 ms with
// FP32 MFMA tiles (planes 16.1), 6.0 ms so (planes 4.8 + 1.0); a frame of 100 emitters of one
// plane 87 -> 30 us.  (Item, emitter and crop size in vector registers and the 64-bit offsets of a
// lane's sixteen pixels, formed once per plane, spilled 44 registers on the 64-row tile: 2.5 GB
// written and as much read per call, 6.5-6.7 ms.  The 64-row tile of N = 128, alone of all, still
// spills 10, 44 bytes a lane: beside 620 MiB of intensities it writes 23 MiB at one workgroup a CU
// and 119 at two.)  Waves of 32 pupil rows (eight of them) took 7.0 + 1.55 ms; table rows of the
// second product requested ahead of the split of T gave 2.75 -> 3.09 ms on the 64-row tile (they
// spill) and 1.20 -> 1.12 ms on the 32-row tile, where they are.
template <int N, int SP>
struct PlaneTile {
  static constexpr int WM = N >= 128 ? 64 : 32;
  using Cfg = HgCfg<2 * N, SP, 16, WM, SP>;
  static constexpr int NW = Cfg::NT / 64;
  static constexpr int COMBOS = SP == 64 ? (4 + NW - 1) / NW : 1;   // 32 x 32 image blocks per wave
  static constexpr int KPW = SP == 64 ? N / 16 : N / 16 / NW;       // k-steps per wave
  static_assert(SP == 64 || N / 16 % NW == 0, "whole k-steps per wave");
  static constexpr int PART = SP == 64 ? 0 : NW * 2 * 32 * 33 * 4;  // partial sums of a 32 x 32 image
  static constexpr int T_BYTES = (int)hg_panel_bytes(N, 2 * SP);
  static constexpr int LDS_BYTES =
      Cfg::LDS_BYTES > T_BYTES ? (Cfg::LDS_BYTES > PART ? Cfg::LDS_BYTES : PART) : (T_BYTES > PART ? T_BYTES : PART);
  // waves of a SIMD to leave registers for: at four (128 registers) two workgroups of six waves fit a
  // CU, at 130 registers one (4096 crops of at most 16 pixels, 9 planes, N = 96: 1.14 ms, 1.69 with one)
  static constexpr int OCC = SP == 32 && (N == 64 || N == 96) ? 4 : 2;
  static constexpr int PIX = SP == 64 ? 16 * COMBOS : (1024 + Cfg::NT - 1) / Cfg::NT;   // intensities per lane
};

template <int N, int SP>
__device__ __forceinline__ void batch_plane(const BatchArgs& a, const BatchParam& bp, int slot, int d, char* lds,
                                            int tid) {
  using P = PlaneTile<N, SP>;
  using Cfg = typename P::Cfg;
  const int lane = tid & 63, w = tid >> 6, h = lane >> 5, l32 = lane & 31;
  const int S = bp.S, r0 = 32 - S / 2;
  const double zrev = ((d - 0.5 * (bp.D - 1)) * a.pitch + bp.zoff) * (1.0 / kTwoPi);
  float isum[P::PIX];
#pragma unroll
  for (int r = 0; r < P::PIX; ++r) isum[r] = 0.f;
  FoldDefocusLoader<Cfg, 1> la;
  const float2* pf = a.Pf + (size_t)slot * 3 * N * N;
  la.Pf = pf;
  la.kszf = a.ksz;
  la.zrev[0] = zrev;
  la.w = N;
  la.nhp = N;   // row stride of ksz
  HgPanelLoader<Cfg, SP> lb;
  lb.src = a.tab + r0;
  lb.ld = kTabRows;
  typename FoldDefocusLoader<Cfg, 1>::Regs ra;
  typename HgPanelLoader<Cfg, SP>::Regs rb;
  if constexpr (SP == 32) {
    ra = la.load(0, tid);
    rb = lb.load(0, tid);
  }
#pragma unroll 1
  for (int c = 0; c < 3; ++c) {
    if constexpr (SP == 64) {
      la.Pf = pf + (size_t)c * N * N;
      ra = la.load(0, tid);
      rb = lb.load(0, tid);
    }
    hg8 fh[P::KPW], fl[P::KPW];   // table rows of this wave's image block, over its k-steps
    auto fetch = [&](int mb, int ks0) {
      const hg8* ap = reinterpret_cast<const hg8*>(a.tab) + r0 + 32 * mb + l32;
#pragma unroll
      for (int u = 0; u < P::KPW; ++u) {
        fh[u] = ap[(4 * (ks0 + u) + h) * kTabRows];
        fl[u] = ap[(4 * (ks0 + u) + 2 + h) * kTabRows];
      }
    };
    {
      HgAcc<Cfg> acc;
      acc.zero();
      hg_mainloop_pre<Cfg>(acc, la, lb, ra, rb, 0, N, lds, tid, w * P::WM, 0, lane);
      // every wave has left the stage buffers
      if constexpr (SP == 32) {
        // the table rows of the second product and the next component's first stage (the last
        // component reloads its own, unused) arrive while T is split and written; at SP = 64
        // the registers are taken
        la.Pf = pf + (size_t)min(c + 1, 2) * N * N;
        ra = la.load(0, tid);
        rb = lb.load(0, tid);
        fetch(0, w * P::KPW);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int i = 0; i < Cfg::TM; ++i)
#pragma unroll
        for (int j = 0; j < Cfg::TN; ++j) {
          float v[16];
#pragma unroll
          for (int r = 0; r < 16; ++r) v[r] = acc.c[i][j][r] * a.tscale;
          uint4 piece[4];
          hg_split16(v, piece);
          uint4* o = reinterpret_cast<uint4*>(lds) + (size_t)(4 * (w * P::WM / 32 + i)) * (2 * SP) + h * SP + 32 * j + l32;
#pragma unroll
          for (int p = 0; p < 4; ++p) o[p * 2 * SP] = piece[p];
        }
    }
    __syncthreads();
    const float escale = component_scale(a.escale, c);
    float2* Ec = a.E ? a.E + 3 * bp.off + ((size_t)(d * 3 + c) * S) * S : nullptr;
    // E' block of columns nb over k-steps [ks0, ks0 + KPW).  The cross products of all k go
    // first: the accumulators are then 2^-11 of their final size and their roundings do not
    // count.
    auto product = [&](int nb, int ks0, hg16& er, hg16& ei) {
      const hg8* bt = reinterpret_cast<const hg8*>(lds) + 32 * nb + l32;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        er[r] = 0.f;
        ei[r] = 0.f;
      }
#pragma unroll
      for (int u = 0; u < P::KPW; ++u) {
        const hg8* t = bt + (4 * (ks0 + u) + h) * 2 * SP;
        er = __builtin_amdgcn_mfma_f32_32x32x16_f16(fh[u], t[4 * SP], er, 0, 0, 0);
        ei = __builtin_amdgcn_mfma_f32_32x32x16_f16(fh[u], t[5 * SP], ei, 0, 0, 0);
        er = __builtin_amdgcn_mfma_f32_32x32x16_f16(fl[u], t[0], er, 0, 0, 0);
        ei = __builtin_amdgcn_mfma_f32_32x32x16_f16(fl[u], t[SP], ei, 0, 0, 0);
      }
#pragma unroll
      for (int u = 0; u < P::KPW; ++u) {
        const hg8* t = bt + (4 * (ks0 + u) + h) * 2 * SP;
        er = __builtin_amdgcn_mfma_f32_32x32x16_f16(fh[u], t[0], er, 0, 0, 0);
        ei = __builtin_amdgcn_mfma_f32_32x32x16_f16(fh[u], t[SP], ei, 0, 0, 0);
      }
    };
    // E = -i E' = (Im E', -Re E')
    if constexpr (SP == 64) {
#pragma unroll
      for (int q = 0; q < P::COMBOS; ++q) {
        const int blk = w + q * P::NW;
        if (blk >= 4) break;
        hg16 er, ei;
        fetch(blk >> 1, 0);
        product(blk & 1, 0, er, ei);
        const int n = 32 * (blk & 1) + l32, m0 = 32 * (blk >> 1) + 4 * h;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float x = ei[r] * escale, y = -er[r] * escale;
          isum[16 * q + r] += x * x + y * y;
          er[r] = x;
          ei[r] = y;
        }
        if (Ec) {
          // row steps formed here: the sixteen offsets, kept over the components, spill
          int step = __builtin_amdgcn_readfirstlane(S);
          asm("" : "+s"(step));
          const unsigned o = m0 * step + n;
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int dm = 8 * (r >> 2) + (r & 3);
            if (m0 + dm < S && n < S) Ec[o + dm * step] = make_float2(er[r], ei[r]);
          }
        }
      }
      __syncthreads();   // T is consumed
    } else {
      hg16 er, ei;
      product(0, w * P::KPW, er, ei);
      __syncthreads();   // T is consumed: the partial sums take its place
      float* part = reinterpret_cast<float*>(lds);
      float* pre = part + w * 2 * 32 * 33;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = 8 * (r >> 2) + 4 * h + (r & 3);
        pre[m * 33 + l32] = er[r];
        pre[32 * 33 + m * 33 + l32] = ei[r];
      }
      __syncthreads();
#pragma unroll
      for (int q = 0; q < P::PIX; ++q) {
        const int e = tid + Cfg::NT * q, m = e >> 5, n = e & 31;
        if (1024 % Cfg::NT != 0 && e >= 1024) break;
        float sr = 0.f, si = 0.f;
#pragma unroll
        for (int ww = 0; ww < P::NW; ++ww) {
          sr += part[ww * 2 * 32 * 33 + m * 33 + n];
          si += part[ww * 2 * 32 * 33 + 32 * 33 + m * 33 + n];
        }
        const float x = si * escale, y = -sr * escale;
        isum[q] += x * x + y * y;
        if (Ec && m < S && n < S) Ec[m * S + n] = make_float2(x, y);
      }
      __syncthreads();
    }
  }
  if (a.I) {
    float* Ip = a.I + bp.off + (size_t)d * S * S;
    if constexpr (SP == 64) {
#pragma unroll
      for (int q = 0; q < P::COMBOS; ++q) {
        const int blk = w + q * P::NW;
        if (blk >= 4) break;
        const int n = 32 * (blk & 1) + l32, m0 = 32 * (blk >> 1) + 4 * h;
        const int step = S;
        const unsigned o = m0 * step + n;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int dm = 8 * (r >> 2) + (r & 3);
          if (m0 + dm < S && n < S) Ip[o + dm * step] = isum[16 * q + r];
        }
      }
    } else {
#pragma unroll
      for (int q = 0; q < P::PIX; ++q) {
        const int e = tid + Cfg::NT * q, m = e >> 5, n = e & 31;
        if (m < S && n < S) Ip[m * S + n] = isum[q];
      }
    }
  }
}

// Memory that nothing writes while the kernel runs, read over the scalar path.
template <class T>
__device__ __forceinline__ auto as_constant(const T* p) {
  return (const T __attribute__((address_space(4)))*)p;
}

// Persistent plane kernel of tile class cls (one launch per class), which serves queues 8 cls
// .. 8 cls + 7.  Workgroup ids are dealt round-robin over the 8 XCDs, so workgroup b serves
// queue b % 8 of the class: the (emitter, plane) items of the emitters assigned to that queue,
// in order, so that the planes of one emitter run at the same time on one XCD and its folded
// pupil is read from that XCD's L2.
// The next item is drawn while the current one is computed.  A workgroup exits when its
// queue is exhausted; the grid has at least 8 workgroups, one per queue.
template <int N, int SP>
__global__ void __launch_bounds__((PlaneTile<N, SP>::Cfg::NT), (PlaneTile<N, SP>::OCC))
    batch_planes_kernel(BatchArgs a, int cls) {
  extern __shared__ __align__(16) char blds[];
  __shared__ long long item[2];
  const int tid = threadIdx.x;
  const int x = 8 * cls + (blockIdx.x & 7);
  // the lists are uploaded before the launch and an item is the same in every lane: scalar loads
  const auto pre = as_constant(a.pre);
  const auto qoff = as_constant(a.qoff);
  const int lo = qoff[x], hi = qoff[x + 1];
  const long long end = pre[hi];
  if (tid == 0) item[0] = (long long)atomicAdd(&a.counter[x], 1ull);
  __syncthreads();
  for (int turn = 0;; turn ^= 1) {
    const long long vit = item[turn];
    const int it_lo = __builtin_amdgcn_readfirstlane((int)vit), it_hi = __builtin_amdgcn_readfirstlane((int)(vit >> 32));
    const long long it = (long long)((unsigned long long)(unsigned)it_hi << 32 | (unsigned)it_lo);
    if (it >= end) break;
    long long next = 0;
    if (tid == 0) next = (long long)atomicAdd(&a.counter[x], 1ull);
    // emitter e of the queue with pre[e] <= it < pre[e + 1]
    int e0 = lo, e1 = hi - 1;
    while (e0 < e1) {
      const int mid = (e0 + e1 + 1) >> 1;
      if (pre[mid] <= it) e0 = mid; else e1 = mid - 1;
    }
    const int slot = as_constant(a.list)[e0];
    const int d = (int)(it - pre[e0]);
    const auto p = as_constant(a.params) + slot;
    BatchParam bp;
    bp.zoff = p->zoff;
    bp.off = p->off;
    bp.S = p->S;
    bp.D = p->D;
    batch_plane<N, SP>(a, bp, slot, d, blds, tid);
    if (tid == 0) item[turn ^ 1] = next;   // read after the barriers of the next plane, or below
    __syncthreads();
  }
}

// Every pupil size and tile class its own instantiation, indexed [N / 32 - 1][class].
typedef void (*PlaneKernel)(BatchArgs, int);
struct PlaneLaunch {
  PlaneKernel k;
  int threads, lds;
};
template <int N, int SP>
static PlaneLaunch plane_launch() {
  return PlaneLaunch{batch_planes_kernel<N, SP>, PlaneTile<N, SP>::Cfg::NT, PlaneTile<N, SP>::LDS_BYTES};
}
static const PlaneLaunch kPlanes[4][2] = {{plane_launch<32, 32>(), plane_launch<32, 64>()},
                                          {plane_launch<64, 32>(), plane_launch<64, 64>()},
                                          {plane_launch<96, 32>(), plane_launch<96, 64>()},
                                          {plane_launch<128, 32>(), plane_launch<128, 64>()}};

}  // namespace rw

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
namespace rw {
// each crop bucket on its own tile class, two workgroups per CU.  k_stage (8 or 16) is part of
// the configuration and of saved plans; the matrix instruction takes 16 pupil rows at once, so
// both run the same kernel.
static rwpsf_batch_config default_config() {
  rwpsf_batch_config c{};
  c.wg_per_cu = 2;
  for (int q = 0; q < 4; ++q) {
    c.tile_rows[q] = 16 * (q + 1);
    c.k_stage[q] = 16;
  }
  return c;
}
static bool config_valid(const rwpsf_batch_config& c) {
  if (c.wg_per_cu < 1 || c.wg_per_cu > kMaxWgPerCu) return false;
  for (int q = 0; q < 4; ++q) {
    if (c.tile_rows[q] % 16 != 0 || c.tile_rows[q] < 16 * (q + 1) || c.tile_rows[q] > 64) return false;
    if (c.k_stage[q] != 8 && c.k_stage[q] != 16) return false;
  }
  return true;
}
static bool config_equal(const rwpsf_batch_config& x, const rwpsf_batch_config& y) {
  return x.wg_per_cu == y.wg_per_cu && std::equal(x.tile_rows, x.tile_rows + 4, y.tile_rows) &&
         std::equal(x.k_stage, x.k_stage + 4, y.k_stage);
}
}  // namespace rw

struct rwpsf_batch {
  int device = 0;
  rwpsf_optics opt{};
  int N = 0, max_emitters = 0, num_cus = 0;
  double px = 0, pitch = 0, k = 0, s_max = 0;
  std::vector<void*> allocations;
  float2* d_Q = nullptr;
  double* d_ksz = nullptr;
  double4* d_gl = nullptr;      // [N*N] Gibson-Lanni phase tables, or null
  uint4* d_tab = nullptr;       // folded DFT table of both axes, a split-f16 panel of 96 rows
  rw::PupilScales scales;
  float2* d_pf = nullptr;       // [max][3][N][N] folded pupils
  long long items = 0;          // (emitter, plane) items of the staged call
  long long class_items[rw::kTileClasses] = {};   // of them, in the 32- and 64-row tile classes
  int class_grid[rw::kTileClasses] = {};          // persistent grid of each class (0 = class not launched)
  float* d_basis = nullptr;
  char* d_upload = nullptr;     // see off_coef() and the others
  unsigned long long* d_counter = nullptr;   // [8] queue counters
  char* h_staging = nullptr;    // pinned mirror of d_upload
  size_t upload_bytes = 0;
  hipEvent_t upload_done = nullptr;
  bool upload_pending = false;
  rwpsf_batch_config cfg = rw::default_config();
  bool use_graph = false;
  hipGraphExec_t gexec = nullptr;
  struct Key {
    int n = -1;
    void* I = nullptr;
    void* E = nullptr;
    rwpsf_batch_config cfg{};
    int grid[rw::kTileClasses] = {};   // the captured launches: a replay must launch the same classes
    hipStream_t st = nullptr;
  } gkey;
  ~rwpsf_batch() {   // teardown: failures cannot be reported and are ignored
    if (gexec) (void)hipGraphExecDestroy(gexec);
    if (upload_done) (void)hipEventDestroy(upload_done);
    if (h_staging) (void)hipHostFree(h_staging);
    for (void* p : allocations) (void)hipFree(p);
  }
};

namespace rw {

static int batch_validate(const rwpsf_batch* b, int n, const rwpsf_emitter* e) {
  if (!b || n < 1 || n > b->max_emitters || !e) return RWPSF_ERR_INVALID_ARG;
  for (int i = 0; i < n; ++i) {
    const rwpsf_emitter& x = e[i];
    if (!std::isfinite(x.x0_nm) || !std::isfinite(x.y0_nm) || !std::isfinite(x.z_nm))
      return RWPSF_ERR_INVALID_ARG;
    if (b->opt.gibson_lanni && (!std::isfinite(x.t_s_nm) || x.t_s_nm < 0.0)) return RWPSF_ERR_INVALID_ARG;
    if (std::fabs(x.x0_nm) > 4 * b->px || std::fabs(x.y0_nm) > 4 * b->px) return RWPSF_ERR_INVALID_ARG;
    if (x.crop < 1 || x.crop > RWPSF_BATCH_MAX_CROP || x.planes < 1 || x.planes > 4096)
      return RWPSF_ERR_INVALID_ARG;
    for (int q = 0; q < RWPSF_BATCH_MAX_ZERNIKE; ++q)
      if (!std::isfinite(x.zernike_waves[q])) return RWPSF_ERR_INVALID_ARG;
  }
  return RWPSF_OK;
}

template <class T>
static int balloc(rwpsf_batch* b, T** p, size_t count) {
  void* d = nullptr;
  hipError_t e = hipMalloc(&d, std::max<size_t>(16, count * sizeof(T)));
  if (e != hipSuccess) {
    set_hip_error(e);
    return RWPSF_ERR_OOM;
  }
  b->allocations.push_back(d);
  *p = (T*)d;
  return RWPSF_OK;
}

// Upload block: params [max] | coef [max][23] | list [max] | pre [max + 1] | qoff [17]
static size_t off_coef(const rwpsf_batch* b) { return sizeof(BatchParam) * b->max_emitters; }
static size_t off_list(const rwpsf_batch* b) { return off_coef(b) + sizeof(float) * kBasisRows * b->max_emitters; }
static size_t off_pre(const rwpsf_batch* b) {
  return (off_list(b) + sizeof(int) * b->max_emitters + 7) / 8 * 8;
}
static size_t off_qoff(const rwpsf_batch* b) { return off_pre(b) + sizeof(long long) * (b->max_emitters + 1); }
static size_t upload_size(const rwpsf_batch* b) { return off_qoff(b) + sizeof(int) * (kQueues + 1); }

// Tile of a configuration's tile rows: 16 and 48 run on the next larger one.
static int tile_of(int rows) { return rows > 32 ? 64 : 32; }

static int class_grid(int num_cus, int wg_per_cu, long long items) {
  const long long want = std::max<long long>(8, std::min<long long>(items, (long long)num_cus * wg_per_cu));
  return items == 0 ? 0 : (int)std::min<long long>(want, (long long)num_cus * kMaxWgPerCu);
}

// Fill the pinned staging area: cost-sorted params, the coefficient matrix, and the
// (emitter, plane) queues: per tile class, eight queues, the class's emitters dealt
// longest first to its least-loaded queue.
static void batch_stage(rwpsf_batch* b, int n, const rwpsf_emitter* e) {
  std::vector<long long> off(n + 1, 0);
  for (int i = 0; i < n; ++i) off[i + 1] = off[i] + (long long)e[i].planes * e[i].crop * e[i].crop;
  std::vector<int> order(n);
  std::iota(order.begin(), order.end(), 0);
  auto sp_of = [&](int i) { return tile_of(b->cfg.tile_rows[(e[i].crop - 1) / 16]); };
  auto cost = [&](int i) { return (double)e[i].planes * sp_of(i) * (b->N + sp_of(i)); };
  std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return cost(x) > cost(y); });
  BatchParam* prm = (BatchParam*)b->h_staging;
  float* coef = (float*)(b->h_staging + off_coef(b));
  for (int slot = 0; slot < n; ++slot) {
    const int i = order[slot];
    prm[slot].zoff = -e[i].z_nm;
    prm[slot].ts = b->opt.gibson_lanni ? e[i].t_s_nm : 0.0;
    prm[slot].off = off[i];
    prm[slot].S = e[i].crop;
    prm[slot].D = e[i].planes;
    prm[slot].SP = sp_of(i);
    prm[slot].pad = 0;
    float* cf = coef + (size_t)slot * kBasisRows;
    for (int q = 0; q < RWPSF_BATCH_MAX_ZERNIKE; ++q) cf[q] = (float)e[i].zernike_waves[q];
    cf[RWPSF_BATCH_MAX_ZERNIKE] = (float)(-b->k * e[i].x0_nm);
    cf[RWPSF_BATCH_MAX_ZERNIKE + 1] = (float)(-b->k * e[i].y0_nm);
  }
  std::vector<int> queue(n);
  double load[kQueues] = {};
  int count[kQueues] = {};
  for (int t = 0; t < kTileClasses; ++t) b->class_items[t] = 0;
  for (int slot = 0; slot < n; ++slot) {
    const int t = prm[slot].SP > 32;
    const int x = 8 * t + (int)(std::min_element(load + 8 * t, load + 8 * t + 8) - (load + 8 * t));
    queue[slot] = x;
    load[x] += cost(order[slot]);
    count[x] += 1;
    b->class_items[t] += prm[slot].D;
  }
  int* list = (int*)(b->h_staging + off_list(b));
  long long* pre = (long long*)(b->h_staging + off_pre(b));
  int* qoff = (int*)(b->h_staging + off_qoff(b));
  qoff[0] = 0;
  for (int x = 0; x < kQueues; ++x) qoff[x + 1] = qoff[x] + count[x];
  int fill[kQueues];
  for (int x = 0; x < kQueues; ++x) fill[x] = qoff[x];
  for (int slot = 0; slot < n; ++slot) list[fill[queue[slot]]++] = slot;
  pre[0] = 0;
  for (int i = 0; i < n; ++i) pre[i + 1] = pre[i] + prm[list[i]].D;
  b->items = pre[n];
  // persistent grid of each class: at least one workgroup per queue, no more than the
  // configured residency, none for an empty class
  for (int t = 0; t < kTileClasses; ++t) b->class_grid[t] = class_grid(b->num_cus, b->cfg.wg_per_cu, b->class_items[t]);
}

// Copy the staged parameter block to the device and record upload_done right after it,
// so that the next call may restage the pinned area while this call's kernels still run.
static int batch_upload(rwpsf_batch* b, hipStream_t st) {
  int rc;
  if ((rc = hip_check(hipMemcpyAsync(b->d_upload, b->h_staging, b->upload_bytes, hipMemcpyHostToDevice, st))) ||
      (rc = hip_check(hipEventRecord(b->upload_done, st))))
    return rc;
  b->upload_pending = true;
  return RWPSF_OK;
}

// The kernels of one call (they read the uploaded block in stream order): the fold, which also
// resets the queues, and one persistent launch per tile class.  This is what a graph captures.
static int batch_kernels(rwpsf_batch* b, int n, float* I, float2* E, hipStream_t st) {
  int rc;
  BatchArgs a{};
  a.params = (const BatchParam*)b->d_upload;
  a.Q = b->d_Q;
  a.ksz = b->d_ksz;
  a.coef = (const float*)(b->d_upload + off_coef(b));
  a.basis = b->d_basis;
  a.gl = b->d_gl;
  a.tab = b->d_tab;
  a.tscale = b->scales.tscale;
  a.escale = b->scales.escale;
  a.Pf = b->d_pf;
  a.list = (const int*)(b->d_upload + off_list(b));
  a.pre = (const long long*)(b->d_upload + off_pre(b));
  a.qoff = (const int*)(b->d_upload + off_qoff(b));
  a.I = I;
  a.E = E;
  a.counter = b->d_counter;
  a.n = n;
  a.N = b->N;
  a.pitch = b->pitch;
  // as many emitters per workgroup as leave four workgroups for each CU: the tables of a cell
  // (116 floats) are read once per group
  const int cells = b->N * b->N / 4 / 256;
  a.group = (int)std::min<long long>(16, std::max<long long>(1, (long long)n * cells / (4 * b->num_cus)));
  hipLaunchKernelGGL(batch_fold_kernel, dim3(cells * ((n + a.group - 1) / a.group)), dim3(256), 0, st, a);
  if ((rc = hip_check(hipGetLastError()))) return rc;
  // one launch per tile class, the tall tiles first; at least one workgroup per queue and
  // no more than the configured residency
  for (int t = kTileClasses - 1; t >= 0; --t) {
    const int grid = b->class_grid[t];
    if (grid == 0) continue;
    const PlaneLaunch& pl = kPlanes[b->N / 32 - 1][t];
    hipLaunchKernelGGL(pl.k, dim3(grid), dim3(pl.threads), pl.lds, st, a, t);
    if ((rc = hip_check(hipGetLastError()))) return rc;
  }
  return RWPSF_OK;
}

static int batch_enqueue(rwpsf_batch* b, int n, float* I, float2* E, hipStream_t st) {
  const int rc = batch_upload(b, st);
  return rc ? rc : batch_kernels(b, n, I, E, st);
}

}  // namespace rw

extern "C" {

int rwpsf_batch_offsets(int n, const rwpsf_emitter* e, int64_t* off) {
  if (n < 0 || (n > 0 && !e) || !off) return RWPSF_ERR_INVALID_ARG;
  off[0] = 0;
  for (int i = 0; i < n; ++i) {
    if (e[i].crop < 1 || e[i].planes < 1) return RWPSF_ERR_INVALID_ARG;
    off[i + 1] = off[i] + (int64_t)e[i].planes * e[i].crop * e[i].crop;
  }
  return RWPSF_OK;
}

int rwpsf_batch_create(const rwpsf_optics* o, int n_pupil, double pixel_nm, double pitch_nm,
                       int max_emitters, rwpsf_batch** out) {
  using namespace rw;
  if (!out) return RWPSF_ERR_INVALID_ARG;
  *out = nullptr;
  double zero = 0.0;
  rwpsf_grid g{1, 1, 1.0, 1.0, 1, &zero};
  rwpsf_numerics nm{RWPSF_FORM_FOURIER, n_pupil, 2, 8, RWPSF_MODEL_VECTORIAL, RWPSF_THETA_GAUSS};
  int st = validate_plan(o, &g, &nm);
  if (st != RWPSF_OK) return st;
  if (n_pupil < 32 || n_pupil > 128 || n_pupil % 32 != 0) return RWPSF_ERR_INVALID_ARG;
  if (!(pixel_nm > 0) || !std::isfinite(pixel_nm) || !(pitch_nm >= 0) || !std::isfinite(pitch_nm))
    return RWPSF_ERR_INVALID_ARG;
  if (max_emitters < 1 || max_emitters > (1 << 20)) return RWPSF_ERR_INVALID_ARG;
  int dev_count = 0;
  if (hipGetDeviceCount(&dev_count) != hipSuccess || dev_count < 1) return RWPSF_ERR_NO_DEVICE;
  rwpsf_batch* b = new (std::nothrow) rwpsf_batch();
  if (!b) return RWPSF_ERR_OOM;
  if (hipGetDevice(&b->device) != hipSuccess ||
      hipDeviceGetAttribute(&b->num_cus, hipDeviceAttributeMultiprocessorCount, b->device) != hipSuccess ||
      b->num_cus < 1) {
    delete b;
    return RWPSF_ERR_NO_DEVICE;
  }
  b->opt = *o;
  b->N = n_pupil;
  b->px = pixel_nm;
  b->pitch = pitch_nm;
  b->max_emitters = max_emitters;
  b->k = kTwoPi * o->n_i / o->wavelength_nm;
  b->s_max = o->na / o->n_i;
  const int N = n_pupil;
  const size_t NN = (size_t)N * N;
  std::vector<float2> Q(3 * NN, make_float2(0.f, 0.f));
  std::vector<double> ksz(NN, 0.0);
  std::vector<double4> gl(o->gibson_lanni ? NN : 0, make_double4(0.0, 0.0, 0.0, 0.0));
  std::vector<double> bound(o->gibson_lanni ? NN : 0, 1.0);   // largest amplitude of the layer's factor per cell
  GLParams glp{};
  glp.k0 = kTwoPi / o->wavelength_nm;
  glp.n_i = o->n_i;
  glp.n_s = o->n_s;
  glp.n_g = o->n_g;
  glp.n_g_d = o->n_g_design;
  glp.n_i_d = o->n_i_design;
  glp.t_g = o->t_g_nm;
  glp.t_g_d = o->t_g_design_nm;
  glp.t_i_d = o->t_i_design_nm;
  std::vector<float> basis((size_t)kBasisRows * NN, 0.f);
  const double ds = 2.0 * b->s_max / N;
  int pref_exp = 0;   // Q carries the mantissa of the prefactor, escale its power of two
  const double pref = std::frexp(o->focal_length * b->k / kTwoPi, &pref_exp);
  for (int j = 0; j < N; ++j)
    for (int l = 0; l < N; ++l) {
      const long u = 2L * j + 1 - N, v = 2L * l + 1 - N;
      const size_t cell = (size_t)j * N + l;
      const double sx = u * b->s_max / N, sy = v * b->s_max / N;
      basis[(size_t)RWPSF_BATCH_MAX_ZERNIKE * NN + cell] = (float)sx;
      basis[(size_t)(RWPSF_BATCH_MAX_ZERNIKE + 1) * NN + cell] = (float)sy;
      const double ru = (double)u / N, rv = (double)v / N, r = std::sqrt(ru * ru + rv * rv);
      for (int q = 0; q < RWPSF_BATCH_MAX_ZERNIKE; ++q)
        basis[(size_t)q * NN + cell] =
            (float)(kTwoPi * zernike_noll(q + 1, r, r > 0 ? ru / r : 1.0, r > 0 ? rv / r : 0.0));
      if (u * u + v * v > (long)N * N) continue;
      std::complex<double> e[3];
      base_pupil_cell(*o, 3, ds, sx, sy, e);
      for (int c = 0; c < 3; ++c) Q[c * NN + cell] = make_float2((float)(pref * e[c].real()), (float)(pref * e[c].imag()));
      ksz[cell] = b->k * std::sqrt(1.0 - (sx * sx + sy * sy));
      if (o->gibson_lanni) {
        // the phase is affine in t_s (t_i is affine in it and each layer's term is linear
        // in its thickness): store its value at t_s = 0 and its slope
        const double sin_t = std::sqrt(sx * sx + sy * sy), T = 1.0e4;
        double r0, i0, r1, i1;
        gl_opd(glp, 0.0, sin_t, &r0, &i0);
        gl_opd(glp, T, sin_t, &r1, &i1);
        gl[cell] = make_double4(r0, i0, (r1 - r0) / T, (i1 - i0) / T);
        // the decay exp(-(i0 + t_s slope)) is largest at t_s = 0 (the slope is not negative)
        bound[cell] = std::exp(std::min(std::max(0.0, -i0), 600.0));
      }
    }
  b->scales = pupil_scales(Q, 3, N, N, bound.empty() ? nullptr : bound.data(), pref_exp);
  b->upload_bytes = upload_size(b);
  int rc;
  if ((rc = balloc(b, &b->d_Q, 3 * NN)) || (rc = balloc(b, &b->d_ksz, NN)) ||
      (rc = balloc(b, &b->d_tab, hg_panel_bytes(N, kTabRows) / sizeof(uint4))) ||
      (rc = balloc(b, &b->d_pf, (size_t)max_emitters * 3 * NN)) ||
      (rc = balloc(b, &b->d_basis, (size_t)kBasisRows * NN)) ||
      (rc = balloc(b, &b->d_upload, b->upload_bytes)) ||
      (rc = balloc(b, &b->d_counter, kQueues)) || (o->gibson_lanni && (rc = balloc(b, &b->d_gl, NN)))) {
    delete b;
    return rc;
  }
  const hipError_t he = hipHostMalloc((void**)&b->h_staging, b->upload_bytes, hipHostMallocDefault);
  if (he != hipSuccess) {
    set_hip_error(he);
    b->h_staging = nullptr;
    delete b;
    return RWPSF_ERR_OOM;
  }
  std::memset(b->h_staging, 0, b->upload_bytes);
  if ((rc = hip_check(hipEventCreateWithFlags(&b->upload_done, hipEventDisableTiming))) ||
      (rc = hip_check(hipMemcpy(b->d_Q, Q.data(), Q.size() * sizeof(float2), hipMemcpyHostToDevice))) ||
      (rc = hip_check(hipMemcpy(b->d_ksz, ksz.data(), ksz.size() * sizeof(double), hipMemcpyHostToDevice))) ||
      // (pixel r of the table at (r - 32) pixel: 64 "pixels" centred on row 32, and 32 more)
      (rc = hip_check(launch_dft_panel(b->d_tab, kTabRows, kTabRows, 32, N, N, b->k, b->s_max, pixel_nm, nullptr))) ||
      (o->gibson_lanni &&
       (rc = hip_check(hipMemcpy(b->d_gl, gl.data(), gl.size() * sizeof(double4), hipMemcpyHostToDevice)))) ||
      (rc = hip_check(hipMemcpy(b->d_basis, basis.data(), basis.size() * sizeof(float), hipMemcpyHostToDevice))) ||
      (rc = hip_check(hipMemcpy(b->d_upload, b->h_staging, b->upload_bytes, hipMemcpyHostToDevice))) ||
      (rc = hip_check(hipDeviceSynchronize()))) {
    delete b;
    return rc;
  }
  for (int t = 0; t < 2; ++t) {
    const PlaneLaunch& pl = kPlanes[N / 32 - 1][t];
    if ((rc = hip_check(hipFuncSetAttribute((const void*)pl.k, hipFuncAttributeMaxDynamicSharedMemorySize, pl.lds)))) {
      delete b;
      return rc;
    }
  }
  *out = b;
  return RWPSF_OK;
}

void rwpsf_batch_destroy(rwpsf_batch* b) {   // teardown: HIP failures are ignored
  if (!b) return;
  int cur = 0;
  const bool had = hipGetDevice(&cur) == hipSuccess;
  (void)hipSetDevice(b->device);
  (void)hipDeviceSynchronize();
  delete b;
  if (had) (void)hipSetDevice(cur);
}

int rwpsf_batch_set_graph(rwpsf_batch* b, int enable) {
  if (!b) return RWPSF_ERR_INVALID_ARG;
  b->use_graph = enable != 0;
  return RWPSF_OK;
}

int rwpsf_batch_set_config(rwpsf_batch* b, const rwpsf_batch_config* c) {
  if (!b || !c || !rw::config_valid(*c)) return RWPSF_ERR_INVALID_ARG;
  b->cfg = *c;
  return RWPSF_OK;
}

int rwpsf_batch_get_config(const rwpsf_batch* b, rwpsf_batch_config* c) {
  if (!b || !c) return RWPSF_ERR_INVALID_ARG;
  *c = b->cfg;
  return RWPSF_OK;
}

int rwpsf_batch_compute(rwpsf_batch* b, int n, const rwpsf_emitter* e, float* I, void* E, void* stream) {
  using namespace rw;
  int rc = batch_validate(b, n, e);
  if (rc) return rc;
  if (!I && !E) return RWPSF_ERR_INVALID_ARG;
  int cur = -1;
  if (hipGetDevice(&cur) != hipSuccess || cur != b->device) return RWPSF_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  if (b->use_graph && !st) return RWPSF_ERR_INVALID_ARG;   // the legacy default stream cannot be captured
  // the previous upload must have left the pinned staging area before it is rewritten
  if (b->upload_pending && (rc = hip_check(hipEventSynchronize(b->upload_done)))) return rc;
  batch_stage(b, n, e);
  if ((rc = batch_upload(b, st))) return rc;
  if (!b->use_graph) {
    rc = batch_kernels(b, n, I, (float2*)E, st);
  } else {
    const bool same = b->gexec && b->gkey.n == n && b->gkey.I == I && b->gkey.E == E &&
                      config_equal(b->gkey.cfg, b->cfg) &&
                      std::equal(b->class_grid, b->class_grid + kTileClasses, b->gkey.grid) && b->gkey.st == st;
    if (!same) {
      if (b->gexec) {
        (void)hipGraphExecDestroy(b->gexec);
        b->gexec = nullptr;
      }
      hipGraph_t g = nullptr;
      if ((rc = hip_check(hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal)))) return rc;
      const int erc = batch_kernels(b, n, I, (float2*)E, st);
      hipError_t ce = hipStreamEndCapture(st, &g);
      if (erc) {
        if (g) (void)hipGraphDestroy(g);
        return erc;
      }
      if ((rc = hip_check(ce))) return rc;
      ce = hipGraphInstantiate(&b->gexec, g, nullptr, nullptr, 0);
      (void)hipGraphDestroy(g);
      if ((rc = hip_check(ce))) return rc;
      b->gkey.n = n;
      b->gkey.I = I;
      b->gkey.E = E;
      b->gkey.cfg = b->cfg;
      std::copy(b->class_grid, b->class_grid + kTileClasses, b->gkey.grid);
      b->gkey.st = st;
    }
    rc = hip_check(hipGraphLaunch(b->gexec, st));
  }
  return rc;
}

}  // extern "C"

namespace rw {

// Autotune cache: a flat JSON object
//   {"key": [wg_per_cu, tile_rows[0..3], k_stage[0..3], ms], ...}
// in the file named by RWPSF_AUTOTUNE_CACHE.  Anything that does not parse is ignored
// (and replaced on the next write).
static std::string tune_key(const rwpsf_batch* b, int n, const rwpsf_emitter* e) {
  int bucket[4] = {0, 0, 0, 0};
  long long planes = 0;
  for (int i = 0; i < n; ++i) {
    bucket[(e[i].crop - 1) / 16] += 1;
    planes += e[i].planes;
  }
  int nb = 1;
  while (nb < n) nb <<= 1;
  char buf[200];
  snprintf(buf, sizeof buf, "N%d_n%d_b%d-%d-%d-%d_meanD%lld_cus%d", b->N, nb, (int)(16.0 * bucket[0] / n),
           (int)(16.0 * bucket[1] / n), (int)(16.0 * bucket[2] / n), (int)(16.0 * bucket[3] / n), planes / n,
           b->num_cus);
  return buf;
}

typedef std::map<std::string, std::pair<rwpsf_batch_config, double>> TuneCache;

static TuneCache cache_read(const char* path) {
  TuneCache m;
  FILE* f = fopen(path, "r");
  if (!f) return m;
  std::string text;
  char chunk[4096];
  size_t got;
  while ((got = fread(chunk, 1, sizeof chunk, f)) > 0) text.append(chunk, got);
  fclose(f);
  size_t pos = text.find('{');
  if (pos == std::string::npos) return {};
  while (true) {
    const size_t k0 = text.find('"', pos);
    if (k0 == std::string::npos) break;
    const size_t k1 = text.find('"', k0 + 1);
    if (k1 == std::string::npos) return {};
    const size_t b0 = text.find('[', k1);
    const size_t b1 = text.find(']', b0 == std::string::npos ? k1 : b0);
    if (b0 == std::string::npos || b1 == std::string::npos) return {};
    rwpsf_batch_config c{};
    double ms = 0;
    if (sscanf(text.c_str() + b0, "[%d , %d , %d , %d , %d , %d , %d , %d , %d , %lf]", &c.wg_per_cu, &c.tile_rows[0],
               &c.tile_rows[1], &c.tile_rows[2], &c.tile_rows[3], &c.k_stage[0], &c.k_stage[1], &c.k_stage[2],
               &c.k_stage[3], &ms) != 10)
      return {};
    if (!config_valid(c)) return {};
    m[text.substr(k0 + 1, k1 - k0 - 1)] = {c, ms};
    pos = b1 + 1;
  }
  return m;
}

static void cache_write(const char* path, const TuneCache& m) {
  const std::string tmp = std::string(path) + ".tmp";
  FILE* f = fopen(tmp.c_str(), "w");
  if (!f) return;
  fprintf(f, "{\n");
  size_t i = 0;
  for (const auto& kv : m) {
    const rwpsf_batch_config& c = kv.second.first;
    fprintf(f, "  \"%s\": [%d, %d, %d, %d, %d, %d, %d, %d, %d, %.6f]%s\n", kv.first.c_str(), c.wg_per_cu,
            c.tile_rows[0], c.tile_rows[1], c.tile_rows[2], c.tile_rows[3], c.k_stage[0], c.k_stage[1], c.k_stage[2],
            c.k_stage[3], kv.second.second, ++i < m.size() ? "," : "");
  }
  fprintf(f, "}\n");
  fclose(f);
  rename(tmp.c_str(), path);
}

// Device time of one call with configuration c: the emitters are staged on the host once,
// then one untimed and two timed enqueues, so the host staging stays outside the window.
static int tune_trial(rwpsf_batch* b, int n, const rwpsf_emitter* e, float* I, hipStream_t st,
                      const rwpsf_batch_config& c, hipEvent_t t0, hipEvent_t t1, float* ms) {
  int rc;
  if (b->upload_pending && (rc = hip_check(hipEventSynchronize(b->upload_done)))) return rc;
  b->cfg = c;
  batch_stage(b, n, e);
  if ((rc = batch_enqueue(b, n, I, nullptr, st))) return rc;
  if ((rc = hip_check(hipEventRecord(t0, st)))) return rc;
  for (int r = 0; r < 2; ++r)
    if ((rc = batch_enqueue(b, n, I, nullptr, st))) return rc;
  if ((rc = hip_check(hipEventRecord(t1, st)))) return rc;
  if ((rc = hip_check(hipEventSynchronize(t1))) || (rc = hip_check(hipEventElapsedTime(ms, t0, t1)))) return rc;
  *ms *= 0.5f;
  return RWPSF_OK;
}

}  // namespace rw

extern "C" {

int rwpsf_batch_autotune(rwpsf_batch* b, int n, const rwpsf_emitter* e, float* I, void* stream,
                         rwpsf_batch_config* best_out, double* best_ms) {
  using namespace rw;
  int rc = batch_validate(b, n, e);
  if (rc) return rc;
  if (!I) return RWPSF_ERR_INVALID_ARG;
  int cur = -1;
  if (hipGetDevice(&cur) != hipSuccess || cur != b->device) return RWPSF_ERR_INVALID_ARG;
  const char* cache_path = getenv("RWPSF_AUTOTUNE_CACHE");
  std::string key;
  TuneCache cache;
  if (cache_path && *cache_path) {
    key = tune_key(b, n, e);
    cache = cache_read(cache_path);
    auto it = cache.find(key);
    if (it != cache.end()) {
      b->cfg = it->second.first;
      if (best_out) *best_out = it->second.first;
      if (best_ms) *best_ms = it->second.second;
      return RWPSF_OK;
    }
  }
  hipStream_t st = (hipStream_t)stream;
  const rwpsf_batch_config saved = b->cfg;
  hipEvent_t t0 = nullptr, t1 = nullptr;
  if ((rc = hip_check(hipEventCreate(&t0))) || (rc = hip_check(hipEventCreate(&t1)))) {
    if (t0) (void)hipEventDestroy(t0);
    return rc;
  }
  // coordinate search from the default: workgroups per CU, then for each crop bucket the
  // taller tile it could share (fewer, fuller launches against more padding).  A candidate that
  // launches what another has launched is not timed again: the choice between the two would be noise.
  long long bucket_items[4] = {};
  for (int i = 0; i < n; ++i) bucket_items[(e[i].crop - 1) / 16] += e[i].planes;
  std::vector<std::vector<int>> tried;
  auto launches = [&](const rwpsf_batch_config& c) {   // grids of the classes, tile of each bucket in use
    long long items[kTileClasses] = {};
    std::vector<int> v;
    for (int q = 0; q < 4; ++q) {
      items[tile_of(c.tile_rows[q]) > 32] += bucket_items[q];
      v.push_back(bucket_items[q] ? tile_of(c.tile_rows[q]) : 0);
    }
    for (long long k : items) v.push_back(class_grid(b->num_cus, c.wg_per_cu, k));
    return v;
  };
  rwpsf_batch_config best = default_config();
  float best_t = 1e30f;
  auto consider = [&](const rwpsf_batch_config& c) {
    const std::vector<int> v = launches(c);
    if (std::find(tried.begin(), tried.end(), v) != tried.end()) return (int)RWPSF_OK;
    tried.push_back(v);
    float ms = 0.f;
    const int r = tune_trial(b, n, e, I, st, c, t0, t1, &ms);
    if (r == RWPSF_OK && ms < best_t) {
      best_t = ms;
      best = c;
    }
    return r;
  };
  rc = consider(best);
  for (int wg = 1; wg <= 3 && !rc; ++wg) {
    if (wg == best.wg_per_cu) continue;
    rwpsf_batch_config c = best;
    c.wg_per_cu = wg;
    rc = consider(c);
  }
  for (int q = 0; q < 3 && !rc; ++q) {
    rwpsf_batch_config c = best;
    c.tile_rows[q] = 64;
    rc = consider(c);
  }
  (void)hipEventDestroy(t0);
  (void)hipEventDestroy(t1);
  b->cfg = rc ? saved : best;
  if (rc) return rc;
  if (best_out) *best_out = best;
  if (best_ms) *best_ms = best_t;
  if (cache_path && *cache_path) {
    cache[key] = {best, best_t};
    cache_write(cache_path, cache);
  }
  return RWPSF_OK;
}

}  // extern "C"
