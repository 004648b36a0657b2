// Learned surrogate of the PSF engine: (21 Noll coefficients, z) -> 64 x 64 intensity.
//
//   x  = (c / 0.05, z / 1000 nm)                                   22 features
//   h1 = relu(x W1 + b1), h2 = relu(h1 W2 + b2), h3 = relu(h2 W3 + b3)   1024 each
//   convolution branch:
//     d1 = relu(T(h3 as 16x8x8; K1) + c1)  16 x 16 x 16
//     d2 = relu(T(d1; K2) + c2)            8 x 32 x 32
//     yd = T(d2; K3) + c3                  64 x 64
//   basis branch: a = h3 Wa + ba (256), yb = a Wb + bb (64 x 64)
//   y = yd + yb
// T: stride-2 transposed convolution, 4 x 4 kernel, 1 pixel padding,
//   out[co, oy, ox] = sum_{ci,ky,kx} in[ci, iy, ix] K[ci, co, ky, kx], oy = 2 iy - 1 + ky.
//
// Dense layers run on the BF16 matrix cores (v_mfma_f32_32x32x16_bf16, FP32
// accumulate).  In the accurate mode every operand is split x = hi + lo with hi,
// lo in BF16 and the product is hi*hi + hi*lo + lo*hi (relative error ~1e-5); the
// fast mode uses hi*hi only.  The forward transposed convolutions run in one fused
// kernel per sample: the first two as implicit GEMMs on v_mfma_f32_16x16x32_bf16 (same
// splitting), the last (one output channel) in FP32, activations in LDS.  Their backward
// runs in one fused FP32 kernel per sample.  Weight gradients of the convolutions
// and all bias gradients are reduced over the batch in a fixed order through
// partial sums; training updates FP32 master weights with Adam.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <vector>

#include "rw_common.h"
#include "rw_plan.h"

namespace rw {

typedef float f16v_s __attribute__((ext_vector_type(16)));
typedef __bf16 bf8_t __attribute__((ext_vector_type(8)));

// ---------------------------------------------------------------- weight gradients of the dense layers
// dW = hin^T gout (K = batch) and db = column sums of gout for every dense layer in one
// launch: the products are independent once the gradients of all layers are known, and each
// alone is too small to fill the GPU (64 x 64 tiles, four 32 x 32 waves).  Both operands are
// k-major in memory: a thread loads eight k of one row (lanes along the rows, coalesced) and
// writes them as one 16-byte piece of BF16 hi and one of lo, in LDS [k / 16][hi 0-7, hi 8-15,
// lo 0-7, lo 8-15][row], from which 32 lanes read 32 consecutive pieces.  The bias sums are
// taken in FP64 by the first row of tiles from the values it stages.  Measured at a batch
// of 256: 19 us for all five layers, against 131 us of separate products (staged as FP32,
// split at every use, no loads in flight) and 50 us of column sums.
struct DwJob {
  const float* hin;    // [K][M]
  const float* gout;   // [K][N], N a multiple of 64
  float *dw, *db;      // [M][N], [N]
  int M, N, tile0;     // first workgroup of the job
};
constexpr int kDwJobs = 5, kDwBK = 64;
struct DwArgs {
  DwJob job[kDwJobs];
  int K;
};
constexpr int kDwPlane = kDwBK / 16 * 4 * 64 * 16;   // bytes of one operand's stage
typedef __bf16 bf2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ void bf_split8(const float* v, bf8_t* hi, bf8_t* lo) {
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    (*hi)[q] = (__bf16)v[q];
    (*lo)[q] = (__bf16)(v[q] - (float)(*hi)[q]);
  }
}

__global__ void __launch_bounds__(256) sg_dw_kernel(DwArgs a) {
  extern __shared__ __align__(16) char dwl[];
  __shared__ double red[256];
  int j = 0;
  while (j + 1 < kDwJobs && (int)blockIdx.x >= a.job[j + 1].tile0) ++j;
  const DwJob jb = a.job[j];
  const int tile = blockIdx.x - jb.tile0, tiles_n = jb.N / 64;
  const int tm = tile / tiles_n, tn = tile % tiles_n;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, h = lane >> 5, l32 = lane & 31;
  const int wm = (w >> 1) * 32, wn = (w & 1) * 32;
  const int row = tid & 63, K = a.K;
  const int cm = min(tm * 64 + row, jb.M - 1), cn = tn * 64 + row;   // rows past M are not stored
  const bool sums = tm == 0;
  f16v_s acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  double bsum = 0.0;
  struct Staged {
    float a[2][8], b[2][8];
  };
  // k groups of eight: thread group w takes groups w and w + 4 of a stage
  auto load = [&](int k0) {
    Staged g;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int k = k0 + 8 * (w + 4 * i) + q, ck = min(k, K - 1);
        const float av = jb.hin[(size_t)ck * jb.M + cm], bv = jb.gout[(size_t)ck * jb.N + cn];
        g.a[i][q] = k < K ? av : 0.f;
        g.b[i][q] = k < K ? bv : 0.f;
      }
    return g;
  };
  auto store = [&](char* st, const Staged& g) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int kg = w + 4 * i, at = ((kg >> 1) * 4 + (kg & 1)) * 64 + row;
      bf8_t hi, lo;
      bf_split8(g.a[i], &hi, &lo);
      reinterpret_cast<bf8_t*>(st)[at] = hi;
      reinterpret_cast<bf8_t*>(st)[at + 128] = lo;
      bf_split8(g.b[i], &hi, &lo);
      reinterpret_cast<bf8_t*>(st + kDwPlane)[at] = hi;
      reinterpret_cast<bf8_t*>(st + kDwPlane)[at + 128] = lo;
      if (sums)
#pragma unroll
        for (int q = 0; q < 8; ++q) bsum += (double)g.b[i][q];
    }
  };
  auto mma = [&](const char* st) {
    const bf8_t* ap = reinterpret_cast<const bf8_t*>(st) + wm + l32;
    const bf8_t* bp = reinterpret_cast<const bf8_t*>(st + kDwPlane) + wn + l32;
#pragma unroll
    for (int u = 0; u < kDwBK / 16; ++u) {
      const bf8_t ah = ap[(4 * u + h) * 64], al = ap[(4 * u + 2 + h) * 64];
      const bf8_t bh = bp[(4 * u + h) * 64], bl = bp[(4 * u + 2 + h) * 64];
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bh, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bl, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bh, acc, 0, 0, 0);
    }
  };
  const int KT = (K + kDwBK - 1) / kDwBK;
  store(dwl, load(0));
  __syncthreads();
  for (int kt = 0; kt < KT - 1; ++kt) {
    const Staged g = load((kt + 1) * kDwBK);
    mma(dwl + (kt & 1) * 2 * kDwPlane);
    store(dwl + ((kt + 1) & 1) * 2 * kDwPlane, g);
    __syncthreads();
  }
  mma(dwl + ((KT - 1) & 1) * 2 * kDwPlane);
  const int n = tn * 64 + wn + l32;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int m = tm * 64 + wm + 8 * (r >> 2) + 4 * h + (r & 3);
    if (m < jb.M) jb.dw[(size_t)m * jb.N + n] = acc[r];
  }
  if (sums) {
    red[tid] = bsum;
    __syncthreads();
    if (tid < 64) jb.db[cn] = (float)((red[tid] + red[tid + 64]) + (red[tid + 128] + red[tid + 192]));
  }
}

// ---------------------------------------------------------------- input layer
// h1 = relu(x W1 + b1) for the 22-feature input layer, in FP32 on the vector units: with
// K = 22 the layer is bound by writing h1, and a matrix-core tile would spend more on
// staging and splitting than on its products.  Thread t owns columns 4t .. 4t + 3 with
// their 22 weights in registers and walks kDense1Rows rows (x of a row is the same for
// the whole workgroup, staged in LDS); bias first, then k in order.
// The features are formed while the workgroup's rows of x are staged (x is also written for
// the backward pass).  A small batch takes fewer rows per workgroup, down to 2, so that it
// still spreads over the CUs (256 rows: 23 us in two launches -> 5 us).
constexpr int kDense1Rows = 64;
__global__ void __launch_bounds__(256) sg_dense1_kernel(const float* __restrict__ coef, const float* __restrict__ z,
                                                        const float* __restrict__ W1, const float* __restrict__ b1,
                                                        int B, int rows, float* __restrict__ x,
                                                        float* __restrict__ h1) {
  const int n = 4 * threadIdx.x;
  float4 w[22];
#pragma unroll
  for (int k = 0; k < 22; ++k) w[k] = *reinterpret_cast<const float4*>(W1 + k * 1024 + n);
  const float4 bias = make_float4(b1[n], b1[n + 1], b1[n + 2], b1[n + 3]);
  const int r0 = blockIdx.x * rows, r1 = min(B, r0 + rows);
  // the workgroup's rows of x, staged once (every lane then reads the same word: a broadcast)
  __shared__ float xs[kDense1Rows * 22];
  for (int i = threadIdx.x; i < (r1 - r0) * 22; i += 256) {
    const int b = r0 + i / 22, f = i % 22;
    const float v = f < 21 ? coef[(size_t)b * 21 + f] * (1.f / 0.05f) : z[b] * (1.f / 1000.f);
    xs[i] = v;
    x[(size_t)r0 * 22 + i] = v;
  }
  __syncthreads();
  for (int m = r0; m < r1; ++m) {
    const float* xm = xs + (m - r0) * 22;
    float4 acc = bias;
#pragma unroll
    for (int k = 0; k < 22; ++k) {
      const float xv = xm[k];
      acc.x = fmaf(xv, w[k].x, acc.x);
      acc.y = fmaf(xv, w[k].y, acc.y);
      acc.z = fmaf(xv, w[k].z, acc.z);
      acc.w = fmaf(xv, w[k].w, acc.w);
    }
    *reinterpret_cast<float4*>(h1 + (size_t)m * 1024 + n) =
        make_float4(fmaxf(acc.x, 0.f), fmaxf(acc.y, 0.f), fmaxf(acc.z, 0.f), fmaxf(acc.w, 0.f));
  }
}

// ---------------------------------------------------------------- dense GEMM, aligned fast path
// C[M][N] = (relu)(A B + bias) for K % 32 == 0 and N % 128 == 0 (the 1024-wide layers
// and the basis branch).  A is FP32 [M][K], split into BF16 hi / lo while it is staged;
// B is given pre-split as k-contiguous BF16 planes Bt_hi / Bt_lo [N][K].  Workgroup
// 128 x 128, 4 waves of 64 x 64 (2 x 2 MFMA blocks of 32 x 32 x 16), k-stage 32, two LDS
// stages; each lane reads its 8 consecutive k of an operand with one 16-byte LDS read.
constexpr int FBM = 128, FBN = 128, FBK = 32, FLD = FBK + 8;   // LDS row: 40 bf16 (80 B)
static_assert(4 * 64 * (64 + 4) * 4 <= 2 * 4 * FBM * FLD * 2, "the epilogue tiles fit in the stage buffers");
constexpr int kGroupM = 8;                                      // row blocks per band (XCD order)
typedef __bf16 bf4_t __attribute__((ext_vector_type(4)));

template <int NSPLIT>
__global__ void __launch_bounds__(256, 2) sg_gemm_fast_kernel(const float* __restrict__ A,
                                                              const __bf16* __restrict__ Bhi,
                                                              const __bf16* __restrict__ Blo,
                                                              float* __restrict__ C, int M, int N, int K,
                                                              const float* __restrict__ bias, int relu,
                                                              int Kc, int accumulate,
                                                              const float* __restrict__ mask) {
  constexpr int PL = FBM * FLD;             // one bf16 plane of a tile
  constexpr int STAGE = 4 * PL;             // A hi, A lo, B hi, B lo
  extern __shared__ __bf16 shb[];
  const int tiles_n = N / FBN;
  int tm = blockIdx.x / tiles_n, tn = blockIdx.x % tiles_n;
  {
    // Workgroups go to the 8 XCDs round robin, and each XCD has its own L2.  When the row
    // blocks divide evenly, XCD x takes a contiguous eighth of them and walks it in bands
    // of kGroupM row blocks, column tile by column tile, so that the workgroups resident
    // on one XCD share A row blocks and B column tiles in its L2 (with the plain order the
    // 8 column tiles of a row block would sit on 8 XCDs and A would be fetched 8 times).
    const int rb = gridDim.x / tiles_n;
    if (rb % (8 * kGroupM) == 0) {
      const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
      const int band = local / (kGroupM * tiles_n), w = local % (kGroupM * tiles_n);
      tm = xcd * (rb >> 3) + band * kGroupM + w % kGroupM;
      tn = w / kGroupM;
    }
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;
  const int row0 = tm * FBM, col0 = tn * FBN;
  // split K: slice blockIdx.y covers k in [kbase, kbase + Kc) and, when there are several
  // slices, writes its raw partial product to slice blockIdx.y of C (reduced afterwards)
  const int kbase = blockIdx.y * Kc;
  if (gridDim.y > 1) C += (size_t)blockIdx.y * M * N;
  f16v_s acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  // A: 128 rows x 32 k = 1024 float4, 4 per thread; B: 128 cols x 32 k bf16 = 512 x 16 B per plane
  struct Staged {
    float4 ra[4];
    uint4 rbh[2], rbl[2];
  };
  // the staged tile is returned by value, so that it stays in registers
  auto load = [&](int k0) {
    Staged g;
    float4* ra = g.ra;
    uint4* rbh = g.rbh;
    uint4* rbl = g.rbl;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int idx = tid + 256 * i, r = idx >> 3, kq = 4 * (idx & 7);
      const int gr = min(row0 + r, M - 1);   // rows past M are computed but not stored
      ra[i] = *reinterpret_cast<const float4*>(A + (size_t)gr * K + kbase + k0 + kq);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int idx = tid + 256 * i, c = idx >> 2, k8 = 8 * (idx & 3);
      rbh[i] = *reinterpret_cast<const uint4*>(Bhi + (size_t)(col0 + c) * K + kbase + k0 + k8);
      if (NSPLIT > 1) rbl[i] = *reinterpret_cast<const uint4*>(Blo + (size_t)(col0 + c) * K + kbase + k0 + k8);
    }
    return g;
  };
  auto store = [&](__bf16* st, const Staged& g) {
    const float4* ra = g.ra;
    const uint4* rbh = g.rbh;
    const uint4* rbl = g.rbl;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int idx = tid + 256 * i, r = idx >> 3, kq = 4 * (idx & 7);
      const float v[4] = {ra[i].x, ra[i].y, ra[i].z, ra[i].w};
      bf4_t h, l;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        h[t] = (__bf16)v[t];
        l[t] = (__bf16)(v[t] - (float)h[t]);
      }
      *reinterpret_cast<bf4_t*>(st + r * FLD + kq) = h;
      if (NSPLIT > 1) *reinterpret_cast<bf4_t*>(st + PL + r * FLD + kq) = l;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int idx = tid + 256 * i, c = idx >> 2, k8 = 8 * (idx & 3);
      *reinterpret_cast<uint4*>(st + 2 * PL + c * FLD + k8) = rbh[i];
      if (NSPLIT > 1) *reinterpret_cast<uint4*>(st + 3 * PL + c * FLD + k8) = rbl[i];
    }
  };
  const int KT = Kc / FBK;
  auto mma = [&](const __bf16* cur) {
#pragma unroll
    for (int ks = 0; ks < FBK; ks += 16) {
      const int kb = ks + 8 * (lane >> 5);
      bf8_t ah[2], al[2], bh[2], bl[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int r = (wm + 32 * i + (lane & 31)) * FLD + kb;
        ah[i] = *reinterpret_cast<const bf8_t*>(cur + r);
        if (NSPLIT > 1) al[i] = *reinterpret_cast<const bf8_t*>(cur + PL + r);
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int c = (wn + 32 * j + (lane & 31)) * FLD + kb;
        bh[j] = *reinterpret_cast<const bf8_t*>(cur + 2 * PL + c);
        if (NSPLIT > 1) bl[j] = *reinterpret_cast<const bf8_t*>(cur + 3 * PL + c);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[i], bh[j], acc[i][j], 0, 0, 0);
          if (NSPLIT > 1) {
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[i], bl[j], acc[i][j], 0, 0, 0);
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al[i], bh[j], acc[i][j], 0, 0, 0);
          }
        }
    }
  };
  // Two stages of global loads in flight: a stage's MFMAs take far less time than a
  // load's latency, so stage kt + 2 is requested while stage kt is multiplied and stage
  // kt + 1 (already in registers) is written to the other LDS buffer.  KT >= 2; the last
  // two stages are peeled, so that no branch surrounds the loads and stores.
  Staged g1 = load(FBK);
  store(shb, load(0));
  __syncthreads();
  for (int kt = 0; kt < KT - 2; ++kt) {
    const Staged g2 = load((kt + 2) * FBK);
    mma(shb + (kt & 1) * STAGE);
    store(shb + ((kt + 1) & 1) * STAGE, g1);
    __syncthreads();
    g1 = g2;
  }
  mma(shb + (KT & 1) * STAGE);
  store(shb + ((KT - 1) & 1) * STAGE, g1);
  __syncthreads();
  mma(shb + ((KT - 1) & 1) * STAGE);
  // Epilogue through LDS (the stage buffers are free now): each wave writes its 64 x 64
  // tile row-major, then stores whole 16-byte row pieces, a quarter of the store
  // instructions of one value per lane per accumulator register.
  __syncthreads();
  constexpr int TLD = 64 + 4;   // floats per LDS row of a wave's tile
  float* tw = reinterpret_cast<float*>(shb) + wave * 64 * TLD;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        tw[(32 * i + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * TLD + 32 * j + (lane & 31)] = acc[i][j][r];
  __syncthreads();
  const bool raw = gridDim.y > 1;
  const int c4 = lane & 15, n = col0 + wn + 4 * c4;
  float4 bn = make_float4(0.f, 0.f, 0.f, 0.f);
  if (bias && !raw) bn = make_float4(bias[n], bias[n + 1], bias[n + 2], bias[n + 3]);   // (bias is 4-byte aligned)
#pragma unroll 4
  for (int it = 0; it < 16; ++it) {
    const int row = 4 * it + (lane >> 4), m = row0 + wm + row;
    if (m < M) {
      float4 v = *reinterpret_cast<const float4*>(tw + row * TLD + 4 * c4);
      float4* dst = reinterpret_cast<float4*>(C + (size_t)m * N + n);
      if (!raw) {
        const float4 prev = accumulate ? *dst : make_float4(0.f, 0.f, 0.f, 0.f);
        v = make_float4(v.x + bn.x + prev.x, v.y + bn.y + prev.y, v.z + bn.z + prev.z, v.w + bn.w + prev.w);
        if (relu) v = make_float4(fmaxf(v.x, 0.f), fmaxf(v.y, 0.f), fmaxf(v.z, 0.f), fmaxf(v.w, 0.f));
        if (mask) {
          const float4 h = *reinterpret_cast<const float4*>(mask + (size_t)m * N + n);
          v = make_float4(h.x > 0.f ? v.x : 0.f, h.y > 0.f ? v.y : 0.f, h.z > 0.f ? v.z : 0.f, h.w > 0.f ? v.w : 0.f);
        }
      }
      *dst = v;
    }
  }
}

// C = (relu)(sum over slices of ws[s] (in slice order) + bias (+ C)), 0 where the mask is not
// positive, after a split-K product
__global__ void sg_splitk_reduce_kernel(const float* __restrict__ ws, int slices, size_t MN, int N,
                                        const float* __restrict__ bias, int relu, int accumulate,
                                        const float* __restrict__ mask, float* __restrict__ C) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= MN) return;
  float v = 0.f;
  for (int s = 0; s < slices; ++s) v += ws[(size_t)s * MN + i];
  if (bias) v += bias[i % N];
  if (accumulate) v += C[i];
  if (relu) v = fmaxf(v, 0.f);
  C[i] = !mask || mask[i] > 0.f ? v : 0.f;
}

// ---------------------------------------------------------------- dense GEMM, few rows
// The same product for a batch of few rows, where 128 x 128 tiles leave most CUs idle and a
// split over K costs a second launch: one 32 x 32 tile per workgroup, the K range split
// over its NW waves, operands loaded straight into the registers of the matrix instruction
// (a lane's eight consecutive k: two 16-byte FP32 loads of A, split there, and one 16-byte
// load of each plane of B), no barrier before the partial sums of the waves are added
// through LDS in wave order.  NW = 1 keeps the one running sum over K of the large tiles: the
// forward products take it, so that a sample's relu decisions do not depend on the batch it
// comes in; the others take the slices that the large tiles split K into at these sizes.  A
// wave is bound by its own chain of loads, splits and dependent MFMAs.  At 256 rows: forward
// layers 16 us on average (128 x 128 tiles 18 us), g W^T with K = 1024 11 us and with K = 4096
// 17 us with its reduction (23 us each).  One, two or three groups of loads in flight and an
// order of tiles by XCD measured the same.
template <int NSPLIT, int NW, bool RAW>
__global__ void __launch_bounds__(NW * 64) sg_gemm_skinny_kernel(const float* __restrict__ A,
                                                                 const __bf16* __restrict__ Bhi,
                                                                 const __bf16* __restrict__ Blo, float* __restrict__ C,
                                                                 int M, int N, int K, const float* __restrict__ bias,
                                                                 int relu, int accumulate,
                                                                 const float* __restrict__ mask) {
  constexpr int G = NW == 1 ? 8 : 4;   // k-steps of 16 loaded together
  extern __shared__ float skl[];   // [NW][32][33]
  const int tiles_n = N / 32;
  const int tm = blockIdx.x / tiles_n, tn = blockIdx.x % tiles_n;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, h = lane >> 5, l32 = lane & 31;
  const int ks = K / (NW * gridDim.y), slice = blockIdx.y * NW + w;   // ks is a multiple of 16 G
  const int kb = slice * ks, ke = kb + ks;
  const float* ap = A + (size_t)min(tm * 32 + l32, M - 1) * K + 8 * h;   // rows past M are not stored
  const size_t bo = (size_t)(tn * 32 + l32) * K + 8 * h;
  f16v_s acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  struct Staged {
    float4 a[G][2];
    bf8_t bh[G], bl[G];
  };
  auto load = [&](int k0) {
    Staged g;
#pragma unroll
    for (int u = 0; u < G; ++u) {
      g.a[u][0] = *reinterpret_cast<const float4*>(ap + k0 + 16 * u);
      g.a[u][1] = *reinterpret_cast<const float4*>(ap + k0 + 16 * u + 4);
      g.bh[u] = *reinterpret_cast<const bf8_t*>(Bhi + bo + k0 + 16 * u);
      if (NSPLIT > 1) g.bl[u] = *reinterpret_cast<const bf8_t*>(Blo + bo + k0 + 16 * u);
    }
    return g;
  };
  Staged cur = load(kb);
  for (int k0 = kb; k0 < ke; k0 += 16 * G) {
    const Staged nxt = load(min(k0 + 16 * G, ke - 16 * G));
#pragma unroll
    for (int u = 0; u < G; ++u) {
      const float v[8] = {cur.a[u][0].x, cur.a[u][0].y, cur.a[u][0].z, cur.a[u][0].w,
                          cur.a[u][1].x, cur.a[u][1].y, cur.a[u][1].z, cur.a[u][1].w};
      bf8_t ah, al;
      bf_split8(v, &ah, &al);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, cur.bh[u], acc, 0, 0, 0);
      if (NSPLIT > 1) {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, cur.bl[u], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, cur.bh[u], acc, 0, 0, 0);
      }
    }
    cur = nxt;
  }
  if (RAW) {   // the slice's product to the workspace
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int m = tm * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
      if (m < M) C[((size_t)slice * M + m) * N + tn * 32 + l32] = acc[r];
    }
    return;
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) skl[(w * 32 + 8 * (r >> 2) + 4 * h + (r & 3)) * 33 + l32] = acc[r];
  __syncthreads();
  for (int e = tid; e < 1024; e += NW * 64) {
    const int r = e >> 5, c = e & 31, m = tm * 32 + r, n = tn * 32 + c;
    if (m >= M) continue;
    float v = 0.f;
#pragma unroll
    for (int q = 0; q < NW; ++q) v += skl[(q * 32 + r) * 33 + c];
    if (bias) v += bias[n];
    const size_t at = (size_t)m * N + n;
    if (accumulate) v += C[at];
    if (relu) v = fmaxf(v, 0.f);
    C[at] = !mask || mask[at] > 0.f ? v : 0.f;
  }
}

// Dense product C = (relu)(A B + bias (+ C)), 0 where the mask is not positive, with B given
// as BF16 planes Bt [N][K].  Up to kSkinnyRows rows take the 32 x 32 tiles (they read A and
// B from L2 once per tile: at 1024 rows the 128 x 128 tiles are faster).  A larger product
// with few tiles is split over K (up to 16 slices, each at least 128 deep) into the workspace
// ws (ws_floats floats) and reduced in slice order, so the result does not depend on the
// launch.
constexpr int kSkinnyRows = 512;
template <int NSPLIT, int NW, bool RAW = false>
static hipError_t sg_skinny_launch(const float* A, const __bf16* Bh, const __bf16* Bl, float* C, int M, int N, int K,
                                   const float* bias, int relu, int accumulate, const float* mask, hipStream_t st,
                                   int wgs = 1) {
  hipLaunchKernelGGL((sg_gemm_skinny_kernel<NSPLIT, NW, RAW>), dim3((M + 31) / 32 * (N / 32), wgs), dim3(NW * 64),
                     RAW ? 0 : NW * 32 * 33 * sizeof(float), st, A, Bh, Bl, C, M, N, K, bias, relu, accumulate, mask);
  return hipGetLastError();
}
static hipError_t sg_gemm_fast(const float* A, const __bf16* Bh, const __bf16* Bl, float* C, int M, int N, int K,
                               const float* bias, int relu, int nsplit, hipStream_t st, int accumulate = 0,
                               const float* mask = nullptr, float* ws = nullptr, size_t ws_floats = 0,
                               int target_wg = 0) {
  if (M <= kSkinnyRows && !ws && K % 128 == 0)   // forward: no split of K
    return nsplit > 1 ? sg_skinny_launch<3, 1>(A, Bh, Bl, C, M, N, K, bias, relu, accumulate, mask, st)
                      : sg_skinny_launch<1, 1>(A, Bh, Bl, C, M, N, K, bias, relu, accumulate, mask, st);
  if (M <= kSkinnyRows) {
    // backward (three products): slices of 256 k where K = 4096, else of 128
    if (K >= 4096) {
      // 16 slices of a tile in one workgroup read 1 MB through one CU's cache (33 us): four
      // workgroups of four slices a tile, and the reduction of the larger products
      const size_t MN = (size_t)M * N;
      if (16 * MN > ws_floats) return hipErrorInvalidValue;
      const hipError_t e = sg_skinny_launch<3, 4, true>(A, Bh, Bl, ws, M, N, K, nullptr, 0, 0, nullptr, st, 4);
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL(sg_splitk_reduce_kernel, dim3((unsigned)((MN + 255) / 256)), dim3(256), 0, st, ws, 16, MN, N,
                         bias, relu, accumulate, mask, C);
      return hipGetLastError();
    }
    if (K >= 1024) return sg_skinny_launch<3, 8>(A, Bh, Bl, C, M, N, K, bias, relu, accumulate, mask, st);
    return sg_skinny_launch<3, 2>(A, Bh, Bl, C, M, N, K, bias, relu, accumulate, mask, st);
  }
  const int tiles = ((M + FBM - 1) / FBM) * (N / FBN);
  int slices = 1;
  while (ws && slices < 16 && tiles * slices * 2 <= target_wg && K % (2 * slices * FBK) == 0 &&
         K / (2 * slices) >= 128 && (size_t)2 * slices * M * N <= ws_floats)
    slices *= 2;
  const dim3 grid(tiles, slices);
  if (K / slices < 2 * FBK) return hipErrorInvalidValue;   // the pipeline needs two k-stages
  const int lds = 2 * 4 * FBM * FLD * (int)sizeof(__bf16);
  float* out = slices > 1 ? ws : C;
  if (nsplit > 1)
    hipLaunchKernelGGL(sg_gemm_fast_kernel<3>, grid, dim3(256), lds, st, A, Bh, Bl, out, M, N, K, bias, relu,
                       K / slices, accumulate, mask);
  else
    hipLaunchKernelGGL(sg_gemm_fast_kernel<1>, grid, dim3(256), lds, st, A, Bh, Bl, out, M, N, K, bias, relu,
                       K / slices, accumulate, mask);
  if (slices > 1) {
    const size_t MN = (size_t)M * N;
    hipLaunchKernelGGL(sg_splitk_reduce_kernel, dim3((unsigned)((MN + 255) / 256)), dim3(256), 0, st, ws, slices, MN,
                       N, bias, relu, accumulate, mask, C);
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------- operand planes of the weights
// BF16 hi / lo planes of the dense weights, in their own order ([K][N], the operand of g W^T)
// and transposed ([N][K], the operand of h W), and the decoder's fragments, in one launch.
// They are brought up to date whenever the weights change (set_state, Adam), so the
// products, also captured ones, find them ready: 10 launches and 66 us of each training step
// before (9 us now), 40 us of each inference call.
struct PlaneJob {
  const float* W;        // [K][N]
  __bf16 *h, *l, *th, *tl;
  int K, N, tile0;
};
constexpr int kPlaneJobs = 4;
struct PlaneArgs {
  PlaneJob job[kPlaneJobs];
  const float *K1, *K2;
  __bf16 *f1h, *f1l, *f2h, *f2l;
  int tiles;             // 32 x 32 tiles of the dense weights; the decoder's workgroups follow
};
__device__ void sg_dec_fragment(int i, const PlaneArgs& a);

__global__ void __launch_bounds__(256) sg_planes_kernel(PlaneArgs a) {
  if ((int)blockIdx.x >= a.tiles) {
    sg_dec_fragment((blockIdx.x - a.tiles) * 256 + threadIdx.x, a);
    return;
  }
  __shared__ float t[32][33];
  int j = 0;
  while (j + 1 < kPlaneJobs && (int)blockIdx.x >= a.job[j + 1].tile0) ++j;
  const PlaneJob jb = a.job[j];
  const int tile = blockIdx.x - jb.tile0, tn = tile % (jb.N / 32), tk = tile / (jb.N / 32);
  const int c = threadIdx.x & 31, r0 = threadIdx.x >> 5;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = r0 + 8 * i;
    const size_t at = (size_t)(32 * tk + r) * jb.N + 32 * tn + c;
    const float v = jb.W[at];
    const __bf16 hi = (__bf16)v;
    jb.h[at] = hi;
    jb.l[at] = (__bf16)(v - (float)hi);
    t[r][c] = v;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = r0 + 8 * i;
    const size_t at = (size_t)(32 * tn + r) * jb.K + 32 * tk + c;
    const float v = t[c][r];
    const __bf16 hi = (__bf16)v;
    jb.th[at] = hi;
    jb.tl[at] = (__bf16)(v - (float)hi);
  }
}

// ---------------------------------------------------------------- elementwise
// Error model of the surrogate: log rel-L2 ~ w . phi(c, z) with the features
// phi = (1, (c_1 / 0.05)^2 .. (c_21 / 0.05)^2, (z / 1000 nm)^2, |z| / 1000 nm).
constexpr int kGateFeatures = 24;
__device__ __forceinline__ float sg_gate_feature(const float* __restrict__ c, float z, int f) {
  if (f == 0) return 1.f;
  if (f <= 21) {
    const float u = c[f - 1] * (1.f / 0.05f);
    return u * u;
  }
  const float t = z * (1.f / 1000.f);
  return f == 22 ? t * t : fabsf(t);
}

__global__ void sg_gate_features_kernel(const float* __restrict__ coef, const float* __restrict__ z, int B,
                                        float* __restrict__ phi) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= B * kGateFeatures) return;
  const int b = i / kGateFeatures, f = i % kGateFeatures;
  phi[i] = sg_gate_feature(coef + (size_t)b * 21, z[b], f);
}

__global__ void sg_gate_predict_kernel(const float* __restrict__ coef, const float* __restrict__ z, int B,
                                       const float* __restrict__ w, float* __restrict__ out) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  float s = 0.f;
#pragma unroll
  for (int f = 0; f < kGateFeatures; ++f) s = fmaf(w[f], sg_gate_feature(coef + (size_t)b * 21, z[b], f), s);
  out[b] = s;
}

// ---------------------------------------------------------------- transposed convolution
// ---------------------------------------------------------------- fused decoder on the matrix cores
// The three transposed convolutions of one sample in one workgroup, activations kept in
// LDS.  Output pixel (2Y + py, 2X + px) of a stride-2, 4 x 4, pad-1 transposed convolution
// takes input rows Y + dy and kernel rows ky with (dy, ky) = (0, 1), (-1, 3) for py = 0 and
// (+1, 0), (0, 2) for py = 1 (the same along x), so each output parity class is a plain
// GEMM over the input pixels: M = pixels, K = (tap, input channel), N = output channels.
//   layer 1 (C0 -> C1 = 16, 8x8 -> 16x16): one GEMM per class (py, px), K = 4 C0, N = 16;
//   layer 2 (C1 -> C2 = 8, 16x16 -> 32x32): one GEMM per row class py with both column
//     classes side by side in N = 2 C2 = 16 (K = 6 C1 over the input columns X-1, X, X+1;
//     the tap a column class does not use has a zero weight);
//   layer 3 (C2 -> 1, 32x32 -> 64x64): N = 1 is a matrix-vector product, done in FP32 on
//     the vector units (a thread owns 2 x 2 input pixels and their 4 x 4 outputs).
// Layers 1 and 2 run v_mfma_f32_16x16x32_bf16: A lane l holds row l % 16 and eight
// consecutive k of group l / 16, B lane l holds column l % 16 and the same eight k, C
// register r of lane l holds row 4 (l / 16) + r, column l % 16.  The weights are A and the
// pixels B, so that a lane ends up with four channels of one pixel and writes them at once.
// Activations sit in LDS channel-last with a zero border, so the eight k of a lane are eight consecutive
// channels of one source pixel (two 16-byte reads), with no bounds tests.  Weights are
// pre-arranged as B fragments ([class][k-step][lane][8] BF16 hi / lo) and held in
// registers for all samples of the workgroup.  The inputs of the two matrix-core layers
// are split into BF16 hi / lo once, when they are written to LDS (each value feeds up to
// 16 fragments).
constexpr int DC0 = 16, DC1 = 16, DC2 = 8;          // decoder channels (layer inputs)
// inputs of the matrix-core layers are held as BF16 hi / lo planes (split once, when
// written), DXb BF16 per pixel (16-byte aligned, padded); the last layer's input in FP32
constexpr int DX0b = DC0 + 8, DX1b = DC1 + 8, DX2 = DC2;
constexpr int DX2H = 34 * 34 * 4;   // floats of one half of the last layer's channels: a pixel's four are 16 bytes
constexpr int DL0b = 10 * 10 * DX0b, DL1b = 18 * 18 * DX1b, DL2 = 34 * 34 * DX2;   // elements per plane
constexpr int DK1 = 4 * DC0 / 32, DK2 = 6 * DC1 / 32;    // k-steps of the layer-1 / layer-2 GEMMs
constexpr int kDecLdsBytes = 2 * (DL0b + DL1b) * 2 + DL2 * 4;
static_assert(DC1 == 16 && 2 * DC2 == 16 && DC0 % 8 == 0 && DC1 % 8 == 0, "decoder tile shapes");
typedef float f4v_t __attribute__((ext_vector_type(4)));

// B fragments: layer 1 [4 classes][DK1][64][8], layer 2 [2 row classes][DK2][64][8], hi and lo
__device__ void sg_dec_fragment(int i, const PlaneArgs& a) {
  const float *K1 = a.K1, *K2 = a.K2;
  const int n1 = 4 * DK1 * 64 * 8, n2 = 2 * DK2 * 64 * 8;
  if (i < n1) {
    const int q = i % 8, l = (i / 8) % 64, s = (i / 512) % DK1, p = i / (512 * DK1);
    const int py = p >> 1, px = p & 1, co = l % 16, k = 32 * s + 8 * (l / 16) + q;
    const int tap = k / DC0, ci = k % DC0, ta = tap >> 1, c = tap & 1;
    const int ky = py ? 2 * ta : 1 + 2 * ta, kx = px ? 2 * c : 1 + 2 * c;
    const float w = K1[((ci * DC1 + co) * 4 + ky) * 4 + kx];
    const __bf16 h = (__bf16)w;
    a.f1h[i] = h;
    a.f1l[i] = (__bf16)(w - (float)h);
  } else if (i < n1 + n2) {
    const int j = i - n1;
    const int q = j % 8, l = (j / 8) % 64, s = (j / 512) % DK2, py = j / (512 * DK2);
    const int n = l % 16, px = n / DC2, co = n % DC2, k = 32 * s + 8 * (l / 16) + q;
    const int t6 = k / DC1, ci = k % DC1, ta = t6 / 3, c3 = t6 % 3;
    const int ky = py ? 2 * ta : 1 + 2 * ta;
    // column tap c3 reads input column X + c3 - 1: px = 0 uses kx = 3, 1 (c3 = 0, 1),
    // px = 1 uses kx = 2, 0 (c3 = 1, 2)
    const int kx = px == 0 ? (c3 == 0 ? 3 : c3 == 1 ? 1 : -1) : (c3 == 0 ? -1 : c3 == 1 ? 2 : 0);
    const float w = kx < 0 ? 0.f : K2[((ci * DC2 + co) * 4 + ky) * 4 + kx];
    const __bf16 h = (__bf16)w;
    a.f2h[j] = h;
    a.f2l[j] = (__bf16)(w - (float)h);
  }
}

// h3 [B][DC0][8][8] (relu applied) -> y [B][64][64] += T(T(T(h3))); d1 [B][DC1][16][16] and d2
// [B][DC2][32][32] (post-relu) are also written when the pointers are not null (training).
// Persistent: workgroup g serves samples g, g + gridDim.x, ...
// LDS is busy 60% of the time, the vector units 52%, with two waves a SIMD to overlap them.  65536
// samples: 1102 us with one channel of a pixel a store, 1000 us with four.  Even and odd columns
// apart, which takes a sixth of the bank conflicts away, changed nothing more.
template <int NSPLIT>
__global__ void __launch_bounds__(256, 2) sg_decoder_kernel(const float* __restrict__ h3, int B,
                                                            const bf8_t* __restrict__ f1h,
                                                            const bf8_t* __restrict__ f1l,
                                                            const bf8_t* __restrict__ f2h,
                                                            const bf8_t* __restrict__ f2l,
                                                            const float* __restrict__ c1,
                                                            const float* __restrict__ c2,
                                                            const float* __restrict__ K3,
                                                            const float* __restrict__ c3,
                                                            float* __restrict__ y, float* __restrict__ d1g,
                                                            float* __restrict__ d2g) {
  extern __shared__ float dls[];
  __bf16* X0h = reinterpret_cast<__bf16*>(dls);   // [10][10][DX0b] hi, then lo
  __bf16* X0l = X0h + DL0b;
  __bf16* X1h = X0l + DL0b;                       // [18][18][DX1b] hi, then lo
  __bf16* X1l = X1h + DL1b;
  float* X2 = reinterpret_cast<float*>(X1l + DL1b);   // [channel half][34][34][4] FP32
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, g = lane >> 4, r16 = lane & 15;
  for (int i = tid; i < kDecLdsBytes / 4; i += 256) dls[i] = 0.f;   // zero borders (interiors are rewritten)
  // B fragments of this wave: layer-1 class p = w, layer-2 row class py2 = w / 2
  bf8_t w1h[DK1], w1l[DK1], w2h[DK2], w2l[DK2];
#pragma unroll
  for (int s = 0; s < DK1; ++s) {
    w1h[s] = f1h[(w * DK1 + s) * 64 + lane];
    if (NSPLIT > 1) w1l[s] = f1l[(w * DK1 + s) * 64 + lane];
  }
  const int py2 = w >> 1;
#pragma unroll
  for (int s = 0; s < DK2; ++s) {
    w2h[s] = f2h[(py2 * DK2 + s) * 64 + lane];
    if (NSPLIT > 1) w2l[s] = f2l[(py2 * DK2 + s) * 64 + lane];
  }
  // accumulator register i of a lane is output channel 4 g + i (layer 2: channel (4 g + i) % DC2 of
  // column class g / 2)
  float bias1[4], bias2[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    bias1[i] = c1[4 * g + i];
    bias2[i] = c2[(4 * g + i) % DC2];
  }
  const float bias3 = c3[0];
  // staged h3 of the next sample: DC0 * 64 floats, 8 per thread as two float4
  constexpr int NV = DC0 * 64 / 4 / 256;
  float4 hv[NV];
  auto fetch = [&](int b) {
#pragma unroll
    for (int v = 0; v < NV; ++v)
      hv[v] = b < B ? *reinterpret_cast<const float4*>(h3 + (size_t)b * DC0 * 64 + 4 * (tid + 256 * v))
                    : make_float4(0.f, 0.f, 0.f, 0.f);
  };
  fetch(blockIdx.x);
  __syncthreads();   // borders zeroed before any interior write
  for (int b = blockIdx.x; b < B; b += gridDim.x) {
    // this sample's basis-branch output under the thread's 4 x 4 outputs of layer 3,
    // requested now so that its latency passes under layers 1 and 2
    float* yo = y + (size_t)b * 4096 + (4 * (tid >> 4)) * 64 + 4 * (tid & 15);
    float4 yprev[4];
#pragma unroll
    for (int oy = 0; oy < 4; ++oy) yprev[oy] = *reinterpret_cast<const float4*>(yo + oy * 64);
    // ---- stage h3 [ci][Y][X] -> X0 [Y+1][X+1][ci]
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const int e = 4 * (tid + 256 * v), ci = e / 64, pix = e % 64;
      const float xs[4] = {hv[v].x, hv[v].y, hv[v].z, hv[v].w};
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int Y = (pix + t) / 8, X = (pix + t) % 8, at = ((Y + 1) * 10 + X + 1) * DX0b + ci;
        const __bf16 h = (__bf16)xs[t];
        X0h[at] = h;
        X0l[at] = (__bf16)(xs[t] - (float)h);
      }
    }
    fetch(b + gridDim.x);
    __syncthreads();
    // ---- layer 1: wave w = class (py, px); the four M-tiles of 16 pixels (Y, X) of the
    // 8 x 8 input, their accumulator chains interleaved
    {
      const int py = w >> 1, px = w & 1;
      f4v_t acc[4];
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) acc[mt] = f4v_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < DK1; ++s) {
        const int k0 = 32 * s + 8 * g, tap = k0 / DC0, ci = k0 % DC0, a = tap >> 1, c = tap & 1;
        const int dy = py ? 1 - a : -a, dx = px ? 1 - c : -c;
        bf8_t ah[4], al[4];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
          const int m = 16 * mt + r16, Y = m >> 3, X = m & 7;
          const int at = ((Y + dy + 1) * 10 + X + dx + 1) * DX0b + ci;
          ah[mt] = *reinterpret_cast<const bf8_t*>(X0h + at);
          al[mt] = NSPLIT > 1 ? *reinterpret_cast<const bf8_t*>(X0l + at) : ah[mt];
        }
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1h[s], ah[mt], acc[mt], 0, 0, 0);
        if (NSPLIT > 1) {
#pragma unroll
          for (int mt = 0; mt < 4; ++mt)
            acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1l[s], ah[mt], acc[mt], 0, 0, 0);
#pragma unroll
          for (int mt = 0; mt < 4; ++mt)
            acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1h[s], al[mt], acc[mt], 0, 0, 0);
        }
      }
      // C: rows 4 g + i (output channels), column r16 (pixel): four channels of a pixel in one store
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
        const int mm = 16 * mt + r16, YY = mm >> 3, XX = mm & 7;
        const int at = ((2 * YY + py + 1) * 18 + 2 * XX + px + 1) * DX1b + 4 * g;
        bf4_t h, l;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float v = fmaxf(acc[mt][i] + bias1[i], 0.f);
          h[i] = (__bf16)v;
          l[i] = (__bf16)(v - (float)h[i]);
        }
        *reinterpret_cast<bf4_t*>(X1h + at) = h;
        *reinterpret_cast<bf4_t*>(X1l + at) = l;
      }
    }
    __syncthreads();
    if (d1g) {   // training: d1 [co][16][16]
      float* o = d1g + (size_t)b * DC1 * 256;
      for (int e = tid; e < DC1 * 256; e += 256) {
        const int co = e / 256, pix = e % 256, at = ((pix / 16 + 1) * 18 + pix % 16 + 1) * DX1b + co;
        o[e] = (float)X1h[at] + (float)X1l[at];   // the value to 2^-16 relative (its sign exactly)
      }
    }
    // ---- layer 2: wave w = row class py2, M-tiles 8 (w & 1) .. + 7 of the 16 x 16 input,
    // in groups of L2G tiles whose accumulator chains are interleaved (a chain's next
    // product waits for the previous one; the group's other chains fill the gap)
    {
      constexpr int L2G = 4;
#pragma unroll 1
      for (int t0 = 0; t0 < 8; t0 += L2G) {
        f4v_t acc[L2G];
#pragma unroll
        for (int u = 0; u < L2G; ++u) acc[u] = f4v_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < DK2; ++s) {
          const int k0 = 32 * s + 8 * g, t6 = k0 / DC1, ci = k0 % DC1, a = t6 / 3, c3 = t6 % 3;
          const int dy = py2 ? 1 - a : -a, dx = c3 - 1;
          bf8_t ah[L2G], al[L2G];
#pragma unroll
          for (int u = 0; u < L2G; ++u) {
            const int m = 16 * (8 * (w & 1) + t0 + u) + r16, Y = m >> 4, X = m & 15;
            const int at = ((Y + dy + 1) * 18 + X + dx + 1) * DX1b + ci;
            ah[u] = *reinterpret_cast<const bf8_t*>(X1h + at);
            al[u] = NSPLIT > 1 ? *reinterpret_cast<const bf8_t*>(X1l + at) : ah[u];
          }
#pragma unroll
          for (int u = 0; u < L2G; ++u) acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w2h[s], ah[u], acc[u], 0, 0, 0);
          if (NSPLIT > 1) {
#pragma unroll
            for (int u = 0; u < L2G; ++u)
              acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w2l[s], ah[u], acc[u], 0, 0, 0);
#pragma unroll
            for (int u = 0; u < L2G; ++u)
              acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w2h[s], al[u], acc[u], 0, 0, 0);
          }
        }
        const int px = g >> 1, half = g & 1;
#pragma unroll
        for (int u = 0; u < L2G; ++u) {
          const int mm = 16 * (8 * (w & 1) + t0 + u) + r16, YY = mm >> 4, XX = mm & 15;
          *reinterpret_cast<float4*>(X2 + half * DX2H + ((2 * YY + py2 + 1) * 34 + 2 * XX + px + 1) * 4) =
              make_float4(fmaxf(acc[u][0] + bias2[0], 0.f), fmaxf(acc[u][1] + bias2[1], 0.f),
                          fmaxf(acc[u][2] + bias2[2], 0.f), fmaxf(acc[u][3] + bias2[3], 0.f));
        }
      }
    }
    __syncthreads();
    if (d2g) {   // training: d2 [co][32][32]
      float* o = d2g + (size_t)b * DC2 * 1024;
      for (int e = tid; e < DC2 * 1024; e += 256) {
        const int co = e / 1024, pix = e % 1024;
        o[e] = X2[co / 4 * DX2H + ((pix / 32 + 1) * 34 + pix % 32 + 1) * 4 + co % 4];
      }
    }
    // ---- layer 3 (FP32): thread owns input pixels (2 Yb + u, 2 Xb + v), u, v in {0, 1},
    // reads the 4 x 4 neighbourhood rows 2 Yb - 1 .. 2 Yb + 2 and writes the 4 x 4 outputs
    {
      const int Yb = tid >> 4, Xb = tid & 15;
      float out[4][4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) out[i][j] = bias3;
#pragma unroll
      for (int hc = 0; hc < DC2; hc += 4) {
        float4 nb[4][4];   // channels hc .. hc + 3 at padded rows 2 Yb .. 2 Yb + 3, cols 2 Xb .. 2 Xb + 3
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            nb[i][j] = *reinterpret_cast<const float4*>(X2 + hc / 4 * DX2H + ((2 * Yb + i) * 34 + 2 * Xb + j) * 4);
#pragma unroll
        for (int cc = 0; cc < 4; ++cc) {
          const int ci = hc + cc;
#pragma unroll
          for (int oy = 0; oy < 4; ++oy)      // output row 4 Yb + oy = 2 (2 Yb + u) + py
#pragma unroll
            for (int ox = 0; ox < 4; ++ox) {
              const int u = oy >> 1, py = oy & 1, v = ox >> 1, px = ox & 1;
#pragma unroll
              for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                  const int dy = py ? 1 - a : -a, dx = px ? 1 - c : -c;
                  const int ky = py ? 2 * a : 1 + 2 * a, kx = px ? 2 * c : 1 + 2 * c;
                  // input pixel (2 Yb + u + dy, 2 Xb + v + dx) sits at nb[u + dy + 1][v + dx + 1]
                  const float4 q = nb[u + dy + 1][v + dx + 1];
                  const float xv = cc == 0 ? q.x : cc == 1 ? q.y : cc == 2 ? q.z : q.w;
                  out[oy][ox] = fmaf(xv, K3[ci * 16 + ky * 4 + kx], out[oy][ox]);
                }
            }
        }
      }
      // y holds the basis branch already: add the convolution branch to it
#pragma unroll
      for (int oy = 0; oy < 4; ++oy) {
        const float4 prev = yprev[oy];
        *reinterpret_cast<float4*>(yo + oy * 64) =
            make_float4(prev.x + out[oy][0], prev.y + out[oy][1], prev.z + out[oy][2], prev.w + out[oy][3]);
      }
    }
    // the next iteration's staging writes X0 only; X1 / X2 are rewritten after its barriers
  }
}

// ---------------------------------------------------------------- decoder backward
// Backward of the three transposed convolutions of a sample in one workgroup, with the loss
// gradient formed on the way: gy = 2 (y - t) / n, then per layer (3, 2, 1) the weight gradient
//   dK[ci][co][ky][kx] = sum_{iy, ix} in[ci][iy][ix] g[co][2 iy - 1 + ky][2 ix - 1 + kx]
// and the data gradient gin[ci][iy][ix] = sum_{co, ky, kx} g[co][..][..] K[ci][co][ky][kx],
// masked by the relu of the layer's input.  Everything stays FP32, on
// v_mfma_f32_16x16x4_f32 (which adds its four k in order): a weight gradient of one co is the
// product [ci][pixel] x [pixel][tap], a data gradient [pixel][(tap, co)] x [(tap, co)][ci].
// Every sum of a sample is one chain in pixel (or tap) order, added to the workgroup's total
// afterwards, as a plain loop over the batch would: in training the sums over a batch cancel
// to 1e-4 of their terms and feed back into the weights, so a different order, no less exact,
// shows in the moments within tens of steps.  The long chains (layer 3's weights and the
// biases) run on waves of their own beside the others' work.  Gradients sit in LDS with a zero
// border, so that no tap needs a bounds test; rows are padded against bank conflicts.  A
// workgroup serves a run of samples and keeps the weight and bias gradients in registers; the
// partial sums of the workgroups are added in a fixed order afterwards.
// Bound by latency: 256 samples are one workgroup per CU, a chain of six phases.  Measured at
// 256 samples: 39 us and 5 us for the reduction, against 730 us for the separate kernels (weights 3
// x 117 us, whose bias sums ran on one thread, their reduction 3 x 64, data 3 x 58, masks).
constexpr int kBwdThreads = 576;   // eight waves and one for the bias sums
constexpr int BX2 = 32 * 32 + 4, BX1 = 16 * 16 + 4, BX0 = 64 + 4;    // channel strides of the layer inputs
constexpr int BL3 = 74, BL2 = 42, BL1 = 20;                          // row strides of the bordered gradients
constexpr int BG2 = 34 * BL2, BG1 = 18 * BL1;                        // channel strides of those
constexpr int kBwdR0 = (66 * BL3 > DC1 * BG1) ? 66 * BL3 : DC1 * BG1;   // gy, then layer 1's gradient
constexpr int kBwdLdsFloats = kBwdR0 + DC2 * BX2 + DC2 * BG2 + DC1 * BX1 + DC0 * BX0 + 128 * 16 + 4096;
static_assert(DC2 * BX2 >= 256 * 16, "K1 takes d2's place");
constexpr int kConvParams = 16 * 16 * 16 + 16 + 16 * 8 * 16 + 8 + 8 * 16 + 1;   // K1 c1 K2 c2 K3 c3, in layout order
static_assert(kBwdLdsFloats * 4 <= 160 * 1024, "one workgroup's LDS");
static_assert(DC0 == 16 && DC1 == 16 && DC2 == 8, "phases below assume these channels");

__global__ void __launch_bounds__(kBwdThreads) sg_decoder_bwd_kernel(
    const float* __restrict__ y, const float* __restrict__ t, const float* __restrict__ h3,
    const float* __restrict__ d1, const float* __restrict__ d2, const float* __restrict__ K1,
    const float* __restrict__ K2, const float* __restrict__ K3, int B, int chunk, float* __restrict__ gy,
    float* __restrict__ g3, float* __restrict__ partial, double* __restrict__ loss_partial) {
  extern __shared__ float bls[];
  float* r0 = bls;               // gy [66][BL3]; later layer 1's gradient [16][18][BL1]
  float* x2 = r0 + kBwdR0;       // d2 [8][BX2]; later K1 as [tap][co][ci]
  float* g2 = x2 + DC2 * BX2;    // layer 2's gradient [8][34][BL2]
  float* x1 = g2 + DC2 * BG2;    // d1 [16][BX1]
  float* x0 = x1 + DC1 * BX1;    // h3 [16][BX0]
  float* k2 = x0 + DC0 * BX0;    // K2 as [tap][co][ci]
  float* gyc = k2 + 128 * 16;    // gy without border, for the bias sum
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, g = lane >> 4, r16 = lane & 15;
  const int ky = r16 >> 2, kx = r16 & 3;   // the lane's tap as a column of a weight gradient
  const float scale = 2.f / (float)((size_t)B * 4096);
  const f4v_t zero4 = {0.f, 0.f, 0.f, 0.f};
  f4v_t a3 = zero4, a2 = zero4, a1[2] = {zero4, zero4};   // totals: wave 0, waves 0-7 (co = w), co = 2 w + u
  float k3[4];
#pragma unroll
  for (int st = 0; st < 4; ++st) k3[st] = r16 < 8 ? K3[r16 * 16 + 4 * st + g] : 0.f;
  float bias3 = 0.f, bias21 = 0.f;   // wave 8: c3; waves 4 and 5: c2 and c1 of column r16
  double lsum = 0.0;
  for (int i = tid; i < DC1 * 8 * 16; i += kBwdThreads) k2[((i & 15) * 8 + ((i >> 4) & 7)) * 16 + (i >> 7)] = K2[i];
  const int b0 = blockIdx.x * chunk, b1 = min(B, b0 + chunk);
  for (int b = b0; b < b1; ++b) {
    __syncthreads();   // the previous sample's (or the staging's) use of the buffers is over
    for (int i = tid; i < kBwdR0; i += kBwdThreads) r0[i] = 0.f;
    for (int i = tid; i < DC2 * BG2; i += kBwdThreads) g2[i] = 0.f;
    for (int i = 4 * tid; i < DC2 * 1024; i += 4 * kBwdThreads)
      *reinterpret_cast<float4*>(x2 + (i >> 10) * BX2 + (i & 1023)) =
          *reinterpret_cast<const float4*>(d2 + (size_t)b * DC2 * 1024 + i);
    for (int i = 4 * tid; i < DC1 * 256; i += 4 * kBwdThreads)
      *reinterpret_cast<float4*>(x1 + (i >> 8) * BX1 + (i & 255)) =
          *reinterpret_cast<const float4*>(d1 + (size_t)b * DC1 * 256 + i);
    for (int i = 4 * tid; i < DC0 * 64; i += 4 * kBwdThreads)
      *reinterpret_cast<float4*>(x0 + (i >> 6) * BX0 + (i & 63)) =
          *reinterpret_cast<const float4*>(h3 + (size_t)b * DC0 * 64 + i);
    __syncthreads();
    for (int i = 4 * tid; i < 4096; i += 4 * kBwdThreads) {
      const float4 yv = *reinterpret_cast<const float4*>(y + (size_t)b * 4096 + i);
      const float* tv = t + (size_t)b * 4096 + i;   // (the caller's array: 4-byte aligned)
      const float e[4] = {yv.x - tv[0], yv.y - tv[1], yv.z - tv[2], yv.w - tv[3]};
      float* o = r0 + ((i >> 6) + 1) * BL3 + (i & 63) + 1;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        o[q] = scale * e[q];
        lsum += (double)e[q] * e[q];
      }
      const float4 gv = make_float4(scale * e[0], scale * e[1], scale * e[2], scale * e[3]);
      *reinterpret_cast<float4*>(gyc + i) = gv;
      *reinterpret_cast<float4*>(gy + (size_t)b * 4096 + i) = gv;
    }
    __syncthreads();
    // ---- layer 3 (one output channel): wave 0 dK3 (rows ci 0-7), waves 1-7 gd2 (columns ci 0-7),
    // wave 8 the first part of the bias sum
    float c3s = 0.f;
    auto bias_run = [&](int i0, int i1) {
      float4 q[8], nq[8];   // 32 values ahead of the chain of additions
#pragma unroll
      for (int e = 0; e < 8; ++e) q[e] = *reinterpret_cast<const float4*>(gyc + i0 + 4 * e);
      for (int i = i0; i < i1; i += 32) {
#pragma unroll
        for (int e = 0; e < 8; ++e) nq[e] = *reinterpret_cast<const float4*>(gyc + min(i + 32, i1 - 32) + 4 * e);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          c3s += q[e].x;
          c3s += q[e].y;
          c3s += q[e].z;
          c3s += q[e].w;
          q[e] = nq[e];
        }
      }
    };
    if (w == 0) {
      f4v_t v = zero4;
#pragma unroll 8
      for (int st = 0; st < 256; ++st) {
        const int px = 4 * st + g, iy = px >> 5, ix = px & 31;
        v = __builtin_amdgcn_mfma_f32_16x16x4f32(x2[(r16 & 7) * BX2 + px], r0[(2 * iy + ky) * BL3 + 2 * ix + kx], v, 0,
                                                 0, 0);
      }
      a3 += v;
    } else if (w == 8) {
      bias_run(0, 1664);
    } else {
      for (int tl = w - 1; tl < 64; tl += 7) {   // 16 pixels of a row
        const int iy = tl >> 1, ix0 = 16 * (tl & 1);
        f4v_t v = zero4;
#pragma unroll
        for (int st = 0; st < 4; ++st)   // k = 4 st + g: ky = st, kx = g
          v = __builtin_amdgcn_mfma_f32_16x16x4f32(r0[(2 * iy + st) * BL3 + 2 * (ix0 + r16) + g], k3[st], v, 0, 0, 0);
        if (r16 < 8)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int ix = ix0 + 4 * g + r;
            g2[r16 * BG2 + (iy + 1) * BL2 + ix + 1] = x2[r16 * BX2 + 32 * iy + ix] > 0.f ? v[r] : 0.f;
          }
      }
    }
    __syncthreads();
    // gy and d2 are done with: layer 1's gradient and K1 take their place
    for (int i = tid; i < DC1 * BG1; i += kBwdThreads) r0[i] = 0.f;
    for (int i = tid; i < DC0 * 256; i += kBwdThreads) x2[((i & 15) * 16 + ((i >> 4) & 15)) * 16 + (i >> 8)] = K1[i];
    // ---- layer 2: wave w < 8 takes co = w of dK2, then image rows 2 w, 2 w + 1 of all ci of gd1
    f4v_t d[2] = {zero4, zero4};
    if (w == 8) {
      bias_run(1664, 2688);
    } else {
      f4v_t v = zero4;
#pragma unroll 4
      for (int st = 0; st < 64; ++st) {
        const int px = 4 * st + g, iy = px >> 4, ix = px & 15;
        v = __builtin_amdgcn_mfma_f32_16x16x4f32(x1[r16 * BX1 + px], g2[w * BG2 + (2 * iy + ky) * BL2 + 2 * ix + kx], v,
                                                 0, 0, 0);
      }
      a2 += v;
#pragma unroll 4
      for (int st = 0; st < 32; ++st) {   // k = 4 st + g: tap st / 2, co = 4 (st % 2) + g
        const float kv = k2[(4 * st + g) * 16 + r16];
        const float* gp = g2 + (4 * (st & 1) + g) * BG2 + (4 * w + (st >> 3)) * BL2 + 2 * r16 + ((st >> 1) & 3);
#pragma unroll
        for (int u = 0; u < 2; ++u) d[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(gp[2 * u * BL2], kv, d[u], 0, 0, 0);
      }
    }
    __syncthreads();   // layer 1's buffer is zeroed
    if (w < 8)
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int iy = 2 * w + u, ix = 4 * g + r;
          r0[r16 * BG1 + (iy + 1) * BL1 + ix + 1] = x1[r16 * BX1 + 16 * iy + ix] > 0.f ? d[u][r] : 0.f;
        }
    __syncthreads();
    // ---- layer 1: wave w < 8 takes co = 2 w, 2 w + 1 of dK1, waves 0-3 then 16 pixels of g3 each
    // (before its mask: the basis branch adds to it), waves 4 and 5 the biases of layers 2 and 1
    if (w == 8) {
      bias_run(2688, 4096);
      bias3 += c3s;
    } else {
      f4v_t v[2] = {zero4, zero4};
#pragma unroll 4
      for (int st = 0; st < 16; ++st) {
        const int px = 4 * st + g, iy = px >> 3, ix = px & 7;
        const float av = x0[r16 * BX0 + px];
#pragma unroll
        for (int u = 0; u < 2; ++u)
          v[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(
              av, r0[(2 * w + u) * BG1 + (2 * iy + ky) * BL1 + 2 * ix + kx], v[u], 0, 0, 0);
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) a1[u] += v[u];
      if (w < 4) {
        const int px = 16 * w + r16, iy = px >> 3, ix = px & 7;
        f4v_t q = zero4;
#pragma unroll 8
        for (int st = 0; st < 64; ++st)   // k = 4 st + g: tap st / 4, co = 4 (st % 4) + g
          q = __builtin_amdgcn_mfma_f32_16x16x4f32(
              r0[(4 * (st & 3) + g) * BG1 + (2 * iy + (st >> 4)) * BL1 + 2 * ix + ((st >> 2) & 3)],
              x2[(4 * st + g) * 16 + r16], q, 0, 0, 0);
        *reinterpret_cast<float4*>(g3 + (size_t)b * 1024 + r16 * 64 + 16 * w + 4 * g) =
            make_float4(q[0], q[1], q[2], q[3]);
      } else if (w < 6) {
        // biases: a product with rows of ones adds the pixels (k) of each co (column) in order
        f4v_t q = zero4;
        if (w == 4) {
          const float* gp = g2 + (r16 & 7) * BG2 + BL2 + 1 + g;
#pragma unroll 8
          for (int st = 0; st < 256; ++st)
            q = __builtin_amdgcn_mfma_f32_16x16x4f32(1.f, gp[(st >> 3) * BL2 + 4 * (st & 7)], q, 0, 0, 0);
        } else {
          const float* gp = r0 + r16 * BG1 + BL1 + 1 + g;
#pragma unroll 8
          for (int st = 0; st < 64; ++st)
            q = __builtin_amdgcn_mfma_f32_16x16x4f32(1.f, gp[(st >> 2) * BL1 + 4 * (st & 3)], q, 0, 0, 0);
        }
        bias21 += q[0];
      }
    }
  }
  // ---- this workgroup's partial sums
  __syncthreads();
  float* dst = partial + (size_t)blockIdx.x * kConvParams;
  if (w == 4 && lane < 8) dst[4096 + 16 + 2048 + lane] = bias21;
  if (w == 5 && lane < 16) dst[4096 + lane] = bias21;
  if (w == 8) {
    if (lane == 0) dst[kConvParams - 1] = bias3;
  } else {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int ci = 4 * g + r;
#pragma unroll
      for (int u = 0; u < 2; ++u) dst[(ci * 16 + 2 * w + u) * 16 + r16] = a1[u][r];
      dst[4096 + 16 + (ci * 8 + w) * 16 + r16] = a2[r];
      if (w == 0 && ci < 8) dst[4096 + 16 + 2048 + 8 + ci * 16 + r16] = a3[r];
    }
  }
  double* ld = reinterpret_cast<double*>(bls);
  ld[tid] = lsum;
  __syncthreads();
  if (tid < 64) {
    double v = 0.0;
    for (int q = 0; q < kBwdThreads / 64; ++q) v += ld[tid + 64 * q];
    ld[tid] = v;
  }
  __syncthreads();
  if (tid == 0) {
    double v = 0.0;
    for (int q = 0; q < 64; ++q) v += ld[q];
    loss_partial[blockIdx.x] = v;
  }
}

// out[p] = sum over chunks of partial[chunk][p], FP64, in a fixed order (eight runs of chunks,
// then the runs); the last workgroup sums the loss partials the same way.
__global__ void __launch_bounds__(256) sg_reduce_partials_kernel(const float* __restrict__ partial, int chunks, int n,
                                                                 float* __restrict__ out,
                                                                 const double* __restrict__ loss_partial,
                                                                 double inv, float* __restrict__ loss) {
  __shared__ double red[256];
  const int tid = threadIdx.x, l = tid & 31, run = tid >> 5;
  const bool lossy = blockIdx.x == gridDim.x - 1;
  const int p = blockIdx.x * 32 + l;
  const int per = (chunks + 7) / 8, c0 = run * per, c1 = min(chunks, c0 + per);
  double s = 0.0;
  if (lossy) {
    for (int c = tid; c < chunks; c += 256) s += loss_partial[c];
  } else if (p < n) {
#pragma unroll 8
    for (int c = c0; c < c1; ++c) s += partial[(size_t)c * n + p];
  }
  red[tid] = s;
  __syncthreads();
  if (lossy) {
    for (int h = 128; h > 0; h >>= 1) {
      if (tid < h) red[tid] += red[tid + h];
      __syncthreads();
    }
    if (tid == 0 && loss) loss[0] = (float)(red[0] * inv);
  } else if (run == 0 && p < n) {
    s = red[l];
    for (int q = 1; q < 8; ++q) s += red[32 * q + l];
    out[p] = (float)s;
  }
}

__global__ void sg_adam_kernel(float* __restrict__ w, const float* __restrict__ g, float* __restrict__ m,
                               float* __restrict__ v, size_t n, float lr, float b1, float b2, float eps,
                               float c1, float c2) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  w[i] -= lr * (mi * c1) / (sqrtf(vi * c2) + eps);
}

}  // namespace rw

// ---------------------------------------------------------------- host side
namespace {
constexpr int kBasis = 256;   // rank of the linear crop basis
struct Layout {
  size_t W1, b1, W2, b2, W3, b3, K1, c1, K2, c2, K3, c3, Wa, ba, Wb, bb, total;
};
Layout layout() {
  Layout L{};
  size_t o = 0;
  auto take = [&](size_t n) { size_t r = o; o += n; return r; };
  L.W1 = take(22 * 1024); L.b1 = take(1024);
  L.W2 = take(1024 * 1024); L.b2 = take(1024);
  L.W3 = take(1024 * 1024); L.b3 = take(1024);
  L.K1 = take(16 * 16 * 16); L.c1 = take(16);
  L.K2 = take(16 * 8 * 16); L.c2 = take(8);
  L.K3 = take(8 * 1 * 16); L.c3 = take(1);
  L.Wa = take(1024 * kBasis); L.ba = take(kBasis);
  L.Wb = take(kBasis * 4096); L.bb = take(4096);
  L.total = o;
  return L;
}
constexpr int kMaxChunks = 256;   // partial sums of the convolution weight gradients per step
constexpr size_t kSplitKFloats = (size_t)16 << 20;   // split-K workspace of the training products
}  // namespace

struct rwpsf_sg {
  int device = 0, max_batch = 0;
  Layout L{};
  std::vector<void*> allocations;
  float *w = nullptr, *g = nullptr, *m = nullptr, *v = nullptr;   // [L.total]
  float *x = nullptr, *h1 = nullptr, *h2 = nullptr, *h3 = nullptr, *d1 = nullptr, *d2 = nullptr, *y = nullptr;
  float *g1 = nullptr, *g2 = nullptr, *g3 = nullptr, *gy = nullptr;
  float *a = nullptr, *ga = nullptr;   // basis coefficients [B][kBasis] and their gradient
  float* partial = nullptr;   // conv weight partials
  __bf16* decw = nullptr;     // B fragments of the decoder's matrix-core layers (hi / lo)
  int num_cus = 0;
  __bf16* wsplit = nullptr;   // BF16 hi / lo planes of W2, W3, Wa, Wb, [N][K]
  __bf16* wsplit_t = nullptr; // the same weights split in their own order (operands of g W^T)
  float* ws = nullptr;        // split-K partial products
  double* loss_partial = nullptr;
  int64_t step = 0;
  ~rwpsf_sg() {   // teardown: failures cannot be reported and are ignored
    for (void* p : allocations) (void)hipFree(p);
  }
};

namespace rw {

template <class T>
static int sg_alloc(rwpsf_sg* s, T** p, size_t count) {
  void* d = nullptr;
  hipError_t e = hipMalloc(&d, std::max<size_t>(16, count * sizeof(T)));
  if (e != hipSuccess) {
    set_hip_error(e);
    return RWPSF_ERR_OOM;
  }
  s->allocations.push_back(d);
  *p = (T*)d;
  return RWPSF_OK;
}

// Operand planes: [N][K] of W2, W3, Wa, Wb (t: hi, lo of each) in wsplit, the same weights in
// their own order (o) in wsplit_t, and the decoder's fragments.
struct SgPlanes {
  __bf16 *t[8], *o[8];
  __bf16 *f1h, *f1l, *f2h, *f2l;
};
static SgPlanes sg_plane_ptrs(const rwpsf_sg* s) {
  const size_t n[4] = {1024 * 1024, 1024 * 1024, 1024 * (size_t)kBasis, (size_t)kBasis * 4096};
  SgPlanes P;
  size_t at = 0;
  for (int i = 0; i < 4; ++i)
    for (int q = 0; q < 2; ++q) {
      P.t[2 * i + q] = s->wsplit + at;
      P.o[2 * i + q] = s->wsplit_t + at;
      at += n[i];
    }
  P.f1h = s->decw;
  P.f1l = P.f1h + 4 * DK1 * 64 * 8;
  P.f2h = P.f1l + 4 * DK1 * 64 * 8;
  P.f2l = P.f2h + 2 * DK2 * 64 * 8;
  return P;
}

// Bring the operand planes up to date with the weights.
static int sg_update_planes(rwpsf_sg* s, hipStream_t st) {
  const Layout& L = s->L;
  const SgPlanes P = sg_plane_ptrs(s);
  const struct { size_t off; int K, N; } m[4] = {{L.W2, 1024, 1024}, {L.W3, 1024, 1024}, {L.Wa, 1024, kBasis}, {L.Wb, kBasis, 4096}};
  PlaneArgs a{};
  for (int i = 0; i < 4; ++i) {
    a.job[i] = PlaneJob{s->w + m[i].off, P.o[2 * i], P.o[2 * i + 1], P.t[2 * i], P.t[2 * i + 1], m[i].K, m[i].N, a.tiles};
    a.tiles += m[i].K / 32 * (m[i].N / 32);
  }
  a.K1 = s->w + L.K1;
  a.K2 = s->w + L.K2;
  a.f1h = P.f1h;
  a.f1l = P.f1l;
  a.f2h = P.f2h;
  a.f2l = P.f2l;
  const int frags = (4 * DK1 + 2 * DK2) * 64 * 8;
  hipLaunchKernelGGL(sg_planes_kernel, dim3(a.tiles + (frags + 255) / 256), dim3(256), 0, st, a);
  return hip_check(hipGetLastError());
}

// keep: also write d1 and d2 (the backward pass needs them)
static int sg_forward_impl(rwpsf_sg* s, int B, const float* coef, const float* z, float* out, int nsplit,
                           bool keep, hipStream_t st) {
  const Layout& L = s->L;
  int rc;
  // (W1 is the first parameter block, so its rows are 16-byte aligned)
  const int rows = std::max(2, std::min(kDense1Rows, B / (2 * s->num_cus)));
  hipLaunchKernelGGL(sg_dense1_kernel, dim3((B + rows - 1) / rows), dim3(256), 0, st, coef, z, s->w + L.W1,
                     s->w + L.b1, B, rows, s->x, s->h1);
  if ((rc = hip_check(hipGetLastError()))) return rc;
  const SgPlanes P = sg_plane_ptrs(s);
  const __bf16 *w2h = P.t[0], *w2l = P.t[1], *w3h = P.t[2], *w3l = P.t[3];
  const __bf16 *wah = P.t[4], *wal = P.t[5], *wbh = P.t[6], *wbl = P.t[7];
  if ((rc = hip_check(sg_gemm_fast(s->h1, w2h, w2l, s->h2, B, 1024, 1024, s->w + L.b2, 1, nsplit, st)))) return rc;
  if ((rc = hip_check(sg_gemm_fast(s->h2, w3h, w3l, s->h3, B, 1024, 1024, s->w + L.b3, 1, nsplit, st)))) return rc;
  // basis branch (linear): a = h3 Wa + ba, out = a Wb + bb; the decoder then adds its output
  if ((rc = hip_check(sg_gemm_fast(s->h3, wah, wal, s->a, B, kBasis, 1024, s->w + L.ba, 0, nsplit, st)))) return rc;
  if ((rc = hip_check(sg_gemm_fast(s->a, wbh, wbl, out, B, 4096, kBasis, s->w + L.bb, 0, nsplit, st)))) return rc;
  // decoder: one persistent launch
  const int grid = std::min(B, 2 * s->num_cus);
  const bf8_t* F1h = reinterpret_cast<const bf8_t*>(P.f1h);
  const bf8_t* F1l = reinterpret_cast<const bf8_t*>(P.f1l);
  const bf8_t* F2h = reinterpret_cast<const bf8_t*>(P.f2h);
  const bf8_t* F2l = reinterpret_cast<const bf8_t*>(P.f2l);
  float* d1 = keep ? s->d1 : nullptr;
  float* d2 = keep ? s->d2 : nullptr;
  if (nsplit > 1)
    hipLaunchKernelGGL(sg_decoder_kernel<3>, dim3(grid), dim3(256), kDecLdsBytes, st, s->h3, B, F1h, F1l, F2h, F2l,
                       s->w + L.c1, s->w + L.c2, s->w + L.K3, s->w + L.c3, out, d1, d2);
  else
    hipLaunchKernelGGL(sg_decoder_kernel<1>, dim3(grid), dim3(256), kDecLdsBytes, st, s->h3, B, F1h, F1l, F2h, F2l,
                       s->w + L.c1, s->w + L.c2, s->w + L.K3, s->w + L.c3, out, d1, d2);
  return hip_check(hipGetLastError());
}

static int sg_backward_impl(rwpsf_sg* s, int B, const float* target, float* loss, hipStream_t st) {
  const Layout& L = s->L;
  int rc;
  // loss gradient and the convolution branch
  const int chunk = (B + kMaxChunks - 1) / kMaxChunks;   // samples per partial sum
  const int chunks = (B + chunk - 1) / chunk;
  hipLaunchKernelGGL(sg_decoder_bwd_kernel, dim3(chunks), dim3(kBwdThreads), kBwdLdsFloats * sizeof(float), st, s->y,
                     target, s->h3, s->d1, s->d2, s->w + L.K1, s->w + L.K2, s->w + L.K3, B, chunk, s->gy, s->g3,
                     s->partial, s->loss_partial);
  if ((rc = hip_check(hipGetLastError()))) return rc;
  // (the convolution parameters K1 c1 K2 c2 K3 c3 are adjacent in the layout)
  hipLaunchKernelGGL(sg_reduce_partials_kernel, dim3((kConvParams + 31) / 32 + 1), dim3(256), 0, st, s->partial, chunks,
                     kConvParams, s->g + L.K1, s->loss_partial, 1.0 / ((double)B * 4096.0), loss);
  if ((rc = hip_check(hipGetLastError()))) return rc;
  // gradients down the dense layers: ga = gy Wb^T; g3 += ga Wa^T (h3 feeds both branches), then
  // g2 = g3 W3^T and g1 = g2 W2^T, each masked by its layer's relu
  const SgPlanes P = sg_plane_ptrs(s);
  const int twg = 2 * s->num_cus;
  if ((rc = hip_check(sg_gemm_fast(s->gy, P.o[6], P.o[7], s->ga, B, kBasis, 4096, nullptr, 0, 3, st, 0, nullptr, s->ws,
                                   kSplitKFloats, twg))) ||
      (rc = hip_check(sg_gemm_fast(s->ga, P.o[4], P.o[5], s->g3, B, 1024, kBasis, nullptr, 0, 3, st, 1, s->h3, s->ws,
                                   kSplitKFloats, twg))) ||
      (rc = hip_check(sg_gemm_fast(s->g3, P.o[2], P.o[3], s->g2, B, 1024, 1024, nullptr, 0, 3, st, 0, s->h2, s->ws,
                                   kSplitKFloats, twg))) ||
      (rc = hip_check(sg_gemm_fast(s->g2, P.o[0], P.o[1], s->g1, B, 1024, 1024, nullptr, 0, 3, st, 0, s->h1, s->ws,
                                   kSplitKFloats, twg))))
    return rc;
  // dW = hin^T gout and db of all five dense layers
  const struct { const float *hin, *gout; size_t W, b; int M, N; } dw[kDwJobs] = {
      {s->a, s->gy, L.Wb, L.bb, kBasis, 4096}, {s->h2, s->g3, L.W3, L.b3, 1024, 1024},
      {s->h1, s->g2, L.W2, L.b2, 1024, 1024}, {s->h3, s->ga, L.Wa, L.ba, 1024, kBasis},
      {s->x, s->g1, L.W1, L.b1, 22, 1024}};
  DwArgs da{};
  da.K = B;
  int tiles = 0;
  for (int i = 0; i < kDwJobs; ++i) {
    da.job[i] = DwJob{dw[i].hin, dw[i].gout, s->g + dw[i].W, s->g + dw[i].b, dw[i].M, dw[i].N, tiles};
    tiles += (dw[i].M + 63) / 64 * (dw[i].N / 64);
  }
  hipLaunchKernelGGL(sg_dw_kernel, dim3(tiles), dim3(256), 4 * kDwPlane, st, da);
  return hip_check(hipGetLastError());
}

}  // namespace rw

extern "C" {

size_t rwpsf_sg_param_count(void) { return layout().total; }

int rwpsf_sg_create(int max_batch, rwpsf_sg** out) {
  using namespace rw;
  if (!out || max_batch < 1 || max_batch > (1 << 20)) return RWPSF_ERR_INVALID_ARG;
  *out = nullptr;
  int dev_count = 0;
  if (hipGetDeviceCount(&dev_count) != hipSuccess || dev_count < 1) return RWPSF_ERR_NO_DEVICE;
  rwpsf_sg* s = new (std::nothrow) rwpsf_sg();
  if (!s) return RWPSF_ERR_OOM;
  if (hipGetDevice(&s->device) != hipSuccess) {
    delete s;
    return RWPSF_ERR_NO_DEVICE;
  }
  s->max_batch = max_batch;
  s->L = layout();
  const size_t P = s->L.total, B = (size_t)max_batch;
  const int chunks = std::min(max_batch, kMaxChunks);
  int rc;
  if ((rc = sg_alloc(s, &s->w, P)) || (rc = sg_alloc(s, &s->g, P)) || (rc = sg_alloc(s, &s->m, P)) ||
      (rc = sg_alloc(s, &s->v, P)) || (rc = sg_alloc(s, &s->x, B * 22)) || (rc = sg_alloc(s, &s->h1, B * 1024)) ||
      (rc = sg_alloc(s, &s->h2, B * 1024)) || (rc = sg_alloc(s, &s->h3, B * 1024)) ||
      (rc = sg_alloc(s, &s->d1, B * 4096)) || (rc = sg_alloc(s, &s->d2, B * 8192)) ||
      (rc = sg_alloc(s, &s->y, B * 4096)) ||
      (rc = sg_alloc(s, &s->g1, B * 1024)) || (rc = sg_alloc(s, &s->g2, B * 1024)) ||
      (rc = sg_alloc(s, &s->g3, B * 1024)) || (rc = sg_alloc(s, &s->gy, B * 4096)) ||
      (rc = sg_alloc(s, &s->partial, (size_t)chunks * kConvParams)) ||
      (rc = sg_alloc(s, &s->loss_partial, 256)) || (rc = sg_alloc(s, &s->decw, 2 * (4 * DK1 + 2 * DK2) * 64 * 8)) ||
      (rc = sg_alloc(s, &s->a, B * kBasis)) || (rc = sg_alloc(s, &s->ga, B * kBasis)) ||
      (rc = sg_alloc(s, &s->wsplit, 2 * (1024 * 1024 + 1024 * 1024 + 1024 * kBasis + kBasis * 4096))) ||
      (rc = sg_alloc(s, &s->wsplit_t, 2 * (1024 * 1024 + 1024 * 1024 + 1024 * kBasis + kBasis * 4096))) ||
      (rc = sg_alloc(s, &s->ws, kSplitKFloats))) {
    delete s;
    return rc;
  }
  if (hipDeviceGetAttribute(&s->num_cus, hipDeviceAttributeMultiprocessorCount, s->device) != hipSuccess ||
      s->num_cus < 1) {
    delete s;
    return RWPSF_ERR_NO_DEVICE;
  }
  const int fast_lds = 2 * 4 * FBM * FLD * (int)sizeof(__bf16);
  const struct { const void* k; int bytes; } lds[] = {
      {(const void*)sg_gemm_fast_kernel<1>, fast_lds}, {(const void*)sg_gemm_fast_kernel<3>, fast_lds},
      {(const void*)sg_dw_kernel, 4 * kDwPlane}, {(const void*)sg_decoder_bwd_kernel, kBwdLdsFloats * 4},
      {(const void*)sg_decoder_kernel<1>, kDecLdsBytes}, {(const void*)sg_decoder_kernel<3>, kDecLdsBytes}};
  for (const auto& l : lds)
    if ((rc = hip_check(hipFuncSetAttribute(l.k, hipFuncAttributeMaxDynamicSharedMemorySize, l.bytes)))) {
      delete s;
      return rc;
    }
  if ((rc = hip_check(hipMemset(s->m, 0, P * sizeof(float)))) || (rc = hip_check(hipMemset(s->v, 0, P * sizeof(float)))) ||
      (rc = hip_check(hipMemset(s->w, 0, P * sizeof(float)))) || (rc = sg_update_planes(s, nullptr)) ||
      (rc = hip_check(hipDeviceSynchronize()))) {
    delete s;
    return rc;
  }
  *out = s;
  return RWPSF_OK;
}

void rwpsf_sg_destroy(rwpsf_sg* s) {   // teardown: HIP failures are ignored
  if (!s) return;
  (void)hipDeviceSynchronize();
  delete s;
}

int rwpsf_sg_set_state(rwpsf_sg* s, const float* w, const float* m, const float* v, int64_t step) {
  if (!s || !w) return RWPSF_ERR_INVALID_ARG;
  const size_t bytes = s->L.total * sizeof(float);
  int rc;
  if ((rc = rw::hip_check(hipMemcpy(s->w, w, bytes, hipMemcpyHostToDevice)))) return rc;
  if (m && (rc = rw::hip_check(hipMemcpy(s->m, m, bytes, hipMemcpyHostToDevice)))) return rc;
  if (v && (rc = rw::hip_check(hipMemcpy(s->v, v, bytes, hipMemcpyHostToDevice)))) return rc;
  s->step = step;
  // on the null stream of the handle's device; the caller's next stream may not order after it
  int cur = 0;
  if ((rc = rw::hip_check(hipGetDevice(&cur))) || (rc = rw::hip_check(hipSetDevice(s->device)))) return rc;
  rc = rw::sg_update_planes(s, nullptr);
  if (!rc) rc = rw::hip_check(hipDeviceSynchronize());
  const int back = rw::hip_check(hipSetDevice(cur));
  return rc ? rc : back;
}

int rwpsf_sg_get_state(const rwpsf_sg* s, float* w, float* m, float* v, float* g, int64_t* step) {
  if (!s) return RWPSF_ERR_INVALID_ARG;
  const size_t bytes = s->L.total * sizeof(float);
  int rc;
  if ((rc = rw::hip_check(hipDeviceSynchronize()))) return rc;
  if (w && (rc = rw::hip_check(hipMemcpy(w, s->w, bytes, hipMemcpyDeviceToHost)))) return rc;
  if (m && (rc = rw::hip_check(hipMemcpy(m, s->m, bytes, hipMemcpyDeviceToHost)))) return rc;
  if (v && (rc = rw::hip_check(hipMemcpy(v, s->v, bytes, hipMemcpyDeviceToHost)))) return rc;
  if (g && (rc = rw::hip_check(hipMemcpy(g, s->g, bytes, hipMemcpyDeviceToHost)))) return rc;
  if (step) *step = s->step;
  return RWPSF_OK;
}

int rwpsf_sg_forward(rwpsf_sg* s, int B, const float* coef, const float* z, float* out, int precision,
                     void* stream) {
  if (!s || B < 1 || B > s->max_batch || !coef || !z || !out) return RWPSF_ERR_INVALID_ARG;
  if (precision != RWPSF_SG_BF16X3 && precision != RWPSF_SG_BF16) return RWPSF_ERR_INVALID_ARG;
  return rw::sg_forward_impl(s, B, coef, z, out, precision == RWPSF_SG_BF16X3 ? 3 : 1, false, (hipStream_t)stream);
}

int rwpsf_sg_gradient(rwpsf_sg* s, int B, const float* coef, const float* z, const float* target, float* loss,
                      void* stream) {
  if (!s || B < 1 || B > s->max_batch || !coef || !z || !target) return RWPSF_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  int rc = rw::sg_forward_impl(s, B, coef, z, s->y, 3, true, st);
  if (rc) return rc;
  return rw::sg_backward_impl(s, B, target, loss, st);
}

int rwpsf_sg_error_features(int B, const float* coef, const float* z, float* phi, void* stream) {
  if (B < 1 || !coef || !z || !phi) return RWPSF_ERR_INVALID_ARG;
  const long long n = (long long)B * rw::kGateFeatures;
  hipLaunchKernelGGL(rw::sg_gate_features_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0,
                     (hipStream_t)stream, coef, z, B, phi);
  return rw::hip_check(hipGetLastError());
}

int rwpsf_sg_error_predict(int B, const float* coef, const float* z, const float* weights, float* log_err,
                           void* stream) {
  if (B < 1 || !coef || !z || !weights || !log_err) return RWPSF_ERR_INVALID_ARG;
  hipLaunchKernelGGL(rw::sg_gate_predict_kernel, dim3((B + 255) / 256), dim3(256), 0, (hipStream_t)stream, coef, z, B,
                     weights, log_err);
  return rw::hip_check(hipGetLastError());
}

int rwpsf_sg_adam(rwpsf_sg* s, float lr, float beta1, float beta2, float eps, void* stream) {
  if (!s || !(lr > 0) || !(beta1 >= 0 && beta1 < 1) || !(beta2 >= 0 && beta2 < 1) || !(eps > 0))
    return RWPSF_ERR_INVALID_ARG;
  s->step += 1;
  const float c1 = (float)(1.0 / (1.0 - std::pow((double)beta1, (double)s->step)));
  const float c2 = (float)(1.0 / (1.0 - std::pow((double)beta2, (double)s->step)));
  const size_t n = s->L.total;
  hipLaunchKernelGGL(rw::sg_adam_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream, s->w,
                     s->g, s->m, s->v, n, lr, beta1, beta2, eps, c1, c2);
  const int rc = rw::hip_check(hipGetLastError());
  return rc ? rc : rw::sg_update_planes(s, (hipStream_t)stream);
}

}  // extern "C"
