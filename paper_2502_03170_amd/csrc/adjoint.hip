// Hand-written adjoint of the Fourier form.
//
// Forward (per stack b, plane z, component c): E = Ax' P~ Ay^T with
// P~ = P_{b,c} exp(i k s_z z), P_{b,c} = Q_c exp(i Phi_b) (read from the forward's
// mirror-folded pupils: each lane recovers its own mirror cell from the four parities).
// For a real loss L(I), I = sum_c |E_c|^2, with g = dL/dI:
//   dL/dPhi[j,l] = sum_{b,z,c} Im( G[j,l] conj(P~[j,l]) ),  G = Ax'^H (2 g E) conj(Ay)
//   dL/dW0 = dL/dPhi,  dL/dc_q = 2 pi sum_cells dL/dPhi Z_q.
// The pupil grid is mirror-symmetric (s[N-1-j] = -s[j]), so with theta = k s_jf x_m and
// phi = k s_lf y_n (jf, lf < N/2 the folded indices, j' = N-1-jf, l' = N-1-lf):
//   H[m][lf], H[m][l'] = Hc -+ i Hs,   Hc, Hs = sum_n (2 g E)[m][n] {cos, sin} phi
//   G = i pref (CC -+ i CS -+ i SC ...)  with  CC = sum_m cos theta Hc, CS = sum_m cos theta Hs,
//   SC = sum_m sin theta Hc, SS = sum_m sin theta Hs (pref = f k / 2 pi), i.e.
//   G[jf,lf] = i pref (CC - iCS - iSC - SS)    G[jf,l'] = i pref (CC + iCS - iSC + SS)
//   G[j',lf] = i pref (CC - iCS + iSC + SS)    G[j',l'] = i pref (CC + iCS + iSC - SS)
// Kernels:
//   adj_scale_kernel  the power of two of each plane of 2 g E (its operand halves are f16)
//   adj_kernel        both contractions as real GEMMs on the F16 matrix cores with split
//                     operands (hgemm.h), H in LDS; sums CC .. SS conj(exp(i k s_z z)) over a run
//                     of planes, then takes mirrors and pupil: one partial of dL/dPhi per
//                     (stack, component, run), no atomics
//   adj_reduce_*      dL/dPhi = sum of the partials in a fixed order (FP64), dL/dW0
//   adj_zernike_kernel dL/dc_q by a fixed-shape tree reduction (FP64)
// The result does not depend on scheduling: every sum runs in a fixed order.
#include <algorithm>
#include <cmath>
#include <complex>
#include <vector>

#include "hgemm.h"
#include "rw_common.h"
#include "rw_fourier.h"
#include "rw_plan.h"

namespace rw {

// Wide loads of the caller's arrays, which are aligned as their elements are (the hardware takes any
// multiple of four bytes).
typedef float any4 __attribute__((ext_vector_type(4), aligned(4)));
typedef float any2 __attribute__((ext_vector_type(2), aligned(4)));

constexpr int kScalePixels = 4096, kScaleGroups = 1024;   // scales of the planes: pixels of a workgroup, workgroups
constexpr int kAdjStacks = 64;    // stacks per launch (their z offsets are passed by value)
constexpr int kAdjThreads = 512;  // eight waves
constexpr int kAdjCols = 32;      // folded y cells per workgroup
constexpr int kAdjChunk = 64;     // pixels per chunk, along x and along y
constexpr int kAdjPanel = kAdjChunk * 128 * 4;   // bytes of the field and of the H panel
constexpr int kAdjTab = kAdjChunk * 2 * kAdjCols * 4;
constexpr int kAdjRows = 256;     // folded x rows 2jf + p per workgroup, 32 a wave
constexpr int kAdjLds = 2 * kAdjPanel + kAdjTab + kAdjChunk * kAdjRows * 4;

// Split-f16 panel of one axis' folded table for contractions over its pixels, [pixel / 16]
// [piece][col][8 halves], 2^kTabExp {cos, sin}(k s_f x): columns 2f + p, or with `blocks` runs of
// 32 cells of one p, 64 (f / 32) + 32 p + f % 32.  Zero for f >= ceil(N / 2).
__global__ void adj_panel_kernel(_Float16* __restrict__ panel, int pixels, int n, int w, double k, double s_max,
                                 double pitch, int blocks) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= pixels * (w / 2)) return;
  const int x = idx % pixels, f = idx / pixels;
  double v[2] = {0.0, 0.0};
  if (f < (n + 1) / 2) {
    const double ph = k * ((2.0 * f + 1.0 - n) * s_max / n) * ((double)(x - pixels / 2) * pitch);
    sincos(ph, &v[1], &v[0]);
  }
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const double y = ldexp(v[p], kTabExp);
    const int col = blocks ? 64 * (f / 32) + 32 * p + f % 32 : 2 * f + p;
    _Float16* o = panel + ((size_t)(x / 16 * 4 + x % 16 / 8) * w + col) * 8 + x % 8;
    const _Float16 hi = (_Float16)(float)y;
    o[0] = hi;
    o[(size_t)2 * w * 8] = (_Float16)(float)(y - (double)(float)hi);
  }
}

// exp(i k s_z z) of every plan plane on the folded cells (FP64 phase reduced mod 2 pi before the
// FP32 sincos); 1 where k s_z is 0.
__global__ void adj_defocus_kernel(const double* __restrict__ kszf, const double* __restrict__ z, int nz, int cells,
                                   float2* __restrict__ D) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)nz * cells) return;
  const int zi = (int)(idx / cells), cell = (int)(idx % cells);
  float sn, cs;
  sincosf((float)reduce_2pi(kszf[cell] * z[zi]), &sn, &cs);
  D[idx] = make_float2(cs, sn);
}

// Scale of every (stack, plane, component): the exponent e that puts the largest part x of 2 g E 2^e
// in [2^13, 2^14), 0 for an empty or not finite plane.
__device__ __forceinline__ int adj_exponent(float x) {
  int b = 0;
  if (!(x > 0.f && x < INFINITY)) return 0;
  frexpf(x, &b);   // x in [2^(b-1), 2^b)
  return 14 - b;
}

// The largest parts of a plane: `parts` workgroups per (stack, plane), each a run of its pixels
// (a multiple of 4 in all).  One writes the plane's scales, several their maxima for adj_exponent_kernel.
// Bound by its loads in flight: a call of few, large planes needs several workgroups a plane (2 planes
// of 512 x 512 pixels: 181 us with one workgroup a plane, 6.4 with 64; 10 of 256 x 256: 49 us, 6.4
// with 16).
__global__ void __launch_bounds__(256) adj_scale_kernel(const float2* __restrict__ E, const float* __restrict__ g,
                                                        int pixels, int parts, int* __restrict__ ex,
                                                        float* __restrict__ maxima) {
  const size_t item = blockIdx.x / parts;
  const any4* e4 = reinterpret_cast<const any4*>(E + item * 3 * pixels);
  const any2* g2 = reinterpret_cast<const any2*>(g + item * pixels);
  const int pairs = pixels / 2, run = (pairs + parts - 1) / parts;
  const int i0 = (blockIdx.x % parts) * run, i1 = min(pairs, i0 + run);
  float m[3] = {0.f, 0.f, 0.f};
  for (int i = i0 + threadIdx.x; i < i1; i += 256) {
    const any2 f = g2[i];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const any4 v = e4[(size_t)c * pairs + i];
      m[c] = fmaxf(m[c], fmaxf(fmaxf(fabsf(2.f * f.x * v.x), fabsf(2.f * f.x * v.y)),
                               fmaxf(fabsf(2.f * f.y * v.z), fabsf(2.f * f.y * v.w))));
    }
  }
  __shared__ float red[3][4];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) m[c] = fmaxf(m[c], __shfl_xor(m[c], d));
    if ((threadIdx.x & 63) == 0) red[c][threadIdx.x >> 6] = m[c];
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    const float* r = red[threadIdx.x];
    const float x = fmaxf(fmaxf(r[0], r[1]), fmaxf(r[2], r[3]));
    if (parts == 1)
      ex[item * 3 + threadIdx.x] = adj_exponent(x);
    else
      maxima[(size_t)blockIdx.x * 3 + threadIdx.x] = x;
  }
}

// The scales from the maxima of the runs: one thread per (stack, plane, component).
__global__ void adj_exponent_kernel(const float* __restrict__ maxima, int parts, int count, int* __restrict__ ex) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const float* m = maxima + ((size_t)(i / 3) * parts) * 3 + i % 3;
  float x = 0.f;
#pragma unroll 8
  for (int p = 0; p < parts; ++p) x = fmaxf(x, m[3 * p]);
  ex[i] = adj_exponent(x);
}

struct AdjArgs {
  const float2* E;     // [stacks][nz][3][nx][ny] (the caller's fields)
  const float* g;      // [stacks][nz][nx][ny]
  const int* ex;       // [stacks][nz][3] scales
  const uint4* X;      // panel of w columns 2jf + p, k = m
  const uint4* Y;      // panel of w columns 64 (lf / 32) + 32 p + lf % 32, k = n
  const float2* D;     // [nz][nhp][nhp] exp(i k s_z z) of the plan's planes
  const float2* Pf;    // [launch's stacks][3][w][w] mirror-folded pupils (the forward's fold)
  const double* kszf;  // [nhp][nhp]
  float* partial;      // [launch's stacks * 3 * zgroups * MC][np][np], MC chunks along x
  double zoff[kAdjStacks];
  int s0, nstk, nz, nx, ny, w, n, row_groups;
  int zgroups, zper;   // planes are split into zgroups runs of zper (the last may be shorter)
  int hshift;          // H is stored with 2^-hshift
  float gexp[3];       // powers of two of the result
};

// One (stack, component, run of planes, 64 pixel rows, 32 folded y cells, 256 folded x rows) per
// workgroup of eight waves (waves past a smaller pupil's rows only take part in H: giving them a
// share of the contraction over x was no faster, and its partial sums cancel less exactly).  A
// step is a chunk of 64 x 64 pixels of one plane:
//   H[m][p, lf]      = sum_n (2 g E)[m][n] {cos, sin} phi    128 rows (m, re / im) x 64 columns
//   G[2jf + p][p, ri, lf] += sum_m {cos, sin} theta H        a wave: 32 rows x four blocks of 32
//                                                            columns, one per (p, re / im)
// H stays in LDS as a split panel.  A lane ends up with CC, CS, SC, SS of the same eight cells.
// The defocus and the pupil are the same function of z for all four mirrors and no function of z,
// so that per plane only  Z += {CC, CS, SC, SS} conj(D_z)  is summed (16 FMAs a folded cell); the
// mirrors and the pupil are taken once per run.
// While a step is multiplied the next one is split into LDS and the one after it is on its way
// from memory.  The field chunk, 2 g E 2^e split in halves, is 32-row blocks of 16 pixel rows m as
// rows 8 (m / 4) + 4 ri + m % 4, so that an accumulator lane holds 16 consecutive m of one part.
// Bound by latency: eight waves of 253 registers fill a CU, and its steps run one after the
// other between barriers (matrix cores busy a third of the time, vector units another, LDS a
// fifth).  64 stacks of 64 x 64 x 21 on a 256 x 256 pupil, the whole of 2 g E to the partial
// sums: 1140 us as two FP32 MFMA kernels with H in memory (2 x 120 + 2 x 450), 310 so and 27 for
// the scales.  Without the sum over planes 268, without G 190, without H 232.  The x table in
// registers spilled (406 us: a spill's reload waits for the loads in flight); the two waves of a
// SIMD in opposite order 370 against 328; all LDS reads of H first, or three chains, 305-307.
// MULTI: more than one chunk along y, so that H and the y table pass from step to step.  16 stacks
// of 128 x 128 x 21 at N = 256, a whole adjoint: 555 us with 89 registers spilled, most of them
// addresses kept over the planes, 366 with 30.
template <bool MULTI>
__global__ void __launch_bounds__(kAdjThreads, 2) adj_kernel(AdjArgs a) {
  extern __shared__ __align__(16) char alds[];
  uint4* As = reinterpret_cast<uint4*>(alds);
  uint4* Hs = reinterpret_cast<uint4*>(alds + kAdjPanel);
  uint4* Ts = reinterpret_cast<uint4*>(alds + 2 * kAdjPanel);
  uint4* Xs = reinterpret_cast<uint4*>(alds + 2 * kAdjPanel + kAdjTab);
  const int tiles_n = a.w / (2 * kAdjCols);
  const int MC = (a.nx + kAdjChunk - 1) / kAdjChunk, NC = MULTI ? (a.ny + kAdjChunk - 1) / kAdjChunk : 1;
  const int nblocks = a.nstk * 3 * a.zgroups * MC * a.row_groups * tiles_n;
  int id = xcd_remap(blockIdx.x, nblocks);
  const int tn = id % tiles_n; id /= tiles_n;
  const int rg = id % a.row_groups; id /= a.row_groups;
  const int c = id % 3; id /= 3;
  const int mc = id % MC; id /= MC;
  const int zg = id % a.zgroups, s = id / a.zgroups;
  const int z_begin = zg * a.zper, z_end = min(a.nz, z_begin + a.zper);
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row0 = rg * kAdjRows + wave * 32;   // folded x rows 2jf + p of this wave
  const bool active = row0 < a.w;
  const int nhp = a.w / 2, lf = kAdjCols * tn + l32, jf0 = row0 / 2;
  const size_t plane = (size_t)a.nx * a.ny;
  const size_t gs = (size_t)(a.s0 + s);

  // this thread's share of a chunk: eight pixels of row ml from nl
  const int ml = (lane & 7) + 8 * wave, nl = lane & ~7;
  struct Regs {
    float4 v[4], f[2];
    uint4 t[MULTI ? 2 : 1];   // of the y table
    int e;
    float two;   // 0 past the edges (such pixels are loaded from pixel 0)
  };
  const int m = kAdjChunk * mc + ml;
  auto load = [&](int zi, int nc) {
    Regs r;
    const int n = kAdjChunk * nc + nl;
    const size_t pl = gs * a.nz + zi;
    const bool ok = m < a.nx && n < a.ny;
    const size_t off = ok ? (size_t)m * a.ny + n : 0;
    const any4* ep = reinterpret_cast<const any4*>(a.E + (pl * 3 + c) * plane + off);
    const any4* gp = reinterpret_cast<const any4*>(a.g + pl * plane + off);
#pragma unroll
    for (int i = 0; i < 4; ++i) r.v[i] = make_float4(ep[i].x, ep[i].y, ep[i].z, ep[i].w);
#pragma unroll
    for (int i = 0; i < 2; ++i) r.f[i] = make_float4(gp[i].x, gp[i].y, gp[i].z, gp[i].w);
    r.two = ok ? 2.f : 0.f;
    r.e = a.ex[pl * 3 + c];
    if constexpr (MULTI) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int idx = tid + i * kAdjThreads, q = min(16 * nc + idx / 64, a.ny / 4 - 1);
        r.t[i] = a.Y[(size_t)q * a.w + 2 * kAdjCols * tn + idx % 64];
      }
    }
    return r;
  };
  auto store = [&](const Regs& r) {
    float x[8], y[8];
    const float* v = reinterpret_cast<const float*>(r.v);
    const float* f = reinterpret_cast<const float*>(r.f);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float ff = r.two * f[i];
      x[i] = ldexpf(ff * v[2 * i], r.e);
      y[i] = ldexpf(ff * v[2 * i + 1], r.e);
    }
    const int row = 32 * (ml >> 4) + 8 * ((ml >> 2) & 3) + (ml & 3);
    uint4* o = As + (size_t)(4 * (nl >> 4) + ((nl >> 3) & 1)) * 128 + row;
    unsigned hi[4], lo[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) hg_split2(x[2 * i], x[2 * i + 1], &hi[i], &lo[i]);
    o[0] = make_uint4(hi[0], hi[1], hi[2], hi[3]);
    o[256] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
#pragma unroll
    for (int i = 0; i < 4; ++i) hg_split2(y[2 * i], y[2 * i + 1], &hi[i], &lo[i]);
    o[4] = make_uint4(hi[0], hi[1], hi[2], hi[3]);
    o[260] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
    if constexpr (MULTI) {
#pragma unroll
      for (int i = 0; i < 2; ++i) Ts[tid + i * kAdjThreads] = r.t[i];
    }
  };
  int zl = z_begin, nl_c = 0;   // chunk that is loaded next
  auto advance = [&]() {
    if (!MULTI || ++nl_c == NC) {
      nl_c = 0;
      zl = min(zl + 1, z_end - 1);
    }
  };
  Regs cur = load(zl, nl_c);
  advance();
  if constexpr (!MULTI) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int idx = tid + i * kAdjThreads, q = min(idx / 64, a.ny / 4 - 1);
      Ts[idx] = a.Y[(size_t)q * a.w + 2 * kAdjCols * tn + idx % 64];
    }
  }
  // x rows past the table repeat its last row
#pragma unroll
  for (int idx = tid; idx < kAdjChunk / 4 * kAdjRows; idx += kAdjThreads) {
    const int q = min(kAdjChunk / 4 * mc + idx / kAdjRows, a.nx / 4 - 1);
    Xs[idx] = a.X[(size_t)q * a.w + min(rg * kAdjRows + idx % kAdjRows, a.w - 1)];
  }
  hg16 zero;
#pragma unroll
  for (int r = 0; r < 16; ++r) zero[r] = 0.f;
  hg16 zacc[4] = {zero, zero, zero, zero}, acc[4] = {zero, zero, zero, zero};
  hg16 hx = zero, hm = zero;   // cross products and main product of this wave's block of H
  float2 d[8];                 // defocus of the plane in acc
#pragma unroll
  for (int q = 0; q < 8; ++q) d[q] = make_float2(0.f, 0.f);
  int e_acc = 0, e_cur = cur.e;
  store(cur);
  cur = load(zl, nl_c);
  const float hscale = ldexpf(1.f, -a.hshift);
  // The lane half of an LDS read in its base, so that the reads of a loop are one address and
  // constants; in its step with one chunk, where registers are left (328 us, in the base 357).
  const int hbase = MULTI ? h : 0, hstep = MULTI ? 0 : h;
  const int hb = wave >> 1, hp = wave & 1;   // 16 pixel rows and the parity of this wave's block of H
  // Z += acc conj(D).  Blocks 0, 1 (2, 3) hold the parts of C* and S* at y parity 0 (1); even
  // registers are x parity 0, odd ones 1.
  auto add_plane = [&]() {
    const int eu = a.hshift - e_acc - 2 * kTabExp;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const float cs = ldexpf(d[q].x, eu), sn = ldexpf(d[q].y, eu);
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          const int r = 2 * q + p;
          const float xr = acc[2 * b][r], xi = acc[2 * b + 1][r];
          zacc[2 * b][r] = fmaf(xi, sn, fmaf(xr, cs, zacc[2 * b][r]));
          zacc[2 * b + 1][r] = fmaf(-xr, sn, fmaf(xi, cs, zacc[2 * b + 1][r]));
        }
    }
  };
  auto transform_y = [&]() {
    const hg8* ap = reinterpret_cast<const hg8*>(As) + 32 * hb + l32 + hbase * 128;
    const hg8* bp = reinterpret_cast<const hg8*>(Ts) + 32 * hp + l32 + hbase * 64;
#pragma unroll
    for (int u = 0; u < kAdjChunk / 16; ++u) {
      const hg8 ah = ap[(4 * u + hstep) * 128], al = ap[(4 * u + 2 + hstep) * 128];
      const hg8 bh = bp[(4 * u + hstep) * 64], bl = bp[(4 * u + 2 + hstep) * 64];
      hx = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bl, hx, 0, 0, 0);
      hm = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bh, hm, 0, 0, 0);
      hx = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, bh, hx, 0, 0, 0);
    }
  };
#pragma unroll 1
  for (int zi = z_begin; zi < z_end; ++zi) {
    __syncthreads();   // the chunk is in LDS, H of the plane before is consumed
    add_plane();       // of the plane before, a share of it behind every matrix instruction
    hx = zero;
    hm = zero;
    transform_y();
#pragma unroll
    for (int g = 0; g < 12; ++g) {
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);   // LDS reads
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // matrix
      __builtin_amdgcn_sched_group_barrier(0x002, 12, 0);  // vector
    }
    if constexpr (MULTI) {
#pragma unroll 1
      for (int nc = 1; nc < NC; ++nc) {
        __syncthreads();
        store(cur);
        advance();
        cur = load(zl, nl_c);
        __syncthreads();
        transform_y();
      }
    }
    {
      // lane half h holds the part ri = h of 16 consecutive m at column (hp, l32)
      float v[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) v[r] = (hm[r] + hx[r]) * hscale;
      uint4 piece[4];
      hg_split16(v, piece);
      uint4* o = Hs + (size_t)(4 * hb) * 128 + 32 * (2 * hp + h) + l32;
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i * 128] = piece[i];
    }
    __syncthreads();   // H is in LDS, the chunk is consumed
    // the defocus before the next chunk: loads return in order
    const float2* Dz = a.D + ((size_t)zi * nhp + (active ? jf0 : 0)) * nhp;
    if constexpr (MULTI) {
      unsigned o = 2 * h * nhp + lf;
      asm("" : "+v"(o));   // formed for each plane: eight addresses kept spill (one chunk: 359 us)
#pragma unroll
      for (int q = 0; q < 8; ++q) d[q] = (Dz + (4 * (q >> 1) + (q & 1)) * nhp)[o];
    } else {
#pragma unroll
      for (int q = 0; q < 8; ++q) d[q] = (Dz + lf)[(size_t)(4 * (q >> 1) + 2 * h + (q & 1)) * nhp];
    }
    e_acc = e_cur;
    __builtin_amdgcn_sched_barrier(0);
    e_cur = cur.e;
    store(cur);   // after the last plane once more, unused
    advance();
    cur = load(zl, nl_c);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = zero;
    const hg8* bp = reinterpret_cast<const hg8*>(Hs) + l32 + hbase * 128;
    const hg8* xp = reinterpret_cast<const hg8*>(Xs) + 32 * wave + l32 + hbase * kAdjRows;
#pragma unroll
    for (int k16 = 0; k16 < kAdjChunk / 16; ++k16) {
      const hg8 xh = xp[(4 * k16 + hstep) * kAdjRows], xl = xp[(4 * k16 + 2 + hstep) * kAdjRows];
      hg8 bh[4], bl[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        bh[j] = bp[(4 * k16 + hstep) * 128 + 32 * j];
        bl[j] = bp[(4 * k16 + 2 + hstep) * 128 + 32 * j];
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(xh, bl[j], acc[j], 0, 0, 0);
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(xl, bh[j], acc[j], 0, 0, 0);
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(xh, bh[j], acc[j], 0, 0, 0);
    }
  }
  add_plane();
  if (!active) return;
  const int nh = (a.n + 1) / 2;
  const size_t npp = (size_t)a.w * a.w;
  const float2* Pf = a.Pf + ((size_t)s * 3 + c) * npp;
  float* out = a.partial + ((((size_t)s * 3 + c) * a.zgroups + zg) * MC + mc) * npp;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const int jf = jf0 + 4 * (q >> 1) + 2 * h + (q & 1);
    if (jf >= nh || lf >= nh) continue;
    const int j1 = a.n - 1 - jf, l1 = a.n - 1 - lf;
    // the pupil at mirror (a, b) from the four parities of the folded cell:
    //   P_ab = sum_{pj, pl} (-1)^(a pj + b pl) (-i)^(pj + pl) Pf_{pj, pl}
    // over 2 per folded axis with two mirrors (a self-mirrored row has no odd part), times the
    // stack's own defocus
    const float4 f0 = *reinterpret_cast<const float4*>(Pf + (size_t)(2 * jf) * a.w + 2 * lf);
    const float4 f1 = *reinterpret_cast<const float4*>(Pf + (size_t)(2 * jf + 1) * a.w + 2 * lf);
    const float scale = (jf != j1 ? 0.5f : 1.f) * (lf != l1 ? 0.5f : 1.f) * a.gexp[c];
    float sn, cs;
    sincosf((float)reduce_2pi(a.kszf[(size_t)jf * nhp + lf] * a.zoff[s]), &sn, &cs);
    const float ccr = zacc[0][2 * q], cci = zacc[1][2 * q], scr = zacc[0][2 * q + 1], sci = zacc[1][2 * q + 1];
    const float csr = zacc[2][2 * q], csi = zacc[3][2 * q], ssr = zacc[2][2 * q + 1], ssi = zacc[3][2 * q + 1];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const float sb = (m & 1) ? -1.f : 1.f, sa = (m & 2) ? -1.f : 1.f;
      const int jc = (m & 2) ? j1 : jf, lc = (m & 1) ? l1 : lf;
      if (((m & 2) && jc == jf) || ((m & 1) && lc == lf)) continue;
      // (-i) (x + i y) = y - i x
      const float ur = scale * ((f0.x + sb * f0.w) + sa * (f1.y - sb * f1.z));
      const float ui = scale * ((f0.y - sb * f0.z) - sa * (f1.x + sb * f1.w));
      const float pr = ur * cs - ui * sn, pi = ur * sn + ui * cs;
      // G = i T, T = CC - sb i CS - sa i SC - sa sb SS; Im(G conj(P~)) = Re(T) Pr + Im(T) Pi
      const float tr = (ccr + sb * csi) + sa * (sci - sb * ssr);
      const float ti = (cci - sb * csr) - sa * (scr + sb * ssi);
      out[(size_t)jc * a.w + lc] = tr * pr + ti * pi;
    }
  }
}

// dL/dPhi on the N x N cells: the partials of a launch are summed in group order (FP64) in two
// levels -- runs of kReduceRun groups (grid.y runs) into rows 1, 2, .. of `runs`, then the rows in
// order; row 0 is the sum over the launches before.
constexpr int kReduceRun = 32;

__global__ void adj_reduce_runs_kernel(const float* __restrict__ partial, int groups, int n, int np,
                                       double* __restrict__ runs) {
  const int cell = blockIdx.x * blockDim.x + threadIdx.x;
  if (cell >= n * n) return;
  const int j = cell / n, l = cell % n;
  const size_t pc = (size_t)j * np + l, npp = (size_t)np * np;
  const int g0 = blockIdx.y * kReduceRun, g1 = min(groups, g0 + kReduceRun);
  double s = 0.0;
#pragma unroll 8
  for (int g = g0; g < g1; ++g) s += (double)partial[g * npp + pc];
  runs[(size_t)(blockIdx.y + 1) * n * n + cell] = s;
}

// The sum over the launches so far: rows row0 .. nruns into row 0.
__global__ void adj_total_kernel(double* __restrict__ runs, int row0, int nruns, int nn) {
  const int cell = blockIdx.x * blockDim.x + threadIdx.x;
  if (cell >= nn) return;
  double s = 0.0;
#pragma unroll 8
  for (int r = row0; r <= nruns; ++r) s += runs[(size_t)r * nn + cell];
  runs[cell] = s;
}

// Second level, dL/dW0, and each workgroup's share of dL/dc_q = 2 pi sum_cells dL/dPhi Z_q
// (a tree over the lanes, then the four waves in order).
constexpr int kReduceThreads = 256;
__global__ void __launch_bounds__(kReduceThreads) adj_reduce_kernel(const double* __restrict__ runs, int row0,
                                                                    int nruns, int n, float* __restrict__ dW0,
                                                                    const float* __restrict__ ztab, int n_zernike,
                                                                    double* __restrict__ shares) {
  __shared__ double red[RWPSF_MAX_ZERNIKE][kReduceThreads / 64];
  const int nn = n * n, cell = blockIdx.x * kReduceThreads + threadIdx.x;
  const bool in = cell < nn;
  double s = 0.0;
  if (in) {
#pragma unroll 8
    for (int r = row0; r <= nruns; ++r) s += runs[(size_t)r * nn + cell];
    if (dW0) dW0[cell] = (float)s;
  }
  for (int q0 = 0; q0 < n_zernike; q0 += 6) {   // six terms' loads and trees in flight
    double v[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) v[i] = in ? s * (double)ztab[(size_t)min(q0 + i, n_zernike - 1) * nn + cell] : 0.0;
#pragma unroll
    for (int d = 32; d > 0; d >>= 1)
#pragma unroll
      for (int i = 0; i < 6; ++i) v[i] += __shfl_xor(v[i], d);
    if ((threadIdx.x & 63) == 0)
#pragma unroll
      for (int i = 0; i < 6; ++i)
        if (q0 + i < n_zernike) red[q0 + i][threadIdx.x >> 6] = v[i];
  }
  __syncthreads();
  if ((int)threadIdx.x < n_zernike) {
    const double* r = red[threadIdx.x];
    shares[(size_t)threadIdx.x * gridDim.x + blockIdx.x] = (r[0] + r[1]) + (r[2] + r[3]);
  }
}

// dL/dc_q from the shares: one workgroup per q, fixed-shape tree.  (One workgroup of 1024 per q
// over all cells instead took 30 us at 256 x 256 cells; shares and this 9 with the reduction.)
__global__ void __launch_bounds__(kReduceThreads) adj_zernike_kernel(const double* __restrict__ shares, int count,
                                                                     float* __restrict__ dc) {
  __shared__ double red[kReduceThreads / 64];
  double v = 0.0;
  for (int i = threadIdx.x; i < count; i += kReduceThreads) v += shares[(size_t)blockIdx.x * count + i];
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) dc[blockIdx.x] = (float)(kTwoPi * ((red[0] + red[1]) + (red[2] + red[3])));
}

// How a call is spread over workgroups and launches.  The partial sums of a launch take at most
// kAdjPartialBytes, or one run of all planes of one stack where that is more (1.5 GiB at the largest
// image and pupil): wide images and large pupils take longer runs, then fewer stacks a launch.  (All
// partial sums of a call at once were 41 GB for 1024 stacks of 256 x 256 x 21 at N = 512.)
constexpr size_t kAdjPartialBytes = (size_t)1 << 30;
struct AdjSplit {
  void (*k)(AdjArgs);
  int row_groups, zgroups, zper, chunks_x;
  int stacks;   // of a launch, at most
  int groups(int n) const { return 3 * std::min(n, stacks) * zgroups * chunks_x; }   // partial sums of a launch
};
static AdjSplit adjoint_split(const rwpsf_plan* p, int n) {
  const int w = 2 * p->nhp, nz = p->grid.nz;
  const int mc = (p->grid.nx + kAdjChunk - 1) / kAdjChunk, nc = (p->grid.ny + kAdjChunk - 1) / kAdjChunk;
  AdjSplit r{nc > 1 ? adj_kernel<true> : adj_kernel<false>, (w + kAdjRows - 1) / kAdjRows, 1, nz, mc, kAdjStacks};
  const size_t fit = kAdjPartialBytes / ((size_t)3 * mc * p->np * p->np * sizeof(float));   // runs of planes of a launch
  const int shortest = fit > 0 ? (int)((nz + fit - 1) / fit) : nz;
  // Runs of planes: one workgroup fits a CU (256 of them), a plane takes a step per chunk along y
  // and the pupil at the end of a run costs about three.  The shortest runs (they are summed in
  // FP32, the partial sums in FP64) within 15% of the least number of rounds times length.
  const long long base = (long long)std::min(n, kAdjStacks) * 3 * mc * r.row_groups * (w / (2 * kAdjCols));
  auto cost = [&](int zper) {
    return ((base * ((nz + zper - 1) / zper) + 255) / 256) * ((long long)zper * nc + 3);
  };
  long long best = cost(nz);
  for (int zper = shortest; zper < nz; ++zper) best = std::min(best, cost(zper));
  for (r.zper = shortest; 20 * cost(r.zper) > 23 * best;) ++r.zper;
  r.zgroups = (nz + r.zper - 1) / r.zper;
  r.stacks = (int)std::max<size_t>(1, std::min<size_t>(kAdjStacks, fit / r.zgroups));
  return r;
}

// Lazily built adjoint tables and workspace of a Fourier plan.
static int adjoint_prepare(rwpsf_plan* p, int n_stacks, const AdjSplit& sp) {
  const int nx = p->grid.nx, ny = p->grid.ny, nz = p->grid.nz, N = p->num.n_pupil, np = p->np;
  const int nhp = p->nhp, w = 2 * nhp;
  int st;
  if (!p->adj_ready) {   // set last; a try that failed on the way leaves what it has allocated to the next
    const double s_max = p->s_max, k = p->k;
    const size_t cells = (size_t)nhp * nhp;
    if ((st = dev_need(p, &p->d_adjTx, hg_panel_bytes(nx, w) / sizeof(uint4)))) return st;
    if ((st = dev_need(p, &p->d_adjTy, hg_panel_bytes(ny, w) / sizeof(uint4)))) return st;
    if ((st = dev_need(p, &p->d_shares, (size_t)RWPSF_MAX_ZERNIKE * ((N * N + kReduceThreads - 1) / kReduceThreads))))
      return st;
    if ((st = dev_need(p, &p->d_adjPf, (size_t)kAdjStacks * 3 * w * w))) return st;   // of a whole launch
    if ((st = dev_need(p, &p->d_adjD, nz * cells))) return st;
    if ((st = dev_need(p, &p->d_adjMax, (size_t)3 * kScaleGroups))) return st;
    hipLaunchKernelGGL(adj_panel_kernel, dim3((nx * nhp + 255) / 256), dim3(256), 0, 0, (_Float16*)p->d_adjTx, nx, N, w,
                       k, s_max, p->grid.dx_nm, 0);
    hipLaunchKernelGGL(adj_panel_kernel, dim3((ny * nhp + 255) / 256), dim3(256), 0, 0, (_Float16*)p->d_adjTy, ny, N, w,
                       k, s_max, p->grid.dy_nm, 1);
    hipLaunchKernelGGL(adj_defocus_kernel, dim3((unsigned)((nz * cells + 255) / 256)), dim3(256), 0, 0, p->d_kszf,
                       p->d_z, nz, (int)cells, p->d_adjD);
    if ((st = hip_check(hipGetLastError()))) return st;
    // the tables are written on the null stream; the caller's stream may not order after it
    if ((st = hip_check(hipDeviceSynchronize()))) return st;
    if ((st = hip_check(hipFuncSetAttribute((const void*)sp.k, hipFuncAttributeMaxDynamicSharedMemorySize, kAdjLds))))
      return st;
    p->adj_ready = true;
  }
  if (p->adj_stacks < n_stacks) {
    int* d = nullptr;
    if ((st = dev_alloc(p, &d, (size_t)n_stacks * nz * 3))) return st;
    p->d_adjEx = d;
    p->adj_stacks = n_stacks;
  }
  if (p->partial_stacks < std::min(n_stacks, kAdjStacks)) {
    // Room for every call of up to that many stacks: one of fewer may have more runs of planes, and
    // must not have to allocate after a larger one (it may be under capture).  In powers of two, as
    // what is replaced stays with the plan.
    int most = 1;
    while (most < std::min(n_stacks, kAdjStacks)) most *= 2;
    int groups = 0;
    for (int n = 1; n <= most; ++n) groups = std::max(groups, adjoint_split(p, n).groups(n));
    float* d = nullptr;
    if ((st = dev_alloc(p, &d, (size_t)groups * np * np))) return st;
    double* r = nullptr;
    if ((st = dev_alloc(p, &r, (size_t)((groups + kReduceRun - 1) / kReduceRun + 1) * N * N))) {
      dev_release(p, d, (size_t)groups * np * np);
      return st;
    }
    p->d_partial = d;
    p->d_runs = r;
    p->partial_stacks = most;
  }
  return RWPSF_OK;
}

int fourier_adjoint(rwpsf_plan* p, int n, const rwpsf_stack* s, const float2* E, const float* dLdI,
                    int n_zernike, float* dc, float* dW0, hipStream_t st) {
  const int nx = p->grid.nx, ny = p->grid.ny, nz = p->grid.nz, N = p->num.n_pupil, np = p->np;
  if (nx % 16 || ny % 16) return RWPSF_ERR_UNSUPPORTED;   // whole MFMA k-steps along x and y
  const AdjSplit sp = adjoint_split(p, n);
  int rc = adjoint_prepare(p, n, sp);
  if (rc) return rc;
  const int w = 2 * p->nhp;
  int tr = p->time_begin(RWPSF_KERNEL_ADJ_H, st);
  // workgroups per plane: runs of at least kScalePixels, while there are fewer than four for each of 256 CUs
  const int items = n * nz;
  const int parts = std::max(1, std::min(nx * ny / kScalePixels, kScaleGroups / items));
  hipLaunchKernelGGL(adj_scale_kernel, dim3((unsigned)items * parts), dim3(256), 0, st, E, dLdI, nx * ny, parts,
                     p->d_adjEx, p->d_adjMax);
  if ((rc = hip_check(hipGetLastError()))) return rc;
  if (parts > 1) {
    hipLaunchKernelGGL(adj_exponent_kernel, dim3((unsigned)(3 * items + 63) / 64), dim3(64), 0, st, p->d_adjMax, parts,
                       3 * items, p->d_adjEx);
    if ((rc = hip_check(hipGetLastError()))) return rc;
  }
  p->time_end(tr, st);
  const int rblocks = (N * N + kReduceThreads - 1) / kReduceThreads;
  for (int b0 = 0; b0 < n; b0 += sp.stacks) {
    const int nb = std::min(sp.stacks, n - b0);
    if ((rc = fourier_build_folded(p, s + b0, nb, p->d_adjPf, st))) return rc;
    AdjArgs a{};
    a.E = E;
    a.g = dLdI;
    a.ex = p->d_adjEx;
    a.X = p->d_adjTx;
    a.Y = p->d_adjTy;
    a.D = p->d_adjD;
    a.Pf = p->d_adjPf;
    a.kszf = p->d_kszf;
    a.partial = p->d_partial;
    for (int i = 0; i < nb; ++i) a.zoff[i] = s[b0 + i].z_offset_nm;
    a.s0 = b0;
    a.nstk = nb;
    a.nz = nz;
    a.nx = nx;
    a.ny = ny;
    a.w = w;
    a.n = N;
    a.row_groups = sp.row_groups;
    a.zgroups = sp.zgroups;
    a.zper = sp.zper;
    // |H 2^(e + kTabExp)| <= ny 2^14 2^kTabExp is stored below 2^15
    a.hshift = kTabExp - 1;
    while ((1 << (a.hshift - kTabExp + 1)) < ny) ++a.hshift;
    // G conj(P~) needs the prefactor f k / 2 pi once: the folded pupils carry its mantissa and
    // 2^pf_exp
    int pref_exp = 0;
    std::frexp(p->opt.focal_length * p->k / kTwoPi, &pref_exp);
    for (int c = 0; c < 3; ++c) a.gexp[c] = std::ldexp(1.f, pref_exp - p->scales.pf_exp[c]);
    const int blocks = nb * 3 * sp.zgroups * sp.chunks_x * sp.row_groups * (w / (2 * kAdjCols));
    tr = p->time_begin(RWPSF_KERNEL_ADJ_G, st);
    hipLaunchKernelGGL(sp.k, dim3(blocks), dim3(kAdjThreads), kAdjLds, st, a);
    if ((rc = hip_check(hipGetLastError()))) return rc;
    p->time_end(tr, st);
    // this launch's partial sums, with those of the launches before
    tr = p->time_begin(RWPSF_KERNEL_ADJ_REDUCE, st);
    const int groups = sp.groups(nb), nruns = (groups + kReduceRun - 1) / kReduceRun, row0 = b0 == 0 ? 1 : 0;
    hipLaunchKernelGGL(adj_reduce_runs_kernel, dim3((N * N + 255) / 256, nruns), dim3(256), 0, st, p->d_partial,
                       groups, N, np, p->d_runs);
    if ((rc = hip_check(hipGetLastError()))) return rc;
    if (b0 + nb < n) {
      hipLaunchKernelGGL(adj_total_kernel, dim3((N * N + 255) / 256), dim3(256), 0, st, p->d_runs, row0, nruns, N * N);
      if ((rc = hip_check(hipGetLastError()))) return rc;
    } else {
      hipLaunchKernelGGL(adj_reduce_kernel, dim3(rblocks), dim3(kReduceThreads), 0, st, p->d_runs, row0, nruns, N, dW0,
                         p->d_ztab, n_zernike, p->d_shares);
      if ((rc = hip_check(hipGetLastError()))) return rc;
      if (n_zernike > 0) {
        hipLaunchKernelGGL(adj_zernike_kernel, dim3(n_zernike), dim3(kReduceThreads), 0, st, p->d_shares, rblocks, dc);
        if ((rc = hip_check(hipGetLastError()))) return rc;
      }
    }
    p->time_end(tr, st);
  }
  return RWPSF_OK;
}

}  // namespace rw
