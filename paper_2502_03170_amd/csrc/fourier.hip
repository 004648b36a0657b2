// Fourier (Cartesian) form of the vectorial Richards-Wolf integral on gfx950.
//
// Sec. 3.3 eq. "cartesian vectorial" with the correction factors of Sec. 3.4:
// each z-plane of each field component is the 2-D transform of the pupil
//   P~_c[j,l] = P_c[j,l] exp(i k s_z z),  P_c = ds^2 a exp(iW) e_inf,c / s_z
// to the pixel grid, E_c = C sum_{j,l} P~_c[j,l] e^{i k (s_x[j] x + s_y[l] y)},
// C = -i f k / 2 pi.  The sample grid is symmetric (s[n-1-j] = -s[j]), so each 1-D
// transform folds into even and odd parts with real coefficients cos / sin, and the
// separable transform becomes two real GEMMs with half the flops of the complex matrix DFT,
// run on the F16 matrix cores with split operands at FP32-level accuracy (hgemm.h):
//   K1  pupil_build_folded   mirror-folded pupils Pf (four parities per folded cell)
//                     of up to 16 stacks, each cell's P_c formed on the way (FP64
//                     phase: Gibson-Lanni, Zernike, free phase map, lateral emitter
//                     shift); the chirp-z path takes the unfolded P_c of pupil_build
//   K2  gemm_pupil    T = Pf~ B1 (fold along y); the defocus factor is formed while the
//                     pupil tile is staged (FP64 phase, reduced mod 2 pi, FP32 sincos)
//   K3  gemm_image    E'_c = A2 T_c (fold along x) for c = x, y, z in one workgroup,
//                     writing E = -i E' and I = sum_c |E_c|^2 from registers.
#include <algorithm>

#include "hfold.h"
#include "hgemm.h"
#include "rw_common.h"
#include "rw_fourier.h"

namespace rw {

// --------------------------------------------------------------------------
// Plan-time table: orthonormal Noll Zernike basis on the cell-centred pupil grid.
// --------------------------------------------------------------------------
__global__ void zernike_table_kernel(float* __restrict__ out, int n, int nj) {
  const int cell = blockIdx.x * blockDim.x + threadIdx.x;
  if (cell >= n * n) return;
  const int j = cell / n, l = cell % n;
  const double u = (2.0 * j + 1.0 - n) / n, v = (2.0 * l + 1.0 - n) / n;  // unit-disk coords
  const double r = sqrt(u * u + v * v);
  const double cp = r > 0 ? u / r : 1.0, sp = r > 0 ? v / r : 0.0;
  for (int q = 1; q <= nj; ++q)
    out[(size_t)(q - 1) * n * n + cell] = (float)zernike_noll(q, r, cp, sp);
}

// Plan-time table: one thread per (row r, folded cell f), FP64 sine and cosine.
__global__ void dft_panel_kernel(_Float16* __restrict__ panel, int rows, int count, int centre, int n, int w, double k,
                                 double s_max, double pitch) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= rows * (w / 2)) return;
  const int r = idx % rows, f = idx / rows;
  double v[2] = {0.0, 0.0};
  if (r < count && f < (n + 1) / 2) {
    const double ph = k * ((2.0 * f + 1.0 - n) * s_max / n) * ((double)(r - centre) * pitch);
    sincos(ph, &v[1], &v[0]);
  }
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const double x = ldexp(v[p], kTabExp);
    const int kk = 2 * f + p;
    _Float16* o = panel + ((size_t)(kk / 16 * 4 + kk % 16 / 8) * rows + r) * 8 + kk % 8;
    const _Float16 hi = (_Float16)(float)x;
    o[0] = hi;
    o[(size_t)2 * rows * 8] = (_Float16)(float)(x - (double)(float)hi);
  }
}

// --------------------------------------------------------------------------
// K1: base pupil of each stack.
// --------------------------------------------------------------------------
// What a pupil cell's phase needs of the cell alone, with room for NZ Zernike terms.  Their
// loads are unrolled, so that a thread has them all in flight at once instead of waiting for
// each in turn.
template <int NZ>
struct PupilCell {
  int cell;   // unpadded index: Zernike table and user phase map
  double sx, sy, sin_t;
  float zv[NZ > 0 ? NZ : 1];
};
template <int NZ>
__device__ __forceinline__ PupilCell<NZ> pupil_cell(const PupilGeom& a, const float* __restrict__ ztab, int j, int l) {
  PupilCell<NZ> p;
  const int n = a.n;
  p.cell = j * n + l;
  p.sx = (2.0 * j + 1.0 - n) * a.s_max / n;
  p.sy = (2.0 * l + 1.0 - n) * a.s_max / n;
  p.sin_t = sqrt(p.sx * p.sx + p.sy * p.sy);
#pragma unroll
  for (int k = 0; k < NZ; ++k) p.zv[k] = k < a.max_zernike ? ztab[(size_t)k * n * n + p.cell] : 0.f;
  return p;
}

// exp(i W) (times the evanescent decay of a Gibson-Lanni layer) at a cell, for stack st with the
// coefficients (waves) in coef and the value w0 of its phase map (the table values of terms past
// max_zernike are 0).
template <int NZ, class Stack>
__device__ __forceinline__ float2 pupil_phase_factor(const PupilGeom& a, const Stack& st, const double* coef, float w0,
                                                     const PupilCell<NZ>& p) {
  double w_re = 0.0, w_im = 0.0;
  if (a.gibson_lanni) gl_opd(a.gl, st.t_s, p.sin_t, &w_re, &w_im);
  w_re -= a.k * (p.sx * st.x0 + p.sy * st.y0);
  w_re += (double)w0;
  double waves = 0.0;
#pragma unroll
  for (int k = 0; k < NZ; ++k) waves += coef[k] * (double)p.zv[k];
  w_re += kTwoPi * waves;
  // the evanescent decay in FP32 (relative error ~1e-7, far below the tolerance); the phase
  // reduced in FP64
  const float amp = w_im > 0.0 ? expf((float)-w_im) : 1.f;
  float sn, cs;
  sincospif(half_turns(w_re), &sn, &cs);
  return make_float2(amp * cs, amp * sn);
}

// One thread per (padded cell, stack): grid.y is the stack.
__global__ void __launch_bounds__(256) pupil_build_kernel(PupilArgs a, const float2* __restrict__ Q,
                                                          const float* __restrict__ ztab,
                                                          float2* __restrict__ P) {
  const int n = a.n, np = a.np;
  const size_t npp = (size_t)np * np;
  const int pcell = blockIdx.x * blockDim.x + threadIdx.x;   // padded cell
  const int s = blockIdx.y;
  if (pcell >= np * np) return;
  const int j = pcell / np, l = pcell % np;
  const int nc = a.nc;
  float2* out = P + (size_t)s * nc * npp + pcell;
  float2 q[3] = {make_float2(0.f, 0.f), make_float2(0.f, 0.f), make_float2(0.f, 0.f)};
  bool inside = false;
  if (j < n && l < n)
    for (int c = 0; c < nc; ++c) {
      q[c] = Q[c * npp + pcell];
      inside = inside || q[c].x != 0.f || q[c].y != 0.f;
    }
  if (!inside) {
    for (int c = 0; c < nc; ++c) out[c * npp] = make_float2(0.f, 0.f);
    return;
  }
  const PupilCell<RWPSF_MAX_ZERNIKE> pc = pupil_cell<RWPSF_MAX_ZERNIKE>(a, ztab, j, l);
  const float2 e = pupil_phase_factor(a, a.s[s], a.s[s].coef, a.s[s].w0 ? a.s[s].w0[pc.cell] : 0.f, pc);
  for (int c = 0; c < nc; ++c) out[c * npp] = make_float2(q[c].x * e.x - q[c].y * e.y, q[c].x * e.y + q[c].y * e.x);
}

// --------------------------------------------------------------------------
// K1 of the Fourier form: mirror-folded pupils.
//
// The cell-centred grid is symmetric, s[n-1-j] = -s[j], so with jf < nh = ceil(n/2)
// and its mirror j' = n-1-jf each 1-D transform splits into even and odd parts:
//   sum_j p_j e^{i k s_j x} = sum_jf cos(k s_jf x) (p_jf + p_j') + sin(k s_jf x) i (p_jf - p_j')
// Folding both pupil axes gives, per folded cell (jf, lf) and parities (pj, pl),
//   Pf_{pj,pl} = i^(pj+pl) sum_{a,b in {0,1}} (-1)^(a pj + b pl) P[mir_a(jf), mir_b(lf)]
// (a mirror equal to the cell itself -- the middle row of an odd n -- is counted once
// and has no odd part).  Both transforms then have real coefficients (cos, sin), so
// each is one real GEMM with half the flops of the complex one.  The defocus factor
// depends on s_x^2 + s_y^2 only and is the same for all four mirrors.
// Layout: Pf[s][c][q = 2 jf + pj][kk = 2 lf + pl], complex, (2 nhp) x (2 nhp).
// The four mirror cells' pupils are formed in registers, so P never reaches memory.
// --------------------------------------------------------------------------
// The values of v in the four lanes of this lane's quad (DPP quad_perm(k, k, k, k)).
__device__ __forceinline__ float4 quad_values(float v) {
  const int b = __float_as_int(v);
  return make_float4(__int_as_float(__builtin_amdgcn_update_dpp(0, b, 0x00, 0xF, 0xF, false)),
                     __int_as_float(__builtin_amdgcn_update_dpp(0, b, 0x55, 0xF, 0xF, false)),
                     __int_as_float(__builtin_amdgcn_update_dpp(0, b, 0xAA, 0xF, 0xF, false)),
                     __int_as_float(__builtin_amdgcn_update_dpp(0, b, 0xFF, 0xF, 0xF, false)));
}

// Four lanes per folded cell, which go through a group of stacks (grid.y): lane m of a quad
// forms the pupil of mirror m = 2 a + b, i.e. of cell (mir_a(jf), mir_b(lf)), broadcasts it to
// the quad (DPP quad permutes) and writes parity (pj, pl) = (m / 2, m % 2) of every channel.
// A lane keeps its base pupil and its table values for the whole group, and the coefficients
// of 16 stacks fit one launch.  64 stacks of 256 x 256 cells: 8 launches of 15.4 us with a lane
// per cell and stack, 4 of 15.2 us so (groups of 8 or 16 and unrolling by two change nothing: 25
// MB leave each launch); one stack of 64 x 64 cells without aberrations 19 -> 5.3 us with room
// for the terms in use only.
constexpr int kFoldGroup = 4;
template <int NZ>
__global__ void __launch_bounds__(256) pupil_build_folded_kernel(FoldArgs a, const float2* __restrict__ Q,
                                                                 const float* __restrict__ ztab,
                                                                 float2* __restrict__ Pf, int nhp, int group) {
  const int n = a.n, np = a.np, nh = (a.n + 1) / 2;
  const int gid = blockIdx.x * blockDim.x + threadIdx.x;
  const int cell = gid >> 2, m = gid & 3;
  if (cell >= nhp * nhp) return;   // whole quads
  const int jf = cell / nhp, lf = cell % nhp;
  const int pj = m >> 1, pl = m & 1;
  const size_t npp = (size_t)np * np, fpp = (size_t)4 * nhp * nhp;
  const int w = 2 * nhp, nc = a.nc;
  const int s0 = blockIdx.y * group, s1 = min(s0 + group, a.nstk);
  const float2 zero = make_float2(0.f, 0.f);
  const bool cells = jf < nh && lf < nh;   // whole quads
  const int j1 = n - 1 - jf, l1 = n - 1 - lf;
  const bool dj = j1 != jf, dl = l1 != lf;
  // this lane's mirror; a mirror equal to the cell itself is absent (zero)
  const int j = pj ? j1 : jf, l = pl ? l1 : lf;
  const bool present = cells && (pj ? dj : true) && (pl ? dl : true);
  float2 q[3];
  bool inside = false;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    q[c] = present && c < nc ? Q[c * npp + (size_t)j * np + l] : zero;
    inside = inside || q[c].x != 0.f || q[c].y != 0.f;
  }
  PupilCell<NZ> pc{};
  if (inside) {
    pc = pupil_cell<NZ>(a, ztab, j, l);
  }
  // the mirror's sign in this lane's parity: (-1)^(a pj + b pl) for mirror (a, b)
  const float s01 = pl ? -1.f : 1.f, s10 = pj ? -1.f : 1.f;
  const bool odd_ok = (!pj || dj) && (!pl || dl);   // odd parts of a self-mirrored row vanish
  const float* map = nullptr;
  float w0 = 0.f;
#pragma unroll 1
  for (int s = s0; s < s1; ++s) {
    if (a.s[s].w0 != map) {   // the map of the stack before is the usual one
      map = a.s[s].w0;
      w0 = map && inside ? map[pc.cell] : 0.f;
    }
    float2* out = Pf + (size_t)s * nc * fpp + (size_t)(2 * jf + pj) * w + 2 * lf + pl;
    float2 p[3] = {zero, zero, zero};
    if (inside) {
      const float2 e = pupil_phase_factor(a, a.s[s], a.coef + s * a.max_zernike, w0, pc);
#pragma unroll
      for (int c = 0; c < 3; ++c) p[c] = make_float2(q[c].x * e.x - q[c].y * e.y, q[c].x * e.y + q[c].y * e.x);
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      if (c >= nc) break;
      const float4 vr = quad_values(p[c].x), vi = quad_values(p[c].y);
      // mirrors (0,0) + s01 (0,1) + s10 [(1,0) + s01 (1,1)]
      float re = (vr.x + s01 * vr.y) + s10 * (vr.z + s01 * vr.w);
      float im = (vi.x + s01 * vi.y) + s10 * (vi.z + s01 * vi.w);
      if (!odd_ok) re = im = 0.f;
      // times i^(pj + pl)
      float2 v;
      if (pj + pl == 0) v = make_float2(re, im);
      else if (pj + pl == 1) v = make_float2(-im, re);
      else v = make_float2(-re, -im);
      out[c * fpp] = v;
    }
  }
}

// --------------------------------------------------------------------------
// K2, K3: the two GEMMs (the pupil operand's loader is in hfold.h).
// --------------------------------------------------------------------------
// Measured on 16 stacks of 128 x 128 x 64 at a 256 x 256 pupil (fields and intensity): the
// call took 1305 us with FP32 MFMA tiles and takes 660 us (pupil GEMM 860 -> 345-400 us, image
// GEMM 480 -> 310-345 us, whose 0.8 GB of T and 0.47 GB of output are 4 TB/s of HBM); one
// 201 x 201 image 52 -> 22 us.  The pupil GEMM's pipes hardly overlap: its MFMAs alone need
// 115 us, without them it takes 257 us, without global loads 247 us; one plane per tile
// (the pupil then crosses L2 twice as often) 372 us, other tile shapes and occupancies
// (128 x 128, eight waves, k-stages of 32) 372-450 us.
// Tiles.  Pupil GEMM: 128 rows of two planes x 128 columns (four 64 x 128 waves, two
// workgroups per CU), 64 columns for outputs of at most 64 pixels; image GEMM: 128 (n, re /
// im) rows x 128 pixels m.  Launches that would underfill the GPU take the 64 x 64 tiles.
using CfgPupil = HgCfg<256, 128, 16, 64, 128>;
using CfgPupilN = HgCfg<256, 64, 16, 64, 64>;
using CfgPupilS = HgCfg<64, 64, 32, 32, 32>;
using CfgImage = HgCfg<128, 128, 32, 64, 64>;
using CfgImageM = HgCfg<128, 64, 32, 64, 32>;
using CfgImageS = HgCfg<64, 64, 32, 32, 32>;
static_assert((4 * kFoldPad) % (CfgPupil::BM / 2) == 0 && (2 * kFoldPad) % 32 == 0, "pupil GEMM padding");
static_assert(kPadY % CfgPupil::BN == 0 && kPadX % CfgImage::BN == 0 && (2 * kPadSmall) % CfgImage::BM == 0 &&
                  kPadSmall % CfgPupilS::BN == 0 && kPadSmall % CfgImageS::BN == 0,
              "output padding");

// K2: T[s][z][c] = (Pf~ B1), i.e. the complex [2 nhp] x [nyp] matrix
// T[q][n] = sum_kk Pf~[q][kk] B1[kk][n], B1[2lf][n] = cos(k s_lf y_n), B1[2lf+1][n] = sin(...),
// written as a panel of rows 2n + ri with k = q for K3: a lane's 16 accumulators are the 16
// consecutive q of one row, and the 64 lanes of a store cover 1 KB without gaps.
template <class Cfg, int PZ, int OCC>
__global__ void __launch_bounds__(Cfg::NT, OCC) gemm_pupil_kernel(Gemm1Args a) {
  extern __shared__ __align__(16) char hlds[];
  constexpr int BR = Cfg::BM / PZ;   // pupil rows of the tile
  const int w = 2 * a.nhp;
  const int tiles_m = 2 * w / BR;
  const int tiles_n = a.nyp / Cfg::BN;
  const int zgroups = (a.nzs + PZ - 1) / PZ;
  const int nblocks = a.nstk * zgroups * a.nc * tiles_m * tiles_n;
  int id = xcd_remap(blockIdx.x, nblocks);
  const int tn = id % tiles_n; id /= tiles_n;
  const int tm = id % tiles_m; id /= tiles_m;
  const int zi = id % zgroups * PZ; id /= zgroups;
  const int c = id % a.nc; id /= a.nc;
  const int s = id;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wrow = (wave / Cfg::WAVES_N) * Cfg::WM, wcol = (wave % Cfg::WAVES_N) * Cfg::WN;
  const size_t fpp = (size_t)w * w;
  const int row0 = tm * BR, col0 = tn * Cfg::BN;
  const int jf0 = row0 / 4;

  FoldDefocusLoader<Cfg, PZ> la;
  la.Pf = a.Pf + ((size_t)s * a.nc + c) * fpp + (size_t)(2 * jf0) * w;
  la.kszf = a.kszf + (size_t)jf0 * a.nhp;
#pragma unroll
  for (int z = 0; z < PZ; ++z) la.zrev[z] = (a.z[a.z0 + min(zi + z, a.nzs - 1)] + a.zoff[s]) * (1.0 / kTwoPi);
  la.w = w;
  la.nhp = a.nhp;
  HgPanelLoader<Cfg, Cfg::BN> lb;
  lb.src = a.B1 + col0;
  lb.ld = a.nyp;

  // The pupil is zero outside the disk (2j+1-n)^2 + (2l+1-n)^2 <= n^2: this row block
  // needs the folded columns lf that its row nearest the centre (largest jf) reaches.
  int k_begin = 0, k_end = w;
  {
    const int n = a.n, nh = (a.n + 1) / 2;
    const int jf_hi = min(jf0 + BR / 4, nh) - 1;
    if (jf_hi < jf0) {
      k_end = Cfg::BK;   // padding rows only: one (zero) stage
    } else {
      const int umin = abs(2 * jf_hi + 1 - n);
      const int vmax = (int)floorf(sqrtf((float)n * n - (float)umin * umin)) + 1;   // generous
      const int lf_lo = max(0, (n - 1 - vmax) / 2);
      k_begin = (2 * lf_lo / Cfg::BK) * Cfg::BK;
    }
  }
  HgAcc<Cfg> acc;
  acc.zero();
  hg_mainloop<Cfg>(acc, la, lb, k_begin, k_end, hlds, tid, wrow, wcol, lane);

  // each wave's rows belong to one plane
  static_assert(BR % Cfg::WM == 0, "a wave stays within a plane");
  const int zw = zi + wrow / BR, prow = row0 + wrow % BR;
  if (zw >= a.nzs) return;
  uint4* T = a.T + (((size_t)s * a.nzs + zw) * a.nc + c) * (hg_panel_bytes(w, 2 * a.nyp) / 16);
  const int ri = lane >> 5;
#pragma unroll
  for (int i = 0; i < Cfg::TM; ++i)
#pragma unroll
    for (int jj = 0; jj < Cfg::TN; ++jj) {
      const int n = col0 + wcol + 32 * jj + (lane & 31);
      float v[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) v[r] = acc.c[i][jj][r] * a.tscale;
      uint4 piece[4];
      hg_split16(v, piece);
      uint4* o = T + (size_t)(4 * ((prow + 32 * i) / 32)) * (2 * a.nyp) + 2 * n + ri;
#pragma unroll
      for (int p = 0; p < 4; ++p) o[(size_t)p * (2 * a.nyp)] = piece[p];
    }
}

// K3: E'[(n, ri)][m] = sum_kk T[kk][(n, ri)] A2[kk][m] with A2[2jf][m] = cos(k s_jf x_m),
// A2[2jf+1][m] = sin(...), for all channels in one workgroup; E = -i E' (times the
// prefactor) and I = sum_c |E_c|^2 are written from registers: accumulators 4g .. 4g + 3 of
// a lane are two neighbouring pixels (re, im) of one image row m, one 16-byte store.
// One channel: the GEMM (its first stage already in ra, rb), then the next channel's first
// stage is loaded, then this channel's fields are stored and its intensity accumulated.
// The loads go first so that the wait before they are staged in LDS does not also wait
// for the stores.
template <class Cfg, bool FULL, bool HAS_E, class LA, class LB>
__device__ __forceinline__ void image_channel(const Gemm2Args& a, char* lds, int c, LA& la, const LB& lb,
                                              typename LA::Regs& ra, typename LB::Regs& rb, const uint4* tsrc,
                                              size_t tch, float2* E, int row0, int col0,
                                              float (*isum)[Cfg::TN][8]) {
  const int w = 2 * a.nhp;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wrow = (wave / Cfg::WAVES_N) * Cfg::WM, wcol = (wave % Cfg::WAVES_N) * Cfg::WN;
  HgAcc<Cfg> acc;
  acc.zero();
  hg_mainloop_pre<Cfg>(acc, la, lb, ra, rb, 0, w, lds, tid, wrow, wcol, lane);
  // first stage of the next channel (the last channel reloads its own, unused)
  la.src = tsrc + (size_t)min(c + 1, a.nc - 1) * tch;
  ra = la.load(0, tid);
  rb = lb.load(0, tid);
  __builtin_amdgcn_sched_barrier(0);
  const float escale = component_scale(a.escale, c);
#pragma unroll
  for (int i = 0; i < Cfg::TM; ++i)
#pragma unroll
    for (int jj = 0; jj < Cfg::TN; ++jj) {
      const int m = col0 + wcol + 32 * jj + (lane & 31);
      const int n0 = (row0 + wrow + 32 * i) / 2 + 2 * (lane >> 5);
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int n = n0 + 4 * g;
        // E = -i E' = (Im E', -Re E')
        const float4 e = make_float4(acc.c[i][jj][4 * g + 1] * escale, acc.c[i][jj][4 * g] * -escale,
                                     acc.c[i][jj][4 * g + 3] * escale, acc.c[i][jj][4 * g + 2] * -escale);
        isum[i][jj][2 * g] += e.x * e.x + e.y * e.y;
        isum[i][jj][2 * g + 1] += e.z * e.z + e.w * e.w;
        if (HAS_E) {
          float2* o = E + (size_t)m * a.ny + n;
          if (FULL) {
            *reinterpret_cast<float4*>(o) = e;
          } else if (m < a.nx) {
            if (n < a.ny) o[0] = make_float2(e.x, e.y);
            if (n + 1 < a.ny) o[1] = make_float2(e.z, e.w);
          }
        }
      }
    }
}

// One output tile of K3 for every channel.  FULL: the tile lies inside the nx x ny image
// and its rows are 16-byte aligned, so its stores need no per-lane bounds and run as
// straight-line 16-byte (fields) and 8-byte (intensity) stores.
template <class Cfg, bool FULL, bool HAS_E>
__device__ __forceinline__ void image_tile(const Gemm2Args& a, char* lds, int s, int zi, int row0, int col0) {
  const int w = 2 * a.nhp;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wrow = (wave / Cfg::WAVES_N) * Cfg::WM, wcol = (wave % Cfg::WAVES_N) * Cfg::WN;
  const size_t plane = (size_t)a.nx * a.ny;
  const size_t gstk = (size_t)(a.s_base + s), gz = (size_t)(a.z0 + zi);
  float isum[Cfg::TM][Cfg::TN][8];
#pragma unroll
  for (int i = 0; i < Cfg::TM; ++i)
#pragma unroll
    for (int jj = 0; jj < Cfg::TN; ++jj)
#pragma unroll
      for (int r = 0; r < 8; ++r) isum[i][jj][r] = 0.f;

  const size_t tch = hg_panel_bytes(w, 2 * a.nyp) / 16;   // 16-byte pieces per channel of T
  const uint4* tsrc = a.T + ((size_t)s * a.nzs + zi) * a.nc * tch + row0;
  HgPanelLoader<Cfg, Cfg::BM> la;
  la.src = tsrc;
  la.ld = 2 * a.nyp;
  HgPanelLoader<Cfg, Cfg::BN> lb;
  lb.src = a.A2 + col0;
  lb.ld = a.nxp;
  auto ra = la.load(0, tid);
  auto rb = lb.load(0, tid);
  float2* E0 = HAS_E ? a.E + (gstk * a.nz + gz) * a.nc * plane : nullptr;
#pragma unroll 1
  for (int c = 0; c < a.nc; ++c)
    image_channel<Cfg, FULL, HAS_E>(a, lds, c, la, lb, ra, rb, tsrc, tch, HAS_E ? E0 + c * plane : nullptr, row0,
                                    col0, isum);
  if (a.I) {
    float* I = a.I + (gstk * a.nz + gz) * plane;
#pragma unroll
    for (int i = 0; i < Cfg::TM; ++i)
#pragma unroll
      for (int jj = 0; jj < Cfg::TN; ++jj) {
        const int m = col0 + wcol + 32 * jj + (lane & 31);
        const int n0 = (row0 + wrow + 32 * i) / 2 + 2 * (lane >> 5);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int n = n0 + 4 * g;
          float* o = I + (size_t)m * a.ny + n;
          if (FULL) {
            *reinterpret_cast<float2*>(o) = make_float2(isum[i][jj][2 * g], isum[i][jj][2 * g + 1]);
          } else if (m < a.nx) {
            if (n < a.ny) o[0] = isum[i][jj][2 * g];
            if (n + 1 < a.ny) o[1] = isum[i][jj][2 * g + 1];
          }
        }
      }
  }
}

template <class Cfg, int OCC>
__global__ void __launch_bounds__(Cfg::NT, OCC) gemm_image_kernel(Gemm2Args a) {
  extern __shared__ __align__(16) char hlds[];
  const int tiles_m = 2 * a.nyp / Cfg::BM;
  const int tiles_n = a.nxp / Cfg::BN;
  const int nblocks = a.nstk * a.nzs * tiles_m * tiles_n;
  int id = xcd_remap(blockIdx.x, nblocks);
  const int tn = id % tiles_n; id /= tiles_n;
  const int tm = id % tiles_m; id /= tiles_m;
  const int zi = id % a.nzs; id /= a.nzs;
  const int s = id;
  const int row0 = tm * Cfg::BM, col0 = tn * Cfg::BN;
  const bool full = a.vec && row0 + Cfg::BM <= 2 * a.ny && col0 + Cfg::BN <= a.nx;
  if (a.E) {
    if (full)
      image_tile<Cfg, true, true>(a, hlds, s, zi, row0, col0);
    else
      image_tile<Cfg, false, true>(a, hlds, s, zi, row0, col0);
  } else {
    if (full)
      image_tile<Cfg, true, false>(a, hlds, s, zi, row0, col0);
    else
      image_tile<Cfg, false, false>(a, hlds, s, zi, row0, col0);
  }
}

// K3 for launches of few tiles: the channels side by side in a workgroup, four waves and stage
// buffers each, instead of one after the other; |E_c|^2 meet in LDS and are added in channel
// order.  Such a launch is a chain of K / 32 stages on a part of the CUs: one 201 x 201 image on a
// 256 x 256 pupil (32 tiles) 13.6 -> 11.4 us, the whole call 24.8 -> 22.4.  With more tiles than
// CUs it is slower (1008 tiles 28 -> 49 us: one such workgroup fills a CU's LDS).
template <class Cfg>
__global__ void __launch_bounds__(3 * Cfg::NT, 1) gemm_image_few_kernel(Gemm2Args a) {
  static_assert(Cfg::TM == 1 && Cfg::TN == 1, "one block a wave");
  extern __shared__ __align__(16) char hlds[];
  const int tiles_m = 2 * a.nyp / Cfg::BM, tiles_n = a.nxp / Cfg::BN;
  int id = blockIdx.x;
  const int tn = id % tiles_n; id /= tiles_n;
  const int tm = id % tiles_m; id /= tiles_m;
  const int zi = id % a.nzs, s = id / a.nzs;
  const int row0 = tm * Cfg::BM, col0 = tn * Cfg::BN;
  const int c = __builtin_amdgcn_readfirstlane(threadIdx.x / Cfg::NT), tid = threadIdx.x % Cfg::NT;
  const int lane = tid & 63, wave = tid >> 6;
  const int wrow = (wave / Cfg::WAVES_N) * Cfg::WM, wcol = (wave % Cfg::WAVES_N) * Cfg::WN;
  const int w = 2 * a.nhp;
  const size_t plane = (size_t)a.nx * a.ny;
  const size_t at = (size_t)(a.s_base + s) * a.nz + a.z0 + zi;
  HgPanelLoader<Cfg, Cfg::BM> la;
  la.src = a.T + (((size_t)s * a.nzs + zi) * a.nc + c) * (hg_panel_bytes(w, 2 * a.nyp) / 16) + row0;
  la.ld = 2 * a.nyp;
  HgPanelLoader<Cfg, Cfg::BN> lb;
  lb.src = a.A2 + col0;
  lb.ld = a.nxp;
  char* lds = hlds + c * Cfg::LDS_BYTES;
  HgAcc<Cfg> acc;
  acc.zero();
  hg_mainloop<Cfg>(acc, la, lb, 0, w, lds, tid, wrow, wcol, lane);
  const int m = col0 + wcol + (lane & 31);
  const int n0 = (row0 + wrow) / 2 + 2 * (lane >> 5);
  const float escale = component_scale(a.escale, c);
  float* sq = reinterpret_cast<float*>(lds);   // [8][NT]: this channel's share of the lane's eight intensities
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int n = n0 + 4 * g;
    // E = -i E' = (Im E', -Re E')
    const float4 e = make_float4(acc.c[0][0][4 * g + 1] * escale, acc.c[0][0][4 * g] * -escale,
                                 acc.c[0][0][4 * g + 3] * escale, acc.c[0][0][4 * g + 2] * -escale);
    sq[(2 * g) * Cfg::NT + tid] = e.x * e.x + e.y * e.y;
    sq[(2 * g + 1) * Cfg::NT + tid] = e.z * e.z + e.w * e.w;
    if (a.E && m < a.nx) {
      float2* o = a.E + (at * a.nc + c) * plane + (size_t)m * a.ny + n;
      if (n < a.ny) o[0] = make_float2(e.x, e.y);
      if (n + 1 < a.ny) o[1] = make_float2(e.z, e.w);
    }
  }
  __syncthreads();
  if (!a.I || c > 0 || m >= a.nx) return;
  float* I = a.I + at * plane + (size_t)m * a.ny;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const int n = n0 + 4 * (q >> 1) + (q & 1);
    float v = 0.f;
    for (int k = 0; k < a.nc; ++k) v += reinterpret_cast<const float*>(hlds + k * Cfg::LDS_BYTES)[q * Cfg::NT + tid];
    if (n < a.ny) I[n] = v;
  }
}

// --------------------------------------------------------------------------
// Host-side launchers
// --------------------------------------------------------------------------
hipError_t launch_zernike_table(float* out, int n, int nj, hipStream_t st) {
  const int cells = n * n;
  hipLaunchKernelGGL(zernike_table_kernel, dim3((cells + 255) / 256), dim3(256), 0, st, out, n, nj);
  return hipGetLastError();
}

hipError_t launch_dft_panel(uint4* panel, int rows, int count, int centre, int n, int w, double k, double s_max,
                            double pitch, hipStream_t st) {
  const int total = rows * (w / 2);
  hipLaunchKernelGGL(dft_panel_kernel, dim3((total + 255) / 256), dim3(256), 0, st, (_Float16*)panel, rows, count, centre, n,
                     w, k, s_max, pitch);
  return hipGetLastError();
}

hipError_t launch_pupil_build(const PupilArgs& a, const float2* Q, const float* ztab, float2* P,
                              hipStream_t st) {
  const int cells = a.np * a.np;
  hipLaunchKernelGGL(pupil_build_kernel, dim3((cells + 255) / 256, a.nstk), dim3(256), 0, st, a, Q, ztab, P);
  return hipGetLastError();
}

hipError_t launch_pupil_build_folded(const FoldArgs& a, const float2* Q, const float* ztab, float2* Pf, int nhp,
                                     hipStream_t st) {
  const int blocks = (4 * nhp * nhp + 255) / 256;
  // stacks per thread: as many as leave four workgroups for each of 256 CUs
  const int group = std::min(kFoldGroup, std::max(1, a.nstk * blocks / 1024));
  // (room for 24 terms keeps two more waves on a SIMD than room for all 36)
  const auto kernel = a.max_zernike == 0    ? pupil_build_folded_kernel<0>
                      : a.max_zernike <= 24 ? pupil_build_folded_kernel<24>
                                            : pupil_build_folded_kernel<RWPSF_MAX_ZERNIKE>;
  hipLaunchKernelGGL(kernel, dim3(blocks, (a.nstk + group - 1) / group), dim3(256), 0, st, a, Q,
                     ztab, Pf, nhp, group);
  return hipGetLastError();
}

template <class Cfg, int PZ, int OCC>
static hipError_t gemm_pupil_launch(const Gemm1Args& a, hipStream_t st) {
  const int tiles = (4 * a.nhp * PZ / Cfg::BM) * (a.nyp / Cfg::BN);
  const int nblocks = a.nstk * ((a.nzs + PZ - 1) / PZ) * a.nc * tiles;
  hipLaunchKernelGGL((gemm_pupil_kernel<Cfg, PZ, OCC>), dim3(nblocks), dim3(Cfg::NT), Cfg::LDS_BYTES, st, a);
  return hipGetLastError();
}

template <class Cfg, int OCC>
static hipError_t gemm_image_launch(const Gemm2Args& a, hipStream_t st) {
  const int tiles = (2 * a.nyp / Cfg::BM) * (a.nxp / Cfg::BN);
  const int nblocks = a.nstk * a.nzs * tiles;
  hipLaunchKernelGGL((gemm_image_kernel<Cfg, OCC>), dim3(nblocks), dim3(Cfg::NT), Cfg::LDS_BYTES, st, a);
  return hipGetLastError();
}

// Compute units of the current device (queried once per device).
int device_cus() {
  static int cus[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cus[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cus[dev] = n;
  }
  return cus[dev];
}

// A launch whose large tiles would give fewer than two workgroups per CU (a few planes, e.g.
// one image) takes the small tiles instead: its time is then set by how many CUs work on
// it, not by the tile efficiency.
hipError_t launch_gemm_pupil(const Gemm1Args& a, hipStream_t st) {
  const long long work = (long long)a.nstk * a.nzs * a.nc;
  const bool few = work * ((4 * a.nhp + 127) / 128) * ((a.nyp + 127) / 128) < 2LL * device_cus();
  if (few) return gemm_pupil_launch<CfgPupilS, 1, 2>(a, st);
  if (a.nyp % 128 == 0) return gemm_pupil_launch<CfgPupil, 2, 2>(a, st);
  return gemm_pupil_launch<CfgPupilN, 2, 2>(a, st);
}

hipError_t launch_gemm_image(const Gemm2Args& a, hipStream_t st) {
  const long long work = (long long)a.nstk * a.nzs;
  const bool few = work * ((a.nxp + 127) / 128) * ((2 * a.nyp + 127) / 128) < 2LL * device_cus();
  const long long blocks = work * (2 * a.nyp / CfgImageS::BM) * (a.nxp / CfgImageS::BN);
  if (few && blocks > device_cus()) return gemm_image_launch<CfgImageS, 2>(a, st);
  if (few) {
    hipLaunchKernelGGL(gemm_image_few_kernel<CfgImageS>, dim3((unsigned)blocks), dim3(a.nc * CfgImageS::NT),
                       a.nc * CfgImageS::LDS_BYTES, st, a);
    return hipGetLastError();
  }
  if (a.nxp % 128 == 0) return gemm_image_launch<CfgImage, 2>(a, st);
  return gemm_image_launch<CfgImageM, 2>(a, st);
}

hipError_t fourier_kernel_attributes() {
  const void* k[7] = {(const void*)gemm_pupil_kernel<CfgPupil, 2, 2>, (const void*)gemm_pupil_kernel<CfgPupilN, 2, 2>,
                      (const void*)gemm_pupil_kernel<CfgPupilS, 1, 2>, (const void*)gemm_image_kernel<CfgImage, 2>,
                      (const void*)gemm_image_kernel<CfgImageM, 2>, (const void*)gemm_image_kernel<CfgImageS, 2>,
                      (const void*)gemm_image_few_kernel<CfgImageS>};
  const int bytes[7] = {CfgPupil::LDS_BYTES, CfgPupilN::LDS_BYTES, CfgPupilS::LDS_BYTES,
                        CfgImage::LDS_BYTES, CfgImageM::LDS_BYTES, CfgImageS::LDS_BYTES, 3 * CfgImageS::LDS_BYTES};
  for (int i = 0; i < 7; ++i) {
    const hipError_t e = hipFuncSetAttribute(k[i], hipFuncAttributeMaxDynamicSharedMemorySize, bytes[i]);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace rw
