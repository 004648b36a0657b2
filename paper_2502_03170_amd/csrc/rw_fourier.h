// Kernel argument blocks and launchers of the Fourier form (internal).
#pragma once

#include "rw_common.h"

namespace rw {

constexpr int kPupilStacks = 8;  // stacks per launch of unfolded pupils (the size of their workspace)
constexpr int kFoldStacks = 16;  // stacks per launch of folded pupils, fewer if each has more than
constexpr int kFoldTerms = 384;  // 23 Zernike terms: they share this room (by-value arguments stay < 4 KB)
constexpr int kGemmStacks = 64;  // stacks per GEMM launch (folded pupils of several launches): fewer
                                 // kernel prologues and tails, and small outputs need many stacks per
                                 // launch to fill the GPU

struct PupilStack {
  double t_s, x0, y0;
  double coef[RWPSF_MAX_ZERNIKE];   // waves
  const float* w0;
};

// Channels: nc = 3 (vectorial model, x, y, z) or 1 (scalar model); every per-channel
// array below holds nc channels.
struct PupilGeom {
  int n, np, nstk, max_zernike, gibson_lanni, nc;   // n: pupil cells per axis, np: padded stride
  double s_max, k;
  GLParams gl;
};
struct PupilArgs : PupilGeom {
  PupilStack s[kPupilStacks];
};
static_assert(sizeof(PupilArgs) <= 4000, "kernel arguments are passed by value (4 KB limit)");

// Arguments of the folded pupils: the coefficients are packed, max_zernike a stack (a read of
// RWPSF_MAX_ZERNIKE from any stack's first stays inside; past the stack's own terms it meets the next
// stack's, which are finite as the caller gave them, times zero).
struct FoldStack {
  double t_s, x0, y0;
  const float* w0;
};
struct FoldArgs : PupilGeom {
  FoldStack s[kFoldStacks];
  double coef[kFoldTerms];          // waves
};
static_assert(sizeof(FoldArgs) <= 4000, "kernel arguments are passed by value (4 KB limit)");

// Device operands are zero-padded: np = n rounded up to 64, nxp = nx rounded up
// to 128, nyp = ny rounded up to 128 (64 for axes of at most 64 pixels), and the folded pupil axis nh = ceil(n/2) to
// nhp = nh rounded up to 32 (so 2 nhp = np).

// Operands of the two GEMMs are split in f16 halves (hgemm.h).  Their power-of-two scales
// (PupilScales) keep the halves in range: Q, and with it the folded pupils, carries 2^pf_exp, so that no
// folded value (a sum over up to four mirrors, each of unit phase factor times the given largest
// amplitude of the cell) exceeds 2^15, each component by itself (at a numerical aperture of 0.02 the
// y component of x-polarised light is 2^-14 of the x component; with one scale for both its halves were
// subnormal, its error 5.1e-7 of its own norm, 1.7e-7 in FP32 products, 9.8e-8 so); the DFT tables carry
// 2^kTabExp; T = Pf B1, bounded by the largest row sum of |Pf|, is multiplied by tscale to stay under 2^15
// when it is split (rows over cells differ by a few bits from component to component: one tscale for
// all).  The halves then neither overflow nor, down to about 2^-18 of the bounds, lose bits to subnormal
// halves.  escale, a power of two, turns the image GEMM's sums into fields.
constexpr int kTabExp = 6;
// escale of component c, formed from the packed exponents on the scalar path (an array of three in the
// arguments is a load on the critical path of a loop over components: 1 us of a call's 33).
__device__ __forceinline__ float component_scale(unsigned exps, int c) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(ldexpf(1.f, (int)(exps >> 10 * c & 1023) - 512))));
}
// Scales of Q [nc][np][np] on the N x N cells, with the prefactor's mantissa; amplitude [np][np] or
// null.  Multiplies Q by them.
PupilScales pupil_scales(std::vector<float2>& Q, int nc, int N, int np, const double* amplitude, int pref_exp);

struct Gemm1Args {
  const float2* Pf;    // [nstk][nc][2 nhp][2 nhp]
  const double* kszf;  // [nhp][nhp] k s_z on the folded cells
  const double* z;     // plan planes
  const uint4* B1;     // panel of nyp rows n, k = 2lf + p: cos / sin (k s_y[lf] y_n)
  uint4* T;            // [nstk][nzs][nc] panels of 2 nyp rows 2n + ri, k = q
  double zoff[kGemmStacks];
  float tscale;
  int n, nhp, nyp, nstk, z0, nzs, nc;   // n: pupil cells per axis
};

struct Gemm2Args {
  const uint4* A2;     // panel of nxp rows m, k = 2jf + p: cos / sin (k s_x[jf] x_m)
  const uint4* T;      // [nstk][nzs][nc] panels of 2 nyp rows 2n + ri, k = q
  float2* E;           // [stacks][nz][nc][nx][ny] or null
  float* I;            // [stacks][nz][nx][ny] or null
  unsigned escale;     // packed powers of two: the prefactor's over the operand scales
  int vec;             // E and I rows allow 16- and 8-byte stores (ny even, aligned outputs)
  int nhp, nxp, nyp, nx, ny, nz, nstk, s_base, z0, nzs, nc;
};

inline int round_up(int v, int m) { return (v + m - 1) / m * m; }
constexpr int kPadPupil = 64, kPadX = 128, kPadY = 128, kFoldPad = 32, kPadSmall = 64;
// padding of an output axis of n pixels: 64 for n <= 64, else a multiple of 128
inline int pad_axis(int n) { return n <= kPadSmall ? kPadSmall : round_up(n, kPadX); }

hipError_t launch_zernike_table(float* out, int n, int nj, hipStream_t st);
// DFT table of `count` output pixels (pixel r at (r - centre) pitch) as a split-f16 panel
// of `rows` rows, k = 2f + p: 2^kTabExp {cos, sin}(wavenumber s_f x_r), zero past count and n
hipError_t launch_dft_panel(uint4* panel, int rows, int count, int centre, int n, int w, double wavenumber,
                            double s_max, double pitch, hipStream_t st);
hipError_t launch_pupil_build(const PupilArgs& a, const float2* Q, const float* ztab, float2* P,
                              hipStream_t st);
// Pf [nstk][nc][2 nhp][2 nhp] of the stacks of a (its np field is the stride of Q)
hipError_t launch_pupil_build_folded(const FoldArgs& a, const float2* Q, const float* ztab, float2* Pf, int nhp,
                                     hipStream_t st);
hipError_t launch_gemm_pupil(const Gemm1Args& a, hipStream_t st);
hipError_t launch_gemm_image(const Gemm2Args& a, hipStream_t st);
hipError_t fourier_kernel_attributes();
int device_cus();   // compute units of the current device

}  // namespace rw
