// Internal declarations of the rwpsf library (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <vector>

#include "rwpsf.h"

#define RW_HD __host__ __device__ inline

namespace rw {

constexpr double kPi = 3.14159265358979323846;
constexpr double kTwoPi = 6.28318530717958647692;

// ---------------------------------------------------------------------------
// Bessel functions of the first kind, J_n(x) = (1/pi) int_0^pi cos(n t - x sin t) dt.
// The integrand is 2 pi periodic and even about pi, so the M-point trapezoid rule
// on [0, 2 pi) is exact up to the aliased orders J_{n +- M} (Jacobi-Anger).  J_nu(x)
// decays past the turning point nu = x on the scale x^(1/3) (Airy transition), so
// M = n + x + 12 x^(1/3) + 32 keeps the aliased terms below 1e-20.
// ---------------------------------------------------------------------------
RW_HD double bessel_j(int n, double x) {
  if (x == 0.0) return n == 0 ? 1.0 : 0.0;
  const double ax = fabs(x);
  int m = n + (int)ceil(ax + 12.0 * cbrt(ax)) + 32;
  m += m & 1;
  const double h = kTwoPi / m;
  double s = 0.0;
  for (int i = 0; i < m; ++i) {
    const double t = h * i;
    s += cos(n * t - x * sin(t));
  }
  return s / m;
}

// ---------------------------------------------------------------------------
// Noll-indexed Zernike polynomials, orthonormal on the unit disk (Sec. 3.4.2).
// ---------------------------------------------------------------------------
RW_HD void noll_nm(int j, int* n_out, int* m_out) {
  int n = 0;
  while ((n + 1) * (n + 2) / 2 < j) ++n;
  const int p = j - n * (n + 1) / 2 - 1;
  const int am = (n % 2 == 0) ? 2 * ((p + 1) / 2) : 2 * (p / 2) + 1;
  *n_out = n;
  *m_out = (am == 0) ? 0 : ((j % 2 == 0) ? am : -am);
}

RW_HD double factorial_d(int k) {
  double f = 1.0;
  for (int i = 2; i <= k; ++i) f *= i;
  return f;
}

// Coefficient of r^(n-2s) in R_n^|m|, times the orthonormalisation factor.
RW_HD double zernike_radial_coef(int n, int am, int s) {
  const double sign = (s & 1) ? -1.0 : 1.0;
  return sign * factorial_d(n - s) /
         (factorial_d(s) * factorial_d((n + am) / 2 - s) * factorial_d((n - am) / 2 - s));
}

RW_HD double zernike_noll(int j, double r, double cp, double sp) {
  int n, m;
  noll_nm(j, &n, &m);
  const int am = m < 0 ? -m : m;
  double rad = 0.0;
  for (int s = 0; s <= (n - am) / 2; ++s) rad += zernike_radial_coef(n, am, s) * pow(r, n - 2 * s);
  if (m == 0) return sqrt((double)(n + 1)) * rad;
  // cos(am p), sin(am p) by the angle-addition recurrence
  double c = 1.0, s = 0.0;
  for (int i = 0; i < am; ++i) {
    const double c2 = c * cp - s * sp;
    s = s * cp + c * sp;
    c = c2;
  }
  return sqrt(2.0 * (n + 1)) * rad * (m > 0 ? c : s);
}

// ---------------------------------------------------------------------------
// Gibson-Lanni OPD (Sec. 3.4.1, eq. "stratified layers general formula"), with
// t_i from the focusing condition eq. "gibson lanni t_i" as printed.  Returns
// W = (re, im): a principal-branch square root makes im >= 0 past a critical angle.
// ---------------------------------------------------------------------------
struct GLParams {
  double k0;  // 2 pi / lambda
  double n_i, n_s, n_g, n_g_d, n_i_d;
  double t_g, t_g_d, t_i_d;
};

RW_HD double gl_ti(const GLParams& g, double t_s) {
  return t_s + g.n_i * (-t_s / g.n_s - g.t_g / g.n_g + g.t_g_d / g.n_g_d + g.t_i_d / g.n_i_d);
}

// sqrt(n^2 - q) for real arguments, principal branch: (re, im)
RW_HD void csqrt_real(double v, double* re, double* im) {
  if (v >= 0.0) {
    *re = sqrt(v);
    *im = 0.0;
  } else {
    *re = 0.0;
    *im = sqrt(-v);
  }
}

RW_HD void gl_opd(const GLParams& g, double t_s, double sin_t, double* w_re, double* w_im) {
  const double q = g.n_i * g.n_i * sin_t * sin_t;
  const double t_i = gl_ti(g, t_s);
  const double n[5] = {g.n_s, g.n_i, g.n_i_d, g.n_g, g.n_g_d};
  const double t[5] = {t_s, t_i, -g.t_i_d, g.t_g, -g.t_g_d};
  double re = 0.0, im = 0.0;
  for (int i = 0; i < 5; ++i) {
    double a, b;
    csqrt_real(n[i] * n[i] - q, &a, &b);
    re += t[i] * a;
    im += t[i] * b;
  }
  *w_re = g.k0 * re;
  *w_im = g.k0 * im;
}

// Reduce an FP64 phase to [-pi, pi] before it is rounded to FP32.
RW_HD double reduce_2pi(double p) { return p - kTwoPi * rint(p * (1.0 / kTwoPi)); }

// sin and cos of 2 pi t: t is reduced to [-1/2, 1/2] in FP64 and rounded once to FP32,
// then the hardware sine and cosine, which take their argument in revolutions (on
// [-1/2, 1/2] their largest error measured 1.3e-7, that of sincosf 1.5e-7).
__device__ __forceinline__ void sincos_rev(double t, float* s, float* c) {
  const float r = (float)(t - rint(t));
  *s = __builtin_amdgcn_sinf(r);
  *c = __builtin_amdgcn_cosf(r);
}

// A phase reduced to half turns in [-1, 1], for sincospif: slower than sincos_rev and twice as
// exact, for factors that every plane of an emitter shares.
__device__ __forceinline__ float half_turns(double phase) {
  const double t = phase * (1.0 / kTwoPi);
  return (float)(2.0 * (t - rint(t)));
}

// ---------------------------------------------------------------------------
// Host helpers
// ---------------------------------------------------------------------------
int gauss_legendre(int n, double a, double b, double* x, double* w);
void set_hip_error(hipError_t e);

struct PlanDevice;  // per-form device state

// Power-of-two scales of the Fourier form's operands.
struct PupilScales {
  int pf_exp[3] = {0, 0, 0};              // Q and the folded pupils of a component carry 2^pf_exp
  float tscale = 1.f;                     // T is multiplied by it when it is written
  unsigned escale = 0;                    // fields per unit of the image product's sums: exponents + 512, 10 bits each
};

}  // namespace rw

// ---------------------------------------------------------------------------
// Plan
// ---------------------------------------------------------------------------
struct rwpsf_plan {
  int device = 0;
  rwpsf_optics opt{};
  rwpsf_grid grid{};
  rwpsf_numerics num{};
  std::vector<double> z;
  double k = 0, s_max = 0, theta_max = 0;
  int nc = 3;                   // output channels: 3 (vectorial model) or 1 (scalar model)
  rw::GLParams gl{};
  size_t device_bytes = 0;
  std::vector<void*> allocations;

  // Fourier form (device operands zero-padded to whole GEMM tiles)
  int np = 0, nxp = 0, nyp = 0; // padded pupil size and output widths
  double* d_z = nullptr;        // [nz]
  double* d_ksz = nullptr;      // [np][np] k * s_z (0 outside the disk)
  float2* d_Q = nullptr;        // [3][np][np] ds^2 a e_inf,c / s_z (0 outside)
  int nhp = 0;                  // folded pupil cells per axis, padded (2 nhp = np)
  double* d_kszf = nullptr;     // [nhp][nhp] k * s_z on the folded cells
  uint4* d_B1 = nullptr;        // split-f16 panel of nyp rows n, k = 2lf + p: cos / sin (k s_y[lf] y_n)
  uint4* d_A2 = nullptr;        // split-f16 panel of nxp rows m, k = 2jf + p: cos / sin (k s_x[jf] x_m)
  rw::PupilScales scales;       // of the Fourier form's operands
  float* d_ztab = nullptr;      // [RWPSF_MAX_ZERNIKE][N][N] Noll basis on the pupil cells
  float2* d_P = nullptr;        // workspace [chunk][3][np][np]
  float2* d_Pf = nullptr;       // workspace [chunk][3][2 nhp][2 nhp] folded pupils
  uint4* d_T = nullptr;         // workspace [planes][3] split-f16 panels of 2 nyp rows 2n + ri, k = q
  size_t T_planes = 0;          // capacity of d_T in stack-planes
  // adjoint (built on first use)
  bool adj_ready = false;       // the tables and d_shares, d_adjPf, d_adjD, d_adjMax are complete
  uint4* d_adjTx = nullptr;     // split-f16 panel of 2 nhp columns 2jf + p, k = x pixel
  uint4* d_adjTy = nullptr;     // split-f16 panel of 2 nhp columns 64 (lf / 32) + 32 p + lf % 32, k = y pixel
  int* d_adjEx = nullptr;       // [adj_stacks][nz][3] power-of-two scales of 2 dL/dI E
  int adj_stacks = 0;
  float* d_adjMax = nullptr;    // [workgroups][3] largest parts of 2 dL/dI E in runs of a plane's pixels
  float2* d_adjPf = nullptr;    // [64 stacks][3][2 nhp][2 nhp] folded pupils of an adjoint launch
  float* d_partial = nullptr;   // [groups][np][np] a launch's per-(stack, component, run of planes, part) dL/dPhi
  int partial_stacks = 0;       // calls of up to that many stacks (and of more) have room there
  double* d_shares = nullptr;   // [RWPSF_MAX_ZERNIKE][workgroups of the reduction] shares of dL/dc
  float2* d_adjD = nullptr;     // [nz][nhp][nhp] exp(i k s_z z) of the plan's planes on the folded cells
  double* d_runs = nullptr;     // [1 + partial runs][N][N] sum so far, first level of the dL/dPhi reduction
  int P_stacks = 0;             // capacity of d_P in stacks

  // chirp-z evaluation of the Fourier form
  // FFT lengths, most output columns per workgroup, their stride in LDS
  int czt_Ly = 0, czt_Lx = 0, czt_cb = 0, czt_stride = 0;
  float2* d_czt = nullptr;       // tables: pre/post/chat along y, then along x
  float2 *czt_pre_y = nullptr, *czt_post_y = nullptr, *czt_chat_y = nullptr;
  float2 *czt_pre_x = nullptr, *czt_post_x = nullptr, *czt_chat_x = nullptr;
  float2* d_czt_T = nullptr;     // workspace [planes][3][N][ny]
  size_t czt_planes = 0;

  // Bessel form
  int n_theta_total = 0;        // nodes after the critical-angle split
  double* d_theta = nullptr;    // [T] nodes
  double* d_wtheta = nullptr;   // [T] weights
  double* d_node = nullptr;     // [T] BesselNode: what the pupil of a node takes from the plan
  int bessel_mode = 0;          // 0 vectorial, 1 vectorial with Fresnel factors, 2 scalar
  float* d_btab = nullptr;      // [T][G][R] w_t h_g(t) J_{n_g}(k rho_r sin t)
  uint4* d_bpanel = nullptr;    // d_btab as a split-f16 panel of btab_ld columns, group g times 2^tab_exp[g]
  int btab_ld = 0, tab_exp[5] = {0, 0, 0, 0, 0};
  int phi_exp = 0;              // Phi is split after multiplication by 2^phi_exp
  double* d_fq = nullptr;       // [T][4] Fresnel products q_s, q_p per node (Fresnel mode)
  float2* d_phi = nullptr;      // workspace [T][stacks][nz][V] pupil x defocus (x q_v)
  float2* d_In = nullptr;       // workspace [stacks][nz][V][re/im][G][R]
  int bessel_stacks = 0;        // capacity of the Bessel workspaces
  std::vector<double> fused_cum;   // Bessel, few stacks: accumulated cost per radial base sample
  float* scratch = nullptr;     // device address of the allocation-free entry point's fixed array
  double drho = 0;              // radial sample pitch
  // Bessel-form adjoint (built on first use)
  bool adjb_ready = false;      // all of the following is complete
  uint4* d_bpanelT = nullptr;   // the transposed table [G][R][T] as a split-f16 panel
  int* d_GInEx = nullptr;       // [stacks nz V] exponents of the row pairs of G_In
  float* d_GIn = nullptr;       // workspace [2 stacks nz V] rows of [G][R] gradients of the radial samples
  float* d_GPhi = nullptr;      // workspace [2 stacks nz V][T] gradient of Phi
  double2* d_adjX = nullptr;    // workspace [stacks][T] sum_z conj(G_Phi) Phi
  double* d_adjnode = nullptr;  // [T][7] k cos t, dW/dt_s (re, im), 2 pi Z_{1,4,11,22}
  double* d_dcp = nullptr;      // [max stacks][4] per-stack shares of dL/dc

  // per-kernel timing (opt-in)
  struct TimingRec {
    int kernel;
    hipEvent_t a, b;
  };
  bool timing = false;
  std::vector<TimingRec> timing_recs;
  std::vector<hipEvent_t> event_pool;
  double timing_ms[RWPSF_KERNEL_COUNT] = {};
  int64_t timing_launches[RWPSF_KERNEL_COUNT] = {};
  int time_begin(int kernel, hipStream_t st);   // returns a record index or -1
  void time_end(int rec, hipStream_t st);
  void timing_flush();

  ~rwpsf_plan();
};
