// Device-side shared definitions of the renderer: kernel argument blocks and
// the per-galaxy shape algebra (Section 2, steps 3 and 4).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "fft_reg.hpp"

namespace gfc {

constexpr int kKmax = 16;
// -2 pi^2 log2(e): the Gaussian transform exp(-2 pi^2 q) written as exp2(kQ q).
constexpr float kQ = -0x1.c7a47ep+4f;
// -log2(e) / 2: a real-space Gaussian exp(-u^T S^-1 u / 2) as exp2(kHalfLog2e q).
constexpr float kHalfLog2e = -0x1.715476p-1f;
constexpr float kInv2Pi = 0x1.45f306p-3f;

// Galaxy parameters and everything a render launch needs.
struct RenderArgs {
  const float* x;
  const float* y;
  const float* flux;
  const float* r_e;
  const float* e1;
  const float* e2;
  const int32_t* mix_id;   // may be null (table 0)
  const float* amp;        // [n_tables][kKmax]
  const float* var;        // [n_tables][kKmax]
  const int32_t* K;        // [n_tables]
  int n_tables;
  int kmax;                // max K over the tables
  float flat_v2;           // the second smallest variance of a table, the largest over the tables (see flat_shared)
  float cdinv[4];          // CD^{-1}, row-major (identity by default)
  float pg[6];             // PSF Gaussian: mu_x, mu_y, c_xx, c_xy, c_yy, amp
  const float2* psf_main;  // PSF spectrum, lane-permuted columns 0..W/2-1
  const float2* psf_nyq;   // PSF spectrum, Nyquist column k_x = W/2, [W]
  float* out;              // [n][W][W]
  int64_t n;
  unsigned flags;
  unsigned long long* invalid;  // device counter of invalid galaxies
  // Spatially varying (eigen-)PSF; eig_J == 0 for a constant PSF.
  int eig_J;                // components; their spectra follow each other eig_stride float2 apart
  int eig_degree;           // polynomial degree (0..3)
  int64_t eig_stride;
  const float* eig_coef;    // [J][T], T = (degree + 1)(degree + 2) / 2
  const float* eig_mom;     // [J][6]: sum, sum x, sum y, sum x^2, sum x y, sum y^2 about the centre pixel
  float eig_norm[4];        // x_off, 1 / x_scale, y_off, 1 / y_scale
  const float* psf_px;      // [n] image position of each galaxy (eigen PSF only)
  const float* psf_py;
  // Stamps of several constant PSFs in one launch (serving): galaxy i uses
  // PSF psf_id[i] of these tables instead of psf_main / psf_nyq / pg.  An
  // index outside [0, n_psf) makes the galaxy invalid.  Null psf_id: one PSF.
  const int32_t* psf_id;              // [n]
  const float2* const* psf_main_tab;  // [n_psf] spectra for this W, laid out as psf_main
  const float2* const* psf_nyq_tab;   // [n_psf] Nyquist columns
  const float* pg_tab;                // [n_psf][6] PSF Gaussians
  int n_psf;
  // Galaxies with a mixture of their own (forward render only; mix_id, K and
  // n_tables are then unused): see component_mix.
  int prof;                 // kProfTable, kProfSersic or kProfComposite
  const float* prof_a;      // [n] Sersic index | bulge fraction
  const float* prof_b;      // [n]              | bulge radius ratio
  const float* prof_grid;   // [S] Sersic indices; amp and var are then [S][k1]
  int prof_S;
  int prof_k1, prof_k2;     // components (Sersic: k1; composite: disk, bulge)
  int prof_disk, prof_bulge;  // the composite's tables
};

enum : int { kProfTable = 0, kProfSersic = 1, kProfComposite = 2 };

constexpr int kEigMax = 16;     // eigen-PSF components
constexpr int kEigDegMax = 3;   // polynomial degree

enum : unsigned { kForceFourier = 1u, kForceReal = 2u, kRampLinear = 4u, kLanczos3 = 8u, kAccumulate = 16u };

// Per-galaxy state shared by every step.
struct Galaxy {
  float x0, y0, flux;
  float fx, fy;      // fractional centre (in [0, 1))
  int nx, ny;        // integer centre modulo W
  float b11, b12, b22;  // pixel-space covariance per unit mixture variance
  int table, K;
  bool ok;
};

// Four floats in memory that are aligned as floats are.
typedef float v4f_any __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ bool finitef(float v) { return __builtin_isfinite(v); }

// Step 3: C_i = v_i B with B = A A^T, A = CD^{-1} E.  With c^2, s^2 and cs of
// the position angle written through e1, e2 (Appendix A), E E^T is
// r_e^2/(1+e)^2 [[1+e^2-2e1, 2e2], [2e2, 1+e^2+2e1]] -- no trigonometry.
// A galaxy's inputs as they are stored.
struct GalaxyIn {
  float x, y, flux, re, e1, e2;
  int table;
};

__device__ __forceinline__ GalaxyIn load_galaxy_in(const RenderArgs& p, int64_t g) {
  return GalaxyIn{p.x[g], p.y[g], p.flux[g], p.r_e[g], p.e1[g], p.e2[g], p.mix_id ? p.mix_id[g] : 0};
}

// PROF: the launch may have mixtures of the galaxies' own (p.prof).
template <int W, bool PROF = false>
__device__ __forceinline__ Galaxy make_galaxy(const RenderArgs& p, const GalaxyIn& in) {
  Galaxy G;
  G.x0 = in.x;
  G.y0 = in.y;
  G.flux = in.flux;
  const float re = in.re, e1 = in.e1, e2 = in.e2;
  // The table follows from mix_id alone (an index out of range takes table
  // 0 and makes the galaxy invalid), so its reads need not wait for the
  // other parameters.
  const bool own = PROF && p.prof != kProfTable;
  const bool table_ok = own || (in.table >= 0 && in.table < p.n_tables);
  G.table = !own && table_ok ? in.table : 0;
  G.K = own ? p.prof_k1 + p.prof_k2 : p.K[G.table];
  const float esq = e1 * e1 + e2 * e2;
  G.ok = finitef(G.x0) && finitef(G.y0) && finitef(G.flux) && finitef(re) && finitef(e1) &&
         finitef(e2) && re > 0.f && esq < 1.f && fabsf(G.x0) <= 8388608.f &&
         fabsf(G.y0) <= 8388608.f && table_ok;
  // An invalid galaxy renders as NaN everywhere: a NaN flux propagates
  // through every product of the Fourier and real-space paths.
  if (!G.ok) G.flux = __builtin_nanf("");
  const float fxf = floorf(G.x0), fyf = floorf(G.y0);
  if (p.flags & kLanczos3) {  // rendered at the integer position; the stamp is shifted afterwards
    G.x0 = fxf;
    G.y0 = fyf;
  }
  G.fx = G.ok ? G.x0 - fxf : 0.f;
  G.fy = G.ok ? G.y0 - fyf : 0.f;
  G.nx = G.ok ? ((int)(fxf - (float)W * floorf(fxf * (1.f / W)))) & (W - 1) : 0;
  G.ny = G.ok ? ((int)(fyf - (float)W * floorf(fyf * (1.f / W)))) & (W - 1) : 0;
  // Hardware square root and reciprocal (about 1 ulp each): the covariance
  // needs no correctly rounded operations, and these are a few instructions
  // instead of some thirty.
  const float e = __builtin_amdgcn_sqrtf(esq);
  const float s = (re * re) * __builtin_amdgcn_rcpf((1.f + e) * (1.f + e));
  const float c11 = s * (1.f + esq - 2.f * e1);
  const float c12 = s * (2.f * e2);
  const float c22 = s * (1.f + esq + 2.f * e1);
  // B = M C M^T with M = CD^{-1}
  const float m00 = p.cdinv[0], m01 = p.cdinv[1], m10 = p.cdinv[2], m11 = p.cdinv[3];
  const float p00 = fmaf(m00, c11, m01 * c12), p01 = fmaf(m00, c12, m01 * c22);
  const float p10 = fmaf(m10, c11, m11 * c12), p11 = fmaf(m10, c12, m11 * c22);
  G.b11 = fmaf(p00, m00, p01 * m01);
  G.b12 = fmaf(p00, m10, p01 * m11);
  G.b22 = fmaf(p10, m10, p11 * m11);
  return G;
}

template <int W, bool PROF = false>
__device__ __forceinline__ Galaxy load_galaxy(const RenderArgs& p, int64_t g) {
  return make_galaxy<W, PROF>(p, load_galaxy_in(p, g));
}

// A galaxy's own mixture (p.prof): its place in the Sersic grid, cell s and
// fraction t, or the composite's bulge fraction t and radius ratio r.
struct Profile {
  float t, r;
  int s;
  bool ok;
};

// From the galaxy's prof_a and prof_b values, by the LANES consecutive lanes
// that hold them (a power of two; every lane of the wavefront takes part): a
// lane compares one grid index, so the search is one load deep for any grid
// of up to LANES + 2 indices.
template <int LANES>
__device__ __forceinline__ Profile make_profile(const RenderArgs& p, float a, float b) {
  if (p.prof == kProfComposite)
    return Profile{a, b, 0, a >= 0.f && a <= 1.f && b > 0.f && __builtin_isfinite(b)};
  const float* grid = p.prof_grid;
  const int S = p.prof_S, lane = (int)__lane_id();
  int s = 0;  // the last cell that starts at or below a; 0 if none
  for (int i0 = 1; i0 < S - 1; i0 += LANES) {
    const int i = i0 + (lane & (LANES - 1));
    unsigned long long le = __ballot(i < S - 1 && grid[min(i, S - 1)] <= a);
    if constexpr (LANES < 64) le = (le >> (lane & ~(LANES - 1))) & ((1ull << LANES) - 1ull);
    s += __popcll(le);
  }
  const bool ok = __builtin_isfinite(a) && a >= grid[0] && a <= grid[S - 1];
  const float t = ok ? (a - grid[s]) / (grid[s + 1] - grid[s]) : 0.f;
  return Profile{t, 1.f, s, ok};
}

// Amplitude and variance of component k < G.K.  Sersic: interpolated between
// the cell's two grid indices.  Composite: the disk's components with
// amplitudes (1 - t) A_d, then the bulge's with t A_b and variances r^2 v_b.
template <bool PROF>
__device__ __forceinline__ float2 component_mix(const RenderArgs& p, const Galaxy& G, const Profile& f, int k) {
  if (!PROF || p.prof == kProfTable) return make_float2(p.amp[G.table * kKmax + k], p.var[G.table * kKmax + k]);
  const float t0 = 1.f - f.t;
  if (p.prof == kProfSersic) {
    const int K = p.prof_k1, i = f.s * K + k;
    return make_float2(fmaf(t0, p.amp[i], f.t * p.amp[i + K]), fmaf(t0, p.var[i], f.t * p.var[i + K]));
  }
  const bool disk = k < p.prof_k1;
  const int i = disk ? p.prof_disk * kKmax + k : p.prof_bulge * kKmax + (k - p.prof_k1);
  const float A = p.amp[i], v = p.var[i];
  return disk ? make_float2(t0 * A, v) : make_float2(f.t * A, (f.r * f.r) * v);
}

// Fourier bins where a component's exponent (log2 of its share of the
// component's amplitude) is below -kSkipLog2 may be skipped: every skipped
// value is below 2^-40 of the amplitude, far under FP32 rounding of the stamp.
constexpr float kSkipLog2 = 40.f;

// A lower bound on the smallest eigenvalue of the galaxy's shape matrix B,
// so that q(nu, omega) >= lambda (nu^2 + omega^2): the eigenvalue of the
// FP32 matrix in double precision (no cancellation at any ellipticity),
// less 0.1 per cent.
__device__ __forceinline__ float shape_min_eig(const Galaxy& G) {
  const double a = G.b11, b = G.b12, d = G.b22;
  const double h = 0.5 * (a - d);
  const double lam = 0.5 * (a + d) - sqrt(h * h + b * b);
  return lam > 0.0 ? (float)(0.999 * lam) : 0.f;
}

// A kernel's first argument A, read through a pointer that is renewed
// opaquely at each call: its fields are reloaded through the scalar cache
// there instead of being held in registers from the kernel's start (inside
// a persistent loop, or late in a long kernel).
template <typename A>
__device__ __forceinline__ const A& kernel_args_renewed() {
  typedef const __attribute__((address_space(4))) A* KArgs;
  KArgs pk = (KArgs)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(pk));
  return *(const A*)pk;
}

__device__ __forceinline__ float uniform_f(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}

// For a wavefront (or workgroup) that renders one stamp: the galaxy's values
// are the same in every lane, so they move to scalar registers.  This frees
// vector registers and turns the mixture-table reads into scalar loads.
__device__ __forceinline__ void make_uniform(Galaxy& G) {
  G.x0 = uniform_f(G.x0);
  G.y0 = uniform_f(G.y0);
  G.flux = uniform_f(G.flux);
  G.fx = uniform_f(G.fx);
  G.fy = uniform_f(G.fy);
  G.nx = __builtin_amdgcn_readfirstlane(G.nx);
  G.ny = __builtin_amdgcn_readfirstlane(G.ny);
  G.b11 = uniform_f(G.b11);
  G.b12 = uniform_f(G.b12);
  G.b22 = uniform_f(G.b22);
  G.table = __builtin_amdgcn_readfirstlane(G.table);
  G.K = __builtin_amdgcn_readfirstlane(G.K);
  G.ok = __builtin_amdgcn_readfirstlane((int)G.ok) != 0;
}

// Weight of eigen-PSF component j at normalised position (u, v): the sum
// over polynomial terms u^a v^b (a + b <= degree, ordered by the power of v,
// then of u) of the component's coefficients.  up/vp hold powers 0..3.
__device__ __forceinline__ float eigen_weight(const RenderArgs& p, int j, const float (&up)[kEigDegMax + 1],
                                              const float (&vp)[kEigDegMax + 1]) {
  const int D = p.eig_degree;
  const float* cf = p.eig_coef + j * ((D + 1) * (D + 2) / 2);
  float c = 0.f;
  static_for<0, kEigDegMax + 1>([&](auto bb) {
    constexpr int b = decltype(bb)::value;
    static_for<0, kEigDegMax + 1 - b>([&](auto aa) {
      constexpr int a = decltype(aa)::value;
      if (a + b <= D) c = fmaf(cf[b * (D + 1) - b * (b - 1) / 2 + a], up[a] * vp[b], c);
    });
  });
  return c;
}

// The PSF Gaussian {mu_x, mu_y, c_xx, c_xy, c_yy, amp} of the weighted sum
// of components: moments are linear in the weights.
__device__ __forceinline__ void eigen_gauss(const float (&mom)[6], float (&pg)[6]) {
  const float F = mom[0], rF = 1.f / F;
  const float mx = mom[1] * rF, my = mom[2] * rF;
  pg[0] = mx;
  pg[1] = my;
  pg[2] = fmaf(mom[3], rF, -mx * mx);
  pg[3] = fmaf(mom[4], rF, -mx * my);
  pg[4] = fmaf(mom[5], rF, -my * my);
  pg[5] = F;
}

// (sin(pi r), cos(pi r)) for |r| < 2^22, without the special-value handling
// of the library routine.  r = j/2 + f with j = rint(2 r) and |f| <= 1/4 (f is
// exact); sin(pi f) and cos(pi f) are their Taylor series through f^9 and
// f^10 (truncation below 2e-9 on |f| <= 1/4), and j mod 4 picks the quadrant.
GFC_HD void sincospi_poly(float r, float* s_out, float* c_out) {
  const float j = rintf(2.f * r);
  const float f = fmaf(-0.5f, j, r);
  const float f2 = f * f;
  float sp = fmaf(f2, 0x1.5078340p-4f, -0x1.32d2ccp-1f);  // pi^9/9!, -pi^7/7!
  sp = fmaf(f2, sp, 0x1.466bc6p+1f);                      // pi^5/5!
  sp = fmaf(f2, sp, -0x1.4abbcep+2f);                     // -pi^3/3!
  sp = fmaf(f2, sp, 0x1.921fb6p+1f) * f;                  // pi
  float cp = fmaf(f2, -0x1.a6d1f2p-6f, 0x1.e1f506p-3f);   // -pi^10/10!, pi^8/8!
  cp = fmaf(f2, cp, -0x1.55d3c8p+0f);                     // -pi^6/6!
  cp = fmaf(f2, cp, 0x1.03c1f0p+2f);                      // pi^4/4!
  cp = fmaf(f2, cp, -0x1.3bd3ccp+2f);                     // -pi^2/2!
  cp = fmaf(f2, cp, 1.f);
  const int q = (int)j;
  const float s = (q & 1) ? cp : sp;
  const float c = (q & 1) ? sp : cp;
  *s_out = __builtin_bit_cast(float, __builtin_bit_cast(int, s) ^ ((q & 2) << 30));
  *c_out = __builtin_bit_cast(float, __builtin_bit_cast(int, c) ^ (((q + 1) & 2) << 30));
}

// -2 (n + f) k / W less whole turns, as hi + lo / pi: hi is the rounded sum of
// the products for f and for the exact n k mod W, lo / pi the two roundings.
// Contraction is off: fused with the differences, the first product would put
// its rounding into them, and it would be counted twice.
template <int W>
GFC_HD void shift_arg(float f, int n, int k, float* hi_out, float* lo_out) {
#pragma clang fp contract(off)
  const float g = -2.f * f, nu = (float)k * (1.f / W);
  const float p = g * nu, pe = fmaf(g, nu, -p);
  const int m = (n * k) & (W - 1);
  const float b = (float)(m < W / 2 ? m : m - W) * (-2.f / W);
  const float hi = p + b, bb = hi - p;
  *hi_out = hi;
  *lo_out = 3.14159265f * (((p - (hi - bb)) + (b - bb)) + pe);
}

// exp(-2 pi i (n + f) k / W), the phase of a shift by n + f at frequency
// k = -W/2..W/2: one evaluation at hi, and lo by the first-order terms.
template <int W>
GFC_HD void shift_phase(float f, int n, int k, float* s_out, float* c_out) {
  float hi, lo, s, c;
  shift_arg<W>(f, n, k, &hi, &lo);
  sincospi_poly(hi, &s, &c);
  *s_out = fmaf(lo, c, s);
  *c_out = fmaf(-lo, s, c);
}

// The value held by the even lane of this lane's pair (DPP quad permute
// 0, 0, 2, 2).
__device__ __forceinline__ float pair_even(float v) {
  return __builtin_bit_cast(float,
                            __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xA0, 0xF, 0xF, false));
}

// The value held by the second lane of this lane's stamp, for stamps of W
// consecutive lanes (W >= 64: lane 1 of the wavefront).
template <int W>
__device__ __forceinline__ float stamp_lane1(float v) {
  if constexpr (W >= 64) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 1));
  } else {
    return __shfl(v, ((int)__lane_id() & ~(W - 1)) + 1, 64);
  }
}

// The value held by the next lower (upper) lane of the wavefront, zero in the
// first (last) lane: DPP wave shifts by one.
__device__ __forceinline__ float lane_below(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x138, 0xF, 0xF, true));
}
__device__ __forceinline__ float lane_above(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x130, 0xF, 0xF, true));
}

// v plus the value that the DPP control CTRL brings to this lane.
template <int CTRL>
__device__ __forceinline__ float dpp_add(float v) {
  return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}

// Sum over each aligned group of N lanes (N = 4, 16, 32 or 64); every lane of
// the group receives the total.  Fixed order, the same in every lane, and no
// LDS: adds with DPP operands within a row of 16 lanes (pairs, quads, halves,
// the row), then the swaps of rows and of wavefront halves.
template <int N>
__device__ __forceinline__ float lane_sum(float v) {
  static_assert(N == 4 || N == 16 || N == 32 || N == 64, "4, 16, 32 or 64 lanes");
  v = dpp_add<0xB1>(v);  // quad_perm 1, 0, 3, 2
  v = dpp_add<0x4E>(v);  // quad_perm 2, 3, 0, 1
  if constexpr (N >= 16) {
    v = dpp_add<0x141>(v);  // row_half_mirror
    v = dpp_add<0x140>(v);  // row_mirror
  }
  if constexpr (N >= 32) {
    unsigned a = __builtin_bit_cast(unsigned, v), b = a;
    asm volatile("" : "+v"(b));  // a register of its own: the swap writes both
    const auto s = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    const unsigned s0 = s[0], s1 = s[1];
    v = __builtin_bit_cast(float, s0) + __builtin_bit_cast(float, s1);
  }
  if constexpr (N >= 64) {
    unsigned a = __builtin_bit_cast(unsigned, v), b = a;
    asm volatile("" : "+v"(b));
    const auto s = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    const unsigned s0 = s[0], s1 = s[1];
    v = __builtin_bit_cast(float, s0) + __builtin_bit_cast(float, s1);
  }
  return v;
}

// Value of v in lane k of the wavefront (k uniform).
__device__ __forceinline__ float lane_f(float v, int k) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), k));
}

// A uniform value in a vector register.  An instruction with a scalar operand
// issues every 4.2 cycles per SIMD; with vector operands two wavefronts issue
// together, every 2.3 cycles.
__device__ __forceinline__ float vector_f(float v) {
  float r;
  asm("v_mov_b32 %0, %1" : "=v"(r) : "s"(v));
  return r;
}

// Keeps a value's computation where it stands: the compiler otherwise sinks it
// to a later use, with its operands (more registers) held until then.
__device__ __forceinline__ void formed_here(float2& v) { asm volatile("" : "+v"(v.x), "+v"(v.y)); }

// 2^x on -1 <= x <= 0 as a polynomial with value 1 at 0: a minimax fit of
// degree 6 in the relative error, 2.08e-9.  The coefficients were rounded one
// after the other and those that follow fitted again each time (2.04e-9
// before rounding; all rounded at once 4.2e-8, of one sign).
constexpr int kFlatDeg = 6;
constexpr float kFlat[kFlatDeg + 1] = {1.f,           0x1.62e42cp-1f,  0x1.ebfac0p-3f, 0x1.c69488p-5f,
                                       0x1.39e3fep-7f, 0x1.4e2bbcp-10f, 0x1.c94ddap-14f};

// The flat components of a stamp: those whose exponent v q stays within one
// power of two over the whole frequency grid (|v q| <= v qmax <= 1, qmax the
// largest |q|, at a corner of the grid: q is a convex quadratic form).  Their
// sum is one polynomial in x = q / qmax,
//   sum_k w_k A_k 2^(v_k q) = sum_j a_j x^j,  a_j = kFlat[j] sum_k w_k A_k (v_k qmax)^j,
// seven multiply-adds per bin instead of a multiply, an exponential and a
// multiply-add for each of them (an exponential issues every 8.2 cycles, a
// multiply-add beside it every 4: 16.6 cycles per component and bin, against
// about 17 for the polynomial).  Of eight components log-spaced over 1e-4..10
// r_e^2, four are flat at r_e = 2 px, two at 8 px.
struct FlatSum {
  float a[kFlatDeg + 1];
  float s;  // 1 / qmax
  __device__ __forceinline__ float at(float q) const {
    const float x = q * s;
    float r = fmaf(a[kFlatDeg], x, a[kFlatDeg - 1]);
    static_for<2, kFlatDeg + 1>([&](auto jj) { r = fmaf(r, x, a[kFlatDeg - decltype(jj)::value]); });
    return r;
  }
};

// Whether stamps that share a wavefront (W < 64) look for flat components: if
// every table has two with v W^2 <= 1.1, flat up to r_e = W / 4, where a round
// galaxy has qmax = 0.89 W^2.  A component leaves the wavefront's loop only if
// it is flat in all of its stamps, while one stamp's sum costs every lane the
// polynomial.  It is a rule on the launch's tables, so that a stamp's values
// do not depend on its neighbours.  Times without and with the polynomial,
// r_e 0.5..8 px, 60,000 stamps of 16 x 16 and 30,000 of 32 x 32: eight
// components from 1e-4 r_e^2 30.4 -> 30.6 and 47.0 -> 46.1 us, sixteen 43.4 ->
// 41.0 and 69.5 -> 60.8 us, eight below 1e-5 24.3 -> 19.0 and 41.0 -> 33.3 us;
// where the rule says no, six from 1e-3 26.2 -> 28.4 and 41.9 -> 43.9 us, six
// from 0.02 28.0 -> 30.3 and 43.7 -> 45.8 us, and tables of both kinds mixed
// 28.2 -> 29.5 and 45.0 -> 44.9 us.
template <int W>
__device__ __forceinline__ bool flat_shared(const RenderArgs& p) {
  return p.flat_v2 * (float)(W * W) <= 1.1f;
}

// Lane k of each group of N lanes (for N = 64: of each row of 16) holds
// component k's variance vk and Fourier amplitude wak (w A; zero past the
// table's K).  With two or more flat components in a stamp (one costs the same
// either way), their amplitudes move from wak into the sums f (every lane of
// the group; zeros if the stamp has no such sum); returns whether the lane's
// stamp has one.  N = 64: f in vector registers.
template <int N>
__device__ __forceinline__ bool take_flat(const Galaxy& G, float vk, float& wak, FlatSum& f) {
  const float qmax = fmaxf(-kQ * fmaf(0.25f, G.b11 + G.b22, 0.5f * fabsf(G.b12)), 1e-30f);
  const float t = vk * qmax;
  bool flat = t <= 1.f && wak != 0.f && finitef(wak);
  constexpr int NK = N == 64 ? kKmax : N;
  const unsigned b = (unsigned)(__ballot(flat) >> ((int)__lane_id() & ~(N - 1) & 63)) & (unsigned)((1ull << NK) - 1ull);
  const bool any = __popc(b) >= 2;
  flat = flat && any;
  f.s = __builtin_amdgcn_rcpf(qmax);
  float p = flat ? wak : 0.f;
  const float tf = flat ? t : 0.f;  // t itself may overflow (v r_e^2 beyond 2e36 px^2)
  if constexpr (N == 64) {
    // Row r forms the sums j = r and 4 + r: two sums over 16 lanes in place of
    // seven.  (The sums are paid with no flat component too: at 256 x 256, one
    // to six components, seven cost 1.5-3% of the render.)
    const int r = (int)__lane_id() >> 4;
    const float t2 = tf * tf;
    p = (r & 1) ? p * tf : p;
    p = (r & 2) ? p * t2 : p;
    const float s0 = lane_sum<16>(p), s1 = lane_sum<16>(p * (t2 * t2));
    static_for<0, kFlatDeg + 1>([&](auto jj) {
      constexpr int j = decltype(jj)::value;
      f.a[j] = kFlat[j] * vector_f(lane_f(j < 4 ? s0 : s1, 16 * (j & 3)));
    });
  } else {
    static_for<0, kFlatDeg + 1>([&](auto jj) {
      f.a[decltype(jj)::value] = kFlat[decltype(jj)::value] * lane_sum<N>(p);
      p *= tf;
    });
  }
  if (flat) wak = 0.f;
  return any;
}

// Raw Lanczos-3 value at t (exact zeros at the integers other than 0), for
// the optional pixel-space sub-pixel shift (Section 2, step 8).
__device__ __forceinline__ float lanczos3(float t) {
  if (t == 0.f) return 1.f;
  if (fabsf(t) >= 3.f || t == rintf(t)) return 0.f;
  const float s = sinpif(t) * sinpif(t * (1.f / 3.f));
  return s * (3.f * 0.10132118364233778f) / (t * t);  // sinc(t) sinc(t/3) = 3 sin(pi t) sin(pi t/3) / (pi t)^2
}

// Step 4: Fourier weight of a component whose covariance trace is `tr`.
template <int W>
__device__ __forceinline__ float route_weight(float tr, unsigned flags) {
  if (flags & kForceFourier) return 1.f;
  if (flags & kForceReal) return 0.f;
  const float n = (0.5f * (float)W) * __builtin_amdgcn_rsqf(tr);
  const float t = fminf(fmaxf(n - 3.f, 0.f), 1.f);
  if (flags & kRampLinear) return t;
  return t * t * (3.f - 2.f * t);
}

// d w / d n of route_weight (zero outside the ramp).
template <int W>
__device__ __forceinline__ float route_slope(float n, unsigned flags) {
  if (flags & (kForceFourier | kForceReal)) return 0.f;
  if (!(n > 3.f && n < 4.f)) return 0.f;
  const float t = n - 3.f;
  if (flags & kRampLinear) return 1.f;
  return 6.f * t * (1.f - t);
}

}  // namespace gfc
