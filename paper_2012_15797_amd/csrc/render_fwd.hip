// Forward render kernel for stamp sizes W = 16, 32, 64, 128 (Lang 2020,
// Section 2, steps 3-8), one fused kernel per launch.
//
// A stamp is handled by W lanes (W < 64: 64/W stamps per wavefront; W = 128:
// two wavefronts).  The half spectrum (W/2 + 1 columns) never leaves the chip:
//
//  column phase  lane (c, h), c = 0..W/2-1, h = 0..1, owns column k_x = c and
//                rows k_y = 2m + h.  It evaluates the mixture transform
//                (steps 5-6) on those bins, multiplies by the fractional-shift
//                phase, the flux and the cached PSF spectrum (step 7a), and
//                runs a W/2-point inverse FFT in registers (the even/odd half
//                of the length-W column transform).  Column k_x = W/2 is
//                packed into column 0 as its imaginary part: both columns
//                transform to real vectors because the product is Hermitian.
//  transpose     through LDS; the last radix-2 stage of the column transform
//                is applied while reading back.
//  row phase     lane y owns row y and runs the length-W complex-to-real
//                inverse transform as a W/2-point complex FFT in registers.
//  store         real-space components (step 8) are added to the row in its
//                lane's registers, and half a stamp at a time goes through LDS
//                to memory, four pixels per lane.
// The phases are those of the whole shift, integer parts included, so the
// stamp leaves the transforms in output order.
#include "gfc_device.hpp"
#include "gfc_launch.hpp"

namespace gfc {

template <int W, bool EIG = false>
struct SmallCfg {
  static constexpr int M = W / 2;                // values per lane in the column phase
  // With a varying PSF at 64 x 64, four stamps (one per wavefront) share a
  // workgroup and stream each component spectrum through LDS once for all four.
  static constexpr bool SHARE = EIG && W == 64;
  static constexpr int BLOCK = SHARE ? 256 : (W < 64 ? 64 : W);  // threads per workgroup
  static constexpr int SPB = BLOCK / W;          // stamps per workgroup
  static constexpr bool WAVE1 = W >= 64;         // one stamp per wavefront (or two wavefronts per stamp)
  // Both LDS transposes run in two passes over halves of the data, so a
  // stamp needs half the LDS and more wavefronts fit on a CU.
  static constexpr int T1S = W / 2 + 1;          // float2 per row: W/4 columns x 2 halves + pad
  static constexpr int T1N = M * T1S;            // float2 per stamp; also (W/2) x (W+1) floats
  static constexpr int HR = W / 2;               // rows of the store tile per pass
  // Floats per row of the store tile: 16-byte aligned, and 4 (mod 32) or the
  // like, so that the eight rows of a 16-byte access fall in distinct banks.
  static constexpr int LSO = W + 4;
};

// EIG: the PSF varies over the image (eigen-PSF components with polynomial
// weights); its spectrum and Gaussian are formed per stamp from the
// components' cached spectra and moments.
// W = 128 is held to two wavefronts per SIMD (a small spill costs less than
// running one wavefront per SIMD); the other sizes reach their occupancy freely.
// LZ: the Lanczos-3 sub-pixel shift is applied while storing.
// PT: each galaxy names its (constant) PSF in p.psf_id, and the stamp takes
// that PSF's spectrum and Gaussian from the tables (a serving batch mixes
// PSFs); the one-PSF instantiations compile exactly as without it.
// PROF: each galaxy has a mixture of its own (p.prof).
template <int W, bool EIG, bool LZ, bool PT, bool PROF>
__global__ void __launch_bounds__((SmallCfg<W, EIG>::BLOCK)) __attribute__((amdgpu_waves_per_eu(W == 128 ? 2 : 1)))
render_small_kernel(RenderArgs p) {
  using C = SmallCfg<W, EIG>;
  constexpr int M = C::M;
  constexpr int T1S = C::T1S;
  // The shift's two forms (see the store): up to 64 x 64 on the rows in
  // output order, at 128 x 128 on the finished half stamp in the LDS tile.
  constexpr bool LZF = LZ && W <= 64, LZT = LZ && W == 128;
  constexpr int LS = W + 8;  // floats per row of the LZT tile: four zero pixels on each side
  constexpr int T1N = LZT ? (C::HR + 2) * LS / 2 : C::HR * C::LSO / 2;
  static_assert(T1N >= C::T1N && T1N % 2 == 0, "the transposes fit");
  __shared__ __attribute__((aligned(16))) float2 s_t1[C::SPB][T1N];  // 16-byte aligned: also read as float4
  __shared__ float2 s_py[C::SPB][W + 2];
  __shared__ float2 s_nyq[C::SPB][W];
  // per real-space component, its row constants (amplitude, g, sxy / syy,
  // -log2(e) / (2 syy)) of the store below
  __shared__ float4 s_rc[C::SPB][kKmax];
  __shared__ float s_lw[LZ ? C::SPB : 1][LZT ? 24 : (LZ ? 12 : 1)];  // raw Lanczos weights of the stamp, per wavefront

  const int l = (C::SPB == 1) ? (int)threadIdx.x : (int)threadIdx.x % W;
  int slot = (C::SPB == 1) ? 0 : (int)threadIdx.x / W;
  if constexpr (C::WAVE1 && C::SPB > 1) slot = __builtin_amdgcn_readfirstlane(slot);  // keeps the stamp index scalar
  const int64_t stamp = (int64_t)blockIdx.x * C::SPB + slot;
  const bool live = stamp < p.n;
  Galaxy G = load_galaxy<W, PROF>(p, live ? stamp : p.n - 1);
  Profile prof = {0.f, 0.f, 0, true};
  if constexpr (PROF) {
    const int64_t gs = live ? stamp : p.n - 1;
    prof = make_profile<(W < 64 ? W : 64)>(p, p.prof_a[gs], p.prof_b ? p.prof_b[gs] : 0.f);
    if (!prof.ok) {  // invalid galaxy: NaN stamp, counted
      G.ok = false;
      G.flux = __builtin_nanf("");
    }
  }
  if constexpr (C::WAVE1) {  // one stamp per wavefront: keep its integer shift in SGPRs
    make_uniform(G);
  }
  // This stamp's PSF spectrum (lane-permuted main columns, Nyquist column)
  // and the index of its Gaussian in the table (PT).
  const float2* psfm = p.psf_main;
  const float2* psfn = p.psf_nyq;
  int ps = 0;
  if constexpr (PT) {
    static_assert(!EIG, "a per-galaxy PSF index takes constant PSFs");
    ps = p.psf_id[live ? stamp : p.n - 1];
    if constexpr (C::WAVE1) ps = __builtin_amdgcn_readfirstlane(ps);
    if (ps < 0 || ps >= p.n_psf) {  // invalid galaxy: NaN stamp, counted
      ps = 0;
      G.ok = false;
      G.flux = __builtin_nanf("");
    }
    psfm = p.psf_main_tab[ps];
    psfn = p.psf_nyq_tab[ps];
  }
  // Lanczos-3 weights of the fused shift (taps d = -3..2 along x, then y),
  // formed up front: with one stamp per wavefront they sit in scalar
  // registers until the store.
  float wxn[6], wy[6];
  if constexpr (LZ) {
    const int64_t gs = live ? stamp : p.n - 1;
    const int ll = W > 64 ? l & 63 : l;
    float* lw = s_lw[slot] + (W > 64 ? 12 * (l >> 6) : 0);  // each wavefront its own: no barrier needed
    if (ll < 12) {  // raw weights of taps d = -3..2: x in 0..5, y in 6..11
      const float v = ll < 6 ? p.x[gs] : p.y[gs];
      lw[ll] = lanczos3((float)((ll % 6) - 3) + (v - floorf(v)));
    }
    float wx[6], sx = 0.f, sy = 0.f;
    static_for<0, 6>([&](auto dd) {
      constexpr int d = decltype(dd)::value;
      wx[d] = lw[d];
      wy[d] = lw[6 + d];
      sx += wx[d];
      sy += wy[d];
    });
    const float rx = 1.f / sx, ry = 1.f / sy;
    static_for<0, 6>([&](auto dd) {
      constexpr int d = decltype(dd)::value;
      wxn[d] = wx[d] * rx;
      wy[d] *= ry;
      if constexpr (C::WAVE1) {  // one stamp per wavefront: the weights are uniform
        wxn[d] = uniform_f(wxn[d]);
        wy[d] = uniform_f(wy[d]);
      }
    });
  }
  const float trB = G.b11 + G.b22;

  // ---------------------------------------------------------------- column phase
  const int c = l >> 1, h = l & 1;
  const float nu = (float)c * (1.f / W);
  const float hW = (float)h * (1.f / W);
  // exponent per unit mixture variance: kQ (b11 nu^2 + 2 b12 nu om + b22 om^2)
  const float g0 = kQ * G.b11 * nu * nu;
  const float g1 = 2.f * kQ * G.b12 * nu;
  const float g2 = kQ * G.b22;
  // Row k_y = 2m + h has omega = c_m + h/W with a compile-time c_m, so the
  // quadratic is expanded about h/W: q = e0 + c_m (e1 + c_m g2), two FMAs
  // with an immediate c_m per bin (e0 = q(h/W), e1 = q'(h/W); for h = 0 they
  // are g0 and g1 and the result is the plain quadratic in omega).
  const float e0 = fmaf(hW, fmaf(g2, hW, g1), g0);
  const float e1 = fmaf(2.f * g2, hW, g1);
  float qv[M + 1];
  static_for<0, M>([&](auto mm) {
    constexpr int m = decltype(mm)::value;
    if constexpr (2 * m == W / 2) {
      const float om = h ? (float)(W / 2 + 1 - W) * (1.f / W) : 0.5f;
      qv[m] = fmaf(om, fmaf(g2, om, g1), g0);
    } else if constexpr (m == 0) {
      qv[m] = e0;
    } else {
      constexpr float cm = (2 * m < W / 2) ? (float)(2 * m) * (1.f / W) : (float)(2 * m - W) * (1.f / W);
      qv[m] = fmaf(cm, fmaf(cm, g2, e1), e0);
    }
  });
  // Nyquist column k_x = W/2: lane l takes row k_y = l at nu = +1/2 and -1/2.
  // The corner's omega = -1/2 twins need no evaluation of their own: the
  // mixture transform is even, so (+-1/2, -1/2) equals (-+1/2, +1/2), the
  // pair that lane W/2 (omega = +1/2) holds.  Up to 64 x 64 the -1/2 values
  // need no evaluation either: (-1/2, omega_l) equals (+1/2, -omega_l), lane
  // W - l's, except at the corner, whose (-1/2, +1/2) the h = 1 lanes
  // evaluate in slot M (where the h = 0 lanes hold the Nyquist row's
  // omega = -1/2 twin and the h = 1 lanes would repeat it).
  constexpr bool kMirrorN = W <= 64;
  constexpr int NQ = kMirrorN ? 1 : 2;
  const float omN = (l < W / 2) ? (float)l * (1.f / W) : (l == W / 2 ? 0.5f : (float)(l - W) * (1.f / W));
  const float qa = kQ * G.b11 * 0.25f, qb = kQ * G.b12, qd = kQ * G.b22;
  float qn[2];
  qn[0] = fmaf(omN, fmaf(qd, omN, qb), qa);      // (+1/2, omN)
  qn[1] = fmaf(omN, fmaf(qd, omN, -qb), qa);     // (-1/2, omN)
  qv[M] = fmaf(-0.5f, fmaf(g2, -0.5f, g1), g0);  // Nyquist row, omega = -1/2
  if constexpr (kMirrorN) {
    if (h) qv[M] = fmaf(0.5f, fmaf(qd, 0.5f, -qb), qa);  // the corner (-1/2, +1/2)
  }

  // PSF spectrum of this lane's bins and the PSF Gaussian (step 2; for a
  // varying PSF, the weighted sum of the components at the galaxy's image
  // position, whose transforms and moments are linear in the weights).
  // From 64 up it is read (a varying one summed) in the PSF product itself, 8
  // or 16 bins at a time, rather than all at once while the mixture sums are
  // live: a constant PSF at 64 takes 116 VGPRs instead of 144, a varying one
  // 128 instead of 160 (four wavefronts per SIMD instead of three).  Below, a
  // varying PSF is summed before the mixture loop, while its sums are not yet
  // live (more registers for the reads in flight).
  constexpr bool kPsfStream = W >= 64;
  constexpr bool kPsfFirst = EIG && !kPsfStream;
  float2 Pm[kPsfStream ? 1 : M];
  float2 psfN;
  float pg[6];
  float ck = 0.f;  // varying PSF, one stamp per wavefront: lane k holds component k's weight
  auto psf_terms = [&]() {
    if constexpr (EIG) {
      const int64_t g = live ? stamp : p.n - 1;
      float u = (p.psf_px[g] - p.eig_norm[0]) * p.eig_norm[1];
      float v = (p.psf_py[g] - p.eig_norm[2]) * p.eig_norm[3];
      if constexpr (C::WAVE1) {
        u = uniform_f(u);
        v = uniform_f(v);
      }
      const float up[4] = {1.f, u, u * u, u * u * u}, vp[4] = {1.f, v, v * v, v * v * v};
      float mom[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      psfN = make_float2(0.f, 0.f);
      if constexpr (kPsfStream) {
        // lane k evaluates component k's polynomial (J <= 16 lanes)
        static_assert(C::WAVE1, "one stamp per wavefront");
        const int lk = (int)__lane_id();
        if (lk < p.eig_J) ck = eigen_weight(p, lk, up, vp);
        for (int j = 0; j < p.eig_J; ++j) {
          const float cj = lane_f(ck, j);
          const float2 qn = p.psf_nyq[j * p.eig_stride + l];
          psfN = make_float2(fmaf(cj, qn.x, psfN.x), fmaf(cj, qn.y, psfN.y));
          static_for<0, 6>([&](auto ii) {
            constexpr int i = decltype(ii)::value;
            mom[i] = fmaf(cj, p.eig_mom[j * 6 + i], mom[i]);
          });
        }
      } else {
        static_for<0, M>([&](auto mm) { Pm[decltype(mm)::value] = make_float2(0.f, 0.f); });
        for (int j = 0; j < p.eig_J; ++j) {
          const float cj = eigen_weight(p, j, up, vp);
          const float2* pj = p.psf_main + j * p.eig_stride;
          static_for<0, M>([&](auto mm) {
            constexpr int m = decltype(mm)::value;
            const float2 q = pj[m * W + l];
            Pm[m] = make_float2(fmaf(cj, q.x, Pm[m].x), fmaf(cj, q.y, Pm[m].y));
          });
          const float2 qn = p.psf_nyq[j * p.eig_stride + l];
          psfN = make_float2(fmaf(cj, qn.x, psfN.x), fmaf(cj, qn.y, psfN.y));
          static_for<0, 6>([&](auto ii) {
            constexpr int i = decltype(ii)::value;
            mom[i] = fmaf(cj, p.eig_mom[j * 6 + i], mom[i]);
          });
        }
      }
      eigen_gauss(mom, pg);
    } else {
      if constexpr (!kPsfStream) {
        static_for<0, M>([&](auto mm) {
          constexpr int m = decltype(mm)::value;
          Pm[m] = psfm[m * W + l];
        });
      }
      psfN = psfn[l];
      if constexpr (PT) {
        static_for<0, 6>([&](auto ii) { pg[decltype(ii)::value] = p.pg_tab[6 * ps + decltype(ii)::value]; });
      } else {
        static_for<0, 6>([&](auto ii) { pg[decltype(ii)::value] = p.pg[decltype(ii)::value]; });
      }
    }
  };
  if constexpr (kPsfFirst) psf_terms();

  // The flat components' polynomial initialises the sums, or the first
  // component with a Fourier share (with none, component 0 contributes zeros);
  // the rest accumulate.
  float S[M + 1];
  float SN[2];
  unsigned rmask = 0;  // components with a real-space share: lane k holds v and (1 - w) A
  float vk = 0.f, rak = 0.f;
  auto first_terms = [&](float v, float wa) {
    static_for<0, M + 1>([&](auto mm) {
      constexpr int m = decltype(mm)::value;
      S[m] = wa * __builtin_amdgcn_exp2f(v * qv[m]);
    });
    static_for<0, NQ>([&](auto jj) {
      constexpr int j = decltype(jj)::value;
      SN[j] = wa * __builtin_amdgcn_exp2f(v * qn[j]);
    });
  };
  auto flat_terms = [&](const FlatSum& f) {
    static_for<0, M + 1>([&](auto mm) { S[decltype(mm)::value] = f.at(qv[decltype(mm)::value]); });
    static_for<0, NQ>([&](auto jj) { SN[decltype(jj)::value] = f.at(qn[decltype(jj)::value]); });
  };
  auto add_terms = [&](float v, float wa) {
    static_for<0, M + 1>([&](auto mm) {
      constexpr int m = decltype(mm)::value;
      S[m] = fmaf(wa, __builtin_amdgcn_exp2f(v * qv[m]), S[m]);
    });
    static_for<0, NQ>([&](auto jj) {
      constexpr int j = decltype(jj)::value;
      SN[j] = fmaf(wa, __builtin_amdgcn_exp2f(v * qn[j]), SN[j]);
    });
  };
  if constexpr (C::WAVE1) {
    // One stamp per wavefront: lane k of each row of 16 works out the route
    // weight of component k once, and the loop takes v and w A from lane k.
    const int lk = (int)__lane_id() & (kKmax - 1);
    float wak = 0.f;
    bool rk = false;
    if (lk < G.K) {
      const float2 av = component_mix<PROF>(p, G, prof, lk);
      const float Ak = av.x;
      vk = av.y;
      const float wk = route_weight<W>(vk * trB, p.flags);
      wak = wk * Ak;
      rk = wk < 1.f && Ak != 0.f;
      rak = (1.f - wk) * Ak;
    }
    rmask = (unsigned)__ballot(rk) & ((1u << kKmax) - 1u);
    FlatSum f;
    const bool flat = take_flat<64>(G, vk, wak, f);  // uniform
    unsigned mk = (unsigned)__ballot(wak != 0.f) & ((1u << kKmax) - 1u);
    if (flat) {
      flat_terms(f);
    } else {
      const int k = mk ? __builtin_ctz(mk) : 0;
      first_terms(vector_f(lane_f(vk, k)), vector_f(lane_f(wak, k)));
      mk &= mk - 1;
    }
    for (; mk != 0; mk &= mk - 1) {
      const int k = __builtin_ctz(mk);
      add_terms(vector_f(lane_f(vk, k)), vector_f(lane_f(wak, k)));
    }
  } else {
    // Several stamps per wavefront: lane k of each stamp works out its
    // stamp's component k (K <= W lanes), and the loop takes v and w A from
    // it with a lane permute within the stamp's W lanes.
    float wak = 0.f;
    bool rk = false;
    if (l < G.K) {
      const float2 av = component_mix<PROF>(p, G, prof, l);
      const float Ak = av.x;
      vk = av.y;
      const float wk = route_weight<W>(vk * trB, p.flags);
      wak = wk * Ak;
      rk = wk < 1.f && Ak != 0.f;
      rak = (1.f - wk) * Ak;
    }
    const unsigned long long rb = __ballot(rk);
    rmask = (unsigned)(rb >> ((int)__lane_id() & ~(W - 1))) & (unsigned)((1ull << W) - 1ull);
    FlatSum f;
    const bool flat = flat_shared<W>(p);  // uniform
    if (flat) take_flat<W>(G, vk, wak, f);
    // over the components that any of the wavefront's stamps still needs
    unsigned long long need = __ballot(wak != 0.f);
    need |= need >> 32;
    if constexpr (W == 16) need |= need >> 16;
    unsigned mk = (unsigned)need & ((1u << kKmax) - 1u);
    if (flat) {
      flat_terms(f);
    } else {
      const int k = mk ? __builtin_ctz(mk) : 0;
      first_terms(__shfl(vk, k, W), __shfl(wak, k, W));
      mk &= mk - 1;
    }
    for (; mk != 0; mk &= mk - 1) {
      const int k = __builtin_ctz(mk);
      const float wa = __shfl(wak, k, W);
      if (wa == 0.f) continue;
      add_terms(__shfl(vk, k, W), wa);
    }
  }

  if constexpr (!kPsfFirst) psf_terms();
  if constexpr (kMirrorN) {
    const float mirrored = __shfl(SN[0], (W - l) & (W - 1), W);
    const float cornerv = __shfl(S[M], 1, W);  // lane 1 of the stamp: h = 1
    SN[1] = (l == W / 2) ? cornerv : mirrored;
  }
  // Lane k forms real-space component k's constants once per stamp; they do
  // not depend on the row.
  if (l < kKmax && ((rmask >> l) & 1u)) {
    const float sxx = fmaf(vk, G.b11, pg[2]);
    const float sxy = fmaf(vk, G.b12, pg[3]);
    const float syy = fmaf(vk, G.b22, pg[4]);
    const float det = fmaf(sxx, syy, -(sxy * sxy));
    const float rsyy = __builtin_amdgcn_rcpf(syy);
    s_rc[slot][l] = make_float4(rak * G.flux * pg[5] * kInv2Pi * __builtin_amdgcn_rsqf(det),
                                __builtin_amdgcn_sqrtf(-kHalfLog2e * syy * __builtin_amdgcn_rcpf(det)), sxy * rsyy,
                                kHalfLog2e * rsyy);
  }

  // Fractional-shift phases (shift theorem): exp(-2 pi i (fx nu + fy om)).
  // Every lane evaluates the y phase of row l and one x phase: lanes h = 0
  // that of column c, lanes h = 1 that of nu = +1/2 (the Nyquist column).
  // The h = 1 lane of a pair takes its column's phase from its neighbour;
  // omega = -1/2 is the conjugate of row W/2 (omega = +1/2).
  // The integer parts of the centre go into the phases as well.
  float sy, cy, sxa, cxa;
  shift_phase<W>(G.fy, G.ny, l <= W / 2 ? l : l - W, &sy, &cy);
  shift_phase<W>(G.fx, G.nx, h ? W / 2 : c, &sxa, &cxa);
  const float sx = pair_even(sxa), cx = pair_even(cxa);
  const float sxh = stamp_lane1<W>(sxa), cxh = stamp_lane1<W>(cxa);  // nu = +1/2
  const float fs = G.flux * (1.f / ((float)W * (float)W));
  const float2 pxF = make_float2(fs * cx, fs * sx);
  s_py[slot][l] = make_float2(cy, sy);
  if (l == W / 2) s_py[slot][W] = make_float2(cy, -sy);
  {
    const float2 eM = make_float2(cxh, sxh), eP = make_float2(cxh, -sxh);
    const bool corner = (l == W / 2);
    const float2 pyA = corner ? make_float2(0.5f * cy, 0.5f * sy) : make_float2(cy, sy);
    const float2 pyB = corner ? make_float2(0.5f * cy, -0.5f * sy) : make_float2(0.f, 0.f);
    const float2 plus = cadd(cscale(pyA, SN[0]), cscale(pyB, SN[1]));
    const float2 minus = cadd(cscale(pyA, SN[1]), cscale(pyB, SN[0]));
    const float2 inner = cadd(cmul(eM, plus), cmul(eP, minus));
    s_nyq[slot][l] = cmul(cscale(psfN, 0.5f * fs), inner);
  }
  __syncthreads();

  float2 Z[M];
  auto product = [&](auto mm, float2 P) {  // Z[m] from the PSF's bin m
    constexpr int m = decltype(mm)::value;
    if constexpr (2 * m == W / 2) {
      const float2 q0 = s_py[slot][W / 2 + h];
      const float2 pyA = h ? q0 : cscale(q0, 0.5f);
      const float2 pyB = h ? make_float2(0.f, 0.f) : cscale(s_py[slot][W], 0.5f);
      Z[m] = cmul(cmul(P, pxF), cadd(cscale(pyA, S[m]), cscale(pyB, S[M])));
    } else {
      Z[m] = cscale(cmul(cmul(P, s_py[slot][2 * m + h]), pxF), S[m]);
    }
  };
  if constexpr (EIG && C::SHARE) {
    // Half of the bins at a time, two components at a time: their bins of the
    // half (contiguous in the cache) are copied with 16-byte loads into one
    // half of the workgroup's transpose buffers, which are free until the
    // column FFT, while the four wavefronts sum the two before from the other
    // half.  Reading a half again two steps later is ordered by the barrier in
    // between.  (A component past the last is the last, with weight zero.)
    // 30,000 stamps, 6 components: 196 us, against 213 us with the whole
    // spectrum summed before the mixture loop, at three wavefronts per SIMD.
    constexpr int HB = M / 2;                // bins of a half
    constexpr int NB = HB * W;               // float2 of one component's half
    static_assert(NB / 2 == 2 * C::BLOCK && 4 * NB <= C::SPB * T1N, "two float4 per thread and component; the buffers fit");
    float2* buf = &s_t1[0][0];
    const float4* src = reinterpret_cast<const float4*>(p.psf_main) + threadIdx.x;
    const int64_t sv = p.eig_stride / 2;     // float4 from one component to the next
    const int np = (p.eig_J + 1) >> 1, last = p.eig_J - 1;
    float4 st0, st1, st2, st3;
    auto fetch = [&](int half, int jp) {     // components 2 jp, 2 jp + 1
      const float4* a = src + half * (NB / 2);
      const float4* b = a + min(2 * jp + 1, last) * sv;
      a += 2 * jp * sv;
      st0 = a[0], st1 = a[C::BLOCK], st2 = b[0], st3 = b[C::BLOCK];
    };
    fetch(0, 0);
    int it = 0;
    static_for<0, 2>([&](auto hh) {
      constexpr int half = decltype(hh)::value;
      float2 P[HB];  // (started at zero: the first pair apart takes 136 registers)
      static_for<0, HB>([&](auto ii) { P[decltype(ii)::value] = make_float2(0.f, 0.f); });
      for (int jp = 0; jp < np; ++jp, ++it) {
        float2* b = buf + (it & 1) * (2 * NB);
        float4* dst = reinterpret_cast<float4*>(b) + threadIdx.x;
        dst[0] = st0, dst[C::BLOCK] = st1, dst[NB / 2] = st2, dst[NB / 2 + C::BLOCK] = st3;
        __syncthreads();
        if (jp + 1 < np) fetch(half, jp + 1);  // in flight while these are summed
        else if constexpr (half == 0) fetch(1, 0);
        const float c0 = vector_f(lane_f(ck, 2 * jp)), c1 = vector_f(lane_f(ck, 2 * jp + 1));  // lanes past J hold zero
        static_for<0, HB>([&](auto ii) {
          constexpr int i = decltype(ii)::value;
          const float2 q0 = b[i * W + l], q1 = b[NB + i * W + l];
          P[i] = make_float2(fmaf(c1, q1.x, fmaf(c0, q0.x, P[i].x)), fmaf(c1, q1.y, fmaf(c0, q0.y, P[i].y)));
        });
      }
      static_for<0, HB>([&](auto ii) {
        constexpr int m = half * HB + decltype(ii)::value;
        product(std::integral_constant<int, m>{}, P[decltype(ii)::value]);
        formed_here(Z[m]);
      });
    });
    __syncthreads();  // the buffers take the transpose
  } else if constexpr (EIG && kPsfStream) {
    // Eight bins at a time; each component's eight are in flight while the
    // one before is summed, two components per trip.  (A component past the
    // last is the last, with weight zero.)  5,000 stamps of 128 x 128, 6
    // components: 209 us, against 305 us with all bins of one component read
    // at a time after the mixture loop, which spilled.
    const float2* pj = p.psf_main + l;
    const int last = p.eig_J - 1;
    float2 qa[8], qb[8];
    auto fetch = [&](float2 (&q)[8], auto gg, int j) {
      static_for<0, 8>([&](auto ii) {
        constexpr int i = decltype(ii)::value;
        q[i] = pj[j * p.eig_stride + (8 * decltype(gg)::value + i) * W];
      });
    };
    fetch(qa, std::integral_constant<int, 0>{}, 0);
    static_for<0, M / 8>([&](auto gg) {
      constexpr int g = decltype(gg)::value;
      float2 P[8];
      static_for<0, 8>([&](auto ii) { P[decltype(ii)::value] = make_float2(0.f, 0.f); });
      auto sum = [&](const float2 (&q)[8], int j) {
        const float cj = vector_f(lane_f(ck, j));  // lanes past J hold zero
        static_for<0, 8>([&](auto ii) {
          constexpr int i = decltype(ii)::value;
          P[i] = make_float2(fmaf(cj, q[i].x, P[i].x), fmaf(cj, q[i].y, P[i].y));
        });
      };
      for (int j = 0; j <= last; j += 2) {
        fetch(qb, gg, min(j + 1, last));
        sum(qa, j);
        if (j + 2 <= last) fetch(qa, gg, j + 2);
        else if constexpr (g + 1 < M / 8) fetch(qa, std::integral_constant<int, g + 1>{}, 0);
        sum(qb, j + 1);
      }
      static_for<0, 8>([&](auto ii) {
        constexpr int m = 8 * g + decltype(ii)::value;
        product(std::integral_constant<int, m>{}, P[decltype(ii)::value]);
        formed_here(Z[m]);
      });
    });
  } else {
    static_for<0, M>([&](auto mm) {
      constexpr int m = decltype(mm)::value;
      if constexpr (kPsfStream) product(mm, psfm[m * W + l]);
      else product(mm, Pm[m]);
      if constexpr (kPsfStream && m % 16 == 15) __builtin_amdgcn_sched_barrier(0);  // bounds the loads in flight
    });
  }
  if (c == 0) {  // column 0 carries the Nyquist column as its imaginary part
    static_for<0, M>([&](auto mm) {
      constexpr int m = decltype(mm)::value;
      const float2 xn = s_nyq[slot][2 * m + h];
      Z[m] = make_float2(Z[m].x - xn.y, Z[m].y + xn.x);
    });
  }
  fft<M, +1>(Z);

  // ---------------------------------------------------------------- row phase
  constexpr int NC = W / 2;
  constexpr int QC = W / 4;  // columns per transpose pass
  const int y = l;
  const int jr = y & (M - 1);
  const float2 tw = twiddle_rt<+1, W>(y);
  float2 X[NC + 1];
  static_for<0, 2>([&](auto pp) {
    constexpr int pass = decltype(pp)::value;
    if (c / QC == pass) {
      static_for<0, M>([&](auto jj) {
        constexpr int j = decltype(jj)::value;
        s_t1[slot][j * T1S + (l - 2 * QC * pass)] = Z[j];
      });
    }
    __syncthreads();
    static_for<0, QC>([&](auto cc) {
      constexpr int cl = decltype(cc)::value;
      constexpr int cI = pass * QC + cl;
      const float2 e0 = s_t1[slot][jr * T1S + 2 * cl];
      const float2 e1 = s_t1[slot][jr * T1S + 2 * cl + 1];
      const float2 v = cfma(tw, e1, e0);
      if constexpr (cI == 0) {
        X[0] = make_float2(v.x, 0.f);
        X[NC] = make_float2(v.y, 0.f);
      } else {
        X[cI] = v;
      }
    });
    __syncthreads();
  });
  // complex-to-real: R[k] = (X[k] + conj X[W/2-k]) + i w^k (X[k] - conj X[W/2-k]),
  // w = exp(2 pi i / W).  Bins k and W/2-k share s = X[k] + conj X[W/2-k] and
  // t = w^k (X[k] - conj X[W/2-k]):  R[k] = s + i t,  R[W/2-k] = conj(s) + i conj(t).
  float2 R[NC];
  static_for<0, NC / 2 + 1>([&](auto kk) {
    constexpr int k = decltype(kk)::value;
    float2 lo, hi;
    c2r_pair<+1, W, k>(X[k], cconj(X[NC - k]), lo, hi);
    R[k] = lo;
    if constexpr (k != 0 && 2 * k != NC) R[NC - k] = hi;
  });
  fft<NC, +1>(R);

  // ---------------------------------------------------------------- real space + store
  float* st = reinterpret_cast<float*>(&s_t1[slot][0]);
  if (rmask != 0) {
    const float dy = (float)y - G.y0 - pg[1];
    const float dx0 = (float)(W / 2) - G.x0 - pg[0];  // dx of column W / 2
    for (unsigned mk = rmask; mk != 0; mk &= mk - 1) {
      const float4 rc = s_rc[slot][__builtin_ctz(mk)];
      // Along this lane's row (dy fixed) the quadratic form is
      // dy^2 / syy + (syy / det) (dx - (sxy / syy) dy)^2, completed about the
      // conditional mean, so that the exponent stays a difference of small
      // terms near the peak (an expansion about a fixed column cancels terms
      // of size (W/2)^2 / sxx there): with dx = x + dx0 the exponent is
      // k - u^2, u = g (x + m), two FMAs with an immediate x.  x counts from
      // column W/2, near most galaxies' centres: m is small there and g m
      // rounds by little.  (Counted from column 0, that rounding moved the
      // component along x by up to 2e-6 px at 64 x 64, in every row alike.)
      const float ampr = rc.x, g = rc.y;
      const float k0 = rc.w * dy * dy;
      const float gm = g * fmaf(-rc.z, dy, dx0);
      static_for<0, W / 2>([&](auto xx) {
        constexpr int x = 2 * decltype(xx)::value;  // two columns at a time
        const float u0 = fmaf(g, (float)(x - W / 2), gm);
        const float u1 = fmaf(g, (float)(x + 1 - W / 2), gm);
        R[x >> 1].x = fmaf(ampr, __builtin_amdgcn_exp2f(fmaf(-u0, u0, k0)), R[x >> 1].x);
        R[x >> 1].y = fmaf(ampr, __builtin_amdgcn_exp2f(fmaf(-u1, u1, k0)), R[x >> 1].y);
      });
    }
  }
  float* outp = p.out + (live ? stamp : 0) * (int64_t)(W * W);
  if constexpr (LZF) {
    {
      // Lanczos-3 shift by the fractional position, fused into the store: a
      // lane keeps its whole output column (W <= 64), so the stamp makes one
      // trip to memory.  The rows are filtered along x in the row-owning lane
      // and written to the LDS tile, and the columns are filtered along y in
      // registers as the tile's rows are read.  Taps outside the stamp have
      // weight zero.
      // x filter of this lane's row, with every lane active (in the staging
      // passes below only half the lanes write, and arithmetic there would
      // be issued once per pass)
      float hrow[W];
      static_for<0, W>([&](auto xx) {
        constexpr int x = decltype(xx)::value;
        float hsum = 0.f;
        static_for<0, 6>([&](auto dd) {
          constexpr int d = decltype(dd)::value;
          constexpr int xs = x + d - 3;
          if constexpr (xs >= 0 && xs < W) hsum = fmaf(wxn[d], (xs & 1) ? R[xs >> 1].y : R[xs >> 1].x, hsum);
        });
        hrow[x] = hsum;
      });
      float acc[W];
      static_for<0, W>([&](auto tt) { acc[decltype(tt)::value] = 0.f; });
      static_for<0, 2>([&](auto qq) {
        constexpr int q = decltype(qq)::value;
        if (y / C::HR == q) {
          int row = (y - q * C::HR) * (W + 1);
          asm volatile("" : "+v"(row));
          static_for<0, W>([&](auto xx) {
            constexpr int x = decltype(xx)::value;
            st[row + x] = hrow[x];
          });
        }
        __syncthreads();
        static_for<0, C::HR>([&](auto rr) {
          constexpr int sr = q * C::HR + decltype(rr)::value;  // source row
          const float v = st[(sr - q * C::HR) * (W + 1) + l];
          static_for<0, 6>([&](auto dd) {
            constexpr int d = decltype(dd)::value;
            constexpr int t = sr - d + 3;  // output row fed through tap d
            if constexpr (t >= 0 && t < W) acc[t] = fmaf(wy[d], v, acc[t]);
          });
          // Output row t is complete once its sources t - 3 .. t + 2 within
          // the stamp are in; the last two rows after the final source row.
          constexpr int done = sr - 2;
          if constexpr (done >= 0) {
            if (live) __builtin_nontemporal_store(acc[done], outp + done * W + l);
          }
          __builtin_amdgcn_sched_barrier(0);
        });
        __syncthreads();
      });
      if (live) {
        __builtin_nontemporal_store(acc[W - 2], outp + (W - 2) * W + l);
        __builtin_nontemporal_store(acc[W - 1], outp + (W - 1) * W + l);
      }
    }
  } else {
    float carry[5];  // LZT: rows HR - 5 .. HR - 1 of this lane's column, for the second half
    const int c4 = 4 * (l & (W / 4 - 1)), r4 = l / (W / 4);  // this lane's four columns and first row
    static_for<0, 2>([&](auto qq) {
      constexpr int q = decltype(qq)::value;
      if (y / C::HR == q) {
        int row = (y - q * C::HR) * C::LSO;
        asm volatile("" : "+v"(row));  // one base address; the offsets stay immediate
        static_for<0, W / 4>([&](auto nn) {
          constexpr int n = decltype(nn)::value;
          *reinterpret_cast<float4*>(st + row + 4 * n) = make_float4(R[2 * n].x, R[2 * n].y, R[2 * n + 1].x, R[2 * n + 1].y);
        });
      }
      __syncthreads();
      if constexpr (LZT) {
        // Lanczos-3 shift of the finished pixels, real-space terms included:
        // along y on the lane's column in registers (the first half's last
        // five rows carry over), then along x from the tile, four pixels per
        // lane with the neighbours in three 16-byte reads.  Taps outside the
        // stamp have weight zero: the rows beyond it are left out, the
        // columns beyond it are zeros beside the tile's rows.  5,001 stamps
        // take 147 us; with a pass of its own over the stamps in memory they
        // took 331 us (182 us that pass).
        constexpr int T0 = q == 0 ? 0 : C::HR - 2;            // output rows whose taps are in
        constexpr int NT = q == 0 ? C::HR - 2 : C::HR + 2;
        float val[C::HR];  // this lane's column
        static_for<0, C::HR>([&](auto rr) { val[decltype(rr)::value] = st[decltype(rr)::value * C::LSO + l]; });
        auto src = [&](auto ss) {
          constexpr int sr = decltype(ss)::value;
          if constexpr (sr < q * C::HR) return carry[sr - (C::HR - 5)];
          else return val[sr - q * C::HR];
        };
        __syncthreads();  // every lane has read its column
        static_for<0, NT>([&](auto tt) {
          constexpr int t = T0 + decltype(tt)::value;
          float acc = 0.f;
          static_for<0, 6>([&](auto dd) {
            constexpr int sr = t + decltype(dd)::value - 3;
            if constexpr (sr >= 0 && sr < W) acc = fmaf(wy[decltype(dd)::value], src(std::integral_constant<int, sr>{}), acc);
          });
          st[(t - T0) * LS + 4 + l] = acc;
        });
        if constexpr (q == 0) {
          static_for<0, 5>([&](auto ii) { carry[decltype(ii)::value] = val[C::HR - 5 + decltype(ii)::value]; });
        }
        for (int i = l; i < 2 * NT; i += W)
          *reinterpret_cast<float4*>(st + (i >> 1) * LS + (i & 1) * (W + 4)) = make_float4(0.f, 0.f, 0.f, 0.f);
        __syncthreads();
#pragma unroll 2
        for (int rw = r4; rw < NT; rw += 4) {
          const float4* s4 = reinterpret_cast<const float4*>(st + rw * LS + c4);
          const float4 a = s4[0], b = s4[1], e = s4[2];  // columns c4 - 4 .. c4 + 7
          const float in[12] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w, e.x, e.y, e.z, e.w};
          v4f_any o;
          static_for<0, 4>([&](auto jj) {
            constexpr int j = decltype(jj)::value;
            float h = 0.f;
            static_for<0, 6>([&](auto dd) { h = fmaf(wxn[decltype(dd)::value], in[j + decltype(dd)::value + 1], h); });
            o[j] = h;
          });
          if (live) __builtin_nontemporal_store(o, reinterpret_cast<v4f_any*>(outp + (T0 + rw) * W + c4));
        }
      } else if (live) {
        // Four pixels per lane: beside the arithmetic, four times as many
        // 4-byte stores hold the wavefronts up (64 x 64: 491 us per 100,000
        // stamps with them).  `out` is only promised to be aligned as floats are.
        const bool acc = (p.flags & kAccumulate) != 0;
        float* o = outp + (q * C::HR + r4) * W + c4;
        static_for<0, C::HR / 4>([&](auto ii) {
          constexpr int i = decltype(ii)::value;
          const float4 t = *reinterpret_cast<const float4*>(st + (4 * i + r4) * C::LSO + c4);
          v4f_any v = {t.x, t.y, t.z, t.w};
          v4f_any* dst = reinterpret_cast<v4f_any*>(o + 4 * i * W);
          if (acc) v += *dst;
          __builtin_nontemporal_store(v, dst);  // streamed output
        });
      }
      __syncthreads();
    });
  }
  if (live && !G.ok && l == 0) atomicAdd(p.invalid, 1ull);
}

template <int W, bool EIG, bool LZ, bool PT, bool PROF>
static hipError_t launch_small(const RenderArgs& args, hipStream_t stream) {
  using C = SmallCfg<W, EIG>;
  constexpr int64_t kMaxBlocks = 1 << 30;
  RenderArgs p = args;
  int64_t done = 0;
  while (done < args.n) {
    const int64_t chunk = std::min<int64_t>(args.n - done, kMaxBlocks * C::SPB);
    p.x = args.x + done;
    p.y = args.y + done;
    p.flux = args.flux + done;
    p.r_e = args.r_e + done;
    p.e1 = args.e1 + done;
    p.e2 = args.e2 + done;
    p.mix_id = args.mix_id ? args.mix_id + done : nullptr;
    p.out = args.out + done * (int64_t)W * W;
    p.psf_px = args.psf_px ? args.psf_px + done : nullptr;
    p.psf_py = args.psf_py ? args.psf_py + done : nullptr;
    p.psf_id = args.psf_id ? args.psf_id + done : nullptr;
    p.prof_a = args.prof_a ? args.prof_a + done : nullptr;
    p.prof_b = args.prof_b ? args.prof_b + done : nullptr;
    p.n = chunk;
    const unsigned blocks = (unsigned)((chunk + C::SPB - 1) / C::SPB);
    hipLaunchKernelGGL((render_small_kernel<W, EIG, LZ, PT, PROF>), dim3(blocks), dim3(C::BLOCK), 0, stream, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    done += chunk;
  }
  return hipSuccess;
}

template <int W, bool PROF>
static hipError_t launch_one_psf(const RenderArgs& args, hipStream_t stream) {
  if (args.flags & kLanczos3)
    return args.eig_J > 0 ? launch_small<W, true, true, false, PROF>(args, stream)
                          : launch_small<W, false, true, false, PROF>(args, stream);
  return args.eig_J > 0 ? launch_small<W, true, false, false, PROF>(args, stream)
                        : launch_small<W, false, false, false, PROF>(args, stream);
}

template <int W>
hipError_t launch_render_small(const RenderArgs& args, hipStream_t stream) {
  if (args.psf_id) {  // per-galaxy constant PSFs (eig_J == 0), mixtures from the tables
    if (args.eig_J > 0 || args.prof != kProfTable) return hipErrorInvalidValue;
    return (args.flags & kLanczos3) ? launch_small<W, false, true, true, false>(args, stream)
                                    : launch_small<W, false, false, true, false>(args, stream);
  }
  // Galaxies with mixtures of their own take instantiations of their own: as
  // a test in the shared ones they cost the plain render 1.6% at 128 x 128
  // (253.3 us against 249.2 for 10,000 large galaxies) and 0.5% below.
  return args.prof != kProfTable ? launch_one_psf<W, true>(args, stream) : launch_one_psf<W, false>(args, stream);
}

template hipError_t launch_render_small<16>(const RenderArgs&, hipStream_t);
template hipError_t launch_render_small<32>(const RenderArgs&, hipStream_t);
template hipError_t launch_render_small<64>(const RenderArgs&, hipStream_t);
template hipError_t launch_render_small<128>(const RenderArgs&, hipStream_t);

}  // namespace gfc
