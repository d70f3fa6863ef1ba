// Shared tail of the adjoint kernels: the chain rule from the frequency- and
// pixel-domain sums of one stamp to d loss / d(x, y, flux, log r_e, e1, e2)
// and the per-galaxy amplitude partials (Section 2, steps 3 and 4
// differentiated).
#pragma once

#include "gfc_device.hpp"

namespace gfc {

// Column c of a real image's row spectra from rows transformed as W / 2 packed
// values Z, times the column's phase exp(2 pi i (n + f) c / W) and its weight:
//   pc (e + tw d),  e, d = Z[c] +- conj Z[W/2 - c],  tw = -i exp(-2 pi i c / W).
// Weight: h(k_x) / W^2 with h = 1 on column 0 and 2 elsewhere, halved for the
// factor 2 in e + tw d.  Columns 0 and W / 2 are real, 2 (Re +- Im) of Z[0],
// and are taken together, the second times i: 2 (1 + i) conj Z[0] (phase 1).
// The phase multiplies last, by itself.  Folded with tw into one factor each
// of Z[c] and conj Z[W/2 - c] it saves four multiply-adds in twelve, but the
// factors then are sums of size one to two, which round the small phases of
// the low columns by 2.2e-8 rms instead of 1.1e-8, in every row alike: the x
// gradient of a fit's step erred by 1.3-1.65 times as much.
struct ColumnSplit {
  float2 tw, pc;
  GFC_HD float2 at(float2 zc, float2 zr) const {  // zr = Z[(W/2 - c) mod W/2]
    const float2 b = cconj(zr);
    return cmul(cfma(tw, csub(zc, b), cadd(zc, b)), pc);
  }
};

// wc = exp(-2 pi i c / W)
template <int W>
GFC_HD ColumnSplit column_split(float f, int n, int c, float2 wc) {
  constexpr float wt = 1.f / ((float)W * (float)W);
  float s, co;
  shift_phase<W>(f, n, c, &s, &co);
  ColumnSplit r;
  r.tw = c == 0 ? make_float2(-1.f, 0.f) : rot90<-1>(wc);
  r.pc = c == 0 ? make_float2(0.5f * wt, 0.5f * wt) : make_float2(co * wt, -s * wt);
  return r;
}

// Contributions of mixture component k to the chain rule (dx, dy, dF and the
// three entries of dL/dB), and its amplitude partial written to ap[k].
// pk_sum[k * pk_stride]: the component's Fourier sum p_k; racc[k racc_stride + i]: its
// real-space sums (sum g N, g N z_x, g N z_y, g N z_x^2, g N z_x z_y, g N z_y^2).
struct CompTerms {
  float dx, dy, dF, L11, L12, L22;
};

template <int W>
__device__ inline CompTerms bwd_component_terms(const RenderArgs& p, const Galaxy& G, int k, unsigned rmask,
                                                const float* pk_sum, int pk_stride, const float* racc,
                                                int racc_stride, float* ap) {
  CompTerms c = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (k >= G.K) {
    ap[k] = 0.f;
    return c;
  }
  const float* amp = p.amp + G.table * kKmax;
  const float* var = p.var + G.table * kKmax;
  const float trB = G.b11 + G.b22;
  const float F = G.flux;
  const float pamp = p.pg[5];
  const float v = var[k];
  const float A = amp[k];
  const float tr = v * trB;
  const float w = route_weight<W>(tr, p.flags);
  const float n = (0.5f * (float)W) * __builtin_amdgcn_rsqf(tr);
  const float pk = pk_sum[k * pk_stride];
  float g0 = 0.f;
  if (rmask & (1u << k)) {
    const float* R = racc + racc_stride * k;
    g0 = R[0];
    const float sxx = fmaf(v, G.b11, p.pg[2]);
    const float sxy = fmaf(v, G.b12, p.pg[3]);
    const float syy = fmaf(v, G.b22, p.pg[4]);
    const float det = fmaf(sxx, syy, -(sxy * sxy));
    const float rdet = __builtin_amdgcn_rcpf(det);  // det > 0: a covariance convolved with the PSF's
    const float ixx = syy * rdet, ixy = -sxy * rdet, iyy = sxx * rdet;
    const float rk = (1.f - w) * F * A * pamp;
    c.dx = rk * R[1];
    c.dy = rk * R[2];
    c.L11 = 0.5f * rk * v * (R[3] - ixx * R[0]);
    c.L12 = rk * v * (R[4] - ixy * R[0]);
    c.L22 = 0.5f * rk * v * (R[5] - iyy * R[0]);
  }
  c.dF = A * (w * pk + (1.f - w) * pamp * g0);
  ap[k] = G.ok ? F * (w * pk + (1.f - w) * pamp * g0) : 0.f;
  // smooth routing: dL/dw_k * dw/dn * dn/d(b11 or b22)
  const float dLdw = F * A * (pk - pamp * g0);
  const float dn = -0.5f * n * __builtin_amdgcn_rcpf(trB);
  const float t = route_slope<W>(n, p.flags) * dLdw * dn;
  c.L11 += t;
  c.L22 += t;
  return c;
}

// Sum of CompTerms over each group of 16 lanes (fixed order); every
// lane of the group receives the totals.  Called with every lane active.
__device__ __forceinline__ CompTerms sum16(CompTerms c) {
  c.dx = lane_sum<16>(c.dx);
  c.dy = lane_sum<16>(c.dy);
  c.dF = lane_sum<16>(c.dF);
  c.L11 = lane_sum<16>(c.L11);
  c.L12 = lane_sum<16>(c.L12);
  c.L22 = lane_sum<16>(c.L22);
  return c;
}

// The rest of the chain rule on one lane: ax, ay, a11, a12, a22 are the stamp
// sums of the Fourier-path terms (see the adjoint kernels), tot the summed
// component terms; B -> C0 -> (log r_e, e1, e2).
template <int W>
__device__ inline void bwd_chain_finish(const RenderArgs& p, const Galaxy& G, int64_t gidx, float ax, float ay,
                                        float a11, float a12, float a22, const CompTerms& tot,
                                        float* grad_params) {
  constexpr float kPi = 3.14159265358979f;
  const float F = G.flux;
  const float dxs = fmaf(2.f * kPi * F, ax, tot.dx);
  const float dys = fmaf(2.f * kPi * F, ay, tot.dy);
  const float L11 = fmaf(-2.f * kPi * kPi * F, a11, tot.L11);
  const float L12 = fmaf(-4.f * kPi * kPi * F, a12, tot.L12);
  const float L22 = fmaf(-2.f * kPi * kPi * F, a22, tot.L22);
  // B = M C0 M^T  ->  dL/dC0 = M^T (dL/dB) M with symmetric dL/dB
  const float m00 = p.cdinv[0], m01 = p.cdinv[1], m10 = p.cdinv[2], m11 = p.cdinv[3];
  const float g11 = L11, g12 = 0.5f * L12, g22 = L22;
  // T = (dL/dB) M
  const float t00 = g11 * m00 + g12 * m10, t01 = g11 * m01 + g12 * m11;
  const float t10 = g12 * m00 + g22 * m10, t11 = g12 * m01 + g22 * m11;
  const float c11g = m00 * t00 + m10 * t10;
  const float c12g = 2.f * (m00 * t01 + m10 * t11);
  const float c22g = m01 * t01 + m11 * t11;
  // C0 = s [[1 + e^2 - 2 e1, 2 e2], [2 e2, 1 + e^2 + 2 e1]], s = r_e^2 / (1 + e)^2
  const float re = p.r_e[gidx], e1 = p.e1[gidx], e2 = p.e2[gidx];
  const float esq = e1 * e1 + e2 * e2, e = sqrtf(esq);
  const float r1e = __builtin_amdgcn_rcpf(1.f + e);
  const float s = re * re * (r1e * r1e);
  const float c11 = s * (1.f + esq - 2.f * e1), c12 = 2.f * s * e2, c22 = s * (1.f + esq + 2.f * e1);
  const float dlogre = 2.f * (c11g * c11 + c12g * c12 + c22g * c22);
  float de1 = 0.f, de2 = 0.f;
  if (e > 0.f) {
    // e1 / e and e2 / e stay correctly rounded divisions: e may be as small
    // as the square root of a denormal
    const float ds1 = -2.f * s * r1e * (e1 / e), ds2 = -2.f * s * r1e * (e2 / e);
    const float a11e = 1.f + esq - 2.f * e1, a22e = 1.f + esq + 2.f * e1;
    de1 = c11g * (ds1 * a11e + s * (2.f * e1 - 2.f)) + c12g * (ds1 * 2.f * e2) +
          c22g * (ds1 * a22e + s * (2.f * e1 + 2.f));
    de2 = c11g * (ds2 * a11e + s * 2.f * e2) + c12g * (ds2 * 2.f * e2 + 2.f * s) +
          c22g * (ds2 * a22e + s * 2.f * e2);
  }
  float* gpo = grad_params + gidx * 6;
  gpo[0] = dxs;
  gpo[1] = dys;
  gpo[2] = tot.dF;
  gpo[3] = dlogre;
  gpo[4] = de1;
  gpo[5] = de2;
}

}  // namespace gfc
