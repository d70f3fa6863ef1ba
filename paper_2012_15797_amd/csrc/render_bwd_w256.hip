// Adjoint of the forward render for 256 x 256 stamps (Lang 2020, Section 2,
// steps 3-8, differentiated); same sums as the W <= 128 adjoint.
//
// One 1,024-thread workgroup per stamp, the half spectrum of the upstream
// gradient g kept on the chip: the forward kernel's stages run backwards, with
// its split of the stamp and its exchanges.  g is read once and nothing else
// moves through memory.  What bounds it is VALU issue (about 6,000
// instructions per wavefront and stamp on large galaxies, a quarter of them
// the real-space sums) and the barriers between the phases: the LDS holds one
// stamp per CU.  500 stamps (r_e 10..60 px, 8 components) take 120 us for the
// whole call; one 512-thread workgroup per stamp working through a slab in
// device memory, with 750 B of spilled registers per lane and no skip of
// negligible bins, took 355 us.
//
//  load           eight lanes per row read 32 pixels each of two rows (the
//                 forward's store pattern: whole 128-byte segments) and
//                 accumulate the real-space sums.
//  row phase      per half (128 rows): the row as 128 packed complex values, a
//                 radix-8 stage on the lane, an exchange between the row's
//                 lanes, a 16-point FFT.
//  column read    lane (c, h) reads its 16 rows of the half, of columns c and
//                 128 - c, and forms the row's real-input spectrum on the way.
//  column DFT     the radix-8 stage over the rows 32 apart, an exchange
//                 between the eight lanes of a column, a 32-point FFT: lane
//                 (c, h) ends with the bins k_y = 8m + h of column c.
//  bins           U0 per bin; the component loop in blocks of eight bins with
//                 the forward's skip of negligible blocks.
//  sums           fixed-order reductions, then the chain rule on the first
//                 wavefront.
// The integer centre enters the phases as exact table entries, so g is never
// rolled.
#include "bwd_common.hpp"
#include "gfc_device.hpp"
#include "gfc_internal.hpp"
#include "gfc_launch.hpp"
#include "w256_common.hpp"

namespace gfc {

// The upstream gradient is only promised to be aligned as floats are.
typedef const __attribute__((address_space(1))) v4f_any* GlobalF4;

__global__ void __launch_bounds__(w256::BLOCK)
render_bwd_w256_kernel(RenderArgs p, const float* __restrict__ gout, float* __restrict__ grad_params,
                       float* __restrict__ amp_part) {
  using namespace w256;
  // rows of a half [HROWS][TS] and the exchanges' slices, then the p_k
  // partials [K][BLOCK]
  __shared__ float2 s_buf[LDS_F2];
  __shared__ float2 s_py[W + 2];
  __shared__ float2 s_nyq[W];
  __shared__ float2 s_ux[NC];           // U0 of the Nyquist row's omega = -1/2 twin, per column
  __shared__ float2 s_twc[8 * TWC];     // s_twc[h][8 k + g] = w^(g (8 k + h)), w = exp(2 pi i / 256)
  constexpr int TWR = 17;
  __shared__ float2 s_twr[8 * TWR];     // s_twr[r][n1] = exp(-2 pi i r n1 / 128), rows 17 apart (distinct banks)
  __shared__ float4 s_cmp[kKmax];       // per component: v, w A, w A v, w (zero past the table's K)
  __shared__ float s_rw[kKmax][NWAVE][6];  // real-space sums per wavefront
  __shared__ float s_racc[kKmax * 6];
  __shared__ float s_red[5][NWAVE];
  __shared__ float s_pk[kKmax];
  static_assert(kKmax * BLOCK <= 2 * LDS_F2, "the p_k partials fit in the half buffer");

  const int t = threadIdx.x;
  const int lane = t & 63;
  const int wv = __builtin_amdgcn_readfirstlane(t >> 6);  // wavefront index (scalar)
  const int64_t stamp = blockIdx.x;  // the launcher sizes each grid to its chunk

  // Row phase: rows 8 wv + yl and 128 further down, class r: pixels x = 4 r +
  // 32 q + 0..3, as z[n] = g[2n] + i g[2n+1] for n = 2 r + kk + 16 q in
  // zq[half][kk][q].  Both rows are in flight while the galaxy is formed.
  float2 zq[2][2][8];
  {
    const int yl = lane & 7, r = lane >> 3;
    GlobalF4 row = (GlobalF4)(gout + stamp * (int64_t)(W * W) + (8 * wv + yl) * W) + r;
    static_for<0, 2>([&](auto hh) {
      constexpr int half = decltype(hh)::value;
      static_for<0, 8>([&](auto qq) {
        constexpr int q = decltype(qq)::value;
        const v4f_any v = row[half * (HROWS * W / 4) + 8 * q];
        zq[half][0][q] = make_float2(v.x, v.y);
        zq[half][1][q] = make_float2(v.z, v.w);
      });
    });
  }
  __builtin_amdgcn_sched_barrier(0);
  Galaxy G = load_galaxy<W>(p, stamp);
  make_uniform(G);
  const float trB = G.b11 + G.b22;

  if (t < 256) {
    const int hh = t >> 5, kg = t & 31;  // kg = 8 k + g
    s_twc[hh * TWC + kg] = twiddle_rt<+1, W>((kg & 7) * (8 * (kg >> 3) + hh));
  } else if (t < 256 + 8 * 16) {
    const int r = (t - 256) >> 4, n1 = t & 15;
    s_twr[r * TWR + n1] = twiddle_rt<-1, 128>(r * n1);
  }
  // Lane k of every wavefront works out component k's route weight; the
  // real-space mask is the ballot of w < 1 (whatever A_k: dL/dA_k needs it),
  // and the first wavefront leaves the Fourier-loop constants in LDS.
  unsigned rmask;
  float vk = 0.f;
  {
    float wk = 0.f, ak = 0.f;
    bool rs = false;
    if (lane < G.K) {
      vk = p.var[G.table * kKmax + lane];
      wk = route_weight<W>(vk * trB, p.flags);
      ak = p.amp[G.table * kKmax + lane];
      rs = wk < 1.f;
    }
    rmask = (unsigned)__ballot(rs) & ((1u << kKmax) - 1u);
    if (t < kKmax) {
      const float wa = wk * ak;
      s_cmp[t] = make_float4(vk, wa, wa * vk, wk);
    }
  }

  // Real-space sums.  Along a row (dy fixed) z = S^-1 (dx, dy) has zx = ixx dx
  // + ixy dy and zy = al + be zx with al = dy / syy, be = -sxy / syy, and the
  // quadratic form is q = dy al + zx^2 / ixx.  So a row needs the moments
  // sum g N zx^p (p = 0, 1, 2) only, with the log2 of nrm exp(-q/2) as
  // c0 + c2 zx^2.
  for (unsigned mk = rmask; mk != 0; mk &= mk - 1) {
    const int k = __builtin_ctz(mk);
    const float v = lane_f(vk, k);
    const float sxx = fmaf(v, G.b11, p.pg[2]);
    const float sxy = fmaf(v, G.b12, p.pg[3]);
    const float syy = fmaf(v, G.b22, p.pg[4]);
    const float det = fmaf(sxx, syy, -(sxy * sxy));
    const float rdet = __builtin_amdgcn_rcpf(det);
    const float ixx = syy * rdet, ixy = -sxy * rdet;
    const float rsyy = __builtin_amdgcn_rcpf(syy);
    const float be = -sxy * rsyy;
    const float lnrm = __builtin_amdgcn_logf(kInv2Pi * __builtin_amdgcn_rsqf(det));
    const float c2 = kHalfLog2e * __builtin_amdgcn_rcpf(ixx);
    float a[6];
    static_for<0, 2>([&](auto hh) {
      constexpr int half = decltype(hh)::value;
      const float dy = (float)(half * HROWS + 8 * wv + (lane & 7)) - G.y0 - p.pg[1];
      const float al = dy * rsyy;
      const float zx0 = fmaf(ixx, (float)(4 * (lane >> 3)) - G.x0 - p.pg[0], ixy * dy);
      const float c0 = fmaf(kHalfLog2e * al, dy, lnrm);
      float m0 = 0.f, m1 = 0.f, m2 = 0.f;
      static_for<0, 8>([&](auto qq) {
        constexpr int q = decltype(qq)::value;
        static_for<0, 4>([&](auto ii) {
          constexpr int i = decltype(ii)::value;
          const float2 z = zq[half][i / 2][q];
          const float zx = fmaf(ixx, (float)(32 * q + i), zx0);
          const float zz = zx * zx;
          const float gn = ((i & 1) ? z.y : z.x) * __builtin_amdgcn_exp2f(fmaf(c2, zz, c0));
          m0 += gn;
          m1 = fmaf(gn, zx, m1);
          m2 = fmaf(gn, zz, m2);
        });
      });
      // sum g N (1, zx, zy, zx^2, zx zy, zy^2) from the moments
      const float a2 = fmaf(be, m1, al * m0), a4 = fmaf(be, m2, al * m1), a5 = fmaf(be, a4, al * a2);
      if constexpr (half == 0) {
        a[0] = m0, a[1] = m1, a[2] = a2, a[3] = m2, a[4] = a4, a[5] = a5;
      } else {
        a[0] += m0, a[1] += m1, a[2] += a2, a[3] += m2, a[4] += a4, a[5] += a5;
      }
    });
    static_for<0, 6>([&](auto ii) { a[decltype(ii)::value] = lane_sum<64>(a[decltype(ii)::value]); });
    if (lane == 0) static_for<0, 6>([&](auto ii) { s_rw[k][wv][decltype(ii)::value] = a[decltype(ii)::value]; });
  }
  __syncthreads();  // the tables

  // ------------------------------------------------------------ rows, per half
  const int c = t >> 3, h = t & 7;          // column phase: column c, rows h (mod 8)
  float2 X4[4][8];                          // row spectra: X4[k][q] of row 8k + h + 32q, column c
  static_for<0, 2>([&](auto hh) {
    constexpr int half = decltype(hh)::value;
    int ln = lane;
    asm volatile("" : "+v"(ln));  // recomputed per half, not held across it
    const int yl = ln & 7, r = ln >> 3;
    const int yloc = 8 * wv + yl;
    // Z[8m + r] = sum_{n1} w16^{-n1 m} (w128^{-n1 r} A_{n1}[r]) with
    // A_{n1}[g] = sum_q w8^{-q g} z[n1 + 16 q]: lane r has n1 = 2 r + kk and
    // hands entry g to lane g of the row.
    if constexpr (half == 1) __syncthreads();  // the first half has been read from s_buf
    float2 R[16];
    {
      float2* rxb = s_buf + wv * (8 * TS) + yl * RXS;  // this row's slot, in the wavefront's own rows
      static_for<0, 2>([&](auto kk) {
        constexpr int k = decltype(kk)::value;
        fft<8, -1>(zq[half][k]);
        static_for<0, 8>([&](auto gg) {
          constexpr int g = decltype(gg)::value;
          rxb[9 * r + g] = zq[half][k][g];
        });
        wave_lds_sync();
        static_for<0, 8>([&](auto ii) {
          constexpr int i = decltype(ii)::value;
          R[2 * i + k] = rxb[9 * i + r];
        });
        wave_lds_sync();  // read before the slot is overwritten
      });
    }
    const float2* twr = s_twr + r * TWR;
    static_for<1, 16>([&](auto nn) {
      constexpr int n1 = decltype(nn)::value;
      R[n1] = cmul(R[n1], twr[n1]);
      if constexpr (n1 % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    });
    fft<16, -1>(R);
    {
      float2* row = s_buf + yloc * TS;
      static_for<0, 16>([&](auto mm) {
        constexpr int m = decltype(mm)::value;
        row[8 * m + r] = R[m];
      });
    }
    __syncthreads();
    // Real-input split while reading: Gr2[c] = e + t with e = Z[c] + conj
    // Z[128 - c], t = -i w256^{-c} (Z[c] - conj Z[128 - c]).  Column 0 is the
    // packed pair (Gr2[0], Gr2[128]), both real: 2 (Re +- Im) of Z[0].
    {
      const float2 tw = rot90<-1>(twiddle_rt<-1, W>(c));
      const int cb = (NC - c) & (NC - 1);
      static_for<0, 4>([&](auto kk) {
        constexpr int k = decltype(kk)::value;
        static_for<0, 4>([&](auto qq) {
          constexpr int q = decltype(qq)::value;
          const float2* row = s_buf + (8 * k + h + 32 * q) * TS;
          const float2 a = row[c], b = cconj(row[cb]);
          float2 v = cfma(tw, csub(a, b), cadd(a, b));
          if (c == 0) v = make_float2(2.f * (a.x + a.y), 2.f * (a.x - a.y));
          X4[k][4 * half + q] = v;
        });
        __builtin_amdgcn_sched_barrier(0);
      });
    }
  });
  __syncthreads();  // the second half has been read; s_buf takes the column exchange

  // ------------------------------------------------------------ column DFT
  // G[8m + g] = sum_j w32^{-m j} w^{-g j} sum_q w8^{-g q} X[j + 32 q], j = 8k + h
  float2 Gk[M];  // 2 G[k_y = 8m + h][c]  (c = 0: packed with column 128)
  {
    float2* cxb = s_buf + wv * (8 * CXS) + (lane >> 3) * CXS;  // this column's slot
    static_for<0, 4>([&](auto kk) {
      constexpr int k = decltype(kk)::value;
      __builtin_amdgcn_sched_barrier(0);  // one chunk's twiddle loads in flight at a time
      fft<8, -1>(X4[k]);
      const float2* tw = s_twc + h * TWC + 8 * k;
      static_for<1, 8>([&](auto gg) {
        constexpr int g = decltype(gg)::value;
        X4[k][g] = cmulc(X4[k][g], tw[g]);
      });
      static_for<0, 8>([&](auto gg) {
        constexpr int g = decltype(gg)::value;
        cxb[9 * h + g] = X4[k][g];
      });
      wave_lds_sync();
      static_for<0, 8>([&](auto ii) {
        constexpr int i = decltype(ii)::value;
        Gk[8 * k + i] = cxb[9 * i + h];
      });
      wave_lds_sync();  // read before the next chunk overwrites the slot
    });
    fft<M, -1>(Gk);
  }

  // ------------------------------------------------------------ phases, Nyquist column
  const float nu = (float)c * (1.f / W);
  const float hW = (float)h * (1.f / W);
  // Threads t < W also take row t of column k_x = 128 (nu = +-1/2), threads
  // t < NC the omega = -1/2 twin of the Nyquist row in column t (uniform per
  // wavefront).
  const bool nyq = t < W, twin = t < NC;
  const float omN = (t < W / 2) ? (float)t * (1.f / W) : (t == W / 2 ? 0.5f : (float)(t - W) * (1.f / W));
  float2 py = make_float2(1.f, 0.f);
  if (nyq) {
    float sy, cy;
    sincospi_poly(-2.f * G.fy * omN, &sy, &cy);
    py = cmul(make_float2(cy, sy), twiddle_rt<-1, W>(G.ny * t));
    s_py[t] = py;
    if (t == W / 2) s_py[W] = cconj(py);  // omega = -1/2 (the integer part's phase is real there)
  }
  if (c == 0) {
    static_for<0, M>([&](auto mm) {
      constexpr int m = decltype(mm)::value;
      s_nyq[D * m + h] = Gk[m];
    });
  }
  __syncthreads();
  // Unpack the packed column: Z = G0 + i GN, with G0 and GN Hermitian in k_y.
  if (c == 0) {
    static_for<0, M>([&](auto mm) {
      constexpr int m = decltype(mm)::value;
      const float2 zb = cconj(s_nyq[(W - D * m - h) & (W - 1)]);
      Gk[m] = cscale(cadd(Gk[m], zb), 0.5f);
    });
  }

  // ------------------------------------------------------------ U0
  GlobalF2 psfm = (GlobalF2)p.psf_main;
  float ure[M], uim[M];
  {
    // h(k_x) / W^2 with h = 1 on column 0 and 2 elsewhere, halved for the factor 2 in Gk
    const float colw = (c == 0 ? 0.5f : 1.f) / ((float)W * (float)W);
    float sx, cx;
    sincospi_poly(-2.f * G.fx * nu, &sx, &cx);
    const float2 px = cscale(cmul(make_float2(cx, sx), twiddle_rt<-1, W>(G.nx * c)), colw);
    const int pidx0 = (h >> 2) * (4 * NC) + 4 * c + (h & 3);  // the forward's decimation-4 order
    static_for<0, M>([&](auto mm) {
      constexpr int m = decltype(mm)::value;
      const float2 P = ld2(psfm, pidx0 + 2 * m * (4 * NC));
      const float2 gp2 = cmul(cmulc(P, Gk[m]), px);  // P conj(G) x phase x weight
      float2 u;
      if constexpr (D * m == W / 2) {
        const float2 q0 = s_py[W / 2 + h];
        u = cmul(gp2, h ? q0 : cscale(q0, 0.5f));
        if (h == 0) s_ux[c] = cmul(gp2, cscale(s_py[W], 0.5f));
      } else {
        u = cmul(gp2, s_py[D * m + h]);
      }
      ure[m] = u.x;
      uim[m] = u.y;
      asm volatile("" : "+v"(ure[m]), "+v"(uim[m]));  // formed here, not sunk to its uses with its operands held
      if constexpr (m % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // bounds the loads in flight
    });
  }
  // the Nyquist column's points (+1/2, omN), (-1/2, omN) and the twin (t / W, -1/2)
  float ure3[3] = {0.f, 0.f, 0.f}, uim3[3] = {0.f, 0.f, 0.f};
  if (nyq) {
    const float2 za = s_nyq[t], zb = cconj(s_nyq[(W - t) & (W - 1)]);
    const float2 d = csub(za, zb);
    const float2 GN = make_float2(0.5f * d.y, -0.5f * d.x);  // (za - conj zb) / (2 i)
    // the integer x shift at k_x = 128 is exp(-i pi n_x) = +-1
    const float sgn = (G.nx & 1) ? -0.25f : 0.25f;
    const float2 gamN = cscale(cmulc(ld2((GlobalF2)p.psf_nyq, t), GN), sgn / ((float)W * (float)W));
    float sxh, cxh;
    sincospi_poly(-G.fx, &sxh, &cxh);
    const bool corner = (t == W / 2);
    const float2 pyA = corner ? cscale(py, 0.5f) : py;
    const float2 pyB = corner ? cscale(cconj(py), 0.5f) : make_float2(0.f, 0.f);
    const float2 eM = make_float2(cxh, sxh), eP = make_float2(cxh, -sxh);
    const float2 u1 = cmul(cmul(gamN, eM), pyA), u2 = cmul(cmul(gamN, eP), pyA);
    const float2 u3 = cmul(cmul(gamN, eM), pyB), u4 = cmul(cmul(gamN, eP), pyB);
    // corner twins folded into their partners (the transform is even; see the
    // W <= 128 adjoint)
    ure3[0] = u1.x + u4.x;
    uim3[0] = u1.y - u4.y;
    ure3[1] = u2.x + u3.x;
    uim3[1] = u2.y - u3.y;
  }
  __syncthreads();  // s_ux is written; the p_k partials take s_buf
  if (twin) {
    const float2 u = s_ux[t];
    ure3[2] = u.x;
    uim3[2] = u.y;
  }

  // ------------------------------------------------------------ component loop
  float* s_pkl = reinterpret_cast<float*>(s_buf);  // [kKmax][BLOCK] per-lane p_k partials
  const float lamq = -kQ * shape_min_eig(G);
  float ax = 0.f, ay = 0.f, a11 = 0.f, a12 = 0.f, a22 = 0.f;
  // the irregular points first (wavefronts 0..3): they initialise the partials
  {
    float g3[3] = {0.f, 0.f, 0.f}, S[3] = {0.f, 0.f, 0.f}, S1[3] = {0.f, 0.f, 0.f};
    const float nt = (float)t * (1.f / W);
    if (nyq) {
      const float qa = kQ * G.b11 * 0.25f, qb = kQ * G.b12, qd = kQ * G.b22;
      g3[0] = fmaf(omN, fmaf(qd, omN, qb), qa);
      g3[1] = fmaf(omN, fmaf(qd, omN, -qb), qa);
      g3[2] = kQ * fmaf(nt, fmaf(G.b11, nt, -G.b12), 0.25f * G.b22);
    }
    for (int k = 0; k < G.K; ++k) {
      float pk = 0.f;
      if (nyq) {
        const float4 cp = s_cmp[k];
        static_for<0, 3>([&](auto jj) {
          constexpr int j = decltype(jj)::value;
          const float e = __builtin_amdgcn_exp2f(cp.x * g3[j]);
          S[j] = fmaf(cp.y, e, S[j]);
          S1[j] = fmaf(cp.z, e, S1[j]);
          pk = fmaf(ure3[j], e, pk);
        });
      }
      s_pkl[k * BLOCK + t] = pk;
    }
    if (nyq) {
      const float n3[3] = {0.5f, -0.5f, nt}, o3[3] = {omN, omN, -0.5f};
      static_for<0, 3>([&](auto jj) {
        constexpr int j = decltype(jj)::value;
        const float si = S[j] * uim3[j], r1 = S1[j] * ure3[j];
        ax = fmaf(n3[j], si, ax);
        ay = fmaf(o3[j], si, ay);
        a11 = fmaf(n3[j] * n3[j], r1, a11);
        a12 = fmaf(n3[j] * o3[j], r1, a12);
        a22 = fmaf(o3[j] * o3[j], r1, a22);
      });
    }
  }
  // The regular bins, eight at a time (k_y in [64 b, 64 b + 63]): omega =
  // c_m + h/W with a compile-time c_m, the quadratic expanded about h/W.  A
  // component is negligible in a block (every exponent below -kSkipLog2) when
  // its variance is at least vmax, as in the forward kernel.
  float m_si = 0.f, m_csi = 0.f, m_r = 0.f, m_cr = 0.f, m_ccr = 0.f;
  const float g2 = kQ * G.b22, g1 = 2.f * kQ * G.b12 * nu;
  const float e0 = fmaf(hW, fmaf(g2, hW, g1), kQ * G.b11 * nu * nu);
  const float e1 = fmaf(2.f * g2, hW, g1);
  const float nlo = (float)(8 * wv) * (1.f / W);
  const float r2[4] = {nlo * nlo, fmaf(nlo, nlo, 0.0625f), fmaf(nlo, nlo, (65.f * 65.f) / (256.f * 256.f)),
                       fmaf(nlo, nlo, 1.f / (256.f * 256.f))};
  static_for<0, M / 8>([&](auto bb) {
    constexpr int b = decltype(bb)::value;
    const float vmax = uniform_f(kSkipLog2 * __builtin_amdgcn_rcpf(lamq * r2[b]));  // rcp(0) = +inf
    float gq[8], S[8], S1[8];
    static_for<0, 8>([&](auto jj) {
      constexpr int j = decltype(jj)::value;
      constexpr int m = 8 * b + j;
      if constexpr (D * m == W / 2) {  // k_y = 128 + h: the Nyquist row (+1/2) for h = 0
        const float om = h ? -0.5f + hW : 0.5f;
        gq[j] = fmaf(om, fmaf(g2, om, g1), kQ * G.b11 * nu * nu);
      } else {
        constexpr float cm = (D * m < W / 2) ? (float)(D * m) * (1.f / W) : (float)(D * m - W) * (1.f / W);
        gq[j] = fmaf(cm, fmaf(cm, g2, e1), e0);
      }
      S[j] = 0.f;
      S1[j] = 0.f;
    });
    float4 cpn = s_cmp[0];
    float pkn = s_pkl[t];
    for (int k = 0; k < G.K; ++k) {
      // the next component's constants and partial are read one iteration
      // ahead (clamped into the arrays; the last read is not used)
      const float4 cp = cpn;
      const float before = pkn;
      const int kn = min(k + 1, kKmax - 1);
      cpn = s_cmp[kn];
      pkn = s_pkl[kn * BLOCK + t];
      const float v = uniform_f(cp.x);
      // w = 0: p_k is only ever multiplied by w or by the ramp slope, both zero
      if (uniform_f(cp.w) == 0.f || !(v < vmax)) continue;
      const float wa = cp.y, wav = cp.z;
      float pk[2] = {0.f, 0.f};  // two chains: a smaller rounding error than one
      static_for<0, 8>([&](auto jj) {
        constexpr int j = decltype(jj)::value;
        const float e = __builtin_amdgcn_exp2f(v * gq[j]);
        S[j] = fmaf(wa, e, S[j]);
        S1[j] = fmaf(wav, e, S1[j]);
        pk[j & 1] = fmaf(ure[8 * b + j], e, pk[j & 1]);
      });
      s_pkl[k * BLOCK + t] = before + (pk[0] + pk[1]);
    }
    static_for<0, 8>([&](auto jj) {
      constexpr int j = decltype(jj)::value;
      constexpr int m = 8 * b + j;
      const float si = S[j] * uim[m], r1 = S1[j] * ure[m];
      if constexpr (D * m == W / 2) {
        const float om = h ? -0.5f + hW : 0.5f;
        ax = fmaf(nu, si, ax);
        ay = fmaf(om, si, ay);
        a11 = fmaf(nu * nu, r1, a11);
        a12 = fmaf(nu * om, r1, a12);
        a22 = fmaf(om * om, r1, a22);
      } else {  // omega = c + h/W, nu the lane's: the moments of si and r1 in c
        constexpr float cm = (D * m < W / 2) ? (float)(D * m) * (1.f / W) : (float)(D * m - W) * (1.f / W);
        m_si += si;
        m_csi = fmaf(cm, si, m_csi);
        m_r += r1;
        m_cr = fmaf(cm, r1, m_cr);
        m_ccr = fmaf(cm * cm, r1, m_ccr);
      }
    });
    // Materialise the block's contribution here, so the compiler does not sink
    // the accumulation (and keep this block's sums alive) past later blocks.
    asm volatile("" : "+v"(m_si), "+v"(m_csi), "+v"(m_r), "+v"(m_cr), "+v"(m_ccr));
  });
  ax = fmaf(nu, m_si, ax);
  ay += fmaf(hW, m_si, m_csi);
  a11 = fmaf(nu * nu, m_r, a11);
  a12 = fmaf(nu, fmaf(hW, m_r, m_cr), a12);
  a22 += fmaf(hW, fmaf(hW, m_r, 2.f * m_cr), m_ccr);

  // ------------------------------------------------------------ sums
  ax = lane_sum<64>(ax);
  ay = lane_sum<64>(ay);
  a11 = lane_sum<64>(a11);
  a12 = lane_sum<64>(a12);
  a22 = lane_sum<64>(a22);
  if (lane == 0) {
    s_red[0][wv] = ax;
    s_red[1][wv] = ay;
    s_red[2][wv] = a11;
    s_red[3][wv] = a12;
    s_red[4][wv] = a22;
  }
  __syncthreads();
  // wavefront k sums component k's partials: 16 per lane, then the lanes
  static_assert(NWAVE == kKmax, "one wavefront per component");
  if (wv < G.K) {
    float a[NWAVE];
    static_for<0, NWAVE>([&](auto ii) { a[decltype(ii)::value] = s_pkl[wv * BLOCK + 64 * decltype(ii)::value + lane]; });
    static_for<0, 4>([&](auto ss) {  // as a tree
      constexpr int o = NWAVE >> (1 + decltype(ss)::value);
      static_for<0, o>([&](auto ii) { a[decltype(ii)::value] += a[decltype(ii)::value + o]; });
    });
    const float acc = lane_sum<64>(a[0]);
    if (lane == 0) s_pk[wv] = acc;
  }
  // the real-space sums over the wavefronts, one (component, sum) per thread
  if (t < kKmax * 6) {
    const int k = t / 6, i = t % 6;
    float acc = 0.f;
    if ((rmask >> k) & 1u)
      static_for<0, NWAVE>([&](auto ww) { acc += s_rw[k][decltype(ww)::value][i]; });
    s_racc[t] = acc;
  }
  __syncthreads();
  if (wv == 0) {  // lanes 0..15 take one component each; lane 0 finishes
    const RenderArgs& pc = kernel_args_renewed<RenderArgs>();
    Galaxy Gc = load_galaxy<W>(pc, stamp);  // reloaded: keeps G's registers free in the loops above
    make_uniform(Gc);
    CompTerms ct = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    float sum[5];
    static_for<0, 5>([&](auto ii) {
      constexpr int i = decltype(ii)::value;
      sum[i] = lane_sum<16>(s_red[i][lane & (NWAVE - 1)]);
    });
    if (lane < kKmax)
      ct = bwd_component_terms<W>(pc, Gc, lane, rmask, s_pk, 1, s_racc, amp_part + stamp * kKmax);
    ct = sum16(ct);
    if (lane == 0)
      bwd_chain_finish<W>(pc, Gc, stamp, sum[0], sum[1], sum[2], sum[3], sum[4], ct, grad_params);
  }
}

hipError_t launch_bwd_w256(const RenderArgs& args, const float* gout, float* grad_params, float* amp_part,
                           hipStream_t stream) {
  constexpr int64_t kChunk = (int64_t)1 << 30;  // workgroups per launch
  RenderArgs p = args;
  for (int64_t done = 0; done < args.n; done += kChunk) {
    const int64_t chunk = std::min<int64_t>(args.n - done, kChunk);
    p.x = args.x + done;
    p.y = args.y + done;
    p.flux = args.flux + done;
    p.r_e = args.r_e + done;
    p.e1 = args.e1 + done;
    p.e2 = args.e2 + done;
    p.mix_id = args.mix_id ? args.mix_id + done : nullptr;
    p.n = chunk;
    hipLaunchKernelGGL(render_bwd_w256_kernel, dim3((unsigned)chunk), dim3(w256::BLOCK), 0, stream, p,
                       gout + done * (int64_t)w256::W * w256::W, grad_params + done * 6, amp_part + done * kKmax);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace gfc
