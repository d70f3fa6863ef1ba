// Adjoint of the forward render for W = 64, 128 and 256 (Lang 2020, Section 2,
// steps 3-8, differentiated); the sums are those of the W <= 32 adjoint.
//
// W = 32 D.  One workgroup of 16 D^2 threads per stamp (1, 4 or 16
// wavefronts), 32 bins per thread, the half spectrum of the upstream gradient
// g kept on the chip: the stages of the 256 x 256 forward kernel run
// backwards.  g is read once and nothing else moves through memory.
//
//  load           D lanes per row read 32 pixels each of two rows, W / 2
//                 apart, and accumulate the real-space sums.
//  row phase      per half (W / 2 rows): the row as 16 D packed complex
//                 values: a radix-8 stage on the lane, an exchange between the
//                 row's lanes, 2 D-point FFTs.
//  column read    lane (c, h) reads its 16 rows of the half, of columns c and
//                 W / 2 - c, and forms the row's real-input spectrum on the
//                 way.
//  column DFT     the radix-D stage over the rows 32 apart, an exchange
//                 between the D lanes of a column, a 32-point FFT: lane (c, h)
//                 ends with the bins k_y = D m + h of column c.
//  bins           U0 per bin; the component loop in blocks of eight bins,
//                 negligible blocks skipped as in the 256 x 256 forward.
//  sums           fixed-order reductions, then the chain rule on the first
//                 wavefront.
// The integer centre enters the phases (shift_phase), so g is never
// rolled.
//
// Its time goes to VALU work (4,450-4,900 instructions per wavefront and
// stamp; a wavefront waits for 31% of its time at 64, 35% at 128), at 256 also
// to the barriers: there the LDS holds one stamp per CU.  32 bins per thread
// keep it within 128 registers, and half a stamp at a time within 10 KB of LDS
// per wavefront, so four wavefronts per SIMD are resident.  Whole calls, r_e
// 0.5..8 px, 8 components: 20,000 stamps of 64 x 64 in 172 us, 5,000 of 128 x
// 128 in 165 us (193 us with r_e 10..60 px), 500 of 256 x 256 with r_e 10..60
// px in 105 us.  One lane per row and two per column with the whole g tile in
// LDS (two wavefronts per SIMD) took 199 us at 64 and 315 us (440 us) at 128;
// a slab in device memory took 353 us at 256.
#include "bwd_common.hpp"
#include "gfc_device.hpp"
#include "gfc_internal.hpp"
#include "gfc_launch.hpp"
#include "w256_common.hpp"

namespace gfc {

// The upstream gradient is only promised to be aligned as floats are.
typedef const __attribute__((address_space(1))) v4f_any* GlobalF4;

namespace {

template <int D_>
struct Split {
  static constexpr int D = D_;            // lanes per row and per column
  static constexpr int W = 32 * D;
  static constexpr int NC = W / 2;        // packed columns
  static constexpr int M = 32;            // bins per lane
  static constexpr int K4 = M / D;        // rows of a lane's column that lie within 32 of each other
  static constexpr int BLOCK = NC * D;
  static constexpr int NWAVE = BLOCK / 64;
  static constexpr int HROWS = W / 2;
  static constexpr int LPW = 64 / D;      // rows (columns) that a wavefront holds at a time
  static constexpr int CL = 8 / D;        // residues mod 8 of k_x that a lane takes in the row phase
  static constexpr int N1 = 2 * D;        // length of its FFTs there
  // LDS strides (float2), for a 64-bit access served 16 lanes at a time: the
  // 16 addresses differ mod 16.  At D = 8, 16 lanes are two columns (rows)
  // of eight lanes each; at D = 2 and 4 the lanes of a wavefront run over
  // its columns (rows) first, so they are 16 columns (rows) and the strides
  // between rows are odd.
  static constexpr int TS = D == 8 ? w256::TS : NC + 1;   // rows of the half buffer
  static constexpr int RA = D == 8 ? 9 : 8;               // row exchange: entry (i, residue) at RA i + residue
  static constexpr int RXS = D == 8 ? w256::RXS : 8 * D + 1;
  static constexpr int KC = D == 8 ? 1 : 2;               // rows k exchanged at a time in a column
  static constexpr int CXS = D == 8 ? w256::CXS : (D == 4 ? 33 : 9);  // column exchange: slot of a column
  static constexpr int CA = D == 8 ? 9 : D;               // entry (i, g) of row k at CA i + g + k D D
  static constexpr int BUF = HROWS * TS;
  // after the column exchange: phases, packed Nyquist column and twins
  // behind its slots, later the p_k partials
  static constexpr int PKS = BLOCK + BLOCK / kKmax;       // floats per component of the p_k partials
  static constexpr int PY = NWAVE * LPW * CXS, NYQ = PY + W + 2;
  // the twins lie behind the partials too: they are read while other lanes may
  // already write partials
  static constexpr int UX = std::max(NYQ + W, kKmax * PKS / 2);
  static_assert(UX + NC <= BUF && kKmax * PKS <= 2 * UX, "the overlays fit in the half buffer");
  static_assert(LPW * RXS <= LPW * TS, "a row exchange slice lies in its wavefront's rows");
  static constexpr int TWC = 33, TWR = N1 + 1;            // rows of the twiddle tables
};

}  // namespace

// Four wavefronts per SIMD: 128 VGPRs.
template <int D>
__global__ void __launch_bounds__(Split<D>::BLOCK) __attribute__((amdgpu_waves_per_eu(4)))
render_bwd_split_kernel(RenderArgs p, const float* __restrict__ gout, float* __restrict__ grad_params,
                        float* __restrict__ amp_part) {
  using C = Split<D>;
  constexpr int W = C::W, NC = C::NC, M = C::M, BLOCK = C::BLOCK, NWAVE = C::NWAVE, HROWS = C::HROWS, LPW = C::LPW;
  constexpr int TS = C::TS, TWC = C::TWC, TWR = C::TWR, K4 = C::K4, CL = C::CL, N1 = C::N1;
  // rows of a half [HROWS][TS] and the exchanges' slices, then the overlays,
  // then the p_k partials
  __shared__ float2 s_buf[C::BUF];
  __shared__ float2 s_twc[D * TWC];     // s_twc[h][D k + g] = w^(g (D k + h)), w = exp(2 pi i / W)
  __shared__ float2 s_twr[8 * TWR];     // s_twr[rho][n1] = exp(-2 pi i rho n1 / NC)
  __shared__ float4 s_cmp[kKmax];       // per component: v, w A, w A v, w (zero past the table's K)
  __shared__ float s_rw[kKmax][NWAVE][6];  // real-space sums per wavefront
  __shared__ float s_red[5][NWAVE];
  __shared__ float s_pk[kKmax];
  float2* s_py = s_buf + C::PY;         // y phase of row k_y; [W]: that of omega = -1/2
  float2* s_nyq = s_buf + C::NYQ;
  float2* s_ux = s_buf + C::UX;         // U0 of the Nyquist row's omega = -1/2 twin, per column

  const int t = threadIdx.x;
  const int lane = t & 63;
  const int wv = __builtin_amdgcn_readfirstlane(t >> 6);  // wavefront index (scalar)
  const int64_t stamp = blockIdx.x;  // the launcher sizes each grid to its chunk

  // Row phase: rows LPW wv + yl and W / 2 further down, lane r of the row:
  // pixels x = 4 r + 4 D q + 0..3, as z[n] = g[2n] + i g[2n+1] for n = 2 r + kk
  // + 2 D q in zq[half][kk][q].  Both rows are in flight while the galaxy is
  // formed.
  float2 zq[2][2][8];
  {
    const int yl = lane % LPW, r = lane / LPW;
    GlobalF4 row = (GlobalF4)(gout + stamp * (int64_t)(W * W) + (LPW * wv + yl) * W) + r;
    static_for<0, 2>([&](auto hh) {
      constexpr int half = decltype(hh)::value;
      static_for<0, 8>([&](auto qq) {
        constexpr int q = decltype(qq)::value;
        const v4f_any v = row[half * (HROWS * W / 4) + D * q];
        zq[half][0][q] = make_float2(v.x, v.y);
        zq[half][1][q] = make_float2(v.z, v.w);
      });
    });
  }
  __builtin_amdgcn_sched_barrier(0);
  Galaxy G = load_galaxy<W>(p, stamp);
  make_uniform(G);
  const float trB = G.b11 + G.b22;

  for (int i = t; i < W; i += BLOCK) {  // i = (row h, D k + g)
    const int hh = i / 32, kg = i % 32;
    s_twc[hh * TWC + kg] = twiddle_rt<+1, W>((kg % D) * (D * (kg / D) + hh));
  }
  for (int i = t; i < 8 * N1; i += BLOCK) s_twr[(i / N1) * TWR + i % N1] = twiddle_rt<-1, NC>((i / N1) * (i % N1));
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
  // c0 + c2 zx^2.  zx0 is zx at column W / 2 (plus the lane's 4 r): near most
  // galaxies' centres, where it is small and rounds by little.
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
      const float dy = (float)(half * HROWS + LPW * wv + lane % LPW) - G.y0 - p.pg[1];
      const float al = dy * rsyy;
      const float zx0 = fmaf(ixx, (float)(4 * (lane / LPW) + W / 2) - G.x0 - p.pg[0], ixy * dy);
      const float c0 = fmaf(kHalfLog2e * al, dy, lnrm);
      float m0 = 0.f, m1 = 0.f, m2 = 0.f;
      static_for<0, 8>([&](auto qq) {
        constexpr int q = decltype(qq)::value;
        static_for<0, 4>([&](auto ii) {
          constexpr int i = decltype(ii)::value;
          const float2 z = zq[half][i / 2][q];
          const float zx = fmaf(ixx, (float)(4 * D * q + i - W / 2), zx0);
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
  // Column phase: lane (c, h) takes column c, rows y and bins k_y = h (mod D).
  const int c = D == 8 ? t >> 3 : wv * LPW + lane % LPW;
  const int h = D == 8 ? t & 7 : lane / LPW;
  const float nu = (float)c * (1.f / W);
  // The real-input split, the column's phase and its weight are applied while
  // reading the transformed rows.  The packed column NC never needs to be taken
  // out of column 0 again: every sum over the bins below is the real part of a
  // sum of terms that are Hermitian in k_y on column 0 (a real column's
  // transform times the PSF's, the phases and real even factors), to which i
  // times another such column adds nothing.
  const ColumnSplit split = column_split<W>(G.fx, G.nx, c, twiddle_rt<-1, W>(c));
  float2 X4[K4][D];                         // row spectra: X4[k][q] of row D k + h + 32 q, column c
  static_for<0, 2>([&](auto hh) {
    constexpr int half = decltype(hh)::value;
    int ln = lane;
    asm volatile("" : "+v"(ln));  // recomputed per half, not held across it
    const int yl = ln % LPW, r = ln / LPW;
    const int yloc = LPW * wv + yl;
    // Z[8m + rho] = sum_{n1} w2D^{-n1 m} (wNC^{-n1 rho} A_{n1}[rho]) with
    // A_{n1}[rho] = sum_q w8^{-q rho} z[n1 + 2 D q]: lane r has n1 = 2 r + kk
    // and hands entry rho to lane rho mod D of the row.
    if constexpr (half == 1) __syncthreads();  // the first half has been read from s_buf
    float2 R[CL][N1];
    {
      float2* rxb = s_buf + wv * (LPW * TS) + yl * C::RXS;  // this row's slot, in the wavefront's own rows
      static_for<0, 2>([&](auto kk) {
        constexpr int k = decltype(kk)::value;
        fft<8, -1>(zq[half][k]);
        static_for<0, 8>([&](auto gg) {
          constexpr int g = decltype(gg)::value;
          rxb[C::RA * r + g] = zq[half][k][g];
        });
        wave_lds_sync();
        static_for<0, D>([&](auto ii) {
          static_for<0, CL>([&](auto cc) {
            constexpr int i = decltype(ii)::value, cl = decltype(cc)::value;
            R[cl][2 * i + k] = rxb[C::RA * i + r + D * cl];
          });
        });
        wave_lds_sync();  // read before the slot is overwritten
      });
    }
    float2* row = s_buf + yloc * TS;
    static_for<0, CL>([&](auto cc) {
      constexpr int cl = decltype(cc)::value;
      const float2* twr = s_twr + (r + D * cl) * TWR;
      static_for<1, N1>([&](auto nn) {
        constexpr int n1 = decltype(nn)::value;
        R[cl][n1] = cmul(R[cl][n1], twr[n1]);
        if constexpr (n1 % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // bounds the loads in flight
      });
      fft<N1, -1>(R[cl]);
    });
    static_for<0, CL>([&](auto cc) {
      static_for<0, N1>([&](auto mm) {
        constexpr int cl = decltype(cc)::value, m = decltype(mm)::value;
        row[8 * m + D * cl + r] = R[cl][m];
      });
    });
    __syncthreads();
    {
      const int cb = (NC - c) & (NC - 1);
      static_for<0, K4>([&](auto kk) {
        constexpr int k = decltype(kk)::value;
        static_for<0, D / 2>([&](auto qq) {
          constexpr int q = decltype(qq)::value;
          const float2* rw = s_buf + (D * k + h + 32 * q) * TS;
          X4[k][(D / 2) * half + q] = split.at(rw[c], rw[cb]);
        });
        if constexpr ((k + 1) * D % 8 == 0) __builtin_amdgcn_sched_barrier(0);
      });
    }
  });
  __syncthreads();  // the second half has been read; s_buf takes the column exchange

  // ------------------------------------------------------------ column DFT
  // G[D m + g] = sum_j w32^{-m j} w^{-g j} sum_q wD^{-g q} X[j + 32 q], j = D k + h
  float2 Gk[M];  // G[k_y = D m + h][c] conj(x phase) weight  (c = 0: packed with column NC)
  {
    float2* cxb = s_buf + (D == 8 ? wv * 8 + (lane >> 3) : c) * C::CXS;  // this column's slot
    const float2* twh = s_twc + h * TWC;
    static_for<0, K4 / C::KC>([&](auto kc) {
      constexpr int k0 = decltype(kc)::value * C::KC;
      __builtin_amdgcn_sched_barrier(0);  // one chunk's twiddle loads in flight at a time
      static_for<0, C::KC>([&](auto kk) {
        constexpr int k = k0 + decltype(kk)::value;
        fft<D, -1>(X4[k]);
        static_for<0, D>([&](auto gg) {
          constexpr int g = decltype(gg)::value;
          if constexpr (g > 0) X4[k][g] = cmulc(X4[k][g], twh[D * k + g]);
          cxb[(k - k0) * D * D + C::CA * h + g] = X4[k][g];
        });
      });
      wave_lds_sync();
      static_for<0, C::KC>([&](auto kk) {
        constexpr int k = k0 + decltype(kk)::value;
        static_for<0, D>([&](auto ii) {
          constexpr int i = decltype(ii)::value;
          Gk[D * k + i] = cxb[(k - k0) * D * D + C::CA * i + h];
        });
      });
      wave_lds_sync();  // read before the next chunk overwrites the slot
    });
    fft<M, -1>(Gk);
  }

  // ------------------------------------------------------------ phases, Nyquist column
  const float hW = (float)h * (1.f / W);
  // Threads t < W also take row t of column k_x = W / 2 (nu = +-1/2), threads
  // t < NC the omega = -1/2 twin of the Nyquist row in column t.
  const bool nyq = t < W, twin = t < NC;
  const float omN = (t < W / 2) ? (float)t * (1.f / W) : (t == W / 2 ? 0.5f : (float)(t - W) * (1.f / W));
  float2 py = make_float2(1.f, 0.f);
  if (nyq) {
    float sy, cy;
    shift_phase<W>(G.fy, G.ny, t <= W / 2 ? t : t - W, &sy, &cy);
    py = make_float2(cy, sy);
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
  // ------------------------------------------------------------ U0
  GlobalF2 psfm = (GlobalF2)p.psf_main;
  float ure[M], uim[M];
  {
    // the cache's lane order: bin (k_y, c) at (k_y / P) (P NC) + P c + k_y mod P,
    // P = 2 up to 128 x 128, 4 at 256 x 256
    constexpr int P2 = D == 8 ? 4 : 2;
    const int pidx0 = (h / P2) * (P2 * NC) + P2 * c + h % P2;
    static_for<0, M>([&](auto mm) {
      constexpr int m = decltype(mm)::value;
      const float2 P = ld2(psfm, pidx0 + m * (D * NC));
      const float2 gp2 = cmulc(P, Gk[m]);
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
    const float2 d = csub(za, zb);  // of the packed column G0 + i GN, both Hermitian in k_y
    const float2 GN = make_float2(0.5f * d.y, -0.5f * d.x);  // (za - conj zb) / (2 i), weight as column 0
    // weight 1/2 of each of nu = +-1/2; the integer x shift at k_x = W / 2 is
    // exp(-i pi n_x) = +-1
    const float sgn = (G.nx & 1) ? -0.5f : 0.5f;
    const float2 gamN = cscale(cmulc(ld2((GlobalF2)p.psf_nyq, t), GN), sgn);
    float sxh, cxh;
    sincospi_poly(-G.fx, &sxh, &cxh);
    const bool corner = (t == W / 2);
    const float2 pyA = corner ? cscale(py, 0.5f) : py;
    const float2 pyB = corner ? cscale(cconj(py), 0.5f) : make_float2(0.f, 0.f);
    const float2 eM = make_float2(cxh, sxh), eP = make_float2(cxh, -sxh);
    const float2 u1 = cmul(cmul(gamN, eM), pyA), u2 = cmul(cmul(gamN, eP), pyA);
    const float2 u3 = cmul(cmul(gamN, eM), pyB), u4 = cmul(cmul(gamN, eP), pyB);
    // corner twins folded into their partners (the transform is even; see the
    // W <= 32 adjoint)
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
  // per-lane p_k partials [kKmax][PKS]; the row stride keeps the reduction below
  // free of bank conflicts
  constexpr int LPK = BLOCK / kKmax, PKS = C::PKS;
  float* s_pkl = reinterpret_cast<float*>(s_buf);
  for (int k = 0; k < G.K; ++k) s_pkl[k * PKS + t] = 0.f;
  // Lane k (mod 16) holds component k's constants; the loops take them by lane
  // reads, over the components of a mask: those with w > 0 (else p_k is only
  // ever multiplied by w or by the ramp slope, both zero) that are not
  // negligible: their variance is below vmax = kSkipLog2 / (lambda r^2), r^2
  // the least nu^2 + omega^2 of the points.
  const float4 cmp = s_cmp[lane % kKmax];
  const float lamq = -kQ * shape_min_eig(G);
  auto active = [&](float r2) {
    const float vmax = kSkipLog2 * __builtin_amdgcn_rcpf(lamq * r2);  // rcp(0) = +inf
    return (unsigned)__ballot(cmp.w != 0.f && !(cmp.x >= vmax)) & ((1u << kKmax) - 1u);
  };
  float ax = 0.f, ay = 0.f, a11 = 0.f, a12 = 0.f, a22 = 0.f;
  // the irregular points
  if (nyq) {
    const float nt = (float)t * (1.f / W);
    const float n3[3] = {0.5f, -0.5f, nt}, o3[3] = {omN, omN, -0.5f};
    const float qa = kQ * G.b11 * 0.25f, qb = kQ * G.b12, qd = kQ * G.b22;
    const float g3[3] = {fmaf(omN, fmaf(qd, omN, qb), qa), fmaf(omN, fmaf(qd, omN, -qb), qa),
                         kQ * fmaf(nt, fmaf(G.b11, nt, -G.b12), 0.25f * G.b22)};
    float S[3] = {0.f, 0.f, 0.f}, S1[3] = {0.f, 0.f, 0.f};
    for (unsigned mk = active(0.25f); mk != 0; mk &= mk - 1) {
      const int k = __builtin_ctz(mk);
      const float v = lane_f(cmp.x, k), wa = lane_f(cmp.y, k), wav = lane_f(cmp.z, k);
      float pk = 0.f;
      static_for<0, 3>([&](auto jj) {
        constexpr int j = decltype(jj)::value;
        const float e = __builtin_amdgcn_exp2f(v * g3[j]);
        S[j] = fmaf(wa, e, S[j]);
        S1[j] = fmaf(wav, e, S1[j]);
        pk = fmaf(ure3[j], e, pk);
      });
      s_pkl[k * PKS + t] = pk;
    }
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
  // The regular bins, eight at a time (k_y in [W b / 4, W (b + 1) / 4)): omega =
  // c_m + h/W with a compile-time c_m, the quadratic expanded about h/W.
  // nu^2 + omega^2 >= r2[b] in block b, nu of the wavefront's first column.
  float m_si = 0.f, m_csi = 0.f, m_r = 0.f, m_cr = 0.f, m_ccr = 0.f;
  const float g2 = kQ * G.b22, g1 = 2.f * kQ * G.b12 * nu;
  const float e0 = fmaf(hW, fmaf(g2, hW, g1), kQ * G.b11 * nu * nu);
  const float e1 = fmaf(2.f * g2, hW, g1);
  constexpr float kW1 = 1.f / W;
  const float nlo = (float)((D == 8 ? 8 : LPW) * wv) * kW1;
  const float r2[4] = {nlo * nlo, fmaf(nlo, nlo, 0.0625f), fmaf(nlo, nlo, (0.25f + kW1) * (0.25f + kW1)),
                       fmaf(nlo, nlo, kW1 * kW1)};
  static_for<0, M / 8>([&](auto bb) {
    constexpr int b = decltype(bb)::value;
    float gq[8], S[8], S1[8];
    static_for<0, 8>([&](auto jj) {
      constexpr int j = decltype(jj)::value;
      constexpr int m = 8 * b + j;
      if constexpr (D * m == W / 2) {  // k_y = W / 2 + h: the Nyquist row (+1/2) for h = 0
        const float om = h ? -0.5f + hW : 0.5f;
        gq[j] = fmaf(om, fmaf(g2, om, g1), kQ * G.b11 * nu * nu);
      } else {
        constexpr float cm = (D * m < W / 2) ? (float)(D * m) * (1.f / W) : (float)(D * m - W) * (1.f / W);
        gq[j] = fmaf(cm, fmaf(cm, g2, e1), e0);
      }
    });
    unsigned mk = active(r2[b]);
    {  // the first component initialises the sums (all of them zero with none active: w = 0)
      const int k = __builtin_ctz(mk | (1u << (kKmax - 1)));
      const float before = s_pkl[k * PKS + t];
      const float v = lane_f(cmp.x, k), wa = lane_f(cmp.y, k), wav = lane_f(cmp.z, k);
      float pk[2] = {0.f, 0.f};
      static_for<0, 8>([&](auto jj) {
        constexpr int j = decltype(jj)::value;
        const float e = __builtin_amdgcn_exp2f(v * gq[j]);
        S[j] = wa * e;
        S1[j] = wav * e;
        pk[j & 1] = fmaf(ure[8 * b + j], e, pk[j & 1]);
      });
      s_pkl[k * PKS + t] = before + (pk[0] + pk[1]);
    }
    for (mk &= mk - 1; mk != 0; mk &= mk - 1) {
      const int k = __builtin_ctz(mk);
      const float before = s_pkl[k * PKS + t];  // used after the exponentials
      const float v = lane_f(cmp.x, k), wa = lane_f(cmp.y, k), wav = lane_f(cmp.z, k);
      float pk[2] = {0.f, 0.f};  // two chains: a smaller rounding error than one
      static_for<0, 8>([&](auto jj) {
        constexpr int j = decltype(jj)::value;
        const float e = __builtin_amdgcn_exp2f(v * gq[j]);
        S[j] = fmaf(wa, e, S[j]);
        S1[j] = fmaf(wav, e, S1[j]);
        pk[j & 1] = fmaf(ure[8 * b + j], e, pk[j & 1]);
      });
      s_pkl[k * PKS + t] = before + (pk[0] + pk[1]);
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
  // LPK lanes per component, lane i taking the partials i, i + LPK, ... as a
  // tree, then the lanes
  {
    const int k = t / LPK, i = t % LPK;
    float a[16];
    static_for<0, 16>([&](auto ee) { a[decltype(ee)::value] = s_pkl[k * PKS + i + decltype(ee)::value * LPK]; });
    static_for<0, 4>([&](auto ss) {
      constexpr int o = 8 >> decltype(ss)::value;
      static_for<0, o>([&](auto ii) { a[decltype(ii)::value] += a[decltype(ii)::value + o]; });
    });
    const float acc = lane_sum<LPK>(a[0]);
    if (i == 0) s_pk[k] = acc;
  }
  // the real-space sums over the wavefronts, one (component, sum) per thread,
  // left in the first wavefront's place
  for (int i = t; i < kKmax * 6; i += BLOCK) {
    const int k = i / 6, j = i % 6;
    if ((rmask >> k) & 1u) {
      float acc = s_rw[k][0][j];
      static_for<1, NWAVE>([&](auto ww) { acc += s_rw[k][decltype(ww)::value][j]; });
      s_rw[k][0][j] = acc;
    }
  }
  __syncthreads();
  if (wv == 0) {  // lanes 0..15 take one component each; lane 0 finishes
    CompTerms ct = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    float sum[5];
    static_for<0, 5>([&](auto ii) {
      constexpr int i = decltype(ii)::value;
      sum[i] = s_red[i][0];
      if constexpr (NWAVE == 16) sum[i] = lane_sum<16>(s_red[i][lane & 15]);
      else static_for<1, NWAVE>([&](auto ww) { sum[i] += s_red[i][decltype(ww)::value]; });
    });
    if (lane < kKmax)
      ct = bwd_component_terms<W>(p, G, lane, rmask, s_pk, 1, &s_rw[0][0][0], 6 * NWAVE, amp_part + stamp * kKmax);
    ct = sum16(ct);
    if (lane == 0)
      bwd_chain_finish<W>(p, G, stamp, sum[0], sum[1], sum[2], sum[3], sum[4], ct, grad_params);
  }
}

template <int D>
static hipError_t launch_bwd_split(const RenderArgs& args, const float* gout, float* grad_params, float* amp_part,
                                   hipStream_t stream) {
  using C = Split<D>;
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
    hipLaunchKernelGGL(render_bwd_split_kernel<D>, dim3((unsigned)chunk), dim3(C::BLOCK), 0, stream, p,
                       gout + done * (int64_t)C::W * C::W, grad_params + done * 6, amp_part + done * kKmax);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_bwd_split(const RenderArgs& args, int W, const float* gout, float* grad_params, float* amp_part,
                            hipStream_t stream) {
  switch (W) {
    case 64: return launch_bwd_split<2>(args, gout, grad_params, amp_part, stream);
    case 128: return launch_bwd_split<4>(args, gout, grad_params, amp_part, stream);
    case 256: return launch_bwd_split<8>(args, gout, grad_params, amp_part, stream);
  }
  return hipErrorInvalidValue;
}

}  // namespace gfc
