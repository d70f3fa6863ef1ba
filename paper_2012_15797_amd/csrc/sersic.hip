// General-Sérsic and composite (bulge + disk) galaxies (Lang 2020: Section 1
// on the profile family and its bulge-disk combinations; the closing
// discussion on interpolating mixture parameters between Sérsic indices).
//
// Both reduce to the ordinary render with one mixture per galaxy, which the
// forward kernels form in the lanes that hold the components (make_profile,
// component_mix): a galaxy's one or two profile parameters are read with its
// others.  Tables of 136 bytes per galaxy, written by a launch of their own
// before the render, cost that launch and an allocation: 3 Sersic stamps of
// 64x64 took 33 us, now 11; 20,000 took 104 us, now 98; 20,000 composites 115
// us, now 107.  An invalid profile parameter makes the galaxy invalid: a NaN
// stamp, counted.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "gfc_internal.hpp"
#include "gfc_launch.hpp"

struct gfc_sersic {
  gfc_ctx* ctx = nullptr;
  int S = 0, K = 0;
  float v2 = 0.f;           // the largest of the grid indices' second smallest variances
  float* d_grid = nullptr;  // [S] indices, then amp [S][K], then var [S][K]
};

namespace gfc {
namespace {

// Common tail: validate, fill the cache and launch the render with the
// galaxies' own mixtures as `profile` sets them up.
template <typename SetProfile>
gfc_status render_profiles(gfc_ctx* ctx, gfc_psf* psf, const gfc_mix* mix_like, const gfc_galaxies* gal, int64_t n,
                           int W, unsigned flags, float* out, hipStream_t s, SetProfile profile) {
  // (more stamps than any device's memory holds: 2 TB at 16 x 16)
  if (n > (int64_t)INT32_MAX) return fail(GFC_EINVAL, "at most 2^31 - 1 galaxies per call with per-galaxy mixtures");
  RenderArgs a;
  gfc_status st = fill_render_args(ctx, psf, mix_like, gal, n, W, flags, &a);
  if (st != GFC_OK) return st;
  if (n == 0) return GFC_OK;
  if (!out) return fail(GFC_EINVAL, "null output");
  DeviceGuard guard(ctx->device);
  const PsfSpectrum* spec = nullptr;
  st = psf_cache(psf, W, s, &spec);
  if (st != GFC_OK) return st;
  attach_spectrum(&a, spec);
  profile(&a);
  a.out = out;
  return render_launch(a, W, s);
}

}  // namespace
}  // namespace gfc

using namespace gfc;

extern "C" {

gfc_status gfc_sersic_create(gfc_ctx* ctx, int S, const float* n_grid, int K, const float* amp, const float* var,
                             gfc_sersic** out) {
  if (!ctx || !n_grid || !amp || !var || !out) return fail(GFC_EINVAL, "null argument");
  *out = nullptr;
  if (S < 2 || S > 256) return fail(GFC_EINVAL, "a Sersic family needs 2..256 grid indices");
  if (K < 1 || K > kKmax) return fail(GFC_EINVAL, "a Sersic family needs 1..16 components");
  for (int i = 0; i < S; ++i) {
    if (!std::isfinite(n_grid[i]) || (i > 0 && !(n_grid[i] > n_grid[i - 1])))
      return fail(GFC_EINVAL, "Sersic grid indices must be finite and strictly increasing");
    for (int k = 0; k < K; ++k) {
      if (!std::isfinite(amp[i * K + k])) return fail(GFC_EINVAL, "non-finite Sersic amplitude");
      if (!(var[i * K + k] > 0.f) || !std::isfinite(var[i * K + k]))
        return fail(GFC_EINVAL, "Sersic variances must be positive and finite");
    }
  }
  DeviceGuard guard(ctx->device);
  auto* f = new (std::nothrow) gfc_sersic();
  if (!f) return fail(GFC_ENOMEM, "allocation failed");
  f->ctx = ctx;
  f->S = S;
  f->K = K;
  for (int i = 0; i < S; ++i) {
    float low[2];
    two_smallest(var + (size_t)i * K, K, low);
    f->v2 = std::max(f->v2, low[1]);
  }
  std::vector<float> h((size_t)S + 2 * (size_t)S * K);
  std::memcpy(h.data(), n_grid, S * sizeof(float));
  std::memcpy(h.data() + S, amp, (size_t)S * K * sizeof(float));
  std::memcpy(h.data() + S + (size_t)S * K, var, (size_t)S * K * sizeof(float));
  hipError_t e = hipMalloc(&f->d_grid, h.size() * sizeof(float));
  if (e == hipSuccess) e = hipMemcpy(f->d_grid, h.data(), h.size() * sizeof(float), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    hipFree(f->d_grid);
    delete f;
    return hip_fail(e, "Sersic family upload");
  }
  ctx->n_objects++;
  *out = f;
  return GFC_OK;
}

gfc_status gfc_sersic_destroy(gfc_sersic* f) {
  if (!f) return fail(GFC_EINVAL, "null Sersic family");
  DeviceGuard guard(f->ctx->device);
  hipDeviceSynchronize();
  hipFree(f->d_grid);
  f->ctx->n_objects--;
  delete f;
  return GFC_OK;
}

gfc_status gfc_render_stamps_sersic(gfc_ctx* ctx, gfc_psf* psf, const gfc_sersic* fam, const gfc_galaxies* gal,
                                    const float* sersic_n, int64_t n, int W, unsigned flags, float* out,
                                    void* hip_stream) {
  if (!fam || !gal) return fail(GFC_EINVAL, "null Sersic family or galaxy block");
  if (fam->ctx != ctx) return fail(GFC_EINVAL, "Sersic family belongs to another context");
  if (n > 0 && !sersic_n) return fail(GFC_EINVAL, "null Sersic index array");
  if (gal->mix_id) return fail(GFC_EINVAL, "mix_id is not used with a Sersic family (pass NULL)");
  // a stand-in for the mixture argument: only its context is read before the tables are replaced
  gfc_mix shell;
  shell.ctx = ctx;
  shell.n_tables = 1;
  shell.kmax = fam->K;
  shell.v2 = fam->v2;
  hipStream_t s = (hipStream_t)hip_stream;
  const int S = fam->S, K = fam->K;
  return render_profiles(ctx, psf, &shell, gal, n, W, flags, out, s, [&](RenderArgs* a) {
    a->prof = kProfSersic;
    a->prof_a = sersic_n;
    a->prof_grid = fam->d_grid;
    a->prof_S = S;
    a->prof_k1 = K;
    a->amp = fam->d_grid + S;
    a->var = fam->d_grid + S + (size_t)S * K;
  });
}

gfc_status gfc_render_stamps_composite(gfc_ctx* ctx, gfc_psf* psf, const gfc_mix* mix, int disk_table,
                                       int bulge_table, const gfc_galaxies* gal, const float* bulge_frac,
                                       const float* bulge_rho, int64_t n, int W, unsigned flags, float* out,
                                       void* hip_stream) {
  if (!mix || !gal) return fail(GFC_EINVAL, "null mixture or galaxy block");
  if (disk_table < 0 || disk_table >= mix->n_tables || bulge_table < 0 || bulge_table >= mix->n_tables)
    return fail(GFC_EINVAL, "disk or bulge table out of range");
  if (n > 0 && (!bulge_frac || !bulge_rho)) return fail(GFC_EINVAL, "null bulge fraction or radius ratio");
  if (gal->mix_id) return fail(GFC_EINVAL, "mix_id is not used with a composite (pass NULL)");
  const int Kd = mix->K[disk_table], Kb = mix->K[bulge_table];
  if (Kd + Kb > kKmax) return fail(GFC_EINVAL, "disk and bulge together exceed 16 components");
  hipStream_t s = (hipStream_t)hip_stream;
  return render_profiles(ctx, psf, mix, gal, n, W, flags, out, s, [&](RenderArgs* a) {
    a->prof = kProfComposite;
    a->prof_a = bulge_frac;
    a->prof_b = bulge_rho;
    a->prof_k1 = Kd;
    a->prof_k2 = Kb;
    a->prof_disk = disk_table;
    a->prof_bulge = bulge_table;
    const float* lows[2] = {&mix->low[2 * (size_t)disk_table], &mix->low[2 * (size_t)bulge_table]};
    const float both[4] = {lows[0][0], lows[0][1], lows[1][0], lows[1][1]};
    float low[2];
    two_smallest(both, 4, low);
    a->flat_v2 = low[1];
    a->amp = mix->d_amp;  // a per-call amplitude table is not used here
    a->var = mix->d_var;
  });
}

}  // extern "C"
