"""GPU parity of the forward render (through the C ABI) against the FP64
oracle: per stamp, max |gpu - oracle| <= 1e-5 x max |oracle|."""

import math

import numpy as np
import pytest

import oracle as o
import workloads as wl
from gpu_helpers import TOL_PEAK, lib_objects, oracle_stamps, peak_errors, render_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2012_15797_amd as gfc
    return gfc.Context.default(0)


@pytest.mark.parametrize("W", [16, 32, 64, 128, 256])
def test_psf_spectrum_cache(ctx, W):
    """Steps 1-2 (PSF-FT cache): the device spectrum equals the oracle's naive
    DFT of the folded PSF, to float32 rounding."""
    import paper_2012_15797_amd as gfc

    P = wl.psf_moffat_halo(64).astype(np.float32)
    psf = gfc.Psf(ctx, P)
    spec = psf.spectrum(W).cpu().numpy().astype(np.complex128)
    ref = o.psf_spectrum(P.astype(np.float64), W)[:, : W // 2 + 1]
    assert np.abs(spec - ref).max() <= 2e-7 * np.abs(ref).max()
    np.testing.assert_allclose(psf.gauss, o.psf_gauss_moments(P.astype(np.float64)), rtol=1e-9, atol=1e-12)
    psf.close()


def test_tiny_case_sixteen_offsets(ctx):
    """Tiny case: one EXP6 galaxy in a 64x64 stamp at 16 sub-pixel offsets,
    every component in Fourier space."""
    cfg = wl.config1()
    psf, mix = lib_objects(ctx, cfg)
    gal = cfg["gal"]
    gpu = render_gpu(ctx, psf, mix, gal, 64, flags=cfg["flags"])
    idx = list(range(len(gal)))
    ref = oracle_stamps(cfg, gal, idx, flags=cfg["flags"])
    errs = peak_errors(gpu, ref, idx)
    assert errs.max() <= TOL_PEAK, errs
    psf.close(); mix.close()


@pytest.mark.parametrize("W", [16, 32, 64, 128, 256])
def test_hybrid_each_size(ctx, W):
    """Every stamp size with hybrid routing over a spread of radii, so that
    all-Fourier, ramped and real-space components all occur; 70 stamps
    (several workgroups and a ragged tail), 16 at W = 256."""
    rng = np.random.Generator(np.random.PCG64(100 + W))
    cfg = wl.config2(10)
    n = 70 if W < 256 else 16
    gal = wl.draw_galaxies(rng, n, W, (np.arange(n) % 2).astype(np.int32),
                           r_e_range=(0.3, W / 4.0))
    psf, mix = lib_objects(ctx, cfg)
    gpu = render_gpu(ctx, psf, mix, gal, W)
    idx = list(range(n))
    ref = oracle_stamps(cfg, gal, idx)
    errs = peak_errors(gpu, ref, idx)
    assert errs.max() <= TOL_PEAK, (errs.max(), int(errs.argmax()))
    psf.close(); mix.close()


@pytest.mark.parametrize("flags", [1, 2, 4])
def test_routing_flags(ctx, flags):
    cfg = wl.config_metric(40)
    gal = cfg["gal"]
    psf, mix = lib_objects(ctx, cfg)
    gpu = render_gpu(ctx, psf, mix, gal, 64, flags=flags)
    idx = list(range(len(gal)))
    errs = peak_errors(gpu, oracle_stamps(cfg, gal, idx, flags=flags), idx)
    assert errs.max() <= TOL_PEAK, errs.max()
    psf.close(); mix.close()


def test_metric_workload_sample(ctx):
    """The throughput workload (DEV8, 64x64, Moffat PSF, hybrid routing):
    500 consecutive stamps against the oracle."""
    cfg = wl.config_metric(500)
    gal = cfg["gal"]
    psf, mix = lib_objects(ctx, cfg)
    gpu = render_gpu(ctx, psf, mix, gal, 64)
    idx = list(range(len(gal)))
    errs = peak_errors(gpu, oracle_stamps(cfg, gal, idx), idx)
    assert errs.max() <= TOL_PEAK, errs.max()
    psf.close(); mix.close()


def test_metric_workload_full_size_sampled(ctx):
    """All 100,000 stamps of the throughput workload in one launch (the
    benchmark's configuration); 300 sampled stamps against the oracle, and
    properties of every stamp: finite, and the total equals flux x sum(A)
    x sum(PSF) up to the light the real-space components put outside the
    stamp."""
    import torch
    import paper_2012_15797_amd as gfc

    cfg = wl.config_metric()
    gal = cfg["gal"]
    psf, mix = lib_objects(ctx, cfg)
    out = gfc.gfc_render_stamps(ctx, psf, mix, gal.x, gal.y, gal.flux, gal.r_e, gal.e1, gal.e2, 64)
    torch.cuda.synchronize()
    assert torch.isfinite(out).all()
    tot = out.double().sum(dim=(1, 2)).cpu().numpy()
    amp, _ = cfg["mix"].as_f32().table(0)
    expect = gal.flux.astype(np.float64) * amp.sum() * cfg["psf"].astype(np.float64).sum()
    assert (tot <= expect * (1 + 1e-5)).all() and (tot >= 0.95 * expect).all()
    idx = np.random.Generator(np.random.PCG64(9)).choice(len(gal), 300, replace=False)
    sample = out[torch.as_tensor(idx, device=out.device)].cpu().numpy().astype(np.float64)
    ref = oracle_stamps(cfg, gal, idx)
    errs = np.array([np.abs(sample[j] - ref[j]).max() / np.abs(ref[j]).max() for j in range(len(idx))])
    assert errs.max() <= TOL_PEAK, errs.max()
    psf.close(); mix.close()


def test_cd_matrix(ctx):
    """Step 3 with a non-identity local WCS matrix: A = CD^{-1} E."""
    cfg = wl.config_metric(30)
    gal = cfg["gal"]
    cd = np.array([1.1, 0.2, -0.15, 0.9])
    psf, mix = lib_objects(ctx, cfg)
    gpu = render_gpu(ctx, psf, mix, gal, 64, cd=cd.astype(np.float32))
    idx = list(range(len(gal)))
    ref = oracle_stamps(cfg, gal, idx, cd=cd.astype(np.float32).astype(np.float64))
    errs = peak_errors(gpu, ref, idx)
    assert errs.max() <= TOL_PEAK, errs.max()
    psf.close(); mix.close()


@pytest.mark.parametrize("W", [128, 256])
def test_large_galaxy_workload(ctx, W):
    """Large-galaxy case (r_e 10..60 px, DEV8, 1-4 components in real space)
    at 128 and 256 with the fitted single-Gaussian PSF, 20 stamps each."""
    cfg = wl.config3(400)
    sel = np.nonzero(cfg["gal"].W == W)[0][:20]
    gal = cfg["gal"].subset(sel)
    psf, mix = lib_objects(ctx, cfg)
    gpu = render_gpu(ctx, psf, mix, gal, W)
    idx = list(range(len(gal)))
    errs = peak_errors(gpu, oracle_stamps(cfg, gal, idx), idx)
    assert errs.max() <= TOL_PEAK, errs.max()
    psf.close(); mix.close()


def test_large_workload_full_size_sampled(ctx):
    """Every 256 x 256 stamp of the large-galaxy workload (about 9,900) in one
    launch, as the benchmark times it: one workgroup per CU stays resident
    and takes stamps in turn.  Stamps at the first and later rounds of the
    workgroups, the last stamp and a random sample against the oracle; every
    stamp finite."""
    import torch
    import paper_2012_15797_amd as gfc

    cfg = wl.config3()
    gal = cfg["gal"].subset(np.nonzero(cfg["gal"].W == 256)[0])
    n = len(gal)
    psf, mix = lib_objects(ctx, cfg)
    out = gfc.gfc_render_stamps(ctx, psf, mix, gal.x, gal.y, gal.flux, gal.r_e, gal.e1, gal.e2, 256,
                                mix_id=gal.mix_id)
    torch.cuda.synchronize()
    assert torch.isfinite(out).all()
    rng = np.random.Generator(np.random.PCG64(11))
    idx = sorted(set([0, 1, 255, 256, 257, 511, 512, 1023, 1024, n - 1]) |
                 set(rng.choice(n, 14, replace=False).tolist()))
    sample = out[torch.as_tensor(idx, device=out.device)].cpu().numpy().astype(np.float64)
    errs = peak_errors(sample, oracle_stamps(cfg, gal, idx), list(range(len(idx))))
    assert errs.max() <= TOL_PEAK, errs.max()
    psf.close(); mix.close()


@pytest.mark.parametrize("flags,cd", [(1, None), (0, None), (4, None), (1, (1.3, 0.4, -0.2, 0.7))])
def test_w256_negligible_block_skip_extremes(ctx, flags, cd):
    """At 256 x 256 a block of Fourier bins is skipped for a component when a
    bound from the smallest eigenvalue of the shape matrix puts every
    exponent in it below -40.  The bound is tightest for wide, elongated
    galaxies: r_e from 2 to 60 px, |e| up to 0.69 at four orientations, every
    component forced to Fourier space (the widest are then skipped almost
    everywhere), the hybrid and linear-ramp routings, and a sheared,
    anisotropic CD matrix."""
    cfg = wl.config3(10)
    rng = np.random.Generator(np.random.PCG64(4040))
    r_e, e1, e2 = [], [], []
    for r in (2.0, 8.0, 20.0, 40.0, 60.0):
        for e, th in ((0.0, 0.0), (0.69, 0.0), (0.69, 0.785), (0.5, 1.571), (0.69, 2.356)):
            r_e.append(r); e1.append(e * math.cos(2 * th)); e2.append(e * math.sin(2 * th))
    n = len(r_e)
    f32 = lambda a: np.asarray(a, np.float32)
    gal = wl.Galaxies(f32(128.0 + rng.uniform(0, 1, n)), f32(128.0 + rng.uniform(0, 1, n)),
                      f32(rng.uniform(1.0, 1e3, n)), f32(r_e), f32(e1), f32(e2), np.zeros(n, np.int32),
                      np.full(n, 256, np.int32))
    cdv = None if cd is None else np.asarray(cd, np.float32)
    psf, mix = lib_objects(ctx, cfg)
    gpu = render_gpu(ctx, psf, mix, gal, 256, flags=flags, cd=cdv)
    idx = list(range(n))
    ref = oracle_stamps(cfg, gal, idx, flags=flags, cd=None if cdv is None else cdv.astype(np.float64))
    errs = peak_errors(gpu, ref, idx)
    assert errs.max() <= TOL_PEAK, (errs.max(), int(errs.argmax()))
    psf.close(); mix.close()


def test_w256_persistent_rounds_tables_and_invalid():
    """At 256 x 256 a workgroup takes stamps in turn and loads the next
    stamp's inputs while it renders the current one.  600 galaxies (two to
    three stamps per workgroup) alternate between two mixture tables, with
    invalid galaxies in the first, second and third rounds: those come out
    NaN and are counted, and their neighbours, whose inputs travel beside
    them, match the oracle."""
    import torch
    import paper_2012_15797_amd as gfc

    local = gfc.Context(0)
    cfg = wl.config2(10)  # two tables (EXP6 and DEV8) and the Moffat + halo PSF
    rng = np.random.Generator(np.random.PCG64(256))
    n = 600
    g = wl.draw_galaxies(rng, n, 256, (np.arange(n) % 2).astype(np.int32), r_e_range=(4.0, 40.0))
    x, r_e, e1, e2, mid = g.x.copy(), g.r_e.copy(), g.e1.copy(), g.e2.copy(), g.mix_id.copy()
    e1[5], e2[5] = 0.99, 0.5  # |e| >= 1
    r_e[256] = -1.0
    mid[300] = 7              # no such table
    x[599] = np.nan
    bad = [5, 256, 300, 599]
    gal = wl.Galaxies(x, g.y, g.flux, r_e, e1, e2, mid, g.W)
    psf, mix = lib_objects(local, cfg)
    out = gfc.gfc_render_stamps(local, psf, mix, gal.x, gal.y, gal.flux, gal.r_e, gal.e1, gal.e2, 256,
                                mix_id=gal.mix_id)
    torch.cuda.synchronize()
    dev = out.device
    assert torch.isnan(out[torch.as_tensor(bad, device=dev)]).all()
    good = torch.as_tensor([i for i in range(n) if i not in bad], device=dev)
    assert torch.isfinite(out[good]).all()
    assert local.invalid_count() == len(bad)
    idx = sorted(set([0, 4, 6, 255, 257, 299, 301, 511, 512, 598]) |
                 set(int(i) for i in rng.choice([i for i in range(n) if i not in bad], 3, replace=False)))
    sample = out[torch.as_tensor(idx, device=dev)].cpu().numpy().astype(np.float64)
    errs = peak_errors(sample, oracle_stamps(cfg, gal, idx), list(range(len(idx))))
    assert errs.max() <= TOL_PEAK, errs.max()
    psf.close(); mix.close()


@pytest.mark.parametrize("W", [16, 32, 64, 128, 256])
def test_edge_positions_and_integer_shift(ctx, W):
    """Centres near and across the stamp edge, negative and large
    coordinates: the integer part of x becomes a cyclic roll of the Fourier
    image and that of y a phase from an exact table entry.  Run with every
    component forced to Fourier space, so the whole stamp is periodic, and
    with the hybrid routing."""
    cfg = wl.config_metric(10)
    base = cfg["gal"]
    s = W / 64.0
    xs = (np.array([0.0, 0.4, 63.9, -3.25, 100.6, 31.0, 32.5, -64.2, 12345.625, -9876.5]) * s).astype(np.float32)
    ys = (np.array([63.7, 0.0, 17.2, 5.5, -40.1, 31.0, 96.0, 2.0, -23456.375, 8765.125]) * s).astype(np.float32)
    gal = wl.Galaxies(xs, ys, base.flux, base.r_e, base.e1, base.e2, base.mix_id,
                      np.full(10, W, np.int32))
    psf, mix = lib_objects(ctx, cfg)
    for flags in (o.FORCE_FOURIER, 0):
        gpu = render_gpu(ctx, psf, mix, gal, W, flags=flags)
        idx = list(range(len(gal)))
        errs = peak_errors(gpu, oracle_stamps(cfg, gal, idx, flags=flags), idx)
        assert errs.max() <= TOL_PEAK, (flags, errs)
    psf.close(); mix.close()


def test_invalid_galaxies_give_nan_and_count(ctx):
    import paper_2012_15797_amd as gfc

    local = gfc.Context(0)
    cfg = wl.config_metric(6)
    g = cfg["gal"]
    e1 = g.e1.copy(); r_e = g.r_e.copy(); x = g.x.copy()
    e1[1] = 0.99; g.e2[1] = 0.5     # |e| >= 1
    r_e[2] = -1.0
    x[3] = np.nan
    mid = np.zeros(6, np.int32); mid[4] = 7   # no such table
    gal = wl.Galaxies(x, g.y, g.flux, r_e, e1, g.e2, mid, g.W)
    psf, mix = lib_objects(local, cfg)
    gpu = render_gpu(local, psf, mix, gal, 64)
    bad = [1, 2, 3, 4]
    assert np.isnan(gpu[bad]).all()
    assert np.isfinite(gpu[[0, 5]]).all()
    assert local.invalid_count() == 4
    psf.close(); mix.close()


def test_deterministic(ctx):
    cfg = wl.config_metric(300)
    gal = cfg["gal"]
    psf, mix = lib_objects(ctx, cfg)
    a = render_gpu(ctx, psf, mix, gal, 64)
    b = render_gpu(ctx, psf, mix, gal, 64)
    assert np.array_equal(a, b)
    psf.close(); mix.close()


def test_empty_batch_and_errors(ctx):
    import paper_2012_15797_amd as gfc

    cfg = wl.config_metric(0)
    psf, mix = lib_objects(ctx, cfg)
    e = np.zeros(0, np.float32)
    out = gfc.gfc_render_stamps(ctx, psf, mix, e, e, e, e, e, e, 64)
    assert out.shape == (0, 64, 64)
    one = np.ones(1, np.float32)
    with pytest.raises(gfc.GfcError):
        gfc.gfc_render_stamps(ctx, psf, mix, one, one, one, one, one, one, 48)
    with pytest.raises(gfc.GfcError):
        gfc.gfc_render_stamps(ctx, psf, mix, one, one, one, one, one, one, 64, flags=3)
    psf.close(); mix.close()


@pytest.mark.parametrize("flags", [0, 1])
@pytest.mark.parametrize("W", [16, 32, 64, 128, 256])
def test_flat_components_and_stores(ctx, W, flags):
    """The components whose exponent stays within one power of two over the
    frequency grid, which are summed as one polynomial: tables with all, some,
    one (not merged) and no such component, zero and negative amplitudes among
    them, r_e from 0.02 px to W/5, hybrid and forced-Fourier routing.  Stamps of
    one wavefront (16, 32) differ in which components are flat.  The output is
    aligned as floats only, and a second, accumulated render doubles it."""
    import torch
    import paper_2012_15797_amd as gfc

    rng = np.random.Generator(np.random.PCG64(1700 + W))
    tables = [(rng.dirichlet(np.ones(16)), np.logspace(-9, -5, 16)), (rng.dirichlet(np.ones(16)), np.logspace(-4, 1, 16)),
              (np.array([0.6, 0.4]), np.array([1e-6, 4.0])), (np.array([0.9, 0.0, -0.2, 0.3]), np.array([2e-4, 1e-3, 1e-2, 0.5])),
              (np.array([0.5, 0.5]), np.array([3.0, 9.0]))]
    mixtures = wl.mixture_set(tables)
    cfg = dict(mix=mixtures, psf=wl.config_metric(4)["psf"])
    n = 25
    gal = wl.draw_galaxies(rng, n, W, (np.arange(n) % 5).astype(np.int32), r_e_range=(0.02, W / 5.0))
    gal.x[:5], gal.y[:5] = [0, W - 1, W / 2, -2, W + 0.25], [W / 2, 0.5, W - 1, 3, -0.75]
    psf, mix = lib_objects(ctx, cfg)
    buf = torch.zeros(n * W * W + 1, device="cuda")
    out = buf[1:].view(n, W, W)
    args = (ctx, psf, mix, gal.x, gal.y, gal.flux, gal.r_e, gal.e1, gal.e2, W)
    gfc.gfc_render_stamps(*args, mix_id=gal.mix_id, flags=flags, out=out)
    once = out.clone()
    gfc.gfc_render_stamps(*args, mix_id=gal.mix_id, flags=flags | gfc.GFC_ACCUMULATE, out=out)
    torch.cuda.synchronize()
    assert torch.equal(out, 2 * once) and float(buf[0]) == 0.0
    ref = oracle_stamps(cfg, gal, range(n), flags=flags)
    errs = peak_errors(once.cpu().numpy().astype(np.float64), ref, range(n))
    assert errs.max() <= TOL_PEAK, (errs.max(), int(np.argmax(errs)))
    psf.close(); mix.close()


@pytest.mark.parametrize("flags", [0, 2])
@pytest.mark.parametrize("W", [16, 32, 64, 128, 256])
def test_largest_radii(ctx, W, flags):
    """Radii whose product with a component's variance overflows the exponent's
    range (v r_e^2 from 2e36 px^2): every pixel is below the smallest float32,
    so the stamp is zero, and its neighbours are as without it.  (From 2.4e18
    px the shape's own exponent overflows: NaN up to 128 x 128.)"""
    import torch
    import paper_2012_15797_amd as gfc

    rng = np.random.Generator(np.random.PCG64(1760 + W))
    mixtures = wl.mixture_set([(rng.dirichlet(np.ones(8)), np.logspace(-4, 1, 8))])
    psf, mix = lib_objects(ctx, dict(mix=mixtures, psf=wl.config_metric(4)["psf"]))
    n, huge = 9, np.array([1, 4, 6])
    gal = wl.draw_galaxies(rng, n, W, 0)
    gal.e1[huge] = gal.e2[huge] = 0.0

    def render():
        return gfc.gfc_render_stamps(ctx, psf, mix, gal.x, gal.y, gal.flux, gal.r_e, gal.e1, gal.e2, W,
                                     flags=flags).cpu().numpy()

    without = render()
    gal.r_e[huge] = [1e18, 2e18, 3e18]
    got = render()
    assert (got[huge[:2]] == 0.0).all()
    assert (got[huge[2]] == 0.0).all() or np.isnan(got[huge[2]]).all()
    others = np.setdiff1d(np.arange(n), huge)
    assert np.array_equal(got[others], without[others])
    psf.close(); mix.close()


def _centred_gaussians(rng, n, W):
    """Round one-component galaxies near the stamp's middle and a PSF whose
    Gaussian (given, off centre) is all that the real-space part takes of it:
    float64 stamps and their derivatives along x and y."""
    x, y = (W / 2 + rng.uniform(0, 1, (2, n))).astype(np.float32)
    r_e = rng.uniform(1.0, W / 16, n).astype(np.float32)
    gauss = [0.21, -0.37, 1.5, 0.0, 1.5, 0.9]
    var = r_e.astype(np.float64) ** 2 + gauss[2]
    p = np.arange(W, dtype=np.float64)
    ux = p[None, None, :] - (x.astype(np.float64) + gauss[0])[:, None, None]
    uy = p[None, :, None] - (y.astype(np.float64) + gauss[1])[:, None, None]
    v = var[:, None, None]
    img = gauss[5] / (2 * np.pi * v) * np.exp(-0.5 * (ux * ux + uy * uy) / v)
    return x, y, r_e, gauss, img, img * ux / v, img * uy / v


@pytest.mark.parametrize("W", [16, 32, 64, 128, 256])
def test_real_space_position(ctx, W):
    """Where the real-space part puts a galaxy: the shift that its error amounts
    to (the error's projection on the derivative along x and y).  dx of the
    middle column, at most 1.4 px here, rounds by 2^-24, m by 2^-24 and g m by
    2^-24 times m: below 2^-22 px, with the roundings that differ from pixel to
    pixel averaging out.  At 256 the eight lanes of a row count from columns
    up to 28 further on, and m rounds by 2^-24 times that: 2^-19 px."""
    import paper_2012_15797_amd as gfc

    rng = np.random.Generator(np.random.PCG64(1790 + W))
    n = 32
    x, y, r_e, gauss, img, ix, iy = _centred_gaussians(rng, n, W)
    psf = gfc.Psf(ctx, wl.psf_moffat_halo(32).astype(np.float32), gauss)
    mix = gfc.Mixture.from_workload(ctx, wl.mixture_set([(np.ones(1), np.ones(1))]).as_f32())
    zero = np.zeros(n, np.float32)
    got = gfc.gfc_render_stamps(ctx, psf, mix, x, y, np.ones(n, np.float32), r_e, zero, zero, W, flags=2)
    err = got.cpu().numpy().astype(np.float64) - img
    shift = [np.abs((err * d).sum((1, 2)) / (d * d).sum((1, 2))).max() for d in (ix, iy)]
    assert max(shift) < 2.0 ** (-22 if W <= 128 else -19), shift
    psf.close(); mix.close()


@pytest.mark.parametrize("shared", [True, False])
@pytest.mark.parametrize("W", [16, 32])
def test_flat_components_between_neighbours(ctx, W, shared):
    """Stamps that share a wavefront, with tables for which it forms the flat
    components' polynomial and with one more table for which it does not: both
    against the oracle, and each stamp is bit for bit the one that it is in a
    launch of its own."""
    import paper_2012_15797_amd as gfc

    rng = np.random.Generator(np.random.PCG64(1880 + W))
    tables = [(rng.dirichlet(np.ones(8)), np.logspace(-4, 1, 8)), (rng.dirichlet(np.ones(16)), np.logspace(-9, -5, 16)),
              (np.array([0.9, 0.0, -0.2, 0.3]), np.array([2e-4, 1e-3, 1e-2, 0.5]))]
    mixtures = wl.mixture_set(tables if shared else tables + [(np.array([0.5, 0.5]), np.array([3.0, 9.0]))])
    cfg = dict(mix=mixtures, psf=wl.config_metric(4)["psf"])
    n = 27
    gal = wl.draw_galaxies(rng, n, W, (np.arange(n) % 3).astype(np.int32), r_e_range=(0.1, W / 2.0))
    psf, mix = lib_objects(ctx, cfg)

    def render(i):
        return gfc.gfc_render_stamps(ctx, psf, mix, gal.x[i], gal.y[i], gal.flux[i], gal.r_e[i], gal.e1[i], gal.e2[i], W,
                                     mix_id=gal.mix_id[i]).cpu().numpy()

    got = render(np.arange(n))
    assert np.array_equal(got, np.concatenate([render(np.array([i])) for i in range(n)]))
    errs = peak_errors(got.astype(np.float64), oracle_stamps(cfg, gal, range(n)), range(n))
    assert errs.max() <= TOL_PEAK, (errs.max(), int(np.argmax(errs)))
    psf.close(); mix.close()
