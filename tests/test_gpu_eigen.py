"""GPU parity of the spatially varying (eigen-)PSF render, through the C ABI,
against the FP64 eigen-PSF oracle (oracle/eigen.py), which sums the
component images in pixel space before transforming; the library sums the
cached component transforms and moments per galaxy.  Bar: per stamp,
max |gpu - oracle| <= 1e-5 x max |oracle|."""

import numpy as np
import pytest

import oracle as o
from oracle import eigen as oe
import workloads as wl
from gpu_helpers import TOL_PEAK

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2012_15797_amd as gfc
    return gfc.Context.default(0)


@pytest.fixture(scope="module")
def eig():
    return wl.eigen_psf_moffat(64, 2)


def _lib(ctx, eig, mixtures):
    import paper_2012_15797_amd as gfc
    psf = gfc.Psf.eigen(ctx, eig["comps"], eig["coef"], eig["degree"], eig["norm"])
    mix = gfc.Mixture.from_workload(ctx, mixtures.as_f32())
    return psf, mix


def _render(ctx, psf, mix, gal, W, px, py, flags=0):
    import torch
    import paper_2012_15797_amd as gfc
    out = gfc.gfc_render_stamps(ctx, psf, mix, gal.x, gal.y, gal.flux, gal.r_e, gal.e1, gal.e2, W,
                                mix_id=gal.mix_id, flags=flags, psf_x=px, psf_y=py)
    torch.cuda.synchronize()
    return out.cpu().numpy().astype(np.float64)


def _eig64(eig):
    """The oracle sees the float32 components the library was given."""
    return dict(eig, comps=np.asarray(eig["comps"], np.float32).astype(np.float64))


def _check(gpu, ref, idx):
    errs = np.array([np.abs(gpu[i] - r).max() / np.abs(r).max() for i, r in zip(idx, ref)])
    assert errs.max() <= TOL_PEAK, (errs.max(), int(np.argmax(errs)))
    return errs


def test_component_spectra_cache(ctx, eig):
    """The cache holds one spectrum per component, equal to the oracle's DFT
    of each component image."""
    import paper_2012_15797_amd as gfc
    psf = gfc.Psf.eigen(ctx, eig["comps"], eig["coef"], eig["degree"], eig["norm"])
    spec = psf.spectrum(64).cpu().numpy().astype(np.complex128)
    assert spec.shape == (6, 64, 33)
    for j in range(6):
        ref = o.psf_spectrum(np.asarray(eig["comps"][j], np.float64), 64)[:, :33]
        assert np.abs(spec[j] - ref).max() <= 2e-7 * np.abs(ref).max()
    psf.close()


@pytest.mark.parametrize("W", [16, 32, 64, 128, 256])
def test_eigen_each_size(ctx, eig, W):
    """Hybrid routing over a spread of radii and positions across the whole
    field (the PSF width and ellipticity drift with position)."""
    rng = np.random.Generator(np.random.PCG64(800 + W))
    cfg = wl.config2(10)
    n = 40 if W < 256 else 10
    gal = wl.draw_galaxies(rng, n, W, (np.arange(n) % 2).astype(np.int32), r_e_range=(0.3, W / 4.0))
    px = rng.uniform(0, 4096, n).astype(np.float32)
    py = rng.uniform(0, 4096, n).astype(np.float32)
    psf, mix = _lib(ctx, eig, cfg["mix"])
    gpu = _render(ctx, psf, mix, gal, W, px, py)
    idx = list(range(n))
    ref = oe.render_batch_eigen(_eig64(eig), cfg["mix"].as_f32(), gal, px, py, idx=idx)
    _check(gpu, ref, idx)
    psf.close(); mix.close()


@pytest.mark.parametrize("flags", [1, 2])
def test_eigen_routing_flags(ctx, eig, flags):
    """All-Fourier and all-real-space: the latter uses only the per-position
    moment Gaussian of the varying PSF."""
    rng = np.random.Generator(np.random.PCG64(850 + flags))
    cfg = wl.config_metric(10)
    n = 30
    gal = wl.draw_galaxies(rng, n, 64, 0, r_e_range=(0.5, 6.0))
    px = rng.uniform(0, 4096, n).astype(np.float32)
    py = rng.uniform(0, 4096, n).astype(np.float32)
    psf, mix = _lib(ctx, eig, cfg["mix"])
    gpu = _render(ctx, psf, mix, gal, 64, px, py, flags=flags)
    idx = list(range(n))
    ref = oe.render_batch_eigen(_eig64(eig), cfg["mix"].as_f32(), gal, px, py, flags=flags, idx=idx)
    _check(gpu, ref, idx)
    psf.close(); mix.close()


def test_single_component_matches_constant_psf(ctx):
    """J = 1, degree 0, weight 1 renders the constant PSF (to float32
    rounding of the moment Gaussian)."""
    import paper_2012_15797_amd as gfc
    cfg = wl.config_metric(40)
    gal = cfg["gal"]
    P = cfg["psf"]
    a = gfc.Psf(ctx, P)
    b = gfc.Psf.eigen(ctx, P[None], [[1.0]], 0, [0.0, 1.0, 0.0, 1.0])
    mix = gfc.Mixture.from_workload(ctx, cfg["mix"].as_f32())
    ra = _render(ctx, a, mix, gal, 64, None, None)
    rb = _render(ctx, b, mix, gal, 64, np.zeros(40, np.float32), np.zeros(40, np.float32))
    peak = np.abs(ra).max(axis=(1, 2))
    assert (np.abs(ra - rb).max(axis=(1, 2)) <= 2e-6 * peak).all()
    a.close(); b.close(); mix.close()


@pytest.mark.parametrize("J", [1, 2, 3, 15, 16])
@pytest.mark.parametrize("W", [32, 64, 128, 256])
def test_eigen_component_counts(ctx, eig, W, J):
    """Odd and even component counts up to the largest (the components are
    summed two at a time, the one past the last with weight zero), five stamps
    (a partial workgroup of four at 64): the first components carry the PSF,
    the rest small multiples of its parts."""
    rng = np.random.Generator(np.random.PCG64(880 + J))
    base = np.asarray(eig["comps"], np.float32)
    comps = np.stack([base[0] if j == 0 else base[j % 6] * np.float32(0.3 if j < 6 else 0.01 * j) for j in range(J)])
    coef = np.zeros((J, 6))
    coef[0, 0] = 1.0
    coef[1:] = rng.normal(0.0, 0.2, (J - 1, 6))
    e = dict(comps=comps, coef=coef, degree=2, norm=eig["norm"])
    cfg = wl.config_metric(10)
    n = 5
    gal = wl.draw_galaxies(rng, n, W, 0, r_e_range=(0.5, W / 6.0))
    px, py = (rng.uniform(0, 4096, n).astype(np.float32) for _ in range(2))
    psf, mix = _lib(ctx, e, cfg["mix"])
    gpu = _render(ctx, psf, mix, gal, W, px, py)
    ref = oe.render_batch_eigen(_eig64(e), cfg["mix"].as_f32(), gal, px, py, idx=range(n))
    _check(gpu, ref, range(n))
    psf.close(); mix.close()


def test_full_size_eigen_workload_sampled(ctx):
    """The 100,000-stamp eigen-PSF workload in one launch, sampled."""
    cfg = wl.config_eigen()
    gal = cfg["gal"]
    psf, mix = _lib(ctx, cfg["eig"], cfg["mix"])
    gpu = _render(ctx, psf, mix, gal, 64, cfg["psf_x"], cfg["psf_y"])
    assert np.isfinite(gpu).all()
    rng = np.random.Generator(np.random.PCG64(870))
    idx = sorted(set(rng.choice(len(gal), 120, replace=False).tolist()) | {0, len(gal) - 1})
    ref = oe.render_batch_eigen(_eig64(cfg["eig"]), cfg["mix"].as_f32(), gal, cfg["psf_x"], cfg["psf_y"],
                                idx=idx)
    _check(gpu, ref, idx)
    psf.close(); mix.close()


def test_eigen_errors(ctx, eig):
    import paper_2012_15797_amd as gfc
    cfg = wl.config_metric(10)
    gal = cfg["gal"]
    psf, mix = _lib(ctx, eig, cfg["mix"])
    with pytest.raises(gfc.GfcError) as e:  # positions are required
        gfc.gfc_render_stamps(ctx, psf, mix, gal.x, gal.y, gal.flux, gal.r_e, gal.e1, gal.e2, 64)
    assert e.value.status == -1
    with pytest.raises(gfc.GfcError) as e:
        psf.gauss
    assert e.value.status == -2
    import torch
    g = torch.zeros((10, 64, 64), device="cuda")
    with pytest.raises(gfc.GfcError) as e:
        gfc.gfc_render_stamps_backward(ctx, psf, mix, gal.x, gal.y, gal.flux, gal.r_e, gal.e1, gal.e2, 64, g)
    assert e.value.status == -2
    with pytest.raises(gfc.GfcError) as e:  # degree out of range
        gfc.Psf.eigen(ctx, eig["comps"][:1], np.ones((1, 15)), 4, eig["norm"])
    assert e.value.status == -1
    psf.close(); mix.close()
