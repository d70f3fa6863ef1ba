"""GPU parity of the adjoint (gfc_render_stamps_backward, through the C ABI)
against the FP64 derivative oracle, which itself is pinned to central finite
differences on the CPU (tests/test_oracle_grad.py).

Bar: for each parameter, |gpu - oracle| <= 1e-4 |oracle| wherever |oracle| is
at least 1e-2 of its rms over the case's galaxies; below that 1e-5 rms is
added (gradients that cancel to nearly zero, or galaxies far fainter than the
case's brightest, whose float32 rounding is set by the size of the summed
terms, not by the result)."""

import math

import numpy as np
import pytest

import oracle as o
import workloads as wl
from gpu_helpers import assert_grads_close as assert_close, gpu_grads, lib_objects, oracle_grads
from oracle.grad import PARAMS

pytestmark = pytest.mark.gpu

@pytest.fixture(scope="module")
def ctx():
    import paper_2012_15797_amd as gfc
    return gfc.Context.default(0)


@pytest.mark.parametrize("W", [16, 32, 64, 128, 256])
def test_backward_each_size(ctx, W):
    rng = np.random.Generator(np.random.PCG64(300 + W))
    cfg = wl.config2(10)
    n = 40 if W < 128 else (12 if W == 128 else 10)
    gal = wl.draw_galaxies(rng, n, W, (np.arange(n) % 2).astype(np.int32), r_e_range=(0.4, W / 5.0))
    g = rng.standard_normal((n, W, W)).astype(np.float32)
    psf, mix = lib_objects(ctx, cfg)
    gp, ga = gpu_grads(ctx, psf, mix, gal, W, g)
    rp, ra, ra_abs = oracle_grads(cfg, gal, g)
    assert_close(gp, rp, f"params W={W}")
    assert_close(ga, ra, f"amplitudes W={W}", scale=ra_abs)
    psf.close(); mix.close()


def test_backward_w256_across_chunks(ctx):
    """W = 256 runs in chunks of 1024 stamps over one reused device slab;
    galaxies on both sides of the chunk boundary, and the last, are checked
    against the oracle (the others must be finite)."""
    rng = np.random.Generator(np.random.PCG64(310))
    cfg = wl.config2(10)
    W, n = 256, 1030
    gal = wl.draw_galaxies(rng, n, W, (np.arange(n) % 2).astype(np.int32), r_e_range=(0.4, W / 5.0))
    g = rng.standard_normal((n, W, W)).astype(np.float32)
    psf, mix = lib_objects(ctx, cfg)
    gp, _ = gpu_grads(ctx, psf, mix, gal, W, g)
    assert np.isfinite(gp).all()
    idx = [0, 1, 1022, 1023, 1024, 1025, 1029]
    rp, _, _ = oracle_grads(cfg, gal.subset(idx), g[idx])
    assert_close(gp[idx], rp, "params W=256 chunk boundary")
    psf.close(); mix.close()


@pytest.mark.parametrize("W", [32, 64, 128, 256])
@pytest.mark.parametrize("case", ["positions", "skip", "sheared"])
def test_backward_routes(ctx, case, W):
    """The adjoint where its parts can go wrong: centres on integers of either
    parity, negative and outside the stamp (from 64 up the integer part is a
    phase, its sign the Nyquist column's); the skip of negligible blocks at
    its extremes (r_e W/128 and W/4 px, |e| = 0.69 at four orientations); a
    sheared CD matrix with a 16-component table, and an upstream gradient that
    is aligned as floats only."""
    import torch
    import paper_2012_15797_amd as gfc

    rng = np.random.Generator(np.random.PCG64(320 + W))
    cfg = wl.config_metric(10)
    n, cd, mix_src = 8, None, cfg["mix"].as_f32()
    gal = wl.draw_galaxies(rng, n, W, 0, r_e_range=(W / 128, W / 4))
    if case == "positions":
        h = W // 2
        gal.x[:] = [h, h - 1, 0, -3.25, W - 0.5, W + 2.75, h + 1.5, h / 2]
        gal.y[:] = [h - 1, h, W - 0.75, 5, -1.5, h + 3, 0.75, 1.5 * h]
    elif case == "skip":
        gal.r_e[:] = np.repeat([W / 128, W / 4], 4)
        gal.e1[:], gal.e2[:] = np.tile([0.69, -0.69, 0, 0], 2), np.tile([0, 0, 0.69, -0.69], 2)
    else:
        cd = np.array([1.3, 0.4, -0.5, 0.8], np.float32)
        v = np.logspace(-4, 1, 16)[None, :]
        mix_src = wl.Mixtures(np.array([16], np.int32), rng.dirichlet(np.ones(16))[None, :], v).as_f32()
    g = rng.standard_normal((n, W, W)).astype(np.float32)
    psf = gfc.Psf(ctx, cfg["psf"])
    mix = gfc.Mixture.from_workload(ctx, mix_src)
    buf = torch.empty(n * W * W + 1, device="cuda")
    gt = buf[1:].view(n, W, W)  # 4-byte aligned
    gt.copy_(torch.as_tensor(g))
    gp, ga = gfc.gfc_render_stamps_backward(ctx, psf, mix, gal.x, gal.y, gal.flux, gal.r_e, gal.e1, gal.e2, W, gt,
                                            cd=cd)
    torch.cuda.synchronize()
    rp, ra, ra_abs = oracle_grads(cfg, gal, g, cd=None if cd is None else cd.astype(np.float64), mix=mix_src)
    assert_close(gp.cpu().numpy(), rp, f"params W={W} {case}")
    assert_close(ga.cpu().numpy(), ra, f"amplitudes W={W} {case}", scale=ra_abs)
    psf.close(); mix.close()


@pytest.mark.parametrize("flags", [1, 2, 4])
def test_backward_routing_flags(ctx, flags):
    rng = np.random.Generator(np.random.PCG64(400 + flags))
    cfg = wl.config_metric(10)
    W, n = 32, 30
    gal = wl.draw_galaxies(rng, n, W, 0, r_e_range=(0.4, 6.0))
    g = rng.standard_normal((n, W, W)).astype(np.float32)
    psf, mix = lib_objects(ctx, cfg)
    gp, ga = gpu_grads(ctx, psf, mix, gal, W, g, flags=flags)
    rp, ra, ra_abs = oracle_grads(cfg, gal, g, flags=flags)
    assert_close(gp, rp, f"params flags={flags}")
    assert_close(ga, ra, f"amplitudes flags={flags}", scale=ra_abs)
    psf.close(); mix.close()


@pytest.mark.parametrize("W", [16, 64, 128, 256])
def test_backward_forced_real_each_size(ctx, W):
    """Every component in real space (GFC_FORCE_REAL = 2): the adjoint's
    pixel-space sums alone carry the shape, position and amplitude terms, at
    each kernel's stamp size (the 256 kernel sums over 512 threads)."""
    rng = np.random.Generator(np.random.PCG64(450 + W))
    cfg = wl.config2(10)
    n = 16 if W < 128 else 6
    gal = wl.draw_galaxies(rng, n, W, (np.arange(n) % 2).astype(np.int32), r_e_range=(0.4, W / 5.0))
    g = rng.standard_normal((n, W, W)).astype(np.float32)
    psf, mix = lib_objects(ctx, cfg)
    gp, ga = gpu_grads(ctx, psf, mix, gal, W, g, flags=2)
    rp, ra, ra_abs = oracle_grads(cfg, gal, g, flags=2)
    assert_close(gp, rp, f"params W={W} forced real")
    assert_close(ga, ra, f"amplitudes W={W} forced real", scale=ra_abs)
    psf.close(); mix.close()


def test_backward_fit_workload(ctx):
    """The differentiation workload: DEV8, 64x64, upstream gradient
    (I - T) / sigma^2 with T = render at perturbed parameters plus noise of
    0.01 x peak; 40 galaxies."""
    cfg = wl.config5(40)
    gal, tgt = cfg["gal"], cfg["target_gal"]
    idx = list(range(len(gal)))
    I = np.stack(o.render_batch(cfg["psf"].astype(np.float64), cfg["mix"].as_f32(), gal, idx=idx))
    T = np.stack(o.render_batch(cfg["psf"].astype(np.float64), cfg["mix"].as_f32(), tgt, idx=idx))
    peak = np.abs(T).max(axis=(1, 2), keepdims=True)
    sigma = 0.01 * peak
    T = T + sigma * wl.generate.noise_field(cfg["noise_seed"], len(gal), 64)
    g = ((I - T) / sigma**2).astype(np.float32)
    psf, mix = lib_objects(ctx, cfg)
    gp, ga = gpu_grads(ctx, psf, mix, gal, 64, g)
    rp, ra, ra_abs = oracle_grads(cfg, gal, g)
    assert_close(gp, rp, "params fit workload")
    assert_close(ga, ra, "amplitudes fit workload", scale=ra_abs)
    psf.close(); mix.close()


def test_backward_cd_matrix(ctx):
    rng = np.random.Generator(np.random.PCG64(500))
    cfg = wl.config_metric(10)
    W, n = 32, 20
    gal = wl.draw_galaxies(rng, n, W, 0, r_e_range=(0.4, 6.0))
    g = rng.standard_normal((n, W, W)).astype(np.float32)
    cd = np.array([0.9, 0.15, -0.2, 1.1], np.float32)
    psf, mix = lib_objects(ctx, cfg)
    gp, ga = gpu_grads(ctx, psf, mix, gal, W, g, cd=cd)
    rp, ra, ra_abs = oracle_grads(cfg, gal, g, cd=cd.astype(np.float64))
    assert_close(gp, rp, "params cd")
    assert_close(ga, ra, "amplitudes cd", scale=ra_abs)
    psf.close(); mix.close()


def test_backward_deterministic_and_accumulating(ctx):
    import torch
    import paper_2012_15797_amd as gfc

    rng = np.random.Generator(np.random.PCG64(600))
    cfg = wl.config_metric(10)
    W, n = 64, 300
    gal = wl.draw_galaxies(rng, n, W, 0)
    g = torch.as_tensor(rng.standard_normal((n, W, W)).astype(np.float32)).cuda()
    psf, mix = lib_objects(ctx, cfg)
    args = (ctx, psf, mix, gal.x, gal.y, gal.flux, gal.r_e, gal.e1, gal.e2, W, g)
    gp1, ga1 = gfc.gfc_render_stamps_backward(*args)
    gp2, ga2 = gfc.gfc_render_stamps_backward(*args)
    assert torch.equal(gp1, gp2) and torch.equal(ga1, ga2)
    acc = torch.zeros_like(ga1)
    gfc.gfc_render_stamps_backward(*args, grad_amp=acc)
    gfc.gfc_render_stamps_backward(*args, grad_amp=acc)
    torch.cuda.synchronize()
    assert torch.allclose(acc, 2 * ga1, rtol=1e-6, atol=0)
    # grad_amp NULL: no amplitude reduction, the parameter gradients unchanged
    gp3, ga3 = gfc.gfc_render_stamps_backward(*args, amp_grad=False)
    torch.cuda.synchronize()
    assert ga3 is None and torch.equal(gp3, gp1)
    psf.close(); mix.close()


@pytest.mark.parametrize("W", [16, 128, 256])
def test_backward_without_amplitude_gradient(ctx, W):
    """grad_amp NULL launches no amplitude reduction and leaves the parameter
    gradients bit for bit as they are with it (the bench times the adjoint
    kernel alone this way)."""
    import torch
    import paper_2012_15797_amd as gfc

    rng = np.random.Generator(np.random.PCG64(650 + W))
    cfg = wl.config2(10)
    n = 37 if W < 128 else 9
    gal = wl.draw_galaxies(rng, n, W, (np.arange(n) % 2).astype(np.int32), r_e_range=(0.4, W / 5.0))
    g = torch.as_tensor(rng.standard_normal((n, W, W)).astype(np.float32)).cuda()
    psf, mix = lib_objects(ctx, cfg)
    args = (ctx, psf, mix, gal.x, gal.y, gal.flux, gal.r_e, gal.e1, gal.e2, W, g)
    gp1, ga1 = gfc.gfc_render_stamps_backward(*args, mix_id=gal.mix_id)
    gp2, ga2 = gfc.gfc_render_stamps_backward(*args, mix_id=gal.mix_id, amp_grad=False)
    torch.cuda.synchronize()
    assert ga2 is None and bool(torch.isfinite(ga1).all())
    assert torch.equal(gp1, gp2)
    psf.close(); mix.close()


def test_autograd_function_matches_adjoint(ctx):
    """torch.autograd through RenderStamps gives the library adjoint, with the
    log r_e chain applied (dL/dr_e = dL/dlog r_e / r_e) and amplitude
    gradients for a torch-held amplitude table."""
    import torch
    import paper_2012_15797_amd as gfc

    rng = np.random.Generator(np.random.PCG64(700))
    cfg = wl.config_metric(10)
    W, n = 32, 25
    gal = wl.draw_galaxies(rng, n, W, 0, r_e_range=(0.5, 5.0))
    psf, mix = lib_objects(ctx, cfg)
    dev = torch.device("cuda")
    t = lambda a: torch.tensor(a, device=dev, requires_grad=True)
    x, y, fl, re, e1, e2 = map(t, (gal.x, gal.y, gal.flux, gal.r_e, gal.e1, gal.e2))
    m = cfg["mix"].as_f32()
    table = np.asarray(m.amp, np.float32)
    new_amp = (table * np.linspace(0.5, 1.5, 16, dtype=np.float32)[None, :]).astype(np.float32)
    amp = torch.tensor(new_amp, device=dev, requires_grad=True)
    g = torch.as_tensor(rng.standard_normal((n, W, W)).astype(np.float32), device=dev)
    before = gfc.gfc_render_stamps(ctx, psf, mix, gal.x, gal.y, gal.flux, gal.r_e, gal.e1, gal.e2, W)
    out = gfc.render(psf, mix, x, y, fl, re, e1, e2, W, amp=amp)
    (out * g).sum().backward()
    gp, ga = gfc.gfc_render_stamps_backward(ctx, psf, mix, gal.x, gal.y, gal.flux, gal.r_e, gal.e1,
                                            gal.e2, W, g, mix_amp=amp.detach())
    torch.cuda.synchronize()
    # the per-call amplitudes leave the shared mixture as it was ...
    after = gfc.gfc_render_stamps(ctx, psf, mix, gal.x, gal.y, gal.flux, gal.r_e, gal.e1, gal.e2, W)
    torch.cuda.synchronize()
    assert torch.equal(before, after) and not torch.equal(before, out.detach())
    # ... and render as a mixture made with them would
    mix2 = gfc.Mixture(ctx, np.asarray(m.K, np.int32), new_amp, np.asarray(m.var, np.float32))
    ref = gfc.gfc_render_stamps(ctx, psf, mix2, gal.x, gal.y, gal.flux, gal.r_e, gal.e1, gal.e2, W)
    torch.cuda.synchronize()
    assert torch.equal(out.detach(), ref)
    mix2.close()
    for i, tt in enumerate((x, y, fl)):
        assert torch.allclose(tt.grad, gp[:, i])
    assert torch.allclose(re.grad, gp[:, 3] / re.detach())
    assert torch.allclose(e1.grad, gp[:, 4]) and torch.allclose(e2.grad, gp[:, 5])
    assert torch.allclose(amp.grad, ga)
    psf.close(); mix.close()


_PER_GALAXY = {}  # contributions from the first case, compared bit for bit by the others


@pytest.mark.parametrize("n_tables", [1700, 70000, (1 << 20) // 14 + 1])
def test_amplitude_sums_across_chunks_and_tables(ctx, n_tables):
    """The per-table amplitude sums over 1,700 galaxies (14 chunks of 128 in
    the two-pass reduction, the last one ragged).  Every table is a copy of
    one mixture, so a call that gives each galaxy its own table returns each
    galaxy's contribution exactly (one term per sum); a call with four shared
    tables must then equal their float64 sums per table.  70,000 tables take
    two launches of the first pass (at most 65,535 tables per grid row); with
    74,899 the chunk partials would pass 64 MiB and the one-pass reduction
    runs instead (its single-term sums must equal the others bit for bit)."""
    import torch
    import paper_2012_15797_amd as gfc

    n, W = 1700, 16
    rng = np.random.Generator(np.random.PCG64(700))  # the same galaxies in every case
    cfg = wl.config_metric(10)
    m = cfg["mix"].as_f32()
    K = np.full(n_tables, int(m.K[0]), np.int32)
    amp = np.broadcast_to(np.asarray(m.amp, np.float32)[:1], (n_tables, 16))
    var = np.broadcast_to(np.asarray(m.var, np.float32)[:1], (n_tables, 16))
    psf = gfc.Psf(ctx, cfg["psf"], cfg.get("psf_gauss"))
    mix = gfc.Mixture(ctx, K, amp, var)
    gal = wl.draw_galaxies(rng, n, W, 0)
    g = torch.as_tensor(rng.standard_normal((n, W, W)).astype(np.float32)).cuda()

    def amp_sums(mix_id):
        _, ga = gfc.gfc_render_stamps_backward(ctx, psf, mix, gal.x, gal.y, gal.flux, gal.r_e, gal.e1, gal.e2,
                                               W, g, mix_id=np.asarray(mix_id, np.int32))
        torch.cuda.synchronize()
        return ga.cpu().numpy()

    own = np.arange(n) % n_tables
    per_gal = amp_sums(own)[own].astype(np.float64)  # [n, 16], galaxy i's contribution
    used = np.array(sorted({0, min(65535, n_tables - 1), n_tables // 3, n_tables - 1}))
    shared = used[rng.integers(0, len(used), n)]
    got = amp_sums(shared)
    ref = np.zeros((n_tables, 16))
    scale = np.zeros((n_tables, 16))
    np.add.at(ref, shared, per_gal)
    np.add.at(scale, shared, np.abs(per_gal))
    err = np.abs(got - ref)
    assert (err <= 1e-5 * scale).all(), float((err / np.maximum(scale, 1e-300)).max())
    unused = np.setdiff1d(np.arange(n_tables), used)
    assert (got[unused] == 0).all()
    first = _PER_GALAXY.setdefault("per_gal", per_gal)
    assert np.array_equal(per_gal, first)
    psf.close(); mix.close()


@pytest.mark.parametrize("n,n_tables", [(1, 1), (64, 16), (65, 2), (2048, 3), (2049, 3), (2048, 17)])
def test_amplitude_sums_in_one_launch(ctx, n, n_tables):
    """The amplitude sums on both sides of the one-launch reduction's limits
    (2,048 galaxies, 16 tables) and at its row remainders, added to what
    grad_amp held.  Each galaxy's contribution is taken from a call with one
    galaxy per table.  A sum of at most 2,049 terms passes through at most 33
    additions in a thread and 10 after it, each rounding by 2^-24 of the sum
    of the terms' sizes."""
    import torch
    import paper_2012_15797_amd as gfc

    W = 16
    rng = np.random.Generator(np.random.PCG64(710 + n + n_tables))
    cfg = wl.config_metric(10)
    m = cfg["mix"].as_f32()

    def tables(t):
        return gfc.Mixture(ctx, np.full(t, int(m.K[0]), np.int32),
                           np.broadcast_to(np.asarray(m.amp, np.float32)[:1], (t, 16)),
                           np.broadcast_to(np.asarray(m.var, np.float32)[:1], (t, 16)))

    psf = gfc.Psf(ctx, cfg["psf"], cfg.get("psf_gauss"))
    gal = wl.draw_galaxies(rng, n, W, 0)
    g = torch.as_tensor(rng.standard_normal((n, W, W)).astype(np.float32)).cuda()

    def amp_sums(mix, mix_id, into=None):
        _, ga = gfc.gfc_render_stamps_backward(ctx, psf, mix, gal.x, gal.y, gal.flux, gal.r_e, gal.e1, gal.e2, W, g,
                                               mix_id=np.asarray(mix_id, np.int32), grad_amp=into)
        torch.cuda.synchronize()
        return ga.cpu().numpy().astype(np.float64)

    own, mix = tables(max(n, 17)), tables(n_tables)
    per_gal = amp_sums(own, np.arange(n))[:n]
    mid = rng.integers(0, n_tables, n)
    held = rng.standard_normal((n_tables, 16)).astype(np.float32)
    got = amp_sums(mix, mid, torch.as_tensor(held).cuda())
    ref, scale = held.astype(np.float64), np.abs(held).astype(np.float64)
    np.add.at(ref, mid, per_gal)
    np.add.at(scale, mid, np.abs(per_gal))
    assert (np.abs(got - ref) <= 44 * 2.0 ** -24 * scale).all()
    psf.close(); own.close(); mix.close()


def test_workspace_when_torch_has_no_memory(ctx, monkeypatch):
    """With nothing left in torch's allocator for the adjoint's scratch the
    library allocates it: the call gives the same gradients, and a failure is
    the library's own (GfcError)."""
    import torch
    import paper_2012_15797_amd as gfc
    from paper_2012_15797_amd import api

    rng = np.random.Generator(np.random.PCG64(1850))
    cfg = wl.config_metric(10)
    n, W = 70, 32
    gal = wl.draw_galaxies(rng, n, W, 0)
    g = torch.as_tensor(rng.standard_normal((n, W, W)).astype(np.float32)).cuda()
    psf = gfc.Psf(ctx, cfg["psf"])
    mix = gfc.Mixture.from_workload(ctx, cfg["mix"].as_f32())

    def adjoint():
        out = gfc.gfc_render_stamps_backward(ctx, psf, mix, gal.x, gal.y, gal.flux, gal.r_e, gal.e1, gal.e2, W, g)
        torch.cuda.synchronize()
        return [t.cpu() for t in out]

    usual = adjoint()
    empty, refused = torch.empty, []

    def no_scratch(*args, **kwargs):
        if kwargs.get("dtype") is torch.uint8:
            refused.append(args)
            raise torch.OutOfMemoryError("no memory left")
        return empty(*args, **kwargs)

    monkeypatch.setattr(api.torch, "empty", no_scratch)
    got = adjoint()
    assert refused
    assert all(torch.equal(a, b) for a, b in zip(usual, got))
    psf.close(); mix.close()
