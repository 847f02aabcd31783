"""The rays per wave that a launch takes by itself, against plans that name them: many small images, whose
waves run out of lanes long before they run out of tiles, and images around one and a third rounds of
tiles.  The launch's own choice is no more than 1.15 times as slow as the faster of 64 and 32 rays, and its
images are theirs bit for bit.  The cut-off with many frequencies against the same call with an
optical-depth-aware step that limits nothing: no slower, the same images and counters."""
import math

import numpy as np
import pytest

import synthetic as S

pytestmark = pytest.mark.gpu


def fastest(R, ctx, cams, gh, nu, opts, plan=None):
    prec = opts.transfer_prec
    own = R.get_plan(ctx, len(nu), prec)
    if plan is not None:
        own_rays = own.rays_per_wave
        own.rays_per_wave = plan
        R.set_plan(ctx, len(nu), prec, own)
    runs = [ctx.trace_batch(cams, [gh] * len(cams), nu, opts) for _ in range(8)]
    if plan is not None:
        own.rays_per_wave = own_rays
        R.set_plan(ctx, len(nu), prec, own)
    return min(r[2].kernel_ms for r in runs), runs[-1][0]


@pytest.mark.parametrize("nx,ny,images,n_nu,prec,cut", [(32, 31, 100, 5, "F32", True), (32, 31, 100, 8, "F64", False),
                                                        (64, 40, 24, 12, "F32", True), (64, 64, 16, 6, "F32", False),
                                                        (540, 540, 1, 12, "F32", False), (600, 380, 1, 8, "F64", False)])
def test_own_choice_is_no_slower(nx, ny, images, n_nu, prec, cut):
    from paper_1801_10452_amd import raptor as R
    ctx = R.Context(0)
    gh = ctx.upload_grid(S.make_grid(128, 128, a_gen=0.9375, dtype=np.float32))
    cams = [S.Camera(spin=0.9375, incl_deg=60.0, nx=nx, ny=ny)] * images
    nu = list(np.geomspace(1e9, 7e9, n_nu)) if cut else list(np.geomspace(2e10, 1e12, n_nu))
    opts = R.default_opts(transfer_prec=getattr(R, prec), tau_cutoff=math.log(1000.0) if cut else 0.0)
    ms, img = fastest(R, ctx, cams, gh, nu, opts)
    named = {rays: fastest(R, ctx, cams, gh, nu, opts, rays) for rays in (64, 32)}
    print(f"[rays per wave] {images} x {nx} x {ny}, {n_nu} frequencies: {ms:.2f} ms, named "
          f"{ {k: round(v[0], 2) for k, v in named.items()} }", flush=True)
    for rays, (_, other) in named.items():
        assert np.array_equal(img, other), rays
    assert ms <= 1.15 * min(v[0] for v in named.values())
    ctx.close()


@pytest.mark.parametrize("nx,ny,images,n_nu,prec,closure,cut", [
    (64, 40, 24, 32, "F32", "EXACT", True), (32, 31, 20, 16, "F64", "EXACT", True), (13, 7, 1, 13, "F64", "EXACT", True),
    (230, 230, 1, 24, "F64", "K2_PAPER", True), (64, 40, 24, 17, "F32", "CONST", False),
    (512, 512, 1, 32, "F32", "CONST", False)])
def test_cutoff_with_many_frequencies(nx, ny, images, n_nu, prec, closure, cut):
    from paper_1801_10452_amd import raptor as R
    ctx = R.Context(0)
    gh = ctx.upload_grid(S.make_grid(128, 128, a_gen=0.9375, dtype=np.float32))
    cams = [S.Camera(spin=0.9375, incl_deg=60.0, nx=nx, ny=ny)] * images
    nu = list(np.geomspace(1e9, 7e9, n_nu))
    kw = dict(transfer_prec=getattr(R, prec), closure=getattr(R, "CLOSURE_" + closure), const_j=1e-20, const_alpha=1e-14,
              tau_cutoff=math.log(1000.0) if cut else 0.0)
    ms, img = fastest(R, ctx, cams, gh, nu, R.default_opts(**kw))
    each_ms, each = fastest(R, ctx, cams, gh, nu, R.default_opts(tau_step=1e30, **kw))
    print(f"[many frequencies] {images} x {nx} x {ny}, {n_nu} frequencies, {closure}: {ms:.2f} ms, each sample after its "
          f"step {each_ms:.2f}", flush=True)
    assert np.array_equal(img, each)
    st, st1 = (ctx.trace_batch(cams, [gh] * images, nu, R.default_opts(**k))[2] for k in (kw, dict(kw, tau_step=1e30)))
    for f in ("rays", "ray_steps", "samples", "n_pole", "n_opaque", "n_zamo_fallback"):
        assert getattr(st, f) == getattr(st1, f), f
    assert ms <= 1.15 * each_ms
    ctx.close()


def test_cutoff_route_in_graphs_and_without_allocation():
    """The same launch direct, replayed as a graph between other launches, without allocation, and under
    plans that name 64, 32 and 16 rays and each number of waves: the same images bit for bit."""
    import torch
    from paper_1801_10452_amd import raptor as R
    ctx = R.Context(0)
    gh = ctx.upload_grid(S.make_grid(64, 64, a_gen=0.9375, dtype=np.float32))
    cams = [S.Camera(spin=0.9375, incl_deg=60.0, nx=37, ny=21), S.Camera(spin=0.9375, incl_deg=30.0, nx=9, ny=40)]
    nu = list(np.geomspace(1e9, 7e9, 17))
    kw = dict(transfer_prec=R.F32, tau_cutoff=math.log(1000.0))
    ref, ref_flux, st = ctx.trace_batch(cams, [gh] * 2, nu, R.default_opts(**kw))
    assert st.n_opaque > 0
    images = torch.empty(ref.size, dtype=torch.float64, device="cuda")
    flux = torch.empty(2 * 17, dtype=torch.float64, device="cuda")
    for k in range(3):
        images.zero_()
        ctx.trace_batch(cams, [gh] * 2, nu, R.default_opts(mem=R.MEM_DEVICE, launch=R.LAUNCH_GRAPH, **kw), images, flux)
        assert np.array_equal(images.cpu().numpy(), ref) and np.array_equal(flux.cpu().numpy(), ref_flux.ravel()), k
        ctx.trace_spectrum(cams[0], gh, nu[:1 + k], R.default_opts(transfer_prec=R.F32))
    images.zero_()
    R.trace_batch_noalloc(ctx, cams, [gh] * 2, nu, R.default_opts(mem=R.MEM_DEVICE, **kw), images, flux)
    assert np.array_equal(images.cpu().numpy(), ref) and np.array_equal(flux.cpu().numpy(), ref_flux.ravel())
    for rays in (0, 16, 32, 64):
        for waves in (1, 2, 3):
            R.set_plan(ctx, 17, R.F32, R.make_plan(rays_per_wave=rays, min_waves_per_simd=waves))
            got, got_flux, _ = ctx.trace_batch(cams, [gh] * 2, nu, R.default_opts(**kw))
            assert np.array_equal(got, ref) and np.array_equal(got_flux, ref_flux), (rays, waves)
    ctx.close()
