"""The waves' sample ring at every number of rays per wave a launch takes by itself (64, 32, 16, 8 or
4, by the rays and frequencies of the launch): a batch of copies of one small image gives each copy
bit for bit as a call of that image alone, which the oracle checks; the batch sizes lie in each
class.  Frequency counts at the edges of the evaluation groups and of the kernel's classes; also
with the optical-depth cut-off and the optical-depth-aware step, which limit what the ring holds."""
import math

import numpy as np
import pytest

import synthetic as S
from tests.gpu_common import oracle_opts, rel_err, report

pytestmark = pytest.mark.gpu

COPIES = [8, 24, 100, 420]   # of 32 x 31 rays: 8, 16, 32 and 64 rays per wave with one frequency


@pytest.fixture(scope="module")
def R():
    from paper_1801_10452_amd import raptor
    return raptor


@pytest.fixture(scope="module")
def ctx(R):
    c = R.Context(0)
    yield c
    c.close()


MODES = {"plain": {}, "cutoff": dict(tau_cutoff=math.log(1000.0)),
         "tau_step": dict(tau_cutoff=math.log(1000.0), tau_step=0.2)}
MODES.update(cutoff_down=MODES["cutoff"], cutoff_mixed=MODES["cutoff"])


def frequencies(n_nu, mode):
    """The cut-off needs rays opaque at every frequency: low ones, where the torus is thick.  Mixed:
    shuffled, and up to where only the innermost rays are opaque, so that the frequency that decides
    lies in any group of the evaluation."""
    if mode == "plain":
        return list(np.geomspace(5e9, 1e13, n_nu))
    nu = np.geomspace(1e9, 7e9 if mode == "cutoff_mixed" else 3e9, n_nu)
    if mode == "cutoff_mixed":
        nu = np.random.RandomState(1).permutation(nu)
    return list(nu[::-1] if mode == "cutoff_down" else nu)


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n_nu,mode", [(1, "plain"), (1, "cutoff"), (1, "tau_step"), (3, "plain"), (3, "cutoff"),
                                       (4, "tau_step"), (5, "plain"), (5, "cutoff"), (6, "cutoff_mixed"),
                                       (8, "cutoff_down"), (9, "cutoff"), (12, "tau_step"), (17, "plain"),
                                       (24, "cutoff_mixed"), (27, "cutoff_down"), (32, "plain"),
                                       (32, "cutoff_mixed")])
def test_rays_per_wave_of_a_launch(R, ctx, orc, prec, n_nu, mode):
    cam = S.Camera(spin=0.9375, incl_deg=60.0, nx=32, ny=31, fov_half=18.0)
    grid = S.make_grid(64, 64, a_gen=0.9375, dtype=np.float64)
    gh = ctx.upload_grid(grid)
    nu = frequencies(n_nu, mode)
    opts = R.default_opts(transfer_prec=R.F32 if prec == "f32" else R.F64, **MODES[mode])
    status = np.zeros((cam.ny, cam.nx), np.int32)
    steps = np.zeros((cam.ny, cam.nx), np.int32)
    one, flux, st = ctx.trace_spectrum(cam, gh, nu, opts, ray_status=status, ray_steps=steps)
    ref, _, ref_st = orc.trace_image(cam, orc.GridHandle(grid), oracle_opts(orc, opts), nu)
    err = rel_err(one, ref)
    report(f"ring {prec} {n_nu} {mode}", err)
    assert err.max() <= 1e-6
    if prec == "f64":
        assert (status.ravel() == ref_st[:, 0]).all() and (steps.ravel() == ref_st[:, 1]).all()
        # the counters hold what the rays took, also where the cut-off drops samples queued behind it
        assert st.ray_steps == ref_st[:, 1].sum() and st.samples == ref_st[:, 2].sum()
    if mode != "plain":
        assert st.n_opaque > 0
    for n in COPIES if mode != "tau_step" else COPIES[:2]:
        imgs, fl, bst = ctx.trace_batch([cam] * n, [gh] * n, nu, opts)
        assert np.array_equal(imgs.reshape(n, n_nu, cam.ny, cam.nx), np.broadcast_to(one, (n,) + one.shape)), n
        assert (fl == flux).all()
        assert (bst.rays, bst.ray_steps, bst.samples, bst.n_opaque) == tuple(
            n * v for v in (st.rays, st.ray_steps, st.samples, st.n_opaque)), n
    ctx.release_grid(gh)


@pytest.mark.parametrize("n_nu", [1, 3, 6, 20])
def test_learned_closure_rays_per_wave(R, ctx, n_nu):
    cam = S.Camera(spin=0.5, incl_deg=50.0, nx=32, ny=31)
    gh = ctx.upload_grid(S.make_grid(64, 64, a_gen=0.5, dtype=np.float32))
    R.mlp_init(ctx)
    nu = list(np.geomspace(2e10, 1e12, n_nu))
    opts = R.default_opts(transfer_prec=R.F32, closure=R.CLOSURE_MLP)
    one, flux, st = ctx.trace_spectrum(cam, gh, nu, opts)
    assert np.isfinite(one).all() and one.max() > 0
    for n in (6, 30, 140):
        imgs, fl, bst = ctx.trace_batch([cam] * n, [gh] * n, nu, opts)
        assert np.array_equal(imgs.reshape(n, n_nu, cam.ny, cam.nx), np.broadcast_to(one, (n,) + one.shape)), n
        assert (bst.samples, bst.n_mlp_fallback, bst.n_mlp_dropped) == tuple(
            n * v for v in (st.samples, st.n_mlp_fallback, st.n_mlp_dropped))
    ctx.release_grid(gh)


def test_grids_of_different_radial_range(R, ctx, orc):
    """Two grids whose radial ranges differ in one batch: each ray tests its own grid's range."""
    g1 = S.make_grid(48, 40, a_gen=0.5, dtype=np.float64, r_out=50.0)
    g2 = S.make_grid(48, 40, a_gen=0.5, dtype=np.float64, r_in=2.0, r_out=20.0)
    h = [ctx.upload_grid(g1), ctx.upload_grid(g2)]
    cams = [S.Camera(0.5, 60.0, 17, 9), S.Camera(0.5, 60.0, 17, 9)]
    imgs, _, _ = ctx.trace_batch(cams, h, [230e9])
    for k, g in enumerate((g1, g2)):
        ref, _, _ = orc.trace_image(cams[k], orc.GridHandle(g), oracle_opts(orc, R.default_opts()), [230e9])
        assert rel_err(imgs[k * 153:(k + 1) * 153].reshape(9, 17), ref[0]).max() <= 1e-6
    for x in h:
        ctx.release_grid(x)
