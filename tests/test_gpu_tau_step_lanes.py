"""The optical-depth-aware step's rounds share each sample's frequencies among the lanes that the
step's samples leave free: one to 64 samples a round, frequency counts that divide evenly into lanes
and groups of four and that do not, 64, 32 and 16 rays per wave, against the oracle, bit for bit the
same whatever the rays, and in a batch as each image alone."""
import math

import numpy as np
import pytest

import synthetic as S
from tests.gpu_common import oracle_opts, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n_nu,cut", [(1, False), (2, True), (3, False), (5, True), (7, False), (13, True), (17, False),
                                      (31, True), (32, False)])
def test_frequencies_shared_among_lanes(orc, prec, n_nu, cut):
    from paper_1801_10452_amd import raptor as R
    ctx = R.Context(0)
    tp = R.F32 if prec == "f32" else R.F64
    grid = S.make_grid(48, 40, a_gen=0.7, dtype=np.float64)
    gh = ctx.upload_grid(grid)
    cams = [S.Camera(spin=0.7, incl_deg=65.0, nx=13, ny=11, fov_half=14.0),
            S.Camera(spin=0.7, incl_deg=65.0, nx=3, ny=1, fov_half=6.0)]
    nu = list(np.geomspace(1e9, 4e9, n_nu)) if cut else list(np.geomspace(2e10, 1e13, n_nu))
    opts = R.default_opts(transfer_prec=tp, tau_step=0.2, tau_cutoff=math.log(1000.0) if cut else 0.0)
    one = []
    for cam in cams:
        status = np.zeros((cam.ny, cam.nx), np.int32)
        steps = np.zeros((cam.ny, cam.nx), np.int32)
        img, _, st = ctx.trace_spectrum(cam, gh, nu, opts, ray_status=status, ray_steps=steps)
        ref, _, info = orc.trace_image(cam, orc.GridHandle(grid), oracle_opts(orc, opts), nu)
        assert rel_err(img, ref).max() <= 1e-6
        if prec == "f64":
            assert (status.ravel() == info[:, 0]).all() and (steps.ravel() == info[:, 1]).all()
            assert (st.ray_steps, st.samples) == (info[:, 1].sum(), info[:, 2].sum())
        assert (st.n_opaque > 0) == cut
        one.append(img.ravel())
    for rays, w in ((64, 2), (32, 3), (16, 3)):
        R.set_plan(ctx, n_nu, tp, R.make_plan(rays_per_wave=rays, min_waves_per_simd=w))
        for n in (1, 40):
            imgs, _, _ = ctx.trace_batch(cams * n, [gh] * (2 * n), nu, opts)
            assert np.array_equal(imgs.reshape(n, -1), np.broadcast_to(np.concatenate(one),
                                                                       (n, one[0].size + one[1].size))), (rays, n)
    ctx.close()
