"""A plan's rays per wave: installed, the launch chooses them (0); a plan that names 64, 32 or 16 runs
and reports that many.  Wide tiles and partial refills of waves of 64 rays give the same images bit for
bit as the installed plan, for every integrator and with the optical-depth-aware step."""
import numpy as np
import pytest

import synthetic as S

pytestmark = pytest.mark.gpu


@pytest.fixture
def R():
    from paper_1801_10452_amd import raptor
    return raptor


def test_the_plan_says_what_runs(R):
    ctx = R.Context(0)
    for n_nu in (1, 4, 8, 24):
        for prec in (R.F32, R.F64):
            got = R.get_plan(ctx, n_nu, prec)
            assert got.rays_per_wave == 0
            made = R.make_plan()
            for f in ("threads", "blocks_per_cu", "refill_threshold", "tile_width", "rays_per_wave"):
                assert getattr(made, f) == getattr(got, f)
    # 24 frequencies: the rows of a wave's rays fill its LDS, so the rays set how many groups fit
    groups = []
    for rays in (64, 32, 16, 0):
        R.set_plan(ctx, 24, R.F32, R.make_plan(rays_per_wave=rays, tile_width=8))
        plan = R.get_plan(ctx, 24, R.F32)
        assert plan.rays_per_wave == rays
        groups.append(R.kernel_info(ctx, 24, R.F32, plan)["blocks_per_cu"])
    assert groups[0] < groups[1] <= groups[2] and groups[3] == groups[2]
    ctx.close()


PLANS = [dict(refill_threshold=1), dict(refill_threshold=8, tile_width=16), dict(refill_threshold=32, tile_width=64),
         dict(tile_width=32, min_waves_per_simd=3), dict(tile_width=64, threads=64, refill_threshold=16),
         dict(blocks_per_cu=1, min_waves_per_simd=1, tile_width=16), dict(blocks_per_cu=1, threads=64, refill_threshold=3)]


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("integ,n_nu,tau", [("RK4", 1, 0.0), ("RK4", 4, 0.0), ("RK4", 12, 0.0), ("RK2", 4, 0.0),
                                            ("VERLET", 1, 0.0), ("VERLET", 4, 0.3), ("RK4", 4, 0.3)])
def test_plans_of_64_rays_give_the_same_images(R, prec, integ, n_nu, tau):
    ctx = R.Context(0)
    # ragged for every tile; several tiles for a wave when one work-group runs per compute unit
    cams = [S.Camera(spin=0.9375, incl_deg=60.0, nx=101, ny=67), S.Camera(spin=0.9375, incl_deg=20.0, nx=9, ny=130)] * 12
    gh = ctx.upload_grid(S.make_grid(64, 64, a_gen=0.9375, dtype=np.float32))
    nu = list(np.geomspace(22e9, 1e12, n_nu))
    tp = R.F32 if prec == "f32" else R.F64
    opts = R.default_opts(transfer_prec=tp, integrator=getattr(R, integ), tau_step=tau)
    ref, ref_flux, ref_st = ctx.trace_batch(cams, [gh] * len(cams), nu, opts)
    assert ref.max() > 0
    for pl in PLANS:
        R.set_plan(ctx, n_nu, tp, R.make_plan(rays_per_wave=64, **pl))
        img, flux, st = ctx.trace_batch(cams, [gh] * len(cams), nu, opts)
        assert np.array_equal(img, ref) and np.array_equal(flux, ref_flux), pl
        assert (st.rays, st.ray_steps, st.samples) == (ref_st.rays, ref_st.ray_steps, ref_st.samples), pl
    ctx.close()
