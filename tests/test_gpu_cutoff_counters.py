"""The counters of a call with the optical-depth cut-off hold what the rays took up to their stops,
however their samples were queued: the same as with every sample evaluated before its ray's next step
(an optical-depth-aware step that limits nothing), in a batch of copies as many times the single
image's, and where the oracle counts them, the oracle's.  Frequency counts of one evaluation group
and of several, whose rounds may evaluate a group twice."""
import math

import numpy as np
import pytest

import synthetic as S
from tests.gpu_common import oracle_opts, rel_err

pytestmark = pytest.mark.gpu

CUT = dict(tau_cutoff=math.log(1000.0))
COUNTERS = ("rays", "ray_steps", "samples", "n_pole", "n_opaque", "n_zamo_fallback", "n_mlp_fallback",
            "n_mlp_dropped")


def counters(st):
    return {k: getattr(st, k) for k in COUNTERS}


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("closure,n_nu", [("EXACT", 1), ("EXACT", 4), ("EXACT", 6), ("EXACT", 24), ("MLP", 1),
                                          ("MLP", 3), ("MLP", 5), ("MLP", 12)])
def test_counters_of_stopped_rays(orc, prec, closure, n_nu):
    """a = 0 on Keplerian orbits, which turn superluminal inside r = 3.  The second camera looks from 3
    degrees off the axis, which the rays of its middle column (no angular momentum) run along and
    cross: their steps hang on the last bit, so that the oracle counts only the first camera's."""
    from paper_1801_10452_amd import raptor as R
    ctx = R.Context(0)
    R.mlp_init(ctx, 7)
    kw = dict(transfer_prec=R.F32 if prec == "f32" else R.F64, closure=getattr(R, "CLOSURE_" + closure), **CUT)
    # where the torus is thick: the exact closure needs lower frequencies than the random network
    lo, hi = (5e8, 3e9) if closure == "EXACT" else (1e9, 2e10)
    nu = list(np.random.RandomState(1).permutation(np.geomspace(lo, hi, n_nu))) if n_nu > 1 else [0.4 * hi]
    cams = [S.Camera(spin=0.0, incl_deg=60.0, nx=24, ny=23, fov_half=8.0),
            S.Camera(spin=0.0, incl_deg=3.0, nx=31, ny=17, fov_half=9.0)]
    g = [S.make_grid(48, 40, a_gen=0.0, dtype=np.float64, r_out=50.0),
         S.make_grid(48, 40, a_gen=0.0, dtype=np.float64, r_in=2.0, r_out=15.0)]
    h = [ctx.upload_grid(x) for x in g]
    total = dict.fromkeys(COUNTERS, 0)
    one = []
    for cam, grid, gh in zip(cams, g, h):
        opts = R.default_opts(**kw)
        img, _, st = ctx.trace_spectrum(cam, gh, nu, opts)
        each, _, st1 = ctx.trace_spectrum(cam, gh, nu, R.default_opts(tau_step=1e30, **kw))
        print(f"[counters {prec} {closure} {n_nu}] {counters(st)}", flush=True)
        assert counters(st) == counters(st1)
        assert rel_err(img, each).max() <= (1e-12 if prec == "f64" else 1e-6)
        if closure == "EXACT" and prec == "f64" and cam is cams[0]:
            _, _, info = orc.trace_image(cam, orc.GridHandle(grid), oracle_opts(orc, opts), nu)
            assert (st.ray_steps, st.samples) == (info[:, 1].sum(), info[:, 2].sum())
        one.append(img.ravel())
        for k in COUNTERS:
            total[k] += getattr(st, k)
    assert total["n_opaque"] > 0 and total["n_pole"] > 0 and total["n_zamo_fallback"] > 0
    if closure == "MLP":
        assert total["n_mlp_fallback"] > 0
    for n in (1, 12, 150):
        imgs, _, st = ctx.trace_batch(cams * n, h * n, nu, R.default_opts(**kw))
        assert np.array_equal(imgs.reshape(n, -1), np.broadcast_to(np.concatenate(one), (n, one[0].size + one[1].size)))
        assert counters(st) == {k: n * v for k, v in total.items()}, n
    ctx.close()
