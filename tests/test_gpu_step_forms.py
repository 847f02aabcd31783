"""The two forms of the RK4 step -- angles chained through short rotations, and full-size shifts,
chosen by eps (the line lies at 0.0625) and, below it, by the sizes of the angles themselves --
against the oracle: identical termination codes and step counts, pixels within 1e-6."""
import numpy as np
import pytest

import synthetic as S
from tests.gpu_common import oracle_opts, rel_err, report

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eps", [0.0125, 0.0625, 0.0626, 0.25])
@pytest.mark.parametrize("spin,incl", [(0.9375, 60.0), (-0.9, 4.0)])
def test_step_forms_match_the_oracle(orc, eps, spin, incl):
    """a = -0.9 seen from 4 degrees off the pole: rays close to the axis, whose angle offsets leave
    the short rotations' range also at a small eps."""
    from paper_1801_10452_amd import raptor as R
    ctx = R.Context(0)
    grid = S.make_grid(48, 40, a_gen=spin, dtype=np.float64)
    cam = S.Camera(spin=spin, incl_deg=incl, nx=18, ny=18, fov_half=12.0)
    opts = R.default_opts(eps=eps, max_steps=100000)
    gh = ctx.upload_grid(grid)
    status = np.zeros((cam.ny, cam.nx), np.int32)
    steps = np.zeros((cam.ny, cam.nx), np.int32)
    img, _, _ = ctx.trace_spectrum(cam, gh, [230e9], opts, ray_status=status, ray_steps=steps)
    ref, _, ref_st = orc.trace_image(cam, orc.GridHandle(grid), oracle_opts(orc, opts), [230e9])
    err = rel_err(img, ref)
    report(f"step forms eps={eps} a={spin}", err)
    assert (status.ravel() == ref_st[:, 0]).all() and (steps.ravel() == ref_st[:, 1]).all()
    assert err.max() <= 1e-6
    ctx.close()
