"""The thin-disk kernel's two forms of the RK4 step (angles chained through short rotations up to eps =
0.0625, full-size shifts beyond it or where a rotation is too large) against the oracle, from a camera near
the plane's pole and one at 60 degrees: identical status and step counts, pixels within 1e-6."""
import numpy as np
import pytest

import synthetic as S
from tests.gpu_common import oracle_opts, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eps", [0.0125, 0.0625, 0.0626, 0.25])
@pytest.mark.parametrize("spin,incl", [(0.9375, 60.0), (-0.9, 4.0)])
def test_disk_step_forms_match_the_oracle(orc, eps, spin, incl):
    from paper_1801_10452_amd import raptor as R
    ctx = R.Context(0)
    cam = S.Camera(spin=spin, incl_deg=incl, nx=18, ny=18, fov_half=12.0)
    opts = R.default_opts(eps=eps, max_steps=100000)
    status = np.zeros((cam.ny, cam.nx), np.int32)
    steps = np.zeros((cam.ny, cam.nx), np.int32)
    I, g, _, _ = ctx.trace_disk(cam, opts, 20.0, 32, 0.0, 2.0, ray_status=status, ray_steps=steps)
    og, oI, ost = orc.trace_disk_image(cam, oracle_opts(orc, opts), 20.0)
    assert np.array_equal(status.ravel(), ost[:, 0]) and np.array_equal(steps.ravel(), ost[:, 1])
    assert rel_err(g, og).max() <= 1e-6 and rel_err(I, oI).max() <= 1e-6
    ctx.close()
