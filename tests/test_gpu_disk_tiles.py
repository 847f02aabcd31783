"""The thin-disk kernel's tiles (8 x 8 pixels) at ragged image sizes and for each integrator, and the
line profile's chunks and groups of bins, against the oracle: identical status and step counts, pixels
within 1e-6, the binning of the same pixels to the rounding of its sums."""
import numpy as np
import pytest

import synthetic as S
from tests.gpu_common import oracle_opts, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,n_bins,integ,eps", [(1, 1, 1, "RK4", 0.05), (7, 9, 17, "RK2", 0.05),
                                                    (65, 3, 300, "VERLET", 0.05), (8, 130, 16, "RK4", 0.1),
                                                    (93, 88, 33, "RK4", 0.05)])
def test_ragged_disk_images(orc, nx, ny, n_bins, integ, eps):
    from paper_1801_10452_amd import raptor as R
    ctx = R.Context(0)
    cam = S.Camera(spin=0.7, incl_deg=70.0, nx=nx, ny=ny, fov_half=14.0)
    opts = R.default_opts(integrator=getattr(R, integ), eps=eps)
    status = np.zeros((ny, nx), np.int32)
    steps = np.zeros((ny, nx), np.int32)
    I, g, prof, st = ctx.trace_disk(cam, opts, 15.0, n_bins, 0.0, 2.0, ray_status=status, ray_steps=steps)
    og, oI, ost = orc.trace_disk_image(cam, oracle_opts(orc, opts), 15.0)
    assert np.array_equal(status.ravel(), ost[:, 0]) and np.array_equal(steps.ravel(), ost[:, 1])
    assert st.ray_steps == ost[:, 1].sum() and st.samples == (ost[:, 0] == orc.DISK).sum()
    assert rel_err(g, og).max() <= 1e-6 and rel_err(I, oI).max() <= 1e-6
    assert np.allclose(prof, orc.disk_profile(cam, g, I, n_bins, 0.0, 2.0), rtol=1e-12, atol=0)
    ctx.close()
