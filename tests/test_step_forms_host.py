"""The forms of the RK4 step on the host: rk4_try_block, which the trace kernel takes, against rk4_step and
its shifts of the angle, bit for bit; rk4_try_chained, the thin-disk kernel's, against the same to its
rounding.  Whole rays of a camera near the equator and of one four degrees off the pole, whose rays next to
the axis leave the polynomials' ranges: a form that refuses a step leaves the state as it was."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <algorithm>
#include <cmath>
#include <cstring>
#include "ks_geodesic.hpp"
// out: steps, steps the block form refused, steps the chained form refused, steps on which the block form
// differs, refused steps that changed the state, largest error of the chained form (position and wave
// vector, relative to the terms of the step) and of its sine and cosine in units of the steps taken
extern "C" void compare(double a, double incl_deg, double eps, int n, double fov, int max_steps, double* out)
{
    const rk::Spin<double> sp = rk::make_spin(a, 1.0);
    const double incl = incl_deg * M_PI / 180.0;
    const auto cam = rk::camera_frame(a, 1.0, 1e4, incl, std::sin(incl), std::cos(incl), 0.0);
    for (int i = 0; i < 7; ++i) out[i] = 0.0;
    for (int p = 0; p < n * n; ++p) {
        double y[8], s, c;
        rk::camera_ray(cam, fov * (2.0 * (p % n + 0.5) / n - 1.0), fov * (2.0 * (p / n + 0.5) / n - 1.0), y);
        rt::sincos_small(y[2], &s, &c);
        double ts = s, tc = c, since = 0.0;   // the chained form's carried sine and cosine
        for (int k = 0; k < max_steps && y[1] > 1.05 * (1.0 + std::sqrt(1.0 - a * a)) && y[1] <= 1e4; ++k) {
            const double dl = -rk::step_size(eps, y);
            double y0[8], y1[8], s1 = s, c1 = c, y2[8];
            std::memcpy(y0, y, sizeof y);
            std::memcpy(y1, y, sizeof y);
            std::memcpy(y2, y, sizeof y);
            rk::rk4_step(sp, y, dl, s, c);
            double ns, nc;
            rk::sincos_shift(y0[2], s, c, y[2], &ns, &nc);
            out[0] += 1.0;
            if (rk::rk4_try_block(sp, y1, dl, &s1, &c1))
                out[3] += std::memcmp(y, y1, sizeof y) != 0 || ns != s1 || nc != c1;
            else {
                out[1] += 1.0;
                out[4] += std::memcmp(y0, y1, sizeof y) != 0 || s1 != s || c1 != c;
            }
            double us = ts, uc = tc;
            if (rk::rk4_try_chained(sp, y2, dl, &us, &uc)) {
                double kmax = 0.0;
                for (int i = 4; i < 8; ++i) kmax = std::max(kmax, std::max(std::fabs(y0[i]), std::fabs(y[i])));
                const double move = std::fabs(dl) * kmax;
                for (int i = 0; i < 8; ++i) {
                    const double scale = i < 4 ? std::fabs(y0[i]) + move : kmax * (1.0 + move);
                    out[5] = std::max(out[5], std::fabs(y2[i] - y[i]) / scale);
                }
                since += 1.0;
                ts = us;
                tc = uc;
                // carried along the reference's angles
                double ds, dc;
                rk::sincos_shift(y2[2], ts, tc, y[2], &ds, &dc);
                ts = ds;
                tc = dc;
                out[6] = std::max(out[6], std::max(std::fabs(ts - std::sin(y[2])), std::fabs(tc - std::cos(y[2]))) /
                                              (since + 1.0));
            } else {
                out[2] += 1.0;
                out[4] += std::memcmp(y0, y2, sizeof y) != 0 || us != ts || uc != tc;
                rt::sincos_small(y[2], &ts, &tc);
                since = 0.0;
            }
            s = ns;
            c = nc;
            if (rk::reflect_pole(y)) {
                rt::sincos_small(y[2], &s, &c);
                ts = s;
                tc = c;
                since = 0.0;
            }
        }
    }
}
"""


@pytest.fixture(scope="module")
def compare(tmp_path_factory):
    from paper_1801_10452_amd.build import CSRC, HIPCC
    d = tmp_path_factory.mktemp("forms")
    (d / "forms.hip").write_text(SOURCE)
    subprocess.check_call([HIPCC, "-x", "hip", "--cuda-host-only", "-std=c++17", "-O2", "-mfma", "-fPIC", "-shared",
                           "-I" + CSRC, str(d / "forms.hip"), "-o", str(d / "forms.so")])
    f = C.CDLL(str(d / "forms.so")).compare
    f.argtypes = [C.c_double] * 3 + [C.c_int, C.c_double, C.c_int, C.POINTER(C.c_double)]
    f.restype = None

    def call(*args):
        out = (C.c_double * 7)()
        f(*args, out)
        return np.array(out)
    return call


@pytest.mark.parametrize("eps", [0.0125, 0.05, 0.0625, 0.25])
@pytest.mark.parametrize("a,incl", [(0.9375, 60.0), (-0.9, 4.0), (0.0, 85.0)])
def test_step_forms_agree(compare, a, incl, eps):
    steps, block_refused, chained_refused, differ, touched, err, angle = compare(a, incl, eps, 14, 12.0, 20000)
    print(f"[step forms a={a} i={incl} eps={eps}] {steps:.0f} steps, refused {block_refused:.0f} and "
          f"{chained_refused:.0f}, chained {err:.1e}, angle {angle:.1e} a step")
    assert steps > 5000 and differ == 0 and touched == 0
    assert chained_refused >= block_refused
    if eps == 0.25:
        assert block_refused > 0 and chained_refused > 0
    # some five hundred roundings of half a unit, of terms up to twenty times the scale
    assert err <= 500 * 2.0 ** -53 * 20
    # sine and cosine: three roundings in each of the two rotations of a step, and the reference's own
    assert angle <= 8 * 2.0 ** -53
