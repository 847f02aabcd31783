"""The network calls on host arrays share one scratch per context: results at ragged sizes, after a
larger call and beyond what the scratch keeps, equal those of a fresh context, and the closure's are
the forward pass scaled back and cut off, formed here in double."""
import numpy as np
import pytest

import synthetic as S

pytestmark = pytest.mark.gpu

LO, HI = np.float32([-4.605170185988091, -2.302585092994046, -0.999]), np.float32([18.420680743952367, 4.605170185988092, 0.999])


@pytest.mark.parametrize("n", [1, 63, 257, 4097, 1700000])
@pytest.mark.parametrize("form", ["MLP_SPLIT", "MLP_F32"])
def test_net_calls(n, form):
    from paper_1801_10452_amd import raptor as R
    if form == "MLP_F32" and n > 5000:
        pytest.skip("the reference form is slow")
    form = getattr(R, form)
    raw = S.mlp_samples(n, seed=5).astype(np.float32)
    x = 2.0 * (raw - LO) / (HI - LO) - np.float32(1.0)
    fresh, used = R.Context(0), R.Context(0)
    for c in (fresh, used):
        R.mlp_init(c, 7)
    big = S.mlp_samples(9001, seed=6).astype(np.float32)
    R.mlp_closure(used, big)
    R.mlp_backward(used, big, np.ones((9001, 2), np.float32))
    y = R.mlp_forward(fresh, x, form)
    net, exact = R.mlp_closure(fresh, raw, form)
    net2, exact2 = R.mlp_closure(used, raw, form)
    assert np.array_equal(net, net2) and np.array_equal(exact, exact2)
    assert np.array_equal(y, R.mlp_forward(used, x, form))
    if n <= 9001:
        dy = np.ones((n, 2), np.float32)
        assert np.array_equal(R.mlp_backward(fresh, x, dy), R.mlp_backward(used, x, dy))
    r = raw.astype(np.float64)
    t = np.cbrt(np.exp(r[:, 0]) / ((2.0 / 9.0) * np.exp(2.0 * r[:, 1]) * np.sqrt(1.0 - r[:, 2] ** 2)))
    want = y.astype(np.float64) * [6.0, 9.0] + [4.0, -6.5] - t[:, None]
    # three float roundings, of the product, of the sum and of the result
    tol = 3 * 2.0 ** -24 * (np.abs(y) * [6.0, 9.0] + [4.0, 6.5] + t[:, None])
    assert (np.abs(net - want) <= tol).all()
    fresh.close()
    used.close()
