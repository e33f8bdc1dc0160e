"""L-BFGS products that overflow: infinities reach the rows that the formula
gives them, whether or not the last tile of rows is whole."""
import numpy as np
import pytest

from gpu_util import dev, host, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 3, 127, 128, 129, 1000])
@pytest.mark.parametrize("with_h0", [False, True])
def test_overflowed_product(n, with_h0):
    spx = require_gpu()
    s, y, g, h0 = np.full(n, -1.0), np.ones(n), np.zeros(n), np.full(n, 2.0)
    s[0], g[0] = 1e10, 1e300
    with np.errstate(all="ignore"):
        d = s @ y
        c = -np.inf  # s.g = 1e310
        a = (h0 if with_h0 else 1.0) * (g + y * c)
        e = (np.sum(y * a) + d * c) / d
        want = a - s * e  # not a number in row 0, -inf in the others
    H = spx.lbfgs_create(n, 1)
    for fused in (False, True):
        if fused:
            p = H.update_apply(dev(s), dev(y), dev(g), dev(h0) if with_h0 else None)
        else:
            H.update(dev(s), dev(y))
            p = H.apply(dev(g), dev(h0) if with_h0 else None)
        assert np.array_equal(host(p), want, equal_nan=True)
