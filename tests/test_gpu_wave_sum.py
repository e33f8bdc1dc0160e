"""The order of a workgroup's sums: the per-workgroup partials of the
bandwidth-reference read kernel, one pair of values per thread, bitwise
against the butterfly (lane l adds lane l ^ 32, then l ^ 16, ... l ^ 1) and
the waves added in order."""
import numpy as np
import pytest

from gpu_util import bits, dev, host, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed", [0, 1])
def test_wave_sum_is_the_butterfly(seed):
    spx = require_gpu()
    rng = np.random.default_rng(seed)
    blocks = 2048
    x = rng.uniform(-1, 1, blocks * 512) * 2.0 ** rng.integers(-30, 31, blocks * 512)
    s = x.reshape(blocks, 4, 64, 2)
    s = s[..., 0] + s[..., 1]
    lane = np.arange(64)
    for d in (32, 16, 8, 4, 2, 1):
        s = s + s[..., lane ^ d]
    want = np.zeros(blocks)
    for w in range(4):
        want = want + s[:, w, 0]
    assert np.array_equal(bits(host(spx.stream_sum(dev(x)))), bits(want))
