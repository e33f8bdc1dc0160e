"""L-BFGS with one to five pairs: a wave per tile for one and two, the new pair
stored by the pass over S up to four, at tile counts about what a workgroup
and the grid take, with the ring wrapping."""
import numpy as np
import pytest

from paper_2406_08646_amd import workloads as W
from gpu_util import bits, dev, host, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("n", [1, 127, 129, 4 * 128, 4 * 128 + 1, 5 * 128 + 64, 512 * 4 * 128 + 3,
                               4096 * 128 - 1, 2048 * 4 * 128 + 129])
def test_few_pairs(orc, n, m):
    """After every push the product of a stored pair and of a pair stored with
    the apply is the oracle's within the rounding of its dot products, and the
    same bits."""
    spx = require_gpu()
    pushes = m + 2
    print(f"lbfgs few n={n} m={m}", flush=True)
    S, Y, g, h0 = W.lbfgs_history(n, pushes, seed=n + m)
    pairs = [(dev(np.ascontiguousarray(S[:, k])), dev(np.ascontiguousarray(Y[:, k])))
             for k in range(pushes)]
    gd, hd = dev(g), dev(h0)
    one, fused = spx.lbfgs_create(n, m), spx.lbfgs_create(n, m)
    for k, (s, y) in enumerate(pairs):
        h = hd if k % 2 else None
        one.update(s, y)
        p = host(one.apply(gd, h))
        assert np.array_equal(bits(p), bits(host(fused.update_apply(s, y, gd, h))))
        lo = max(0, k + 1 - m)
        ref = orc.lbfgs_dense(S[:, lo:k + 1], Y[:, lo:k + 1], g, h0 if k % 2 else np.ones(n))
        err = np.linalg.norm(p - ref) / np.linalg.norm(ref)
        assert err <= max(1e-12, 2.2e-16 * n), (k, err)
