"""GPU limited-memory BFGS product at the edges of its tiling: 128-row tiles,
a quarter of the pairs per wave, results held over 72 tiles a workgroup, or 8
where long passes over few pairs take more workgroups."""
import numpy as np
import pytest
import torch

from paper_2406_08646_amd import workloads as W
from gpu_util import dev, host, require_gpu

pytestmark = pytest.mark.gpu


def tol(n):
    """Rounding bound of the dot products of length n (about n eps), twice."""
    return max(1e-12, 2.2e-16 * n)


@pytest.mark.parametrize("n,m,pushes", [
    (1, 1, 2), (2, 3, 2), (127, 4, 4), (128, 5, 7), (129, 16, 17), (1000, 17, 17),
    (513 * 128 + 1, 13, 14),     # more tiles than workgroups, a ragged last one
    (4096, 49, 64), (4097, 64, 64),
    (512 * 72 * 128 + 129, 9, 10),  # a workgroup's held results written twice
    (4095 * 128, 8, 8), (4096 * 128 - 1, 8, 9),  # either side of the eight-workgroup form
    (2048 * 8 * 128 + 130, 3, 4)])  # and its held results written twice
@pytest.mark.parametrize("offset", [0, 1])
def test_lbfgs_tiles(orc, n, m, pushes, offset):
    """p against the oracle after the pushes, with every vector on or 8 bytes
    off a 16-byte boundary; nothing past p's end is written."""
    spx = require_gpu()
    print(f"lbfgs tiles n={n} m={m} pushes={pushes} offset={offset}", flush=True)
    S, Y, g, h0 = W.lbfgs_history(n, pushes, seed=7 + m)

    def at(v):
        b = torch.zeros(n + offset + 2, dtype=torch.float64, device="cuda")
        b[offset:offset + n] = dev(v)
        return b[offset:offset + n]

    L = spx.lbfgs_create(n, m)
    for k in range(pushes):
        L.update(at(np.ascontiguousarray(S[:, k])), at(np.ascontiguousarray(Y[:, k])))
    lo = max(0, pushes - m)
    for h in (h0, None):
        ref = orc.lbfgs_dense(S[:, lo:], Y[:, lo:], g, h if h is not None else np.ones(n))
        buf = torch.full((n + offset + 2,), 7.0, dtype=torch.float64, device="cuda")
        L.apply(at(g), at(h) if h is not None else None, p=buf[offset:offset + n])
        b = host(buf)
        err = np.linalg.norm(b[offset:offset + n] - ref) / np.linalg.norm(ref)
        assert err <= tol(n), err
        assert np.all(b[:offset] == 7.0) and np.all(b[offset + n:] == 7.0)


@pytest.mark.parametrize("m", [1, 2])
def test_lbfgs_diagonal_without_reciprocal(orc, m):
    """s.y so small that 1 / (s.y) overflows: the quotients are still those of
    the division.  s.y near 4e-310 keeps a relative 1.3e-14."""
    spx = require_gpu()
    n = 4
    S, Y = np.full((n, 1), 1e-155), np.full((n, 1), 1e-155)
    g, h0 = np.full(n, 1e-155), np.full(n, 0.5)
    L = spx.lbfgs_create(n, m)
    L.update(dev(np.ascontiguousarray(S[:, 0])), dev(np.ascontiguousarray(Y[:, 0])))
    p = host(L.apply(dev(g), dev(h0))) * 1e155
    ref = orc.lbfgs_dense(S, Y, g, h0) * 1e155
    assert np.all(np.isfinite(ref)) and np.linalg.norm(p - ref) <= 1e-12 * np.linalg.norm(ref)
