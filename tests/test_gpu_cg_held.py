"""CG with the matrix and vectors held in one compute unit: the persistent
batched form bitwise against persistent BiCG (which walks memory; on
symmetric systems the two have the same recurrences and sums), and the
single-system form against the oracle, at the edges of their sizes."""
import math

import numpy as np
import pytest

from paper_2406_08646_amd import workloads as W
from gpu_util import assemble, bits, dev, host, require_gpu

pytestmark = pytest.mark.gpu


def five_point(L, rng):
    c = rng.uniform(1.0, 2.0, 2 * L * (L - 1) + 4 * L)
    nh = L * (L - 1)
    return W.five_point_system(L, c[:nh], c[nh:2 * nh], c[2 * nh:])


def seven_point(L, rng):
    """The 3-D counterpart, from edges, with 0.05 on the diagonal."""
    k = np.arange(L**3).reshape(L, L, L)
    i, j, v = [k.ravel()], [k.ravel()], [np.full(L**3, 0.05)]
    for a, b in ((k[1:], k[:-1]), (k[:, 1:], k[:, :-1]), (k[:, :, 1:], k[:, :, :-1])):
        a, b, c = a.ravel(), b.ravel(), rng.uniform(1.0, 2.0, a.size)
        i += [a, a, b, b]
        j += [a, b, a, b]
        v += [c, -c, -c, c]
    return W.CooProblem(n=L**3, i=np.concatenate(i).astype(np.int32),
                        j=np.concatenate(j).astype(np.int32), v=np.concatenate(v))


def q1(N, dim, rng):
    return W.q1_poisson(N, dim, kappa=np.exp(rng.standard_normal(N**dim)))


# the largest systems: 256 threads with rows of 5, 9 and 27 entries, then 512
# standing for 1024 with 5, 7 and (x and D^-1 in LDS) 5
@pytest.mark.parametrize("kind,sides", [("five", [1, 2, 16, 31, 32]), ("q2", [1, 5, 15, 16, 31]),
                                        ("q3", [1, 2, 6, 9]), ("five", [3, 33, 45, 63, 64]),
                                        ("seven", [2, 11, 15, 16]), ("five", [32, 65, 72, 78])])
def test_held_batch_is_persistent_bicg_bit_for_bit(kind, sides):
    spx = require_gpu()
    rng = np.random.default_rng(len(sides) + sides[-1])
    make = {"five": lambda L: five_point(L, rng), "seven": lambda L: seven_point(L, rng),
            "q2": lambda L: q1(L, 2, rng), "q3": lambda L: q1(L, 3, rng)}[kind]
    probs = [make(L) for L in sides]
    batch = spx.batch_create([assemble(spx, p) for p in probs])
    b = dev(rng.uniform(-1, 1, batch.total))
    x0 = dev(rng.uniform(-1, 1, batch.total))
    for args in (dict(rtol=1e-10), dict(rtol=1e-10, maxit=7), dict(rtol=0.0, maxit=0)):
        xc, ic, rc, sc = batch.batch_cg(b, x=x0.clone(), persistent=1, **args)
        xb, ib, rb, sb = batch.batch_bicg(b, x=x0.clone(), persistent=1, **args)
        assert sc == sb and ic == ib and rc == rb
        assert np.array_equal(bits(host(xc)), bits(host(xb)))


@pytest.mark.parametrize("kind,side", [("five", 1), ("five", 16), ("five", 17), ("five", 32),
                                       ("five", 33), ("five", 45), ("q2", 44), ("q3", 5)])
def test_held_solve_matches_oracle(orc, kind, side):
    spx = require_gpu()
    rng = np.random.default_rng(side)
    prob = five_point(side, rng) if kind == "five" else q1(side, int(kind[1]), rng)
    b, x0 = rng.uniform(-1, 1, prob.n), rng.uniform(-1, 1, prob.n)
    ref = orc.assemble(prob.n, prob.i, prob.j, prob.v)
    A = assemble(spx, prob)
    ores = orc.pcg(ref, b, 1e-10)
    oref = orc.pcg(ref, b, 1e-13)
    res = A.cg_solve(dev(b), rtol=1e-10)
    assert res.status == 0 and res.relres <= 1e-10 * (1 + 1e-3)
    assert abs(res.iters - ores.iters) <= max(2, math.ceil(0.01 * ores.iters))
    again = A.cg_solve_transpose(dev(b), x=dev(x0), rtol=1e-10)
    assert again.status == 0 and again.relres <= 1e-10 * (1 + 1e-3)
    # both within the residuals' bound of the same solution
    D = np.zeros((prob.n, prob.n))
    D[np.repeat(np.arange(prob.n), np.diff(ref.rowptr)), ref.col] = ref.val
    lam = np.linalg.eigvalsh(D)[0]
    tol = 2 * 1.001e-10 * np.linalg.norm(b) / lam
    assert np.linalg.norm(host(res.x) - oref.x) <= tol
    assert np.linalg.norm(host(again.x) - oref.x) <= tol
    r = A.cg_solve(dev(b), rtol=1e-14, maxit=1)
    assert r.iters == 1 and (r.status == spx.NOT_CONVERGED or prob.n == 1)


def test_held_solve_statuses():
    spx = require_gpu()
    k = np.arange(300, dtype=np.int32)
    for d, status in ((np.where(k == 299, 0.0, 2.0), spx.ZERO_DIAGONAL),
                      (np.where(k == 299, -1.0, 1.0), spx.BREAKDOWN)):
        Z = spx.coo_preallocate(300, dev(k), dev(k))
        Z.set_values_coo(dev(d))
        r = Z.cg_solve(dev(np.where(k == 299, 1.0, 0.0)), rtol=1e-8)
        assert r.status == status and r.iters == 0
    # the last rows empty: no entry to load for them
    E = spx.coo_preallocate(300, dev(k[:290]), dev(k[:290]))
    E.set_values_coo(dev(np.ones(290)))
    assert E.cg_solve(dev(np.ones(300)), rtol=1e-8).status == spx.ZERO_DIAGONAL
