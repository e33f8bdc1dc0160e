"""The resident CG solve (one cooperative launch: fp64, and the fp32 inner
solve of the refinement) against the oracle at the sizes where its shares
change: one workgroup and several, a ragged last one, one, two and four rows
per thread; a pattern whose window does not fit; every status."""
import math

import numpy as np
import pytest

from paper_2406_08646_amd import workloads as W
from gpu_util import assemble, dev, host, require_gpu

pytestmark = pytest.mark.gpu


def five_point(L, seed):
    """Coefficients in [1, 2]: the smallest eigenvalue is at least the
    constant-coefficient operator's, 8 sin^2(pi / (2 (L + 1)))."""
    rng = np.random.default_rng(seed)
    c = rng.uniform(1.0, 2.0, 2 * L * (L - 1) + 4 * L)
    nh = L * (L - 1)
    prob = W.five_point_system(L, c[:nh], c[nh:2 * nh], c[2 * nh:])
    return prob, rng.uniform(-1, 1, prob.n), 8 * math.sin(math.pi / (2 * (L + 1))) ** 2


def scattered(n, seed):
    """Symmetric, eight random off-diagonal entries of size at most 1 a row
    pair, diagonal 1 above the row's absolute sum: eigenvalues at least 1,
    and a workgroup's rows touch x everywhere."""
    rng = np.random.default_rng(seed)
    i = np.repeat(np.arange(n), 4)
    j = rng.integers(0, n, 4 * n)
    v = rng.uniform(-1, 1, 4 * n)
    d = 1.0 + np.bincount(i, np.abs(v), n) + np.bincount(j, np.abs(v), n)
    k = np.arange(n)
    prob = W.CooProblem(n=n, i=np.concatenate([i, j, k]).astype(np.int32),
                        j=np.concatenate([j, i, k]).astype(np.int32), v=np.concatenate([v, v, d]))
    return prob, rng.uniform(-1, 1, n), 1.0


@pytest.mark.parametrize("case", [17, 36, 64, 181, 363, 513, "scattered"])
def test_resident_solve_matches_oracle(orc, case):
    spx = require_gpu()
    prob, b, lam = scattered(60000, 5) if case == "scattered" else five_point(case, case)
    ref = orc.assemble(prob.n, prob.i, prob.j, prob.v)
    A = assemble(spx, prob)
    ores = orc.pcg(ref, b, 1e-8)
    x0 = np.random.default_rng(1).uniform(-1, 1, prob.n)
    print(f"resident: {case} n={prob.n} oracle {ores.iters} it", flush=True)
    for start in (None, x0):
        for solve in (A.cg_solve, A.cg_solve_transpose):
            res = solve(dev(b), x=None if start is None else dev(start), rtol=1e-8)
            assert res.status == 0 and res.relres <= 1e-8 * (1 + 1e-3)
            if start is None:
                assert abs(res.iters - ores.iters) <= max(2, math.ceil(0.01 * ores.iters))
            x = host(res.x)
            err = np.linalg.norm(b - orc.spmv(ref, x)) + np.linalg.norm(b - orc.spmv(ref, ores.x))
            assert np.linalg.norm(x - ores.x) <= err / lam * (1 + 1e-6)
    om = orc.pcg_mixed(ref, b, 1e-10, 1e-4)
    m = A.cg_solve_mixed(dev(b), rtol_outer=1e-10, rtol_inner=1e-4)
    assert m.status == 0 and m.relres <= 1e-10
    assert abs(m.outer - om.outer) <= 1 and abs(m.inner - om.inner) <= max(3, 0.05 * om.inner)


def test_resident_solve_statuses():
    spx = require_gpu()
    prob, b, _ = five_point(40, 3)
    C = assemble(spx, prob)
    for maxit in (0, 1, 3):
        r = C.cg_solve(dev(b), rtol=1e-12, maxit=maxit)
        assert r.status == spx.NOT_CONVERGED and r.iters == maxit
    r = C.cg_solve(dev(np.zeros(prob.n)), rtol=1e-8)
    assert r.status == 0 and r.iters == 0 and np.all(host(r.x) == 0)
    x = host(C.cg_solve(dev(b), rtol=1e-10).x)
    r = C.cg_solve(dev(b), x=dev(x), rtol=1e-9)
    assert r.status == 0 and r.iters == 0 and np.array_equal(host(r.x), x)
    m = C.cg_solve_mixed(dev(b), maxit_outer=1, maxit_inner=2)
    assert m.status == spx.NOT_CONVERGED and m.inner == 2
    k = np.arange(1000, dtype=np.int32)
    for d, status in ((np.where(k == 700, 0.0, 2.0), spx.ZERO_DIAGONAL),
                      (np.where(k == 700, -1.0, 1.0), spx.BREAKDOWN)):
        Z = spx.coo_preallocate(1000, dev(k), dev(k))
        Z.set_values_coo(dev(d))
        r = Z.cg_solve(dev(np.where(k == 700, 1.0, 0.0)), rtol=1e-8)
        assert r.status == status and r.iters == 0
        assert Z.cg_solve_mixed(dev(np.where(k == 700, 1.0, 0.0))).status == status
    # one step on a multiple of the identity, and b reached exactly
    I = spx.coo_preallocate(1000, dev(k), dev(k))
    I.set_values_coo(dev(np.full(1000, 4.0)))
    r = I.cg_solve(dev(np.ones(1000)), rtol=1e-14)
    assert r.status == 0 and r.iters == 1 and np.all(host(r.x) == 0.25)


def test_resident_solves_from_two_threads():
    """Two handles solved at once from two threads on two streams: the
    launches take turns, each result bitwise that of the solve alone."""
    spx = require_gpu()
    import threading

    import torch

    systems = []
    for L, seed in ((150, 1), (300, 2)):
        prob, b, _ = five_point(L, seed)
        A, bd = assemble(spx, prob), dev(b)
        systems.append((A, bd, host(A.cg_solve(bd, rtol=1e-8).x)))
    torch.cuda.synchronize()
    wrong = []

    def work(A, bd, want):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            for _ in range(4):
                r = A.cg_solve(bd, rtol=1e-8)
                if r.status != 0 or not np.array_equal(r.x.cpu().numpy(), want):
                    wrong.append(r.status)

    threads = [threading.Thread(target=work, args=s) for s in systems]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
