"""The resident CG solve takes the form of the recurrences that the solve has
without it: the textbook one above 2,000,000 entries (one, two and four rows
per thread) and, with rows of more than 9 entries, up to 2048 rows; and its
statuses there."""
import math

import numpy as np
import pytest

from paper_2406_08646_amd import workloads as W
from gpu_util import assemble, bits, dev, host, require_gpu
from test_gpu_cg_resident import five_point

pytestmark = pytest.mark.gpu


def q1(N, dim, seed):
    rng = np.random.default_rng(seed)
    prob = W.q1_poisson(N, dim, kappa=np.exp(0.3 * rng.standard_normal(N**dim)))
    return prob, rng.uniform(-1, 1, prob.n)


@pytest.mark.parametrize("make", [lambda: q1(45, 3, 1), lambda: q1(489, 2, 2),
                                  lambda: five_point(641, 3)[:2]], ids=["27", "9", "5"])
def test_resident_textbook_above_two_million_entries(orc, make):
    spx = require_gpu()
    prob, b = make()
    ref = orc.assemble(prob.n, prob.i, prob.j, prob.v)
    A = assemble(spx, prob)
    assert A.nnz > 2000000 and A.get_option(spx.OPT_CG_VARIANT) == 0
    print(f"resident textbook n={prob.n} nnz={A.nnz}", flush=True)
    bd, rtol = dev(b), 1e-9
    auto = A.cg_solve(bd, rtol=rtol)
    short = A.cg_solve(bd, rtol=rtol, maxit=9)
    A.set_option(spx.OPT_CG_VARIANT, 1)
    single = A.cg_solve(bd, rtol=rtol, maxit=9)
    A.set_option(spx.OPT_CG_VARIANT, -1)
    A.set_option(spx.OPT_SMALL_SOLVE, 0)
    launches = A.cg_solve(bd, rtol=rtol)
    assert auto.status == launches.status == 0
    # the other form's rounding differs within nine iterations
    assert short.iters == single.iters == 9
    assert not np.array_equal(bits(host(short.x)), bits(host(single.x)))
    assert abs(auto.iters - launches.iters) <= max(2, math.ceil(0.01 * launches.iters))
    assert auto.relres <= rtol * (1 + 1e-3)
    assert np.linalg.norm(b - orc.spmv(ref, host(auto.x))) <= rtol * (1 + 1e-3) * np.linalg.norm(b)


@pytest.mark.parametrize("N", [6, 8, 11])  # 343 to 1728 rows of up to 27 entries
def test_resident_textbook_up_to_2048_rows(orc, N):
    spx = require_gpu()
    prob, b = q1(N, 3, N)
    ref = orc.assemble(prob.n, prob.i, prob.j, prob.v)
    A = assemble(spx, prob)
    ores = orc.pcg(ref, b, 1e-10)
    for solve in (A.cg_solve, A.cg_solve_transpose, A.cg_solve_noalloc):
        res = solve(dev(b), x=dev(np.zeros(prob.n)), rtol=1e-10)
        assert res.status == 0 and res.relres <= 1e-10 * (1 + 1e-3)
        assert abs(res.iters - ores.iters) <= 2
        D = np.zeros((prob.n, prob.n))
        D[np.repeat(np.arange(prob.n), np.diff(ref.rowptr)), ref.col] = ref.val
        tol = 2 * 1.001e-10 * np.linalg.norm(b) / np.linalg.eigvalsh(D)[0]
        assert np.linalg.norm(host(res.x) - ores.x) <= tol
    short = A.cg_solve(dev(b), rtol=1e-14, maxit=9)
    A.set_option(spx.OPT_CG_VARIANT, 1)
    assert not np.array_equal(bits(host(short.x)),
                              bits(host(A.cg_solve(dev(b), rtol=1e-14, maxit=9).x)))


def test_resident_textbook_statuses():
    """Diagonal systems whose rows also store ten zeros, so that neither the
    register-held solve nor the single-reduction form takes them."""
    spx = require_gpu()
    n = 1000
    k = np.arange(n)
    i = np.repeat(k, 11)
    j = (i + np.tile(np.arange(11), n)) % n

    def system(d):
        A = spx.coo_preallocate(n, dev(i.astype(np.int32)), dev(j.astype(np.int32)))
        A.set_values_coo(dev(np.where(i == j, d[i], 0.0)))
        return A

    unit = dev(np.where(k == 700, 1.0, 0.0))
    for d, status in ((np.where(k == 700, 0.0, 2.0), spx.ZERO_DIAGONAL),
                      (np.where(k == 700, -1.0, 1.0), spx.BREAKDOWN)):
        r = system(d).cg_solve(unit, rtol=1e-8)
        assert r.status == status and r.iters == 0 and np.all(host(r.x) == 0)
    I = system(np.full(n, 4.0))
    r = I.cg_solve(dev(np.ones(n)), rtol=1e-14)
    assert r.status == 0 and r.iters == 1 and np.all(host(r.x) == 0.25)
    r = I.cg_solve(dev(np.zeros(n)), rtol=1e-8)
    assert r.status == 0 and r.iters == 0 and np.all(host(r.x) == 0)
    prob, b = q1(8, 3, 1)
    A = assemble(spx, prob)
    for maxit in (0, 1, 3):
        r = A.cg_solve(dev(b), rtol=1e-12, maxit=maxit)
        assert r.status == spx.NOT_CONVERGED and r.iters == maxit
