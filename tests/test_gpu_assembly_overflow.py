"""Assembly of patterns whose row tile overflows (one row of more triplets
than a tile holds) on so many rows that the window index's scratch spans the
leftovers of the row sort, which exceed any place in the index: single
triplets, runs of equal rows and a vector, below the size up to which the
host learns of the overflow last.  Bitwise against the oracle."""
import numpy as np
import pytest

from paper_2406_08646_amd import workloads as W
from gpu_util import bits, csr_equal, dev, host, require_gpu

pytestmark = pytest.mark.gpu


def spread(n, ncoo, heavy, run, seed):
    """`heavy` triplets of row 0 among others of random rows, each named
    `run` times in a row."""
    rng = np.random.default_rng(seed)
    rows = np.concatenate([np.zeros(heavy // run, np.int64),
                           rng.integers(1, n, (ncoo - heavy) // run)])
    i = np.repeat(rng.permutation(rows), run)
    j = rng.integers(0, n, i.size)
    return W.CooProblem(n=n, i=i.astype(np.int32), j=j.astype(np.int32),
                        v=rng.uniform(-1, 1, i.size))


@pytest.mark.parametrize("n,ncoo,heavy,run", [(4000000, 200000, 2000, 1),
                                              (1 << 22, 250000, 1100, 1),
                                              (3000000, 250000, 2000, 4)])
def test_overflowed_tile_many_rows_bitwise(orc, n, ncoo, heavy, run):
    spx = require_gpu()
    prob = spread(n, ncoo, heavy, run, heavy)
    print(f"overflow n={n} ncoo={prob.ncoo}", flush=True)
    A = spx.coo_preallocate(n, dev(prob.i), dev(prob.j))
    A.set_values_coo(dev(prob.v))
    ref = orc.assemble(n, prob.i, prob.j, prob.v)
    csr_equal(ref, *(host(t) for t in A.get_csr()))
    jmap, perm = (host(t) for t in A.get_coo_maps())
    assert np.array_equal(jmap.astype(np.int64), ref.jmap) and np.array_equal(perm, ref.perm)
    x = np.random.default_rng(0).uniform(-1, 1, n)
    y, want = host(A.matmult(dev(x))), orc.spmv(ref, x)
    assert np.all(np.abs(y - want) <= 1e-12 * orc.abs_spmv(ref, x) + 1e-300)


def test_overflowed_vector_many_rows_bitwise(orc):
    spx = require_gpu()
    prob = spread(4000000, 200000, 2000, 1, 7)
    print("overflow, vector", flush=True)
    x = np.random.default_rng(1).uniform(-1, 1, prob.n)
    V = spx.vec_coo_preallocate(prob.n, dev(prob.i))
    got = dev(x)
    V.set_values_coo(dev(prob.v), got, mode=spx.ADD_VALUES)
    assert np.array_equal(bits(host(got)), bits(orc.vec_coo(prob.n, prob.i, prob.v, x, mode=1)))


@pytest.mark.parametrize("run", [1, 7])
@pytest.mark.parametrize("longest", [1023, 1024, 1025, 1535, 1537, 2600, 300000])
def test_long_row_at_every_place_bitwise(orc, longest, run):
    """One row of about a tile's capacity, or far above, after 0 to 600 other
    triplets (the tile boundary falls at its start, inside and at its end)."""
    spx = require_gpu()
    rng = np.random.default_rng(longest)
    for before in (0, 1, 511, 512, 600):
        rows = np.concatenate([np.arange(before) // 3, np.full(longest // run, 300),
                               301 + np.arange(700) // 2])
        i = np.repeat(rows, run)
        prob = W.CooProblem(n=2000, i=i.astype(np.int32),
                            j=rng.integers(0, 2000, i.size).astype(np.int32),
                            v=rng.uniform(-1, 1, i.size))
        A = spx.coo_preallocate(prob.n, dev(prob.i), dev(prob.j))
        A.set_values_coo(dev(prob.v))
        ref = orc.assemble(prob.n, prob.i, prob.j, prob.v)
        csr_equal(ref, *(host(t) for t in A.get_csr()))
        assert np.array_equal(host(A.get_coo_maps()[1]), ref.perm)


@pytest.mark.parametrize("n", [1, 3, 500])
def test_rows_as_full_as_tiles_bitwise(orc, n):
    """Exactly as many triplets as the rows' tiles hold, and one more."""
    spx = require_gpu()
    rng = np.random.default_rng(n)
    for extra in (0, 1):
        i = np.concatenate([np.repeat(np.arange(n), 1024), np.full(extra, n // 2)])
        prob = W.CooProblem(n=n, i=i.astype(np.int32),
                            j=rng.integers(0, n, i.size).astype(np.int32),
                            v=rng.uniform(-1, 1, i.size))
        A = spx.coo_preallocate(n, dev(prob.i), dev(prob.j))
        A.set_values_coo(dev(prob.v))
        ref = orc.assemble(n, prob.i, prob.j, prob.v)
        csr_equal(ref, *(host(t) for t in A.get_csr()))
