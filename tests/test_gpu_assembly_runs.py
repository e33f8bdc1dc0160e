"""Assembly of streams that name the same row several times in a row (the
symbolic stage sorts those runs instead of the triplets) bitwise against the
oracle: runs of every length around the tile edges, rows and runs too long
for a tile (the full sort), empty rows, both sides of the size up to which
the pattern's arrays are sized by the triplets, index arrays off a 16-byte
boundary, and streams with ignored triplets (no runs)."""
import numpy as np
import pytest
import torch

from paper_2406_08646_amd import workloads as W
from gpu_util import bits, csr_equal, dev, host, require_gpu

pytestmark = pytest.mark.gpu


def runs(rng, n, lengths, span, gaps=1):
    """Runs of the given lengths in random rows (multiples of gaps), columns
    within span of the row, many of them twice."""
    row = (rng.integers(0, max(1, n // gaps), len(lengths)) * gaps).clip(0, n - 1)
    i = np.repeat(row, lengths)
    j = (i + rng.integers(-span, span + 1, i.size)).clip(0, n - 1)
    v = np.ldexp(rng.uniform(-1, 1, i.size), rng.integers(-30, 31, i.size))
    return W.CooProblem(n=n, i=i.astype(np.int32), j=j.astype(np.int32), v=v)


def check(orc, spx, prob, shift=0):
    def index(a):
        t = torch.zeros(a.size + shift, dtype=torch.int32, device="cuda")
        t[shift:] = dev(a)
        return t[shift:]

    A = spx.coo_preallocate(prob.n, index(prob.i), index(prob.j))
    A.set_values_coo(dev(prob.v))
    ref = orc.assemble(prob.n, prob.i, prob.j, prob.v)
    csr_equal(ref, *(host(t) for t in A.get_csr()))
    jmap, perm = (host(t) for t in A.get_coo_maps())
    assert np.array_equal(jmap.astype(np.int64), ref.jmap) and np.array_equal(perm, ref.perm)
    x = np.random.default_rng(0).uniform(-1, 1, prob.n)
    assert np.array_equal(bits(host(A.matmult(dev(x)))), bits(orc.spmv(ref, x)))
    yt = host(A.matmult_transpose(dev(x)))
    scale = np.bincount(prob.j, np.abs(prob.v * x[prob.i]), prob.n)
    assert np.all(np.abs(yt - orc.spmv_transpose(ref, x)) <= 1e-12 * scale + 1e-300)
    A.destroy()


@pytest.mark.parametrize("n,nrun,lo,hi,gaps,shift", [
    (1, 40, 2, 9, 1, 0),            # one row
    (900, 700, 2, 2, 1, 0),         # the shortest runs that are sorted
    (900, 900, 8, 8, 1, 0),         # element rows
    (900, 900, 1, 15, 1, 1),        # ragged, index arrays off a boundary
    (70000, 9000, 3, 9, 7, 3),      # most rows empty, the last ones too
    (400, 400, 60, 70, 1, 0),       # a few rows per tile
    (300, 60, 400, 600, 1, 0),      # rows about a tile long
    (50, 40, 900, 1100, 1, 0),      # runs around the capacity: the full sort
    (5000, 40000, 4, 10, 1, 0),     # above 2^18 triplets
    (300, 300, 1000, 1100, 1, 2),   # above 2^18 triplets, the full sort
    (5000000, 30000, 2, 12, 1, 0),  # more than 2^22 rows: the full sort
])
def test_runs_bitwise(orc, n, nrun, lo, hi, gaps, shift):
    spx = require_gpu()
    rng = np.random.default_rng(n + nrun + hi)
    prob = runs(rng, n, rng.integers(lo, hi + 1, nrun), 40, gaps)
    print(f"runs n={n} ncoo={prob.ncoo}", flush=True)
    check(orc, spx, prob, shift)


@pytest.mark.parametrize("drop", [0.001, 0.5])
def test_runs_with_ignored_triplets_bitwise(orc, drop):
    spx = require_gpu()
    rng = np.random.default_rng(3)
    prob = runs(rng, 3000, rng.integers(4, 9, 4000), 30)
    gone = rng.random(prob.ncoo) < drop
    keep = ~gone
    A = spx.coo_preallocate(prob.n, dev(np.where(gone, -1, prob.i).astype(np.int32)), dev(prob.j))
    A.set_values_coo(dev(prob.v))
    ref = orc.assemble(prob.n, prob.i[keep], prob.j[keep], prob.v[keep])
    csr_equal(ref, *(host(t) for t in A.get_csr()))
    perm = host(A.get_coo_maps()[1])
    assert np.array_equal(perm, np.flatnonzero(keep)[ref.perm])


def test_one_triplet_per_tile_boundary(orc):
    """Row counts and run starts exactly on the 512-item tile edges."""
    spx = require_gpu()
    for per in (1, 2, 511, 512, 513, 1024):
        i = np.repeat(np.arange(6), per)
        j = np.tile(np.arange(per) % 6, 6)
        prob = W.CooProblem(n=6, i=i.astype(np.int32), j=j.astype(np.int32),
                            v=np.arange(i.size, dtype=np.float64))
        check(orc, spx, prob)
