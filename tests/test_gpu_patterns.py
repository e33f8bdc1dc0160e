"""GPU products and solves of patterns whose rows repeat (the pattern walk):
list lengths, window sizes and tile loads at the edges of its forms, patterns
just past them, empty rows, ragged last tiles and values that must not
spread, against the oracle."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2406_08646_amd import workloads as W
from gpu_util import dev, host, require_gpu, spmv_within

pytestmark = pytest.mark.gpu


def bits(a):
    return np.ascontiguousarray(a).view(np.int64)


def from_lists(n, lists, pick, seed):
    """Row r has the columns r + o of lists[pick(r)] that exist, and random
    values; symmetric in structure only if the lists are."""
    rows = np.arange(n)
    which = pick(rows)
    I, J = [], []
    for k, offs in enumerate(lists):
        r = rows[which == k]
        for o in offs:
            c = r + o
            ok = (c >= 0) & (c < n)
            I.append(r[ok])
            J.append(c[ok])
    i, j = np.concatenate(I).astype(np.int32), np.concatenate(J).astype(np.int32)
    v = np.random.default_rng(seed).uniform(-1, 1, i.size)
    return W.CooProblem(n=n, i=i, j=j, v=v)


def run_of(length):
    return [list(range(-(length // 2), length - length // 2))]


def groups(count):
    """3 entries around each of `count` places 640 columns apart: 4 or 5 (6)
    blocks each."""
    return [[640 * g + d for g in range(count) for d in (0, 1, 2)]]


CASES = {}
for L in (1, 2, 5, 6, 9, 10, 27, 28, 32, 33):
    CASES[f"length{L}"] = lambda L=L: from_lists(2100, run_of(L), lambda r: 0 * r, L)
for G in (3, 4, 5, 6, 7, 8):
    CASES[f"groups{G}"] = lambda G=G: from_lists(7000, groups(G), lambda r: 0 * r, 50 + G)
for K in (1, 3, 15, 16, 17, 40):  # lists in every tile
    CASES[f"lists{K}"] = lambda K=K: from_lists(
        3000, [[-40 - k, -1, 0, 1, 3 + k] for k in range(K)], lambda r, K=K: r % K, 100 + K)
CASES["empty_rows"] = lambda: from_lists(1500, [[], [-1, 0, 1], [0]], lambda r: r % 7 % 3, 7)
CASES["empty_tile"] = lambda: from_lists(1500, [[], [-1, 0, 1]],
                                         lambda r: ((r < 256) | (r >= 600)).astype(int), 8)
CASES["tile"] = lambda: from_lists(256, run_of(7), lambda r: 0 * r, 9)
CASES["rows257"] = lambda: from_lists(257, run_of(7), lambda r: 0 * r, 10)
CASES["row1"] = lambda: from_lists(1, run_of(1), lambda r: 0 * r, 11)


@pytest.mark.parametrize("case", sorted(CASES))
def test_pattern_products_bitwise(orc, case):
    """Products and transposed products have the oracle's bits, also where x
    holds infinities and NaN that only some rows meet."""
    spx = require_gpu()
    prob = CASES[case]()
    print(case, prob.n, flush=True)
    A = spx.coo_preallocate(prob.n, dev(prob.i), dev(prob.j))
    A.set_values_coo(dev(prob.v))
    A.set_option(spx.OPT_SPMV_VARIANT, 4)
    ref = orc.assemble(prob.n, prob.i, prob.j, prob.v)
    x = np.random.default_rng(3).uniform(-1, 1, prob.n)
    for bad in (None, np.inf, np.nan):
        if bad is not None:
            x[prob.n // 3] = bad
        for y, y_ref in ((A.matmult(dev(x)), orc.spmv(ref, x)),
                         (A.matmult_transpose(dev(x)), orc.spmv_transpose(ref, x))):
            y = host(y)
            assert np.array_equal(np.isnan(y), np.isnan(y_ref))
            ok = ~np.isnan(y)
            assert np.array_equal(bits(y[ok]), bits(y_ref[ok]))


@pytest.mark.parametrize("shape,points", [((41, 37), 5), ((60, 43), 9), ((19, 17, 23), 27),
                                          ((13, 16, 33), 7)])
def test_pattern_solves(orc, shape, points):
    """CG, transposed CG and the mixed-precision solve on symmetric stencils:
    the solution's residual, by the oracle's product, meets the tolerance."""
    spx = require_gpu()
    dim = len(shape)
    n = int(np.prod(shape))
    idx = np.arange(n).reshape(shape)
    I, J, V = [], [], []
    for o in np.ndindex(*(3,) * dim):
        o = [k - 1 for k in o]
        if points in (5, 7) and np.abs(o).sum() > 1:
            continue
        src = idx[tuple(slice(max(0, -k), s - max(0, k)) for k, s in zip(o, shape))].ravel()
        dst = idx[tuple(slice(max(0, k), s - max(0, -k)) for k, s in zip(o, shape))].ravel()
        I.append(src)
        J.append(dst)
        V.append(np.full(src.size, points - 0.99 if not any(o) else -1.0))
    i, j = np.concatenate(I).astype(np.int32), np.concatenate(J).astype(np.int32)
    v = np.concatenate(V)
    print(shape, points, flush=True)
    A = spx.coo_preallocate(n, dev(i), dev(j))
    A.set_values_coo(dev(v))
    A.set_option(spx.OPT_SPMV_VARIANT, 4)
    ref = orc.assemble(n, i, j, v)
    b = np.random.default_rng(5).uniform(-1, 1, n)
    for r in (A.cg_solve(dev(b), rtol=1e-10), A.cg_solve_transpose(dev(b), rtol=1e-10),
              A.cg_solve_mixed(dev(b), rtol_outer=1e-10, rtol_inner=1e-4)):
        assert r.status == 0
        # the recursive residual's drift from the true one stays well below rtol
        assert np.linalg.norm(b - orc.spmv(ref, host(r.x))) <= 2e-10 * np.linalg.norm(b)


# stencils on ragged meshes of more than one 256-row tile per CU (27n: four);
# 27 points with windows of up to 24 blocks or, in 27w, more
SPMM_SHAPES = {"5": ((311, 299), 5), "9": ((307, 303), 9), "27": ((47, 44, 43), 27),
               "27w": ((51, 51, 51), 27), "27n": ((62, 64, 70), 27)}


@pytest.mark.parametrize("name", sorted(SPMM_SHAPES))
def test_pattern_spmm_bitwise(orc, name):
    """Y = A X for every width that changes the form, contiguous, strided and
    off a 16-byte boundary, has the bits of the gathering kernel (which takes
    16 strided columns), and the oracle's values; nothing is written past a
    row."""
    spx = require_gpu()
    shape, points = SPMM_SHAPES[name]
    dim, n = len(shape), int(np.prod(shape))
    idx = np.arange(n).reshape(shape)
    I, J = [], []
    for o in np.ndindex(*(3,) * dim):
        o = [k - 1 for k in o]
        if points == 5 and np.abs(o).sum() > 1:
            continue
        I.append(idx[tuple(slice(max(0, -k), s - max(0, k)) for k, s in zip(o, shape))].ravel())
        J.append(idx[tuple(slice(max(0, k), s - max(0, -k)) for k, s in zip(o, shape))].ravel())
    i, j = np.concatenate(I).astype(np.int32), np.concatenate(J).astype(np.int32)
    rng = np.random.default_rng(31)
    v = rng.uniform(-1, 1, i.size)
    A = spx.coo_preallocate(n, dev(i), dev(j))
    A.set_values_coo(dev(v))
    ref = orc.assemble(n, i, j, v)
    lib = spx.load_library()
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    for nrhs, pad, shift in ((1, 0, 0), (2, 0, 0), (2, 0, 1), (3, 0, 0), (4, 2, 0), (5, 0, 0),
                             (6, 0, 0), (7, 1, 0), (8, 0, 0), (11, 0, 0), (12, 0, 0), (15, 3, 1),
                             (16, 0, 0), (16, 1, 0),
                             (17, 0, 0), (24, 0, 0), (32, 0, 0), (33, 1, 0)):
        print(name, n, nrhs, pad, shift, flush=True)
        ld = nrhs + pad
        Xh = rng.uniform(-1, 1, (n, nrhs))
        X = torch.zeros(n * ld + 2, dtype=torch.float64, device="cuda")
        Y = torch.full((n * ld + 2,), 7.0, dtype=torch.float64, device="cuda")
        X[shift:shift + n * ld].view(n, ld)[:, :nrhs] = dev(Xh)
        rc = lib.spx_spmm(A.handle, nrhs, ctypes.c_void_p(X.data_ptr() + 8 * shift), ld,
                          ctypes.c_void_p(Y.data_ptr() + 8 * shift), ld, stream)
        assert rc == 0
        Yh = host(Y)
        body = Yh[shift:shift + n * ld].reshape(n, ld)
        assert np.all(body[:, nrhs:] == 7.0) and np.all(Yh[:shift] == 7.0)
        assert np.all(Yh[shift + n * ld:] == 7.0)
        for c in range(0, nrhs, 16):
            Xg = torch.zeros(n, 18, dtype=torch.float64, device="cuda")
            k = min(16, nrhs - c)
            Xg[:, :k] = dev(np.ascontiguousarray(Xh[:, c:c + k]))
            Yg = torch.zeros(n, 18, dtype=torch.float64, device="cuda")
            assert lib.spx_spmm(A.handle, 16, ctypes.c_void_p(Xg.data_ptr()), 18,
                                ctypes.c_void_p(Yg.data_ptr()), 18, stream) == 0
            assert np.array_equal(bits(body[:, c:c + k]), bits(host(Yg)[:, :k]))
    # the last product against the oracle
    spmv_within(body[:, 0], orc.spmv(ref, Xh[:, 0]), orc.abs_spmv(ref, Xh[:, 0]))


def test_pattern_products_under_capture():
    """A captured product and product of several vectors, both of the forms
    that raise their LDS limit, replay with the eager bits on new inputs."""
    spx = require_gpu()
    idx = np.arange(62 * 64 * 70).reshape(62, 64, 70)
    I, J = [], []
    for o in np.ndindex(3, 3, 3):
        o = [k - 1 for k in o]
        I.append(idx[tuple(slice(max(0, -k), s - max(0, k)) for k, s in zip(o, idx.shape))].ravel())
        J.append(idx[tuple(slice(max(0, k), s - max(0, -k)) for k, s in zip(o, idx.shape))].ravel())
    i, j = np.concatenate(I).astype(np.int32), np.concatenate(J).astype(np.int32)
    n = idx.size
    A = spx.coo_preallocate(n, dev(i), dev(j))
    A.set_values_coo(dev(np.random.default_rng(41).uniform(-1, 1, i.size)))
    x, X = (torch.zeros(n, k, dtype=torch.float64, device="cuda").squeeze(1) for k in (1, 4))
    y, Y = torch.empty_like(x), torch.empty_like(X)
    A.matmult(x, y)
    A.spmm(X, Y)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        A.matmult(x, y)
        A.spmm(X, Y)
    for seed in range(3):
        x.copy_(dev(np.random.default_rng(seed).uniform(-1, 1, n)))
        X.copy_(dev(np.random.default_rng(seed + 9).uniform(-1, 1, (n, 4))))
        y.fill_(7.0)
        Y.fill_(7.0)
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(bits(host(y)), bits(host(A.matmult(x))))
        assert np.array_equal(bits(host(Y)), bits(host(A.spmm(X))))
