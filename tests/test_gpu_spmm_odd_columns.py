"""Products of an odd number of columns by row patterns where X and Y have even
strides and end at the last row's last column: the bits of the gathering
kernel, whatever follows, and nothing written past a row."""
import ctypes

import numpy as np
import pytest
import torch

from gpu_util import bits, dev, host, require_gpu

pytestmark = pytest.mark.gpu

# more than one 256-row tile per CU (5many: ten, from where 6 columns have
# their form), a ragged last one, and each window class
SHAPES = {"5": ((311, 299), 5), "5many": ((811, 811), 5), "9": ((307, 303), 9), "27": ((47, 44, 43), 27),
          "27w": ((51, 51, 51), 27), "27n": ((62, 64, 70), 27)}


@pytest.mark.parametrize("name", sorted(SHAPES))
def test_odd_columns_end_with_the_block(name):
    spx = require_gpu()
    shape, points = SHAPES[name]
    n, idx = int(np.prod(shape)), np.arange(np.prod(shape)).reshape(shape)
    I, J = [], []
    for o in np.ndindex(*(3,) * len(shape)):
        o = [k - 1 for k in o]
        if points == 5 and np.abs(o).sum() > 1:
            continue
        I.append(idx[tuple(slice(max(0, -k), s - max(0, k)) for k, s in zip(o, shape))].ravel())
        J.append(idx[tuple(slice(max(0, k), s - max(0, -k)) for k, s in zip(o, shape))].ravel())
    rng = np.random.default_rng(5)
    A = spx.coo_preallocate(n, dev(np.concatenate(I).astype(np.int32)),
                            dev(np.concatenate(J).astype(np.int32)))
    A.set_values_coo(dev(rng.uniform(-1, 1, A.ncoo)))
    lib, stream = spx.load_library(), torch.cuda.current_stream().cuda_stream

    def product(nrhs, X, ldx, Y, ldy):
        assert lib.spx_spmm(A.handle, nrhs, ctypes.c_void_p(X.data_ptr()), ldx,
                            ctypes.c_void_p(Y.data_ptr()), ldy, stream) == 0

    for nrhs, ld in ((1, 2), (3, 4), (5, 6), (5, 8), (7, 8), (9, 10), (13, 14), (17, 18), (23, 24),
                     (31, 32)):
        if name == "5many" and nrhs > 7:
            break
        print(name, n, nrhs, ld, flush=True)
        used = (n - 1) * ld + nrhs
        X = torch.full((used + 64,), float("nan"), dtype=torch.float64, device="cuda")
        Y = torch.full((used + 64,), 7.0, dtype=torch.float64, device="cuda")
        Xh = rng.uniform(-1, 1, (n, nrhs))
        X.as_strided((n, nrhs), (ld, 1)).copy_(dev(Xh))
        product(nrhs, X, ld, Y, ld)
        got = host(Y.as_strided((n, nrhs), (ld, 1)).contiguous())
        # 16 strided columns at a time take the gathering kernel
        for c in range(0, nrhs, 16):
            k = min(16, nrhs - c)
            Xg, Yg = (torch.zeros(n, 18, dtype=torch.float64, device="cuda") for _ in range(2))
            Xg[:, :k] = dev(np.ascontiguousarray(Xh[:, c:c + k]))
            product(16, Xg, 18, Yg, 18)
            assert np.array_equal(bits(got[:, c:c + k]), bits(host(Yg)[:, :k]))
        Y.as_strided((n, nrhs), (ld, 1)).fill_(7.0)
        assert bool((Y == 7.0).all())
