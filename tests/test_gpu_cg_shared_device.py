"""Solves in a second process while another one, which has solved by
cooperative launches, still holds the device's queue for them: the launch is
refused there, and a pattern that met the refusal must not ask again on every
solve."""
import os
import subprocess
import sys

import numpy as np
import pytest

from paper_2406_08646_amd import workloads as W
from gpu_util import assemble, dev, require_gpu

pytestmark = pytest.mark.gpu

CHILD = """
import sys, time
sys.path.insert(0, sys.argv[1])
import numpy as np, torch
from paper_2406_08646_amd import spx, workloads as W
def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()
prob = W.q1_poisson(128, 2)
A = spx.coo_preallocate(prob.n, dev(prob.i), dev(prob.j))
A.set_values_coo(dev(prob.v))
b = dev(np.random.default_rng(0).uniform(-1, 1, prob.n))
def best(solve, count):
    times = []
    for _ in range(count):
        torch.cuda.synchronize()
        t = time.perf_counter()
        r = solve(b)
        torch.cuda.synchronize()
        times.append(time.perf_counter() - t)
        assert r.status == 0
    return min(times)
for name in ("cg_solve", "cg_solve_mixed"):
    solve = getattr(A, name)
    A.set_option(spx.OPT_SMALL_SOLVE, 1)
    first = best(solve, 1)
    auto = best(solve, 4)
    A.set_option(spx.OPT_SMALL_SOLVE, 0)
    best(solve, 1)
    launches = best(solve, 4)
    print(f"{name}: first {first * 1e3:.2f} ms, then {auto * 1e3:.2f}, by launches {launches * 1e3:.2f}",
          flush=True)
    assert auto <= 2 * launches
"""


def test_refused_launch_is_not_repeated():
    spx = require_gpu()
    prob = W.q1_poisson(64, 2)
    A = assemble(spx, prob)
    assert A.cg_solve(dev(np.ones(prob.n)), rtol=1e-8).status == 0
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    out = subprocess.run([sys.executable, "-u", "-c", CHILD, root], capture_output=True, text=True,
                         timeout=100)
    print(out.stdout, out.stderr, flush=True)
    assert out.returncode == 0
