"""Graphs captured while systems with runs of columns come and go beside one without (run by test_gpu_serve_graphs.py
in a process of its own): arguments: the counting library, the HIP runtime."""

import ctypes
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path[:0] = [ROOT, os.path.join(ROOT, "tests")]

C = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
assert C.count_init(sys.argv[2].encode()) == 0

import numpy as np  # noqa: E402
import torch  # noqa: E402

torch.zeros(1, device="cuda")

from paper_2105_06176_amd.ppcg import OK, Server, Solver  # noqa: E402
from test_gpu_stencil import runs  # noqa: E402
from workloads import poisson2d, rhs_from_solution, xstar_uniform  # noqa: E402

VISITS = 12
long, short = poisson2d(2000), runs(40, 40, 40, 1, 1, 1)
bl, bs = (rhs_from_solution(A, xstar_uniform(A.n, 3)) for A in (long, short))
S = Solver(short, tol=1e-6, vec_mem="host")
alone = torch.empty(short.n, dtype=torch.float64)
S.solve(torch.as_tensor(bs), out=alone)
S.close()
server = Server()
rid = server.submit(long, bl, 0.0, "fp64")
server.step()
before = C.count_graphs()
for _ in range(VISITS):
    v = server.submit(short, bs, 1e-6, "fp64")
    got = None
    while got is None:
        server.step()
        assert server.poll(rid) is None, "the long request ended before the visits"
        got = server.poll(v)
    assert got[1]["status"] == OK and np.array_equal(got[0], alone.numpy())
    server.step()  # the long one alone
print("GRAPHS", C.count_graphs() - before, flush=True)
server.close()
