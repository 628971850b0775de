"""Device allocations of ppcg_create (run by test_gpu_list_sample.py in a process of its own): arguments: the counting
library, the HIP runtime."""

import ctypes
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path[:0] = [ROOT, os.path.join(ROOT, "tests")]

C = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
assert C.count_init(sys.argv[2].encode()) == 0

import torch  # noqa: E402

torch.zeros(1, device="cuda")

from paper_2105_06176_amd.ppcg import Solver  # noqa: E402
from test_gpu_list_sample import unit_diagonal  # noqa: E402
from workloads import poisson2d, random_spd, stencil27_lognormal  # noqa: E402


def allocations(A):
    before = C.count_mallocs()
    S = Solver(A)
    S.close()
    return C.count_mallocs() - before


for A in (random_spd(30000), stencil27_lognormal(30, seed=1)):
    allocations(A)  # the signature's choices are timed here
    print("COUNT", allocations(A), allocations(unit_diagonal(A)), flush=True)
print("LISTS", allocations(poisson2d(64)), flush=True)
