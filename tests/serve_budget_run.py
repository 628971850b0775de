"""Peak of the device memory that a server's requests take (run by test_gpu_serve_budget.py in a process of its own):
arguments: the counting library, the HIP runtime's soname, the budget in bytes."""

import ctypes
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path[:0] = [ROOT, os.path.join(ROOT, "tests")]

counter, runtime, budget = sys.argv[1], sys.argv[2], float(sys.argv[3])
C = ctypes.CDLL(counter, mode=ctypes.RTLD_GLOBAL)
C.count_used.restype = C.count_most.restype = ctypes.c_size_t
assert C.count_init(runtime.encode()) == 0

import torch  # noqa: E402

torch.zeros(1, device="cuda")

from paper_2105_06176_amd import ppcg  # noqa: E402
from test_gpu_serve_pool import burst  # noqa: E402

before = C.count_used()
server = ppcg.Server(budget_bytes=budget)
own = C.count_used()  # the engine's tables
assert own > before  # the counters are in place
C.count_reset()
errors = []
burst(server, 3, errors)
assert not errors, errors
print("PEAK", C.count_most() - own, flush=True)
server.close()
assert C.count_used() == before
