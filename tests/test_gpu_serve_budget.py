"""The device memory of a server's requests: in use and idle together, what a burst takes stays within the budget, and
a handle holds no more than its footprint."""

import os
import subprocess
import sys

import pytest

from paper_2105_06176_amd import ppcg
from paper_2105_06176_amd.ppcg import Solver
from test_gpu_stencil import runs
from workloads import poisson3d, poisson125, random_spd

pytestmark = pytest.mark.gpu
HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def counter(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("count") / "hip_count.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", out, os.path.join(HERE, "hip_count.c"), "-ldl",
                    "-lpthread"], check=True)
    return out


def runtime():
    """The HIP runtime that this process has loaded."""
    with open("/proc/self/maps") as f:
        return next(ln.split()[-1] for ln in f if "libamdhip64.so" in ln)


@pytest.mark.parametrize("budget", [24 << 20, 40 << 20])
def test_a_burst_stays_within_the_budget(counter, budget):
    """Three rounds of six systems, the largest of which takes 18 MiB while it is prepared: the device memory in use and
    idle, beside the server's own, at its highest (64 KiB for its work tables, which grow to 8 bytes per tile)."""
    ppcg.lib()
    r = subprocess.run([sys.executable, os.path.join(HERE, "serve_budget_run.py"), counter, runtime(), str(budget)],
                       capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    peak = int(r.stdout.split("PEAK")[1])
    print(f"budget {budget >> 20} MiB, at most {peak / 2**20:.1f} MiB")
    assert peak <= budget + (64 << 10)


MATS = {"list_padding_1.5": lambda: runs(16, 16, 16, 2, 2, 2), "poisson125_40": lambda: poisson125(40),
        "poisson3d_64": lambda: poisson3d(64), "random_20000": lambda: random_spd(20000),
        "random_100": lambda: random_spd(100), "poisson3d_9": lambda: poisson3d(9)}


@pytest.mark.parametrize("name", sorted(MATS))
@pytest.mark.parametrize("prec", ["fp64", "mixed", "mixed_values"])
@pytest.mark.parametrize("flags", [0, ppcg.FLAG_ITER_FUSED | ppcg.FLAG_SELL_VALUE_TABLE])
def test_a_handle_holds_at_most_its_footprint(name, prec, flags):
    A = MATS[name]()
    S = Solver(A, precision=prec, flags=flags)
    mi = S.matrix_info()
    S.close()
    vectors = 88.0 * A.n + (48.0 * A.n if prec == "mixed" else 0.0)
    assert vectors + 12.0 * mi["nnz_stored"] < mi["device_bytes"]
    assert mi["device_bytes"] <= ppcg.footprint_bytes(A.n, A.nnz, prec)
