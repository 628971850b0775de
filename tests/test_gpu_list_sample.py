"""Which matrices of a constant diagonal are tried for chunk lists: a sample of the chunks may only rule out what the
layout itself would refuse."""

import subprocess
import sys

import numpy as np
import pytest

import oracle
from paper_2105_06176_amd import ppcg
from paper_2105_06176_amd.ppcg import Solver
from test_gpu_serve_budget import HERE, counter, runtime  # noqa: F401 (counter: a fixture)
from test_gpu_stencil import box, dev, host, runs, tridiagonal
from workloads import CSR, poisson2d, poisson3d, random_spd, rhs_from_solution, stencil27_lognormal, xstar_uniform

pytestmark = pytest.mark.gpu


def unit_diagonal(A):
    """A scaled from both sides to a diagonal of ones."""
    rows = np.repeat(np.arange(A.n), np.diff(A.rp))
    on = rows == A.ci
    s = np.empty(A.n)
    s[rows[on]] = 1.0 / np.sqrt(A.val[on])
    val = A.val * s[rows] * s[A.ci]
    val[on] = 1.0
    return CSR(A.n, A.rp, A.ci, val, A.name + "_unit")


def one_other(n, at):
    """-1 beside the diagonal but for one couple of rows."""
    off = np.full(n - 1, -1.0)
    off[at] = -0.75
    return tridiagonal(n, off)


LISTS = {"poisson2d_301": lambda: poisson2d(301), "unit_poisson3d_40": lambda: unit_diagonal(poisson3d(40)),
         "box_63_9_11": lambda: box(63, 9, 11), "runs_16_16_16": lambda: runs(16, 16, 16, 2, 2, 2),
         "two_chunks": lambda: tridiagonal(65, np.full(64, -1.0))}
OTHERS = {"unit_random": lambda: unit_diagonal(random_spd(30000)),
          "unit_stencil27": lambda: unit_diagonal(stencil27_lognormal(30, seed=1)),
          "a_value_in_the_first_chunk": lambda: one_other(20000, 5),
          "a_value_in_a_chunk_between": lambda: one_other(20000, 10 * 64 + 70)}


@pytest.mark.parametrize("name", sorted(LISTS) + sorted(OTHERS))
def test_automatic_choice(name):
    A = {**LISTS, **OTHERS}[name]()
    b = rhs_from_solution(A, xstar_uniform(A.n, 3))
    S = Solver(A, fixed_iters=8)
    mi = S.matrix_info()
    lists = mi["bytes_spmv"] == 16.0 * ((A.n + 63) // 64) + (8.0 if mi["iter_launches"] == 1 else 16.0) * A.n
    assert lists == (name in LISTS)
    x, info = S.solve(dev(b))
    ref = oracle.pipecg(A, b, fixed_iters=8)
    assert info["status"] == ppcg.OK and info["iters"] == ref.iters
    assert np.linalg.norm(host(x) - ref.x) <= 1e-10 * np.linalg.norm(ref.x)
    S.close()


def test_no_layout_is_tried_in_vain(counter):  # noqa: F811
    """The same pattern with a varying and a constant diagonal: as many allocations.  A small matrix on lists: 19 (21 with
    a sizing pass of its own)."""
    ppcg.lib()
    r = subprocess.run([sys.executable, HERE + "/create_count_run.py", counter, runtime()], capture_output=True,
                       text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    counts, lists = r.stdout.split("LISTS")
    for line in counts.split("COUNT")[1:]:
        varying, constant = map(int, line.split()[:2])
        assert constant == varying, r.stdout
    assert int(lists) <= 19, r.stdout
