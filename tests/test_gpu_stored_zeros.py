"""Zeros that a matrix stores are entries: 0 * Inf and 0 * NaN are NaN in the row sum, in whatever storage the handle
chose, and they take part in the iteration like any other value."""

import numpy as np
import pytest

import oracle
from paper_2105_06176_amd import ppcg
from paper_2105_06176_amd.ppcg import Solver
from test_gpu_stencil import dev, host, tridiagonal
from workloads import rhs_from_solution, xstar_uniform

pytestmark = pytest.mark.gpu


def some_zeros(n):
    off = np.full(n - 1, -1.0)
    off[5::9] = 0.0
    return tridiagonal(n, off)


def all_zeros(n):
    """Diagonal matrix with stored zeros beside the diagonal: one value per entry of every chunk's list."""
    return tridiagonal(n, np.zeros(n - 1))


@pytest.mark.parametrize("gen", [some_zeros, all_zeros])
@pytest.mark.parametrize("n", [700, 6400])
@pytest.mark.parametrize("special", [np.inf, -np.inf, np.nan])
def test_spmv_multiplies_stored_zeros(gen, n, special):
    A = gen(n)
    S = Solver(A)
    x = xstar_uniform(n, 3)
    # inside the matrix: every row there has all the entries of its chunk's list
    x[[n // 2, n // 2 + 5, n // 2 + 6]] = special
    assert np.array_equal(host(S.spmv(dev(x))), oracle.spmv(A, x), equal_nan=True)
    S.close()


@pytest.mark.parametrize("n", [700, 6400])
def test_solve_with_stored_zeros(n):
    A = some_zeros(n)
    b = rhs_from_solution(A, xstar_uniform(n, 4))
    S = Solver(A, fixed_iters=15)
    x, info = S.solve(dev(b))
    ref = oracle.pipecg(A, b, fixed_iters=15)
    assert info["status"] == ppcg.OK and info["iters"] == ref.iters
    assert np.linalg.norm(host(x) - ref.x) <= 1e-10 * np.linalg.norm(ref.x)
    S.close()
