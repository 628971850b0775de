"""Classic PCG with the CSR-vector SpMV at the edges of its tiles: 512 rows up to 524,288 rows on 256 compute units, then
1,024 and 1,536; last tiles of one row, and of a whole one."""

import numpy as np
import pytest

import oracle
from paper_2105_06176_amd import ppcg
from paper_2105_06176_amd.ppcg import Solver
from test_gpu_stencil import dev, host, tridiagonal
from workloads import random_spd, rhs_from_solution, xstar_uniform

pytestmark = pytest.mark.gpu


def matrix(n):
    return random_spd(n, seed=3) if n < 100000 else tridiagonal(n, np.full(n - 1, -1.0))


@pytest.mark.parametrize("n", [1, 2, 511, 512, 513, 30001, 524287, 524288, 524289, 1048576, 1048577, 1100003])
@pytest.mark.parametrize("prec", ["fp64", "mixed_values"])
def test_fixed_iterates_match_oracle(n, prec):
    A = matrix(n) if n > 2 else tridiagonal(n, np.full(n - 1, -1.0))
    b = rhs_from_solution(A, xstar_uniform(n, 3))
    k = min(n, 5)
    if prec == "mixed_values" and n < 100000:  # values that FP32 holds
        A.val[:] = A.val.astype(np.float32)
        b = rhs_from_solution(A, xstar_uniform(n, 3))
    S = Solver(A, fixed_iters=k, method="pcg", spmv_format="csr_vector", precision=prec, inner_tol=1e-30)
    x, info = S.solve(dev(b))
    ref = oracle.pcg(A, b, fixed_iters=k)
    assert info["status"] == ppcg.OK and info["iters"] == ref.iters
    assert np.linalg.norm(host(x) - ref.x) <= 1e-10 * np.linalg.norm(ref.x)
    S.close()


@pytest.mark.parametrize("n", [513, 524289])
def test_fp32_vectors_reach_the_tolerance(n):
    A = matrix(n)
    b = rhs_from_solution(A, xstar_uniform(n, 3))
    S = Solver(A, tol=1e-10, method="pcg", spmv_format="csr_vector", precision="mixed")
    x, info = S.solve(dev(b))
    assert info["status"] == ppcg.OK and oracle.true_relres(A, b, host(x)) <= 1e-10
    S.close()
