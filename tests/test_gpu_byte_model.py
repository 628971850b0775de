"""What ppcg_matrix_info says that an iteration reads, on matrices of chunk lists, from the kernels' own loads."""

import pytest

from paper_2105_06176_amd import ppcg
from paper_2105_06176_amd.ppcg import Solver
from workloads import poisson2d, poisson3d, poisson125

pytestmark = pytest.mark.gpu
GENS = [lambda: poisson2d(301), lambda: poisson3d(40), lambda: poisson125(40)]


def info(A, **options):
    S = Solver(A, spmv_format="sell", **options)
    mi = S.matrix_info()
    S.close()
    return mi


@pytest.mark.parametrize("gen", GENS)
def test_fp32_values_are_counted_per_entry(gen):
    """PIPECG with FP32 values streams 4 bytes per entry, a column of 0, 2 or 4 bytes, and two FP64 vectors."""
    A = gen()
    mi = info(A, precision="mixed_values")
    chunks = (A.n + 63) // 64
    assert mi["value_bytes"] == 4 and mi["iter_launches"] == 2
    vectors, matrix = 16.0 * A.n, (4.0 + mi["col_index_bytes"]) * A.nnz
    assert 0 <= mi["bytes_spmv"] - vectors - matrix <= 12.0 * (chunks + 1)


@pytest.mark.parametrize("gen", GENS)
@pytest.mark.parametrize("prec,vector", [("fp64", 8), ("mixed_values", 8), ("mixed", 4)])
def test_classic_pcg_reads_the_lists(gen, prec, vector):
    A = gen()
    mi = info(A, precision=prec, method="pcg")
    assert mi["bytes_spmv"] == 16.0 * ((A.n + 63) // 64) + 4.0 * vector * A.n


@pytest.mark.parametrize("gen", GENS)
def test_fp64_reads_the_lists(gen):
    A = gen()
    mi = info(A)
    assert mi["iter_launches"] == 1
    assert mi["bytes_spmv"] == 16.0 * ((A.n + 63) // 64) + 8.0 * A.n  # n stays in registers


@pytest.mark.parametrize("gen", GENS)
def test_reported_values_of_list_matrices(gen):
    """The diagonal, -1 and the padding's 0.0; no bytes per value in FP64 by either method."""
    A = gen()
    for options in ({}, {"flags": ppcg.FLAG_SELL_VALUE_TABLE}, {"method": "pcg"}):
        mi = info(A, **options)
        assert (mi["distinct_values"], mi["value_bytes"], mi["col_index_bytes"]) == (3, 1, 0), options
    mi = info(A, flags=ppcg.FLAG_SELL_FULL_VALUES)
    assert (mi["distinct_values"], mi["value_bytes"]) == (0, 8)
