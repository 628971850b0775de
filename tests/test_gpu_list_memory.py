"""Device memory of handles whose matrix was tried for chunk lists, from ppcg_matrix_info."""

import pytest

from paper_2105_06176_amd import ppcg
from paper_2105_06176_amd.ppcg import Solver
from test_gpu_stencil import halves
from workloads import poisson3d

pytestmark = pytest.mark.gpu
SHARED = ppcg.FLAG_ITER_FUSED | ppcg.FLAG_SELL_SHARED_OFFSETS


def info(A, flags):
    S = Solver(A, spmv_format="sell", flags=flags)
    mi = S.matrix_info()
    S.close()
    return mi


@pytest.mark.parametrize("n", [6400, 50000])
def test_refused_lists_leave_nothing(n):
    """Two values of one entry in a chunk: the same storage with a value table and without, and no lists' memory."""
    A = halves(n, n // 2 + 20)
    plain, table = info(A, SHARED | ppcg.FLAG_SELL_FULL_VALUES), info(A, SHARED | ppcg.FLAG_SELL_VALUE_TABLE)
    assert table["distinct_values"] == 4  # 4, -1, -0.5 and the padding's 0
    # (the timing of 16-bit columns may keep them in either handle)
    extra, col16 = table["device_bytes"] - plain["device_bytes"], 2 * table["nnz_stored"]
    assert extra - (table["nnz_stored"] + 8 * 4) in (-col16, 0, col16)


@pytest.mark.parametrize("side", [64, 100])
def test_lists_need_no_second_vector_to_gather_from(side):
    """Eleven vectors, the inverse diagonal, the stored entries (with 16-bit columns where their timing kept them), and
    0.3 or 0.9 MB by their sizes for padding, partial sums, chunk extents and lists; a second vector would be 2.1 or 8."""
    A = poisson3d(side)
    mi = info(A, SHARED)
    assert mi["bytes_spmv"] < 9.0 * A.n  # lists
    rest = mi["device_bytes"] - 96.0 * A.n - 12.0 * mi["nnz_stored"]
    assert any(0 <= rest - col16 <= 2 * A.n for col16 in (0, 2 * mi["nnz_stored"]))
