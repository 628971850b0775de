"""The single-launch iteration on chunks described by lists alone (offsets,
values and lane masks per 64 rows) against the oracle and, bit for bit,
against the same iteration on per-entry columns.

The rows of both storages add the same products in the same order (a missing
entry adds an exact zero), so equality is exact; against the oracle the
iterates are held to the 1e-10 bar of every fixed-iteration test.
"""

import numpy as np
import pytest

import oracle
from paper_2105_06176_amd import ppcg
from paper_2105_06176_amd.ppcg import Solver, solve_batch
from workloads import CSR, poisson2d, poisson3d, poisson125, rhs_from_solution, shifted, xstar_uniform
from workloads.gen import _constant_stencil

pytestmark = pytest.mark.gpu

FORM = ppcg.FLAG_ITER_FUSED | ppcg.FLAG_SELL_VALUE_TABLE
LISTS, COLUMNS = FORM | ppcg.FLAG_SELL_SHARED_OFFSETS, FORM | ppcg.FLAG_SELL_NO_SHARED_OFFSETS


def dev(a):
    import torch

    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64)).cuda()


def host(t):
    return t.cpu().numpy()


def tridiagonal(n, off, diag=4.0):
    """off[i] couples rows i and i + 1; an entry is stored also where it is 0."""
    import scipy.sparse as sp

    M = sp.diags([np.ones(n - 1), np.ones(n), np.ones(n - 1)], [-1, 0, 1], format="csr")
    M.sort_indices()
    rows = np.repeat(np.arange(n), np.diff(M.indptr))
    lo = np.minimum(rows, M.indices)
    val = np.where(rows == M.indices, diag, np.append(off, 0.0)[lo])
    return CSR(n, M.indptr.astype(np.int32), M.indices.astype(np.int32), val.astype(np.float64), f"tri{n}")


def box(nx, ny, nz):
    offs = [(0, 0, -1), (0, -1, 0), (-1, 0, 0), (0, 0, 0), (1, 0, 0), (0, 1, 0), (0, 0, 1)]
    return _constant_stencil((nx, ny, nz), offs, 6.5, -1.0, f"box_{nx}_{ny}_{nz}")


def halves(n, cut):
    """Off-diagonals -1 before row `cut`, -0.5 after it."""
    return tridiagonal(n, np.where(np.arange(n - 1) < cut, -1.0, -0.5))


def stored_zeros(n):
    off = np.full(n - 1, -1.0)
    off[::7] = 0.0
    off[3::11] = -0.0
    return tridiagonal(n, off)


# matrix, iterations, whether each entry of a chunk's list has one value
CASES = {
    "one_row": (lambda: CSR(1, np.array([0, 1], np.int32), np.zeros(1, np.int32), np.array([2.0])), 1, True),
    "65_rows": (lambda: tridiagonal(65, np.full(64, -1.0)), 5, True),
    "diagonal_only": (lambda: CSR(5000, np.arange(5001, dtype=np.int32), np.arange(5000, dtype=np.int32),
                                  np.full(5000, 3.0)), 1, True),
    "poisson2d_67": (lambda: poisson2d(67), 30, True),
    "poisson2d_301": (lambda: poisson2d(301), 25, True),
    "poisson3d_17": (lambda: poisson3d(17), 12, True),
    "lines_of_3": (lambda: box(3, 40, 30), 15, True),
    "lines_of_64": (lambda: box(64, 9, 11), 15, True),
    "lines_of_63": (lambda: box(63, 9, 11), 15, True),
    "poisson125_40": (lambda: poisson125(40), 8, True),
    "halves_on_a_chunk_border": (lambda: halves(6400, 3199), 20, False),  # the entry 3199-3200 crosses the chunks
    "halves_inside_a_chunk": (lambda: halves(6400, 3220), 20, False),
    "stored_zeros": (lambda: stored_zeros(5003), 20, False),  # -0.0 is a value of its own beside -1
    "five_rows_per_thread": (lambda: poisson3d(124), 5, True),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_lists_equal_columns_and_oracle(name):
    gen, k, lists = CASES[name]
    A = gen()
    b = rhs_from_solution(A, xstar_uniform(A.n, 3))
    S = Solver(A, fixed_iters=k, spmv_format="sell", flags=LISTS)
    N = Solver(A, fixed_iters=k, spmv_format="sell", flags=COLUMNS)
    mi = S.matrix_info()
    if A.n > 64:  # beside the gathered vector: 16 bytes per 64 rows, or at least one per entry
        per_row = (mi["bytes_spmv"] - 8.0 * A.n) / A.n
        assert (per_row < 0.9) == (lists and mi["col_index_bytes"] == 0), per_row
    if name.startswith("poisson2d") or "125" in name:
        assert mi["col_index_bytes"] == 0
    x, info = S.solve(dev(b))
    y, _ = N.solve(dev(b))
    ref = oracle.pipecg(A, b, fixed_iters=k)
    assert info["status"] == ppcg.OK and info["iters"] == ref.iters
    assert np.array_equal(host(x), host(y))
    assert np.linalg.norm(host(x) - ref.x) <= 1e-10 * np.linalg.norm(ref.x)
    for s in (S, N):
        s.close()


def runs(nx, ny, nz, rx, ry, rz):
    """Runs of 2 rx + 1 consecutive columns, (2 ry + 1) (2 rz + 1) of them."""
    offs = [(i, j, k) for k in range(-rz, rz + 1) for j in range(-ry, ry + 1) for i in range(-rx, rx + 1)]
    return _constant_stencil((nx, ny, nz), offs, len(offs) - 0.5, -1.0, f"runs_{nx}_{ny}_{nz}_{rx}{ry}{rz}")


# steps of three runs, what remains after them, runs on the edges of the vector and of its lines
RUNS = [(1000, 1, 1, 2, 0, 0), (100, 60, 1, 2, 1, 0), (61, 97, 1, 2, 2, 0), (90, 70, 1, 1, 1, 0), (40, 40, 40, 1, 1, 1),
        (64, 60, 30, 1, 1, 1), (53, 50, 41, 2, 2, 2), (65, 40, 40, 2, 1, 2), (101, 50, 1, 3, 1, 0)]
# rows sorted by length: per-entry columns
SORTED = [(33, 20, 17, 1, 1, 1), (3, 40, 40, 1, 1, 1), (5, 30, 31, 2, 2, 2), (37, 11, 13, 2, 2, 2)]


@pytest.mark.parametrize("shape", RUNS + SORTED, ids=lambda t: "_".join(map(str, t)))
def test_runs_equal_columns_and_oracle(shape):
    A = runs(*shape)
    b = rhs_from_solution(A, xstar_uniform(A.n, 4))
    S = Solver(A, fixed_iters=8, spmv_format="sell", flags=LISTS)
    N = Solver(A, fixed_iters=8, spmv_format="sell", flags=COLUMNS)
    assert (S.matrix_info()["col_index_bytes"] == 0) == (shape in RUNS)
    x, info = S.solve(dev(b))
    y, _ = N.solve(dev(b))
    ref = oracle.pipecg(A, b, fixed_iters=8)
    assert info["status"] == ppcg.OK and info["iters"] == ref.iters
    assert np.array_equal(host(x), host(y))
    assert np.linalg.norm(host(x) - ref.x) <= 1e-10 * np.linalg.norm(ref.x)
    S.close()
    N.close()


# matrix, whether the lists are taken untimed (else left to the timing)
AUTO = {
    "runs_16_16_16": (lambda: runs(16, 16, 16, 2, 2, 2), True),
    "runs_17_30_23": (lambda: runs(17, 30, 23, 2, 2, 2), True),
    "runs_33_20_17": (lambda: runs(33, 20, 17, 1, 1, 1), True),
    "runs_5_30_31": (lambda: runs(5, 30, 31, 2, 2, 2), False),  # 2.1 stored entries per entry
    "poisson2d_33": (lambda: poisson2d(33), True),
    "box_24_40_18": (lambda: box(24, 40, 18), True),
    "halves": (lambda: halves(6400, 3220), False),  # two values of an entry in a chunk
    "one_row": (CASES["one_row"][0], True),
}


@pytest.mark.parametrize("name", sorted(AUTO))
@pytest.mark.parametrize("k", [1, 9])
def test_automatic_choice_and_oracle(name, k):
    gen, lists = AUTO[name]
    A = gen()
    k = min(k, A.n)
    b = rhs_from_solution(A, xstar_uniform(A.n, 6))
    ref = oracle.pipecg(A, b, fixed_iters=k)
    for _ in range(2):  # the second handle meets what the first one left
        S = Solver(A, fixed_iters=k)
        if lists:
            assert S.matrix_info()["col_index_bytes"] == 0
        x, info = S.solve(dev(b))
        assert info["status"] == ppcg.OK and info["iters"] == ref.iters
        assert np.linalg.norm(host(x) - ref.x) <= 1e-10 * np.linalg.norm(ref.x)
        S.close()


def test_batch_with_and_without_runs_equals_solo_bitwise():
    mats = [poisson3d(20), runs(53, 50, 41, 2, 2, 2), poisson2d(80), runs(40, 40, 40, 1, 1, 1)]
    bs = [rhs_from_solution(A, xstar_uniform(A.n, 5 + i)) for i, A in enumerate(mats)]
    solvers = [Solver(A, tol=1e-9, spmv_format="sell", flags=LISTS) for A in mats]
    solo = [s.solve(dev(b)) for s, b in zip(solvers, bs)]
    for _ in range(2):
        xs, infos = solve_batch(solvers, [dev(b) for b in bs])
        for x, info, (y, one) in zip(xs, infos, solo):
            assert info["iters"] == one["iters"] and np.array_equal(host(x), host(y))
    for s in solvers:
        s.close()


@pytest.mark.parametrize("name", ["poisson2d_67", "lines_of_63", "poisson125_40", "halves_inside_a_chunk"])
def test_spmv_and_initial_guess_on_lists(name):
    """The SpMV, the initialisation from a guess and the true residual read the lists too (no value table is built):
    bit for bit the oracle's product and the per-entry columns' solve."""
    gen, k, _ = CASES[name]
    A = gen()
    b = rhs_from_solution(A, xstar_uniform(A.n, 3))
    x0 = xstar_uniform(A.n, 8)
    S = Solver(A, fixed_iters=k, spmv_format="sell", flags=ppcg.FLAG_ITER_FUSED | ppcg.FLAG_SELL_SHARED_OFFSETS)
    N = Solver(A, fixed_iters=k, spmv_format="sell", flags=COLUMNS)
    assert np.array_equal(host(S.spmv(dev(x0))), oracle.spmv(A, x0))
    x, info = S.solve(dev(b), x0=dev(x0))
    y, other = N.solve(dev(b), x0=dev(x0))
    assert np.array_equal(host(x), host(y)) and info["rel_resid_true"] == other["rel_resid_true"]
    for s in (S, N):
        s.close()


@pytest.mark.parametrize("gen", [lambda: poisson2d(67), lambda: box(63, 9, 11), lambda: poisson3d(40)])
@pytest.mark.parametrize("prec", ["fp64", "mixed", "mixed_values"])
def test_classic_pcg_on_lists(gen, prec):
    """Algorithm 1 reads the lists in every precision (FP32 values are the rounded list values): bit for bit the
    per-entry columns' solve, with the tiles of its two launches ragged at these sizes."""
    A = gen()
    b = rhs_from_solution(A, xstar_uniform(A.n, 6))
    res = []
    for flags in (ppcg.FLAG_SELL_SHARED_OFFSETS, ppcg.FLAG_SELL_NO_SHARED_OFFSETS):
        S = Solver(A, tol=1e-10, method="pcg", precision=prec, spmv_format="sell", flags=flags)
        x, info = S.solve(dev(b))
        assert info["status"] == ppcg.OK and oracle.true_relres(A, b, host(x)) <= 1e-10
        res.append((host(x), info["iters"], info["outer_iters"]))
        S.close()
    assert np.array_equal(res[0][0], res[1][0]) and res[0][1:] == res[1][1:]


@pytest.mark.parametrize("gen", [lambda: tridiagonal(2, np.full(1, -1.0)), lambda: tridiagonal(63, np.full(62, -1.0)),
                                 lambda: tridiagonal(1025, np.full(1024, -1.0)), lambda: poisson2d(32),
                                 lambda: poisson2d(63), lambda: poisson2d(64), lambda: box(15, 16, 17),
                                 lambda: halves(4000, 2020)])
def test_one_workgroup_kernel_reads_every_storage_alike(gen):
    """At most 4,096 rows: the matrix from lists, staged in LDS through the value table, or from memory; 1 to 4 rows
    per thread, full and ragged wavefronts.  Equal bit for bit, and the oracle's iterates to 1e-10."""
    A = gen()
    b = rhs_from_solution(A, xstar_uniform(A.n, 5))
    k = min(20, A.n - 1)
    xs = []
    for flags in (0, ppcg.FLAG_SELL_VALUE_TABLE | ppcg.FLAG_SELL_NO_SHARED_OFFSETS, ppcg.FLAG_SELL_FULL_VALUES):
        S = Solver(A, fixed_iters=k, spmv_format="sell", flags=flags)
        x, info = S.solve(dev(b))
        ref = oracle.pipecg(A, b, fixed_iters=k)
        assert info["iters"] == ref.iters
        assert np.linalg.norm(host(x) - ref.x) <= 1e-10 * np.linalg.norm(ref.x)
        xs.append(host(x))
        S.close()
    assert np.array_equal(xs[0], xs[1]) and np.array_equal(xs[0], xs[2])


def test_batch_of_list_and_column_systems_equals_solo_bitwise():
    """Both kernels in one batch, twice (captured graphs replayed), with systems that end at different times."""
    mats = [poisson2d(80), shifted(poisson2d(121), 0.3), poisson3d(33), box(31, 17, 20), poisson2d(40)]
    flags = [0, LISTS, COLUMNS, 0, 0]
    bs = [rhs_from_solution(A, xstar_uniform(A.n, 9 + i)) for i, A in enumerate(mats)]
    solvers = [Solver(A, tol=1e-10, spmv_format="sell", flags=f) for A, f in zip(mats, flags)]
    solo = [s.solve(dev(b)) for s, b in zip(solvers, bs)]
    for _ in range(2):
        xs, infos = solve_batch(solvers, [dev(b) for b in bs])
        for A, b, x, info, (sx, si) in zip(mats, bs, xs, infos, solo):
            assert np.array_equal(host(x), host(sx)) and info["iters"] == si["iters"], A.name
            assert oracle.true_relres(A, b, host(x)) <= 1e-10
            assert abs(info["iters"] - oracle.pipecg(A, b, tol=1e-10).iters) <= 2
    for s in solvers:
        s.close()
