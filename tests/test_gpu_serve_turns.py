"""Large requests of a server iterate in turn, smaller ones beside them; the length of a lone request's chunks."""

import numpy as np
import pytest
import torch

from paper_2105_06176_amd import ppcg
from paper_2105_06176_amd.ppcg import Server, Solver
from workloads import poisson2d, poisson3d, rhs_from_solution, xstar_uniform

pytestmark = pytest.mark.gpu


def problem(A):
    return rhs_from_solution(A, xstar_uniform(A.n, 3))


def alone(A, b, tol):
    S = Solver(A, tol=tol, vec_mem="host")
    x = torch.empty(A.n, dtype=torch.float64)
    _, info = S.solve(torch.as_tensor(b), out=x)
    mi = S.matrix_info()
    S.close()
    return x.numpy(), info, mi


def drain(server, ids):
    """Results, the order of the ends, the most active at a time."""
    res, order, most = {}, [], 0
    while len(res) < len(ids):
        active, _ = server.step()
        most = max(most, active)
        for rid in ids:
            if rid not in res:
                r = server.poll(rid)
                if r is not None:
                    res[rid] = r
                    order.append(rid)
    return res, order, most


def test_large_requests_take_turns():
    """Ten systems of 78 MB an iteration: three of them fit 256 MiB (up to three more are counted as active while their
    solutions are copied out), each with its solo result."""
    A = poisson2d(1000)
    b = problem(A)
    x, info, mi = alone(A, b, 1e-8)
    assert 256 * 2**20 // mi["bytes_per_iter"] == 3
    server = Server()
    ids = [server.submit(A, b, 1e-8, "fp64") for _ in range(10)]
    res, _, most = drain(server, ids)
    server.close()
    for rid in ids:
        assert np.array_equal(res[rid][0], x) and res[rid][1]["iters"] == info["iters"]
    assert most <= 6


def test_a_small_request_passes_a_waiting_large_one():
    A, small = poisson2d(1000), poisson2d(60)
    b, bs = problem(A), problem(small)
    x, info, _ = alone(small, bs, 1e-8)
    server = Server()
    large = [server.submit(A, b, 1e-8, "fp64") for _ in range(5)]
    rid = server.submit(small, bs, 1e-8, "fp64")
    res, order, _ = drain(server, large + [rid])
    server.close()
    assert all(res[k][1]["status"] == ppcg.OK for k in large)
    assert np.array_equal(res[rid][0], x) and res[rid][1]["iters"] == info["iters"]
    assert order.index(rid) < len(order) - 2  # before the two that waited


@pytest.mark.parametrize("gen,chunk", [(lambda: poisson3d(160), 8), (lambda: poisson2d(150), 32)])
def test_chunks_of_a_lone_request(gen, chunk):
    """Iterations between two polls with nothing else to run: as many as move 5e9 bytes, 8 to 32.  The start, the end
    and the wait for the solution take up to six steps."""
    A = gen()
    b = problem(A)
    mi = alone(A, b, 1e-3)[2]
    assert chunk * mi["bytes_per_iter"] <= 5e9 and (chunk == 32 or 2 * chunk * mi["bytes_per_iter"] > 5e9)
    server = Server()
    rid = server.submit(A, b, 1e-6, "fp64")
    steps, got = 0, None
    while got is None:
        server.step()
        steps += 1
        got = server.poll(rid)
    server.close()
    iters = got[1]["iters"]
    assert iters >= 5 * chunk
    assert iters // chunk <= steps <= iters // chunk + 6, (iters, steps)
