"""Device memory that a server keeps between its requests: reused by later ones of other sizes and precisions, held
within the budget, and given back with the server."""

import threading

import numpy as np
import pytest

import oracle
from paper_2105_06176_amd import ppcg
from paper_2105_06176_amd.ppcg import Server
from workloads import poisson2d, poisson3d, random_spd, rhs_from_solution, shifted, xstar_uniform

pytestmark = pytest.mark.gpu

SYSTEMS = [poisson2d(40), random_spd(3000), poisson3d(20), shifted(poisson2d(91), 0.2), poisson2d(64), random_spd(20000)]


def burst(server, rounds, errors):
    """The systems in another order each round, each checked against its tolerance and the exact solution."""
    try:
        for r in range(rounds):
            todo = {}
            for k in np.roll(np.arange(len(SYSTEMS)), r):
                A = SYSTEMS[k]
                xs = xstar_uniform(A.n, 10 * r + int(k))
                b = rhs_from_solution(A, xs)
                prec = "mixed" if (r + k) % 4 == 3 else "fp64"
                todo[server.submit(A, b, 1e-10, prec)] = (A, b)
            while todo:
                server.step()
                for rid in list(todo):
                    got = server.poll(rid)
                    if got is not None:
                        A, b = todo.pop(rid)
                        x, info = got
                        assert info["status"] == ppcg.OK
                        assert oracle.true_relres(A, b, x) <= 2e-10
    except BaseException as e:  # noqa: BLE001 - reported by the test
        errors.append(e)


def two_servers(budget):
    errors = []
    servers = [Server(budget_bytes=budget) for _ in range(2)]
    threads = [threading.Thread(target=burst, args=(s, 3, errors)) for s in servers]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for s in servers:
        s.close()
    assert not errors, errors


@pytest.mark.parametrize("budget", [0.0, 30e6])
def test_bursts_reuse_memory_and_give_it_back(budget):
    import torch

    two_servers(budget)  # what the runtime allocates once
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    two_servers(budget)
    assert before - torch.cuda.mem_get_info()[0] < 16 << 20
