"""Tile shapes of the single-launch form that only some storages or sizes reach: k_fused's rows per thread on
constant-coefficient grids (which otherwise iterate on chunk lists), and k_stencil above 8.4 million rows, where the
ring of residuals is on again and a thread sums more than two tiles' records."""

import numpy as np
import pytest

import oracle
from paper_2105_06176_amd import ppcg
from paper_2105_06176_amd.ppcg import Solver
from test_gpu_fused import CASES, FUSED
from test_gpu_stencil import COLUMNS, LISTS, dev, host
from workloads import rhs_from_solution, xstar_uniform

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["c1_poisson2d_64", "poisson2d_100_ragged", "poisson3d_40", "tile_and_68_rows",
                                  "poisson2d_600_three_rows", "poisson3d_124_five_rows",
                                  "poisson2d_2000_sixteen_rows"])
def test_k_fused_tile_shapes(name):
    gen, ks, _ = CASES[name]
    A = gen()
    b = rhs_from_solution(A, xstar_uniform(A.n, 3))
    S = Solver(A, fixed_iters=1, spmv_format="sell", flags=FUSED | ppcg.FLAG_SELL_NO_SHARED_OFFSETS)
    mi = S.matrix_info()
    assert mi["iter_launches"] == 1 and mi["bytes_spmv"] > 12.0 * A.n  # per-entry storage
    for k in ks:
        S.set_options(fixed_iters=k)
        x, info = S.solve(dev(b))
        ref = oracle.pipecg(A, b, fixed_iters=k)
        assert info["status"] == ppcg.OK and info["iters"] == k
        assert np.linalg.norm(host(x) - ref.x) <= 1e-10 * np.linalg.norm(ref.x)
    S.close()


def device_box(nx, ny, nz):
    """7-point CSR on the device, x varying fastest."""
    import torch

    n = nx * ny * nz
    i = torch.arange(n, dtype=torch.int32, device="cuda")
    x, y, z = i % nx, i // nx % ny, i // (nx * ny)
    ok = torch.stack([z > 0, y > 0, x > 0, x >= 0, x < nx - 1, y < ny - 1, z < nz - 1], 1)
    step = torch.tensor([-nx * ny, -nx, -1, 0, 1, nx, nx * ny], dtype=torch.int32, device="cuda")
    val = torch.tensor([-1.0, -1.0, -1.0, 6.5, -1.0, -1.0, -1.0], dtype=torch.float64, device="cuda")
    rp = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    rp[1:] = torch.cumsum(ok.sum(1), 0)
    return rp, (i[:, None] + step)[ok], val.expand(n, 7)[ok]


@pytest.mark.parametrize("shape", [(210, 210, 204), (181, 211, 131), (250, 400, 250)], ids=lambda s: "_".join(map(str, s)))
def test_lists_equal_columns_on_large_boxes(shape):
    """8,996,400 rows: 1,099 tiles of 8,192 rows.  5,003,021 rows: the ring
    on again above 4.79 million.  25,000,000 rows: the most that lists take, byte offsets of ten vectors up to 2e9."""
    import torch

    A = device_box(*shape)
    n = shape[0] * shape[1] * shape[2]
    g = torch.Generator(device="cuda").manual_seed(5)
    b = torch.rand(n, dtype=torch.float64, device="cuda", generator=g) - 0.5
    xs = []
    for flags in (LISTS, COLUMNS):
        S = Solver(A, fixed_iters=7, spmv_format="sell", flags=flags)
        assert (S.matrix_info()["bytes_spmv"] < 9.0 * n) == (flags == LISTS)
        x, info = S.solve(b)
        assert info["status"] == ppcg.OK and info["iters"] == 7
        xs.append(x)
        S.close()
    assert torch.equal(xs[0], xs[1])
