"""The transposed 3D operator on grids whose march tiles hold several rows and
planes, with shorter last tiles along y and z (5 rows x 3 planes and 4 x 4),
and on one whose rows take two tiles: A^T x and A x against the oracle's
product, and a transposed solve by its true residual.

The stored block of a node pair is one 3 x 3 block for both orders of the
pair, so the transpose has the same blocks transposed.  A^T x sums about 100
products per entry; 1e-13 of the largest is allowed."""
import numpy as np
import pytest

import oracle
from tests.gpu_helpers import load, make_ctx, need_gpu, random_cells
from tests.helpers import full_from_half

pytestmark = pytest.mark.gpu

RTOL = 1e-12


def transposed(M):
    return np.ascontiguousarray(M.reshape(M.shape[0], 3, 3, -1).transpose(0, 2, 1, 3).reshape(M.shape))


def dev(a):
    import torch

    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64)).cuda()


@pytest.mark.parametrize("mass", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", [(96, 47, 33), (63, 31, 62), (37, 50, 29)])
def test_transposed_march_over_rows_and_planes(shape, mass):
    need_gpu()
    from paper_2509_11100_amd import relsim

    g = oracle.Grid(dim=3, nx=shape[0], ny=shape[1], nz=shape[2], dx=1.0, dy=0.9, dz=1.1, dt=0.4)
    rng = np.random.default_rng(11)
    n = 3 * g.N
    kw = {"mass_fp32": True} if mass == "fp32" else {}
    ctx = make_ctx(g, "mixed" if mass == "fp32" else "fp64", n, rtol=RTOL, **kw)
    parts = load(ctx, *random_cells(g, n, rng, empty_frac=0.2))
    J, M = relsim.deposit_moments(ctx, parts, dev((2 * rng.random((3, g.N)) - 1) * 2.0))
    x = 2 * rng.random((3, g.N)) - 1
    Mf = full_from_half(g, M.cpu().numpy().astype(np.float64))
    Mt = transposed(Mf)
    for got, ref in ((relsim.apply_AT(ctx, M, dev(x)), oracle.apply_A(g, Mt, x)),
                     (relsim.apply_A(ctx, M, dev(x)), oracle.apply_A(g, Mf, x))):
        assert np.abs(got.cpu().numpy() - ref).max() <= 1e-13 * np.abs(ref).max()
    if mass == "fp32":
        return  # the Python call of the transposed solve takes M in FP64 only
    l_th, l_E, l_B = (2 * rng.random((3, g.N)) - 1 for _ in range(3))
    mu, lE, lB = ctx.grid(), ctx.grid(), ctx.grid()
    it, rr = relsim.field_solve_adjoint(ctx, M, dev(l_th), dev(l_E), dev(l_B), mu, lE, lB)
    b = l_th + l_E / g.theta - g.c * g.dt * oracle.curl_cn(g, l_B)
    mu = mu.cpu().numpy()
    res = np.linalg.norm(b - oracle.apply_A(g, Mt, mu)) / np.linalg.norm(b)
    assert it > 0 and rr <= RTOL and abs(res - rr) <= 1e-13
    ref = l_B + g.c * g.theta * g.dt * oracle.curl_nc(g, mu)
    assert np.abs(lB.cpu().numpy() - ref).max() <= 1e-13 * np.abs(ref).max()
