"""Cycles longer than the operator's kernel sums the dots of (16 columns in 2D, 8
in 3D; from there a kernel of their own has them, 16 vectors at a time): solves
of more than 34 steps in cycles of 64 and of 20, by the true residual
that the oracle's operator gives (1e-13 for its rounding and the solver's)."""
import numpy as np
import pytest

import oracle
from tests.gpu_helpers import load, make_ctx, need_gpu, random_cells
from tests.helpers import full_from_half

pytestmark = pytest.mark.gpu

RTOL = 1e-11


def dev(a):
    import torch

    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64)).cuda()


@pytest.mark.parametrize("restart", [20, 64])
@pytest.mark.parametrize("mass", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", [(37, 29), (300, 211), (13, 11, 9), (70, 26, 19)])
def test_long_cycles(shape, mass, restart):
    need_gpu()
    from paper_2509_11100_amd import relsim

    dim = len(shape)
    g = oracle.Grid(dim=dim, nx=shape[0], ny=shape[1], nz=shape[2] if dim == 3 else 1, dx=1.0, dy=0.9, dz=1.1, dt=0.4)
    rng = np.random.default_rng(29)
    n = 4 * g.N
    kw = {"mass_fp32": True} if mass == "fp32" else {}
    ctx = make_ctx(g, "mixed" if mass == "fp32" else "fp64", n, rtol=RTOL, gmres_restart=restart, **kw)
    parts = load(ctx, *random_cells(g, n, rng, empty_frac=0.2))
    E, B = (2 * rng.random((3, g.N)) - 1) * 0.5, (2 * rng.random((3, g.N)) - 1) * 2.0
    J, M = relsim.deposit_moments(ctx, parts, dev(B))
    M *= 40.0  # more steps: the curl-curl term and the identity matter less
    Eth, _, _, it, rr = relsim.field_solve(ctx, M, J, dev(E), dev(B))
    assert it > 34 and rr <= RTOL
    Mf = full_from_half(g, M.cpu().numpy().astype(np.float64))
    b = oracle.rhs(g, E, B, J.cpu().numpy())
    res = np.linalg.norm(b - oracle.apply_A(g, Mf, Eth.cpu().numpy())) / np.linalg.norm(b)
    assert abs(res - rr) <= 1e-13
    if mass == "fp32":
        return  # the Python call of the transposed solve takes M in FP64 only
    zero = ctx.grid()
    mu, lE, lB = ctx.grid(), ctx.grid(), ctx.grid()
    it, rr = relsim.field_solve_adjoint(ctx, M, dev(b), zero, zero, mu, lE, lB)
    assert it > 34 and rr <= RTOL
    Mt = np.ascontiguousarray(Mf.reshape(Mf.shape[0], 3, 3, -1).transpose(0, 2, 1, 3).reshape(Mf.shape))
    res = np.linalg.norm(b - oracle.apply_A(g, Mt, mu.cpu().numpy())) / np.linalg.norm(b)
    assert abs(res - rr) <= 1e-13
