"""The end of a GMRES cycle, which every block of a kernel finds for itself
while one block records it: solves of many short cycles on grids of many
blocks come out the same bit for bit every time, and their residual is the
oracle's (b formed and A applied on the host; both round at a few 1e-16 of
||A|| ||x|| + ||b||, 1e-13 allowed)."""
import numpy as np
import pytest

import oracle
from tests.gpu_helpers import load, make_ctx, need_gpu, random_cells
from tests.helpers import full_from_half

pytestmark = pytest.mark.gpu

RTOL = 1e-10


@pytest.mark.parametrize("restart", [1, 2, 5])
@pytest.mark.parametrize("shape", [(300, 211), (48, 41, 37)])
def test_short_cycles_on_many_blocks_repeat_bit_for_bit(shape, restart):
    need_gpu()
    import torch

    from paper_2509_11100_amd import relsim

    dim = len(shape)
    g = oracle.Grid(dim=dim, nx=shape[0], ny=shape[1], nz=shape[2] if dim == 3 else 1, dx=1.0, dy=0.9, dz=1.1, dt=0.4)
    rng = np.random.default_rng(7)
    n = 3 * g.N
    ctx = make_ctx(g, "fp64", n, rtol=RTOL, gmres_restart=restart, gmres_maxit=2000)
    parts = load(ctx, *random_cells(g, n, rng))
    E, B = (2 * rng.random((3, g.N)) - 1) * 0.5, (2 * rng.random((3, g.N)) - 1) * 2.0
    Et, Bt = torch.as_tensor(E).cuda(), torch.as_tensor(B).cuda()
    J, M = relsim.deposit_moments(ctx, parts, Bt)
    first = relsim.field_solve(ctx, M, J, Et, Bt)
    for _ in range(4):
        again = relsim.field_solve(ctx, M, J, Et, Bt)
        assert again[3:] == first[3:]
        assert all(torch.equal(a, b) for a, b in zip(first[:3], again[:3]))
    b = oracle.rhs(g, E, B, J.cpu().numpy())
    res = np.linalg.norm(b - oracle.apply_A(g, full_from_half(g, M.cpu().numpy()), first[0].cpu().numpy()))
    assert first[4] <= RTOL and abs(res / np.linalg.norm(b) - first[4]) <= 1e-13
