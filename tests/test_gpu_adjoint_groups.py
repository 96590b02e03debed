"""The particle adjoints' lane groups.  The group width follows from the mean
occupancy (64 lanes per cell from 256 particles on, down to 8), and the small
grids of the oracle tests take 64 lanes; here the same particles, all at once
(64 lanes) and in interleaved parts (32, 16 and 8 lanes), give the same
cotangents: per particle, and summed over the parts on the grid.  Both sides
form the same FP64 terms; the grid sums add up to a few thousand of them in
another order (1e-12 of the largest)."""
import numpy as np
import pytest

import oracle
from tests.gpu_helpers import load, make_ctx, need_gpu, random_cells

pytestmark = pytest.mark.gpu

GRIDS = {
    "2d": oracle.Grid(dim=2, nx=130, ny=64, dx=1.0, dy=0.9, dt=0.4),
    "3d": oracle.Grid(dim=3, nx=24, ny=20, nz=18, dx=1.0, dy=0.9, dz=1.1, dt=0.4, q=(1.0, -1.0, 2.0),
                      m=(1.0, 1.0, 3.0)),
}


def cotangents(ctx, g, state, fields, lam):
    import torch

    from paper_2509_11100_amd import relsim

    parts = load(ctx, *state)
    _ = parts.cell  # the adjoints need the cell ids written
    B, Eth, mu = fields
    dev = dict(dtype=torch.float64, device="cuda")
    lx, lu = (torch.as_tensor(np.ascontiguousarray(a)).cuda() for a in lam)
    out = {"lx": torch.empty_like(lx), "lu": torch.empty_like(lu)}
    lE, lB = torch.ones((3, g.N), **dev), torch.ones((3, g.N), **dev)  # accumulated into
    relsim.push_adjoint(ctx, parts, Eth, B, None, lx, lu, out["lx"], out["lu"], lE, lB)
    lBd = torch.zeros((3, g.N), **dev)
    relsim.deposit_adjoint(ctx, parts, B, Eth, mu, out["lx"], out["lu"], lBd)
    return {k: v.cpu().numpy() for k, v in out.items()}, [(t.cpu().numpy() - o) for t, o in ((lE, 1), (lB, 1),
                                                                                             (lBd, 0))]


@pytest.mark.parametrize("gname", list(GRIDS))
def test_group_widths_give_the_same_cotangents(gname):
    need_gpu()
    import torch

    g = GRIDS[gname]
    n = 260 * g.N
    rng = np.random.default_rng(17)
    cell, sp, off, u, w = random_cells(g, n, rng, umax=2.0)
    order = np.argsort(cell.astype(np.int64) * len(g.q) + sp, kind="stable")
    cell, sp, off, u, w = cell[order], sp[order], off[:, order], u[:, order], w[order]
    fields = [torch.as_tensor((2 * rng.random((3, g.N)) - 1) * s).cuda() for s in (2.0, 0.5, 0.3)]
    lx, lu = rng.standard_normal((g.dim, n)), rng.standard_normal((3, n))
    ctx = make_ctx(g, "fp64", n)
    whole, grid = cotangents(ctx, g, (cell, sp, off, u, w), fields, (lx, lu))
    for k in (2, 4, 16):
        sums = [0.0, 0.0, 0.0]
        for part in range(k):
            s = slice(part, n, k)
            got, gg = cotangents(ctx, g, (cell[s], sp[s], off[:, s], u[:, s], w[s]), fields, (lx[:, s], lu[:, s]))
            for name in got:
                ref = whole[name][:, s]
                assert np.abs(got[name] - ref).max() <= 1e-13 * np.abs(ref).max()
            sums = [a + b for a, b in zip(sums, gg)]
        for a, b in zip(sums, grid):
            assert np.abs(a - b).max() <= 1e-12 * np.abs(b).max()
