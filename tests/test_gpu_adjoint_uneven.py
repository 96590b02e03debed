"""The particle adjoints' lane groups on cells filled unevenly, as a sheet's: a
third of the cells empty, three rows holding most of the particles, species
missing from many cells.  As on evenly filled cells, the same particles all at
once (32 lanes per cell) and in interleaved parts (16 and 8 lanes) give the same
cotangents: per particle (1e-13), and summed over the parts on the grid, where
up to ten thousand terms are added in another order (1e-12 of the largest)."""
import numpy as np
import pytest

from tests.gpu_helpers import make_ctx, need_gpu, random_cells
from tests.test_gpu_adjoint_groups import GRIDS, cotangents

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gname", list(GRIDS))
def test_uneven_cells_give_the_same_cotangents(gname):
    need_gpu()
    import torch

    g = GRIDS[gname]
    S = len(g.q)
    n = 150 * g.N
    rng = np.random.default_rng(19)
    cell, sp, off, u, w = random_cells(g, n, rng, umax=2.0, empty_frac=0.33)
    crowded = rng.random(n) < 0.7
    cell[crowded] = (cell[crowded] % g.nx) + g.nx * (g.ny // 2 + rng.integers(0, 3, int(crowded.sum())))
    sp[cell % 3 == 0] = S - 1
    sp[cell % 5 == 0] = 0
    off[:, :3] = [[0.0], [0.5], [1.0 - 2.0 ** -53]][: g.dim]
    order = np.argsort(cell.astype(np.int64) * S + sp, kind="stable")
    cell, sp, off, u, w = cell[order], sp[order], off[:, order], u[:, order], w[order]
    fields = [torch.as_tensor((2 * rng.random((3, g.N)) - 1) * s).cuda() for s in (2.0, 0.5, 0.3)]
    lx, lu = rng.standard_normal((g.dim, n)), rng.standard_normal((3, n))
    ctx = make_ctx(g, "fp64", n)
    whole, grid = cotangents(ctx, g, (cell, sp, off, u, w), fields, (lx, lu))
    for k in (2, 8):
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
