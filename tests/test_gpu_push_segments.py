"""The push passes' row segments on extents that no power of two divides: the
last segment of a row is shorter and the last tiles reach past the grid.  The
push with re-sort against the push in place followed by a stable sort on the
host (bit for bit), and its kinetic sum against relsim_energy (both sum the
same FP64 terms, to 1e-13)."""
import numpy as np
import pytest

import oracle
from tests.gpu_helpers import host_state, load, make_ctx, need_gpu, random_cells

pytestmark = pytest.mark.gpu

# cells per wave (counting pass, scatter) at these occupancies: (8, 8), (2, 1)
# beside a crowded band of rows, (8, 4) and (16, 16)
CASES = {
    "2d_131x129": (oracle.Grid(dim=2, nx=131, ny=129, dx=1.0, dy=0.9, dt=0.4), 60000, 0.0),
    "2d_67x65_crowded_rows": (oracle.Grid(dim=2, nx=67, ny=65, dx=1.0, dy=0.9, dt=0.4), 300000, 0.9),
    "2d_203x101_three_species": (oracle.Grid(dim=2, nx=203, ny=101, dx=1.0, dy=1.1, dt=0.4, q=(1.0, -1.0, 2.0),
                                             m=(1.0, 1.0, 3.0)), 700000, 0.0),
    # crowded segments split over several waves: 2 parts of 2 cells (counting
    # pass) and 3 (scatter), the 1-cell segments at the rows' ends whole; 5 and
    # 8 parts of 8 cells
    "2d_97x89_split_three_species": (oracle.Grid(dim=2, nx=97, ny=89, dx=1.0, dy=1.1, dt=0.4, q=(1.0, -1.0, 2.0),
                                                 m=(1.0, 1.0, 3.0)), 120000, 0.7),
    "3d_29x27x23_split": (oracle.Grid(dim=3, nx=29, ny=27, nz=23, dx=1.0, dy=0.9, dz=1.1, dt=0.4), 100000, 0.5),
    "3d_37x35x33": (oracle.Grid(dim=3, nx=37, ny=35, nz=33, dx=1.0, dy=0.9, dz=1.1, dt=0.4), 50000, 0.0),
}


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("name", list(CASES))
def test_resort_on_extents_that_segments_do_not_divide(name, precision):
    need_gpu()
    import torch

    from paper_2509_11100_amd import relsim

    g, n, crowded = CASES[name]
    rng = np.random.default_rng(31)
    cell, sp, off, u, w = random_cells(g, n, rng, umax=2.0)
    band = rng.random(n) < crowded  # this share of the particles sits in three rows
    cell[band] = (cell[band] % g.nx) + g.nx * (g.ny // 2 + rng.integers(0, 3, int(band.sum())))
    B = torch.as_tensor((2 * rng.random((3, g.N)) - 1) * 2.0).cuda()
    E = torch.as_tensor((2 * rng.random((3, g.N)) - 1) * 0.5).cuda()
    ctx = make_ctx(g, precision, n)
    parts = load(ctx, cell, sp, off, u, w)
    ctx2 = make_ctx(g, precision, n)
    flat = load(ctx2, *parts.to_host())
    relsim.push(ctx2, flat, E, B, resort=False)
    perm = torch.empty(n, dtype=torch.int32, device="cuda")
    relsim.push(ctx, parts, E, B, resort=True, new_index=perm)
    W = relsim.energy_pushed(ctx, E, B)
    ref = relsim.energy(ctx, parts, E, B)
    assert np.all(np.abs(W - ref) <= 1e-13 * np.abs(ref))
    assert relsim.placement_clamps(ctx) == 0

    s1, s2 = host_state(g, parts), host_state(g, flat)
    S, N, ext = len(g.q), g.N, [g.nx, g.ny, g.nz]
    f = flat.to_host()[2]
    c = s2["cell"].astype(np.int64)
    coords = [c % g.nx, (c // g.nx) % g.ny, c // (g.nx * g.ny)]
    one = f.dtype.type(1)
    for d in range(g.dim):
        m = np.where(f[d] >= 1, 1, np.where(f[d] < 0, -1, 0))
        moved = (f[d] - m.astype(f.dtype)).astype(f.dtype)
        edge = (m == -1) & (moved == one)  # just below 0: stays, at the face
        f[d] = np.where(edge, 0, moved)
        coords[d] = (coords[d] + np.where(edge, 0, m)) % ext[d]
    bins = (coords[0] + g.nx * (coords[1] + (g.ny * coords[2] if g.dim == 3 else 0))) * S + s2["species"]
    order = np.argsort(bins, kind="stable")
    np.testing.assert_array_equal(s1["bin_start"], np.searchsorted(np.sort(bins), np.arange(N * S + 1)))
    np.testing.assert_array_equal(s1["off"], f[:, order].astype(np.float64))
    np.testing.assert_array_equal(s1["u"], s2["u"][:, order])
    np.testing.assert_array_equal(s1["w"], s2["w"][order])
    np.testing.assert_array_equal(perm.cpu().numpy()[order], np.arange(n))
