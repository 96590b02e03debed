"""The lanes per cell that the 2D FP64 deposit takes by itself: 8 instead of 4
where the launch would have few waves or the plasma more than two species.  The
result is that of the group asked for, bit for bit (each group width adds a
cell's particles in an order of its own), and the widths differ by the rounding
of sums of up to a few hundred terms (1e-13 of the largest)."""
import numpy as np
import pytest

import oracle
from tests.gpu_helpers import load, make_ctx, need_gpu, random_cells

pytestmark = pytest.mark.gpu

# cells, species, particles per cell, lanes
CASES = [((130, 64), 2, 24, 8), ((130, 64), 2, 23, 4), ((257, 256), 2, 24, 4), ((257, 256), 3, 24, 8)]


@pytest.mark.parametrize("shape,species,mean,lanes", CASES)
def test_fp64_deposit_group(shape, species, mean, lanes):
    need_gpu()
    import torch

    from paper_2509_11100_amd import relsim

    g = oracle.Grid(dim=2, nx=shape[0], ny=shape[1], dx=1.0, dy=0.9, dt=0.4, q=(1.0, -1.0, 2.0)[:species],
                    m=(1.0, 1.0, 3.0)[:species])
    rng = np.random.default_rng(23)
    n = mean * g.N
    state = random_cells(g, n, rng, empty_frac=0.2)
    B = torch.as_tensor((2 * rng.random((3, g.N)) - 1) * 2.0).cuda()
    out = {}
    for group in (0, 4, 8):
        ctx = make_ctx(g, "fp64", n, group=group)
        out[group] = relsim.deposit_moments(ctx, load(ctx, *state), B)
    for a, b in zip(out[0], out[lanes]):
        assert torch.equal(a, b)
    for a, b in zip(out[4], out[8]):
        assert float((a - b).abs().max()) <= 1e-13 * float(a.abs().max())
