"""The 2D FP64 deposit of more than 1024 waves, whose next record waits in LDS
(smaller launches keep it in registers): cells with 0, 1, G - 1, G, G + 1, 2 G,
2 G + 1 and 5 G - 1 particles side by side at every lane-group width G, against
the oracle (1e-12, as the other deposit tests), without and with a per-particle
gbar (here gamma itself), and on both sides of the 1024 waves the same sums bit
for bit."""
import numpy as np
import pytest

import oracle
from tests.gpu_helpers import host_state, load, make_ctx, need_gpu
from tests.helpers import full_from_half

pytestmark = pytest.mark.gpu


def ragged(g, group, rng):
    counts = np.array([0, 1, group - 1, group, group + 1, 2 * group, 2 * group + 1, 5 * group - 1])
    cell = np.repeat(np.arange(g.N, dtype=np.int32), counts[rng.integers(0, 8, g.N)])
    n = len(cell)
    return cell, rng.integers(0, 3, n).astype(np.uint8), rng.random((2, n)), (2 * rng.random((3, n)) - 1) * 2.0, \
        0.5 + rng.random(n)


@pytest.mark.parametrize("given", [False, True])
@pytest.mark.parametrize("group", [4, 8, 16, 32, 64])
def test_ragged_cells_of_many_waves(group, given):
    need_gpu()
    import torch

    from paper_2509_11100_amd import relsim

    ny = 1100 * (64 // group) // 37 + 1
    g = oracle.Grid(dim=2, nx=37, ny=ny, dx=1.0, dy=0.9, dt=0.4, q=(1.0, -1.0, 2.0), m=(1.0, 1.0, 3.0))
    rng = np.random.default_rng(43 + group)
    state = ragged(g, group, rng)
    n = len(state[0])
    B = (2 * rng.random((3, g.N)) - 1) * 2.0
    ctx = make_ctx(g, "fp64", n, group=group)
    parts = load(ctx, *state)
    st = host_state(g, parts)
    gbar = torch.as_tensor(np.sqrt(1 + (st["u"] ** 2).sum(0) / g.c**2)).cuda() if given else None
    J, M = relsim.deposit_moments(ctx, parts, torch.as_tensor(B).cuda(), gbar=gbar)
    Jr, Mr = oracle.deposit(g, st["x"], st["u"], st["w"], st["species"], B)
    assert np.linalg.norm(J.cpu().numpy() - Jr) <= 1e-12 * np.linalg.norm(Jr)
    assert np.linalg.norm(full_from_half(g, M.cpu().numpy()) - Mr) <= 1e-12 * np.linalg.norm(Mr)


@pytest.mark.parametrize("group", [4, 16, 64])
def test_both_sides_of_the_limit_add_alike(group):
    """Rows of cells in the middle of a grid of 1024 waves and of one with a few
    rows more see the same particles and fields."""
    need_gpu()
    import torch

    from paper_2509_11100_amd import relsim

    rows = 1024 * (64 // group) // 32
    rng = np.random.default_rng(47 + group)
    out = []
    for ny in (rows, rows + 3):
        g = oracle.Grid(dim=2, nx=32, ny=ny, dx=1.0, dy=0.9, dt=0.4, q=(1.0, -1.0, 2.0), m=(1.0, 1.0, 3.0))
        if not out:
            small, B = ragged(g, group, rng), (2 * rng.random((3, g.N + 96)) - 1) * 2.0
        ctx = make_ctx(g, "fp64", len(small[0]), group=group)
        J, M = relsim.deposit_moments(ctx, load(ctx, *small), torch.as_tensor(B[:, : g.N].copy()).cuda())
        # nodes whose cells and fields do not wrap around
        out.append((J[:, 64 : 32 * (rows - 2)], M[..., 64 : 32 * (rows - 2)]))
    for a, b in zip(*out):
        assert torch.equal(a, b)
