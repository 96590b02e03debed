"""The 2D deposit's rounds at every lane-group width G: cells with 0, 1, G - 1,
G, G + 1, 2 G, 2 G + 1 and 5 G - 1 particles side by side, so that groups end in
different rounds and rounds start off their 64-byte boundaries, against the
oracle (the bounds of the other deposit tests: FP64 1e-12, FP32 particles
1e-5), without and with a per-particle gbar (here gamma itself, so that the
result is the same)."""
import numpy as np
import pytest

import oracle
from tests.gpu_helpers import host_state, load, make_ctx, need_gpu
from tests.helpers import full_from_half

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("given", [False, True])
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("mixed", 1e-5)])
@pytest.mark.parametrize("group", [4, 8, 16, 32, 64])
def test_ragged_cells_at_every_group_width(group, precision, tol, given):
    need_gpu()
    import torch

    from paper_2509_11100_amd import relsim

    g = oracle.Grid(dim=2, nx=9, ny=7, dx=1.0, dy=0.9, dt=0.4, q=(1.0, -1.0, 2.0), m=(1.0, 1.0, 3.0))
    rng = np.random.default_rng(41 + group)
    counts = np.array([0, 1, group - 1, group, group + 1, 2 * group, 2 * group + 1, 5 * group - 1])
    cell = np.repeat(np.arange(g.N, dtype=np.int32), counts[rng.integers(0, 8, g.N)])
    n = len(cell)
    sp = rng.integers(0, 3, n).astype(np.uint8)
    B = (2 * rng.random((3, g.N)) - 1) * 2.0
    ctx = make_ctx(g, precision, n, group=group)
    parts = load(ctx, cell, sp, rng.random((2, n)), (2 * rng.random((3, n)) - 1) * 2.0, 0.5 + rng.random(n))
    st = host_state(g, parts)
    gbar = None
    if given:
        gbar = torch.as_tensor(np.sqrt(1 + (st["u"] ** 2).sum(0) / g.c**2)).cuda()
        gbar = gbar.float() if precision == "mixed" else gbar
    J, M = relsim.deposit_moments(ctx, parts, torch.as_tensor(B).cuda(), gbar=gbar)
    Jr, Mr = oracle.deposit(g, st["x"], st["u"], st["w"], st["species"], B)
    assert np.linalg.norm(J.cpu().numpy() - Jr) <= tol * np.linalg.norm(Jr)
    full = full_from_half(g, M.cpu().numpy())
    assert np.linalg.norm(full - Mr) <= tol * np.linalg.norm(Mr)
