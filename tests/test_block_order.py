"""The order in which the XCDs take work items (csrc/block_order.h), compiled
for the host: every order is a permutation, and the blocks of 64 consecutive
cells in the 2D deposit stay on one XCD (two where a run ends inside them),
on small grids and in what is left after the last whole round of chunks too."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_11100_amd", "csrc")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("order")
    src = d / "order.cpp"
    src.write_text('#define __host__\n#define __device__\n#include "block_order.h"\nextern "C" {\n'
                   "int bands(int b, int nb) { return relsim::xcd_bands(b, nb); }\n"
                   "int chunks(int b, int nb, int chunk) { return relsim::xcd_chunks(b, nb, chunk); }\n"
                   "int deposit(int b, int nb, int G, int ncells) { return relsim::deposit_block(b, nb, G, ncells); }\n"
                   "int even(int n, int cap, int most) { return relsim::even_tile(n, cap, most); }\n"
                   "int side(int dim, int nseg, int C) { return relsim::tile_segments(dim, nseg, C); }\n}\n")
    so = d / "order.so"
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(so)], check=True)
    return C.CDLL(str(so))


@pytest.mark.parametrize("nb", [1, 7, 8, 9, 63, 64, 65, 511, 512, 4100, 10007])
def test_orders_are_permutations(lib, nb):
    assert sorted(lib.bands(b, nb) for b in range(nb)) == list(range(nb))
    for chunk in (1, 3, 8, 64, 100, 512):
        assert sorted(lib.chunks(b, nb, chunk) for b in range(nb)) == list(range(nb))


@pytest.mark.parametrize("G", [4, 8, 16, 64])
@pytest.mark.parametrize("ncells", [32 * 32, 64 * 32, 61 * 63, 100 * 77, 200 * 102, 214 * 371, 300 * 211, 512 * 256])
def test_deposit_blocks_of_64_cells_share_an_xcd(lib, ncells, G):
    per = 64 // G  # cells of a block
    nb = (ncells + per - 1) // per
    xcd = np.full(nb, -1)
    for b in range(nb):
        xcd[lib.deposit(b, nb, G, ncells)] = b % 8
    assert xcd.min() == 0  # every block taken
    runs = np.array([len(set(xcd[i:i + G])) for i in range(0, nb - nb % 8 - G, G)])
    assert runs.max() <= 2 and np.count_nonzero(runs == 2) <= 8


@pytest.mark.parametrize("cap", [1, 2, 4, 8, 16, 32])
def test_even_tiles_stay_below_their_bound(lib, cap):
    most = cap + cap // 4
    for n in range(1, 200):
        t = lib.even(n, cap, most)
        assert 1 <= t <= min(n, most)
        assert -(-n // t) * t < n + t  # the last tile holds some of the places
    assert lib.even(4 * cap, cap, most) == cap


def test_3d_tiles_are_one_segment_wide(lib):
    for nseg in range(1, 40):
        for C in (1, 2, 4, 8, 16, 32, 64):
            assert lib.side(3, nseg, C) == 1
            assert 1 <= lib.side(2, nseg, C) <= max(1, 32 // C)
