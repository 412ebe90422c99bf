"""Few hills onto a bias grid (a private list's one hill of a step, one or two
walkers of a shared list, short lists), at the edges of the kernel's tiles
(up to 256 columns, four rows a thread) and of the rules that choose it, and
grids with more tiles than a step launches workgroups for, against the FP64
oracle's node values of the stored list at the bound of the other node tests
(1e-12 of the grid's largest |V|, |dV/dxi|).
"""
import numpy as np
import pytest
import torch

from paper_2301_04835_amd import synth

from gpu_util import dev
from test_gpu_grid_tiles import check, make, points

pytestmark = pytest.mark.gpu

SHAPES = [([2], False), ([255], False), ([256], True), ([513], False), ([2, 2], False), ([3, 300], False),
          ([70, 5], False), ([33, 65], False), ([300, 2], True), ([2, 257], True), ([2, 3, 5], False),
          ([5, 4, 70], False), ([9, 8, 3], True)]


def deposits(s, sigma, ref, nb, mixed, W, shared, lists, start=5):
    """Two deposits on top of `start` hills a list, a step without one between."""
    for w in lists:
        s.hills_set(w, points(start, len(nb), mixed, 7 + w).astype(np.float32), np.ones(start, np.float32))
    pos = dev(np.concatenate([synth.chain_template(22, 40 + w % 50) for w in range(W)]))
    for rep in range(2):
        s.deposit(dev(points(W, len(nb), mixed, 50 + rep)))
        s.step(pos, forces=torch.zeros_like(pos, dtype=torch.float32), step=1)
        s.check()
        for w in lists:
            assert check(s, ref, sigma, w) == start + (rep + 1) * (W if shared else 1)


@pytest.mark.parametrize("nb,mixed", SHAPES)
@pytest.mark.parametrize("W,shared", [(1, False), (40, False), (2, True), (3, True)])
def test_deposits(gpu, nb, mixed, W, shared):
    s, sigma, ref = make(nb, mixed, W, shared)
    deposits(s, sigma, ref, nb, mixed, W, shared, [0] if shared or W == 1 else [0, 17, W - 1])


@pytest.mark.parametrize("nb,mixed", SHAPES)
def test_short_lists(gpu, nb, mixed):
    s, sigma, ref = make(nb, mixed)
    for K in (1, 2, 8, 9, 16, 32, 33, 64, 65):
        s.hills_set(0, points(K, len(nb), mixed, 100 + K).astype(np.float32),
                    np.linspace(0.5, 1.5, K).astype(np.float32))
        assert check(s, ref, sigma) == K
    s.hills_set(0, np.zeros((0, len(nb)), np.float32), np.zeros(0, np.float32))
    V, G = s.grid_get(0)
    assert not V.any() and not G.any()


@pytest.mark.parametrize("nb,W,shared", [([130, 130], 300, False), ([40, 7, 9], 300, False), ([1100, 1100], 3, True),
                                         ([1100, 1100], 2, True), ([40000], 70, True), ([300000], 3, True)])
def test_more_tiles_than_workgroups(gpu, nb, W, shared):
    """Each workgroup takes several tiles, and the count moves once they are
    all done."""
    s, sigma, ref = make(nb, False, W, shared)
    deposits(s, sigma, ref, nb, False, W, shared, [0] if shared else [0, 150, W - 1])


def test_long_grid_of_a_short_list(gpu):
    """One CV, more than 512 x 64 nodes: lists up to 64 hills."""
    s, sigma, ref = make([40000], False)
    for K in (64, 65):
        s.hills_set(0, points(K, 1, False, K).astype(np.float32), np.ones(K, np.float32))
        assert check(s, ref, sigma) == K
