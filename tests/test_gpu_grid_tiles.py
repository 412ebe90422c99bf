"""The tiled sums that put hills onto a bias grid, at the edges of their tiles
(32 x 32 nodes, 64 nodes in one CV) and of their hill stages (16 hills, four
groups of them), against the FP64 oracle's node values of the stored list.

Tolerance: both sides sum the same float32-stored hills in FP64; a node value
is a product of at most three exponentials and a sum of K <= 200 terms, each
within a few ulp: 1e-12 of the grid's largest |V| (|dV/dxi|), the bound of
the grid's other node tests.
"""
import numpy as np
import pytest
import torch

from oracle.grid import BiasGrid
from paper_2301_04835_amd import Sampler, synth

from gpu_util import dev

pytestmark = pytest.mark.gpu

PI = np.pi
RG_LO, RG_HI = 0.2, 0.6


def make(nb, mixed, W=1, shared=False, cap=256):
    """Walkers of 22 atoms with len(nb) CVs: dihedrals, the last one a radius
    of gyration when mixed."""
    D = len(nb)
    nd = D - (1 if mixed else 0)
    s = Sampler(0)
    for d in range(nd):
        s.add_dihedral([d, d + 1, d + 2, d + 3])
    if mixed:
        s.add_gyration(list(range(12)))
    s.set_walkers(np.arange(W + 1) * 22, hill_capacity=[cap] if shared else [cap] * W, shared=shared)
    sigma = [0.35, 2.0, 0.5][:nd] + ([0.04] if mixed else [])
    s.metad(sigma, 1.2, 300.0, 6.0, 500, cap)
    lo, hi = [-PI] * nd + [RG_LO] * (D - nd), [PI] * nd + [RG_HI] * (D - nd)
    s.metad_grid(lo, hi, nb)
    s.bind()
    return s, sigma, BiasGrid(lo, hi, nb, [True] * nd + [False] * (D - nd))


def points(K, D, mixed, seed):
    g = np.random.default_rng(seed)
    x = g.uniform(-PI, PI, size=(K, D))
    if mixed:
        x[:, -1] = g.uniform(RG_LO, RG_HI, size=K)
    x[0, :D - 1 if mixed else D] = 0.0  # half a period from the node at -pi
    return x


def check(s, ref, sigma, walker=0):
    C, H = s.hills_get(walker)
    ref.set_hills(C.astype(np.float64), H.astype(np.float64), sigma)
    V, G = s.grid_get(walker)
    sV, sG = np.max(np.abs(ref.V)), np.max(np.abs(ref.G))
    eV = np.max(np.abs(V - ref.V.reshape(-1)))
    eG = np.max(np.abs(G.T - ref.G.reshape(-1, ref.D)))
    assert eV <= 1e-12 * sV and eG <= 1e-12 * sG, (eV / sV, eG / sG)
    return len(H)


@pytest.mark.parametrize("nb,mixed", [([2], False), ([63], False), ([65], False), ([63], True), ([130], True),
                                      ([2, 2], False), ([32, 32], False), ([33, 31], False), ([31, 64], True),
                                      ([5, 97], False), ([2, 3, 5], False), ([7, 6, 33], False), ([3, 11, 31], True)])
def test_list_onto_nodes(gpu, nb, mixed):
    s, sigma, ref = make(nb, mixed)
    for K in (1, 15, 16, 17, 64, 65, 200):
        x = points(K, len(nb), mixed, 100 + K)
        s.hills_set(0, x.astype(np.float32), np.linspace(0.5, 1.5, K).astype(np.float32))
        assert check(s, ref, sigma) == K
    s.hills_set(0, np.zeros((0, len(nb)), np.float32), np.zeros(0, np.float32))
    V, G = s.grid_get(0)
    assert not V.any() and not G.any()


@pytest.mark.parametrize("nb,mixed", [([65], False), ([33, 31], False), ([40, 64], True), ([7, 6, 33], False)])
@pytest.mark.parametrize("W,shared", [(1, False), (3, False), (17, True)])
def test_deposits_onto_nodes(gpu, nb, mixed, W, shared):
    """Deposits (one hill per walker) on top of a starting list, twice, and a
    launch that finds nothing to add in between."""
    s, sigma, ref = make(nb, mixed, W, shared)
    lists = [0] if shared else list(range(W))
    for w in lists:
        x = points(20, len(nb), mixed, 7 + w)
        s.hills_set(w, x.astype(np.float32), np.ones(20, np.float32))
    pos = dev(np.concatenate([synth.chain_template(22, 40 + w) for w in range(W)]))
    for rep in range(2):
        s.deposit(dev(points(W, len(nb), mixed, 50 + rep)))
        s.step(pos, forces=torch.zeros_like(pos, dtype=torch.float32), step=1)
        s.check()
        for w in lists:
            assert check(s, ref, sigma, w) == 20 + (rep + 1) * (W if shared else 1)
