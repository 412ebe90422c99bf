"""Surrogate steps whose fallback rows sum many walkers one after the other
through the same LDS: 1,024 walkers outside certified cells are 32 to a row.

A walker's records do not depend on the row that formed them, so V, dV/dxi and
forces equal, bit for bit, those of the same walkers in contexts of 32, where
every row sums one.
"""
import numpy as np
import pytest
import torch

from paper_2301_04835_amd import Sampler, synth

from gpu_util import dev

pytestmark = pytest.mark.gpu

ATOMS, K, CAP = 22, 5000, 9000


def step(pos, dims):
    """One surrogate step with every walker on the exact fallback."""
    W = len(pos) // ATOMS
    g = np.random.default_rng(7)
    s = Sampler(0)
    for d in range(dims):
        s.add_dihedral([d, d + 1, d + 2, d + 3])
    s.set_walkers(np.arange(W + 1) * ATOMS, [CAP], shared=True)
    s.metad([0.3] * dims, 1.0, 300.0, 6.0, 0, CAP)
    s.surrogate(64, max_samples=1024, max_batch=1024, cert_n=8, tol_force=1e-9)
    s.bind()
    s.hills_set(0, synth.uniform_centers(K, dims, 41), synth.uniform_heights(K, 42))
    s.surrogate_params(g.normal(size=s.surrogate_param_count()).astype(np.float32))
    s.surrogate_certify()
    s.surrogate_enable(True)
    P = dev(pos)
    out = []
    for _ in range(3):
        F = torch.zeros_like(P)
        V = torch.empty(W, dtype=torch.float64, device=P.device)
        dV = torch.empty((W, dims), dtype=torch.float64, device=P.device)
        s.step(P, forces=F, step=3, V_out=V, dV_out=dV)
        s.check()
        assert s.surrogate_fallback_count() == W
        out.append([t.cpu().numpy() for t in (V, dV, F.reshape(W, ATOMS, 3))])
    return out


@pytest.mark.parametrize("dims", [1, 2, 3])
def test_rows_of_many_walkers(gpu, dims):
    W = 1024
    pos = np.concatenate([synth.chain_template(ATOMS, 100 + w) for w in range(W)]).astype(np.float32)
    together = step(pos, dims)
    for w in range(0, W, 256):
        alone = step(pos[w * ATOMS:(w + 32) * ATOMS], dims)[0]
        for rep in together:
            for a, b in zip(rep, alone):
                assert np.array_equal(a[w:w + 32], b)
