"""Private lists of more tiles than one wavefront finalizes (256): the
workgroup's finalize with its four records in flight a lane, the force table's
branch in it, and its deposit, against the FP64 oracle.

Tolerances: hill_v_rel_bound and hill_grad_bound, the derived bounds of a
float32 hill sum, the gradient's Hessian term from the oracle's CV tolerance
(1e-9 rad: both sides evaluate the dihedral in FP64).
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2301_04835_amd import Sampler, synth

from gpu_util import TWO_PI, dev, hill_grad_bound, hill_v_rel_bound, rel_inf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("K", [130 * 1024, 256 * 1024 - 600, 256 * 1024 + 5, 767 * 1024, 769 * 1024 + 3, 1100000])
def test_step_of_long_lists(gpu, K, dtype):
    """Two walkers, one with a long list in tiles of 1,024 hills, one with a
    short one; a depositing step, then one on the grown lists."""
    ks, sigma, cvs = [K, 700], [0.5, 0.6], synth.backbone_cvs(4)
    g = np.random.default_rng(K)
    n = 22
    pos = np.concatenate([synth.chain_template(n, 5), synth.chain_template(n, 6)]).astype(dtype)
    s = Sampler(0)
    s.add_cvs(cvs)
    s.set_walkers([0, n, 2 * n], [k + 300 for k in ks])
    s.metad(sigma, 1.2, 300.0, 6.0, 1)
    s.bind()
    s.set_tuning(1024, 0)
    lists = []
    for w, k in enumerate(ks):
        C = g.uniform(-np.pi, np.pi, (k, 2)).astype(np.float32)
        H = g.uniform(0.5, 1.5, k).astype(np.float32)
        s.hills_set(w, C, H)
        lists.append((C, H))
    P = dev(pos)
    for rep in range(2):
        F = torch.zeros((2 * n, 3), dtype=torch.float32, device=gpu)
        xi = torch.zeros((2, 2), dtype=torch.float64, device=gpu)
        V = torch.zeros(2, dtype=torch.float64, device=gpu)
        dV = torch.zeros((2, 2), dtype=torch.float64, device=gpu)
        s.step(P, forces=F, xi_out=xi, V_out=V, dV_out=dV)
        s.check()
        x, Vh, dVh, Fh = (t.cpu().numpy() for t in (xi, V, dV, F))
        for w in range(2):
            C, H = (a.astype(np.float64) for a in lists[w])
            xr, J = oracle.cv_eval(pos[w * n:(w + 1) * n].astype(np.float64), cvs)
            assert np.max(np.abs(x[w] - xr)) <= 1e-9
            Vr, dVr = oracle.hillsum_batch(x[w:w + 1], None, C, H, sigma, [TWO_PI] * 2, nthreads=8)
            assert abs(Vh[w] - Vr[0]) <= hill_v_rel_bound(x[w], C, H, sigma, [TWO_PI] * 2) * Vr[0]
            assert np.all(np.abs(dVh[w] - dVr[0]) <=
                          hill_grad_bound(x[w], C, H, sigma, [TWO_PI] * 2, np.zeros((2, 2)), np.zeros(2)))
            assert rel_inf(Fh[w * n:(w + 1) * n], -np.tensordot(dVh[w], J, axes=(0, 0))) <= 1e-5
            lists[w] = s.hills_get(w)
            assert len(lists[w][1]) == ks[w] + rep + 1
            assert np.max(np.abs(lists[w][0][-1] - x[w])) <= 1e-6
