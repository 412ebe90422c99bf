"""The shared-list sum with two and four queries per lane, which lists with
room for 65,536 hills take from 1,024 and for 65,536 from 8,192 queries on,
and the finalize kernels that move a list's count when several workgroups
share the deposit, against the FP64 oracle on sampled queries.

Tolerances: as derived for the sizes of the other sums (V 3e-6 relative,
dV/dxi 1e-5 of its term scale).
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2301_04835_amd import Sampler, synth

from gpu_util import dev
from test_gpu_shared_sizes import SETS, close, cvs_of, draw, reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", list(SETS) + ["mixed_last", "one_angle"])
def test_points_with_more_queries_per_lane(gpu, name):
    D, per = {**SETS, "mixed_last": (2, [False, True]), "one_angle": (3, [False, True, False])}[name]
    sigma = [0.9, 0.7, 1.1][:D]
    g = np.random.default_rng(D)
    s = Sampler(0)
    s.add_cvs(cvs_of(per))
    s.metad(sigma, 1.0, 300.0, 6.0, 500, 70000)
    s.bind()
    many = draw(8300, per, g)
    pick = np.r_[0:5, 120:132, 1020:1030, 8188:8194, 8290:8300]
    for K in (1, 257, 3000):
        C, H = draw(K, per, g).astype(np.float32), g.uniform(0.5, 1.5, K).astype(np.float32)
        s.hills_set(0, C, H)
        ref = reference(many[pick], C, H, sigma, per)
        for n in (1023, 1024, 1025, 8191, 8192, 8193, 8300):
            at = pick[pick < n]
            V, dV = s.bias_eval(dev(many[:n]))
            close(V.cpu().numpy()[at], dV.cpu().numpy()[at], tuple(r[:len(at)] for r in ref))


@pytest.mark.parametrize("name", ["dihedral", "two", "three", "mixed"])
@pytest.mark.parametrize("W,cap", [(300, 2000), (1030, 70000), (8200, 70000)])
def test_steps_of_many_walkers(gpu, name, W, cap):
    """A step with its deposit, sampled walkers against the oracle; the list
    then holds every walker's hill, and a second step sums them."""
    D, per = SETS[name]
    sigma = [0.9, 0.7, 1.1][:D]
    g = np.random.default_rng(W)
    cvs, n, K = cvs_of(per), 7, 900
    pos = np.concatenate([synth.chain_template(n, 60 + w % 500) for w in range(W)]).astype(np.float32)
    s = Sampler(0)
    s.add_cvs(cvs)
    s.set_walkers(np.arange(W + 1) * n, [cap], shared=True)
    s.metad(sigma, 1.2, 300.0, 6.0, 1, cap)
    s.bind()
    C, H = draw(K, per, g).astype(np.float32), g.uniform(0.5, 1.5, K).astype(np.float32)
    s.hills_set(0, C, H)
    P = dev(pos)
    F = torch.zeros((W * n, 3), dtype=torch.float32, device=gpu)
    pick = np.unique(np.r_[0:4, 62:66, 126:130, 254:258, W // 2, W - 4:W])
    pick = pick[pick < W]
    for rep in range(2 if W < 8000 else 1):
        xi = torch.zeros((W, D), dtype=torch.float64, device=gpu)
        V = torch.zeros(W, dtype=torch.float64, device=gpu)
        dV = torch.zeros((W, D), dtype=torch.float64, device=gpu)
        F.zero_()
        s.step(P, forces=F, xi_out=xi, V_out=V, dV_out=dV)
        s.check()
        x, Vh, dVh = xi.cpu().numpy(), V.cpu().numpy(), dV.cpu().numpy()
        close(Vh[pick], dVh[pick], reference(x[pick], C, H, sigma, per))
        Fh = F.cpu().numpy().astype(np.float64)
        for w in pick:
            xr, J = oracle.cv_eval(pos[w * n:(w + 1) * n].astype(np.float64), cvs)
            assert np.max(np.abs(x[w] - xr)) <= 1e-9
            Fr = -np.tensordot(dVh[w], J, axes=(0, 0))
            assert np.max(np.abs(Fh[w * n:(w + 1) * n] - Fr)) <= 1e-5 * np.max(np.abs(Fr))
        C, H = s.hills_get(0)
        assert len(H) == K + (rep + 1) * W
        assert np.max(np.abs(C[-W:] - x)) <= 1e-6
