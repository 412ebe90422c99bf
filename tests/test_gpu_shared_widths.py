"""The shared-list sum with narrow hills on periodic CVs, on both sides of the
width below which it keeps scaled displacements (0.005 rad), against the FP64
oracle on the stored float32 centres.

Points lie within three widths of a hill and the hills within four widths of
a common centre, so that every exponent is below 25 per CV.  Tolerance: the
exponent q is rounded once to float32 (2^-24 q of a term, whose weight in V
falls as 2^-q; below 2e-6 for the near hills that make up V) and the float32
Gaussian and product add 2e-7; the FP64 displacement's 1e-15 rad is 1e-10
widths.  V within 3e-6 relative, dV/dxi within 1e-5 of its term scale, the
bounds of the wide hills.
"""
import numpy as np
import pytest
import torch

from paper_2301_04835_amd import Sampler, synth

from gpu_util import dev
from test_gpu_shared_sizes import close, cvs_of, reference

pytestmark = pytest.mark.gpu

WIDTHS = [1e-5, 1e-4, 0.0049, 0.0051, 0.05]


def around(x0, n, sigma, k, g):
    """n points within k widths of x0 (a clipped normal), on the torus where
    the first CV's centre lies at its seam."""
    return x0 + np.clip(g.normal(scale=k / 2, size=(n, len(x0))), -k, k) * np.asarray(sigma)


@pytest.mark.parametrize("per", [[True], [True, True], [True, False], [True, True, True], [False, True, True]])
@pytest.mark.parametrize("width", WIDTHS)
def test_points(gpu, width, per):
    D = len(per)
    sigma = [width if p else 0.05 for p in per]
    g = np.random.default_rng(int(width * 1e6) + D)
    s = Sampler(0)
    s.add_cvs(cvs_of(per))
    s.metad(sigma, 1.0, 300.0, 6.0, 500, 4000)
    s.bind()
    x0 = np.array([0.3, np.pi, -1.7])[:D]  # the second at the seam
    for K, n in ((1, 3), (700, 70), (3000, 1030)):
        C = around(x0, K, sigma, 4.0, g).astype(np.float32)
        H = g.uniform(0.5, 1.5, K).astype(np.float32)
        s.hills_set(0, C, H)
        xi = C[g.integers(0, K, n)].astype(np.float64) + np.clip(g.normal(size=(n, D)), -3, 3) * sigma
        V, dV = s.bias_eval(dev(xi))
        close(V.cpu().numpy(), dV.cpu().numpy(), reference(xi, C, H, sigma, per))


@pytest.mark.parametrize("width", WIDTHS)
def test_step_of_dihedrals(gpu, width):
    """A step of walkers that share narrow hills around their own CVs, and its
    deposit."""
    W, n, K = 40, 10, 400
    per, sigma = [True, True], [width, width]
    g = np.random.default_rng(3)
    pos = np.tile(synth.chain_template(n, 9), (W, 1))
    s = Sampler(0)
    s.add_cvs(cvs_of(per))
    s.set_walkers(np.arange(W + 1) * n, [1000], shared=True)
    s.metad(sigma, 1.2, 300.0, 6.0, 1, 1000)
    s.bind()
    P, F = dev(pos), torch.zeros((W * n, 3), dtype=torch.float32, device=gpu)
    xi = torch.zeros((W, 2), dtype=torch.float64, device=gpu)
    V = torch.zeros(W, dtype=torch.float64, device=gpu)
    dV = torch.zeros((W, 2), dtype=torch.float64, device=gpu)
    x0 = s.eval_cv(P)[0].cpu().numpy()[0]
    C = around(x0, K, sigma, 4.0, g).astype(np.float32)
    H = g.uniform(0.5, 1.5, K).astype(np.float32)
    s.hills_set(0, C, H)
    s.step(P, forces=F, xi_out=xi, V_out=V, dV_out=dV)
    s.check()
    x = xi.cpu().numpy()
    assert np.max(np.abs(x - x0)) <= 1e-12
    close(V.cpu().numpy(), dV.cpu().numpy(), reference(x, C, H, sigma, per))
    assert torch.any(F != 0)
    C, H = s.hills_get(0)
    assert len(H) == K + W
