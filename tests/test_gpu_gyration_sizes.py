"""Radii of gyration of many walkers at the sizes where a thread of the kernel
holds one member or four (256), against the FP64 oracle: values 1e-9, forces
of a harmonic bias 1e-6 of the walker's largest (float32)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2301_04835_amd import Sampler
from gpu_util import dev, rel_inf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n", [2, 6, 255, 256, 257])
def test_walkers_radii(gpu, n, dtype):
    W = 70
    pos = np.random.default_rng(n).uniform(0.0, 2.0, size=(W * n, 3)).astype(dtype)
    s = Sampler(0)
    s.add_gyration(list(range(n)))
    s.set_walkers(np.arange(W + 1) * n)
    s.harmonic([50.0], np.full((W, 1), 0.5))
    s.bind()
    F = torch.zeros((W * n, 3), dtype=torch.float32, device=gpu)
    xi = torch.zeros((W, 1), dtype=torch.float64, device=gpu)
    s.step(dev(pos), forces=F, xi_out=xi)
    s.check()
    for w in (0, 1, 63, 64, W - 1):
        xr, J = oracle.cv_eval(pos[w * n:(w + 1) * n].astype(np.float64), [{"kind": "gyration", "idx": list(range(n))}])
        assert abs(xi[w, 0].item() - xr[0]) <= 1e-9 * xr[0]
        assert rel_inf(F[w * n:(w + 1) * n].cpu().numpy(), -50.0 * (xr[0] - 0.5) * J[0]) <= 1e-6
