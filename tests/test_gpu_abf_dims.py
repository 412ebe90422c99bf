"""ABF with one and three CVs, in one launch (few touched atoms) and in two
(more than 512), against the FP64 oracle at the 1e-5 of the ABF tests: per
step the bias along xi and the forces, at the end the histogram (exact) and
the force sums."""
import numpy as np
import pytest
import torch

import oracle
from paper_2301_04835_amd import Sampler, synth

from gpu_util import dev, rel_inf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("many", [False, True])
@pytest.mark.parametrize("D", [1, 3])
def test_abf_dims(gpu, D, many):
    W, n, T = 2, 700, 12
    m = 600 if many else 60
    box = np.full(3, 40.0)
    cvs = [{"kind": "gyration", "idx": list(range(m))},
           synth.backbone_cvs(4)[0],
           {"kind": "coordination", "a": list(range(m, m + 30)), "b": list(range(m + 30, m + 100)), "r0": 0.5, "n": 6,
            "m": 12, "rcut": 0.0, "normalize": False}][:D]
    g = np.random.default_rng(70 + D)
    tmpl = [synth.chain_template(n, 40 + w) for w in range(W)]
    at = np.array([oracle.cv_eval(tm.astype(np.float64), cvs, box)[0] for tm in tmpl])
    lo = [at[:, 0].min() - 0.6, -np.pi, 0.0][:D]
    hi = [at[:, 0].max() + 0.6, np.pi, 3.0 * at[:, -1].max() + 1.0][:D]
    nb, thr = [12, 3, 2][:D], 2
    s = Sampler(0)
    s.add_cvs(cvs)
    s.set_box(box)
    s.set_walkers(np.arange(W + 1) * n)
    s.abf(lo, hi, nb, thr)
    s.bind()
    assert (len(np.unique(s.jac_layout()[0])) > 512) == many
    grids = [oracle.AbfGrid(lo, hi, nb, [False, True, False][:D], thr) for _ in range(W)]
    Fb = torch.zeros((W * n, 3), dtype=torch.float32, device=gpu)
    dV = torch.zeros((W, D), dtype=torch.float64, device=gpu)
    for t in range(T):
        pos = np.concatenate([tm + 0.2 * g.normal(size=tm.shape) for tm in tmpl]).astype(np.float32)
        q = g.normal(0.0, 50.0, size=pos.shape).astype(np.float32)
        Fb.zero_()
        s.step(dev(pos), forces=Fb, step=t, dV_out=dV, sys_forces=dev(q))
        bg, Fg = -dV.cpu().numpy(), Fb.cpu().numpy()
        for w in range(W):
            sl = slice(w * n, (w + 1) * n)
            xi, J = oracle.cv_eval(pos[sl].astype(np.float64), cvs, box)
            b, F, _, _ = oracle.abf_step(grids[w], xi, J, q[sl].astype(np.float64))
            if np.any(b != 0):
                assert rel_inf(bg[w], b) <= 1e-5 and rel_inf(Fg[sl], F) <= 1e-5
            else:
                assert np.all(bg[w] == 0) and np.all(Fg[sl] == 0)
    s.check()
    for w in range(W):
        N, Fsum = s.abf_grid(w)
        assert np.array_equal(N.astype(np.int64), grids[w].N)
        nz = grids[w].N > 0
        assert rel_inf(Fsum[nz], grids[w].Fsum[nz]) <= 1e-5
