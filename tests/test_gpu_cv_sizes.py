"""Group sizes around what a thread of the CV kernels keeps and stages: 256
members a round, four rounds in registers (gyration), 1,024 partners in LDS
(all-pairs coordination numbers), against the FP64 oracle.  Tolerances of the
CV tests: gyration 1e-9 (Jacobian stored in float32: 1e-6), coordination
number 1e-6 (Jacobian 1e-5)."""
import numpy as np
import pytest

import oracle
from paper_2301_04835_amd import Sampler
from gpu_util import dense_jac, dev, rel_inf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n", [1, 255, 257, 1024, 1025, 2300])
def test_cv_group_sizes(gpu, n, dtype):
    g = np.random.default_rng(n)
    N = n + 40
    pos = g.uniform(0.0, 3.0, size=(N, 3)).astype(dtype)
    atoms = g.permutation(N).tolist()
    cvs = [{"kind": "coordination", "a": atoms[n:n + 33], "b": atoms[:n], "r0": 0.5, "n": 6, "m": 12, "rcut": 0.0,
            "normalize": False}]
    if n > 1:  # the radius of one atom is zero and has no gradient
        cvs.append({"kind": "gyration", "idx": atoms[:n]})
    box = [3.1, 3.0, 3.3]
    s = Sampler(0)
    s.add_cvs(cvs)
    s.set_box(box)
    s.set_walkers(np.array([0, N], dtype=np.int64))
    s.bind()
    xi, J = s.eval_cv(dev(pos))
    xr, Jr = oracle.cv_eval(pos.astype(np.float64), cvs, np.array(box))
    xi = xi.cpu().numpy()[0]
    atom, cvi = s.jac_layout()
    Jd = dense_jac(J[0].cpu().numpy(), atom, cvi, N, len(cvs))
    assert abs(xi[0] - xr[0]) <= 1e-6 * abs(xr[0])
    assert rel_inf(Jd[0], Jr[0]) <= 1e-5
    if n > 1:
        assert abs(xi[1] - xr[1]) <= 1e-9 * abs(xr[1])
        assert rel_inf(Jd[1], Jr[1]) <= 1e-6
