"""The two ways in which the cell build places members, in turns (groups
crowded into a few cells, or whose slots do not fit LDS) and by counting:
values and the vector-Jacobian product against the FP64 oracle (1e-6 relative,
1e-5 inf-norm, the bars of the cell path), bitwise the same again, at group
sizes around the build's chunks (1,024 members) and the largest whose slots fit
(8,128 members beside 16,384 cells)."""
import numpy as np
import pytest
import torch

from oracle import methods
from gpu_util import dev, rel_inf
from test_gpu_cell_cull import cell_ctx, pair_cvs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("na,L", [(600, 19.3), (1023, 19.3), (1024, 19.3), (1025, 19.3), (8192, 19.3), (8193, 19.3),
                                  (9000, 3.7), (41000, 3.7)])
def test_crowded_groups(gpu, na, L, dtype):
    """Three quarters of group a in a few cells around the box corner (they
    wrap), the rest anywhere; group b nearby."""
    g = np.random.default_rng(na)
    nb, L3 = 30, np.full(3, L)
    n = na + nb
    pos = g.uniform(0.0, 1.0, size=(n, 3)) * L3
    some = np.flatnonzero(g.random(n) < 0.75)
    pos[some] = g.normal(scale=0.1, size=(len(some), 3))
    pos[na:na + 20] = g.normal(scale=0.4, size=(20, 3))
    check(pos.astype(dtype), na, nb, L3, gpu)


@pytest.mark.parametrize("na,L", [(1024, 19.3), (4097, 9.0), (8128, 19.3), (8129, 19.3), (20000, 10.0)])
def test_even_groups(gpu, na, L):
    """The group all over the box: counted where the slots fit."""
    g = np.random.default_rng(na)
    pos = g.uniform(0.0, L, size=(na + 30, 3)).astype(np.float32)
    check(pos, na, 30, np.full(3, L), gpu)


def check(pos, na, nb, L3, gpu):
    n = na + nb
    cvs = pair_cvs(na, nb, (6, 12))[:1]
    s = cell_ctx(cvs, L3, n)
    assert s.cell_list_cvs() == 1
    P = dev(pos)
    xi = s.eval_cv(P)[0].cpu().numpy()[0]
    pb = torch.zeros((n, 3), dtype=torch.float32, device=gpu)
    s.cv_vjp(P, dev(np.ones((1, 1))), pb)
    xr, J = methods.cv_eval(pos.astype(np.float64), cvs, L3)
    assert abs(xi[0] - xr[0]) <= 1e-6 * abs(xr[0])
    assert rel_inf(pb.cpu().numpy(), J[0]) <= 1e-5
    pb2 = torch.zeros_like(pb)
    s.cv_vjp(P, dev(np.ones((1, 1))), pb2)
    assert np.array_equal(s.eval_cv(P)[0].cpu().numpy()[0], xi) and torch.equal(pb, pb2)
