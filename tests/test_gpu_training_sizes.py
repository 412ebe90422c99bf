"""Loss, gradient and Adam updates of the network at the edges of the training
kernel's workgroups (16 samples, 8 at 128 units) and of the update kernel's
gradient slices, for every width and CV count, against the FP64 oracle.

Tolerances: those of the full-batch gradient test (loss 1e-5, each parameter
block 1e-4 of its largest entry: FP32 arithmetic and the bf16 pair rounding
the oracle repeats); they do not grow with fewer samples, every sample's
terms carrying the same relative error.  After two Adam steps a weight differs
from the oracle's by at most that relative gradient error times the step, and
the sign of an entry at the noise level may flip: 99% of the weights within
1e-3 of the learning rate, all within two steps of it.
"""
import numpy as np
import pytest

from oracle import mlp
from paper_2301_04835_amd import synth

from gpu_util import dev
from test_gpu_surrogate import bf16_dict, make_ctx, rand_params, to_dict, to_flat

pytestmark = pytest.mark.gpu

RG = {"kind": "gyration", "idx": [0, 1, 2, 3, 4, 5]}
SETS = {1: ([RG], [False]), 2: (synth.backbone_cvs(0)[:1] + [RG], [True, False]),
        3: (synth.backbone_cvs(0) + [RG], [True, True, False])}


def samples(D, periodic, n, seed):
    g = np.random.default_rng(seed)
    xi = np.stack([g.uniform(-np.pi, np.pi, n) if p else 0.9 + 0.3 * g.normal(size=n) for p in periodic], 1)
    return xi, 2.0 + 3.0 * g.normal(size=n), 2.0 * g.normal(size=(n, D))


@pytest.mark.parametrize("H", [64, 128])
@pytest.mark.parametrize("D", [1, 2, 3])
def test_loss_gradient_sizes(gpu, H, D):
    cvs, periodic = SETS[D]
    s = make_ctx(cvs, H, D, max_batch=512)
    mu, sd = np.full(D, 0.9), np.full(D, 0.25)
    s.surrogate_norm(mu, sd)
    P = rand_params(H, D, 130 + D)
    s.surrogate_params(P)
    s.surrogate_output(1.5, 0.5)
    for n in (1, 7, 8, 9, 15, 16, 17, 255, 257, 512):
        xi, V, G = samples(D, periodic, n, 140 + n)
        loss, grad = s.surrogate_loss_grad(dev(xi), dev(V), dev(G), 0.7, 1.3)
        L, gr, _, _ = mlp.loss_and_grads(bf16_dict(P, H, D), xi, (V - 0.5) / 1.5, G / 1.5, 0.7, 1.3, periodic, mu, sd,
                                         act_round=mlp.round_bf16x2)
        gk = to_dict(grad, H, D)
        worst = max(np.max(np.abs(gk[k] - gr[k])) / np.max(np.abs(gr[k])) for k in gr)
        assert abs(loss - L) <= 1e-5 * L and worst <= 1e-4, (n, loss, L, worst)


@pytest.mark.parametrize("H,D", [(64, 2), (128, 3)])
def test_adam_over_a_ragged_batch(gpu, H, D):
    """Two steps over 300 samples in batches of 200: the second takes the
    remaining 100, fewer records than gradient slices at 64 units."""
    cvs, periodic = SETS[D]
    s = make_ctx(cvs, H, D, max_batch=512)
    mu, sd = np.full(D, 0.9), np.full(D, 0.25)
    s.surrogate_norm(mu, sd)
    P = rand_params(H, D, 150)
    s.surrogate_params(P)
    xi, V, G = samples(D, periodic, 300, 151)
    lr = 1e-3
    s.surrogate_fit(dev(xi), dev(V), dev(G), batch=200, steps=2, lr=lr, lr_final=lr, alpha=1.0, beta=0.5)
    got = s.surrogate_params()
    Q = to_dict(P, H, D)
    m = {k: np.zeros_like(v) for k, v in Q.items()}
    v = {k: np.zeros_like(x) for k, x in Q.items()}
    for t, sl in ((1, slice(0, 200)), (2, slice(200, 300))):
        Q = {k: x.astype(np.float32).astype(np.float64) for k, x in Q.items()}
        _, g, _, _ = mlp.loss_and_grads({k: mlp.round_bf16(x) for k, x in Q.items()}, xi[sl], V[sl], G[sl], 1.0, 0.5,
                                        periodic, mu, sd, act_round=mlp.round_bf16x2)
        Q, m, v = mlp.adam_step(Q, g, m, v, t, lr)
    d = np.abs(got - to_flat(Q))
    assert np.quantile(d, 0.99) <= 1e-3 * lr + 2e-7 and np.max(d) <= 2 * lr + 2e-7, (np.quantile(d, 0.99), np.max(d))
