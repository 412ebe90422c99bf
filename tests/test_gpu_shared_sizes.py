"""The shared-list sum at the edges of its splits -- lanes per query (4 to
64), queries per lane (1, 2, 4), hill stages (256) and steps (4 hills per lane
group) -- for every periodicity, and its deposits' hill count, against the
FP64 oracle.

Tolerances: a term's exponent q is formed in FP64 and rounded once to float32,
so the term carries 2^-24 q, and the float32 Gaussian and product 2e-7 more;
with these widths q stays below 25 for every pair (half a turn or two
standard deviations in each CV), so a term, and V, is within 3e-6 relative
(one far hill alone can be that far; near hills dominate longer lists).
dV/dxi: 1e-5 of the term scale sum_k e_k |D_kd| / sigma_d^2 (terms cancel).
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2301_04835_amd import Sampler, synth

from gpu_util import TWO_PI, dev

pytestmark = pytest.mark.gpu

RG = {"kind": "gyration", "idx": [0, 1, 2, 3, 4, 5]}
SETS = {"dihedral": (1, [True]), "two": (2, [True, True]), "three": (3, [True] * 3), "rg": (1, [False]),
        "mixed": (2, [True, False]), "mixed3": (3, [True, False, True])}


def cvs_of(per):
    return [{"kind": "dihedral", "idx": [d, d + 1, d + 2, d + 3]} if p else RG for d, p in enumerate(per)]


def draw(K, per, g):
    return np.stack([g.uniform(-np.pi, np.pi, K) if p else g.normal(0.9, 0.3, K) for p in per], 1)


def reference(xi, C, H, sigma, per):
    """V, dV/dxi and the term scale of the gradient."""
    V, dV = oracle.hillsum_batch(xi, None, C.astype(np.float64), H.astype(np.float64), sigma,
                                 [TWO_PI if p else 0.0 for p in per], nthreads=8)
    S = np.zeros_like(dV)
    for i in range(len(xi)):
        d = xi[i] - C.astype(np.float64)
        for k, p in enumerate(per):
            if p:
                d[:, k] -= TWO_PI * np.rint(d[:, k] / TWO_PI)
        e = H * np.exp(-np.sum(d * d / (2 * np.square(sigma)), 1))
        S[i] = np.sum(e[:, None] * np.abs(d), 0) / np.square(sigma)
    return V, dV, S


def close(V, dV, ref):
    Vr, dVr, S = ref
    assert np.all(np.abs(V - Vr) <= 3e-6 * Vr), np.max(np.abs(V - Vr) / Vr)
    assert np.all(np.abs(dV - dVr) <= 1e-5 * S), np.max(np.abs(dV - dVr) / S)


@pytest.mark.parametrize("name", list(SETS))
def test_points_and_hills_at_the_edges(gpu, name):
    D, per = SETS[name]
    sigma = [0.9, 0.7, 1.1][:D]
    g = np.random.default_rng(D)
    s = Sampler(0)
    s.add_cvs(cvs_of(per))
    s.metad(sigma, 1.0, 300.0, 6.0, 500, 20000)
    s.bind()
    many = draw(8300, per, g)
    for K in (1, 3, 4, 5, 255, 256, 257, 1023, 5000):
        C, H = draw(K, per, g).astype(np.float32), g.uniform(0.5, 1.5, K).astype(np.float32)
        s.hills_set(0, C, H)
        for n in (1, 2, 4, 5, 8, 9, 16, 17, 32, 33, 63, 64, 65):
            V, dV = s.bias_eval(dev(many[:n]))
            close(V.cpu().numpy(), dV.cpu().numpy(), reference(many[:n], C, H, sigma, per))
    pick = np.r_[0:5, 120:132, 1020:1030, 8188:8194, 8290:8300]
    ref = reference(many[pick], C, H, sigma, per)
    for n in (1023, 1024, 1025, 8191, 8192, 8193, 8300):
        at = pick[pick < n]
        V, dV = s.bias_eval(dev(many[:n]))
        close(V.cpu().numpy()[at], dV.cpu().numpy()[at], tuple(r[:len(at)] for r in ref))


@pytest.mark.parametrize("name", ["dihedral", "two", "three", "mixed"])
@pytest.mark.parametrize("W,K,cap", [(1, 700, 1000), (3, 40, 1000), (33, 9000, 30000), (70, 300, 20000)])
def test_step_and_deposits(gpu, name, W, K, cap):
    """A step (CVs in the sum for dihedral sets), its deposit and a second
    step on the grown list, in float32 and float64 positions; then a list too
    full to take the walkers' hills keeps its count."""
    D, per = SETS[name]
    sigma = [0.9, 0.7, 1.1][:D]
    g = np.random.default_rng(W + K)
    cvs = cvs_of(per)
    n = 10
    pos = np.concatenate([synth.chain_template(n, 60 + w) for w in range(W)])
    for dtype in (np.float32, np.float64):
        p = pos.astype(dtype)
        s = Sampler(0)
        s.add_cvs(cvs)
        s.set_walkers(np.arange(W + 1) * n, [cap], shared=True)
        s.metad(sigma, 1.2, 300.0, 6.0, 1, cap)
        s.bind()
        C, H = draw(K, per, g).astype(np.float32), g.uniform(0.5, 1.5, K).astype(np.float32)
        s.hills_set(0, C, H)
        P, F = dev(p), torch.zeros((W * n, 3), dtype=torch.float32, device=gpu)
        xr = np.zeros((W, D))
        Js = []
        for w in range(W):
            xr[w], J = oracle.cv_eval(p[w * n:(w + 1) * n].astype(np.float64), cvs)
            Js.append(J)
        for rep in range(2):
            xi = torch.zeros((W, D), dtype=torch.float64, device=gpu)
            V = torch.zeros(W, dtype=torch.float64, device=gpu)
            dV = torch.zeros((W, D), dtype=torch.float64, device=gpu)
            F.zero_()
            s.step(P, forces=F, xi_out=xi, V_out=V, dV_out=dV)
            s.check()
            assert np.max(np.abs(xi.cpu().numpy() - xr)) <= 1e-9
            ref = reference(xr, C, H, sigma, per)
            close(V.cpu().numpy(), dV.cpu().numpy(), ref)
            Fh = F.cpu().numpy().astype(np.float64)
            for w in range(W):
                Fr = -np.tensordot(dV.cpu().numpy()[w], Js[w], axes=(0, 0))
                assert np.max(np.abs(Fh[w * n:(w + 1) * n] - Fr)) <= 1e-5 * np.max(np.abs(Fr))
            C, H = s.hills_get(0)
            assert len(H) == K + (rep + 1) * W
            assert np.max(np.abs(C[-W:] - xr)) <= 1e-6
        full = draw(cap - W + 1, per, g).astype(np.float32)
        s.hills_set(0, full, np.ones(len(full), np.float32))
        s.deposit(dev(xr))
        with pytest.raises(Exception):
            s.check()
        assert s.hill_counts()[0] == len(full)
