"""Times of calls next to those of their neighbours: a form of a call may not
cost a multiple of another that does the same work.  Each bound lies midway
between what was measured and the fault it stands against; times are the best
of several rounds in one process.
"""
import numpy as np
import pytest
import torch

from paper_2301_04835_amd import Sampler, synth

from gpu_util import dev

pytestmark = pytest.mark.gpu

RG = {"kind": "gyration", "idx": [0, 1, 2, 3, 4, 5]}


def best_us(call, reps, rounds=7):
    call()
    torch.cuda.synchronize()
    t = []
    for _ in range(rounds):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(reps):
            call()
        b.record()
        torch.cuda.synchronize()
        t.append(a.elapsed_time(b) * 1e3 / reps)
    return min(t)


def eval_us(per, n, K):
    g = np.random.default_rng(n)
    s = Sampler(0)
    s.add_cvs([{"kind": "dihedral", "idx": [d, d + 1, d + 2, d + 3]} if p else RG for d, p in enumerate(per)])
    s.metad([0.35 if p else 0.03 for p in per], 1.0, 300.0, 6.0, 500, K)
    s.bind()
    draw = lambda m: np.stack([g.uniform(-np.pi, np.pi, m) if p else g.normal(0.25, 0.05, m) for p in per], 1)
    s.hills_set(0, draw(K).astype(np.float32), np.ones(K, np.float32))
    x = dev(draw(n))
    V = torch.empty(n, dtype=torch.float64, device=x.device)
    dV = torch.empty((n, len(per)), dtype=torch.float64, device=x.device)
    return best_us(lambda: s.bias_eval_noalloc(x, V, dV), 3)


@pytest.mark.parametrize("n", [700, 8191, 20000])
@pytest.mark.parametrize("per", [[True, False], [False, True], [True, False, True], [False, True, False]])
def test_mixed_sets_sum_as_fast_as_angles(gpu, per, n):
    """A CV without a period takes two operations a pair, an angle four."""
    mixed, angles = eval_us(per, n, 200000), eval_us([True] * len(per), n, 200000)
    print(per, n, round(mixed, 1), round(angles, 1))
    assert mixed <= 1.15 * angles


@pytest.mark.parametrize("D", [1, 2, 3])
def test_short_lists_stay_fast_with_many_points(gpu, D):
    """1,000 hills: one point more, at the sizes where queries per lane may
    change, costs nothing (1.4 times with four a lane on 128 workgroups)."""
    below, above = eval_us([True] * D, 8191, 1000), eval_us([True] * D, 8192, 1000)
    print(D, round(below, 1), round(above, 1))
    assert above <= 1.2 * below


@pytest.mark.parametrize("D", [1, 2, 3])
def test_windows_take_no_second_round(gpu, D):
    """2,048 windows fit the chip at once, as 1,700 do (1.3 times otherwise)."""
    t = []
    for W in (1700, 2048):
        pos = np.concatenate([synth.chain_template(22, 60 + w % 64) for w in range(W)]).astype(np.float32)
        s = Sampler(0)
        s.add_cvs([{"kind": "dihedral", "idx": [d, d + 1, d + 2, d + 3]} for d in range(D)])
        s.set_walkers(np.arange(W + 1) * 22)
        s.harmonic([100.0] * D, np.zeros((W, D)))
        s.bind()
        P = dev(pos)
        F = torch.zeros_like(P)
        s.graph_capture(20, P, forces=F)
        t.append(best_us(s.graph_launch, 5) / 20)
    print(D, [round(x, 2) for x in t])
    assert t[1] <= 1.12 * t[0]


@pytest.mark.parametrize("nb", [[4096], [1000, 2], [2, 1000]])
def test_private_grids_take_their_hill_side_by_side(gpu, nb):
    """A step in which each of 32 walkers puts one hill onto its own grid, next
    to one walker's (1.8 times and more with tiles of matrix products)."""
    t = []
    for W in (1, 32):
        D = len(nb)
        s = Sampler(0)
        for d in range(D):
            s.add_dihedral([d, d + 1, d + 2, d + 3])
        s.set_walkers(np.arange(W + 1) * 22, hill_capacity=[20000] * W)
        s.metad([0.35] * D, 1.2, 300.0, 6.0, 1)
        s.metad_grid([-np.pi] * D, [np.pi] * D, nb)
        s.bind()
        P = dev(np.concatenate([synth.chain_template(22, 40 + w) for w in range(W)]).astype(np.float32))
        F = torch.zeros_like(P)
        s.graph_capture(20, P, forces=F)
        t.append(best_us(s.graph_launch, 5) / 20)
        s.check()
    print(nb, [round(x, 2) for x in t])
    assert t[1] <= 1.6 * t[0]


@pytest.mark.parametrize("n,box", [(20000, 40.0), (20000, 80.0), (41000, 60.0)])
def test_crowded_cells_sort_in_linear_time(gpu, n, box):
    """A droplet at water's density in a large box, whose cells hold hundreds of
    members, next to the same atoms all over a box of the usual density (3.9 and
    17 times with every member counting its cell's)."""
    t = []
    g = np.random.default_rng(n)
    for L in ((2 * n / 23.0) ** (1 / 3), box):
        x = g.random((2 * n, 3)) * L
        if L == box:
            v = g.normal(size=(2 * n, 3))
            r = (2 * n / 33.0 * 0.75 / np.pi) ** (1 / 3) * g.random((2 * n, 1)) ** (1 / 3)
            x = L / 2 + r * v / np.linalg.norm(v, axis=1, keepdims=True)
        s = Sampler(0)
        s.add_coordination(list(range(n)), list(range(n, 2 * n)), 0.5, rcut=1.2)
        s.set_box([L] * 3)
        s.set_walkers(np.array([0, 2 * n], dtype=np.int64))
        s.set_cell_lists(1)
        s.metad([0.2], 1.0, 300.0, None, 500, 1000)
        s.bind()
        P = dev(x.astype(np.float32))
        F = torch.zeros_like(P)
        s.step(P, forces=F)
        s.check()
        t.append(min(s.time_cell(P, F, reps=5)[0] for _ in range(3)) * 1e3)
    print(n, box, [round(x, 1) for x in t])
    assert t[1] <= 2.8 * t[0]
