"""A list onto the nodes in slices, with 64 x 64 node tiles or 32 x 32 ones, at
the edges of the tiles and with fewer and more hills than the slices take at
a time, against the FP64 oracle's node values (the tolerance of the tiled
sums' tests: up to 1,500 terms of FP64 rounding, below 1e-12 of the grid's
largest value)."""
import numpy as np
import pytest

from gpu_util import dev  # noqa: F401  (the GPU helpers' import check)
from test_gpu_grid_tiles import check, make, points

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb,mixed", [([130], False), ([4096], False), ([64, 64], False), ([63, 65], True),
                                      ([65, 128], False), ([129, 70], True), ([200, 40], False), ([2, 33, 61], False),
                                      ([9, 7, 64], True), ([13, 12, 13], False)])
def test_list_in_slices(gpu, nb, mixed):
    s, sigma, ref = make(nb, mixed, cap=1500)
    for K in (1, 127, 129, 1500):
        x = points(K, len(nb), mixed, 300 + K)
        s.hills_set(0, x.astype(np.float32), np.linspace(0.5, 1.5, K).astype(np.float32))
        assert check(s, ref, sigma) == K
    s.hills_set(0, np.zeros((0, len(nb)), np.float32), np.zeros(0, np.float32))
    V, G = s.grid_get(0)
    assert not V.any() and not G.any()


def test_second_list_in_slices(gpu):
    """Each walker's own grid from its own list, the others left alone."""
    s, sigma, ref = make([70, 65], False, W=3, cap=300)
    for w, K in ((1, 300), (2, 40), (0, 7)):
        x = points(K, 2, False, 50 + w)
        s.hills_set(w, x.astype(np.float32), np.linspace(0.5, 1.5, K).astype(np.float32))
    assert [check(s, ref, sigma, w) for w in range(3)] == [7, 300, 40]
