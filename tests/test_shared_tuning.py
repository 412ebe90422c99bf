"""A caller's number of workgroups for the shared sum (sx_set_tuning's grid) is
taken as it is, up to whole chunks; the default gives every compute unit the
same number.  Host arithmetic of the launch, no GPU."""
import ctypes

import pytest

from paper_2301_04835_amd import _lib


@pytest.fixture(scope="module")
def chunks():
    import os
    if not os.path.exists(_lib.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    f = _lib.load()._ZN2sx13shared_chunksElli
    f.restype, f.argtypes = ctypes.c_int32, [ctypes.c_int64, ctypes.c_int64, ctypes.c_int32]
    return f


@pytest.mark.parametrize("nq,blocks", [(1, 1), (64, 1), (100, 2), (256, 4), (1000, 16)])
@pytest.mark.parametrize("target", [1, 100, 255, 256, 300, 511, 700, 1024, 3000])
def test_explicit_number(chunks, nq, blocks, target):
    cap = 16000000 // nq // 256 * 256  # one query a lane up to 2^26 pairs
    stages = cap // 256
    assert chunks(cap, nq, target) == min(stages, -(-target // blocks))


@pytest.mark.parametrize("cap", [1, 255, 256, 257, 1000, 20000, 65536, 10 ** 6, 1 << 23])
@pytest.mark.parametrize("nq", [1, 5, 32, 33, 64, 65, 256, 1000, 1024, 8191, 8192, 40000, 65536])
def test_default_fits_the_records(chunks, cap, nq):
    """No more chunks than stages, and no more records than a batch of 65,536
    points reserves (and than 16 MiB)."""
    n, stages = chunks(cap, nq, 0), -(-cap // 256)
    assert 1 <= n <= stages
    assert n * nq <= min(stages, 8) * 65536
