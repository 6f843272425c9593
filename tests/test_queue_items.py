"""Host side of the batched launches: the work queue's (set, block) items, against the same items
listed one by one and sorted by cost."""
import ctypes
import time

import numpy as np
import pytest

from paper_2511_11430_amd import _lib

P64 = ctypes.POINTER(ctypes.c_int64)


def _queue_items(lane, loop, per):
    f = _lib.load()["_ZN3vpm11queue_itemsEiPKlS1_S1_P15HIP_vector_typeIiLj2EE"]
    f.restype = ctypes.c_int64
    f.argtypes = [ctypes.c_int32, P64, P64, P64, ctypes.c_void_p]
    arrs = [np.ascontiguousarray(v, dtype=np.int64) for v in (np.r_[0, np.cumsum(lane)], np.r_[0, np.cumsum(loop)], per)]
    p = [a.ctypes.data_as(P64) for a in arrs]
    n = f(len(lane), *p, None)
    out = np.full((n, 2), -1, dtype=np.int32)
    seconds = []
    for _ in range(30):
        t0 = time.perf_counter()
        assert f(len(lane), *p, out.ctypes.data) == n
        seconds.append(time.perf_counter() - t0)
    return out, min(seconds)


def _one_by_one(lane, loop, per):
    items = [((no + 1) * min(pb, nl - k * pb), b, k) for b, (nl, no, pb) in enumerate(zip(lane, loop, per))
             for k in range(-(-nl // pb))]
    return np.array([(b, k) for _, b, k in sorted(items, key=lambda i: -i[0])], dtype=np.int32).reshape(-1, 2)


# sets of a multiple of a block, of one particle, empty ones, equal sets, a short block as dear as another set's whole one
@pytest.mark.parametrize("lane,loop,per", [
    ([64, 0, 1, 130, 64, 128], [64, 0, 1, 130, 64, 128], [64] * 6),
    ([100, 36, 36], [63, 127, 127], [64, 32, 32]),
    ([0, 0], [5, 0], [16, 16]),
    ([7] * 9, [0, 3] * 4 + [0], [1, 2, 4, 8, 256] * 1 + [3, 5, 6, 7]),
])
def test_items_in_decreasing_cost(lane, loop, per):
    assert np.array_equal(_queue_items(lane, loop, per)[0], _one_by_one(lane, loop, per))


def test_items_of_many_uneven_sets():
    """64 uneven sets in blocks of 64 (11000 items): the order, and that it costs no sort of every item
    (1.5 ns per item measured, 11 with one)."""
    n = np.exp(np.random.default_rng([64, 512, 50000]).uniform(np.log(512), np.log(50000), 64)).astype(int).tolist()
    out, seconds = _queue_items(n, n, [64] * 64)
    assert len(out) > 8000 and np.array_equal(out, _one_by_one(n, n, [64] * 64))
    assert seconds < 5e-9 * len(out)
