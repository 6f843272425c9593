"""Calls whose lanes no single launch holds (2^32 and more are refused): host rules, no memory needed."""
import ctypes

import pytest

import paper_2511_11430_amd as vpm
from paper_2511_11430_amd import _lib


def _lanes(n_tgt, n_seg, per_pair):
    f = _lib.load()["_ZN3vpm13segment_lanesElli"]
    f.restype, f.argtypes = ctypes.c_int, [ctypes.c_int64, ctypes.c_int64, ctypes.c_int]
    return f(n_tgt, n_seg, per_pair)


@pytest.mark.parametrize("per_pair", [100, 260])
@pytest.mark.parametrize("n_seg", [0, 1, 64, 65, 4096, 1 << 30])
def test_segment_lanes_fit_a_launch(n_seg, per_pair):
    for n in (1, 1000, 1 << 24, (1 << 30) - 64, 1 << 30, (1 << 31) - 1):
        lanes = _lanes(n, n_seg, per_pair)
        assert lanes in (1, 4, 16, 64) and -(-n * lanes // 256) * 256 < 1 << 32, n
    # and as few lanes as 64 segments need, as many as a few targets need
    assert _lanes(400000, 64, per_pair) == 1 and _lanes(1000, 4096, per_pair) == 64


def test_batches_of_a_billion_targets_are_not_sliced():
    """One set of a billion targets over one source beside a dense one: sliced, a workgroup per 64 targets,
    it would not fit a launch; the queue of whole blocks does (its workspace: an item per 128 targets)."""
    src, tgt = [0, 1, 200001], [0, 1 << 30, (1 << 30) + 256]
    up = lambda b: (b + 255) // 256 * 256
    plain = 256 + 2 * up(8 * 3) + up(8 * ((1 << 23) + 2))
    assert vpm.vpm_workspace_size(vpm.F32C, src, tgt, self_eval=False) == plain
    # a small one of the same shape is sliced
    assert vpm.vpm_workspace_size(vpm.F32C, src, [0, 1 << 20, (1 << 20) + 256], self_eval=False) > \
        256 + 2 * up(8 * 3) + up(8 * ((1 << 13) + 2))
