"""fm_batch_walk without a GPU: null arguments are refused."""
import ctypes

import pytest

fm = pytest.importorskip("paper_2609_14982_amd")


def test_walk_query_refuses_null():
    w = fm.binding.fm_walk()
    assert fm.load().fm_batch_walk(None, 0, ctypes.byref(w)) == fm.binding.FM_EINVAL
    assert fm.load().fm_batch_walk(None, 1, None) == fm.binding.FM_EINVAL
