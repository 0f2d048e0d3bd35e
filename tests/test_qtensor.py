"""QTensor on host tensors (nothing is launched): sizes are the types they were."""
import ctypes

import pytest


@pytest.fixture(scope="module")
def q2d():
    import paper_2607_24953_amd as q
    return q


def test_sizes_of_other_types_stay_refused(q2d):
    """2048.0 equals 2048 as a cache key."""
    q2d.QTensor(q2d.FP4_2D, 64, 2048, "cpu")
    with pytest.raises((TypeError, ctypes.ArgumentError)):
        q2d.QTensor(q2d.FP4_2D, 64, 2048.0, "cpu")
    q2d.QTensor(q2d.FP4_2D, 64, 1, "cpu")
