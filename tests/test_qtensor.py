"""QTensor's buffers (host tensors stand in for device ones; nothing is launched): their
memory can be kept and given back by orientation, and sizes are the types they were."""
import ctypes
import gc
import weakref

import pytest
import torch


@pytest.fixture(scope="module")
def q2d():
    import paper_2607_24953_amd as q
    return q


def storage(t):
    return t.untyped_storage().nbytes()


@pytest.mark.parametrize("fmt", ["FP4_2D", "FP4_1D", "MXFP8"])
@pytest.mark.parametrize("rows,cols", [(4096, 4096), (8193, 1100)])
def test_one_orientation_holds_its_own_memory(q2d, fmt, rows, cols):
    q = q2d.QTensor(getattr(q2d, fmt), rows, cols, "cpu")
    for codes, scales in ((q.codes, q.scales), (q.codes_t, q.scales_t)):
        own = codes.numel() + scales.numel()
        assert own <= storage(codes) <= own + 512 and storage(scales) <= own + 512
    kept, want = q.codes, q.codes.data_ptr()
    other = weakref.ref(q._stores[1])
    del q, codes, scales
    gc.collect()
    assert other() is None and kept.data_ptr() == want


def test_dropped_orientation_gives_its_memory_back(q2d):
    q = q2d.QTensor(q2d.FP4_2D, 4096, 4096, "cpu")
    q.codes_t.fill_(1)
    other = weakref.ref(q._stores[1])
    q.codes_t = None
    q.scales_t = None
    assert other() is None and q.codes_t is None and q.scales_t is None
    # a call that needs it finds no buffer
    assert not q.desc.codes_t and not q.desc.scales_t
    fake = 0x1000
    assert q2d._lib.q2d_gemm(q.ptr(), 1, q.ptr(), 1, fake, 0, 4096, 0, None) == 1
    assert q.codes.shape == (4096, 2048) and q.desc.codes == q.codes.data_ptr()


@pytest.mark.parametrize("orientations", [(True, False), (False, True), (True, True), (False, False)])
@pytest.mark.parametrize("rows,cols", [(33, 70), (4096, 2500)])
def test_unwanted_orientations_have_no_buffer(q2d, orientations, rows, cols):
    q = q2d.QTensor(q2d.FP4_2D, rows, cols, "cpu", orientations=orientations)
    for want, names in zip(orientations, (("codes", "scales"), ("codes_t", "scales_t"))):
        for n in names:
            t = getattr(q, n)
            assert (t is not None) == want
            assert (getattr(q.desc, n) or 0) == (t.data_ptr() if want else 0)
            if want:
                assert t.data_ptr() % 16 == 0 and t.shape[1] == getattr(q.desc, "ld_" + n)


def test_sizes_of_other_types_stay_refused(q2d):
    """2048.0 equals 2048 as a cache key."""
    q2d.QTensor(q2d.FP4_2D, 64, 2048, "cpu")
    with pytest.raises((TypeError, ctypes.ArgumentError)):
        q2d.QTensor(q2d.FP4_2D, 64, 2048.0, "cpu")
    q2d.QTensor(q2d.FP4_2D, 64, 1, "cpu")
