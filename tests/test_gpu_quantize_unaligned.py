"""Quantizers on contiguous rows of any pitch and alignment (vector loads aligned to
the element only, partial sub-blocks at the right edge, Philox blocks that
straddle rows): every byte against the oracle, for widths around the 8-column
sub-block and the 128-column strip, odd pitches, and views whose base lies off a
16-byte boundary."""
import numpy as np
import pytest
import torch

import oracle
import synth
from helpers import assert_same_bytes, gpu_buffers, grouped_written, poison

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
VIEWS = [(131, 523, 0, 0, 523), (67, 300, 3, 1, 257), (40, 259, 0, 3, 256), (129, 144, 1, 7, 129), (33, 20, 0, 5, 9),
         (64, 1111, 2, 0, 1104), (9, 8, 0, 1, 7)]


@pytest.fixture(scope="module")
def q2d():
    import paper_2607_24953_amd as q
    return q


def views(dtype):
    """(label, device view, the same view on the host)"""
    for R, P, r0, c0, C in VIEWS:
        base = synth.normal((R, P), 1.0, R + P, dtype, device=DEV)
        synth.add_outlier_channels(base, 7, frac=0.02)
        yield "%s %s" % ((R, P, r0, c0, C), dtype), base[r0:, c0:c0 + C], base.cpu()[r0:, c0:c0 + C]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("mode", ["rtn", "sr"])
def test_unaligned_rows(q2d, dtype, mode):
    for label, x, h in views(dtype):
        assert x.stride() == h.stride()
        for block in (32, 64):
            q = q2d.QTensor(q2d.FP4_2D, *x.shape, DEV, block)
            poison(q)
            q2d.q2d_quantize(x, mode, 2**33 + 5, 2**40 + 3, out=q, block=block)
            assert_same_bytes(gpu_buffers(q), oracle.quantize_fp4_2d(h, mode, 2**33 + 5, 2**40 + 3, block=block), label)
        q = q2d.QTensor(q2d.FP4_1D, *x.shape, DEV)
        poison(q)
        q2d.q2d_quantize_1d(x, mode, 11, 4, out=q)
        assert_same_bytes(gpu_buffers(q), oracle.quantize_fp4_1d(h, mode, 11, 4), label + " 1d")


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_unaligned_rows_mxfp8(q2d, dtype):
    for label, x, h in views(dtype):
        q = q2d.QTensor(q2d.MXFP8, *x.shape, DEV)
        poison(q)
        q2d.mxfp8_quantize(x, out=q)
        assert_same_bytes(gpu_buffers(q), oracle.quantize_mxfp8(h), label)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("mode", ["rtn", "sr"])
def test_unaligned_rows_grouped(q2d, dtype, mode):
    """Segments of odd lengths start at any storage index modulo 8."""
    off = np.cumsum([0, 1, 0, 37, 130, 5, 64])
    for P, c0, C in ((301, 1, 299), (264, 0, 264), (65, 2, 33)):
        base = synth.normal((int(off[-1]), P), 1.0, P, dtype, device=DEV)
        x, h = base[:, c0:c0 + C], base.cpu()[:, c0:c0 + C]
        o = oracle.quantize_fp4_grouped(h, off, mode, 5, 6)
        q = q2d.q2d_grouped_quantize(x, torch.from_numpy(off).to(DEV), mode, 5, 6)
        P_rows = int(np.sum((np.diff(off) + 127) // 128 * 128))
        got = grouped_written(q, P_rows)
        for k, v in got.items():
            w = o[k][:P_rows] if k == "codes" else o[k][:P_rows // 32] if k == "scales" else \
                o[k][:, :P_rows // 2] if k == "codes_t" else o[k][:, :P_rows // 32]
            assert np.array_equal(v, w), (k, P, c0, C)
