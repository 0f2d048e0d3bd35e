"""Stochastic rounding of views that reach past storage index 2^35, where the upper word
of the Philox counter is no longer 0: every byte against the oracle, on rows before,
across and behind that index, with rows on 16-byte boundaries and off them."""
import mmap

import numpy as np
import pytest
import torch

import oracle
import synth
from helpers import assert_same_bytes, gpu_buffers, grouped_written, poison

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
ROWS, COLS = 34, 300
ELEMENTS = 33 * 2 ** 30 + COLS                  # 71 GB of bf16, of which only the rows are touched


@pytest.fixture(scope="module")
def q2d():
    import paper_2607_24953_amd as q
    return q


@pytest.fixture(scope="module")
def spans():
    if torch.cuda.mem_get_info()[0] < 4 * ELEMENTS:
        pytest.skip("needs 71 GB of device memory, half of what is free at most")
    dev = torch.empty(ELEMENTS, dtype=torch.bfloat16, device=DEV)
    # address space only: anonymous, without reserve (0x4000: MAP_NORESERVE)
    buf = mmap.mmap(-1, 2 * ELEMENTS, flags=mmap.MAP_PRIVATE | mmap.MAP_ANONYMOUS | 0x4000)
    yield dev, torch.frombuffer(buf, dtype=torch.bfloat16, count=ELEMENTS)
    del dev
    torch.cuda.empty_cache()


# row 32 starts 256 or 64 elements before storage index 2^35
@pytest.mark.parametrize("pitch", [2 ** 30 - 8, 2 ** 30 - 2])
def test_storage_index_past_2_35(q2d, spans, pitch):
    x, h = (s.as_strided((ROWS, COLS), (pitch, 1)) for s in spans)
    h.copy_(synth.normal((ROWS, COLS), 1.0, 5, torch.bfloat16))
    x.copy_(h)
    for block in (32, 64):
        q = q2d.QTensor(q2d.FP4_2D, ROWS, COLS, DEV, block)
        poison(q)
        q2d.q2d_quantize(x, "sr", 2 ** 33 + 5, 2 ** 40 + 3, out=q, block=block)
        assert_same_bytes(gpu_buffers(q), oracle.quantize_fp4_2d(h, "sr", 2 ** 33 + 5, 2 ** 40 + 3, block=block), str(block))
    q = q2d.QTensor(q2d.FP4_1D, ROWS, COLS, DEV)
    poison(q)
    q2d.q2d_quantize_1d(x, "sr", 11, 4, out=q)
    assert_same_bytes(gpu_buffers(q), oracle.quantize_fp4_1d(h, "sr", 11, 4), "1d")
    off = np.array([0, 3, 3, ROWS])
    o = oracle.quantize_fp4_grouped(h, off, "sr", 5, 6)
    got = grouped_written(q2d.q2d_grouped_quantize(x, torch.from_numpy(off).to(DEV), "sr", 5, 6), 256)
    for k, v in got.items():
        w = o[k][:256] if k == "codes" else o[k][:8] if k == "scales" else o[k][:, :128] if k == "codes_t" else o[k][:, :8]
        assert np.array_equal(v, w), k
