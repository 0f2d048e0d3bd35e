"""Which kernel a call launches, by size and alignment, found on the CPU by recording
the launches (launches.py)."""
import pytest

from launches import record


@pytest.mark.parametrize("fn,extra", [("quantize", {}), ("quantize", {"block": 64}), ("quantize_1d", {})])
@pytest.mark.parametrize("dt", ["bf16", "f32"])
def test_stochastic_rounding_past_index_2_35_keeps_vector_loads(tmp_path, fn, extra, dt):
    rows = 40
    calls = [dict(fn=fn, R=rows, C=4096, sr=sr, dt=dt, stride_r=pitch, **extra)
             for sr in (0, 1) for pitch in (2 ** 25, 2 ** 30, 2 ** 30 + 2)]
    vec = [launches[0]["args"][1] for launches in record(calls, tmp_path)]
    # nearest (no draws), then stochastic: below the index, past it on and off 16-byte boundaries
    assert vec == [2, 2, 1, 2, 4, 3]
