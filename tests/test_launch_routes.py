"""Which kernel a call launches, by size and alignment, found on the CPU by recording
the launches (launches.py)."""
import pytest

import large_tiles
import test_gpu_gemm_small as small
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


FORMATS = {"2d": 0, "a1": 1, "b1": 2, "a1b1": 3}


def test_large_fp4_problems_take_the_persistent_kernel(tmp_path):
    calls = [dict(fn="gemm", M=M, N=N, K=K, c_dt=c_dt, fmt=fmt, acc=acc, ta=t, tb=t)
             for M, N, K in large_tiles.SHORT_K + large_tiles.FP4 for fmt in FORMATS
             for c_dt in ("f32", "bf16") for acc in (0, 1) for t in (0, 1)]
    for c, launches in zip(calls, record(calls, tmp_path)):
        assert [(l["kernel"], l["args"]) for l in launches] == \
            [("gemm_fp4_persistent_kernel", (int(c["c_dt"] == "bf16"), c["acc"], 0, FORMATS[c["fmt"]], 0, 0))], c


def test_large_mxfp8_problems_take_the_256_kernel(tmp_path):
    calls = [dict(fn="gemm", M=M, N=N, K=K, c_dt=c_dt, fmt="mxfp8", acc=acc)
             for M, N, K in large_tiles.MXFP8 + [large_tiles.MXFP8_ONE_PRODUCT] for c_dt in ("f32", "bf16") for acc in (0, 1)]
    for c, launches in zip(calls, record(calls, tmp_path)):
        assert [(l["kernel"], l["args"]) for l in launches] == \
            [("gemm_fp8_256_kernel", (int(c["c_dt"] == "bf16"), c["acc"], int((c["K"] + 127) // 128 % 4 == 0)))], c


def test_large_quantized_outputs_take_the_persistent_kernel(tmp_path):
    M, N, K = large_tiles.QUANTIZED
    calls = [dict(fn="gemm_quantized", M=M, N=N, K=K, fmt=fmt, sr=sr) for fmt in FORMATS for sr in (0, 1)]
    for c, launches in zip(calls, record(calls, tmp_path)):
        assert [(l["kernel"], l["args"]) for l in launches] == \
            [("gemm_fp4_persistent_kernel", (0, 0, 0, FORMATS[c["fmt"]], 1, c["sr"]))], c


def test_large_grouped_problems_take_the_persistent_kernel(tmp_path):
    calls = [dict(fn="grouped_gemm", S=sum(counts), N=N, K=K, E=len(counts), tb=tb, c_dt=c_dt, ldc=N + pad, acc=acc)
             for counts, N, K in large_tiles.GROUPED for tb in (0, 1) for c_dt in ("f32", "bf16") for pad in (0, 3)
             for acc in (0, 1)]
    for c, launches in zip(calls, record(calls, tmp_path)):
        assert [(l["kernel"], l["args"]) for l in launches] == \
            [("gemm_fp4_persistent_kernel", (int(c["c_dt"] == "bf16"), c["acc"], 1, 0, 0, 0))], c


@pytest.mark.parametrize("fmt", ["2d", "a1", "mxfp8"])
def test_small_shapes_cover_every_small_tile(tmp_path, fmt):
    """Every tile kernel, with whole and (FP4) half-filled last stages."""
    calls = [dict(fn="gemm", M=M, N=N, K=K, fmt=fmt, c_dt="f32") for M, N, K in small.SHAPES]
    seen = set()
    for c, launches in zip(calls, record(calls, tmp_path)):
        l, = launches
        odd = (c["K"] + 127) // 128 % 2
        seen.add((l["kernel"], l["args"][1:4] if "tile" in l["kernel"] else l["args"][1:3], odd))
    tiles = [("gemm_ksplit_kernel", (1, 1)), ("gemm_ksplit_kernel", (2, 2)), ("gemm_tile_kernel", (2, 2, 3)),
             ("gemm_tile_kernel", (2, 2, 2))]
    assert seen >= {(*t, odd) for t in tiles for odd in (0, 1)}, seen


def test_shared_launches_keep_the_order_of_overlapping_results(tmp_path):
    """One descriptor for X and W, one buffer for dX and dW: the second result replaces or
    adds to the first one's, so each goes out on its own."""
    calls = [dict(fn=fn, T=256, N=256, K=384, dt="f32", sr=1, same=same, acc=acc)
             for fn, acc in (("linear_fwd", 0), ("linear_bwd", 0), ("linear_bwd", 1)) for same in (0, 1)]
    calls = [{k: v for k, v in c.items() if k != "acc" or c["fn"] == "linear_bwd"} for c in calls]
    assert [len(launches) for launches in record(calls, tmp_path)] == [2, 3, 2, 3, 2, 3]
