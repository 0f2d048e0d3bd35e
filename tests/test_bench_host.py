"""Host-side logic of bench.py (no GPU): kernel-name classification of the
rocprofv3 traces, the algorithmic byte counts behind the roofline figures, the
split of a trace by workload, and the one-GPU guard."""
import os
import subprocess
import sys

import pytest
import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402

P = "void q2d::(anonymous namespace)::"


@pytest.mark.parametrize("name,kind", [
    (P + "gemm_fp4_persistent_kernel<true, false, 0, 0, false, false>(q2d::GemmArgs, int, int, q2d::GroupedArgs)", "gemm_fp4"),
    (P + "gemm_fp4_persistent_kernel<false, true, 0, 3, false, false>(q2d::GemmArgs, int, int, q2d::GroupedArgs)", "gemm_fp4"),
    (P + "gemm_fp4_persistent_kernel<true, false, 1, 0, false, false>(q2d::GemmArgs, int, int, q2d::GroupedArgs)",
     "gemm_fp4_grouped"),
    (P + "gemm_fp4_persistent_kernel<false, false, 2, 0, false, false>(q2d::GemmArgs, int, int, q2d::GroupedArgs)",
     "gemm_fp4_grouped_k"),
    (P + "gemm_fp4_persistent_kernel<false, false, 0, 1, true, false>(q2d::GemmArgs, int, int, q2d::GroupedArgs)",
     "gemm_fp4_yq"),
    (P + "gemm_fp4_persistent_kernel<false, false, 0, 0, true, false>(q2d::GemmArgs, int, int, q2d::GroupedArgs)",
     "gemm_fp4_yq"),
    (P + "gemm_fp4_persistent_kernel<false, false, 0, 0, true, true>(q2d::GemmArgs, int, int, q2d::GroupedArgs)",
     "gemm_fp4_dxq"),
    (P + "gemm_fp8_256_kernel<true, false, true>(q2d::GemmArgs, int, int)", "gemm_fp8"),
    (P + "gemm_ksplit_kernel<0, 1, 1, true, true>(q2d::(anonymous namespace)::Pair)", "gemm_fp4"),
    (P + "gemm_ksplit_kernel<1, 2, 2, false, false>(q2d::(anonymous namespace)::Pair)", "gemm_fp8"),
    (P + "gemm_tile_kernel<0, 2, 2, 3, 1, true, false>(q2d::(anonymous namespace)::Pair)", "gemm_fp4"),
    (P + "gemm_tile_kernel<1, 2, 2, 2, 1, true, true>(q2d::(anonymous namespace)::Pair)", "gemm_fp8"),
    (P + "gemm_tile_grouped_kernel<true>(q2d::GemmArgs, q2d::GroupedArgs, unsigned int)", "gemm_fp4_grouped"),
    (P + "gemm_tile_quant_kernel<2, 1, false>(q2d::GemmArgs, unsigned int, unsigned int)", "gemm_fp4_yq"),
    (P + "gemm_tile_quant_kernel<3, 0, true>(q2d::GemmArgs, unsigned int, unsigned int)", "gemm_fp4_dxq"),
    (P + "fp4_quantize_kernel<unsigned short, 2, false, 4, false, 2, false, false>(q2d::QuantArgs, q2d::QuantArgs, unsigned int)",
     "quant_fp4"),
    (P + "fp4_quantize_kernel<float, 1, true, 1, false, 1, false, true>(q2d::QuantArgs, q2d::QuantArgs, unsigned int)",
     "quant_fp4"),
    (P + "fp4_quantize_kernel<float, 2, true, 4, true, 2, false, false>(q2d::QuantArgs, q2d::QuantArgs, unsigned int)",
     "quant_fp4_grouped"),
    (P + "fp4_quantize_kernel<unsigned short, 4, true, 4, false, 2, true, false>(q2d::QuantArgs, q2d::QuantArgs, unsigned int)",
     "quant_fp4_1d"),
    (P + "mxfp8_quantize_kernel<false, 2>(q2d::QuantArgs)", "quant_mxfp8"),
    # (not one of the library's)
    ("gemm_kernel<0, true>(int)", None),
    ("void at::native::vectorized_elementwise_kernel<4, at::native::FillFunctor<float>>(int, float, float)", None),
])
def test_kind_of(name, kind):
    assert bench.kind_of(name) == kind


def test_every_kind_has_peak_kernel_and_source():
    for k in bench.KIND_PEAK:
        assert k in bench.KIND_KERNEL and k in bench.KIND_SOURCES


def test_byte_counts():
    t = torch.empty((64, 96), dtype=torch.bfloat16)
    n = 64 * 96
    assert bench.quant_bytes(t) == n * 2 + n + n / 1024
    assert bench.quant_bytes(t, "fp4_1d") == n * 2 + n + 2 * n / 32
    assert bench.quant_bytes(t, "mxfp8") == n * 2 + 2 * n + 2 * n / 32
    # A [M, K], B [N, K] FP4 codes with 2D scales, bf16 C [M, N]
    M, N, K = 256, 128, 512
    assert bench.gemm_bytes(M * K, N * K, M * N * 2) == (M * K + N * K) * (0.5 + 1 / 1024) + M * N * 2
    assert bench.gemm_bytes(M * K, N * K, 0, "fp4", True, False) == M * K * (0.5 + 1 / 32) + N * K * (0.5 + 1 / 1024)


def test_phase_owners():
    assert bench.phase_owners(5, [("a", 2), ("b", 3)]) == ["a", "a", "b", "b", "b"]
    with pytest.raises(ValueError):
        bench.phase_owners(4, [("a", 2), ("b", 3)])


def test_more_than_one_gpu_is_refused():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True,
                       text=True, timeout=120)
    assert r.returncode == 2 and "one GPU" in r.stderr


def test_result_line_is_short_and_the_detail_complete(tmp_path):
    import json
    kinds = {"gemm_fp4": {"achieved": 1.0, "launches_timed": 3}}
    rec = {"metric": "m", "value": 1.5, "kinds": kinds,
           "other_workloads": {"w%d" % i: {"TFLOP/s": 2.0, "ms_per_step": 3.0, "kinds": kinds, "launches": 7,
                                           "per_kernel": {"X" * 40: 1}} for i in range(8)}}
    line, detail = bench.printed(rec)
    got = json.loads(line)
    assert got["value"] == 1.5 and got["kinds"] == kinds
    assert got["other_workloads"]["w7"] == {"TFLOP/s": 2.0, "ms_per_step": 3.0}
    # both in one log, in either order: the record read back is the complete one
    for lines in ((detail, line), (line, detail)):
        log = tmp_path / "log"
        log.write_text("\n".join(("bench: measured", *lines)) + "\n")
        assert bench._json_line(str(log)) == rec
    log.write_text(line + "\n")
    assert bench._json_line(str(log)) == got
    assert json.loads(bench.printed({"value": 1})[0]) == {"value": 1}
