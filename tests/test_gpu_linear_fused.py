"""The linear layer's shared launches (X and W quantized together, dX and dW in one
grid of small tiles) give what the separate calls give, byte for byte: tensors of
one and of several workgroup shapes, a ragged and an odd width (rows read in
different ways), mixed rounding, 64 x 64 blocks beside 32 x 32 ones, output types in
every combination, and an accumulated dW; results that share memory keep their order."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module")
def q2d():
    import paper_2607_24953_amd as q
    return q


@pytest.mark.parametrize("T,N,K", [(1, 8, 40), (100, 70, 33), (128, 256, 256), (500, 1000, 1304), (2000, 1100, 2048),
                                   (2300, 4096, 768), (4096, 300, 4000)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("mx,mw,fmt1d,bx,bw", [("rtn", "rtn", 0, 32, 32), ("sr", "sr", 0, 32, 32), ("rtn", "sr", 0, 32, 32),
                                               ("sr-floor", "sr", 0, 32, 64), ("rtn", "rtn", 1, 32, 32)])
def test_linear_equals_separate_calls(q2d, T, N, K, dtype, mx, mw, fmt1d, bx, bw):
    X = synth.normal((T, K), 1.0, T + K, dtype, device=DEV)
    W = synth.normal((N, K), 0.02, N + K, dtype, device=DEV)
    dY = synth.normal((T, N), 1e-3, T + N, dtype, device=DEV)
    qX = q2d.QTensor(q2d.FP4_1D if fmt1d else q2d.FP4_2D, T, K, DEV, 32 if fmt1d else bx)
    qW = q2d.QTensor(q2d.FP4_2D, N, K, DEV, bw)
    Y, _, _ = q2d.q2d_linear_fwd(X, W, mx, mw, 7, 3, 4, y_dtype=dtype, qX=qX, qW=qW)
    sX = q2d.q2d_quantize_1d(X, mx, 7, 3) if fmt1d else q2d.q2d_quantize(X, mx, 7, 3, block=bx)
    sW = q2d.q2d_quantize(W, mw, 7, 4, block=bw)
    for a, b in ((qX, sX), (qW, sW)):
        for k in ("codes", "codes_t", "scales", "scales_t"):
            assert torch.equal(getattr(a, k), getattr(b, k)), k
    assert torch.equal(Y, q2d.q2d_gemm(sX, 0, sW, 0, out_dtype=dtype))
    sdY = q2d.q2d_quantize(dY, "sr", 7, 5)
    for dx_dt, dw_dt in ((dtype, torch.float32), (torch.float32, torch.bfloat16), (torch.bfloat16, torch.bfloat16)):
        dX, dW, qdY = q2d.q2d_linear_bwd(dY, qX, qW, "sr", 7, 5, dx_dtype=dx_dt, dw_dtype=dw_dt)
        # sums of FP4 products of similar scale are exact in float32, whatever the tiles
        assert torch.equal(qdY.codes, sdY.codes)
        assert torch.equal(dX, q2d.q2d_gemm(sdY, 0, sW, 1, out_dtype=dx_dt))
        want = q2d.q2d_gemm(sdY, 1, sX, 1, out_dtype=dw_dt)
        assert torch.equal(dW, want)
        acc = want.clone()
        q2d.q2d_linear_bwd(dY, qX, qW, "sr", 7, 5, dx_dtype=dx_dt, dw_dtype=dw_dt, dW=acc, accumulate_dw=True)
        if dw_dt == torch.float32:
            assert torch.equal(acc, 2 * want)           # the same sums again, and doubling is exact
        else:
            assert torch.allclose(acc.float(), 2 * want.float(), rtol=2.0 ** -7, atol=0)


def test_results_in_one_buffer(q2d):
    """One descriptor for X and W (the second quantization stays), one buffer for dX and an
    accumulated dW (their sum): as from the calls one after the other."""
    n = 256
    X, W = (synth.normal((n, n), 1.0, k, torch.float32, device=DEV) for k in (1, 2))
    q = q2d.QTensor(q2d.FP4_2D, n, n, DEV)
    Y, _, _ = q2d.q2d_linear_fwd(X, W, "sr", "sr", 7, 3, 4, y_dtype=torch.float32, qX=q, qW=q)
    sW = q2d.q2d_quantize(W, "sr", 7, 4)
    for k in ("codes", "codes_t", "scales", "scales_t"):
        assert torch.equal(getattr(q, k), getattr(sW, k)), k
    assert torch.equal(Y, q2d.q2d_gemm(sW, 0, sW, 0))
    dY = synth.normal((n, n), 1e-3, 5, torch.float32, device=DEV)
    sX, sdY = q2d.q2d_quantize(X, "sr", 7, 3), q2d.q2d_quantize(dY, "sr", 7, 5)
    out = torch.empty((n, n), device=DEV)
    q2d.q2d_linear_bwd(dY, sX, sW, "sr", 7, 5, dx_dtype=torch.float32, dX=out, dW=out, accumulate_dw=True)
    want = q2d.q2d_gemm(sdY, 0, sW, 1)
    q2d.q2d_gemm(sdY, 1, sX, 1, out=want, accumulate=True)
    assert torch.equal(out, want)
