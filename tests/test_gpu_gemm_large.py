"""GPU parity of the 256 x 256 GEMM kernels where they can go wrong: ragged M and N,
short K with several tiles a workgroup, 1D operands, accumulation, odd pitches and
misaligned outputs, blocks that are not finite, quantized outputs, ragged-M grouped
products.  The shapes are large enough for the tile choice to pick these kernels
(test_launch_routes.py checks that it does); references are float64 products, on the
GPU, of the values that q2d_dequantize gives for each operand.

float32 outputs of FP4 operands: relative Frobenius error <= 1e-5; MXFP8: the
elementwise bound derived from the matrix instruction's arithmetic; bf16: one rounding."""
from fractions import Fraction

import numpy as np
import pytest
import torch

import fp8_mfma_model as fm
import large_tiles
import oracle
import synth
from helpers import BUFS, assert_same_bytes, gpu_buffers
from test_gpu_fp8_mfma import gemm as gemm_of_codes, random_operand

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
BF16, F32 = torch.bfloat16, torch.float32
FORMATS = ("2d", "a1", "b1", "a1b1")


@pytest.fixture(scope="module")
def q2d():
    import paper_2607_24953_amd as q
    return q


@pytest.fixture(autouse=True)
def free_memory():
    yield
    torch.cuda.empty_cache()


def quantized(q2d, M, N, K, ta, tb, fmt, seed=0):
    """The two operands and the float64 product of their values."""
    A = synth.normal((K, M) if ta else (M, K), 1.0, M + K + seed, BF16, device=DEV)
    B = synth.normal((K, N) if tb else (N, K), 0.02, N + K + seed + 1, BF16, device=DEV)
    synth.add_outlier_channels(A, 5, frac=0.02)
    if fmt == "b64":
        qa, qb = q2d.q2d_quantize(A, block=64), q2d.q2d_quantize(B, "sr", 3, block=64)
        return qa, qb, product(q2d, qa, ta, qb, tb)
    qa = q2d.mxfp8_quantize(A) if fmt == "mxfp8" else q2d.q2d_quantize_1d(A) if "a1" in fmt else q2d.q2d_quantize(A)
    qb = q2d.mxfp8_quantize(B) if fmt == "mxfp8" else q2d.q2d_quantize_1d(B) if "b1" in fmt else q2d.q2d_quantize(B, "sr", 3)
    return qa, qb, product(q2d, qa, ta, qb, tb)


def product(q2d, qa, ta, qb, tb):
    a, b = q2d.q2d_dequantize(qa, ta).double(), q2d.q2d_dequantize(qb, tb).double()
    a = a.t().contiguous() if ta else a
    b = b if tb else b.t().contiguous()
    return a @ b


def check_f32(c, ref):
    assert float(torch.linalg.norm(c.double() - ref) / torch.linalg.norm(ref)) <= 1e-5


def check_bf16(c, ref):
    tol = ref.abs() * 2.0 ** -8 + 1e-5 * float(ref.square().mean().sqrt()) + 1e-38
    assert bool(((c.double() - ref).abs() <= tol).all())


def check_out(c, ref):
    (check_bf16 if c.dtype == BF16 else check_f32)(c, ref)


@pytest.mark.parametrize("M,N,K", large_tiles.SHORT_K + large_tiles.FP4)
@pytest.mark.parametrize("fmt,ta,tb", [("2d", 0, 0), ("2d", 1, 1), ("a1", 0, 0), ("b1", 1, 1), ("a1b1", 0, 1), ("b64", 0, 1)])
def test_fp4(q2d, M, N, K, fmt, ta, tb):
    qa, qb, ref = quantized(q2d, M, N, K, ta, tb, fmt)
    c32 = q2d.q2d_gemm(qa, ta, qb, tb, out_dtype=F32)
    check_f32(c32, ref)
    again = q2d.q2d_gemm(qa, ta, qb, tb, out_dtype=F32)
    assert torch.equal(c32, again)              # the result does not depend on timing
    q2d.q2d_gemm(qa, ta, qb, tb, out=again, accumulate=True)
    check_f32(again, 2 * ref)
    del c32, again
    check_bf16(q2d.q2d_gemm(qa, ta, qb, tb, out_dtype=BF16), ref)
    c0 = synth.normal((M, N), 0.5, 11, BF16, device=DEV)
    c16 = c0.clone()
    q2d.q2d_gemm(qa, ta, qb, tb, out=c16, accumulate=True)
    check_bf16(c16, ref + c0.double())


def strided(q2d, run, M, N, ref, dtype, pad, base, acc):
    """run(out, accumulate) into a view with an even or odd row pitch or a base one
    element off; nothing outside the view changes."""
    ld = N + pad
    flat = synth.normal((M * ld + 2,), 0.5, 33, dtype, device=DEV)
    before = flat.clone()
    c = flat[base:base + M * ld].view(M, ld)[:, :N]
    want = ref + c.double() if acc else ref
    run(c, acc)
    check_out(c, want)
    inside = torch.zeros(M * ld + 2, dtype=torch.bool, device=DEV)
    inside[base:base + M * ld].view(M, ld)[:, :N] = True
    assert torch.equal(flat[~inside], before[~inside])


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("pad,base", [(6, 0), (1, 0), (2, 1)])
@pytest.mark.parametrize("acc", [False, True])
def test_fp4_strided_output(q2d, dtype, pad, base, acc):
    M, N, K = large_tiles.FP4[1]
    qa, qb, ref = quantized(q2d, M, N, K, 0, 0, "2d")
    strided(q2d, lambda c, a: q2d.q2d_gemm(qa, 0, qb, 0, out=c, accumulate=a), M, N, ref, dtype, pad, base, acc)


@pytest.mark.parametrize("M,N,K", large_tiles.MXFP8)
@pytest.mark.parametrize("ta,tb", [(0, 0), (1, 1)])
def test_mxfp8(q2d, M, N, K, ta, tb):
    qa, qb, ref = quantized(q2d, M, N, K, ta, tb, "mxfp8")

    def fields(q, t):
        d = dict(gpu_buffers(q), rows=q.rows, cols=q.cols)
        return fm.operand_fields(d, bool(t))
    bound = torch.from_numpy(fm.error_bound(*fields(qa, ta), *fields(qb, tb))).to(DEV)
    c = q2d.q2d_gemm(qa, ta, qb, tb, out_dtype=F32)
    assert bool(((c.double() - ref).abs() <= bound).all())
    # the other outputs hold the same float32 sums: rounded once, or added to C
    c16 = q2d.q2d_gemm(qa, ta, qb, tb, out_dtype=BF16)
    assert torch.equal(c16, c.to(BF16))
    c0 = synth.normal((M, N), 0.5, 43, F32, device=DEV)
    acc = c0.clone()
    q2d.q2d_gemm(qa, ta, qb, tb, out=acc, accumulate=True)
    assert torch.equal(acc, c0 + c)
    acc = c0.to(BF16)
    want = (c + acc.float()).to(BF16)
    q2d.q2d_gemm(qa, ta, qb, tb, out=acc, accumulate=True)
    assert torch.equal(acc, want)


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("pad,base", [(6, 0), (1, 0), (2, 1)])
@pytest.mark.parametrize("shape", [1, 3])
def test_mxfp8_strided_output(q2d, dtype, pad, base, shape):
    M, N, K = large_tiles.MXFP8[shape]
    qa, qb, _ = quantized(q2d, M, N, K, 0, 0, "mxfp8")
    for acc in (False, True):
        # contiguous float32 output: checked in test_mxfp8
        ref = q2d.q2d_gemm(qa, 0, qb, 0, out_dtype=F32).double()
        strided(q2d, lambda c, a: q2d.q2d_gemm(qa, 0, qb, 0, out=c, accumulate=a), M, N, ref, dtype, pad, base, acc)


def test_mxfp8_single_instruction_bit_exact(q2d):
    """One instruction for each of 16400 x 16400 outputs; 512 sampled ones against the
    model of the instruction's arithmetic."""
    M, N, K = large_tiles.MXFP8_ONE_PRODUCT
    rng = np.random.default_rng(22)
    A, sA = random_operand(rng, M, K, 124, 131)
    B, sB = random_operand(rng, N, K, 124, 131)
    C = gemm_of_codes(q2d, A, sA, B, sB)
    for m, n in zip(rng.integers(0, M, 512), rng.integers(0, N, 512)):
        assert Fraction(float(C[m, n])) == fm.dot(A[m], sA[m], B[n], sB[n]), (m, n)


@pytest.mark.parametrize("fmt,t", [("2d", 0), ("2d", 1), ("a1b1", 0)])
def test_fp4_non_finite_blocks(q2d, fmt, t):
    """Exactly the outputs whose dot product meets a block with a NaN or an infinity
    are NaN."""
    M, N, K = large_tiles.FP4[0]
    A = synth.normal((K, M) if t else (M, K), 1.0, 91, F32, device=DEV)
    B = synth.normal((K, N) if t else (N, K), 0.02, 92, F32, device=DEV)
    A[5, 7] = float("nan")
    A[-1, -1] = float("inf")
    quantize = q2d.q2d_quantize_1d if fmt == "a1b1" else q2d.q2d_quantize
    qa, qb = quantize(A), quantize(B)
    ref = product(q2d, qa, t, qb, t)
    nan = ref.isnan()
    assert bool(nan.any()) and not bool(nan.all())
    for dtype in (F32, BF16):
        c = q2d.q2d_gemm(qa, t, qb, t, out_dtype=dtype)
        assert torch.equal(c.isnan(), nan)
        check_out(c[~nan], ref[~nan])


@pytest.mark.parametrize("fmt", FORMATS)
@pytest.mark.parametrize("mode", ["rtn", "sr"])
def test_fp4_quantized_output(q2d, fmt, mode):
    """Operands on the E2M1 grid with unit scales make the float32 sums exact, so every
    byte of the quantized output is the oracle's."""
    M, N, K = large_tiles.QUANTIZED
    g = torch.Generator(device=DEV)
    g.manual_seed(M + N)
    grid = torch.tensor([0, .5, 1, 1.5, 2, 3, 4, 6], device=DEV)

    def matrix(rows):
        x = grid[torch.randint(0, 8, (rows, K), generator=g, device=DEV)]
        x = x * (1 - 2 * torch.randint(0, 2, (rows, K), generator=g, device=DEV)).float()
        x[::32, :] = 6.0
        x[:, ::32] = 6.0
        return x

    a, b = matrix(M), matrix(N)
    qa = q2d.q2d_quantize_1d(a) if "a1" in fmt else q2d.q2d_quantize(a)
    qb = q2d.q2d_quantize_1d(b) if "b1" in fmt else q2d.q2d_quantize(b)
    got = q2d.q2d_gemm_quantized(qa, 0, qb, 0, mode, seed=2 ** 40 + 1, offset=9)
    again = q2d.q2d_gemm_quantized(qa, 0, qb, 0, mode, seed=2 ** 40 + 1, offset=9)
    assert all(torch.equal(getattr(got, k), getattr(again, k)) for k in BUFS)
    c = (a.double() @ b.double().t().contiguous()).float().cpu()
    assert_same_bytes(gpu_buffers(got), oracle.quantize_fp4_2d(c, mode, 2 ** 40 + 1, 9), "%s %s" % (fmt, mode))


@pytest.mark.parametrize("counts,N,K", large_tiles.GROUPED)
@pytest.mark.parametrize("tb", [0, 1])
@pytest.mark.parametrize("dtype,pad,base", [(F32, 0, 0), (BF16, 0, 0), (BF16, 3, 0), (BF16, 2, 1), (F32, 3, 0)])
def test_grouped_ragged_m(q2d, counts, N, K, tb, dtype, pad, base):
    """Empty experts, single rows and segments around a tile; odd row pitches and a base
    one element off (the rest stays as it was), accumulation."""
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    E, S = len(counts), int(off[-1])
    X = synth.normal((S, K), 1.0, S + K, BF16, device=DEV)
    W = synth.normal((E * K, N) if tb else (E * N, K), 0.02, N + K, BF16, device=DEV)
    offs = torch.from_numpy(off).to(DEV)
    qx, qw = q2d.q2d_grouped_quantize(X, offs), q2d.q2d_quantize(W)
    flat = synth.normal((S * (N + pad) + 2,), 0.5, 3, dtype, device=DEV)
    before = flat.clone()
    c = flat[base:base + S * (N + pad)].view(S, N + pad)[:, :N]
    q2d.q2d_grouped_gemm(qx, 0, qw, tb, offs, out=c)
    got = c.clone()
    q2d.q2d_grouped_gemm(qx, 0, qw, tb, offs, out=c, accumulate=True)
    inside = torch.zeros(flat.shape, dtype=torch.bool, device=DEV)
    inside[base:base + S * (N + pad)].view(S, N + pad)[:, :N] = True
    assert torch.equal(flat[~inside], before[~inside])
    w = q2d.q2d_dequantize(qw).double()
    for e in range(E):
        a, b = int(off[e]), int(off[e + 1])
        if a == b:
            continue
        x = q2d.q2d_dequantize(q2d.q2d_quantize(X[a:b].contiguous())).double()
        ref = x @ (w[e * K:(e + 1) * K] if tb else w[e * N:(e + 1) * N].t().contiguous())
        check_out(got[a:b], ref)
        check_out(c[a:b], ref + got[a:b].double())
