"""GPU parity of the small-tile GEMM kernels against the float64 oracle, at the
sizes where they can go wrong: one and several tiles of every kind with ragged
M and N (clamped operand rows, masked stores), K of 1 to 32 units of 128 (shorter
than, equal to and longer than the LDS rings; odd numbers of units, where the last
128-byte stage is half empty), one to four waves with work in the K-split kernel.

float32 outputs of FP4 operands: relative Frobenius error <= 1e-5; MXFP8: the
elementwise bound derived from the matrix instruction's arithmetic; bf16: one
rounding.  The size rule gives, from the top: 32 x 32, 64 x 64, 128 x 128 tiles
one and two a CU."""
import numpy as np
import pytest
import torch

import fp8_mfma_model as fm
import oracle
import synth
from helpers import assert_same_bytes, check_bf16, gpu_buffers, rel_frob

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
SHAPES = [(1, 1, 1), (33, 31, 65), (100, 290, 640), (16, 260, 1700), (31, 700, 300),
          (500, 600, 1300), (250, 1000, 1792), (256, 2048, 4096),
          (700, 1100, 1300), (900, 1030, 1792), (1003, 1111, 1999),
          (2100, 2050, 700), (1800, 3000, 1700),
          # odd numbers of units on both rings of the 128 x 128 tiles, one to three units
          (1003, 1111, 1900), (1500, 1600, 300), (520, 4100, 100), (2100, 2050, 100), (2100, 2050, 370), (1800, 3000, 1650)]


@pytest.fixture(scope="module")
def q2d():
    import paper_2607_24953_amd as q
    return q


def operands(q2d, fmt, M, N, K, ta, tb):
    A = synth.normal((K, M) if ta else (M, K), 1.0, M + K, torch.bfloat16, device=DEV)
    B = synth.normal((K, N) if tb else (N, K), 0.02, N + K + 1, torch.bfloat16, device=DEV)
    synth.add_outlier_channels(A, 5, frac=0.02)
    if fmt == "mxfp8":
        return q2d.mxfp8_quantize(A), oracle.quantize_mxfp8(A.cpu()), q2d.mxfp8_quantize(B), oracle.quantize_mxfp8(B.cpu())
    if "a1" in fmt:
        qa, oa = q2d.q2d_quantize_1d(A), oracle.quantize_fp4_1d(A.cpu(), "rtn")
    else:
        qa, oa = q2d.q2d_quantize(A), oracle.quantize_fp4_2d(A.cpu(), "rtn")
    if "b1" in fmt:
        return qa, oa, q2d.q2d_quantize_1d(B), oracle.quantize_fp4_1d(B.cpu(), "rtn")
    return qa, oa, q2d.q2d_quantize(B), oracle.quantize_fp4_2d(B.cpu(), "rtn")


def values(o, t, fmt, which):
    return oracle.operand(o, bool(t), "mxfp8" if fmt == "mxfp8" else "fp4_1d" if which in fmt else "fp4")


@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("fmt,ta,tb", [("2d", 0, 0), ("2d", 1, 1), ("a1", 0, 0), ("b1", 1, 1), ("a1b1", 0, 1),
                                       ("mxfp8", 0, 0), ("mxfp8", 1, 1)])
def test_small_gemm(q2d, M, N, K, fmt, ta, tb):
    qa, oa, qb, ob = operands(q2d, fmt, M, N, K, ta, tb)
    a64, b64 = values(oa, ta, fmt, "a1"), values(ob, tb, fmt, "b1")
    ref = oracle.gemm(a64, b64)
    c = q2d.q2d_gemm(qa, ta, qb, tb, out_dtype=torch.float32).cpu().numpy().astype(np.float64)
    if fmt == "mxfp8":
        av, am = fm.operand_fields(oa, bool(ta))
        bv, bm = fm.operand_fields(ob, bool(tb))
        assert np.all(np.abs(c - ref) <= fm.error_bound(av, am, bv, bm))
        # one bf16 rounding of the float32 result, which is the same in both outputs
        ref = c
    else:
        assert rel_frob(c, ref) <= 1e-5
    check_bf16(q2d.q2d_gemm(qa, ta, qb, tb, out_dtype=torch.bfloat16), ref)


@pytest.mark.parametrize("M,N,K", [(33, 63, 300), (500, 600, 1300), (900, 1030, 1792), (2100, 2050, 700)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("pad,base,acc", [(6, 0, False), (1, 0, True), (2, 1, False)])
def test_small_gemm_strided_output(q2d, M, N, K, dtype, pad, base, acc):
    """Into a view with an even or odd row pitch or a base one element off, with and
    without accumulation; nothing outside the view changes."""
    qa, oa, qb, ob = operands(q2d, "2d", M, N, K, 0, 0)
    ref = oracle.gemm(oracle.operand(oa, False), oracle.operand(ob, False))
    ld = N + pad
    flat = synth.normal((M * ld + 2,), 0.5, 33, dtype, device=DEV)
    before = flat.clone()
    c = flat[base:base + M * ld].view(M, ld)[:, :N]
    c0 = c.float().cpu().numpy().astype(np.float64)
    q2d.q2d_gemm(qa, 0, qb, 0, out=c, accumulate=acc)
    want = ref + c0 if acc else ref
    if dtype == torch.bfloat16:
        check_bf16(c, want)
    else:
        assert rel_frob(c.cpu().numpy(), want) <= 1e-5
    inside = torch.zeros(M * ld + 2, dtype=torch.bool, device=DEV)
    inside[base:base + M * ld].view(M, ld)[:, :N] = True
    assert torch.equal(flat[~inside], before[~inside])
    if not acc:
        again = c.clone()
        q2d.q2d_gemm(qa, 0, qb, 0, out=c)
        assert torch.equal(c, again)            # the K split adds in a fixed order


@pytest.mark.parametrize("counts,N,K", [((1, 0, 127, 128, 129, 40), 160, 384), ((300,) * 7, 640, 128),
                                        ((0, 5, 260, 33) * 15, 1024, 640)])
@pytest.mark.parametrize("tb", [0, 1])
@pytest.mark.parametrize("dtype,pad", [(torch.float32, 0), (torch.bfloat16, 0), (torch.bfloat16, 1)])
def test_small_grouped_gemm(q2d, counts, N, K, tb, dtype, pad):
    """Ragged-M products with few tiles (128 x 128 tiles): empty experts, segments of
    one row and around a tile, odd numbers of K units, several tiles a workgroup, an
    odd row pitch, accumulation.  Per expert against the float64 oracle."""
    if tb and K % 128:
        pytest.skip("transposed weights need K of whole 128")
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    E, S = len(counts), int(off[-1])
    X = synth.normal((S, K), 1.0, S + K, torch.bfloat16, device=DEV)
    W = synth.normal((E * K, N) if tb else (E * N, K), 0.02, N + K, torch.bfloat16, device=DEV)
    offs = torch.from_numpy(off).to(DEV)
    qx, qw = q2d.q2d_grouped_quantize(X, offs), q2d.q2d_quantize(W)
    flat = synth.normal((S, N + pad), 0.5, 3, dtype, device=DEV)
    before = flat.clone()
    c = flat[:, :N]
    q2d.q2d_grouped_gemm(qx, 0, qw, tb, offs, out=c)
    got = c.clone()
    q2d.q2d_grouped_gemm(qx, 0, qw, tb, offs, out=c, accumulate=True)
    assert torch.equal(flat[:, N:], before[:, N:])
    ow = oracle.operand(oracle.quantize_fp4_2d(W.cpu(), "rtn"), False)
    for e in range(E):
        a, b = int(off[e]), int(off[e + 1])
        if a == b:
            continue
        xe = oracle.operand(oracle.quantize_fp4_2d(X[a:b].cpu().contiguous(), "rtn"), False)
        we = ow[e * K:(e + 1) * K].T if tb else ow[e * N:(e + 1) * N]
        ref = oracle.gemm(xe, we)
        if dtype == torch.bfloat16:
            check_bf16(got[a:b], ref)
            check_bf16(c[a:b], ref + got[a:b].double().cpu().numpy())
        else:
            assert rel_frob(got[a:b].cpu().numpy(), ref) <= 1e-5
            assert rel_frob(c[a:b].cpu().numpy(), 2 * ref) <= 1e-5


@pytest.mark.parametrize("M,N,K,fmt", [(130, 200, 384, "2d"), (700, 1032, 1300, "a1"), (1500, 3000, 640, "2d"),
                                       (2100, 4000, 384, "b1"), (4090, 4088, 4100, "2d")])
@pytest.mark.parametrize("mode", ["rtn", "sr"])
def test_small_gemm_quantized(q2d, M, N, K, fmt, mode):
    """FP4 outputs from 128 x 128 tiles, one and two workgroups a CU, and (last) from
    the persistent kernel: operands on the E2M1 grid with unit scales make the
    float32 sums exact, so every byte is the oracle's."""
    rng = np.random.default_rng(M + N)
    grid = np.array([0, .5, 1, 1.5, 2, 3, 4, 6], np.float32)

    def matrix(rows):
        x = grid[rng.integers(0, 8, (rows, K))] * rng.choice(np.array([-1, 1], np.float32), (rows, K))
        x[::32, :] = 6.0
        x[:, ::32] = 6.0
        return torch.from_numpy(x)

    a, b = matrix(M), matrix(N)
    qa = q2d.q2d_quantize_1d(a.to(DEV)) if fmt == "a1" else q2d.q2d_quantize(a.to(DEV))
    qb = q2d.q2d_quantize_1d(b.to(DEV)) if fmt == "b1" else q2d.q2d_quantize(b.to(DEV))
    got = q2d.q2d_gemm_quantized(qa, 0, qb, 0, mode, seed=2**40 + 1, offset=9)
    want = oracle.gemm_quantized(a.numpy().astype(np.float64), b.numpy().astype(np.float64), mode, 2**40 + 1, 9)
    assert_same_bytes(gpu_buffers(got), want, "%s %s" % ((M, N, K), mode))
