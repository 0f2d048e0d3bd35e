"""Which kernels a call of the C ABI launches, found without a GPU: the calls run in a
process of their own over a recording stand-in for the HIP runtime (256 CUs), with
addresses that are never read.

record([call, ...]) -> one list of launches per call.  A call is a dict with the
entry point in "fn" and the sizes it takes:
  quantize, quantize_1d, mxfp8      R C dt [sr] [block] [stride_r] [x]
  grouped_quantize                  S C E dt [sr]
  gemm                              M N K ta tb fmt c_dt [ldc] [c] [acc]
  gemm_quantized                    M N K ta tb fmt [sr]
  grouped_gemm                      S N K E ta tb c_dt [ldc]
  linear_fwd, linear_bwd            T N K dt [oned] [block]; same: one descriptor for X and W,
                                    one buffer for dX and dW
fmt: "2d", "mxfp8", or which operands have 1D blocks ("a1", "b1", "a1b1").
dt, c_dt: "f32" or "bf16".  x, c: the address (its alignment matters).
A launch is a dict: kernel, args (its template arguments), grid, block, lds (dynamic)."""
import ctypes
import json
import os
import re
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2607_24953_amd", "libq2d.so")
DT = {"f32": 0, "bf16": 1}
FP4_2D, MXFP8, FP4_1D = 0, 1, 2
BASE = 1 << 32


def kernel_name(mangled: str):
    """(name, template arguments) of a kernel in libq2d's anonymous namespace, or None."""
    m = re.search(r"_GLOBAL__N_1(\d+)", mangled)
    if m is None:
        return None
    name = mangled[m.end():m.end() + int(m.group(1))]
    args = re.match(r"I((?:[ft]|L[a-z]\d+E)+)E", mangled[m.end() + len(name):])
    if args is None:
        return name, ()
    return name, tuple({"f": "float", "t": "bf16"}.get(a) or int(a[2:-1])
                       for a in re.findall(r"[ft]|L[a-z]\d+E", args.group(1)))


class _Tensor(ctypes.Structure):
    _fields_ = [("fmt", ctypes.c_int32), ("block", ctypes.c_int32), ("rows", ctypes.c_int64), ("cols", ctypes.c_int64),
                ("codes", ctypes.c_void_p), ("ld_codes", ctypes.c_int64),
                ("codes_t", ctypes.c_void_p), ("ld_codes_t", ctypes.c_int64),
                ("scales", ctypes.c_void_p), ("ld_scales", ctypes.c_int64),
                ("scales_t", ctypes.c_void_p), ("ld_scales_t", ctypes.c_int64)]


class _Launch(ctypes.Structure):
    _fields_ = [("name", ctypes.c_char_p), ("grid", ctypes.c_uint32), ("block", ctypes.c_uint32), ("lds", ctypes.c_uint64)]


def record(calls, tmp_path):
    if shutil.which("gcc") is None:
        import pytest
        pytest.skip("gcc not found")
    so = os.path.join(str(tmp_path), "launch_recorder.so")
    if not os.path.exists(so):
        subprocess.run(["gcc", "-std=c99", "-O1", "-Wall", "-shared", "-fPIC", "-o", so,
                        os.path.join(HERE, "launch_recorder.c")], check=True)
    run = subprocess.run([sys.executable, os.path.abspath(__file__), so], input=json.dumps(calls), capture_output=True,
                         text=True, timeout=300)
    assert run.returncode == 0, run.stderr[-4000:]
    out = json.loads(run.stdout)
    for launches in out:
        for l in launches:
            name = kernel_name(l.pop("name"))
            assert name is not None, l
            l["kernel"], l["args"] = name
    return out


def _main(so):
    rec = ctypes.CDLL(so, mode=ctypes.RTLD_GLOBAL)
    rec.recorded_launch.restype = ctypes.POINTER(_Launch)
    lib = ctypes.CDLL(LIB)
    P, I64, U64 = ctypes.c_void_p, ctypes.c_int64, ctypes.c_uint64

    def tensor(fmt, rows, cols, block=32, nseg=0):
        t = _Tensor()
        r = lib.q2d_grouped_tensor_init(ctypes.byref(t), I64(rows), I64(cols), nseg, block, None) if nseg else \
            lib.q2d_tensor_init(ctypes.byref(t), fmt, I64(rows), I64(cols), block, None)
        assert r == 0, r
        t.codes, t.codes_t, t.scales, t.scales_t = (BASE * i for i in (2, 3, 4, 5))
        return ctypes.byref(t)

    def operand(fmt, oned, rows, cols, trans):
        f = MXFP8 if fmt == "mxfp8" else FP4_1D if oned else FP4_2D
        return tensor(f, cols, rows) if trans else tensor(f, rows, cols)

    def call(fn, dt="bf16", sr=0, block=32, x=BASE, c=BASE, acc=0, c_dt="bf16", ldc=0, ta=0, tb=0, fmt="2d", R=0, C=0,
             S=0, E=0, T=0, M=0, N=0, K=0, stride_r=0, oned=0, same=0):
        d, s = DT[dt], U64(1)
        if fn in ("quantize", "quantize_1d"):
            out = tensor(FP4_1D if fn == "quantize_1d" else FP4_2D, R, C, block)
            return getattr(lib, "q2d_" + fn)(P(x), d, I64(R), I64(C), I64(stride_r or C), I64(1), block, sr, s, s, out, None)
        if fn == "mxfp8":
            return lib.mxfp8_quantize(P(x), d, I64(R), I64(C), I64(stride_r or C), I64(1), tensor(MXFP8, R, C), None)
        if fn == "grouped_quantize":
            return lib.q2d_grouped_quantize(P(x), d, I64(S), I64(C), I64(C), E, P(BASE * 6), 32, sr, s, s,
                                            tensor(FP4_2D, S, C, 32, E), None)
        if fn in ("gemm", "gemm_quantized"):
            a, b = operand(fmt, "a1" in fmt, M, K, ta), operand(fmt, "b1" in fmt, N, K, tb)
            if fn == "gemm":
                return lib.q2d_gemm(a, ta, b, tb, P(c), DT[c_dt], I64(ldc or N), acc, None)
            return lib.q2d_gemm_quantized(a, ta, b, tb, sr, s, s, tensor(FP4_2D, M, N), None)
        if fn == "grouped_gemm":
            a = tensor(FP4_2D, S, M if ta else K, 32, E)
            b = tensor(FP4_2D, S, N, 32, E) if ta else tensor(FP4_2D, E * K, N) if tb else tensor(FP4_2D, E * N, K)
            return lib.q2d_grouped_gemm(a, ta, b, tb, E, P(BASE * 6), I64(S), P(c), DT[c_dt], I64(ldc or N), acc, None)
        qx, qw = tensor(FP4_1D if oned else FP4_2D, T, K, 32 if oned else block), tensor(FP4_2D, N, K, block)
        if not same:
            for k in ("codes", "codes_t", "scales", "scales_t"):
                setattr(qw._obj, k, getattr(qw._obj, k) + BASE // 2)
        if fn == "linear_fwd":
            return lib.q2d_linear_fwd(P(x), P(BASE * 7), d, I64(T), I64(N), I64(K), sr, sr, s, s, s, qx, qw, P(c), d, None)
        assert fn == "linear_bwd", fn
        return lib.q2d_linear_bwd(P(x), d, qx, qw, 1, s, s, tensor(FP4_2D, T, N, block), P(c), d,
                                  P(c if same else BASE * 8), d, acc, None)

    out = []
    for kw in json.load(sys.stdin):
        rec.record_clear()
        status = call(**kw)
        assert status == 0, (kw, status)
        got = [rec.recorded_launch(i).contents for i in range(rec.recorded())]
        out.append([dict(name=l.name.decode(), grid=l.grid, block=l.block, lds=l.lds) for l in got])
    json.dump(out, sys.stdout)


if __name__ == "__main__":
    _main(sys.argv[1])
