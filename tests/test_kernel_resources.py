"""Resources of the built quantizer kernels, read from the library's own code object
metadata (no GPU needed): an input array that lands in scratch memory costs each
kernel its whole input once more in memory traffic, without any wrong result."""
import os
import re
import struct
import subprocess

import pytest

from launches import kernel_name, record

READELF = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(path):
    """gfx950 code objects of the offload bundles in a host library."""
    data = open(path, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, p)
            triple = data[p + 24:p + 24 + length].decode()
            p += 24 + length
            if "gfx950" in triple and size:
                yield data[at + off:at + off + size]
        at = data.find(MAGIC, at + 24)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Kernel name with its template arguments -> scratch and LDS bytes, VGPRs."""
    import paper_2607_24953_amd as q2d
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    found = {}
    for i, obj in enumerate(code_objects(q2d.lib_path)):
        f = tmp_path_factory.mktemp("co") / ("%d.co" % i)
        f.write_bytes(obj)
        text = subprocess.run([READELF, "--notes", str(f)], check=True, capture_output=True, text=True).stdout
        for part in re.split(r"\n  - ", text)[1:]:
            field = {k: re.search(r"\.%s:\s*'?([\w.]+)" % k, part) for k in
                     ("symbol", "private_segment_fixed_size", "group_segment_fixed_size", "vgpr_count")}
            if field["symbol"] is None:
                continue
            name = kernel_name(field["symbol"].group(1))
            if name is not None:
                found[name] = tuple(int(field[k].group(1)) for k in
                                    ("private_segment_fixed_size", "group_segment_fixed_size", "vgpr_count"))
    return found


def select(kernels, name, **want):
    """{arguments: (scratch, lds, vgprs)} of the kernels of that name whose arguments match."""
    fields = {"fp4_quantize_kernel": ("type", "vec", "sr", "wr", "grouped", "wc", "oned", "pair"),
              "mxfp8_quantize_kernel": ("f32", "vec")}[name]
    out = {}
    for (n, args), res in kernels.items():
        if n != name:
            continue
        assert len(args) == len(fields), args
        got = dict(zip(fields, args))
        if all(got[k] == v for k, v in want.items()):
            out[args] = res
    assert out, (name, want)
    return out


@pytest.mark.parametrize("vec", [1, 2, 3, 4])
def test_vector_load_quantizers_use_no_scratch(kernels, vec):
    found = select(kernels, "fp4_quantize_kernel", vec=vec)
    if vec <= 2:
        found.update(select(kernels, "mxfp8_quantize_kernel", vec=vec))
    for args, (scratch, _, _) in found.items():
        # (the grouped float32 kernels with round to nearest spill at their bound of 128 VGPRs)
        most = 96 if args[:5] == ("float", vec, 0, 4, 1) else 0
        assert scratch <= most, (args, scratch)


STREAMING = [dict(fn="quantize", R=16384, C=4096, sr=sr, block=block, dt=dt, stride_r=pitch)
             for sr in (0, 1) for block in (32, 64) for dt in ("bf16", "f32") for pitch in (0, 4099)] + \
            [dict(fn="quantize_1d", R=16384, C=C, sr=sr, dt=dt, stride_r=pitch)
             for sr in (0, 1) for C, dt, pitch in ((4096, "bf16", 0), (11008, "bf16", 0), (4096, "f32", 0), (4096, "bf16", 4099))] + \
            [dict(fn="grouped_quantize", S=131072, C=2048, E=128, sr=sr) for sr in (0, 1)] + \
            [dict(fn="mxfp8", R=16384, C=4096)]


def test_streaming_quantizers_fit_two_workgroups(kernels, tmp_path):
    """Inputs that stream from HBM: two workgroups of every quantizer fit a CU's 160 KB
    of LDS, own and dynamic together."""
    for call, launches in zip(STREAMING, record(STREAMING, tmp_path)):
        for l in launches:
            own = kernels[l["kernel"], l["args"]][1]
            assert 2 * (own + l["lds"]) <= 160 * 1024, (call, l, own)


def test_stochastic_64_blocks_are_not_held(kernels, tmp_path):
    """Their maximum is known behind a barrier only: as many workgroups as fit."""
    calls = [c for c in STREAMING if c["fn"] == "quantize" and c["sr"] == 1 and c["block"] == 64]
    for call, launches in zip(calls, record(calls, tmp_path)):
        assert [l["lds"] for l in launches] == [0], call
