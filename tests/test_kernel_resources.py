"""What kernels the library that was built here holds, from the metadata of its code objects (no GPU needed)."""
import dataclasses
import os
import re
import struct

import pytest

from paper_2603_20661_amd import synth

B = pytest.importorskip("paper_2603_20661_amd.binding", reason="libwww.so is not built")
msgpack = pytest.importorskip("msgpack")
LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_20661_amd", "libwww.so")


def _code_objects(data):
    """gfx950 ELF images of the offload bundles in the library"""
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := data.find(magic, at)) >= 0:
        n, pos = struct.unpack_from("<Q", data, at + 24)[0], at + 32
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, pos)
            if b"gfx950" in data[pos + 24:pos + 24 + idlen]:
                yield data[at + off:at + off + size]
            pos += 24 + idlen
        at += 24


def _kernels():
    out = {}
    for elf in _code_objects(open(LIB, "rb").read()):
        phoff, phsize, phnum = struct.unpack_from("<Q", elf, 32)[0], *struct.unpack_from("<HH", elf, 54)
        for i in range(phnum):
            kind, _, off, _, _, size = struct.unpack_from("<IIQQQQ", elf, phoff + i * phsize)
            if kind != 4:   # PT_NOTE
                continue
            namesz, descsz, typ = struct.unpack_from("<III", elf, off)
            if typ == 32:   # NT_AMDGPU_METADATA
                at = off + 12 + (namesz + 3) // 4 * 4
                for k in msgpack.unpackb(elf[at:at + descsz])["amdhsa.kernels"]:
                    out[k[".name"]] = k
    return out


def test_fp32_decode_kernels_of_64_tokens_spill_no_more_than_measured():
    """bytes of scratch per lane of the residual and gate/up kernels; with 196 and 176 they were 3 to 10 % slower"""
    kernels = _kernels()
    for epi, most in ((1, 148), (2, 172)):
        found = [k for name, k in kernels.items() if name.startswith(f"_Z18skinny_gemm_kernelILi4ELi1ELi{epi}ELi1EE")]
        assert len(found) == 1 and found[0][".private_segment_fixed_size"] <= most, (epi, [k[".private_segment_fixed_size"] for k in found])


def _shapes():
    """models from the smallest width to the widest, both head sizes, few and many kv heads, small and large vocabularies"""
    for d in (128, 256, 384, 512, 640, 1024, 1536, 2048, 3072, 4096, 5120, 8192):
        for hd in (64, 128):
            for heads, kv in ((max(1, d // hd), max(1, d // hd // 8)), (2, 2), (32, 32)):
                if heads % kv or heads // kv not in (1, 2, 4, 8):
                    continue
                for ffn, vocab in ((384, 512), (768, 50304), (2816, 32000), (14336, 128256)):
                    yield synth.ModelShape("any", 2, d, heads, kv, hd, ffn, vocab, 1e-5, 1e4, 1, seed=0)


def test_every_route_has_a_kernel_and_every_small_decode_kernel_a_route():
    """a shape without a kernel would leave its product out; a kernel without a shape is built for nothing"""
    wmode = {synth.WDTYPE_F32: 1, synth.WDTYPE_BF16: 0, synth.WDTYPE_FP8WO: 2, synth.WDTYPE_INT4WO_128: 3}
    epi = {"qkv": 0, "o": 1, "gate_up": 2, "down": 1, "lm_head": 3}
    reached = set()
    for shape in _shapes():
        for wd, wm in wmode.items():
            cfg = B.make_config(dataclasses.replace(shape, weight_dtype=wd), 300, 64, 4096, 4096)
            for batch in (1, 8, 9, 16, 17, 32, 33, 64, 65, 128, 200, 300):
                for gemm in B.GEMMS:
                    kernel, tokens, rows, _, _ = B.www_debug_route(cfg, gemm, batch)     # raises if there is none
                    if kernel == "decode_small":
                        groups = rows // 16
                        r = 2 if wd == synth.WDTYPE_F32 else min(groups, 4)
                        reached.add((wm, epi[gemm], r, groups // r, {8: 1, 16: 2, 32: 4}[tokens]))
    built = {tuple(map(int, m.groups())) for m in (re.match(r"_Z17small_gemm_kernelILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)E", k) for k in _kernels()) if m}
    assert reached == built, (sorted(reached - built), sorted(built - reached))


def test_every_decode_kernel_of_33_to_64_sequences_has_a_route():
    """and is named by the route hook; their rows fill whole workgroups"""
    wmode = {synth.WDTYPE_F32: 1, synth.WDTYPE_BF16: 0, synth.WDTYPE_FP8WO: 2, synth.WDTYPE_INT4WO_128: 3}
    reached = set()
    for shape in _shapes():
        for wd, wm in wmode.items():
            cfg = B.make_config(dataclasses.replace(shape, weight_dtype=wd), 64, 64, 64, 4096)
            for gemm in B.GEMMS:
                for batch in (32, 33, 64):
                    kernel, tokens, rows, splits, _ = B.www_debug_route(cfg, gemm, batch)
                    if kernel == "decode_mid":
                        assert batch > 32 and gemm in ("o", "down") and tokens == 64 and splits > 1 and shape.d_model % rows == 0
                        reached.add((wm, rows // 16))
    built = {tuple(map(int, m.groups())) for m in (re.match(r"_Z15mid_gemm_kernelILi(\d+)ELi(\d+)E", k) for k in _kernels()) if m}
    assert reached == built == {(0, 2), (0, 4), (2, 2)}


def test_sampling_kernels_use_no_scratch_memory():
    """in 80 bytes a lane, groups of four elements chosen by address, the in-place kernel took 3 % longer at 8193 tokens than the code before it, 8 % more at 128 256"""
    kernels = {k: v for k, v in _kernels().items() if "sample_" in k}
    assert len(kernels) >= 6
    assert {k for k, v in kernels.items() if v[".private_segment_fixed_size"]} == set()
