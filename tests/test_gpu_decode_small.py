"""GPU: the decode GEMMs of steps of up to 32 sequences, at the edges of their token groups (8, 16 and 32 columns), with k ranges
that end inside a chunk, row groups that do not fill a tile, split k ranges, and every weight format.  Bounds of the parity tests."""
import dataclasses

import pytest

from paper_2603_20661_amd import synth
from test_gpu_parity import WIDE8B, WIDE8B_FP8, WIDE8B_Q128, check, run_job

pytestmark = pytest.mark.gpu

# 20 k blocks in the QKV GEMM, 129 (132 for int4) in the down projection, 514 row groups in the gate/up GEMM
H128 = synth.ModelShape("small128", 1, 640, 4, 1, 128, 4112, 528, 1e-5, 1e4, synth.WDTYPE_BF16, seed=501)
H64 = dataclasses.replace(H128, name="small64", n_q_heads=8, n_kv_heads=2, head_dim=64, seed=502)
FORMATS = [H128, H64, dataclasses.replace(H128, name="small128qk", qk_norm=1, seed=503), dataclasses.replace(H64, name="small64qk", qk_norm=1, seed=504),
           dataclasses.replace(H128, name="small128fp8", weight_dtype=synth.WDTYPE_FP8WO, seed=505),
           dataclasses.replace(H64, name="small64int4", ffn_dim=4224, weight_dtype=synth.WDTYPE_INT4WO_128, seed=506),
           dataclasses.replace(H128, name="small128int4", ffn_dim=4128, weight_dtype=synth.WDTYPE_INT4WO_32, seed=507),
           dataclasses.replace(H128, name="small128f32", weight_dtype=synth.WDTYPE_F32, seed=508),
           dataclasses.replace(H64, name="small64f32", weight_dtype=synth.WDTYPE_F32, seed=509),
           dataclasses.replace(H128, name="small512f32", d_model=512, ffn_dim=1040, weight_dtype=synth.WDTYPE_F32, seed=510)]


def route(shape, gemm, batch):
    """(kernel, tokens and rows per workgroup, k splits, -) of a GEMM of a step"""
    from paper_2603_20661_amd import binding as B
    return B.www_debug_route(B.make_config(shape, batch, 64, 64, 4096), gemm, batch)


@pytest.mark.parametrize("batch", [1, 8, 9, 17, 32])
@pytest.mark.parametrize("shape", FORMATS, ids=lambda s: s.name)
def test_formats_and_token_groups(shape, batch):
    lens = 2 + synth.uniform_i32(batch, 9, batch, 20)
    check(run_job(shape, lens, 2, seed=510 + batch), f"{shape.name} batch {batch}")


FULL_WIDTH = [(WIDE8B_Q128, 5, {"qkv": (64, 2), "down": (64, 4), "gate_up": (128, 1), "lm_head": (512, 1)}),
              (WIDE8B, 12, {"qkv": (64, 2), "down": (64, 4), "gate_up": (128, 1), "lm_head": (512, 1)}),
              (WIDE8B_FP8, 24, {"qkv": (64, 2), "down": (64, 4), "gate_up": (128, 1), "lm_head": (128, 1)})]


@pytest.mark.parametrize("shape,batch,expected", FULL_WIDTH, ids=lambda v: getattr(v, "name", str(v) if isinstance(v, int) else ""))
def test_full_width_tiles(shape, batch, expected):
    """several row groups per wavefront, k splits in narrow GEMMs, two and eight wavefronts side by side in the wide ones"""
    assert {g: route(shape, g, batch)[2:4] for g in ("qkv", "down", "gate_up", "lm_head")} == expected   # rows per workgroup, k splits
    lens = 2 + synth.uniform_i32(batch, 9, batch, 20)
    check(run_job(dataclasses.replace(shape, n_layers=1), lens, 2, seed=540 + batch), f"{shape.name} batch {batch}")


def test_int4_gate_up_of_two_token_groups():
    """128 rows a workgroup; the formats above have its 64"""
    assert route(WIDE8B_Q128, "gate_up", 20)[:4] == ("decode_small", 32, 128, 1)
    lens = 2 + synth.uniform_i32(20, 9, 20, 20)
    check(run_job(dataclasses.replace(WIDE8B_Q128, n_layers=1), lens, 2, seed=575), "int4 gate/up, 20 sequences")


def test_widest_sums_of_squares():
    """d_model = 8192: 512 entries per token, twice what the kernels request up front"""
    shape = dataclasses.replace(H128, name="small8192", d_model=8192, n_q_heads=2, n_kv_heads=2, ffn_dim=528, vocab=272, seed=520)
    for batch in (3, 20):
        check(run_job(shape, 2 + synth.uniform_i32(batch, 9, batch, 6), 2, seed=560 + batch), f"d_model 8192 batch {batch}")


# 344 row groups and 144 k blocks in the O projection, 400 and 172 in the QKV product: the general kernel's rows suit 17 to 32 tokens better
GENERAL = synth.ModelShape("small5504", 1, 5504, 40, 5, 128, 528, 272, 1e-5, 1e4, synth.WDTYPE_BF16, seed=521)


@pytest.mark.parametrize("shape", [dataclasses.replace(GENERAL, qk_norm=1), dataclasses.replace(GENERAL, name="small5504fp8", weight_dtype=synth.WDTYPE_FP8WO)],
                         ids=lambda s: s.name)
def test_narrow_products_in_the_general_kernel(shape):
    batch = 20
    assert route(shape, "qkv", batch)[:2] == route(shape, "o", batch)[:2] == ("decode", 32) and route(shape, "down", batch)[0] == "decode_small"
    check(run_job(shape, 2 + synth.uniform_i32(batch, 9, batch, 6), 2, seed=580), f"{shape.name} batch {batch}")
