"""Which kernel the sizes of a call lead to, evaluated on the host (256 compute units)."""
import dataclasses

import pytest

from paper_2603_20661_amd import synth

B = pytest.importorskip("paper_2603_20661_amd.binding", reason="libwww.so is not built")


def config(shape, max_batch=256):
    return B.make_config(shape, max_batch, 64, 16384, 4096)


@pytest.mark.parametrize("base", [synth.M1B, synth.M8B], ids=lambda s: s.name)
def test_fp32_weights_keep_the_general_decode_kernel(base):
    """two weight planes: above a small model's k ranges the kernel for few tokens takes up to 1.7 times as long"""
    cfg = config(dataclasses.replace(base, weight_dtype=synth.WDTYPE_F32))
    for batch in (1, 8, 9, 16, 17, 32):
        for gemm in B.GEMMS:
            assert B.www_debug_route(cfg, gemm, batch)[0] == "decode", (gemm, batch)
    small = config(dataclasses.replace(base, d_model=512, n_q_heads=8, n_kv_heads=2, head_dim=64, weight_dtype=synth.WDTYPE_F32))
    for batch in (1, 16, 32):
        assert B.www_debug_route(small, "qkv", batch)[0] == B.www_debug_route(small, "o", batch)[0] == "decode_small"


def test_widths_beyond_the_measured_models():
    """products whose rows and k range suit the general decode kernel better than workgroups of few rows"""
    wide = dataclasses.replace(synth.M8B, d_model=8192, n_q_heads=64, ffn_dim=28672)
    for wd in (synth.WDTYPE_BF16, synth.WDTYPE_FP8WO):
        cfg = config(dataclasses.replace(wide, weight_dtype=wd))
        assert [B.www_debug_route(cfg, "qkv", b)[0] for b in (16, 32)] == ["decode"] * 2 and B.www_debug_route(cfg, "down", 32)[0] == "decode"
    # 320 row groups: a quarter of the compute units would have two workgroups
    cfg = config(dataclasses.replace(synth.M8B, d_model=5120, n_q_heads=40, n_kv_heads=10, ffn_dim=13824))
    assert B.www_debug_route(cfg, "down", 4)[2:4] != (16, 1)
    # one round of row tiles in the output head
    assert B.www_debug_route(config(synth.M1B), "lm_head", 4)[0] == "decode" and B.www_debug_route(config(synth.M8B), "lm_head", 4)[0] == "decode_small"


@pytest.mark.parametrize("wd", [synth.WDTYPE_BF16, synth.WDTYPE_FP8WO, synth.WDTYPE_INT4WO_128])
@pytest.mark.parametrize("base", [synth.M1B, synth.M8B], ids=lambda s: s.name)
def test_narrow_products_of_few_tokens(base, wd):
    cfg = config(dataclasses.replace(base, weight_dtype=wd))
    for batch in (1, 8, 9, 16, 17, 32):
        for gemm in ("qkv", "o", "down"):
            assert B.www_debug_route(cfg, gemm, batch)[0] == "decode_small", (gemm, batch)
