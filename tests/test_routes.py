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
