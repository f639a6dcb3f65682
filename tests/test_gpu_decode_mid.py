"""GPU: the residual products of steps of 33 to 64 sequences: token groups that are partly or all padding, splits and wavefronts whose range of
k ends early, FP8 units with one k block, both tile heights.  Bounds of the parity tests."""
import dataclasses

import pytest

from paper_2603_20661_amd import synth
from test_gpu_decode_small import route
from test_gpu_parity import check, run_job

pytestmark = pytest.mark.gpu

# 32 and 129 k blocks
ROWS32 = synth.ModelShape("mid640", 1, 640, 8, 2, 128, 4112, 272, 1e-5, 1e4, synth.WDTYPE_BF16, seed=901)
ROWS64 = dataclasses.replace(ROWS32, name="mid2176", d_model=2176, seed=902)
CASES = [(ROWS32, (32, 4), (32, 7)), (ROWS64, (64, 4), (64, 7)), (dataclasses.replace(ROWS32, name="mid640fp8", weight_dtype=synth.WDTYPE_FP8WO), (32, 2), (32, 7))]


@pytest.mark.parametrize("batch", [33, 48, 49, 64])
@pytest.mark.parametrize("shape,o,down", CASES, ids=lambda v: getattr(v, "name", ""))
def test_residual_products(shape, o, down, batch):
    assert (route(shape, "o", batch)[2:4], route(shape, "down", batch)[2:4]) == (o, down)   # rows per workgroup, k splits
    check(run_job(shape, 2 + synth.uniform_i32(batch, 9, batch, 20), 2, seed=910 + batch), f"{shape.name} batch {batch}")

# (shape, ffn_dim, splits of the down product): k blocks a split and in the last one, from which the wavefronts have
LOOPS = [(ROWS32, 9120, 8),       # 36, 33: 4 and 5 chunks
         (ROWS32, 11168, 8),      # 44, 41: 5 and 6; FP8 units 2 and 3
         (ROWS32, 15264, 8),      # 60, 57: 7 and 8; 3 and 4, one of a single block
         (ROWS32, 19392, 8),      # 76, 74: 9 and 10; 4 and 5
         (ROWS32, 23456, 8),      # 92, 89: 11 and 12; 5 and 6, one of a single block
         (ROWS64, 10784, 7),      # 52, 25: 6 and 7, 3 and 4
         (ROWS64, 16928, 7)]      # 76, 73: 9 and 10


@pytest.mark.parametrize("wd", [synth.WDTYPE_BF16, synth.WDTYPE_FP8WO], ids=["bf16", "fp8"])
@pytest.mark.parametrize("shape,ffn,splits", LOOPS, ids=lambda v: getattr(v, "name", str(v)))
def test_ring_of_chunks(shape, ffn, splits, wd):
    """every remainder of the ring of three (FP8: two) chunks, with none, one and two or more rounds of its loop"""
    shape = dataclasses.replace(shape, ffn_dim=ffn, weight_dtype=wd)
    if wd == synth.WDTYPE_FP8WO and shape.d_model > 2048:
        assert route(shape, "down", 64)[0] == "decode"               # (64 rows of FP8 weights: no kernel here)
        return
    for batch in (33, 64):
        assert route(shape, "down", batch)[:4] == ("decode_mid", 64, 16 * (2 if shape.d_model <= 2048 else 4), splits)
        check(run_job(shape, 2 + synth.uniform_i32(batch, 9, batch, 4), 1, seed=930 + batch), f"{shape.name} ffn {ffn} batch {batch}")
