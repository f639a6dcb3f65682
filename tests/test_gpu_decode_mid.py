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
