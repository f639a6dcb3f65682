"""GPU: batches above 64 sequences, where the gate/up and output-head GEMMs take 128 tokens per workgroup (with a split k
range too) and the others 64, and where the last group of tokens is nearly empty, full, or padding only.  Bounds of the
parity tests."""
import dataclasses

import pytest

from paper_2603_20661_amd import synth
from test_gpu_parity import MID64, MID128, MIDF32, check, run_job

pytestmark = pytest.mark.gpu

FP8 = dataclasses.replace(MID128, name="mid128fp8", weight_dtype=synth.WDTYPE_FP8WO, seed=411)
INT4 = dataclasses.replace(MID128, name="mid128int4", ffn_dim=1408, weight_dtype=synth.WDTYPE_INT4WO_128, seed=412)


@pytest.mark.parametrize("shape,batch", [(MID128, 65), (MID128, 128), (MID64, 129), (MID64, 193), (MID128, 180), (FP8, 100), (INT4, 97), (MIDF32, 81)],
                         ids=lambda v: getattr(v, "name", str(v)))
def test_large_batches(shape, batch):
    lens = 3 + synth.uniform_i32(batch, 9, batch, 30)
    check(run_job(shape, lens, 2, seed=140 + batch), f"{shape.name} batch {batch}")


@pytest.mark.parametrize("batch", [18, 35, 49])
def test_groups_of_16_without_sequences(batch):
    lens = 3 + synth.uniform_i32(batch, 9, batch, 30)
    check(run_job(MID128, lens, 2, seed=170 + batch), f"batch {batch}")
