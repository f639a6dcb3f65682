"""GPU: batches above 64 sequences, which the decode GEMMs take in groups of 64 tokens per workgroup, or of 128 in gate/up
GEMMs and output heads that fill the GPU in fewer rounds that way, and where the last group of tokens is nearly empty, full,
or padding only.  Bounds of the parity tests."""
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


WIDE = dataclasses.replace(MID128, name="wide", n_layers=1, ffn_dim=8320, vocab=20000, seed=413)        # 130 and 157 row tiles
WIDE_FP8 = dataclasses.replace(WIDE, name="widefp8", weight_dtype=synth.WDTYPE_FP8WO, seed=414)


@pytest.mark.parametrize("shape", [WIDE, WIDE_FP8], ids=lambda s: s.name)
@pytest.mark.parametrize("batch", [65, 100, 128, 129, 193])     # groups of 128 tokens up to 128 sequences, of 64 behind
def test_wide_gemms(shape, batch):
    lens = 3 + synth.uniform_i32(batch, 9, batch, 12)
    check(run_job(shape, lens, 2, seed=180 + batch), f"{shape.name} batch {batch}")


def test_wide_gemms_with_a_half_empty_group():
    """86 row tiles, 250 sequences: two groups of 128 tokens in the gate/up GEMM, the second of them not full"""
    shape = dataclasses.replace(WIDE, name="wide86", ffn_dim=5504, seed=415)
    check(run_job(shape, 3 + synth.uniform_i32(250, 9, 250, 12), 2, seed=190), "wide86 batch 250")
