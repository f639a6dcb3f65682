"""GPU: the merge of a sequence's partial attention results, at the record counts where its loads, its rounds and its wavefronts' shares end
(2, 4 and 8 loads of two or four records; 16, 32 and 64 records), for every number of query heads per kv head.  Bounds of the parity tests."""
import dataclasses

import pytest

from paper_2603_20661_amd import synth
from test_gpu_parity import check, run_job

pytestmark = pytest.mark.gpu

# one kv head: a sequence of n tokens has ceil(n / 32) records, up to 64 (then 32 of two pairs of blocks, growing again)
SHAPE = synth.ModelShape("merge", 1, 256, 4, 1, 64, 272, 272, 1e-5, 1e4, synth.WDTYPE_F32, seed=801)


@pytest.mark.parametrize("heads,hd", [(1, 128), (2, 128), (4, 128), (8, 128), (1, 64), (2, 64), (4, 64), (8, 64)])
@pytest.mark.parametrize("length", [20, 490, 1000, 1990])
def test_record_counts(heads, hd, length):
    """each case grows by 256 tokens and passes the record counts 1-9, 16-24, 32-40, 63-64 and then 33-36 of twice the length"""
    shape = dataclasses.replace(SHAPE, n_q_heads=heads, head_dim=hd)
    check(run_job(shape, [length], 256, seed=802), f"merge {heads} heads of {hd}, {length} tokens on")
