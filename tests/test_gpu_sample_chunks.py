"""GPU: sampling of rows that are cut into chunks, at the edges of the chunks and of the runs of tokens inside them, with few rows (chunks of up to
8192 tokens) and with more than a round of workgroups (up to 16 384), and with rows whose decisive bin does not fit the lists.  Against the fp64
oracle, with the bound derived in test_gpu_sample_edges.py."""
import numpy as np
import pytest

from paper_2603_20661_amd import synth
from test_gpu_sample_edges import check
from test_gpu_sample_sizes import run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,vocab", [(4, 8193), (5, 16383), (4, 262145), (4, 300001), (90, 16385), (130, 16384), (70, 32769)])
@pytest.mark.parametrize("std", [3.0, 0.05])
def test_chunks_and_runs(batch, vocab, std):
    lg = synth.normal_f32(91, vocab, batch * vocab, std=std).reshape(batch, vocab).copy()
    for k, at in enumerate((0, 255, 256, vocab // 2 - 1, vocab // 2, vocab - 1)):    # certain tokens at the ends of runs and chunks
        if k + 4 < batch:
            lg[k + 4, at] = 60.0
    u = np.linspace(0.0, 0.999, batch).astype(np.float32)
    print(f"batch {batch} vocab {vocab} std {std}", flush=True)
    keep = sorted({*range(min(batch, 12)), batch - 2, batch - 1})                     # rows that the oracle looks at

    def some(lg_all, temperature, top_p, u_all):
        tok, e = run(lg, temperature, top_p, u)
        return tok[keep], e[keep]

    tok = check(lg[keep], 1.0, 0.9, u[keep], some)
    for k, at in enumerate((0, 255, 256, vocab // 2 - 1, vocab // 2, vocab - 1)):
        if k + 4 < batch:
            assert tok[keep.index(k + 4)] == at
