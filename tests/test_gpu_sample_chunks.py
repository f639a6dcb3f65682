"""GPU: sampling of rows that are cut into chunks, at the edges of the chunks and of the runs of tokens inside them, with few rows (chunks of up to
8192 tokens) and with more than a round of workgroups (up to 16 384), and with rows whose decisive bin does not fit the lists.  Against the fp64
oracle, with the bound derived in test_gpu_sample_edges.py."""
import numpy as np
import pytest

from oracle import sample as S
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


@pytest.mark.parametrize("batch,vocab,top_p,std", [(4, 128256, 0.9, 0.4), (40, 128256, 0.9, 0.4), (4, 128256, 0.8, 0.8), (40, 128256, 0.9, 1.0), (4, 262144, 0.9, 1.0),
                                                   (4, 1 << 20, 0.9, 0.8)])
def test_members_that_only_the_chunks_lists_hold(batch, vocab, top_p, std):
    """more members of the decisive bin than the row's list holds (4096), in every chunk no more than its own does"""
    lg = synth.normal_f32(92, vocab & 0xffff, 4 * vocab, std=std).reshape(4, vocab).copy()
    lg[1] = np.round(lg[1] * 64) / 64                                # many equal ones
    lg[2][(lg[2] > 0.1) & (lg[2] < 2)] = 0.5                          # members all equal, or none of them above the bin
    lg[2, ::3] = lg[0, ::3]
    z = np.float32(1.4426950408889634) * np.float32(8)
    for b in (0, 1):
        e, mask, tau = S.nucleus_fast(lg[b], 1.0, top_p)
        n = np.add.reduceat(np.floor(lg[b] * z) == np.floor(lg[b][e == tau][0] * z), np.arange(0, vocab, 8016))
        assert 4096 < n.sum() and n.max() < 1600 / (2 if batch > 16 else 1)
    print(f"batch {batch} vocab {vocab}", flush=True)
    wide = np.tile(lg, (batch // 4, 1))
    u = np.linspace(0.0, 0.999, batch).astype(np.float32)
    keep = [0, 1, 2, 3, batch - 4, batch - 3, batch - 2, batch - 1]

    def some(lg_all, temperature, top_p, u_all):
        tok, e = run(wide, temperature, top_p, u)
        return tok[keep], e[keep]

    check(wide[keep], 1.0, top_p, u[keep], some)
