"""GPU: the plan of the decode attention where its cut points change: chunks of one key pair, a longest sequence of 64
and 65 pairs (one and two pairs a chunk), and chunks that begin in one sequence and end in another.  Bounds of the parity
tests (the cuts only move the rounding of partial softmax sums)."""
import pytest

from paper_2603_20661_amd import synth
from test_gpu_parity import check, run_job

pytestmark = pytest.mark.gpu


def shape(hd, group, n_kv):
    return synth.ModelShape(f"plan{hd}g{group}", 1, 128, n_kv * group, n_kv, hd, 176, 512, 1e-5, 1e4, synth.WDTYPE_BF16, seed=300 + hd + group)


@pytest.mark.parametrize("hd,group,n_kv,lens", [
    (64, 2, 1, [1930]),              # 61 .. 69 pairs in the steps: one pair a chunk, then two
    (128, 1, 1, [1, 2030]),          # the short sequence ends inside the first chunk once there are two pairs in it
    (64, 8, 2, [4000, 31, 32, 33]),  # at least two pairs a chunk throughout
])
def test_cut_points(hd, group, n_kv, lens):
    check(run_job(shape(hd, group, n_kv), lens, 3, seed=90 + hd), f"plan {hd} {lens}")


@pytest.mark.parametrize("length", [32760, 40000])
def test_contexts_beyond_64_chunks(length):
    """A long sequence alone (16 pairs a chunk; at 40 000 tokens more than 64 chunks) and beside others that move its cut
    points (21 and 23 pairs a chunk with 1024 wavefronts), on the same cache.  Each cut rescales one fp32 softmax state (2^-24 relative): some 90 cuts move a
    logit of up to 6 by at most 4e-5."""
    import numpy as np
    from helpers import GpuSession
    s = shape(64, 8, 8)
    lens = np.array([length, 33, 33000, 20000], np.int32)
    cap = lens + 2
    blocks = (cap + 15) // 16
    sess = GpuSession(s, synth.make_blob(s, std=0.1, gain_std=0.1), 4, int(blocks.max()) * 16, int(lens.max()), int(blocks.sum()) + 3)
    table = synth.block_tables(7, cap, int(blocks.sum()) + 3, int(blocks.max()), permute=True)
    try:
        for b in range(4):
            sess.prefill(synth.tokens(8 + b, int(lens[b]), s.vocab), lens[b:b + 1], lens[b:b + 1], table[b:b + 1])
        tok = synth.tokens(13, 4, s.vocab)
        alone, _ = sess.decode(tok[:1], lens[:1] + 1, table[:1])
        beside, _ = sess.decode(tok, lens + 1, table)
    finally:
        sess.close()
    err = float(np.abs(alone[0] - beside[0]).max())
    print(f"{length}: max|dlogit|={err:.2e} of {np.abs(alone[0]).max():.1f}", flush=True)
    assert np.isfinite(beside).all() and 0.5 < np.abs(alone[0]).max() < 6.0
    assert err <= 4e-5
