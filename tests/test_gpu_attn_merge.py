"""GPU: the merge of a sequence's partial attention results, at the record counts where its loads, its rounds and its wavefronts' shares end
(2, 4 and 8 loads of two or four records; 16, 32 and 64 records), for every number of query heads per kv head.  Bounds of the parity tests."""
import dataclasses

import numpy as np
import pytest

from helpers import GpuSession
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


@pytest.mark.parametrize("hd", [64, 128])
def test_the_order_of_the_sums_depends_on_the_number_of_records_alone(hd):
    """equal query heads: each gets the same bits, however many share a kv head"""
    lengths, out = (40, 300, 700, 1070), {}                       # 2, 10, 22 and 34 records
    toks = synth.tokens(804, max(lengths), SHAPE.vocab)
    for heads in (1, 2, 4, 8):
        shape = dataclasses.replace(SHAPE, d_model=128, n_q_heads=heads, head_dim=hd, weight_dtype=synth.WDTYPE_BF16)   # (one chunk of k: never split)
        blob = synth.make_blob(dataclasses.replace(shape, n_q_heads=1), std=0.05, seed=803)
        entries, total = synth.blob_layout(shape)
        wide = np.zeros(total, np.uint8)
        for (name, off, rows, cols, _), (_, off1, rows1, cols1, _) in zip(entries, synth.blob_layout(dataclasses.replace(shape, n_q_heads=1))[0]):
            size = (rows1 * cols1) * (4 if name.endswith("norm") else 2)
            part = blob[off1:off1 + size].reshape(rows1, -1)
            if name.endswith("wqkv"):
                part = np.concatenate([part[:hd]] * heads + [part[hd:]])
            elif name.endswith("wo"):
                part = np.concatenate([part] * heads, axis=1)
            wide[off:off + part.size] = part.reshape(-1)
        from paper_2603_20661_amd import binding as B
        sess = GpuSession(shape, wide, 1, 1088, 16, 68)
        table = np.arange(68, dtype=np.int32)[None]
        try:
            for n, t in enumerate(toks, 1):
                sess.decode([t], [n], table)
                if n in lengths:
                    raw = B.www_debug_read(sess.model, 2, heads * hd * 16, stream=sess.stream).numpy().view(np.uint32)
                    units = raw.reshape(heads, hd // 32, 2, 64, 4)[:, :, :, ::16]                      # [head][32 columns][high, low][lanes of the one token]
                    assert (units == units[:1]).all() and units.any()
                    assert (out.setdefault(n, units[0]) == units[0]).all(), f"{heads} heads, {n} tokens"
        finally:
            sess.close()
