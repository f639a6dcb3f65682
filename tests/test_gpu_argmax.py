"""GPU: the greedy token where many logits are equal, in every kernel with an output head: the lowest index of the largest logit, over row
groups, wavefronts, workgroups and rows that do not fill a workgroup."""
import dataclasses

import numpy as np
import pytest

from helpers import GpuSession
from paper_2603_20661_amd import synth

pytestmark = pytest.mark.gpu

SHAPE = synth.ModelShape("argmax", 1, 256, 4, 1, 64, 272, 2064, 1e-5, 1e4, synth.WDTYPE_BF16, seed=701)
INT4 = dataclasses.replace(SHAPE, name="int4", weight_dtype=synth.WDTYPE_INT4WO_128, ffn_dim=384)
CASES = [(SHAPE, b) for b in (1, 17, 33, 100)] + [(INT4, 3), (INT4, 16), (INT4, 40), (dataclasses.replace(INT4, name="int4wide", vocab=33040), 9),
         (dataclasses.replace(SHAPE, name="f32", weight_dtype=synth.WDTYPE_F32), 4), (dataclasses.replace(SHAPE, name="fp8", weight_dtype=synth.WDTYPE_FP8WO), 8),
         (dataclasses.replace(SHAPE, name="wide", vocab=66064), 5), (dataclasses.replace(SHAPE, name="wide", vocab=66064), 128)]


@pytest.mark.parametrize("shape,batch", CASES, ids=lambda v: getattr(v, "name", str(v)))
@pytest.mark.parametrize("period", [24, 616])
def test_equal_logits(shape, batch, period):
    """row n of the output head is row 7 + n % period, and rows 0 to 6 are zero: the largest logit occurs in many workgroups"""
    blob = synth.make_blob(shape, std=0.05)
    for name, off, rows, cols, dt in synth.blob_layout(shape)[0]:
        if name not in ("lm_head", "lm_head.scale") or rows != shape.vocab:   # (the one scale of an FP8 matrix stays)
            continue
        row_bits = cols * {synth.WDTYPE_F32: 32, synth.WDTYPE_BF16: 16, synth.WDTYPE_FP8WO: 8, synth.WDTYPE_INT4WO_128: 4}[dt]
        m = blob[off:off + rows * row_bits // 8].reshape(rows, -1)
        m[7:] = m[7 + np.arange(rows - 7) % period]
        m[:7] = 0
    lens = 1 + np.arange(batch, dtype=np.int32) % 3
    table = np.arange(batch, dtype=np.int32)[:, None]
    sess = GpuSession(shape, blob, batch, 16, int(lens.sum()), batch)
    try:
        logits, tok = sess.prefill(synth.tokens(3, int(lens.sum()), shape.vocab), lens, lens, table)
        steps = [(logits, tok)]
        for s in range(2):
            steps.append(sess.decode(synth.tokens(4 + s, batch, shape.vocab), lens + 1 + s, table))
    finally:
        sess.close()
    for logits, tok in steps:
        assert np.all((logits == logits.max(-1, keepdims=True)).sum(-1) >= (shape.vocab - 7) // period)
        assert np.array_equal(tok, logits.argmax(-1))
