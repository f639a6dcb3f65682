"""GPU: the prefill GEMM's smaller tiles (128 rows x 128 or 256 tokens, k range split over workgroups) at their edges: one
token, the borders of a group of 32, of a tile and of two tiles, wavefronts without tokens, an odd number of k blocks
(ffn_dim 352: 11), a last row tile that is not full, and calls in which some GEMMs of a layer take these tiles and others
do not.  Bounds of the parity tests."""
import dataclasses

import pytest

from paper_2603_20661_amd import synth
from test_gpu_parity import check, run_job

pytestmark = pytest.mark.gpu

ODD = synth.ModelShape("oddk", 2, 256, 6, 3, 64, 352, 512, 1e-5, 1e4, synth.WDTYPE_BF16, seed=401)
DEEP = synth.ModelShape("deepk", 2, 384, 4, 1, 128, 4112, 512, 1e-5, 1e4, synth.WDTYPE_BF16, seed=402)   # 129 k blocks: splits
DEEP_QKN = dataclasses.replace(DEEP, name="deepkqkn", qk_norm=1, seed=403)


@pytest.mark.parametrize("shape", [ODD, DEEP, DEEP_QKN], ids=lambda s: s.name)
@pytest.mark.parametrize("lens", [[1], [31, 1], [33], [127], [128, 1], [255, 2], [513], [200, 900]], ids=str)
def test_edges(shape, lens):
    check(run_job(shape, lens, 1, seed=sum(lens)), f"{shape.name} {lens}")


@pytest.mark.parametrize("hd,group", [(64, 1), (64, 2), (64, 8), (128, 1), (128, 2), (128, 4), (128, 8)])
@pytest.mark.parametrize("lens,chunk", [([700, 3, 129], 40), ([1100, 260], 130)], ids=str)
def test_key_ranges_of_the_attention(hd, group, lens, chunk):
    """chunks over a cached prefix in calls of few tiles: the keys of a tile are cut into ranges, the last of them with
    queries that see none of its keys or only part of its first pair"""
    n_kv = 2 if group <= 4 else 1
    shape = synth.ModelShape(f"rng{hd}g{group}", 2, 256, n_kv * group, n_kv, hd, 352, 512, 1e-5, 1e4, synth.WDTYPE_BF16, seed=420 + hd + group)
    check(run_job(shape, lens, 1, seed=430 + group, chunk=chunk), f"{shape.name} {lens} chunk {chunk}")
