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
