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


def edges(batch, vocab):
    """tokens in front of which a chunk, a run of tokens or a chunk's reserved head ends, by the launch rule of sample.hip"""
    shorter = -(-vocab // 8192)
    n_chunks = min(shorter if batch * shorter <= 256 else -(-vocab // 16384), 64)
    chunk = -(-vocab // n_chunks)
    length = -(-(-(-chunk // 256)) // (1024 // n_chunks)) * 256
    starts = sorted({0, chunk, (n_chunks // 2) * chunk, (n_chunks - 1) * chunk})
    at = {s + d for s in starts for d in (0, length, 2 * length, 4096, chunk // length * length)}
    return n_chunks, chunk, length, sorted(e for e in at if 0 < e < vocab)


SIZES = [(4, 8193), (5, 16383), (4, 262145), (4, 300001), (90, 16385), (130, 16384), (70, 32769)]


@pytest.mark.parametrize("batch,vocab", SIZES)
def test_tokens_on_either_side_of_an_edge(batch, vocab):
    """two equal tokens that are the nucleus, one behind each edge of chunks, runs and reserved heads and one in front of it, and the row's first and last"""
    n_chunks, chunk, length, at = edges(batch, vocab)
    assert (n_chunks, chunk, length) == {8193: (2, 4097, 256), 16383: (2, 8192, 256), 262145: (33, 7944, 512), 300001: (37, 8109, 512), 16385: (2, 8193, 256),
                                         16384: (1, 16384, 256), 32769: (3, 10923, 256)}[vocab]
    pairs = [(0, vocab - 1), *((e - 1, e) for e in at)]
    pairs += [pairs[0]] * (-len(pairs) % batch)
    for first in range(0, len(pairs), batch):
        some = pairs[first:first + batch]
        lg = synth.normal_f32(93, vocab + first, batch * vocab, std=3.0).reshape(batch, vocab).copy()
        for row, pair in zip(lg, some):
            row[list(pair)] = 60.0
        for side in (0, 1):
            print(f"batch {batch} vocab {vocab} {some[0]} .. {some[-1]}", flush=True)
            tok, _ = run(lg, 1.0, 0.9, np.full(batch, 0.25 + 0.5 * side, np.float32))
            assert tok.tolist() == [pair[side] for pair in some]


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
