"""GPU: prefill calls whose last positions ride along as rows of the GEMMs (hi and lo parts in one group of 32 columns): one to
several such groups, full and nearly empty ones, token counts around a group and a tile, chunks over a cached prefix, every weight
format that rides, both tile kernels and k splits.  Which calls ride, and in which tiles, follows from the sizes by rules on the
host; every test asks them and fails where a changed rule has moved it elsewhere.  The cache entries of the last positions are
checked by the decode steps behind.  Bounds of the parity tests."""
import dataclasses

import numpy as np
import pytest

from helpers import compare
from paper_2603_20661_amd import synth
from test_gpu_parity import WIDE8B, check, run_job

pytestmark = pytest.mark.gpu

H64 = synth.ModelShape("last64", 3, 256, 6, 3, 64, 352, 512, 1e-5, 1e4, synth.WDTYPE_BF16, seed=601)
H128 = synth.ModelShape("last128", 2, 384, 4, 1, 128, 4112, 512, 1e-5, 1e4, synth.WDTYPE_BF16, seed=602)   # k splits
FORMATS = [H64, H128, dataclasses.replace(H64, name="last64qk", qk_norm=1, seed=603), dataclasses.replace(H128, name="last128qk", qk_norm=1, seed=604),
           dataclasses.replace(H128, name="last128fp8", weight_dtype=synth.WDTYPE_FP8WO, seed=605),
           dataclasses.replace(H64, name="last64int4", ffn_dim=384, weight_dtype=synth.WDTYPE_INT4WO_32, seed=606)]


def route(shape, gemm, batch, total):
    """(kernel, tokens per tile, rows per tile, k splits, last positions ride) of a GEMM of a call"""
    from paper_2603_20661_amd import binding as B
    return B.www_debug_route(B.make_config(shape, batch, 64, total, 4096), gemm, batch, total)


def check_scaled(res, what):
    """Bounds for narrow models, whose greedy tokens say little: their logits (standard deviation 0.3 over 512 tokens) have their
    two best within 1e-3 in about 1 % of the rows, and one case agreed in 98.8 % (in 98.8 % as well with tiles of 256 tokens
    alone).  So the error is bounded against the logits' size: operands rounded to 11 bits leave a standard error of about
    2^-11.5 of it after the seven products of two layers, and the largest of 130 000 logits lies at 4.5 of those, 1.6e-3;
    five times that for shapes whose errors add up instead.  A misplaced row is off by the logits' size.  Where the oracle's two
    best are further apart than two such errors the tokens are the same.  That is expected in 0.945 of the rows (the gap of 512
    normal logits is about exponential, with a mean of 0.28 standard deviations), a property of the oracle alone; greedy sequences run into
    cycles, so a case of two may hold as few as five different rows, whose share has a standard deviation of 0.10."""
    o_logits, o_tok, g_logits, g_tok = res
    err, agree, _ = compare(*res)
    size = float(o_logits.std())
    bound = 8e-3 * size
    top2 = np.sort(o_logits, axis=-1)[..., -2:]
    clear = top2[..., 1] - top2[..., 0] > 2 * bound
    print(f"{what}: max|dlogit|={err:.3e} of logits {size:.2f} agreement={agree:.4f} clear rows {clear.mean():.3f}", flush=True)
    assert err <= bound
    assert clear.mean() >= 0.945 - 3 * 0.10 and (o_tok == g_tok)[clear].all()


@pytest.mark.parametrize("batch,total", [(1, 1), (1, 32), (3, 97), (16, 16), (17, 160), (33, 250), (70, 300)], ids=str)
@pytest.mark.parametrize("shape", FORMATS, ids=lambda s: s.name)
def test_groups_of_last_positions(shape, batch, total):
    assert all(route(shape, g, batch, total)[4] for g in ("qkv", "o", "gate_up", "down"))
    lens = [total // batch + (i < total % batch) for i in range(batch)]
    check(run_job(shape, lens, 2, seed=610 + batch + total), f"{shape.name} {batch} sequences, {total} tokens")


@pytest.mark.parametrize("shape", FORMATS[:4], ids=lambda s: s.name)
def test_chunks_over_a_prefix(shape):
    """every chunk's last position rides, the cache entry it leaves is read by the next chunk"""
    for batch, total in ((4, 97), (3, 65), (2, 64), (1, 32), (1, 22)):
        assert route(shape, "qkv", batch, total)[4]
    check(run_job(shape, [150, 33, 1, 96], 2, seed=640, chunk=32), f"{shape.name} chunks of 32")


@pytest.mark.parametrize("lens,gate_up", [([200], ("prefill_small", 256)), ([100, 60, 64], ("prefill_small", 256)), ([300, 2], ("prefill", 192)),
                                          ([310, 140], ("prefill", 256))], ids=str)
def test_large_tiles(lens, gate_up):
    """full-width matrices: the gate/up product takes the largest tiles, the others the smaller ones, with split k ranges"""
    shape = dataclasses.replace(WIDE8B, n_layers=2)
    assert route(shape, "gate_up", len(lens), sum(lens)) == (*gate_up, 128 if gate_up[0] == "prefill_small" else 256, 1, True)
    assert all(route(shape, g, len(lens), sum(lens))[0] == "prefill_small" and route(shape, g, len(lens), sum(lens))[3] > 1 for g in ("o", "down"))
    check(run_job(shape, lens, 1, seed=650 + len(lens)), f"{WIDE8B.name} {lens}")


# products of 8192 rows, for which 192 tokens per tile fill the chip in one round: the residual ones, and the QKV product
NARROW = synth.ModelShape("narrow8192", 2, 8192, 2, 1, 64, 352, 512, 1e-5, 1e4, synth.WDTYPE_BF16, seed=607)
NARROW_QKV = synth.ModelShape("narrowqkv64", 2, 256, 64, 32, 64, 352, 512, 1e-5, 1e4, synth.WDTYPE_BF16, seed=608)
NARROW_QKV128 = dataclasses.replace(NARROW_QKV, name="narrowqkv128", n_q_heads=32, n_kv_heads=16, head_dim=128, qk_norm=1, seed=609)


@pytest.mark.parametrize("lens", [[700, 400], [450, 600, 83]], ids=str)
@pytest.mark.parametrize("shape", [NARROW, NARROW_QKV, NARROW_QKV128, dataclasses.replace(NARROW_QKV, name="narrowf32", weight_dtype=synth.WDTYPE_F32)],
                         ids=lambda s: s.name)
def test_tiles_of_192_tokens(shape, lens):
    """whole tiles, and a last one that the last positions share with tokens; groups of 32 on both sides of the residual stream's
    256-token blocks; fp32 weights: the same tiles without last positions"""
    for g in ("o", "down") if shape is NARROW else ("qkv",):
        assert route(shape, g, len(lens), sum(lens)) == ("prefill", 192, 256, 1, shape.weight_dtype != synth.WDTYPE_F32)
    res = run_job(shape, lens, 1, seed=660 + len(lens))
    return check(res, f"{shape.name} {lens}") if shape is NARROW else check_scaled(res, f"{shape.name} {lens}")


# One product with rows for the large tiles in each of these, the others narrow, so that every kernel and tile of the prefill GEMMs
# has a small case: plain and normalised heads, calls that ride, calls of several layers that keep the decode pass, and fp32 weights
# (which never ride).
WIDE_QKV = synth.ModelShape("wideqkv", 2, 256, 64, 64, 128, 352, 512, 1e-5, 1e4, synth.WDTYPE_BF16, seed=621)
WIDE_QKV_QKN = dataclasses.replace(WIDE_QKV, name="wideqkvqk", qk_norm=1, seed=622)
WIDE_RESID = synth.ModelShape("wideresid", 2, 8192, 2, 1, 64, 352, 512, 1e-5, 1e4, synth.WDTYPE_BF16, seed=623)
WIDE_RESID4 = synth.ModelShape("wideresid4", 2, 4096, 4, 1, 64, 1408, 512, 1e-5, 1e4, synth.WDTYPE_BF16, seed=624)
WIDE_GATE = synth.ModelShape("widegate", 2, 256, 4, 2, 64, 8192, 512, 1e-5, 1e4, synth.WDTYPE_BF16, seed=625)


def _f32(shape):
    return dataclasses.replace(shape, name=shape.name + "f32", weight_dtype=synth.WDTYPE_F32)


ROUTES = [(s, "qkv", *c) for s in (WIDE_QKV, WIDE_QKV_QKN) for c in ((33, 66, "prefill_small", 256, True), (33, 170, "prefill", 192, True),
                                                                      (33, 300, "prefill", 256, True), (2, 2048, "prefill", 256, False))]
ROUTES += [(_f32(s), "qkv", *c) for s in (WIDE_QKV, WIDE_QKV_QKN) for c in ((2, 100, "prefill_small", 128, False), (2, 131, "prefill_small", 256, False),
                                                                            (2, 261, "prefill", 192, False), (2, 391, "prefill", 256, False))]
ROUTES += [(WIDE_GATE, "gate_up", *c) for c in ((33, 170, "prefill_small", 256, True), (33, 417, "prefill", 192, True), (33, 677, "prefill", 256, True),
                                                (2, 3072, "prefill", 256, False))]
ROUTES += [(_f32(WIDE_GATE), "gate_up", *c) for c in ((2, 100, "prefill_small", 128, False), (2, 261, "prefill_small", 256, False),
                                                      (2, 513, "prefill", 192, False), (2, 769, "prefill", 256, False))]
ROUTES += [(WIDE_RESID, "down", *c) for c in ((33, 417, "prefill_small", 256, True), (33, 1024, "prefill", 192, True), (33, 1500, "prefill", 256, True),
                                              (16, 2048, "prefill", 256, False))]
ROUTES += [(WIDE_RESID4, "down", 2, 1408, "prefill_small", 256, False), (_f32(WIDE_RESID), "down", 2, 1025, "prefill", 192, False)]


@pytest.mark.parametrize("shape,gemm,batch,total,kernel,tokens,rides", ROUTES, ids=lambda v: getattr(v, "name", str(v)))
def test_every_kernel_and_tile(shape, gemm, batch, total, kernel, tokens, rides):
    got = route(shape, gemm, batch, total)
    assert (got[0], got[1], got[4]) == (kernel, tokens, rides)
    lens = [total // batch + (i < total % batch) for i in range(batch)]
    lens[0], lens[-1] = lens[0] - lens[-1] // 2, lens[-1] + lens[-1] // 2     # not all of one length
    # Weights of standard deviation 0.32 / sqrt(d_model) everywhere: queries and keys then have the size that 256 columns give them with
    # 0.02.  (With 0.02 the scores of 8192 columns reach 26 and attention nearly picks one key, which turns the rounding of
    # a cached key into 1.6 % of the logits in one row of 264, with or without riding.)
    check_scaled(run_job(shape, lens, 1, seed=670 + total, std=0.32 / shape.d_model ** 0.5), f"{shape.name} {batch} sequences, {total} tokens")
