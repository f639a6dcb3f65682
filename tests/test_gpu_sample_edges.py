"""GPU: sampling where the scores leave the ordinary range: temperatures at which log2(e) * logit / T exceeds any table of
scores (nearly greedy draws), rows that lie far below zero (every token masked with a finite value).  Checked against the
fp64 oracle: the token is a nucleus member, the draw falls into its interval of the running mass, and the scratch buffer
holds the probabilities up to one factor per row.

Bound: a probability is 2^a with a = (x - max) * log2(e) / T; the difference, the factor and the product are each rounded to
fp32 (2^-24 relative), so a is off by at most 3 * 2^-24 * |a| and 2^a by 1.3e-7 * |a| of itself, which is at most 7e-8 of the
largest probability.  A running mass of members down to 2^-44 is then off by less than 6e-6 of the total; 1e-5 is allowed."""
import numpy as np
import pytest

from oracle import sample as S
from paper_2603_20661_amd import synth
from test_gpu_sample_sizes import run

pytestmark = pytest.mark.gpu

BOUND = 1e-5
ROW, CHUNKS = 1000, 20011      # a row of one workgroup, and one that is cut into chunks


def check(lg, temperature, top_p, u, run=run):
    T = float(np.float32(temperature))
    tok, e_gpu = run(lg, temperature, top_p, u)
    for b in range(len(lg)):
        want, e, mask, cum, target = S.sample(lg[b], T, top_p, float(u[b]))
        t = int(tok[b])
        assert 0 <= t < lg.shape[1]
        assert e[t] >= e[mask].min() * (1 - BOUND), f"row {b}: token {t} outside the nucleus (oracle's {want})"
        before, eps = cum[t] - (e[t] if mask[t] else 0.0), BOUND * cum[-1]
        assert before - eps <= target <= cum[t] + eps, f"row {b}: token {t}, oracle's {want}"
        ratio = e_gpu[b].astype(np.float64) / e_gpu[b].max()
        assert np.abs(ratio - e).max() <= BOUND, f"row {b}: scratch is not the unnormalised probabilities"
    return tok


U = np.array([0.0, 0.3, 0.6, 0.999], np.float32)


@pytest.mark.parametrize("vocab", [ROW, 8192, 8193, CHUNKS, 128256])
@pytest.mark.parametrize("temperature", [1e-3, 1e-6, 1e-7, 1e-8, 1e-20, 1e-39])
def test_low_temperatures(vocab, temperature):
    lg = synth.normal_f32(84, vocab, 4 * vocab, std=3.0).reshape(4, vocab).copy()
    lg[1] = np.abs(lg[1]) + 0.5                  # positive only
    lg[2] = -np.abs(lg[2]) - 0.5                 # negative only
    lg[3, [5, vocab - 3]] = lg[3].max() + 1.0    # two equal ones at the top
    tok = check(lg, temperature, 0.9, U)
    if temperature < 1e-6:
        assert [int(t) for t in tok[:3]] == [int(r.argmax()) for r in lg[:3]]
        assert tok[3] == vocab - 3


@pytest.mark.parametrize("vocab", [ROW, CHUNKS])
@pytest.mark.parametrize("value", [-1e8, -1e9, -3e38, np.finfo(np.float32).min], ids=str)
def test_rows_far_below_zero(vocab, value):
    """equal masked tokens: a uniform draw, as over any row of equal logits; and one token a little above the others"""
    lg = np.full((4, vocab), value, np.float32)
    lg[2, vocab - 2] *= np.float32(0.5)
    lg[3, ::3] = -np.inf
    tok = check(lg, 1.0, 0.9, U)
    assert tok[0] == 0 and tok[2] == vocab - 2
    assert abs(int(tok[1]) - 0.3 * vocab) <= 2


@pytest.mark.parametrize("vocab", [ROW, CHUNKS])
def test_infinite_and_unordered_logits(vocab):
    """+inf is the certain token (two of them: one of the two); a NaN is never drawn"""
    lg = synth.normal_f32(85, vocab, 4 * vocab, std=3.0).reshape(4, vocab).copy()
    lg[0, vocab - 5] = np.inf
    lg[1, [3, vocab - 5]] = np.inf
    lg[2, 1:] = np.nan
    lg[3, ::2] = np.nan
    tok, e = run(lg, 1.0, 0.9, np.array([0.999, 0.6, 0.5, 0.5], np.float32))
    assert tok[0] == vocab - 5 and tok[1] == vocab - 5 and tok[2] == 0 and tok[3] % 2 == 1
    assert not np.isnan(e).any()


@pytest.mark.parametrize("vocab", [1 << 19, (1 << 20) + 1, 1_800_000, 1 << 21, 9_000_001], ids=str)
def test_long_flat_rows(vocab):
    """every token near the largest: the masses of a row together are many times one token's.  The fp64 oracle's sums are
    exact for equal tokens; the other row's are off by no more than its probabilities are."""
    lg = np.zeros((3, vocab), np.float32)
    lg[1] = 0.25
    lg[2] = synth.normal_f32(86, vocab & 0xffff, vocab, std=1e-3)
    tok = check(lg, 1.0, 0.9, np.array([0.999, 0.37, 0.62], np.float32))
    assert abs(int(tok[0]) - 0.999 * vocab) <= 2e-5 * vocab


@pytest.mark.parametrize("vocab", [1, 63, ROW, 8192, 8193, CHUNKS, 128256])
@pytest.mark.parametrize("temperature,top_p", [(1.0, 0.9), (0.6, 1.0), (1e-8, 0.9)])
def test_probabilities_replace_the_logits(vocab, temperature, top_p):
    """the same buffer as logits and scratch"""
    import torch
    from paper_2603_20661_amd import binding as B
    lg = synth.normal_f32(87, vocab, 4 * vocab, std=3.0).reshape(4, vocab).copy()
    lg[1, :] = 0.25
    lg[2, 1::2] = -np.inf
    lg[3] *= 1e-3
    print(f"vocab {vocab} T {temperature}", flush=True)
    dev = torch.device("cuda:0")

    def in_place(lg, temperature, top_p, u):
        buf, tok = torch.from_numpy(lg).to(dev), torch.full((4,), -1, dtype=torch.int32, device=dev)
        B.www_sample_top_p(buf, temperature, top_p, torch.from_numpy(u).to(dev), buf, tok)
        torch.cuda.synchronize()
        return tok.cpu().numpy(), buf.cpu().numpy()

    check(lg, temperature, top_p, U, in_place)


def test_buffers_that_overlap_in_part_are_refused():
    import torch
    from paper_2603_20661_amd import binding as B
    dev = torch.device("cuda:0")
    buf = torch.zeros(3 * 64, dtype=torch.float32, device=dev)
    u, tok = torch.zeros(2, dtype=torch.float32, device=dev), torch.full((2,), -1, dtype=torch.int32, device=dev)
    for a, b in ((0, 64), (64, 0), (1, 0), (0, 1)):
        with pytest.raises(B.WwwError) as e:
            B.www_sample_top_p(buf[a:a + 128].view(2, 64), 1.0, 0.9, u, buf[b:b + 128].view(2, 64), tok)
        assert e.value.code == B.E_INVALID_ARG
    torch.cuda.synchronize()
    assert tok.cpu().tolist() == [-1, -1] and not buf.cpu().numpy().any()


@pytest.mark.parametrize("vocab", [2, ROW, CHUNKS])
def test_zeros_of_either_sign_are_equal(vocab):
    """equal probabilities enter the nucleus together, whatever the sign of the zero they come from"""
    lg = np.full((4, vocab), -1.0, np.float32)
    lg[:, :2] = [0.0, -0.0]
    lg[1, :2] = lg[2, :2] = [-0.0, 0.0]
    tok = check(lg, 0.02, 0.5, np.array([0.9, 0.9, 0.2, 0.2], np.float32))
    assert tok.tolist() == [1, 1, 0, 0]


@pytest.mark.parametrize("vocab", [ROW, 8192, CHUNKS])
def test_infinite_temperature(vocab):
    """all tokens equally probable, so all in the nucleus, whatever their logits"""
    lg = synth.normal_f32(88, vocab, 4 * vocab, std=3.0).reshape(4, vocab)
    tok, _ = run(lg, float("inf"), 0.5, U)
    assert tok.tolist() == [int(np.float64(u) * vocab) for u in U]


@pytest.mark.parametrize("vocab", [8192, 8193, 24577])
def test_members_of_the_decisive_bin_in_some_chunks_only(vocab):
    """more members than a chunk's list holds in the first chunk, few, none or equal ones in the others"""
    lg = synth.normal_f32(89, vocab, 4 * vocab, std=0.5).reshape(4, vocab) - 8.0
    lg[:, :3000] = 0.01 * synth.normal_f32(90, vocab, 4 * 3000).reshape(4, 3000)
    lg[1, 5000:5300] = lg[1, 17]
    lg[2, 4500:] = -np.inf
    lg[3, :3000] = 0.125
    for u in (0.01, 0.5, 0.999):
        check(lg, 1.0, 0.6, np.full(4, u, np.float32))


def scores_in_bins(logit, temperature):
    """the kernels' scores, in eighths of an octave: fp32, as in sample.hip"""
    c = np.float32(1.4426950408889634) / np.float32(temperature)
    return np.float32(logit) * (c * np.float32(8))


@pytest.mark.parametrize("vocab", [512, CHUNKS])
def test_the_bin_where_floats_stop_being_halves(vocab):
    """scores of -2^23 and half above it share a bin, the one that decides: five members, not nine"""
    values = np.array([-508772.0, -508772.21875, -508772.25], np.float32)
    assert scores_in_bins(values[1:], 0.7).tolist() == [-8388607.5, -8388608.0]
    lg = np.full((4, vocab), -600000.0, np.float32)
    lg[:, 7] = values[0]
    lg[:, [9, 100, 300, 400]] = values[1]
    lg[:2, vocab - 4:] = values[2]
    lg[2:, [1, 8, 101, vocab - 5]] = values[2]
    tok = check(lg, 0.7, 0.5295, U)
    assert set(tok.tolist()) <= {7, 9, 100, 300, 400}


@pytest.mark.parametrize("vocab", [8192, CHUNKS])
@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_the_lowest_bin_where_no_float_is_its_number(vocab, sign):
    """Beyond 2^24 the bin 255 below the largest has an odd number.  It holds the last 1300 tokens; 1500 lie in the bin above it, the others higher
    still.  A token of the lowest bin is 2^-32 of the largest, so that the last 2^-24 of the whole mass are some 250 of them."""
    line = np.float32(sign * 1.4e6) + np.arange(-600, 600, dtype=np.float32) * np.float32(0.125)
    t = scores_in_bins(line, 0.7).astype(np.int64)
    assert (np.abs(t) > 1 << 24).all() and (np.abs(t) < 1 << 25).all() and (t % 2 == 0).all()
    at = {int(v): x for v, x in zip(t, line)}
    top = max(v for v in at if v % 4 == 2 and {v - 252, v - 254, v - 256} <= set(at))
    lg = np.full((1, vocab), at[top - 252], np.float32)
    lg[0, 1:vocab - 1300:(vocab - 1300) // 1500] = at[top - 254]
    lg[0, vocab - 1300:] = at[top - 256]
    lg[0, 0] = at[top]
    tok, _ = run(lg, 0.7, 1.0, np.array([1.0 - 2.0 ** -24], np.float32))
    _, e, mask, cum, target = S.sample(lg[0], float(np.float32(0.7)), 1.0, 1.0 - 2.0 ** -24)
    # masses are whole multiples of 2^-44 of up to twice the largest, each off by up to one of its 2048 at least and, as derived above, by
    # 32 * 1.3e-7: 5e-4 of what follows the largest
    rest = cum[-1] - cum[0]
    assert mask.all() and cum[tok[0] - 1] - 5e-4 * rest <= target <= cum[tok[0]] + 5e-4 * rest
    assert tok[0] >= vocab - 300
