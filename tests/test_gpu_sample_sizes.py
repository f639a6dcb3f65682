"""GPU: the sampling kernels at the sizes where their paths meet: one workgroup per row up to 8192 tokens, chunks beyond;
rows whose decisive bin holds more elements than the lists (flat rows, ties over the whole row); masked tokens.  Checked
against the fp64 oracle: the token is a nucleus member, the draw falls into its interval of the running mass, and the
scratch buffer holds the probabilities up to one factor per row.  Bound: a probability is 2^a with a = (x - max) *
log2(e) / T, whatever the size of the scores themselves; the difference, the factor and the product are each rounded to fp32, so a
is off by at most 3 * 2^-24 * |a| and 2^a by 1.3e-7 * |a| of itself: at most 7e-8 of the largest probability, and less than
6e-6 for a sum of members down to 2^-44 (scores far outside the ones here: test_gpu_sample_edges.py)."""
import numpy as np
import pytest

from oracle import sample as S
from paper_2603_20661_amd import synth

pytestmark = pytest.mark.gpu


def run(lg, temperature, top_p, u):
    import torch
    from paper_2603_20661_amd import binding as B
    dev = torch.device("cuda:0")
    lg_dev, u_dev = torch.from_numpy(lg).to(dev), torch.from_numpy(u).to(dev)
    scratch = torch.full(lg.shape, float("nan"), dtype=torch.float32, device=dev)
    tok = torch.full((lg.shape[0],), -1, dtype=torch.int32, device=dev)
    B.www_sample_top_p(lg_dev, temperature, top_p, u_dev, scratch, tok)
    torch.cuda.synchronize()
    return tok.cpu().numpy(), scratch.cpu().numpy()


@pytest.mark.parametrize("vocab", [1, 7, 63, 1023, 8191, 8192, 8193, 12289, 16384, 16385, 100003])
@pytest.mark.parametrize("std,temperature,top_p", [(3.0, 1.0, 0.9), (0.02, 1.0, 0.7), (10.0, 0.6, 1.0)])
def test_sizes_where_the_paths_meet(vocab, std, temperature, top_p):
    batch = 5
    lg = synth.normal_f32(83, vocab, batch * vocab, std=std).reshape(batch, vocab).copy()
    lg[1, :] = 0.25                              # one value everywhere
    if vocab > 8:
        lg[2, 1::2] = -np.inf                    # masked tokens
        lg[3, vocab - 2] = lg[3].max() + 30.0    # one certain token, in the last place but one
    u = np.array([0.0, 0.37, 0.62, 0.999, 1.0 - 2.0 ** -24], np.float32)
    print(f"vocab {vocab} std {std}", flush=True)
    tok, e_gpu = run(lg, temperature, top_p, u)
    for b in range(batch):
        want, e, mask, cum, target = S.sample(lg[b], temperature, top_p, float(u[b]))
        t = int(tok[b])
        assert 0 <= t < vocab
        assert e[t] >= e[mask].min() * (1 - 1e-5), f"row {b}: token {t} outside the nucleus (oracle's {want})"
        before, eps = cum[t] - (e[t] if mask[t] else 0.0), 1e-5 * cum[-1]
        assert before - eps <= target <= cum[t] + eps, f"row {b}: token {t}, oracle's {want}"
        ratio = e_gpu[b].astype(np.float64) / e_gpu[b].max()
        assert np.abs(ratio - e).max() <= 1e-5, f"row {b}: scratch is not the unnormalised probabilities"
    if vocab > 8:
        assert tok[3] == vocab - 2
        assert tok[2] % 2 == 0


def test_rows_without_a_finite_logit():
    for vocab in (100, 20000):
        lg = np.full((2, vocab), -np.inf, np.float32)
        tok, _ = run(lg, 1.0, 0.9, np.array([0.0, 0.9], np.float32))
        assert tok.tolist() == [0, 0]
