"""Top-k select and tiers on chosen scores, against the oracle. A layer with
zero predictor matrices scores every neuron by its bias, so any scores can be
given to m2c_predict_rank: the equal-width bins, their candidate lists and
the radix path that takes over where the bins do not suit the scores."""
import numpy as np
import pytest

import oracle
from helpers import say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def scores_of(kind, n, rng):
    s = rng.standard_normal(n).astype(np.float32)
    if kind == "ties":  # a few hundred distinct values: ties inside and across the boundaries
        s = np.round(s * 40).astype(np.float32) / 40
    elif kind == "zeros":  # half the scores tie at +0 / -0
        s[rng.permutation(n)[: n // 2]] = 0.0
        s[rng.permutation(n)[: n // 8]] = -0.0
    elif kind == "outlier":  # all but one neuron in a few bins
        s[n // 2] = 1e30
    elif kind == "nonfinite":
        s[rng.permutation(n)[:6]] = [np.inf, -np.inf, np.nan, -np.nan, np.inf, 0.0][: min(6, n)]
    elif kind == "tiny":
        s *= np.float32(1e-38)
    elif kind == "equal":
        s[:] = -1.5
    elif kind == "crowded":  # one bin holds more neurons than a candidate list
        s = (1.0 + rng.random(n) * 1e-4).astype(np.float32)
        s[0], s[-1] = -1.0, 1.5
    elif kind == "halves":  # bins end where keys change sign
        s = np.where(rng.random(n) < 0.5, -1.0, 1.0).astype(np.float32) * rng.random(n, dtype=np.float32)
    return s


KINDS = ("normal", "ties", "zeros", "outlier", "nonfinite", "tiny", "equal", "crowded", "halves")


# d_ff in each register instance (1, 2, 4, 8, 12, .. 32, 40 scores per thread: both sides of the
# narrow ones' edges, the upper edge of the others), and above the widest (rows read again by each pass)
@pytest.mark.parametrize("d_ff", [1, 63, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 11008, 16384, 20480,
                                  24576, 28672, 28673, 32769, 40960, 40961, 70000])
def test_select_scores(d_ff):
    from paper_2410_14740_amd import m2c
    d, r = 128, 8
    z = np.zeros
    rng = np.random.default_rng(d_ff)
    w = z((d_ff, d), np.float16)
    x = torch.zeros((1, d), dtype=torch.float16, device="cuda")
    tiers = torch.empty((1, d_ff), dtype=torch.uint8, device="cuda")
    sc = torch.empty((1, d_ff), dtype=torch.float32, device="cuda")
    owner = None

    class D:
        pass

    for kind in KINDS:
        data = D()
        data.w_gate = data.w_up = w
        data.w_down = z((d, d_ff), np.float16)
        data.pred_a, data.pred_b = z((r, d), np.float16), z((d_ff, r), np.float16)
        data.bias = scores_of(kind, d_ff, rng)
        L = m2c.Layer(m2c.make_desc(d, d_ff, r, d_ff, 0, staging_slots=-1), data, weights_of=owner)
        owner = owner or L
        want_s = (np.float32(0) + data.bias).astype(np.float32)
        for k in sorted({0, 1, d_ff // 5, d_ff - 1, d_ff}):
            n16, n8 = k // 10, (2 * k) // 5
            say(f"select d_ff={d_ff} {kind} k={k}")
            L.predict_rank(x, 1, k, n16, n8, sc, tiers)
            torch.cuda.synchronize()
            got_s = sc.cpu().numpy()[0]
            assert np.array_equal(got_s.view(np.uint32)[~np.isnan(want_s)],
                                  want_s.view(np.uint32)[~np.isnan(want_s)])
            tm, _ = oracle.select_tiers(got_s, k, n16, n8)
            assert np.array_equal(tiers.cpu().numpy()[0], tm), (kind, k)
        if L is not owner:
            L.close()
    owner.close()
