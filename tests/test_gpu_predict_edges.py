"""Predictor scores bit for bit against the oracle where the kernels' tilings
end: every lane count of the fixed order (r 8 .. 1024, with one and two chunks
per lane), every chunk count of d, rows past d_ff, and batches that leave the
token tiles of 1, 2, 4 and 8 partly empty."""
import numpy as np
import pytest

import oracle
from helpers import say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,r,d_ff,batch", [
    (128, 8, 1, 1), (128, 16, 70, 3), (256, 24, 333, 2), (384, 48, 65, 5), (512, 64, 257, 9),
    (640, 136, 1000, 1), (1024, 256, 513, 8), (1536, 400, 300, 17), (2176, 512, 129, 4),
    (5120, 1024, 200, 1), (5120, 256, 300, 2), (4224, 64, 100, 2), (6144, 520, 90, 2), (8192, 512, 1030, 32), (16384, 1000, 100, 3)])
def test_scores_at_tile_edges(d, r, d_ff, batch):
    from paper_2410_14740_amd import m2c
    from paper_2410_14740_amd import workloads as W
    ld = W.make_layer(1000 + d + r, 0, d, d_ff, r, 1, rhos=(0.5,) * batch, zipf_bias=batch % 2 == 1)
    k = max(1, d_ff // 4)
    say(f"predict d={d} r={r} d_ff={d_ff} batch={batch}")
    L = m2c.Layer(m2c.make_desc(d, d_ff, r, k, 0, max_batch=batch), ld)
    x = torch.from_numpy(ld.x[0].view(np.uint16).copy()).cuda()
    s = torch.empty((batch, d_ff), dtype=torch.float32, device="cuda")
    tiers = torch.empty((batch, d_ff), dtype=torch.uint8, device="cuda")
    L.predict_rank(x, batch, k, k // 3, k // 3, s, tiers)
    torch.cuda.synchronize()
    got = s.cpu().numpy()
    for b in range(batch):
        want = oracle.predict(ld.pred_a, ld.pred_b, ld.bias, ld.x[0, b])[1]
        assert np.array_equal(got[b].view(np.uint32), want.view(np.uint32)), f"row {b}"
    L.close()
