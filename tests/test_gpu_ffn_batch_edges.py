"""Batched FFN where its tiles and steps end: tiers of 0, 1, 8, 16, 31, 32, 33
... items, quantization group counts that are no multiple of 16, one row tile
and two, wide gate/up tiles, and rows of very different magnitude (the wave's exponent of the down
kernel moves between steps), against the oracle. The tolerance is the suite's
FFN tolerance (2e-3 of each value, floored at 1% of the row's rms)."""
import numpy as np
import pytest

import oracle
from helpers import FFN_TOL, r8_errors, say, subset_records

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,batch,counts,xscale", [
    (128, 2, (0, 0, 1), 1.0), (256, 3, (1, 0, 0), 1.0), (384, 8, (8, 16, 31), 1.0),
    (640, 16, (9, 33, 32), 1.0), (1024, 17, (32, 31, 1), 1.0), (2048, 32, (17, 65, 130), 1.0),
    (1152, 31, (0, 40, 0), 1.0), (512, 9, (70, 70, 300), 64.0), (4096, 5, (40, 200, 400), 2.0 ** -8),
    # above 16 rows, at most and more than 256 gate/up tiles of 16 items (8 of FP16)
    (256, 17, (8, 16, 4064), 1.0), (256, 17, (8, 17, 4064), 1.0), (384, 32, (513, 1505, 1603), 1.0)])
def test_batched_ffn_edges(d, batch, counts, xscale):
    from paper_2410_14740_amd import m2c
    from paper_2410_14740_amd import workloads as W
    n = sum(counts)
    d_ff = n + 7
    ld = W.make_layer(500 + d + batch, 0, d, d_ff, 8, 1, rhos=(0.5,) * batch)
    rng = np.random.default_rng(d + batch)
    tm = np.zeros((batch, d_ff), np.uint8)
    ids = np.sort(rng.permutation(d_ff)[:n])
    tier = np.repeat([3, 2, 1], counts).astype(np.uint8)[rng.permutation(n)]
    for i, t in zip(ids, tier):  # each active neuron in one or more rows, one of them at its tier
        rows = rng.permutation(batch)[: rng.integers(1, batch + 1)]
        tm[rows, i] = rng.integers(1, t + 1, len(rows))
        tm[rows[0], i] = t
    x = (ld.x[0].astype(np.float32) * xscale * np.exp2(rng.integers(-6, 7, (batch, 1)))).astype(np.float16)
    L = m2c.Layer(m2c.make_desc(d, d_ff, 8, d_ff, d_ff, max_batch=batch), ld)
    y = torch.zeros((batch, d), dtype=torch.float32, device="cuda")
    say(f"batched FFN d={d} batch={batch} tiers={counts} xscale={xscale}")
    L.cache_plan(torch.from_numpy(tm).cuda(), batch, 0)
    L.cache_fill()
    for _ in range(2):  # the second call adds the same again: scratch left by a call does not matter
        L.sparse_ffn(torch.from_numpy(x.view(np.uint16)).cuda(), batch, y)
    torch.cuda.synchronize()
    recs, row = subset_records(ld, ids)
    masks = ((tm[:, ids] > 0) * (1 << np.arange(batch, dtype=np.uint64))[:, None]).sum(0).astype(np.uint32)
    want = oracle.sparse_ffn(x, np.array([row[int(i)] for i in ids], np.int32), tier, recs, masks)
    for b in range(batch):
        err = r8_errors(y.cpu().numpy()[b] / 2, want[b]).max()
        assert err <= FFN_TOL, f"row {b}: {err:.3e}"
    L.stats()
    L.close()
