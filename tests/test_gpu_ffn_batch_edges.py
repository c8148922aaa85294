"""Batched FFN where its tiles and steps end: tiers of 0, 1, 8, 16, 31, 32, 33
... items, quantization group counts that are no multiple of 16, one row tile
and two, wide gate/up tiles, rows of very different magnitude, and down waves
of several steps whose exponent falls between them, against the oracle. The
tolerance of the first test is the suite's FFN tolerance (2e-3 of each value,
floored at 1% of the row's rms); the second has its own, with its reason."""
import numpy as np
import pytest

import oracle
from helpers import FFN_TOL, r8_errors, say, subset_records

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _tier_map(rng, d_ff, batch, counts):
    """(tier map, active ids, their tiers): each active neuron in one or more
    rows, one of them at its tier."""
    n = sum(counts)
    tm = np.zeros((batch, d_ff), np.uint8)
    ids = np.sort(rng.permutation(d_ff)[:n])
    tier = np.repeat([3, 2, 1], counts).astype(np.uint8)[rng.permutation(n)]
    for i, t in zip(ids, tier):
        rows = rng.permutation(batch)[: rng.integers(1, batch + 1)]
        tm[rows, i] = rng.integers(1, t + 1, len(rows))
        tm[rows[0], i] = t
    return tm, ids, tier


def _run(ld, d, d_ff, batch, x, tm, ids, tier):
    """(the kernels' y, the oracle's)"""
    from paper_2410_14740_amd import m2c
    L = m2c.Layer(m2c.make_desc(d, d_ff, 8, d_ff, d_ff, max_batch=batch), ld)
    y = torch.zeros((batch, d), dtype=torch.float32, device="cuda")
    L.cache_plan(torch.from_numpy(tm).cuda(), batch, 0)
    L.cache_fill()
    for _ in range(2):  # the second call adds the same again: scratch left by a call does not matter
        L.sparse_ffn(torch.from_numpy(x.view(np.uint16)).cuda(), batch, y)
    torch.cuda.synchronize()
    L.stats()
    L.close()
    recs, row = subset_records(ld, ids)
    masks = ((tm[:, ids] > 0) * (1 << np.arange(batch, dtype=np.uint64))[:, None]).sum(0).astype(np.uint32)
    want = oracle.sparse_ffn(x, np.array([row[int(i)] for i in ids], np.int32), tier, recs, masks)
    return y.cpu().numpy() / 2, want


@pytest.mark.parametrize("d,batch,counts,xscale", [
    (128, 2, (0, 0, 1), 1.0), (256, 3, (1, 0, 0), 1.0), (384, 8, (8, 16, 31), 1.0),
    (640, 16, (9, 33, 32), 1.0), (1024, 17, (32, 31, 1), 1.0), (2048, 32, (17, 65, 130), 1.0),
    (1152, 31, (0, 40, 0), 1.0), (512, 9, (70, 70, 300), 64.0), (4096, 5, (40, 200, 400), 2.0 ** -8),
    # above 16 rows, at most and more than 256 gate/up tiles of 16 items (8 of FP16)
    (256, 17, (8, 16, 4064), 1.0), (256, 17, (8, 17, 4064), 1.0), (384, 32, (513, 1505, 1603), 1.0)])
def test_batched_ffn_edges(d, batch, counts, xscale):
    from paper_2410_14740_amd import workloads as W
    d_ff = sum(counts) + 7
    ld = W.make_layer(500 + d + batch, 0, d, d_ff, 8, 1, rhos=(0.5,) * batch)
    rng = np.random.default_rng(d + batch)
    tm, ids, tier = _tier_map(rng, d_ff, batch, counts)
    x = (ld.x[0].astype(np.float32) * xscale * np.exp2(rng.integers(-6, 7, (batch, 1)))).astype(np.float16)
    say(f"batched FFN d={d} batch={batch} tiers={counts} xscale={xscale}")
    y, want = _run(ld, d, d_ff, batch, x, tm, ids, tier)
    for b in range(batch):
        err = r8_errors(y[b], want[b]).max()
        assert err <= FFN_TOL, f"row {b}: {err:.3e}"


# A group's down waves: 4 per workgroup, 512 / (d / 128) workgroups, 32 items of
# one tier per step, so that a wave takes 3 (d 16384: 42 steps for 16 waves), 2
# (d 8192: 49 for 32), 2 (d 4096: 74 for 64), 7 (d 16384, INT4 alone: 100 for 16)
# or 4 (FP16 alone: 50 for 16) steps; with 3 a wave has FP16 and INT8, another INT8
# and INT4 steps.
@pytest.mark.parametrize("batch", [2, 5, 13, 17, 32])
@pytest.mark.parametrize("d,counts", [(16384, (80, 300, 900)), (8192, (100, 400, 1000)),
                                      (4096, (250, 700, 1400)), (16384, (0, 0, 3200)),
                                      (16384, (1600, 0, 0))])
def test_batched_ffn_several_steps_per_wave(d, batch, counts):
    """Waves of several steps, with values that rise and fall by powers of two
    from step to step, so that the running exponent of a row falls while its
    sums are not zero. The sums are fp32 and the codes exact, so an output is
    off by a few 2^-24 of its row's rms times the root of the gate and up dot
    products' length (128 x 6e-8 = 8e-6 for one h at d 16384, less for a sum of
    many). h rounded to fp16 once, as when the low part of the split is lost,
    is 2^-12 of every term, 5e-4 of the rms at the worst output (computed in
    numpy for such values): the tolerance, 2e-5 of the
    rms, lies between."""
    from paper_2410_14740_amd import workloads as W
    n = sum(counts)
    d_ff = n + 3
    ld = W.make_layer(700 + d + batch, 0, d, d_ff, 8, 1, rhos=(0.5,) * batch)
    rng = np.random.default_rng(d + batch + n)
    tm, ids, tier = _tier_map(rng, d_ff, batch, counts)
    for t in (3, 2, 1):  # the work order: ascending id inside a tier, 32 items a step
        of_tier = ids[tier == t]
        e = rng.integers(-6, 7, len(of_tier) // 32 + 1)[np.arange(len(of_tier)) // 32]
        ld.w_up[of_tier] = (ld.w_up[of_tier].astype(np.float32) * np.exp2(e)[:, None]).astype(np.float16)
    x = (ld.x[0].astype(np.float32) * np.exp2(rng.integers(-3, 1, (batch, 1)))).astype(np.float16)
    say(f"batched FFN, several steps per wave: d={d} batch={batch} tiers={counts}")
    y, want = _run(ld, d, d_ff, batch, x, tm, ids, tier)
    for b in range(batch):
        err = np.abs(y[b] - want[b]).max() / np.sqrt(np.mean(want[b] ** 2))
        say(f"  row {b}: {err:.2e} of the rms")
        assert err <= 2e-5, f"row {b}: {err:.3e}"
