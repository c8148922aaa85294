"""Cache plans at the edges of the plan kernels' tiling, against the oracle on
given tier maps: chunks of 256 neurons, rounds of 1024 and sweeps of 8192 LRU
places, orders of many sweeps, of which a workgroup ranks only a part, pools
that start and end inside them, empty pools, and a captured plan replayed
with changing tier maps."""
import numpy as np
import pytest

import oracle
from helpers import say, work_order

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

FIELDS = ("req_ids", "req_tier", "req_hit", "req_slot", "req_mask", "fill_ids", "fill_tier",
          "fill_slot", "fill_from", "evicted_ids")


class _Zero:
    def __init__(self, d, d_ff, r):
        self.w_gate = self.w_up = np.zeros((d_ff, d), np.float16)
        self.w_down = np.zeros((d, d_ff), np.float16)
        self.pred_a, self.pred_b = np.zeros((r, d), np.float16), np.zeros((d_ff, r), np.float16)
        self.bias = None


def _layer(d_ff, k, C, batch=1, flags=0, tier_slots=None):
    from paper_2410_14740_amd import m2c
    return m2c.Layer(m2c.make_desc(128, d_ff, 8, k, C, max_batch=batch, flags=flags,
                                   tier_slots=tier_slots), _Zero(128, d_ff, 8))


def _maps(rng, batch, d_ff, k, steps):
    """Tier maps whose active sets drift, so that hits, refills, evictions
    and (where C < k) bypasses all occur."""
    score = rng.standard_normal((batch, d_ff))
    for _ in range(steps):
        score = 0.8 * score + 0.6 * rng.standard_normal((batch, d_ff))
        tm = np.zeros((batch, d_ff), np.uint8)
        for b in range(batch):
            kk = max(0, k - int(rng.integers(0, 3)))
            order = np.argsort(-score[b])[:kk]
            tm[b, order] = 1
            tm[b, order[: kk // 2]] = 2
            tm[b, order[: kk // 5]] = 3
        yield tm


def _check(L, o, label):
    g = L.read_plan()
    for f in FIELDS:
        assert np.array_equal(g[f], o[f]), f"{label}: {f}"
    ws, wm = work_order(o)
    assert np.array_equal(g["work_slot"], ws) and np.array_equal(g["work_mask"], wm), label
    assert np.array_equal(g["counts"][:13], o["counts"][:13]), label


@pytest.mark.parametrize("d_ff,k,C,batch,dom", [
    (1, 1, 1, 1, 0), (1023, 300, 500, 1, 1), (1024, 300, 0, 1, 0), (1025, 400, 1024, 2, 0),
    (9000, 1500, 8192, 1, 0), (9000, 1500, 8193, 3, 1), (20000, 2500, 17000, 1, 1),
    (66000, 3000, 4097, 1, 0),
    # chunks of 256 neurons and rounds of 1024 places
    (255, 100, 200, 1, 0), (256, 256, 100, 2, 1), (257, 120, 257, 1, 0), (2049, 500, 1025, 5, 0),
    (5000, 800, 2048, 1, 1),
    # orders of several sweeps: bypass beyond them, nearly all new, 13 sweeps, every slot of the largest layer
    (30000, 12000, 9000, 1, 0), (60000, 15000, 40961, 1, 0), (33000, 16000, 16385, 2, 1), (100000, 3000, 100000, 1, 1),
    (262144, 1000, 262144, 2, 0)])
def test_plan_single_arena_edges(d_ff, k, C, batch, dom):
    from paper_2410_14740_amd import m2c
    L = _layer(d_ff, k, C, batch, m2c.FLAG_DOMINANT_HITS if dom else 0)
    cache = oracle.LRUCache(d_ff, C, L.info.staging_slots,
                            oracle.POLICY_DOMINANCE if dom else oracle.POLICY_EXACT)
    for t, tm in enumerate(_maps(np.random.default_rng(d_ff + C), batch, d_ff, k, 5)):
        say(f"plan d_ff={d_ff} C={C} batch={batch} dom={dom} step {t}")
        tiers = torch.from_numpy(tm).cuda()
        L.cache_plan(tiers, batch, 3 * t)
        torch.cuda.synchronize()
        _check(L, cache.plan(tm, 3 * t), f"step {t}")
        slot_of, key, tier, last = m2c.m2c_debug_read_tables(L.handle, d_ff, C)
        assert np.array_equal(slot_of, cache.slot_of)
        assert np.array_equal(key, cache.slot_key[:C])
        assert np.array_equal(tier, cache.slot_tier[:C])
        assert np.array_equal(last, cache.slot_last[:C])
    L.close()


@pytest.mark.parametrize("dom", [0, 1])
@pytest.mark.parametrize("d_ff,k,slots", [
    (1024, 200, {3: 1, 2: 1, 1: 1}), (3000, 700, {3: 1024, 2: 1000, 1: 24}),
    (3000, 700, {3: 0, 2: 0, 1: 300}), (3000, 700, {3: 300, 2: 0, 1: 0}),
    (32768, 4000, {3: 8191, 2: 2, 1: 9000}), (32768, 4000, {3: 800, 2: 8192, 1: 8193}),
    # orders of several sweeps: pools of several each, one inside a sweep, empty ones, one full at the start
    (32768, 3000, {3: 10000, 2: 9000, 1: 13768}), (32768, 9000, {3: 300, 2: 24000, 1: 8468}),
    (32768, 5000, {3: 0, 2: 9000, 1: 20000}), (32768, 12000, {3: 9000, 2: 0, 1: 9001}),
    (20000, 6000, {3: 500, 2: 16384, 1: 100})])
def test_plan_pool_edges(d_ff, k, slots, dom):
    from paper_2410_14740_amd import m2c
    L = _layer(d_ff, k, 0, 1, m2c.FLAG_DOMINANT_HITS if dom else 0, slots)
    S = {t: L.info.pool_slots[t] - slots[t] for t in (1, 2, 3)}
    cache = oracle.TierPoolCache(d_ff, slots, S,
                                 oracle.POLICY_DOMINANCE if dom else oracle.POLICY_EXACT)
    for t, tm in enumerate(_maps(np.random.default_rng(d_ff + k), 1, d_ff, k, 6)):
        say(f"pools d_ff={d_ff} {slots} dom={dom} step {t}")
        L.cache_plan(torch.from_numpy(tm).cuda(), 1, t)
        torch.cuda.synchronize()
        _check(L, cache.plan(tm[0], t), f"step {t}")
        for tr in (1, 2, 3):
            so, key, last = m2c.m2c_debug_read_pool_tables(L.handle, tr, d_ff, slots[tr])
            assert np.array_equal(so, cache.pools[tr].slot_of)
            assert np.array_equal(key, cache.pools[tr].slot_key[: slots[tr]])
            assert np.array_equal(last, cache.pools[tr].slot_last[: slots[tr]])
    L.close()


@pytest.mark.parametrize("pools", [False, True])
def test_plan_captured_and_replayed(pools):
    """A captured plan replays with the step it was captured with; the LRU
    order follows the plans' order, so every replay's plan is the one the
    oracle makes at increasing steps, with eager plans of another layer
    between the replays."""
    d_ff, k = 3000, 500
    slots = {3: 150, 2: 300, 1: 400}
    L = _layer(d_ff, k, 700, tier_slots=slots if pools else None)
    other = _layer(d_ff, k, 700)
    if pools:
        S = {t: L.info.pool_slots[t] - slots[t] for t in (1, 2, 3)}
        cache = oracle.TierPoolCache(d_ff, slots, S)
    else:
        cache = oracle.LRUCache(d_ff, 700, L.info.staging_slots)
    maps = list(_maps(np.random.default_rng(5), 1, d_ff, k, 6))
    tiers = torch.from_numpy(maps[0]).cuda()
    L.cache_plan(tiers, 1, 0)
    torch.cuda.synchronize()
    as_given = (lambda tm: tm[0]) if pools else (lambda tm: tm)
    _check(L, cache.plan(as_given(maps[0]), 0), "eager")
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    say("plan capture")
    with torch.cuda.graph(g, stream=s):
        L.cache_plan(tiers, 1, 1)
    torch.cuda.synchronize()
    for t in range(1, 6):
        say(f"plan replay {t}")
        tiers.copy_(torch.from_numpy(maps[t]))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        _check(L, cache.plan(as_given(maps[t]), t), f"replay {t}")
        other.cache_plan(tiers, 1, t)
        torch.cuda.synchronize()
    del g
    L.close()
    other.close()
