"""The work this library is used for, as cases that can be timed and checked.

Four kinds, all through the public binding (paper_2410_14740_amd.m2c and
.pipeline):

  step    one decode step of one layer on one stream: predict_rank,
          cache_plan, cache_fill, sparse_ffn
  route   what the aux stream does per layer-step: predict_rank and cache_plan
          of every layer, against caches in their steady state
  ffn     what the main stream does per layer-step: sparse_ffn of every layer
          on plans whose records are resident
  stack   a whole decode step of a stack of layers on the three streams of
          pipeline.StackSchedule, fills over the host link included

Weights and predictors are normal fp16 values, decode inputs are AR(1) streams
(consecutive tokens share most of their active neurons), batched layers have a
log-Zipf neuron popularity, as in paper_2410_14740_amd/workloads.py. Layers of
one case share one neuron store, as the benchmark's do; each has its own
predictor, slot cache and plans. Several layers are cycled so that the records
and predictors of a pass come from HBM and not from the Infinity Cache, as
they do in a stack.
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2410_14740_amd import m2c
from paper_2410_14740_amd.pipeline import StackSchedule
from paper_2410_14740_amd.workloads import WORKLOADS, tier_counts

TOKENS = 16  # distinct decode inputs; a state's steps go round them
WARM = 6     # steps a state's cache has seen before the first pass
RHO = 0.9    # correlation of consecutive inputs (batch rows alternate 0.5 / 0.95)
SIGMA_W, SIGMA_P = 0.02, 0.05
QMAX = {1: 7, 2: 127}


def _of(name, workload, kind, layers, batch=1, arena="single", policy="exact", scores=False):
    wl = WORKLOADS[workload]
    k, n16, n8 = wl.counts()
    return {"name": name, "kind": kind, "d": wl.d_model, "d_ff": wl.d_ff, "r": wl.pred_rank,
            "layers": layers, "batch": batch, "k": k, "n16": n16, "n8": n8,
            "slots": wl.cache_slots(), "arena": arena, "policy": policy, "bias": batch > 1,
            "deterministic": False, "scores": scores}


def listed():
    return [
        # one small layer, one token: launches and single-workgroup latency
        _of("step-tiny", "tiny", "step", 1),
        # the test suite's ragged layer (48 chunks of d, 6 of r, d_ff not a
        # multiple of 64), four tokens at once
        {"name": "step-ragged-b4", "kind": "step", "d": 384, "d_ff": 700, "r": 48, "layers": 1,
         "batch": 4, "k": 175, "n16": 58, "n8": 58, "slots": 250, "arena": "single",
         "policy": "exact", "bias": True, "deterministic": False, "scores": False},
        # the aux stream of a 7B decode with the default cache (one arena, exact tiers)
        _of("route-7b", "llama2-7b", "route", 16),
        # the aux stream of the 70B decode with the headline cache policy
        _of("route-70b-pools", "llama2-70b", "route", 8, arena="pools", policy="dominance"),
        # the aux stream of the batched 7B decode (union plans); the scores are asked for
        _of("route-7b-b8", "llama2-7b-b8", "route", 8, batch=8, scores=True),
        # a layer wider than the register select and the ballot plan take
        # (d_ff of the test suite's wide layer)
        {"name": "route-wide", "kind": "route", "d": 1024, "d_ff": 40000, "r": 64, "layers": 4,
         "batch": 1, "k": 4000, "n16": 1000, "n8": 1000, "slots": 6000, "arena": "single",
         "policy": "exact", "bias": False, "deterministic": False, "scores": False},
        # the FFN of a decoded token through 7B-shaped layers
        _of("ffn-7b", "llama2-7b", "ffn", 16),
        # the same at 70B
        _of("ffn-70b", "llama2-70b", "ffn", 8),
        # the batched 7B FFN (union of eight tokens' neurons)
        _of("ffn-7b-b8", "llama2-7b-b8", "ffn", 8, batch=8),
        # the largest call: the most rows a layer takes, 70B shape
        _of("ffn-70b-b32", "llama2-70b", "ffn", 1, batch=32),
        # a token through 7B-shaped layers on the three-stream schedule
        _of("stack-7b", "llama2-7b", "stack", 16, arena="pools", policy="dominance"),
        # the same at 70B, bound by the host link
        _of("stack-70b", "llama2-70b", "stack", 8, arena="pools", policy="dominance"),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["step", "route", "route", "ffn", "ffn", "ffn", "stack"])
    if kind == "step":
        d, d_ff = 128 * log_int(3, 24), log_int(700, 6000)
    elif kind == "route":
        d, d_ff = 128 * log_int(8, 64), log_int(2500, 40000)
        if d_ff > 32768:
            d = 128 * rng.randint(4, 16)
    elif kind == "ffn":
        d, d_ff = 128 * log_int(8, 96), log_int(2500, 28672)
        d_ff = min(d_ff, 8192 * 16384 // d)
    else:
        d, d_ff = 128 * log_int(8, 40), log_int(2500, 13824)
    r = 8 * log_int(4, 64)
    mix = rng.choice([("1/3", "1/3"), ("1/10", "2/5"), ("1/5", "3/10"), ("1/10", "3/10"), ("1", "0")])
    k, n16, n8 = tier_counts(d_ff, "%d/100" % rng.randint(5, 25), *mix)
    batch = 1 if kind == "stack" or rng.random() < 0.5 else log_int(2, 32)
    if kind in ("step", "route"):
        batch = min(batch, 8)
    pools = kind == "stack" or (kind == "route" and batch == 1 and d_ff <= 32768 and rng.random() < 0.5)
    return {"kind": kind, "d": d, "d_ff": d_ff, "r": r,
            "layers": 1 if kind == "step" else rng.randint(2, 6) if batch == 1 else rng.randint(1, 3),
            "batch": batch, "k": k, "n16": n16, "n8": n8,
            "slots": int(d_ff * rng.uniform(0.1, 0.35 if pools else 0.5)),
            "arena": "pools" if pools else "single",
            "policy": rng.choice(["exact", "dominance"]) if pools or kind == "route" else "exact",
            "bias": batch > 1, "deterministic": kind == "ffn" and batch == 1 and rng.random() < 0.25,
            "scores": rng.random() < 0.25}


# ---------------------------------------------------------------------------
# inputs, from the seed alone

def _gen(seed, layer, what):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1009 + layer) * 16 + what)
    return g


def _normal(seed, layer, what, shape, sigma):
    return torch.empty(shape, dtype=torch.float16, device="cuda").normal_(
        0.0, sigma, generator=_gen(seed, layer, what))


def _weights(c, seed):
    d, d_ff = c["d"], c["d_ff"]
    return (_normal(seed, 0, 0, (d_ff, d), SIGMA_W), _normal(seed, 0, 1, (d_ff, d), SIGMA_W),
            _normal(seed, 0, 2, (d, d_ff), SIGMA_W))


def _predictor(c, seed, layer):
    return (_normal(seed, layer, 3, (c["r"], c["d"]), SIGMA_P),
            _normal(seed, layer, 4, (c["d_ff"], c["r"]), SIGMA_P),
            _zipf(c, seed, layer) * (SIGMA_P * SIGMA_P * math.sqrt(c["r"] * c["d"]))
            if c["bias"] else None)


def _zipf(c, seed, layer):
    """log-Zipf popularity in units of the score standard deviation."""
    perm = torch.randperm(c["d_ff"], generator=_gen(seed, layer, 5), device="cuda")
    return (-1.1 * torch.log(perm.double() + 1.0)).float()


def _tokens(c, seed):
    """x [TOKENS][layers][batch][d] fp16, AR(1) along the tokens."""
    B = c["batch"]
    rho = torch.tensor([RHO] if B == 1 else [(0.5, 0.95)[b % 2] for b in range(B)], device="cuda")
    rho = rho.view(1, B, 1)
    shape = (c["layers"], B, c["d"])
    g = _gen(seed, 0, 6)
    x = torch.randn(shape, generator=g, device="cuda")
    out = torch.empty((TOKENS, *shape), dtype=torch.float16, device="cuda")
    for t in range(TOKENS):
        if t:
            x = rho * x + torch.sqrt(1 - rho * rho) * torch.randn(shape, generator=g, device="cuda")
        out[t] = x
    return out


def _tiers_by_rank(scores, c):
    """uint8 tier map of float scores [rows][d_ff]: best n16 FP16, next n8 INT8, rest of k INT4."""
    order = torch.argsort(scores, dim=1, descending=True, stable=True)
    by_rank = torch.zeros(c["d_ff"], dtype=torch.uint8, device=scores.device)
    by_rank[:c["k"]] = 1
    by_rank[:c["n16"] + c["n8"]] = 2
    by_rank[:c["n16"]] = 3
    return torch.zeros(scores.shape, dtype=torch.uint8, device=scores.device).scatter_(
        1, order, by_rank.expand_as(order))


def _given_tiers(c, seed, layer):
    """Tier maps of an ffn case: random scores with the case's popularity."""
    s = torch.randn((c["batch"], c["d_ff"]), generator=_gen(seed, layer, 7), device="cuda")
    return _tiers_by_rank(s + _zipf(c, seed, layer) if c["bias"] else s, c)


def _pool_slots(c):
    counts = {3: c["n16"], 2: c["n8"], 1: c["k"] - c["n16"] - c["n8"]}
    return m2c.pool_slots_for_budget(c["d"], counts, c["slots"] * 6 * c["d"])


_decode_streams = []


def _streams():
    """The program's main, aux and copy streams (a process gets few hardware queues)."""
    if not _decode_streams:
        _decode_streams.extend(torch.cuda.Stream() for _ in range(3))
    return tuple(_decode_streams)


# ---------------------------------------------------------------------------

def prepare(case, seed):
    """Layers with their stores, predictors and warm caches, and the tokens."""
    c = case
    st = SimpleNamespace(c=c, t=0)
    flags = m2c.FLAG_DOMINANT_HITS if c["policy"] == "dominance" else 0
    flags |= m2c.FLAG_DETERMINISTIC_FFN if c["deterministic"] else 0
    pools = c["arena"] == "pools"
    desc = m2c.make_desc(c["d"], c["d_ff"], c["r"], c["k"], c["slots"], max_batch=c["batch"],
                         flags=flags, tier_slots=_pool_slots(c) if pools else None)
    n, B, d, d_ff = c["layers"], c["batch"], c["d"], c["d_ff"]
    host = [w.cpu().numpy() for w in _weights(c, seed)]
    st.layers = []
    for l in range(n):
        a, b, bias = (None if v is None else v.cpu().numpy() for v in _predictor(c, seed, l))
        data = SimpleNamespace(w_gate=host[0], w_up=host[1], w_down=host[2], pred_a=a, pred_b=b,
                               bias=bias)
        st.layers.append(m2c.Layer(desc, data, weights_of=st.layers[0] if l else None))
    del host
    st.x = _tokens(c, seed)
    st.tiers = torch.zeros((n, B, d_ff), dtype=torch.uint8, device="cuda")
    st.y = torch.zeros((n, B, d), dtype=torch.float32, device="cuda")
    st.scores = torch.zeros((n, B, d_ff), dtype=torch.float32, device="cuda") if c["scores"] else None
    L0 = st.layers[0]
    raw = torch.zeros(n * L0.info.plan_bytes + 256, dtype=torch.uint8, device="cuda")
    off = (-raw.data_ptr()) % 256  # plans are 256-byte aligned
    st.plans = raw[off:off + n * L0.info.plan_bytes].view(n, -1)
    st.fields = []
    for f, dt in (("req_ids", torch.int32), ("req_tier", torch.uint8), ("req_hit", torch.uint8),
                  ("req_slot", torch.int32), ("req_mask", torch.int32), ("fill_ids", torch.int32),
                  ("fill_tier", torch.uint8), ("fill_slot", torch.int32),
                  ("fill_from", torch.uint8), ("evicted_ids", torch.int32),
                  ("work_slot", torch.int32), ("work_mask", torch.int32)):
        o, nb = getattr(L0.layout, f), L0.info.plan_capacity * dt.itemsize
        st.fields.append(st.plans[:, o:o + nb].view(dt))
    o = L0.layout.counts
    st.fields.append(st.plans[:, o:o + 4 * m2c.NCOUNTS].view(torch.int32))
    st.sched = None
    if c["kind"] == "ffn":
        for l, L in enumerate(st.layers):
            st.tiers[l] = _given_tiers(c, seed, l)
            L.cache_plan(st.tiers[l], B, 0, plan=st.plans[l])
            L.cache_fill(plan=st.plans[l])
    else:
        if c["kind"] == "stack":
            st.sched = StackSchedule(torch, st.layers, c["k"], c["n16"], c["n8"], st.tiers,
                                     streams=_streams())
        for _ in range(WARM):
            run(st)
    torch.cuda.synchronize()
    return st


def run(state):
    """One pass: a decode step of every layer, or the part of it that the case's kind names."""
    st, c = state, state.c
    B, kind = c["batch"], c["kind"]
    s = torch.cuda.current_stream()
    if kind == "ffn":
        st.y.zero_()
        for l, L in enumerate(st.layers):
            L.sparse_ffn(st.x[0, l], B, st.y[l], stream=s, plan=st.plans[l])
        return st.y
    t = st.t
    st.t += 1
    x = st.x[t % TOKENS]
    if kind == "stack":
        st.y.zero_()
        st.sched.main.wait_stream(s)  # the inputs are resident: only y has to be ready
        st.sched.step(t, lambda l: x[l], lambda l: st.y[l], plan_of=lambda l: st.plans[l])
        s.wait_stream(st.sched.main)
        return st.y, st.tiers
    for l, L in enumerate(st.layers):
        L.predict_rank(x[l], B, c["k"], c["n16"], c["n8"], None if st.scores is None else st.scores[l],
                       st.tiers[l], stream=s)
        L.cache_plan(st.tiers[l], B, t, stream=s, plan=st.plans[l])
    if kind == "route":
        return st.tiers, st.fields, st.scores
    st.y.zero_()
    L = st.layers[0]
    L.cache_fill(stream=s, plan=st.plans[0])
    L.sparse_ffn(x[0], B, st.y[0], stream=s, plan=st.plans[0])
    return st.y, st.tiers, st.scores


# ---------------------------------------------------------------------------

def _record_bytes(d, t):
    return {3: 6 * d, 2: 3 * d + 6 * (d // 128), 1: 3 * d // 2 + 6 * (d // 128)}[t]


def _union(c):
    """Expected required neurons of a step by tier, and (row, neuron) pairs."""
    k, n16, n8, B = c["k"], c["n16"], c["n8"], c["batch"]
    if B == 1:
        return {3: n16, 2: n8, 1: k - n16 - n8}, k
    r = np.random.default_rng(1)
    s = r.standard_normal((B, c["d_ff"]))
    if c["bias"]:
        s = s - 1.1 * np.log(r.permutation(c["d_ff"]) + 1.0)
    rank = np.argsort(np.argsort(-s, axis=1), axis=1).min(axis=0)
    return {3: int((rank < n16).sum()), 2: int(((rank >= n16) & (rank < n16 + n8)).sum()),
            1: int(((rank >= n16 + n8) & (rank < k)).sum())}, k * B


def work(case):
    """Per pass. Every weight byte the math needs once from HBM, inputs and
    outputs once; the host-link bytes of step and stack fills (a share of the
    records that depends on the cache's history) are not counted."""
    c = case
    d, d_ff, r, B, kind = c["d"], c["d_ff"], c["r"], c["batch"], c["kind"]
    by_tier, pairs = _union(c)
    nbytes = flops = 0
    if kind != "ffn":  # predictor, scores if asked for, tier map
        nbytes += 2 * r * (d + d_ff) + 2 * d * B + (4 * d_ff * B if c["scores"] else 0) + d_ff * B
        flops += 2 * r * (d + d_ff) * B
    if kind == "route":  # the plan's lists of the required neurons
        nbytes += 22 * sum(by_tier.values())
    else:
        nbytes += sum(n * _record_bytes(d, t) for t, n in by_tier.items()) + 6 * d * B
        flops += 6 * d * pairs
    return {"bytes": nbytes * c["layers"], "flops": flops * c["layers"]}


def tolerance(case):
    """Scores, tier maps and plans are reproducible bit for bit by contract
    (one fixed fp32 order). The FFN sums in fp32 in no fixed order: over the
    listed cases two runs of one call differ by 7e-8 to 1.6e-7 (rel; max up to
    1e-6), and a call from 64 bits by 1.6e-7 to 3e-7; two implementations can
    be both errors apart."""
    return "exact" if case["kind"] == "route" else {"rel": 2e-6, "max": 2e-5}


# ---------------------------------------------------------------------------
# 64-bit values of run()'s first pass on a new state

def _fixed_order(a, b):
    """Dot products of a's rows with b in the documented fp32 order, so that
    the selection that depends on them is the same; each fmaf is a 64-bit
    product and sum rounded to 32 bits."""
    n = a.shape[1]
    chunks, L = n // 8, 1
    while 2 * L <= min(chunks, 64):
        L *= 2
    acc = torch.zeros((a.shape[0], L), dtype=torch.float64, device=a.device)
    for c0 in range(0, chunks, L):
        m = min(L, chunks - c0)
        for e in range(8):
            cols = torch.arange(c0, c0 + m, device=a.device) * 8 + e
            acc[:, :m] = (acc[:, :m] + a[:, cols].double() * b[cols].double()).float().double()
    lane = torch.arange(L, device=a.device)
    while L > 1:
        L //= 2
        acc = (acc + acc[:, lane ^ L]).float().double()
    return acc[:, 0].float()


def _step_scores(c, pred, x):
    A, Bm, bias = pred
    rows = []
    for xb in x:
        s = _fixed_order(Bm, _fixed_order(A, xb))
        rows.append(s if bias is None else s + bias)
    return torch.stack(rows)


def _dequant(w, tier):
    """fp16 rows -> the values their record of that tier holds, in 64 bits."""
    if tier == 3:
        return w.double()
    g = w.float().view(w.shape[0], -1, 128)
    s = (g.abs().amax(2, keepdim=True) / QMAX[tier]).half().float()
    q = torch.where(s > 0, torch.round(g / s).clamp(-QMAX[tier], QMAX[tier]), torch.zeros_like(g))
    return (q.double() * s.double()).view(w.shape)


def _ffn64(weights, x, tiers, step_tier):
    """sum over active neurons, rows by their own tier map, records at step_tier."""
    wg, wu, wd = weights
    y = torch.zeros((x.shape[0], x.shape[1]), dtype=torch.float64, device="cuda")
    for t in (3, 2, 1):
        of_tier = torch.nonzero(step_tier == t).flatten()
        for i in range(0, len(of_tier), 4096):
            ids = of_tier[i:i + 4096]
            a = x.double() @ _dequant(wg[ids], t).t().contiguous()
            u = x.double() @ _dequant(wu[ids], t).t().contiguous()
            h = a / (1 + torch.exp(-a)) * u * (tiers[:, ids] > 0)
            y += h @ _dequant(wd[:, ids].t().contiguous(), t)
    return y


class _Pools:
    """The per-tier pools of one layer: which tier serves each neuron."""

    def __init__(self, c):
        self.dom, self.C = c["policy"] == "dominance", _pool_slots(c)
        self.of = {t: np.full(c["d_ff"], -1, np.int64) for t in (1, 2, 3)}
        self.key = {t: np.full(self.C[t], -1, np.int64) for t in (1, 2, 3)}
        self.last = {t: np.full(self.C[t], -1, np.int64) for t in (1, 2, 3)}

    def step(self, tm, step):
        tm = tm.copy()
        if self.dom:
            for t in (2, 1):
                want = (tm == t) & (self.of[t] < 0)
                for up in range(t + 1, 4):
                    take = want & (tm == t) & (self.of[up] >= 0)
                    tm[take] = up
        for t in (1, 2, 3):
            of, key, last = self.of[t], self.key[t], self.last[t]
            ids = np.flatnonzero(tm == t)
            last[of[ids][of[ids] >= 0]] = step
            new = ids[of[ids] < 0]
            free = np.flatnonzero(last != step)
            free = free[np.lexsort((free, last[free]))][:len(new)]
            gone = key[free]
            of[gone[gone >= 0]] = -1
            key[free], last[free] = new[:len(free)], step
            of[new[:len(free)]] = free
        return tm


def exact(case, seed):
    c = case
    if c["kind"] == "route":
        if not c["scores"]:
            return None
        x = _tokens(c, seed)[WARM % TOKENS]
        out = []
        for l in range(c["layers"]):
            A, Bm, bias = _predictor(c, seed, l)
            s = (x[l].double() @ A.double().t().contiguous()) @ Bm.double().t().contiguous()
            out.append(s if bias is None else s + bias.double())
        return None, [None] * 13, torch.stack(out)
    weights = _weights(c, seed)
    xs = _tokens(c, seed)
    out, scores = [], []
    for l in range(c["layers"]):
        if c["kind"] == "ffn":
            x, tiers = xs[0, l], _given_tiers(c, seed, l)
            step_tier = tiers.amax(0)
        else:
            pred = _predictor(c, seed, l)
            pools = _Pools(c) if c["arena"] == "pools" else None
            for t in range(0 if pools else WARM, WARM + 1):
                x = xs[t % TOKENS, l]
                s = _step_scores(c, pred, x)
                tiers = _tiers_by_rank(s, c)
                step_tier = tiers.amax(0)
                if pools:
                    step_tier = torch.from_numpy(pools.step(step_tier.cpu().numpy(), t)).cuda()
            scores.append(s.double())
        out.append(_ffn64(weights, x, tiers, step_tier))
    y = torch.stack(out)
    if c["kind"] == "ffn":
        return y
    if c["kind"] == "stack":
        return y, None
    return y, None, torch.stack(scores) if c["scores"] else None
