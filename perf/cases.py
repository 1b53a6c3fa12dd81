"""Performance cases of the batched replay: what its users replay, through the public binding.

A user lays a batch out once (``DeviceBatch``: descriptors and events on the GPU, outputs and scratch
beside them) and replays it with ``replay()`` or ``replay_noalloc()``.  One pass is one such call; its
outputs are the batch's outcomes, pool telemetry and claim telemetry, whole.  Every output is an
integer and must be the same bit for bit.

Inputs are drawn by the package's own generator: case seed -> which pools of a recipe are drawn.
The recipes ("small", "zipf", "nested", ...) are the package's workloads; ``usable`` and ``events`` scale
a recipe's block quantities and claim durations by the ratios that its full-size workload has.
"""
import random

import numpy as np

import paper_2605_24259_amd as rkc
from paper_2605_24259_amd import tracegen as tg

# claim share of a recipe's events (claim slots and their 40-byte records follow from it)
CLAIM_SHARE = {"probe": 0.5, "sweep": 0.5, "small": 0.15, "zipf": 0.15, "nested": 0.2, "zipf_defer": 0.135,
               "zipf_relax": 0.15, "zipf_offload": 0.15}
# pools whose event counts and sizes differ keep between 1/8 and all of their events
RAGGED_LOW = 8


def _pools(name, recipe, pools, events, usable, chains, claims, requests, ragged=False, noalloc=False):
    c = dict(recipe=recipe, pools=pools, events=events, usable=usable, chains=chains, claims=claims,
             requests=requests, ragged=ragged, noalloc=noalloc)
    return dict(c, name=name) if name else c


def _sweep(name, residents, actives, usables):
    c = dict(recipe="sweep", residents=residents, actives=actives, usables=usables)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the 60/70/80 probe under the four policies: one conformance check, all launch latency
        dict(name="probe", recipe="probe"),
        # one scheduler's own pool under a few candidate settings: few pools, each a serial chain
        _pools("zipf_few", "zipf", 64, 1024, 2048, 256, 64, 256),
        # conformance-size pools by the thousand (the "small" workload)
        _pools("small", "small", 4096, 256, 80, 0, 64, 64),
        # a fleet of unlike pools and traces of unlike length, from code that may not allocate
        _pools("small_ragged", "small", 3001, 256, 80, 0, 64, 64, ragged=True, noalloc=True),
        # the capacity sweep: 131,072 cells of one claim and one prefill
        _sweep("sweep", 32, 32, 32),
        # the benchmark workload
        _pools("zipf", "zipf", 65536, 1024, 2048, 256, 64, 256),
        # hard-protection pools: scheduler deferral and retries, and relaxation with a second tier
        _pools("zipf_defer", "zipf_defer", 16384, 1024, 2048, 256, 64, 256),
        _pools("zipf_offload", "zipf_offload", 16384, 1024, 2048, 256, 64, 256),
        # many overlapping claims on few chains, demotion-heavy
        _pools("nested", "nested", 8192, 2048, 16384, 64, 256, 256),
        # longer traces that keep some hundred claims alive over many chains
        _pools("zipf_claims", "zipf", 2048, 2048, 2048, 256, 256, 256),
        # pools of a million tokens of KV
        _pools("wide", "zipf", 512, 4096, 65536, 256, 256, 1024),
        # the largest pools and the longest traces
        _pools("huge", "zipf", 64, 65536, 262144, 256, 4096, 16384),
    ]


def _log(rng, a, b):
    """An integer of [a, b], spread over its logarithm."""
    return min(b, max(a, int(round(a * (b / a) ** rng.random()))))


def draw(rng: random.Random):
    kind = rng.choice(("sweep", "small", "zipf", "zipf", "extended", "nested", "claims", "wide", "huge"))
    if kind == "sweep":
        return _sweep(None, rng.randint(5, 32), rng.randint(5, 32), rng.randint(5, 32))
    if kind == "small":
        return _pools(None, "small", _log(rng, 17, 4096), _log(rng, 40, 256), rng.randint(64, 200), 0, 64, 64,
                      ragged=rng.random() < 0.5, noalloc=rng.random() < 0.5)
    if kind == "zipf":
        return _pools(None, "zipf", _log(rng, 33, 16384), _log(rng, 200, 1024), _log(rng, 1000, 4096),
                      rng.choice((57, 64, 100, 128, 200, 256)), 64, 256, ragged=rng.random() < 0.3)
    if kind == "extended":
        return _pools(None, rng.choice(("zipf_defer", "zipf_relax", "zipf_offload")), _log(rng, 33, 8192),
                      _log(rng, 200, 1024), _log(rng, 1000, 4096), rng.choice((64, 120, 256)), 64, 256,
                      ragged=rng.random() < 0.3)
    if kind == "nested":
        return _pools(None, "nested", _log(rng, 33, 4096), _log(rng, 300, 2048), 16384, rng.randint(30, 64), 256, 256)
    if kind == "claims":
        return _pools(None, "zipf", _log(rng, 33, 2048), _log(rng, 600, 2048), _log(rng, 1000, 4096),
                      rng.randint(70, 256), rng.randint(80, 256), 256)
    if kind == "wide":
        return _pools(None, "zipf", _log(rng, 16, 512), _log(rng, 1000, 4096), _log(rng, 33000, 131072),
                      rng.randint(100, 256), 256, 1024, ragged=rng.random() < 0.3)
    return _pools(None, "zipf", rng.randint(7, 64), _log(rng, 8000, 65536), _log(rng, 100000, 262144), 256, 4096, 16384)


def _scaled(c):
    """Generator overrides of a case: the recipe's ratios at the case's sizes."""
    U, n, recipe = c["usable"], c["events"], c["recipe"]
    p = dict(usable_blocks=U, n_events=n, max_live_claims=c["claims"], max_live_requests=c["requests"])
    if recipe == "small":
        return dict(p, prefill_max=U + U // 5, claim_len_min=max(1, U // 10), claim_len_max=max(1, U * 4 // 5),
                    dur_min=max(1, n // 16), dur_max=max(1, n // 2))
    if recipe == "nested":
        return dict(p, n_chains=c["chains"], dur_min=max(1, n // 16), dur_max=max(1, n // 2))
    # prefills up to 3/4 of the pool, chains of 1/64 to 1/4 of it, claims for 1/16 to 1/2 of the trace;
    # tables of more than 64 claims are kept from overflowing by the generator
    p.update(n_chains=c["chains"], prefill_max=U * 3 // 4, chain_len_min=max(1, U // 64), chain_len_max=max(1, U // 4),
             dur_min=max(1, n // 16), dur_max=max(1, n // 2), claim_cap=c["claims"] if c["claims"] > 64 else 0)
    if recipe == "zipf_offload":
        p["offload_blocks"] = U // 2
    return p


def _offsets(counts):
    return (np.cumsum(counts) - counts).astype(np.int64).view(np.int32).reshape(-1, 2)


def _with_slots(t, share):
    """The trace with a claim table that does not depend on the seed: a record for each CLAIM that the
    recipe's mix draws (and six standard deviations), the pools' spare records spread evenly."""
    P, E = t.n_pools, t.n_events
    cap = int(E * share + 6 * (E * share * (1 - share)) ** 0.5) + 8
    spare = cap - t.n_claim_slots
    d = t.desc.copy()
    d[:, 6] += spare // P + (np.arange(P) < spare % P)
    d[:, 14:16] = _offsets(d[:, 6].astype(np.int64))
    return tg.Trace(d, t.events, cap, t.name)


def _ragged(t, rng):
    """The trace with every pool cut to a length of its own (the case's, whatever the seed), and with
    less room in some."""
    P, n = t.n_pools, t.n_events // t.n_pools
    ne = np.random.default_rng(P * 4096 + n).integers(max(1, n // RAGGED_LOW), n + 1, P)
    ev = t.events.reshape(P, n, 4)
    keep = np.arange(n)[None, :] < ne[:, None]
    slots = ((ev[:, :, 0] & 15) == tg.EV_CLAIM) & keep
    ns = slots.sum(1)
    d = t.desc.copy()
    d[:, 0] = rng.integers(max(1, int(d[0, 0]) * 3 // 4), int(d[0, 0]) + 1, P)
    d[:, 2] = ne
    d[:, 6] = ns
    d[:, 12:14], d[:, 14:16] = _offsets(ne), _offsets(ns)
    return tg.Trace(d, np.ascontiguousarray(ev[keep]), int(ns.sum()), t.name)


def _trace(c, seed):
    rng = np.random.default_rng(seed)
    if c["recipe"] == "probe":
        # the paper's probe, the resident and active sizes moved by the seed
        R, S = 60 - int(rng.integers(0, 20)), 70 - int(rng.integers(0, 20))
        return tg.from_pools([dict(usable_blocks=80, mode=m, n_chains=2,
                                   events=[tg.claim(R, 0, R, hard=1, prio=3), tg.prefill(S, 1, 0)]) for m in range(4)])
    if c["recipe"] == "sweep":
        pick = lambda lo, hi, k: tuple(int(x) for x in np.sort(rng.choice(np.arange(lo, hi), k, replace=False)))  # noqa: E731
        return tg.sweep(pick(8, 257, c["residents"]), pick(8, 257, c["actives"]), pick(16, 513, c["usables"]))
    t = tg.generate(c["recipe"], n_pools=c["pools"], first_pool=(seed % 16384) * 131072, **_scaled(c))
    return _with_slots(_ragged(t, rng) if c["ragged"] else t, CLAIM_SHARE[c["recipe"]])


def prepare(case, seed):
    """What a user's program holds: the batch on the GPU."""
    return case, rkc.DeviceBatch.from_trace(_trace(case, seed), scratch=not case.get("noalloc"))


def run(state):
    case, db = state
    if case.get("noalloc"):
        db.replay_noalloc()
    else:
        db.replay()
    return db.outcomes, db.pool_tel, db.claim_tel


def work(case):
    """Bytes of one pass: a 16-byte event in and a 16-byte outcome out per event, a 40-byte record per
    claim, a 64-byte descriptor in and a 256-byte telemetry record out per pool.  No arithmetic
    beyond integer bookkeeping."""
    if case["recipe"] == "probe":
        pools, events = 4, 8
    elif case["recipe"] == "sweep":
        pools = 4 * case["residents"] * case["actives"] * case["usables"]
        events = 2 * pools
    else:
        pools = case["pools"]
        events = pools * case["events"] * ((1 + 1 / RAGGED_LOW) / 2 if case["ragged"] else 1)
    return {"bytes": events * (32 + 40 * CLAIM_SHARE[case["recipe"]]) + pools * 320, "flops": 0}


def tolerance(case):
    return "exact"
