"""Kernels and dispatch branches at the sizes where they can go wrong, against the oracle, bit for bit."""
import numpy as np
import pytest

from tests import randtrace
from tests.gpu_util import compare_pools, gpu_replay, say

pytestmark = pytest.mark.gpu


# four claim sets with one, two and four 64-chain key groups: the edges of the groups
@pytest.mark.parametrize("n_chains", [64, 65, 128, 129, 256])
def test_claim_sets_over_chain_groups(oracle_mod, n_chains):
    trace = randtrace.many_claims_batch(900 + n_chains, 96, n_events=(300, 900), n_chains=n_chains)
    say(f"case claim sets over {n_chains} chains: {trace.n_pools} pools")
    gpu = gpu_replay(trace)
    ora = oracle_mod.replay(trace.desc, trace.events, trace.n_claim_slots, threads=16)
    assert not ora[3].any()
    assert ora[1][:, 30].max() > 64, "no pool keeps more than one claim set live"
    compare_pools(trace, gpu, ora)


# one lane per pool: partial and whole waves of pools, two events each
@pytest.mark.parametrize("n_pools", [1, 63, 64, 65, 1000])
def test_two_event_pools(oracle_mod, n_pools):
    trace = randtrace.random_batch(700 + n_pools, n_pools, U_range=(2, 14), n_events=(0, 2), defer=True, relax=True,
                                   offload=True, hard_share=0.6)
    say(f"case two-event pools: {n_pools}")
    ora = oracle_mod.replay(trace.desc, trace.events, trace.n_claim_slots, threads=16)
    compare_pools(trace, gpu_replay(trace), ora)


# four events: the smallest batch that goes one lane per pool, and one pool fewer (a wavefront per pool)
@pytest.mark.parametrize("n_pools", [49151, 49152])
def test_four_event_pools(oracle_mod, tg, n_pools):
    base = randtrace.random_batch(801, 4096, U_range=(2, 14), n_events=(1, 4), defer=True, relax=True, offload=True,
                                  hard_share=0.6)
    reps = -(-n_pools // base.n_pools)
    desc = np.tile(base.desc, (reps, 1))
    k = np.repeat(np.arange(reps, dtype=np.int64), base.n_pools)
    for col, field, step in ((12, "event_offset", base.n_events), (14, "claim_slot_offset", base.n_claim_slots)):
        desc[:, col: col + 2] = (np.tile(base.field(field), reps) + k * step).view(np.int32).reshape(-1, 2)
    trace = tg.Trace(np.ascontiguousarray(desc[:n_pools]), np.tile(base.events, (reps, 1)), base.n_claim_slots * reps)
    say(f"case four-event pools: {n_pools}")
    out, pt, ct = gpu_replay(trace)
    o_out, o_pt, o_ct, _ = oracle_mod.replay(base.desc, base.events, base.n_claim_slots, threads=16)
    whole = n_pools // base.n_pools
    assert (out[: whole * base.n_events].reshape(whole, -1, 4) == o_out).all()
    assert (pt[: whole * base.n_pools].reshape(whole, -1, 64) == o_pt).all()
    assert (ct[: whole * base.n_claim_slots].reshape(whole, -1, 10) == o_ct).all()
