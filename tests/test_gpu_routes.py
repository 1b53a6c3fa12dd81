"""Kernels and dispatch branches at the sizes where they can go wrong, against the oracle, bit for bit."""
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
