"""Which kernel a batch goes to, by the host-side rules (no GPU needed)."""
import ctypes

import pytest


def large_pool(n_pools, usable, events, chains, requests, claims, slots=None):
    """Whether the large-pool kernel takes the batch: it needs less scratch there than on the general kernel
    (limits whose scratch would be the same on both are not for this test)."""
    import paper_2605_24259_amd as rkc
    b = rkc.Batch()
    b.n_pools, b.max_usable_blocks, b.max_events, b.max_chains = n_pools, usable, events, chains
    b.max_live_requests, b.max_live_claims, b.max_claim_slots = requests, claims, slots or events // 4 + 1
    need = []
    for b.flags in (0, rkc.FLAG_GENERAL_KERNEL):
        need.append(rkc.load().rkc_scratch_bytes(ctypes.byref(b)))
    assert need[0] <= need[1]
    return need[0] < need[1]


# the largest pools: one a CU in the large-pool kernel, eight in the general one
@pytest.mark.parametrize("n_pools,taken", [(1, True), (256, True), (512, True), (513, False), (1024, False), (3072, False)])
def test_pools_of_a_cu(n_pools, taken):
    assert large_pool(n_pools, 262144, 2048, 256, 16384, 4096) is taken


# three a CU against eight, seven against sixteen, three against two, at and past 2.5 times the rounds
@pytest.mark.parametrize("n_pools,usable,chains,requests,claims,taken", [
    (1536, 65536, 256, 4096, 4096, True), (1537, 65536, 256, 4096, 4096, False), (2048, 65536, 256, 4096, 4096, False),
    (2049, 65536, 256, 4096, 4096, True), (3840, 65536, 256, 4096, 4096, True), (3841, 65536, 256, 4096, 4096, False),
    (3584, 2048, 8, 300, 64, True), (3585, 2048, 8, 300, 64, False), (8192, 2048, 8, 300, 64, True),
    (8192, 65536, 256, 1024, 256, True)])
def test_rounds_of_smaller_tables(n_pools, usable, chains, requests, claims, taken):
    assert large_pool(n_pools, usable, 1024, chains, requests, claims) is taken


# long claim tables, and traces of a few events that take more rounds than on the general kernel
@pytest.mark.parametrize("n_pools,events,claims,taken", [
    (64, 4096, 4096, True), (64, 4096, 4097, False), (600, 4096, 4097, False),
    (256, 7, 4096, True), (512, 7, 4096, False), (512, 8, 4096, True)])
def test_claim_tables_and_short_traces(n_pools, events, claims, taken):
    assert large_pool(n_pools, 100000, events, 256, 16384, claims) is taken


# past the kernel's encoding
@pytest.mark.parametrize("kw,taken", [({}, True), (dict(usable=1 << 20), False), (dict(events=65537), False),
                                      (dict(chains=257), False), (dict(requests=16385), False), (dict(slots=65537), False)])
def test_limits_of_the_encoding(kw, taken):
    lim = dict(usable=(1 << 20) - 1, events=65536, chains=256, requests=16384, claims=4096, slots=65536)
    assert large_pool(64, **dict(lim, **kw)) is taken
