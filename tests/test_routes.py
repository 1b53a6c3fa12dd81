"""Which kernel a batch goes to, by the host-side rules (no GPU needed)."""
import ctypes

import pytest


def batch(n_pools, usable, events, chains, requests, claims, slots=None):
    import paper_2605_24259_amd as rkc
    b = rkc.Batch()
    b.n_pools, b.max_usable_blocks, b.max_events, b.max_chains = n_pools, usable, events, chains
    b.max_live_requests, b.max_live_claims, b.max_claim_slots = requests, claims, slots or events // 4 + 1
    # plausible, aligned device addresses; none is dereferenced by the host-side checks
    b.d_pools, b.d_pool_tel, b.d_scratch = 0x10000, 0x40000, 0x60000
    return b


def large_pool(*args, **kw):
    """Whether the large-pool kernel takes the batch: it needs less scratch there than on the general kernel
    (limits whose scratch would be the same on both are not for this test)."""
    import paper_2605_24259_amd as rkc
    b = batch(*args, **kw)
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


# a batch that goes to the general kernel for its speed only is still taken with the large-pool kernel's scratch
@pytest.mark.parametrize("n_pools,chains,requests,claims", [(513, 256, 4097, 2500), (64, 16, 9000, 5000)])
def test_smaller_scratch_is_taken(n_pools, chains, requests, claims):
    import torch

    import paper_2605_24259_amd as rkc
    if torch.cuda.is_available():
        pytest.skip("needs a machine without a GPU: the accepted calls must stop at their launch")
    lib = rkc.load()
    b = batch(n_pools, 40000, 64, chains, requests, claims)
    general = lib.rkc_scratch_bytes(ctypes.byref(b))
    assert not large_pool(n_pools, 40000, 64, chains, requests, claims)
    refused = taken = None
    low, high = 0, general
    while high - low > 1:  # the least scratch that is not refused
        b.scratch_bytes = (low + high) // 2
        if lib.rkc_replay_batch(ctypes.byref(b), None) == -5:
            low = refused = b.scratch_bytes
        else:
            high = taken = b.scratch_bytes
    # the pools' regions of the large-pool kernel: the nodes of 64 events are in LDS; FIFO, slots, deferral ring,
    # and the claims past 256
    up = lambda n: -(-n // 256) * 256  # noqa: E731
    c = -(-(claims - 256) // 64) * 64
    assert taken == refused + 1 == n_pools * (up(8 * 65) + up(8 * 17) + up(16 * requests) + up(16 * c) + up(8 * c)) < general


def test_builtin_scratch_takes_what_fits_in_either_kernel():
    import paper_2605_24259_amd as rkc
    lib = rkc.load()
    b = batch(513, 40000, 64, 256, 4097, 2500)
    assert lib.rkc_scratch_bytes(ctypes.byref(b)) > rkc.NOALLOC_SCRATCH_BYTES
    assert lib.rkc_replay_batch_noalloc(ctypes.byref(b), None) != -8
    b = batch(600, 40000, 64, 256, 4097, 2500)
    assert lib.rkc_replay_batch_noalloc(ctypes.byref(b), None) == -8
