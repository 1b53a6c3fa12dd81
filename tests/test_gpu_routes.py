"""Kernels and dispatch branches at the sizes where they can go wrong, against the oracle, bit for bit."""
import numpy as np
import pytest

from tests import randtrace
from tests.gpu_util import compare_pools, compare_tiled, gpu_replay, large_pool_route, say, tile

pytestmark = pytest.mark.gpu


# four claim sets over the edges of the 64-chain key groups: one or four groups in the layout for few pools;
# one, two or four past 4,096 pools
@pytest.mark.parametrize("n_pools", [96, 4100])
@pytest.mark.parametrize("n_chains", [64, 65, 128, 129, 256])
def test_claim_sets_over_chain_groups(oracle_mod, n_chains, n_pools):
    base = randtrace.many_claims_batch(900 + n_chains, 96, n_events=(300, 900), n_chains=n_chains)
    say(f"case claim sets over {n_chains} chains: {n_pools} pools")
    ora = oracle_mod.replay(base.desc, base.events, base.n_claim_slots, threads=16)
    assert not ora[3].any()
    assert ora[1][:, 30].max() > 64, "no pool keeps more than one claim set live"
    compare_tiled(gpu_replay(tile(base, n_pools)), ora)


# two events: one wavefront per pool up to 4,096 pools, one lane per pool above (partial and whole waves)
@pytest.mark.parametrize("n_pools", [1, 65, 1000, 4096, 4097, 4159, 4160])
def test_two_event_pools(oracle_mod, n_pools):
    base = randtrace.random_batch(700 + n_pools, min(n_pools, 1000), U_range=(2, 14), n_events=(0, 2), defer=True,
                                  relax=True, offload=True, hard_share=0.6)
    say(f"case two-event pools: {n_pools}")
    ora = oracle_mod.replay(base.desc, base.events, base.n_claim_slots, threads=16)
    compare_tiled(gpu_replay(tile(base, n_pools)), ora)


# four events: the smallest batch that goes one lane per pool, and one pool fewer (a wavefront per pool)
@pytest.mark.parametrize("n_pools", [49151, 49152])
def test_four_event_pools(oracle_mod, n_pools):
    base = randtrace.random_batch(801, 4096, U_range=(2, 14), n_events=(1, 4), defer=True, relax=True, offload=True,
                                  hard_share=0.6)
    say(f"case four-event pools: {n_pools}")
    ora = oracle_mod.replay(base.desc, base.events, base.n_claim_slots, threads=16)
    compare_tiled(gpu_replay(tile(base, n_pools)), ora)


def _big(trace, **limits):
    """The trace with batch limits past the compact kernel's (the large-pool kernel replays it)."""
    import paper_2605_24259_amd as rkc
    lim = dict(trace.limits(), **limits)
    lim["max_usable_blocks"] = max(lim["max_usable_blocks"], 40000)
    assert large_pool_route(trace, lim)
    return rkc.DeviceBatch(trace.desc, trace.events, trace.n_claim_slots, lim).replay().results()


# the large-pool kernel: every feature, table overflows, more pools than CUs and fewer
@pytest.mark.parametrize("n_pools", [40, 700])
@pytest.mark.parametrize("kw", [dict(), dict(defer=True, hard_share=0.7), dict(relax=True, offload=True, hard_share=0.8),
                                dict(defer=True, relax=True, offload=True, hard_share=0.8)],
                         ids=["plain", "defer", "offload", "all"])
def test_large_pool_kernel_random(oracle_mod, n_pools, kw):
    trace = randtrace.random_batch(300 + n_pools, n_pools, U_range=(4, 300), n_events=(1, 400), n_chains=9,
                                   p_malformed=0.01, tight_every=5, **kw)
    say(f"case large-pool random {n_pools} {kw}")
    ora = oracle_mod.replay(trace.desc, trace.events, trace.n_claim_slots, threads=16)
    compare_pools(trace, _big(trace), ora)


# its request ring: tables of 1 to 6 entries, whose ring wraps all the time, and a ring far larger than the lists
@pytest.mark.parametrize("max_live_requests", [6, 16384])
def test_large_pool_kernel_request_ring(oracle_mod, max_live_requests):
    trace = randtrace.many_requests_batch(17, 48, n_events=(900, 1500), n_chains=200, req_cap=1024)
    if max_live_requests < 1024:
        trace.desc[:, 5] = np.minimum(trace.desc[:, 5], max_live_requests)
    say(f"case request ring {max_live_requests}")
    ora = oracle_mod.replay(trace.desc, trace.events, trace.n_claim_slots, threads=16)
    compare_pools(trace, _big(trace, max_live_requests=max_live_requests), ora)


def _full_ring_pool(tg, rng, mode, cap, rounds):
    """A pool that fills its live-request table, then finishes, extends and refills at both ends of it, with
    selectors at the edges of their range; a deferring one also takes its oldest request back in, at the front."""
    late = mode == 3
    evs = []
    if late:
        evs += [tg.claim(3 * cap, 0, 3 * cap, hard=1), tg.prefill(3 * cap + 5, -1, 0)]  # refused for the claim: deferred
    evs += [tg.prefill(1 + i % 2, 1 + i % 9, i % 2) for i in range(cap - late)]
    if late:
        evs += [tg.release(0), tg.retry()]
    evs += [tg.prefill(1, -1, 0)]  # the table is full
    n, top = cap, 2**32 - 1
    for k in range(rounds):
        take = min(n - 1, int(rng.integers(1, 40)))
        for m in range(n, n - take, -1):
            last = top // m * m  # the largest multiple of the list's length, below 2^32
            sel = (0, 1, m - 1, m // 2, m // 2 - 1, m, last - 1, last, top, int(rng.integers(0, top)))[int(rng.integers(0, 10))]
            evs += [tg.extend(1, sel), tg.finish(sel)]
        n -= take
        more = min(cap - n, int(rng.integers(1, 30)))
        evs += [tg.prefill(1, 1 + k % 9, k % 2)] * more
        n += more
    return dict(usable_blocks=6 * cap + 4, mode=mode, n_chains=10, max_live_requests=cap, max_live_claims=2, events=evs,
                defer_limit=2 if late else 0)


# the ring filled to its last entry, and lists of thousands of requests shifted from both sides, with selectors
# at the edges of their range over counts of thousands; the largest ring against the general kernel (the
# oracle takes half a minute)
@pytest.mark.parametrize("cap,rounds,reference", [(1024, 150, "oracle"), (5000, 60, "oracle"), (16384, 25, "general kernel")])
def test_large_pool_kernel_full_ring(oracle_mod, tg, cap, rounds, reference):
    import paper_2605_24259_amd as rkc
    rng = np.random.default_rng(cap)
    trace = tg.from_pools([_full_ring_pool(tg, rng, mode, cap, rounds) for mode in range(4)])
    say(f"case full request ring {cap}")
    if reference == "oracle":
        ref = oracle_mod.replay(trace.desc, trace.events, trace.n_claim_slots, threads=16)
    else:
        ref = gpu_replay(trace, flags=rkc.FLAG_GENERAL_KERNEL)
    assert (ref[1][:, 31] == 1).all()  # each table overflowed once full
    assert ref[1][3, 33] == 1          # the deferred request was served late
    compare_pools(trace, _big(trace, max_live_requests=cap), ref)


# its claim list past the 256 claims kept in LDS, and long lists of both kinds
@pytest.mark.parametrize("claim_cap", [256, 257, 900])
def test_large_pool_kernel_claim_list(oracle_mod, claim_cap):
    trace = randtrace.many_claims_batch(55, 64, n_events=(900, 2500), claim_cap=claim_cap, n_chains=80,
                                        claim_share=0.6, release_share=0.06)
    say(f"case claim list {claim_cap}")
    ora = oracle_mod.replay(trace.desc, trace.events, trace.n_claim_slots, threads=16)
    assert claim_cap < 900 or ora[1][:, 30].max() > 320
    compare_pools(trace, _big(trace, max_live_requests=4096), ora)


def test_large_pool_kernel_long_lists(oracle_mod, tg):
    from tests.test_gpu_group import long_list_pools
    trace = long_list_pools(tg, 103, 8)
    say("case large-pool long lists")
    ora = oracle_mod.replay(trace.desc, trace.events, trace.n_claim_slots, threads=16)
    compare_pools(trace, gpu_replay(trace), ora)


# the edges of its encoding: 2^20 - 1 blocks and 65,536 events go there, one more of either does not; against
# the oracle where that replays the batch in seconds, else against the general kernel
@pytest.mark.parametrize("usable,events,large_pool,reference", [
    ((1 << 20) - 1, 65536, True, "general kernel"), ((1 << 20) - 1, 100, True, "oracle"), (1 << 20, 100, False, "oracle"),
    (300, 65536, True, "oracle"), (300, 65537, False, "oracle")])
def test_large_pool_kernel_limits(oracle_mod, tg, usable, events, large_pool, reference):
    import paper_2605_24259_amd as rkc
    sel = [(i * 2654435761) & 0x7FFFFFFF for i in range(events)]
    evs = []
    for i in range(events):
        k = i % 16
        if i == events - 1:
            evs.append(tg.prefill(usable // 2, 255, usable // 2))
        elif k in (0, 5, 10):
            evs.append(tg.prefill(1 + sel[i] % (usable // 3), sel[i] % 256, (1 + sel[i] % (usable // 3)) // 2))
        elif k in (3, 8):
            evs.append(tg.claim(1 + sel[i] % (usable // 5), sel[i] % 256, hard=i & 1, prio=i & 3, dur=sel[i] % 65536))
        elif k == 12:
            evs.append(tg.release(sel[i]))
        elif k in (4, 14):
            evs.append(tg.finish(sel[i]))
        else:
            evs.append(tg.extend(1 + sel[i] % 50, sel[i]))
    trace = tg.from_pools([dict(usable_blocks=usable, mode=m, n_chains=256, max_live_requests=9000, max_live_claims=300,
                                events=evs) for m in range(4)])
    say(f"case large-pool limits {usable} {events}")
    assert large_pool_route(trace, trace.limits()) == large_pool
    got = gpu_replay(trace)
    assert not (got[1][:, 31] & ~7).any()
    if reference == "oracle":
        ref = oracle_mod.replay(trace.desc, trace.events, trace.n_claim_slots, threads=16)
    else:
        ref = gpu_replay(trace, flags=rkc.FLAG_GENERAL_KERNEL)
    compare_pools(trace, got, ref)


# the compact kernel's layout for few pools at its largest batch and one pool past it, per claim-set
# and key-group instantiation
@pytest.mark.parametrize("n_pools", [4096, 4097])
@pytest.mark.parametrize("n_chains,claims", [(3, 64), (100, 64), (3, 256), (100, 256)])
def test_few_pools_layout(oracle_mod, n_pools, n_chains, claims):
    import paper_2605_24259_amd as rkc
    trace = randtrace.random_batch(77, n_pools, U_range=(4, 60), n_events=(3, 70), n_chains=n_chains, tight_every=9,
                                   caps=(70, claims), defer=True, hard_share=0.4)
    say(f"case few pools {n_pools} {n_chains} {claims}")
    ora = oracle_mod.replay(trace.desc, trace.events, trace.n_claim_slots, threads=16)
    compare_pools(trace, gpu_replay(trace), ora)


# its nodes past the 256 in LDS, and its request list at 256 entries
def test_few_pools_layout_past_lds(oracle_mod):
    trace = randtrace.many_requests_batch(23, 40, n_events=(4000, 6000), n_chains=250)
    say("case few pools past LDS")
    ora = oracle_mod.replay(trace.desc, trace.events, trace.n_claim_slots, threads=16)
    compare_pools(trace, gpu_replay(trace), ora)


# claims that can never fit, with footprints past 16 bits and up to the largest valid one: lead_end of their
# records is the chain's length, whole, in every kernel and layout (claim sets, key groups, few pools and many)
@pytest.mark.parametrize("kernel", ["compact", "two events", "large-pool", "general"])
@pytest.mark.parametrize("n_pools,n_chains,claims", [(48, 8, 64), (48, 8, 256), (48, 130, 64), (48, 130, 256),
                                                     (4100, 8, 64), (4100, 100, 64), (4100, 130, 64), (4100, 8, 256),
                                                     (4100, 100, 256), (4100, 130, 256)])
def test_footprints_past_16_bits(oracle_mod, tg, kernel, n_pools, n_chains, claims):
    import paper_2605_24259_amd as rkc
    sizes = (65535, 65536, 65539, 65546, 131072 + 4, 1 << 24)
    pools = []
    for i in range(48):
        c, pick = (7 * i) % n_chains, sizes[i % len(sizes):] + sizes[:i % len(sizes)]
        evs = [tg.claim(10 + i % 3, c, 10, hard=1)] + [tg.claim(L, c, L - j % 2, hard=j & 1, prio=j & 3)
                                                       for j, L in enumerate(3 * pick)]
        pools.append(dict(usable_blocks=20 + i, mode=i % 4, n_chains=n_chains, max_live_requests=4,
                          max_live_claims=claims, events=evs[:2] if kernel == "two events" else evs))
    base = tg.from_pools(pools)
    say(f"case footprints past 16 bits: {kernel} {n_pools} {n_chains} {claims}")
    ora = oracle_mod.replay(base.desc, base.events, base.n_claim_slots, threads=16)
    assert (ora[0][:, 0] & 255 == 4).sum() >= 48  # MATFAIL
    assert set(ora[2][:, 9]) == {10, 11, 12}
    trace = tile(base, n_pools)
    got = _big(trace) if kernel == "large-pool" else gpu_replay(trace, rkc.FLAG_GENERAL_KERNEL if kernel == "general" else 0)
    compare_tiled(got, ora)


# one claim set over one, two and four key groups with deferral, relaxation and offload, in both layouts
@pytest.mark.parametrize("n_pools", [200, 4100])
@pytest.mark.parametrize("n_chains", [60, 128, 256])
def test_relaxation_over_key_groups(oracle_mod, n_chains, n_pools):
    base = randtrace.random_batch(600 + n_chains, 200, U_range=(40, 400), n_events=(100, 300), n_chains=n_chains,
                                  tight_every=9, caps=(256, 64), defer=True, relax=True, offload=True, hard_share=0.8)
    say(f"case relaxation over {n_chains} chains: {n_pools} pools")
    ora = oracle_mod.replay(base.desc, base.events, base.n_claim_slots, threads=16)
    assert ora[1][:, 36].sum() > 100 and ora[1][:, 38].sum() > 50  # relaxed requests, offloaded claims
    compare_tiled(gpu_replay(tile(base, n_pools)), ora)


# a batch that is faster on the general kernel, but fits the built-in scratch on the large-pool one only
def test_builtin_scratch_of_many_large_tables(oracle_mod):
    import paper_2605_24259_amd as rkc
    base = randtrace.random_batch(88, 150, U_range=(40, 300), n_events=(20, 64), n_chains=16, tight_every=9, caps=(256, 64),
                                  defer=True, hard_share=0.5)
    trace = tile(base, 513)
    lim = dict(trace.limits(), max_usable_blocks=40000, max_chains=256, max_live_requests=4097, max_live_claims=2500)
    say("case built-in scratch of many large tables")
    assert not large_pool_route(trace, lim)
    db = rkc.DeviceBatch(trace.desc, trace.events, trace.n_claim_slots, lim, scratch=False)
    assert db.scratch_needed > rkc.NOALLOC_SCRATCH_BYTES
    ora = oracle_mod.replay(base.desc, base.events, base.n_claim_slots, threads=16)
    compare_tiled(db.replay_noalloc().results(), ora)
