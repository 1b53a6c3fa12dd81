"""The lane-per-pool replay of short traces, compiled for the host, against the oracle: every form of
pool that the rule for it accepts (policies, malformed events, full tables, deferral, relaxation,
offload, bad descriptors), at every event count up to its limit."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from tests import randtrace

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = r"""
#include "rkc_tiny.h"
extern "C" void tiny_replay(int e, int n, const rkc_tiny_limits* g, const rkc_pool_desc* d, const rkc_event* ev,
                            rkc_outcome* o, rkc_pool_telemetry* p, rkc_claim_telemetry* c) {
  for (int i = 0; i < n; i++) {
    if (e == 2) rkc_tiny_pool<2>(*g, d[i], ev, o, p + i, c);
    else rkc_tiny_pool<4>(*g, d[i], ev, o, p + i, c);
  }
}
extern "C" int tiny_serves(int n_pools, int max_events, int max_slots) {
  return rkc_tiny_serves(n_pools, max_events, max_slots);
}
"""


class Limits(ctypes.Structure):
    _fields_ = [("n_events_total", ctypes.c_int64), ("n_slots_total", ctypes.c_int64)] + [
        (k, ctypes.c_int32) for k in ("usable", "events", "chains", "reqs", "claims", "slots")]


@pytest.fixture(scope="module")
def host_lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("tiny")
    src, lib = d / "tiny.cpp", d / "libtiny.so"
    src.write_text(SOURCE)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Wno-unknown-pragmas", "-fsanitize=undefined",
                           "-fno-sanitize-recover", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"), "-I",
                           os.path.join(ROOT, "paper_2605_24259_amd", "csrc"), str(src), "-o", str(lib)])
    return ctypes.CDLL(str(lib))


def host_replay(lib, trace, e):
    L = trace.limits()
    g = Limits(trace.n_events, trace.n_claim_slots, L["max_usable_blocks"], L["max_events"], L["max_chains"],
               L["max_live_requests"], L["max_live_claims"], L["max_claim_slots"])
    out = np.full((max(trace.n_events, 1), 4), 77, np.int32)
    pt = np.full((trace.n_pools, 64), 77, np.int32)
    ct = np.full((max(trace.n_claim_slots, 1), 10), 77, np.int32)
    desc, ev = np.ascontiguousarray(trace.desc), np.ascontiguousarray(trace.events)
    lib.tiny_replay(e, trace.n_pools, ctypes.byref(g), *(ctypes.c_void_p(a.ctypes.data) for a in (desc, ev, out, pt, ct)))
    return out[: trace.n_events], pt, ct[: trace.n_claim_slots]


@pytest.mark.parametrize("e", [2, 4])
@pytest.mark.parametrize("kw", [
    dict(),
    dict(defer=True, hard_share=0.8),
    dict(relax=True, hard_share=0.8),
    dict(relax=True, offload=True, hard_share=0.9),
    dict(relax=True, offload=True, defer=True, hard_share=0.9),
], ids=["plain", "defer", "relax", "offload", "all"])
def test_tiny_replay_matches_oracle(oracle_mod, host_lib, e, kw):
    trace = randtrace.random_batch(1000 + e, 12000, U_range=(2, 14), n_events=(1, e), **kw)
    ora = oracle_mod.replay(trace.desc, trace.events, trace.n_claim_slots, threads=8)
    got = host_replay(host_lib, trace, e)
    for g, o, name in zip(got, ora[:3], ("outcomes", "pool telemetry", "claim telemetry")):
        bad = np.nonzero((g != o).any(1))[0]
        assert bad.size == 0, f"{name}: row {bad[0]}: {g[bad[0]].tolist()} oracle {o[bad[0]].tolist()}"


def test_tiny_replay_of_the_capacity_sweep(oracle_mod, host_lib, tg):
    trace = tg.sweep(residents=(1, 40, 64, 200), actives=(1, 63, 130, 256), usables=tuple(range(1, 400, 7)))
    ora = oracle_mod.replay(trace.desc, trace.events, trace.n_claim_slots, threads=8)
    for g, o in zip(host_replay(host_lib, trace, 2), ora[:3]):
        assert np.array_equal(g, o)


# a lane replays its pools' event types in turn: batches that are resident as wavefronts all at once are
# faster that way (64 pools of two mixed events 6.4 us, by lane 10 us)
@pytest.mark.parametrize("n_pools,events,slots,lane", [
    (1, 2, 8, 0), (64, 2, 8, 0), (4096, 2, 8, 0), (4097, 2, 8, 1), (131072, 1, 1, 1), (4097, 2, 9, 0),
    (4097, 3, 8, 0), (49151, 4, 8, 0), (49152, 3, 8, 1), (49152, 4, 8, 1), (49152, 5, 8, 0)])
def test_batches_of_the_lane_per_pool_replay(host_lib, n_pools, events, slots, lane):
    assert host_lib.tiny_serves(n_pools, events, slots) == lane
