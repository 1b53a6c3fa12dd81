// rkc_tiny.hip -- launch of the lane-per-pool replay of short traces (rkc_tiny.h).
#include <hip/hip_runtime.h>

#include "rkc_lean.h"
#include "rkc_tiny.h"

namespace {

// Bound by latency and by the records' scattered stores: 131,072 pools x 2 events are 2,048 waves, two
// per SIMD, each one chain of descriptor load, event load, replay, stores; 19.6 us for the 56 MB a
// pass reads and writes, 11 us of it at the copy rate.
template <int E>
__global__ __launch_bounds__(64) void rkc_tiny_replay(rkc_tiny_limits g, int n_pools, const rkc_pool_desc* pools,
                                                      const rkc_event* events, rkc_outcome* outcomes,
                                                      rkc_pool_telemetry* tel, rkc_claim_telemetry* claims) {
  const int p = (int)(blockIdx.x * 64 + threadIdx.x);
  if (p >= n_pools) return;
  const rkc_pool_desc d = pools[p];
  rkc_tiny_pool<E>(g, d, events, outcomes, tel + p, claims);
}

template <int E>
rkc_status launch(const rkc_lean_args* a, hipStream_t s) {
  const rkc_tiny_limits g = {a->n_events_total, a->n_slots_total, a->max_usable, a->max_events, a->max_chains,
                             a->max_reqs, a->max_claims, a->max_slots};
  hipLaunchKernelGGL(rkc_tiny_replay<E>, dim3((unsigned)(((uint64_t)a->n_pools + 63) / 64)), dim3(64), 0, s, g, (int)a->n_pools,
                     a->pools, a->events, a->outcomes, a->pool_tel, a->claim_tel);
  return hipGetLastError() == hipSuccess ? RKC_OK : RKC_E_HIP;
}

}  // namespace

bool rkc_tiny_fits(const rkc_lean_args* a) { return rkc_tiny_serves(a->n_pools, a->max_events, a->max_slots); }

rkc_status rkc_tiny_launch(const rkc_lean_args* a, hipStream_t s) {
  return a->max_events <= 2 ? launch<2>(a, s) : launch<4>(a, s);
}
