// rkc_big.h -- internal interface between the C ABI (rkc_replay.hip) and the large-pool replay
// kernel (rkc_big.hip).  Not part of the public ABI.
#ifndef RKC_BIG_H
#define RKC_BIG_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rkc.h"

struct rkc_big_args {
  const rkc_pool_desc* pools;
  const rkc_event* events;
  rkc_outcome* outcomes;
  rkc_pool_telemetry* pool_tel;
  rkc_claim_telemetry* claim_tel;
  void* scratch;
  int64_t n_events_total, n_slots_total;
  int32_t n_pools, max_usable, max_events, max_chains, max_reqs, max_claims, max_slots;
  // layout: request ring entries (a power of two), touch-stack nodes in all and in LDS, LDS and
  // scratch bytes per pool, scratch regions
  uint32_t ring, node_cap, nodes_lds, lds_bytes;
  uint64_t scr_pool_bytes, scr_off_nodes, scr_off_fifo, scr_off_slots, scr_off_defer, scr_off_claims, scr_off_cx;
};

// Fill the layout part of g for batch b; false when b is outside the kernel's limits.
bool rkc_big_layout(const rkc_batch* b, rkc_big_args* g);

// Launch the kernel (one 64-lane workgroup per pool) on stream s.
rkc_status rkc_big_launch(const rkc_big_args* g, hipStream_t s);

#ifdef RKC_CHECK_UNIFORM
unsigned rkc_big_uniform_violations(void);
#endif

#endif
