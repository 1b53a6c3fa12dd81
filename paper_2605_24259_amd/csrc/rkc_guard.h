// rkc_guard.h -- the consistency guard of the kernels that replay a pool by one wavefront.  Plain C++, so
// that it also compiles for the host, where it is tested.
//
// Feasibility is checked before an eviction loop starts and no candidate's run is empty, so every pass takes
// blocks.  A pass that took none (only a wrong build has one) still lowers the blocks left to take, so that the
// loop ends; the blocks it only claims to have taken then count as active and stay counted as evictable, and
// the pool no longer adds up.  That is tested once, when the pool is done: a test in every pass, one
// scalar compare and branch, made the zipf batches 1.4 to 2 % slower (10.09 -> 10.23 ms).
#ifndef RKC_GUARD_H
#define RKC_GUARD_H

#include <stdint.h>

#ifdef __HIPCC__
#define RKC_GUARD_FN __host__ __device__ __forceinline__
#else
#define RKC_GUARD_FN inline
#endif

// Blocks left to take after a pass of an eviction loop that took m of K.
RKC_GUARD_FN uint32_t rkc_left(uint32_t K, uint32_t m) { return K - (m > 1u ? m : 1u); }

// Every usable block is free (F), active (A) or cached, and every cached block is evictable or protected.
RKC_GUARD_FN bool rkc_adds_up(uint32_t U, uint32_t F, uint32_t A, uint32_t cached) { return F + A + cached == U; }

#endif
