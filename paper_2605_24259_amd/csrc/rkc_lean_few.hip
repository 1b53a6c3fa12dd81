// rkc_lean_few.hip -- the compact kernel's instantiations for few pools (all resident at once, so that a
// pool's latency is the time): rkc_lean.hip with FEW set, built as a file of its own to build in parallel.
#define RKC_LEAN_FEW
#include "rkc_lean.hip"
