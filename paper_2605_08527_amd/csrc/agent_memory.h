// Waits on the vector-memory counter, and accesses to memory that workgroups of one launch share.
#pragma once
#include "common.h"

namespace marlaas {

// at most N vector-memory requests of this wave are outstanding (requests complete in order)
template <int N>
__device__ __forceinline__ void wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory"); }

// Memory shared between workgroups inside one launch (partial sums, u, counters) is accessed with
// the agent-scope cache policy on the individual instruction (sc1: the access is performed at the
// level all XCDs share), the way relaxed agent-scope atomics are: no write-back or invalidation of
// a whole L2 is needed, which with 256 workgroups costs tens of microseconds.  A store is performed
// once the vector-memory counter has counted it down.
__device__ __forceinline__ void store4_agent(float* p, f32x4 v) {
  asm volatile("global_store_dwordx4 %0, %1, off sc1" :: "v"(p), "v"(v) : "memory");
}
__device__ __forceinline__ void load4_agent(f32x4& v, const float* p) {     // complete after wait_vm<..>()
  asm volatile("global_load_dwordx4 %0, %1, off sc1" : "=v"(v) : "v"(p) : "memory");
}


}  // namespace marlaas
