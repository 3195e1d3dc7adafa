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

// Launches that exchange u take turns over two areas, each all zero bits when its turn comes: a launch uses one and
// clears what the launch before it used of the other, so that nobody has to find out who is last through (a count of the
// workgroups, with the answer's trip and the clearing behind it: 256 rows of 4096 x 4096 23.1 us, taking turns 22.5; 300 rows,
// 1024 x 3080, 40 adapters of rank 8, 13.2 and 11.9).  The line is asked for behind a workgroup's operands, which would have to
// wait for it.  (Read with the kernel's first loads instead, a layer's four calls of 157 rows took 194 us, not 190.6: its values
// are in the way of the loop's.)  Few rows, whose u is wanted sooner, keep the count: 6 rows 11.5 us, taking turns 12.2.
// Whose turn it is comes from TURN_LINES lines of {count, floats of u in area 0, in area 1, ...}; workgroup b has
// line b mod TURN_LINES.  Every workgroup adds to its line's count once, when it has read the line, the first to each line so
// much that a launch adds 2^TURN_SHIFT to every line, however few workgroups it has: before its own share is in, a workgroup
// finds the launch's number above.
// Fourth word: number (+ 1) of a launch that must not use the area of partial sums, because somebody gave up waiting in the one
// before it and sums may lie there; it clears the area instead.  All workgroups of that launch have to find the same, however
// late they come (one that did not would take what lies there for sums), so the word stays until the launch after it.
struct Turn {
  uint32_t number; int area;
  int64_t u_before;                  // floats of u in the other area
  bool sums_ok, was_not;             // (this launch's, the one's before it)
};
__device__ __forceinline__ const int32_t* turn_line(const int32_t* turns) { return turns + blockIdx.x % TURN_LINES * 32; }
__device__ __forceinline__ Turn turn_of(uint32_t count, uint32_t u0, uint32_t u1, uint32_t sums) {
  uint32_t c = (uint32_t)__builtin_amdgcn_readfirstlane((int)count), n0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)u0);
  uint32_t n1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)u1), gave = (uint32_t)__builtin_amdgcn_readfirstlane((int)sums);
  // (the line has arrived here, and not where its words are used: a barrier waits for no load from memory)
  asm volatile("" : "+s"(c), "+s"(n0), "+s"(n1), "+s"(gave) :: "memory");
  Turn t;
  t.number = c >> TURN_SHIFT;
  t.area = t.number & 1;
  const uint32_t n = t.area ? n0 : n1;
  t.u_before = n < (uint32_t)MID_U_FLOATS ? n : MID_U_FLOATS;
  // (gave 0: nobody ever gave up)
  t.sums_ok = gave != t.number + 1;
  t.was_not = gave == ((t.number - 1) & (~0u >> TURN_SHIFT)) + 1;
  return t;
}
// Once for every workgroup, by one lane, behind a barrier that every wave which reads the line meets with its Turn in hand: one
// that read after the launch's last share would find the next launch's number.  u_floats: what the launch may use of its area.
__device__ __forceinline__ void turn_over(int32_t* turns, const Turn& t, int64_t u_floats) {
  uint32_t line = blockIdx.x % TURN_LINES;
  if (blockIdx.x >= TURN_LINES) {
    (void)__hip_atomic_fetch_add((uint32_t*)turns + line * 32, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return;
  }
  // the first to its line, and the first of all to the lines that a small launch has nobody for
  do {
    uint32_t* l = (uint32_t*)turns + line * 32;
    const uint32_t others = line < gridDim.x ? (gridDim.x - line - 1) / TURN_LINES : 0;
    __hip_atomic_store(l + 1 + t.area, (uint32_t)u_floats, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // done with, or the number would come round; whoever gives up in this launch may have put the next one's there
    if (t.was_not) {
      uint32_t old = ((t.number - 1) & (~0u >> TURN_SHIFT)) + 1;
      (void)__hip_atomic_compare_exchange_strong(l + 3, &old, 0u, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    (void)__hip_atomic_fetch_add(l, (1u << TURN_SHIFT) - others, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    line = line == 0 ? gridDim.x : line + 1;
  } while (blockIdx.x == 0 && line < TURN_LINES);
}
// The same for a workgroup without any other business; all its waves call it.
__device__ __forceinline__ Turn turn_missed(int32_t* turns, int64_t u_floats, bool one) {
  const int4 l = *(const int4*)turn_line(turns);
  const Turn t = turn_of(l.x, l.y, l.z, l.w);
  __syncthreads();
  if (one) turn_over(turns, t, u_floats);
  return t;
}
// Somebody gave up waiting for sums: the next launch leaves their area alone.
__device__ __forceinline__ void turn_gave_up(int32_t* turns, uint32_t number, int lane) {
  if (lane < TURN_LINES) __hip_atomic_store((uint32_t*)turns + lane * 32 + 3, ((number + 1) & (~0u >> TURN_SHIFT)) + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Part `part` of `parts` (workgroups) of n floats, cleared by a workgroup's threads, the last ones first (n a multiple of 4).
__device__ __forceinline__ void clear_share(float* p, int64_t n, int64_t part, int64_t parts) {
  for (int64_t i = (part * blockDim.x + (blockDim.x - 1 - threadIdx.x)) * 4; i < n; i += parts * blockDim.x * 4) store4_agent(p + i, f32x4{0.f, 0.f, 0.f, 0.f});
}

}  // namespace marlaas
