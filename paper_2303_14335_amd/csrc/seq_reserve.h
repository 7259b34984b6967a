// seq_reserve.h - places in the sequence engine's task table and arena
// (seq_types.h), for the tiers' task kernels.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "seq_types.h"
#include "wave_ops.h"

namespace mpld {

// `bytes` of the arena and `pieces` tasks (maybe none) for this wave; false when there is no
// room for them.  What is refused takes nothing: refused waves come back round
// after round, and counts that went on growing would pass 32 bits, and then be
// taken for room.  (Waves that look at the same time may pass the capacity
// together, once.)  All of the atomics are in one branch, on a lane of its own.
__device__ __forceinline__ bool seq_take_room(const SeqArgs& a, uint64_t bytes, int32_t pieces, int32_t& child,
                                              int64_t& at) {
  const uint64_t used = uniform64(__hip_atomic_load(&a.head->arena, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  const int32_t made =
      (int32_t)uniform((uint32_t)__hip_atomic_load(&a.head->tasks, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  if (used + bytes > (uint64_t)a.arena_cap || (pieces != 0 && made > a.task_cap - pieces)) return false;
  uint64_t p = 0;
  int32_t c = 0;
  if (__lane_id() == 63u) {
    p = atomicAdd(&a.head->arena, (unsigned long long)bytes);
    c = atomicAdd(&a.head->tasks, pieces);
  }
  child = (int32_t)rdlane((uint32_t)c, 63u);
  const uint64_t from = rdlane64((uint32_t)p, (uint32_t)(p >> 32), 63u);
  at = (int64_t)from;
  return from + bytes <= (uint64_t)a.arena_cap && (pieces == 0 || child <= a.task_cap - pieces);
}

}  // namespace mpld
