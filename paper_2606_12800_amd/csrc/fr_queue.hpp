// Device queue of tiles for persistent kernels: a tile that is woken while
// idle is queued once; any workgroup takes it, works on it alone and lets go
// of it, or, woken meanwhile, looks at it again.  No workgroup waits for
// another to be resident, and every wait ends.
#pragma once

#include "fr_internal.hpp"

namespace fr {

// Tile states (idle: 0).
constexpr uint32_t ST_PENDING = 1, ST_RUNNING = 2, ST_DONE = 4;
// A workgroup without a tile gives up when neither the queue nor the count of
// tiles left has moved over this many of its own looks (0.27 s; a tile in
// another workgroup's hands is done or let go within some 1000).  Looks, not a
// clock's time: while the whole hardware queue is switched out nobody looks.
constexpr uint32_t STUCK_LOOKS = 1u << 19;

__device__ __forceinline__ uint64_t ld64(const uint64_t* p) {
  return (uint64_t)__hip_atomic_load(reinterpret_cast<unsigned long long*>(const_cast<uint64_t*>(p)),
                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st64(uint64_t* p, uint64_t v) {
  __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), (unsigned long long)v, __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t ld32(const uint32_t* p) {
  return __hip_atomic_load(const_cast<uint32_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st32(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The wavefront's stores are complete (device-coherent ones visible).
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Takes a tile from the queue; -1 when no tiles are left (or the work is
// given up).  One lane of a workgroup.
__device__ inline int32_t take_tile(const TileQueue& Q) {
  TileCtl* C = Q.ctl;
  uint32_t ticket = atomicAdd(&C->head, 1u);
  uint32_t last_tail = 0, last_left = 0, since = 0;
  for (uint32_t it = 0;; ++it) {
    const uint64_t w = ld64(Q.ring + ticket % Q.cap);
    const uint32_t at = (uint32_t)(w >> 32);
    if ((uint32_t)w != 0u && at == ticket) {
      const uint32_t t = (uint32_t)w - 1u;
      // Taken (an entry that is overwritten before this is queued again by
      // the workgroup that overwrote it; whoever comes second finds the tile
      // running).
      atomicCAS(reinterpret_cast<unsigned long long*>(Q.ring + ticket % Q.cap), (unsigned long long)w, 0ull);
      if (atomicCAS(Q.state + t, ST_PENDING, ST_RUNNING) == ST_PENDING) return (int32_t)t;
      ticket = atomicAdd(&C->head, 1u);
      continue;
    }
    if ((uint32_t)w != 0u && (int32_t)(at - ticket) > 0) {
      ticket = atomicAdd(&C->head, 1u);
      continue;
    }
    __builtin_amdgcn_s_sleep(8);
    if (it % 4u != 0u) continue;
    const uint32_t left = ld32(&C->left), tail = ld32(&C->tail);
    if (left == 0u || ld32(&C->stop)) return -1;
    if (left != last_left || tail != last_tail) {
      last_left = left;
      last_tail = tail;
      since = it;
    } else if (it - since > STUCK_LOOKS) {
      atomicExch(&C->stop, 1u);
      if (Q.status) atomicCAS(Q.status, 0, Q.stuck);
      return -1;
    }
  }
}

// Puts tile t (just set pending) into the queue.
__device__ __forceinline__ void push_tile(const TileQueue& Q, uint32_t t) {
  for (;;) {
    const uint32_t ticket = atomicAdd(&Q.ctl->tail, 1u);
    const uint64_t old =
        (uint64_t)atomicExch(reinterpret_cast<unsigned long long*>(Q.ring + ticket % Q.cap),
                             ((unsigned long long)ticket << 32) | (t + 1u));
    if ((uint32_t)old == 0u) return;
    t = (uint32_t)old - 1u;  // an entry not taken yet: queue that tile again
  }
}

// The queue's words at the start: `ntiles` tickets given out.
__device__ __forceinline__ void open_queue(const TileQueue& Q, uint32_t ntiles) {
  Q.ctl->head = 0;
  Q.ctl->tail = ntiles;
  Q.ctl->left = ntiles;
  Q.ctl->stop = 0;
}

}  // namespace fr
