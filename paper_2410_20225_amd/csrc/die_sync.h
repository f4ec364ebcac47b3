// Barrier among the workgroups of one launch that run on the same accelerator die (XCD).
// MI355X hands the workgroups of a launch to its eight dies in turn, so workgroups i, i + 8,
// i + 16, ... share a die and its L2.  Work that is private to a die (the instances dealt to
// one tag machine, and the cells of those instances) can therefore run as a persistent loop
// with this barrier between dependent phases: every wave drains its stores into the shared L2
// before its workgroup arrives (s_waitcnt vmcnt(0)), so no L2 write-back or invalidation and no
// kernel boundary is needed.  The per-CU L1 is NOT
// invalidated: what crosses the barrier must be data the consumer's CU cannot hold an older copy
// of (rows written once per launch and read only afterwards), or be read past the L1.  The first
// barrier of a launch is at device scope, completes wherever the workgroups run, and tells all of them whether they
// share a die; if they do not, they leave.  The later ones count in the die's L2 (atomics are performed there, also the
// one that looks at the count), which takes a third of a round trip through memory.  Every wait is bounded.
// A barrier of 32 workgroups costs about 1 us; with device-scope words and a second one for giving up it was 2.5.
#pragma once
#ifndef __HIPCC_RTC__
#include <hip/hip_runtime.h>
#endif
#include <stdint.h>

namespace tdf {

constexpr uint32_t XCDS = 8;

struct alignas(128) DieSync {
  uint32_t count;      // arrivals at the first barrier
  uint32_t pad;
  uint32_t xcc_mask;   // dies the workgroups of this group actually ran on
  uint32_t abort;      // a workgroup gave up waiting
  alignas(128) uint32_t local;   // arrivals at the later barriers (monotone: G per barrier), and DIE_GAVE_UP
};
constexpr uint32_t DIE_GAVE_UP = 0x80000000u;   // (arrivals stay below: at most 2^25 levels of at most 32 workgroups)

// HW_REG_XCC_ID (20), bits 3:0: the die this wave runs on
__device__ __forceinline__ uint32_t xcc_id() { return __builtin_amdgcn_s_getreg(20 | (0 << 6) | (3 << 11)) & 15u; }

// A barrier in two halves, each called by every thread of each of the G workgroups of a group; `gen` counts the
// group's barriers so far (all workgroups pass the same value).  What lies between the halves overlaps the wait: loads of
// data that no workgroup of the group writes.
// Release: each wave waits until the die's L2 has acknowledged all its outstanding stores (on this
// architecture stores count in vmcnt; the workgroup barrier by itself does not wait for them), then
// the workgroup meets, then one thread announces the arrival.  No L2 write-back is involved.
__device__ __forceinline__ void die_arrive(DieSync* sy, uint32_t gen) {
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x == 0) {   // without waiting for the old value
    if (gen == 0) __hip_atomic_fetch_add(&sy->count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else __hip_atomic_fetch_add(&sy->local, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
}
// Returns false if the wait exceeded spin_ticks (100 MHz ticks), another workgroup had given up, or the workgroups
// are not on one die: the caller then leaves.
__device__ inline bool die_wait(DieSync* sy, uint32_t G, uint32_t gen, long long spin_ticks, uint32_t* sh_ok) {
  if (threadIdx.x == 0) {
    bool ok = true;
    uint32_t nothing = 0;
    asm volatile("" : "+s"(nothing));   // (an atomic that adds nothing, not a load, which the L1 could answer)
    long long t0 = 0;
    for (uint32_t k = 1;; ++k) {
      if (gen == 0) {
        if (__hip_atomic_load(&sy->count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= G) {
          const uint32_t mask = __hip_atomic_load(&sy->xcc_mask, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          ok = (mask & (mask - 1u)) == 0;
          break;
        }
      } else {
        const uint32_t v = __hip_atomic_fetch_add(&sy->local, nothing, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (v >= gen * G) {
          ok = v < DIE_GAVE_UP;
          break;
        }
      }
      __builtin_amdgcn_s_sleep(1);
      if (k % 64u != 0) continue;   // (the clock is read rarely: that takes as long as a look)
      if (t0 == 0) t0 = wall_clock64();
      if (wall_clock64() - t0 > spin_ticks) {
        __hip_atomic_store(&sy->abort, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_fetch_or(&sy->local, DIE_GAVE_UP, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        ok = false;
        break;
      }
    }
    *sh_ok = ok ? 1u : 0u;
  }
  __syncthreads();
  return *sh_ok != 0;
}

}  // namespace tdf
