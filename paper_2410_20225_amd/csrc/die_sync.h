// Workgroups of one launch that run on the same accelerator die (XCD).
// MI355X hands the workgroups of a launch to its eight dies in turn, so workgroups i, i + 8,
// i + 16, ... share a die and its L2.  Work that is private to a die (the instances dealt to
// one tag machine, and the cells of those instances) can therefore run as a persistent loop in which
// workgroups read what others of the die have written: what has reached the shared L2 is there for all of them, with no L2
// write-back or invalidation and no kernel boundary.  The per-CU L1 is NOT invalidated: such data is read past it, or is
// data the reader's CU cannot hold an older copy of.  The barrier below opens such a launch: it is at device scope, completes
// wherever the workgroups run, and tells all of them whether they share a die; if they do not, they leave.
#pragma once
#ifndef __HIPCC_RTC__
#include <hip/hip_runtime.h>
#endif
#include <stdint.h>

namespace tdf {

constexpr uint32_t XCDS = 8;

struct alignas(128) DieSync {
  uint32_t count;      // arrivals at the barrier
  uint32_t beat;       // counted on by workgroups that get somewhere
  uint32_t xcc_mask;   // dies the workgroups of this group actually ran on
  uint32_t abort;      // a workgroup gave up waiting
  uint32_t at;         // about where the workgroups are (the level launches' level)
};

// HW_REG_XCC_ID (20), bits 3:0: the die this wave runs on
__device__ __forceinline__ uint32_t xcc_id() { return __builtin_amdgcn_s_getreg(20 | (0 << 6) | (3 << 11)) & 15u; }

// The first barrier of a launch, called once by every thread of each of the G workgroups of a group, which have put their
// dies into xcc_mask.  Release: each wave waits until the die's L2 has acknowledged all its outstanding stores (on this
// architecture stores count in vmcnt; the workgroup barrier by itself does not wait for them), then
// the workgroup meets, then one thread announces the arrival.  No L2 write-back is involved.
// Returns false if the wait exceeded spin_ticks (100 MHz ticks) or the workgroups are not on one die: the caller then leaves.
__device__ inline bool die_meet(DieSync* sy, uint32_t G, long long spin_ticks, uint32_t* sh_ok) {
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x == 0) {
    bool ok = true;
    __hip_atomic_fetch_add(&sy->count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    long long t0 = 0;
    for (uint32_t k = 1;; ++k) {
      if (__hip_atomic_load(&sy->count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= G) {
        const uint32_t mask = __hip_atomic_load(&sy->xcc_mask, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        ok = (mask & (mask - 1u)) == 0;
        break;
      }
      __builtin_amdgcn_s_sleep(1);
      if (k % 64u != 0) continue;   // (the clock is read rarely: that takes as long as a look)
      if (t0 == 0) t0 = wall_clock64();
      if (wall_clock64() - t0 > spin_ticks) {
        __hip_atomic_store(&sy->abort, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
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
