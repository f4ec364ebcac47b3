// Waves of 64 lanes on the CPU, for tests of wave-synchronous device code: every lane is a fiber, and the
// lanes of a wave meet at each cross-lane operation (ballot, shuffle, readlane).  What the device code relies on holds
// here too: between two such operations the lanes of a wave share no data.  Waves take turns at random places, at
// every cross-lane operation and wherever a lane looks at the clock or sleeps, so that an order of events that is rare
// on the GPU is ordinary here.  Everything runs on one thread: atomics are plain accesses.  x86-64 only.
#pragma once
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>

#include <algorithm>
#include <vector>

#define __HIPCC_RTC__ 1
#define __device__
#define __host__
#define __global__
#define __shared__
#define __forceinline__ inline
#define __launch_bounds__(...)

using std::max;
using std::min;
struct alignas(16) uint4 { uint32_t x, y, z, w; };
inline uint4 make_uint4(uint32_t x, uint32_t y, uint32_t z, uint32_t w) { return uint4{x, y, z, w}; }

extern "C" void hw_switch(void** save, void* load);
asm(R"(
.text
.globl hw_switch
hw_switch:
  pushq %rbp
  pushq %rbx
  pushq %r12
  pushq %r13
  pushq %r14
  pushq %r15
  movq %rsp, (%rdi)
  movq %rsi, %rsp
  popq %r15
  popq %r14
  popq %r13
  popq %r12
  popq %rbx
  popq %rbp
  ret
)");

namespace hw {
constexpr size_t STACK = 64 * 1024;
struct Lane {
  void* sp = nullptr;
  enum { READY, MET, DONE } state = READY;
  uint32_t round = 0;      // cross-lane operations so far
};
struct Wave {
  Lane lane[64];
  uint64_t post[2][64];    // what the lanes brought to the last two cross-lane operations
  uint32_t id = 0, next = 0;
  long long clock = 0;     // the same for all lanes until they meet again
  bool done = false;
  char* lds = nullptr;
};
struct World {
  std::vector<Wave> waves;
  void* main_sp = nullptr;
  Wave* w = nullptr;
  uint32_t l = 0;
  bool yielded = false;
  uint64_t turns = 0, rng = 1;
  uint32_t slow_every = 0;   // wave 0 gets one in so many of its turns only (0: all of them)
  void (*body)(uint32_t wave, char* lds) = nullptr;
};
inline World& world() { static World g; return g; }
inline uint32_t random_u32() {
  uint64_t& s = world().rng;
  s ^= s << 13; s ^= s >> 7; s ^= s << 17;
  return (uint32_t)(s >> 32);
}
inline void back_to_main() { World& g = world(); hw_switch(&g.w->lane[g.l].sp, g.main_sp); }
inline void yield() { world().yielded = true; back_to_main(); }
// All lanes of the wave bring a value; the array of all of them.
inline const uint64_t* meet(uint64_t v) {
  World& g = world();
  Wave* w = g.w;
  Lane& me = w->lane[g.l];
  const uint32_t r = me.round++ & 1;
  w->post[r][g.l] = v;
  me.state = Lane::MET;
  back_to_main();
  return w->post[r];
}
inline void entry() {
  World& g = world();
  g.body(g.w->id, g.w->lds);
  g.w->lane[g.l].state = Lane::DONE;
  back_to_main();
  abort();
}
// Runs `body` in n waves with lds_bytes of LDS each; false if it took more than max_turns.
inline bool run(uint32_t n, size_t lds_bytes, uint64_t seed, uint64_t max_turns, void (*body)(uint32_t, char*)) {
  World& g = world();
  g.body = body;
  g.rng = seed * 0x9E3779B97F4A7C15ull + 1;
  g.waves.assign(n, Wave());
  char* stacks = (char*)mmap(nullptr, STACK * 64 * (size_t)n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (stacks == MAP_FAILED) abort();
  std::vector<std::vector<uint4>> lds(n, std::vector<uint4>(lds_bytes / 16 + 1));
  for (uint32_t k = 0; k < n; ++k) {
    Wave& w = g.waves[k];
    w.id = k;
    w.lds = (char*)lds[k].data();
    memset(w.lds, 0xA5, lds_bytes);
    for (uint32_t i = 0; i < 64; ++i) {
      void** sp = (void**)(stacks + STACK * (64 * (size_t)k + i + 1));
      *--sp = nullptr;             // (where entry would return to)
      *--sp = (void*)&entry;
      for (int r = 0; r < 6; ++r) *--sp = nullptr;
      w.lane[i].sp = sp;
    }
  }
  uint32_t left = n;
  while (left) {
    if (g.turns > max_turns) return false;
    Wave& w = g.waves[random_u32() % n];
    if (w.done) continue;
    if (w.id == 0 && g.slow_every && left > 1 && random_u32() % g.slow_every) continue;
    g.w = &w;
    for (uint32_t quantum = 1 + random_u32() % 24; quantum && !w.done;) {
      bool gave_way = false;
      for (; w.next < 64; ++w.next) {
        Lane& l = w.lane[w.next];
        if (l.state != Lane::READY) continue;
        g.l = w.next;
        g.yielded = false;
        hw_switch(&g.main_sp, l.sp);
        if (g.yielded) { gave_way = true; break; }
      }
      ++g.turns;
      if (gave_way) break;
      // every lane has met the others (or is done): on they go
      uint32_t met = 0, round = w.lane[0].round;
      for (Lane& l : w.lane) {
        if (l.state == Lane::DONE) continue;
        if (l.round != round) { fprintf(stderr, "lanes of a wave at different cross-lane operations\n"); abort(); }
        l.state = Lane::READY;
        ++met;
      }
      if (met == 0) { w.done = true; --left; }
      else if (met != 64) { fprintf(stderr, "a cross-lane operation without all lanes\n"); abort(); }
      w.next = 0;
      w.clock = (long long)g.turns;
      --quantum;
    }
  }
  munmap(stacks, STACK * 64 * (size_t)n);
  return true;
}
}  // namespace hw

struct ThreadIdx { struct X { operator uint32_t() const { return hw::world().l; } } x; };
struct BlockIdx { struct X { operator uint32_t() const { return hw::world().w->id; } } x, y; };
static ThreadIdx threadIdx;
static BlockIdx blockIdx;
inline unsigned __lane_id() { return hw::world().l; }
inline unsigned long long __ballot(bool v) {
  const uint64_t* p = hw::meet(v);
  unsigned long long m = 0;
  for (int i = 0; i < 64; ++i) m |= (unsigned long long)(p[i] != 0) << i;
  return m;
}
template <typename T> inline T hw_take(const uint64_t* p, uint32_t from) { T v; memcpy(&v, &p[from & 63], sizeof v); return v; }
template <typename T> inline uint64_t hw_bits(T v) { uint64_t b = 0; memcpy(&b, &v, sizeof v); return b; }
template <typename T> inline T __shfl(T v, int from) { return hw_take<T>(hw::meet(hw_bits(v)), (uint32_t)from); }
template <typename T> inline T __shfl_xor(T v, int x) { const uint32_t i = hw::world().l; return hw_take<T>(hw::meet(hw_bits(v)), i ^ (uint32_t)x); }
inline int hw_readlane(int v, int from) { return hw_take<int>(hw::meet(hw_bits(v)), (uint32_t)from); }
inline int hw_readfirstlane(int v) { return hw_readlane(v, 0); }
inline int hw_dpp(int old, int v, int ctrl, int row_mask) {
  const int i = (int)hw::world().l, row = i / 16;
  const uint64_t* p = hw::meet(hw_bits(v));
  if (!((row_mask >> row) & 1)) return old;
  if (ctrl > 0x110 && ctrl < 0x120) { const int from = i % 16 - (ctrl - 0x110); return from < 0 ? old : hw_take<int>(p, (uint32_t)(row * 16 + from)); }
  if (ctrl == 0x142) return row == 0 ? old : hw_take<int>(p, (uint32_t)(row * 16 - 1));
  if (ctrl == 0x143) return row < 2 ? old : hw_take<int>(p, 31u);
  abort();
}
#define __builtin_amdgcn_readlane hw_readlane
#define __builtin_amdgcn_readfirstlane hw_readfirstlane
#define __builtin_amdgcn_update_dpp(old, v, ctrl, row, bank, bound) hw_dpp(old, v, ctrl, row)
#define __builtin_amdgcn_s_sleep(n) hw::yield()
#define __builtin_amdgcn_s_waitcnt(n) ((void)0)
#define __builtin_amdgcn_s_getreg(n) 0
inline long long wall_clock64() { hw::yield(); return hw::world().w->clock; }
inline int __popcll(unsigned long long v) { return __builtin_popcountll(v); }
inline int __ffsll(long long v) { return __builtin_ffsll(v); }
inline int __ffs(int v) { return __builtin_ffs(v); }
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __HIP_MEMORY_SCOPE_WORKGROUP 0
#define __HIP_MEMORY_SCOPE_SYSTEM 0
template <typename T> inline T __hip_atomic_load(const T* p, int, int) { return *(const volatile T*)p; }
template <typename T, typename V> inline void __hip_atomic_store(T* p, V v, int, int) { *(volatile T*)p = (T)v; }
template <typename T, typename V> inline T __hip_atomic_fetch_add(T* p, V v, int, int) { const T o = *p; *p = (T)(o + (T)v); return o; }
template <typename T, typename V> inline T __hip_atomic_fetch_or(T* p, V v, int, int) { const T o = *p; *p = (T)(o | (T)v); return o; }
template <typename T, typename V> inline bool __hip_atomic_compare_exchange_strong(T* p, T* expect, V v, int, int, int) {
  if (*p == *expect) { *p = (T)v; return true; }
  *expect = *p;
  return false;
}
template <typename T, typename V> inline T atomicAdd(T* p, V v) { const T o = *p; *p = (T)(o + (T)v); return o; }
template <typename T, typename V> inline T atomicSub(T* p, V v) { const T o = *p; *p = (T)(o - (T)v); return o; }
template <typename T, typename V> inline T atomicOr(T* p, V v) { const T o = *p; *p = (T)(o | (T)v); return o; }
template <typename T, typename V> inline T atomicMax(T* p, V v) { const T o = *p; *p = max(o, (T)v); return o; }
