// Elements that have not been written yet.  Rows that one workgroup of a level tail writes and others wait for hold all ones until
// then (a value that has this pattern, a NaN, is stored as another one), so whether 16-byte chunks of them are there follows
// from the greatest of their elements.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tdf {

typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;   // one 16-byte chunk

template <typename T> struct Unwritten;
// Two elements a word: one instruction a word.  (The compiler, if it sees the comparison behind the maxima, compares every half.)
template <> struct Unwritten<__bf16> {
  static __device__ __forceinline__ uint32_t greatest(uint32_t m, u32x4 c) {
    typedef __attribute__((ext_vector_type(2))) unsigned short u16x2;
    const uint32_t x = c.x, y = c.y, z = c.z, w = c.w;   // (a bit cast of a vector's component itself is the first one's, whichever it names)
    const u16x2 a = __builtin_elementwise_max(__builtin_bit_cast(u16x2, x), __builtin_bit_cast(u16x2, y));
    const u16x2 b = __builtin_elementwise_max(__builtin_bit_cast(u16x2, z), __builtin_bit_cast(u16x2, w));
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, m), __builtin_elementwise_max(a, b)));
  }
  static __device__ __forceinline__ bool waiting(uint32_t m) {
    asm("" : "+v"(m));
    return ((0xFFFEFFFEu - m) & m & 0x80008000u) != 0;   // (a half of ~m is zero)
  }
};
template <> struct Unwritten<float> {
  static __device__ __forceinline__ uint32_t greatest(uint32_t m, u32x4 c) { return max(max(max(m, c.x), c.y), max(c.z, c.w)); }
  static __device__ __forceinline__ bool waiting(uint32_t m) {
    asm("" : "+v"(m));
    return m == 0xFFFFFFFFu;
  }
};

}  // namespace tdf
