// Parts of fp32 values for the 16-bit matrix cores, and the copies that bring
// their operands into LDS (k-means assignment, projection of large batches).
#ifndef DRESD_SPLIT_H
#define DRESD_SPLIT_H

#include "dresd_device.h"

namespace dresd {

typedef uint16_t us8 __attribute__((ext_vector_type(8)));

// Three 16-bit parts of x (f16 when F16, else bf16), each the rounded rest.
template <bool F16>
__device__ __forceinline__ void split3(float x, uint16_t &a, uint16_t &b, uint16_t &c) {
  if constexpr (F16) {
    const _Float16 h = (_Float16)x;
    const float r1 = x - (float)h;
    const _Float16 m = (_Float16)r1;
    const _Float16 l = (_Float16)(r1 - (float)m);
    a = __builtin_bit_cast(uint16_t, h);
    b = __builtin_bit_cast(uint16_t, m);
    c = __builtin_bit_cast(uint16_t, l);
  } else {
    const __bf16 h = (__bf16)x;
    const float r1 = x - (float)h;
    const __bf16 m = (__bf16)r1;
    const __bf16 l = (__bf16)(r1 - (float)m);
    a = __builtin_bit_cast(uint16_t, h);
    b = __builtin_bit_cast(uint16_t, m);
    c = __builtin_bit_cast(uint16_t, l);
  }
}

// Copy 16 bytes per lane into LDS, from base + this lane's offset to lds + 16
// times the lane; see copy1_to_lds.
__device__ __forceinline__ void copy16_to_lds(const void *base, uint32_t off, uint32_t lds) {
  asm volatile(
      "s_mov_b32 m0, %2\n\t"
      "global_load_lds_dwordx4 %0, %1"
      :
      : "v"(off), "s"(base), "s"(lds)
      : "memory");
}

}  // namespace dresd

#endif
