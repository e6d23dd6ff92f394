// Device helpers of the kernels that keep fp32 sums as 16-bit hi / lo operands.
#pragma once
#include <hip/hip_runtime.h>

#include "band_common.h"

namespace spider_impl {

// Split two consecutive fp32 values into packed 16-bit words hi = rnd(x) and
// lo = rnd(x - hi) (x - hi is exact in fp32).
template <int OP, bool XLO>
__device__ __forceinline__ void split2(uint32_t a, uint32_t b, uint32_t* hi, uint32_t* lo) {
  const float fa = __builtin_bit_cast(float, a), fb = __builtin_bit_cast(float, b);
  *hi = pack2<OP>(fa, fb);
  if constexpr (XLO) {
    const f32x2 h = unpack2<OP>(*hi);
    *lo = pack2<OP>(fa - h.x, fb - h.y);
  } else {
    *lo = 0u;
  }
}

// Store 4 fp32 outputs; the line resource drops whatever lies outside [0, nx).
template <bool ALIGNED>
__device__ __forceinline__ void store_f32x4(__amdgpu_buffer_rsrc_t rs, uint32_t voff, f32x4 v) {
  if constexpr (ALIGNED) {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rs, voff, 0, kStoreNT);
  } else {
    // Cast the whole vector: element-wise bit casts of a float vector feeding these
    // stores have been seen to compile to four stores of element 0.
    const u32x4 u = __builtin_bit_cast(u32x4, v);
#pragma unroll
    for (int t = 0; t < 4; ++t) __builtin_amdgcn_raw_buffer_store_b32(u[t], rs, voff + 4 * t, 0, 0);
  }
}

}  // namespace spider_impl
