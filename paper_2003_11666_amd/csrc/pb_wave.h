// Wavefront reductions shared by the kernels of the tick engine.
#pragma once
#include <hip/hip_runtime.h>

namespace pb {

// Cross-lane operand through the data-parallel-primitive path of the vector
// ALU (no LDS round trip): lanes without a source, or in rows masked out,
// read 0.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_src(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROW_MASK, 0xF, false));
}

// Sum over the wavefront, returned to every lane (fixed order).
__device__ __forceinline__ float wave_sum(float v) {
  v += dpp_src<0xB1, 0xF>(v);    // quad_perm [1,0,3,2]
  v += dpp_src<0x4E, 0xF>(v);    // quad_perm [2,3,0,1]
  v += dpp_src<0x141, 0xF>(v);   // row_half_mirror
  v += dpp_src<0x140, 0xF>(v);   // row_mirror: every lane holds the sum of its row of 16
  v += dpp_src<0x142, 0xA>(v);   // row_bcast:15 into rows 1 and 3
  v += dpp_src<0x143, 0xC>(v);   // row_bcast:31 into rows 2 and 3: lane 63 holds the total
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// Sum over each row of 16 lanes, returned to every lane of the row (fixed order).
__device__ __forceinline__ float row_sum(float v) {
  v += dpp_src<0xB1, 0xF>(v);    // quad_perm [1,0,3,2]
  v += dpp_src<0x4E, 0xF>(v);    // quad_perm [2,3,0,1]
  v += dpp_src<0x141, 0xF>(v);   // row_half_mirror
  v += dpp_src<0x140, 0xF>(v);   // row_mirror
  return v;
}

// Maximum over the wavefront, returned to every lane, without LDS: lanes without a source keep their own value.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_or_self(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), CTRL, ROW_MASK, 0xF, false));
}
__device__ __forceinline__ float wave_max_dpp(float v) {
  v = fmaxf(v, dpp_or_self<0xB1, 0xF>(v));
  v = fmaxf(v, dpp_or_self<0x4E, 0xF>(v));
  v = fmaxf(v, dpp_or_self<0x141, 0xF>(v));
  v = fmaxf(v, dpp_or_self<0x140, 0xF>(v));
  v = fmaxf(v, dpp_or_self<0x142, 0xA>(v));
  v = fmaxf(v, dpp_or_self<0x143, 0xC>(v));
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

}  // namespace pb
