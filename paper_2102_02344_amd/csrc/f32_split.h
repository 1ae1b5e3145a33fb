// An fp32 value as the exact sum of three bf16 ones (see gemm_f32.hip).
#pragma once
#include "common.h"

namespace hfta {

constexpr uint32_t F32_TINY = (27u << 24) - 1;             // 2 * bits - 1 of 2^-100: smaller (but zero) is not split

// Four values as three planes of four bf16.  `chk` becomes NaN if one has no finite remainder; `low` holds the smallest
// magnitude but zero, as 2 * bits - 1 of the value itself: zero wraps to the largest, and what its first part rounds to
// zero (below 2^-134) does not look like one.
typedef __bf16 f32s_bf16x2 __attribute__((ext_vector_type(2)));
struct SplitSeen {
  float chk = 0.f;
  uint32_t low = 0xffffffffu;
  __device__ __forceinline__ bool bad() const { return chk != chk || low < F32_TINY; }
};
// the rounded pair; x and y become what it leaves (exact: a two-element dot product with -1 and 0)
__device__ __forceinline__ uint32_t split_pair(float& x, float& y) {
  const uint32_t w = pack_bf16x2(x, y);
  const f32s_bf16x2 h = __builtin_bit_cast(f32s_bf16x2, w);
  uint32_t cx, cy;
  asm("s_mov_b32 %0, 0xbf80" : "=s"(cx));
  asm("s_mov_b32 %0, 0xbf800000" : "=s"(cy));
  x = __builtin_amdgcn_fdot2_f32_bf16(h, __builtin_bit_cast(f32s_bf16x2, cx), x, false);
  y = __builtin_amdgcn_fdot2_f32_bf16(h, __builtin_bit_cast(f32s_bf16x2, cy), y, false);
  return w;
}
__device__ __forceinline__ void split4(const float4& v, uint2 (&o)[3], SplitSeen& seen) {
  float e[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) seen.low = min(seen.low, __float_as_uint(e[i]) * 2u - 1u);
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    o[q].x = split_pair(e[0], e[1]);
    o[q].y = split_pair(e[2], e[3]);
  }
  o[2].x = pack_bf16x2(e[0], e[1]);
  o[2].y = pack_bf16x2(e[2], e[3]);
  const f32s_bf16x2 ones = __builtin_bit_cast(f32s_bf16x2, 0x3f803f80u);
#pragma unroll
  for (int i = 0; i < 2; ++i)
    seen.chk = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(f32s_bf16x2, i ? o[2].y : o[2].x), ones, seen.chk, false);
}

}  // namespace hfta
