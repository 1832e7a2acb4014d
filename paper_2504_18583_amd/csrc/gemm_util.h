// Small device helpers shared by the skinny and the row-block GEMM kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pard {
namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kRsrcWord3 = 0x00020000;   // buffer descriptor word 3 for gfx9-family raw buffers
constexpr int kCachePolicyNT = 2;        // non-temporal: weights are streamed once
constexpr int kWaitVmcnt0 = 0x0F70;      // s_waitcnt vmcnt(0), expcnt and lgkmcnt not waited for

// Sum over the 16 lanes of a DPP row (lanes 16g .. 16g+15), fixed order:
// quad_perm swaps (1 0 3 2), (2 3 0 1), then half-row and row mirrors.
__device__ __forceinline__ float sum16(float x) {
  x += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0xB1, 0xF, 0xF, false));
  x += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x4E, 0xF, 0xF, false));
  x += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x141, 0xF, 0xF, false));
  x += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x140, 0xF, 0xF, false));
  return x;
}

__device__ __forceinline__ bool better(float v, int i, float bv, int bi) {
  return v > bv || (v == bv && i < bi);
}

// The best (value, index) over the 16 lanes of a DPP row, in every lane: the
// same moves as sum16.
template <int CTRL>
__device__ __forceinline__ void best_dpp(float& bv, int& bi) {
  const float ov = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(bv), CTRL, 0xF, 0xF, false));
  const int oi = __builtin_amdgcn_mov_dpp(bi, CTRL, 0xF, 0xF, false);
  if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
}
__device__ __forceinline__ void best16(float& bv, int& bi) {
  best_dpp<0xB1>(bv, bi);
  best_dpp<0x4E>(bv, bi);
  best_dpp<0x141>(bv, bi);
  best_dpp<0x140>(bv, bi);
}

}  // namespace
}  // namespace pard
