// Operands of the FP4 / FP8 matrix instruction and wave reductions, shared by the decode kernels.
#pragma once
#include "rkv_internal.h"

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ v4f mfma_fp4(const v8i& a, const v8i& b, const v4f& c) {
  return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c, 4, 4, 0, 0, 0, 0);
}
__device__ __forceinline__ v4f mfma_fp8_fp4(const v8i& a, const v8i& b, const v4f& c) {
  return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c, 0, 4, 0, 0, 0, 0);
}

// two dwords of 2-bit codes -> four dwords of FP4 nibbles (value = code / 2)
__device__ __forceinline__ v8i unpack_fp4(uint32_t d0, uint32_t d1) {
  v8i r;
  r[0] = (int)(d0 & 0x33333333u);
  r[1] = (int)((d0 >> 2) & 0x33333333u);
  r[2] = (int)(d1 & 0x33333333u);
  r[3] = (int)((d1 >> 2) & 0x33333333u);
  r[4] = r[5] = r[6] = r[7] = 0;
  return r;
}

// one dword of third bits (3-bit codes; bit 4j + k belongs to nibble j of operand dword k) -> four
// dwords of FP4 nibbles (value = bit / 2)
__device__ __forceinline__ v8i unpack_fp4_bits(uint32_t h) {
  v8i r;
  r[0] = (int)(h & 0x11111111u);
  r[1] = (int)((h >> 1) & 0x11111111u);
  r[2] = (int)((h >> 2) & 0x11111111u);
  r[3] = (int)((h >> 3) & 0x11111111u);
  r[4] = r[5] = r[6] = r[7] = 0;
  return r;
}

template <int CTRL>
__device__ __forceinline__ float dpp_f(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}
#define DPP_ROW_MIRROR 0x140
#define DPP_ROW_HALF_MIRROR 0x141
#define DPP_QUAD_MIRROR 0x1B      // quad_perm [3,2,1,0]
#define DPP_QUAD_SWAP 0xB1        // quad_perm [1,0,3,2]

// All-lanes reduction over the 64 lanes of a wave: 4 DPP steps inside each row of 16, then the
// four row results through scalar registers.
template <bool IS_MAX>
__device__ __forceinline__ float wave_allreduce(float x) {
  auto op = [](float a, float b) { return IS_MAX ? fmaxf(a, b) : a + b; };
  x = op(x, dpp_f<DPP_QUAD_SWAP>(x));
  x = op(x, dpp_f<0x4E>(x));                 // quad_perm [2,3,0,1]
  x = op(x, dpp_f<DPP_ROW_HALF_MIRROR>(x));
  x = op(x, dpp_f<DPP_ROW_MIRROR>(x));
  const int xi = __float_as_int(x);
  const float r0 = __int_as_float(__builtin_amdgcn_readlane(xi, 0)), r1 = __int_as_float(__builtin_amdgcn_readlane(xi, 16));
  const float r2 = __int_as_float(__builtin_amdgcn_readlane(xi, 32)), r3 = __int_as_float(__builtin_amdgcn_readlane(xi, 48));
  return op(op(r0, r1), op(r2, r3));
}

// LDS writes of this wave before, its reads behind (other waves do not touch the region)
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
