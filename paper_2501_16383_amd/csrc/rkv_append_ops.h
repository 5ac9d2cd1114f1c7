// Matrix operands, packed extrema and block parameters of the write half's matrix-core kernels.
#pragma once
#include "rkv_internal.h"

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ v8h as_v8h(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  union { uint32_t u[4]; v8h h; } x;
  x.u[0] = a; x.u[1] = b; x.u[2] = c; x.u[3] = d;
  return x.h;
}
__device__ __forceinline__ uint32_t parity_mask(int x, uint32_t m) { return (__popc(x) & 1) ? m : 0u; }

typedef _Float16 h2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ h2 as_h2(uint32_t u) { return __builtin_bit_cast(h2, u); }
__device__ __forceinline__ uint32_t as_u32(h2 h) { return __builtin_bit_cast(uint32_t, h); }
// packed fp16 min / max as single instructions (the builtin forms add a canonicalizing instruction
// per operand, which costs as much as the operation itself)
__device__ __forceinline__ uint32_t pk_min(uint32_t a, uint32_t b) {
  uint32_t r;
  asm("v_pk_min_f16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ uint32_t pk_max(uint32_t a, uint32_t b) {
  uint32_t r;
  asm("v_pk_max_f16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, true);
}

// Eq. 8-9 for one block given its min and max, as quant_params but without IEEE divisions: the
// division by 3 (or 7, or 15) is a multiplication (error below 1.5 ulp of fp32, which can change the fp16 scale
// only within 2^-23 of a rounding boundary) and the reciprocal of the scale is v_rcp_f32 refined by
// one Newton step.
// meta8: FP8 E4M3 scale rounded up, INT8 zero-point.
// inv_qmax: 1 / (2^bits - 1) rounded to fp32.
__device__ __forceinline__ void quant_params_nodiv(float mn, float mx, float& s, float& zero, float& inv_s, bool meta8,
                                                   float inv_qmax = 0.33333334f) {
  const float raw = (mx - mn) * inv_qmax;
  if (meta8) {
    s = rkv_e4m3_round_up(raw);
    if (s == 0.0f) {
      s = rkv_e4m3_round_up(fabsf(mn));
      if (s == 0.0f) s = 1.0f;
    }
  } else {
    s = __half2float(__float2half_rn(raw));
    if (!(s <= 65504.0f)) s = 65504.0f;
    if (s == 0.0f) {
      s = __half2float(__float2half_rn(fabsf(mn)));
      if (!(s <= 65504.0f)) s = 65504.0f;
      if (s == 0.0f) s = 1.0f;
    }
  }
  const float r0 = __builtin_amdgcn_rcpf(s);
  inv_s = fmaf(fmaf(-s, r0, 1.0f), r0, r0);
  zero = -rintf(mn * inv_s);
  zero = meta8 ? fminf(fmaxf(zero, -128.0f), 127.0f) : fminf(fmaxf(zero, -2048.0f), 2048.0f);
}

// value of x in lane `src_lane` (the address operand is the lane number times 4)
__device__ __forceinline__ float lane_read(float x, int src_lane4) {
  return __int_as_float(__builtin_amdgcn_ds_bpermute(src_lane4, __float_as_int(x)));
}

// Eq. 6 with one FMA per element.  Adding 1.5 * 2^23 rounds to an integer, ties to even, as rintf;
// adding the (integer) zero-point in the same FMA keeps that rounding only if the constant added is
// even, so an odd zero-point is raised by one and the clamp bounds and the packing bias move with
// it.  `base` = 1.5 * 2^23 + (zero & 1); `add` = base + zero; codes are float_bits - bits(base).
__device__ __forceinline__ void fused_round_consts(float zero, float& base, float& add) {
  const float odd = (float)((int)zero & 1);
  base = 12582912.0f + odd;
  add = base + zero;
}
