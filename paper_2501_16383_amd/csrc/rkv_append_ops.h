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

// ---- one token's keys as columns (rkv_append_one, append_row_few): a product's columns are sixteen heads, its rows
// channels 16 p + 4 q + r of head `col`, p = 2 w and 2 w + 1 for wave w of four.

// H_128 of the columns' heads, from x[ks] = the head's channels 32 ks + 8 q .. + 7, and H_G over neighbouring columns.
// A operand: lane (row m = col, k-group q) holds H_128[16 p + m][32 ks + 8 q + j], j = 0..7: the parity of (channel & k)
template <int G>
__device__ __forceinline__ void rotate_columns(const uint4 (&x)[4], int w, int col, int q, v4f (&acc)[2]) {
  uint32_t sg[4];
#pragma unroll
  for (int j = 0; j < 4; ++j)
    sg[j] = (0x3C003C00u ^ parity_mask(col & (2 * j) & 7, 0x00008000u)) ^ parity_mask(col & (2 * j + 1) & 7, 0x80000000u);
#pragma unroll
  for (int pp = 0; pp < 2; ++pp) {
    const int p = 2 * w + pp;
    const uint32_t mk = parity_mask(((col >> 3) & 1 & q) ^ ((p & 1) & (q >> 1)), 0x80008000u);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const uint32_t mm = mk ^ parity_mask((p >> 1) & ks, 0x80008000u);
      const v4f zero4 = {0.f, 0.f, 0.f, 0.f};
      acc[pp] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_v8h(sg[0] ^ mm, sg[1] ^ mm, sg[2] ^ mm, sg[3] ^ mm),
                                                       as_v8h(x[ks].x, x[ks].y, x[ks].z, x[ks].w), ks == 0 ? zero4 : acc[pp], 0, 0, 0);
    }
  }
#pragma unroll
  for (int pp = 0; pp < 2; ++pp)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float a = acc[pp][r];
      const float b1 = __uint_as_float(dpp_u<0xB1>(__float_as_uint(a)));             // quad_perm [1,0,3,2]
      a = (col & 1) ? b1 - a : a + b1;
      if constexpr (G == 4) {
        const float b2 = __uint_as_float(dpp_u<0x4E>(__float_as_uint(a)));           // quad_perm [2,3,0,1]
        a = (col & 2) ? b2 - a : a + b2;
      }
      acc[pp][r] = a;
    }
}

// A lane's eight codes (see above) into the dwords of its head `hb` of the rotation group, token t: four codes of product pp at bits 16 (q & 1) + 4 r + 2 (q >> 1)
// of dword (hb, p); third bits: code m = 8 (q & 1) + 2 r + (q >> 1) of dword pp of a pair at bit 4 (m >> 1) + 2 pp + (m & 1) of the pair's.
// code(pp, r): the code; live: the lane that stores (one per column).
template <int HB, typename Code>
__device__ __forceinline__ void store_column_codes(const RkvView& v, int b, int rg, int t, int hb, int w, int q, bool live, Code code) {
  constexpr bool HI = HB == 2, H1 = HB == 1;
  const size_t tile = rkv_k_tilebase(v, b, rg, t >> 4);
  uint32_t third = 0;
#pragma unroll
  for (int pp = 0; pp < 2; ++pp) {
    uint32_t word = 0, upper = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const uint32_t c = code(pp, r);
      word |= (c & 3u) << (16 * (q & 1) + 4 * r + 2 * (q >> 1));
      if constexpr (HI) upper |= (c >> 2) << (16 * (q & 1) + 4 * r + 2 * (q >> 1));
      if constexpr (H1) third |= (c >> 2) << (16 * (q & 1) + 4 * r + 2 * pp + (q >> 1));
    }
    word |= __shfl_xor(word, 16);
    word |= __shfl_xor(word, 32);
    const int p = 2 * w + pp;
    const size_t o = tile + ((((hb >> 1) * 4 + (p >> 1)) * 16 + (t & 15)) * 4) + (hb & 1) * 2 + (p & 1);
    if (live) v.kc[o] = word;
    if constexpr (HI) {
      upper |= __shfl_xor(upper, 16);
      upper |= __shfl_xor(upper, 32);
      if (live) v.kh[o] = upper;
    }
    if constexpr (H1) {
      if (pp == 1) {
        third |= __shfl_xor(third, 16);
        third |= __shfl_xor(third, 32);
        if (live) v.kh[o >> 1] = third;
      }
    }
  }
}
