// Append of one token (a decode step): the keys and values of one rotation group, by 256 threads.  Bit for bit what the bulk
// kernel stores: a matrix product's output depends on its own row and column alone and the channels are summed in the same
// order, so its columns, sixteen tokens there, are the group's heads here (a column per head, repeated); extrema are exact in any order.
//   keys    wave w: channels 32w .. + 31 of every head, two products of 16 channels over K = 128; lane (column, q) holds
//           channels 16p + 4q + r of head column mod G, p = 2w and 2w + 1; H_g between neighbouring lanes; extrema
//           over q by lane exchanges and over the waves through LDS; the four codes of a lane sit at bits 16 (q & 1) + 4 r +
//           2 (q >> 1) of dword (head, p) of the token.
//   values  wave a < G: head a, lane: channels 2 lane and 2 lane + 1, whose bits are put into the dwords of the token's slab.
// One barrier.  What bounds it is the chain row -> extrema -> codes -> store.
// (append_row_few has the same operand, butterfly and packing for whole rows.  One piece of code for both was tried: the order in which the
// compiler then puts them made a decode step 1 % longer on one sequence x 512 tokens, 2.5 % on one x 32768.)
#pragma once
#include "rkv_internal.h"
#include "rkv_append_ops.h"

struct RkvOneLds {
  float2 mm[4][4];                       // [wave][head]
};
template <int G, int HB>
__device__ __forceinline__ void rkv_append_one(const RkvView& v, const __half* __restrict__ krow, const __half* __restrict__ vrow, int t, int b, int rg,
                                               RkvOneLds& lds) {
  constexpr bool HI = HB == 2, H1 = HB == 1;
  constexpr float QMAX = HI ? 15.0f : (H1 ? 7.0f : 3.0f), INV_QMAX = HI ? 0.06666667f : (H1 ? 0.14285715f : 0.33333334f);
  constexpr int n = 128 * G;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15, q = lane >> 4, head = col & (G - 1);
  const bool vact = wave < G;
  const __half* kg = krow + (size_t)rg * n;
  // ---- requests
  uint4 x[4] = {make_uint4(0, 0, 0, 0), make_uint4(0, 0, 0, 0), make_uint4(0, 0, 0, 0), make_uint4(0, 0, 0, 0)};
  if (!v.keys_rotated) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) x[ks] = *reinterpret_cast<const uint4*>(kg + head * RKV_D + 32 * ks + 8 * q);
  }
  const int tau = t & 31, vc0 = (vact ? wave : 0) * RKV_D + 2 * lane;          // values: channels vc0, vc0 + 1 of the group
  const uint32_t vraw = *reinterpret_cast<const uint32_t*>(vrow + (size_t)rg * n + vc0);
  const size_t vb = rkv_v_slabbase(v, b, rg, t >> 5);
  const size_t o0 = vb + rkv_v_off(G, vc0, tau), o1 = vb + rkv_v_off(G, vc0 + 1, tau);
  const uint32_t old0 = v.vc[o0], old1 = v.vc[o1];
  uint32_t oldh0 = 0, oldh1 = 0;
  if constexpr (HI) { oldh0 = v.vh[o0]; oldh1 = v.vh[o1]; }
  if constexpr (H1) { oldh0 = v.vh[o0 >> 1]; oldh1 = v.vh[o1 >> 1]; }
  // ---- keys: rotation
  v4f acc[2];
  if (v.keys_rotated) {
    // the keys already are what enters Eq. 6, in reordered order
#pragma unroll
    for (int pp = 0; pp < 2; ++pp)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[pp][r] = __half2float(kg[v.pinv[rg * n + head * RKV_D + 16 * (2 * wave + pp) + 4 * q + r] - rg * n]);
  } else {
    // A operand: lane (row m, k-group q) holds H_128[16 p + m][32 ks + 8 q + j], j = 0..7: the parity of (channel & k)
    uint32_t sg[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      sg[j] = (0x3C003C00u ^ parity_mask(col & (2 * j) & 7, 0x00008000u)) ^ parity_mask(col & (2 * j + 1) & 7, 0x80000000u);
#pragma unroll
    for (int pp = 0; pp < 2; ++pp) {
      const int p = 2 * wave + pp;
      const uint32_t mk = parity_mask(((col >> 3) & 1 & q) ^ ((p & 1) & (q >> 1)), 0x80008000u);
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const uint32_t mm = mk ^ parity_mask((p >> 1) & ks, 0x80008000u);
        const v4f zero4 = {0.f, 0.f, 0.f, 0.f};
        acc[pp] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_v8h(sg[0] ^ mm, sg[1] ^ mm, sg[2] ^ mm, sg[3] ^ mm),
                                                         as_v8h(x[ks].x, x[ks].y, x[ks].z, x[ks].w), ks == 0 ? zero4 : acc[pp], 0, 0, 0);
      }
    }
    // H_g over the heads: neighbouring columns
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
  {
    float mn = acc[0][0], mx = mn;
#pragma unroll
    for (int pp = 0; pp < 2; ++pp)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        mn = fminf(mn, acc[pp][r]);
        mx = fmaxf(mx, acc[pp][r]);
      }
    mn = fminf(mn, __shfl_xor(mn, 16)); mx = fmaxf(mx, __shfl_xor(mx, 16));
    mn = fminf(mn, __shfl_xor(mn, 32)); mx = fmaxf(mx, __shfl_xor(mx, 32));
    if (lane < G) lds.mm[wave][lane] = make_float2(mn, mx);
  }
  // ---- values (while the waves meet)
  {
    // (min, -max) of the head as one packed pair
    const uint32_t sw = __builtin_amdgcn_perm(vraw, vraw, 0x01000302u);
    uint32_t p = __builtin_amdgcn_perm(pk_max(vraw, sw), pk_min(vraw, sw), 0x05040100u) ^ 0x80000000u;
    p = pk_min(p, dpp_u<0xB1>(p));                                        // quad_perm [1,0,3,2]
    p = pk_min(p, dpp_u<0x4E>(p));                                        // quad_perm [2,3,0,1]
    p = pk_min(p, dpp_u<0x141>(p));                                       // row_half_mirror
    p = pk_min(p, dpp_u<0x140>(p));                                       // row_mirror
    p = pk_min(p, (uint32_t)__shfl_xor((int)p, 16));
    p = pk_min(p, (uint32_t)__shfl_xor((int)p, 32));
    const h2 pr = as_h2(p), raw = as_h2(vraw);
    float sc, zero_v, inv, base, add;
    quant_params_nodiv((float)pr[0], -(float)pr[1], sc, zero_v, inv, v.meta8, INV_QMAX);
    fused_round_consts(zero_v, base, add);
    const float c0 = __builtin_amdgcn_fmed3f(fmaf((float)raw[0], inv, add), base, base + QMAX);
    const float c1 = __builtin_amdgcn_fmed3f(fmaf((float)raw[1], inv, add), base, base + QMAX);
    const uint32_t e0 = __float_as_uint(c0) - __float_as_uint(base), e1 = __float_as_uint(c1) - __float_as_uint(base);
    const int sh = rkv_v_shift(tau);
    if (vact) {
      v.vc[o0] = (old0 & ~(3u << sh)) | (e0 & 3u) << sh;
      v.vc[o1] = (old1 & ~(3u << sh)) | (e1 & 3u) << sh;
      if constexpr (HI) {
        v.vh[o0] = (oldh0 & ~(3u << sh)) | (e0 >> 2) << sh;
        v.vh[o1] = (oldh1 & ~(3u << sh)) | (e1 >> 2) << sh;
      }
      if constexpr (H1) {
        const int bit = 4 * (tau & 7) + (tau >> 3);         // (a channel's dword of third bits holds the whole slab)
        v.vh[o0 >> 1] = (oldh0 & ~(1u << bit)) | (e0 >> 2) << bit;
        v.vh[o1 >> 1] = (oldh1 & ~(1u << bit)) | (e1 >> 2) << bit;
      }
      if (lane == 0) rkv_store_meta(v, v.vm, rkv_meta_index(v, b, t, rg * G + wave), sc, zero_v);
    }
  }
  __syncthreads();
  // ---- keys: Eq. 6-9 on y = (raw rotation) / sqrt(n)
  const float rs = v.keys_rotated ? 1.0f : rsqrtf((float)n);
  const float2 m0 = lds.mm[0][head], m1 = lds.mm[1][head], m2 = lds.mm[2][head], m3 = lds.mm[3][head];
  float sc, zero_h, inv, base, add;
  quant_params_nodiv(fminf(fminf(m0.x, m1.x), fminf(m2.x, m3.x)) * rs, fmaxf(fmaxf(m0.y, m1.y), fmaxf(m2.y, m3.y)) * rs, sc, zero_h, inv,
                     v.meta8, INV_QMAX);
  fused_round_consts(zero_h, base, add);
  const float inv2 = inv * rs;
  if (tid < G) rkv_store_meta(v, v.km, rkv_meta_index(v, b, t, rg * G + tid), sc, zero_h);
  const size_t tile = rkv_k_tilebase(v, b, rg, t >> 4);
  uint32_t third = 0;
#pragma unroll
  for (int pp = 0; pp < 2; ++pp) {
    uint32_t word = 0, upper = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float c = __builtin_amdgcn_fmed3f(fmaf(acc[pp][r], inv2, add), base, base + QMAX);
      const uint32_t code = __float_as_uint(c) - __float_as_uint(base);
      word |= (code & 3u) << (16 * (q & 1) + 4 * r + 2 * (q >> 1));
      if constexpr (HI) upper |= (code >> 2) << (16 * (q & 1) + 4 * r + 2 * (q >> 1));
      if constexpr (H1) third |= (code >> 2) << (16 * (q & 1) + 4 * r + 2 * pp + (q >> 1));
    }
    word |= __shfl_xor(word, 16);
    word |= __shfl_xor(word, 32);
    const int p = 2 * wave + pp;
    const size_t o = tile + ((((head >> 1) * 4 + (p >> 1)) * 16 + (t & 15)) * 4) + (head & 1) * 2 + (p & 1);
    if (lane < G) v.kc[o] = word;
    if constexpr (HI) {
      upper |= __shfl_xor(upper, 16);
      upper |= __shfl_xor(upper, 32);
      if (lane < G) v.kh[o] = upper;
    }
    if constexpr (H1) {
      if (pp == 1) {
        third |= __shfl_xor(third, 16);
        third |= __shfl_xor(third, 32);
        if (lane < G) v.kh[o >> 1] = third;
      }
    }
  }
}
