// Query preparation of the read half: RoPE at the query's position (Eq. 5's q, rotated once per
// step instead of once per key), scaled by 1/sqrt(128), in the layouts the decode kernels read.
#pragma once
#include "rkv_internal.h"

// One channel of the query times the angle (cs, sn), scaled: x cs + sgn partner sn.  (Rounded once, the same wherever it is inlined.)
__device__ __forceinline__ float rkv_prep_q_turn(float x, float partner, float sgn, double cs, double sn) {
  return (float)(fma((double)x, cs, (double)(sgn * partner) * sn) * 0.08838834764831845);
}
// one channel of the query, rotated to position pos and scaled.  Angles from the table (computed in
// double, stored as float) when the position lies inside it - the usual case -, else computed here
__device__ __forceinline__ float rkv_prep_q_rotate(const RkvView& v, float x, float partner, float sgn, int pos, int j) {
  double sn, cs;
  if (pos >= 0 && pos < v.Tpad) {
    const float2 t = v.rope[(size_t)pos * 64 + j];
    cs = t.x;
    sn = t.y;
  } else {
    sincos((double)pos * pow((double)v.theta, -(double)j / 64.0), &sn, &cs);
  }
  return rkv_prep_q_turn(x, partner, sgn, cs, sn);
}

// One output channel c (0..127) of (virtual) query head h of sequence b.
// q~[b][h][c] = RoPE(q, q_pos)[c] / sqrt(128), angles in double (q_pos may lie beyond the table).
// share: 0 for k_decode_shared's operands besides, 2 for the same unrotated, 1 for k_decode_mfma's (Hq == Hkv), -1 for none.
__device__ __forceinline__ void rkv_prep_q_one(const RkvView& v, const __half* __restrict__ q, const int* __restrict__ q_pos,
                                               int at, float* __restrict__ qr, int share, int nq, int h, int b, int c) {
  // v.Hq counts virtual heads when nq > 1 (several query tokens, each at its own position)
  const RkvVHead vh = rkv_virtual_head(v, h, nq);
  // at: the default position
  const int pos = q_pos ? q_pos[b * nq + vh.qi] : at;
  const size_t base = ((size_t)b * v.Hq + h) * RKV_D;                       // where the rotated query goes
  const size_t src = (((size_t)b * nq + vh.qi) * (v.Hq / nq) + vh.h) * RKV_D; // where the raw query is
  int j, partner;
  float sgn;
  if (v.rope_style == 0) {
    j = c & 63;
    partner = c ^ 64;
    sgn = c < 64 ? -1.f : 1.f;
  } else {
    j = c >> 1;
    partner = c ^ 1;
    sgn = (c & 1) ? 1.f : -1.f;
  }
  const float x = __half2float(q[src + c]), p = __half2float(q[src + partner]);
  const int nn = v.rope_style ? (c >> 1) & 15 : c & 15, pp = v.rope_style ? (c >> 5) & 3 : (c >> 4) & 3, half = v.rope_style ? c & 1 : c >> 6;
  if (share == 0 || share == 2) {
    // The kernel that serves all query heads of a KV head at once (k_decode_shared) takes the query
    // as fp16 matrix operands, split into a high and a low part (a float to 2^-23): for each head
    //   [p][high, low][lane group nn / 4][half][nn % 4]   fp16,
    // scaled by a power of two that puts the head's largest component at 2^8 .. 2^11 (what is 2^-11
    // of it still has all bits of its low part), and the scale's inverse behind all heads' operands.
    float mx = fmaxf(fabsf(__half2float(q[src + (c & 63)])), fabsf(__half2float(q[src + (c & 63) + 64])));
#pragma unroll
    for (int i = 32; i > 0; i >>= 1) mx = fmaxf(mx, __shfl_xor(mx, i));
    int ex = 0;
    if (mx > 0.f && mx < INFINITY) frexpf(mx, &ex);
    const float val = rkv_prep_q_rotate(v, x, p, sgn, pos, j);
    qr[base + c] = val;
    __half* img = reinterpret_cast<__half*>(qr + (size_t)v.B * v.Hq * RKV_D);
    const size_t o = (((((size_t)b * v.Hq + h) * 4 + pp) * 2) * 4 + (nn >> 2)) * 8 + 4 * half + (nn & 3);
    if (share == 2) {                                       // (the query as it came, its rotation is on the keys' side: largest component at 2^15 .. 65504, so the power of two never is below one and the product is exact)
      img[o] = __float2half_rn(ldexpf(x, 16 - ex));
      if (c == 0) qr[2 * (size_t)v.B * v.Hq * RKV_D + (size_t)b * v.Hq + h] = ldexpf(0.08838834764831845f, ex - 16);
      return;
    }
    const float y = ldexpf(val, 14 - ex);
    const __half hi = __float2half_rn(y);
    img[o] = hi;
    img[o + 4 * 8] = __float2half_rn(y - __half2float(hi));
    if (c == 0) qr[2 * (size_t)v.B * v.Hq * RKV_D + (size_t)b * v.Hq + h] = ldexpf(1.0f, ex - 14);
    return;
  }
  qr[base + c] = rkv_prep_q_rotate(v, x, p, sgn, pos, j);
  if (share != 1) return;                                   // (scores from the scores kernel, the general kernel: the plain copy only)
  // k_decode_mfma keeps RoPE angles for the first of a lane's four consecutive tokens only, and rotates the query back to
  // tokens 1 and 2 of the four: it gets it at positions pos - r, r = 1 and 2 (<R(t + r) k, R(pos) q> = <R(t) k, R(pos - r) q>, exactly),
  // in its own layout: [b][rot group][r - 1][p 0..3][f / 4][n 0..15][f % 4],  f = KV head a * 2 + half
  // (the 16 channel lanes n read consecutive 16-byte pieces, which LDS serves without bank conflicts) with
  // entry (n, p, half) = channel 16p + n + 64*half (interleaved pairs: 2 (16p + n) + half), pre-multiplied by 2/sqrt(rotation size)
  // (FP4 nibbles hold code/2; 1/sqrt(n) is the normalisation of Eq. 10).
  const int rg = h / v.g, a = h - rg * v.g;                 // (one query head per KV head)
  float* qt = qr + (size_t)v.B * v.Hq * RKV_D;
  const float lane_scale = 2.0f * rsqrtf((float)v.n);
#pragma unroll
  for (int r = 1; r < 3; ++r) {
    const int f = 2 * a + half;
    size_t o = (((size_t)b * v.NRG + rg) * 2 + r - 1) * 4 + pp;
    o = (o * (v.g / 2) + (f >> 2)) * 16 + nn;
    qt[o * 4 + (f & 3)] = rkv_prep_q_rotate(v, x, p, sgn, pos - r, j) * lane_scale;
  }
}
