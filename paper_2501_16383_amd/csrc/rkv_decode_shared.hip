// Read half, matrix-core kernel for several query heads per KV head (grouped queries, several query
// tokens per step): plain reorder (inside blocks of 128), rot_heads 2 or 4, codes of 2 to 4 bits in
// groups of 128, either metadata format, both RoPE pairings.
//
// One workgroup = (sequence, rotation group, chunk of 256 or 128 tokens, up to 32 / G query heads of each of the
// G KV heads), 4 waves; rkv_mfma_chunk and rkv_shared_heads choose.  Rotation, RoPE and unpacking of a key cost vector
// instructions per (token, KV head); they are done once for all the query heads, and the product with the queries is a
// matrix product whose columns are the (query head, KV head) pairs:
//   phase K  wave w: four (two) tiles of 16 tokens.  The operands of the Hadamard product are
//            exchanged against k_decode_mfma's, H_128 tile [16 channels x 128] times codes [128 x 16 tokens]:
//            lane (n, q) then holds channels 16p + 4q + 0..3 and their RoPE partners of token n, which is
//            the layout the next product (v_mfma_f32_16x16x32_f16: [16 tokens x 32 channels] times
//            [32 channels x 16 columns]) takes its left operand in: nothing crosses lanes.
//            The scales and the butterfly over the blocks (H_g) are linear, so they come after the
//            contraction over the channels:
//              score(t, a, h) = sum_blk H_g[a][blk] scale_blk(t) * <RoPE_t(H_128 c_blk(t)), q~(a, h)>:
//            the rotated codes meet the queries of ALL KV heads of the group, sixteen columns per product.
//            Precision: H_128 c is exact, RoPE runs in fp32; both operands (a query at its sequence's end needs no split: QX) are then split into two
//            fp16 numbers each (low at most 2^-11 of its number, high + low the number to 2^-23) and the product is high * high +
//            high * low + low * high, accumulated in fp32; low * low, at most 2^-22 of a term, is left out: with
//            it outputs were 1 to 3 % closer to 64-bit attention and steps 3 to 6 % slower.  Codes are centred on
//            their middle value (the product's C operand starts at minus its share of channel 0), the
//            zero-points with them, so that channel 0 is no larger than the others.  Outputs are 0.4 to 2.0e-6 of the norm
//            away from 64-bit attention on the same codes (2 to 56 rows per KV head, 140 to 25000 tokens), where the same dot
//            products in fp32 on k_decode_mfma were 0.4 to 8e-6 away; where its workgroups had one query head the two
//            were equal within 5 % (30 draws; since then that kernel has centred codes, and this one QX), where they had two this one was 2 to 10 times closer.
//   phase S  wave: softmax statistics and weight digits of four query heads of one KV head; the digits
//            (six base-16 digits of a 24-bit integer, in FP8, see k_decode_mfma) stay in the wave's own LDS.
//   phase V  the same wave: rows = 4 query heads x 4 digits, contraction over 128 tokens of ONE KV head:
//            no part of the operand is zero, the codes are fetched once for all query heads.
// 32 sequences x 8192 tokens, 32 query heads on 8: step 153.5 us with two query heads per workgroup of k_decode_mfma, 85.0 here;
// four query tokens, 8 x 4096 tokens: 98.4 and 48.3 us (one round of two workgroups per compute unit).  Bound by the vector pipe in phase K (16 instructions of
// RoPE and 16 of the split for eight channels of a token and block).
// The variants with 32 columns and 3- or 4-bit codes hold 8 registers in scratch memory.
#include "rkv_internal.h"
#include "rkv_mfma_ops.h"
#include <hip/hip_ext.h>

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));


// four dwords of FP4 nibbles (the other four registers of the operand are not read)
__device__ __forceinline__ v8i as_fp4(const uint4& u) {
  v8i r;
  r[0] = (int)u.x; r[1] = (int)u.y; r[2] = (int)u.z; r[3] = (int)u.w;
  r[4] = r[5] = r[6] = r[7] = 0;
  return r;
}
__device__ __forceinline__ float flip(float x, uint32_t sign) { return __uint_as_float(__float_as_uint(x) ^ sign); }
// Eight floats -> fp16 high and low parts, x = high + low to 2^-23.  x - high is exact: one multiply-add of mixed
// precision each (high * -1 + x) into a float, two of which are rounded by one conversion.  What an instruction costs here (cycles
// of a SIMD, four waves on it, measured): a float multiply-add 2.4, a conversion of two floats or a mixed multiply-add into
// a float 4.2, one into half a register 8.2 - the form with those was 1.5 instructions an element instead of 2, and 82 cycles for
// eight elements instead of 67.
struct Split8 { v8h hi, lo; };
__device__ __forceinline__ Split8 split8(const float (&x)[8]) {
  union { v2h h2[4]; uint32_t u[4]; v8h h8; } hi, lo;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float l0, l1;
    hi.h2[i] = __builtin_convertvector((v2f){x[2 * i], x[2 * i + 1]}, v2h);
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[0,0,0] op_sel_hi:[1,0,0]" : "=v"(l0) : "v"(hi.u[i]), "v"(x[2 * i]));
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(l1) : "v"(hi.u[i]), "v"(x[2 * i + 1]));
    lo.h2[i] = __builtin_convertvector((v2f){l0, l1}, v2h);
  }
  return {hi.h8, lo.h8};
}

// CT: column tiles (16 columns each), of which rs query heads per KV head are used.  TILES: tiles per wave.  HB: bits per code above the low two (planes as in k_decode_mfma).
// q_lim: null, or the last position each of the nq query tokens may attend (v.Hq then counts virtual heads).
// QX: the one query token of a sequence is the last one.  Keys are then rotated by their distance from it, and the query
// needs no rotation: its fp16 numbers are the operand as they came (times a power of two), and the product with its low part
// falls away, a third of the products with the queries.  32 sequences x 8192 tokens, 32 heads on 8: 90.0 -> 85.2 us a step, and outputs 7 % closer to 64-bit attention (100 draws).
// Three workgroups fit a compute unit with one column tile, but for a second plane of codes of four heads over whole chunks (192 registers); the others
// are told so, since the wider codes' take 169 to 175 registers, a few too many, where two are asked for.  us a call with two and three, 32 heads on 8: rotation
// over two heads, 16 sequences x 4096 tokens, 3-bit 42.1 and 39.3, 4-bit 42.4 and 39.7; over four, half chunks, 12 x 4096, 3-bit 34.6 and 32.4, 4-bit 35.5 and 32.8.
template <int G, int CT, int HB, int TILES, bool QX>
__global__ void __launch_bounds__(256, (CT == 1 && (HB == 0 || G == 2 || TILES == 2)) ? 3 : 2) k_decode_shared(RkvView v, const float* __restrict__ qr,
                                                                                     float* __restrict__ part, int nch,
                                                                                     const int* __restrict__ q_lim, int nq, int ns, int rs,
                                                                                     uint32_t inv_ns, uint32_t inv_nrg) {
  constexpr bool HI = HB != 0;
  constexpr int CH = 64 * TILES;                     // tokens
  constexpr int NC = 16 * CT;                        // columns
  constexpr int SC_STRIDE = CH + 4;               // (rows of sixteen columns fall on different LDS banks)
  constexpr int QSTRIDE = NC + 1;                    // 16-byte pieces per row of the query operand
  constexpr int QP = QX ? 16 : 32;                   // 16-byte pieces of the query operand per column
  constexpr int GP = G / 2;                          // packed fp16 pairs per token
  constexpr int DROW = 144, DSET1 = 16 * DROW, DWAVE = 24 * DROW;   // weight digits of a wave: 16 rows of set 0, 8 of set 1, 128 tokens each
  constexpr float MID = HB == 0 ? 1.5f : HB == 1 ? 3.5f : 7.5f;     // middle code
  struct KeyPart {
    uint4 H[8][64];
    uint4 q[QP][QSTRIDE];                            // [(p, high / low (QX: high only), lane group)][column]
    float ks[G][CH];                              // scales of the chunk's tokens
    float kz[G][CH];                              // their zero-points' share: sum_blk H_g[a][blk] scale_blk (zero_blk - MID)
    float2 cs0[CH];                               // RoPE angle of channel pair 0
    float2 step[64];                                 // RoPE rotation by 16 positions
  };
  union Shared {
    KeyPart k;
    uint8_t dig[4][DWAVE];
  };
  __shared__ __attribute__((aligned(16))) Shared sh;
  __shared__ __attribute__((aligned(16))) float s_sc[NC][SC_STRIDE];
  __shared__ __attribute__((aligned(16))) uint32_t s_vm[G][CH];   // values: (scale, zero-point) pairs
  __shared__ int s_sink[64];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = lane & 15, q = lane >> 4;
  __builtin_amdgcn_s_setprio(3);                     // (short phases ahead of the other workgroups' key phases, as in k_decode_mfma)

  // Workgroup -> (sequence, rotation group, chunk, query-head group): as in k_decode_mfma
  const int rep = v.Hq / v.Hkv;
  int rg = blockIdx.y;
  int rrg, chunk, b;
  if (v.lens) {
    const int tot8 = gridDim.x / ns;
    rrg = blockIdx.x / tot8;
    constexpr int SPLIT = RKV_MFMA_CHUNK / CH;       // (the table counts chunks of 256 tokens)
    const int w_ = blockIdx.x - rrg * tot8, w = w_ / SPLIT;
    if (w >= v.cstart[v.B]) return;
    int lo = 0, hi = v.B;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (v.cstart[mid] <= w) lo = mid;
      else hi = mid;
    }
    b = lo;
    chunk = (w - v.cstart[b]) * SPLIT + w_ % SPLIT;
  } else {
    const int xcd = blockIdx.x & 7, rem = blockIdx.x >> 3;
    chunk = inv_ns ? (int)__umulhi((uint32_t)rem, inv_ns) : rem;
    rrg = rem - chunk * ns;
    const int br = blockIdx.y * 8 + xcd;
    if (br >= v.B * v.NRG) return;
    b = inv_nrg ? (int)__umulhi((uint32_t)br, inv_nrg) : br;
    rg = br - b * v.NRG;
  }
  const int len = rkv_len(v, b);
  if (chunk * CH >= len) return;
  const int t0 = chunk * CH;
  const int rsv = min(rs, rep - rrg * rs);           // query heads per KV head that exist
  // virtual head of column col = rr * G + a
  auto head_of = [&](int col) { return (rg * G + col % G) * rep + rrg * rs + col / G; };

  // ---- requests, back to back
  const size_t nqh = (size_t)v.B * v.Hq;
  const uint4* qimg = reinterpret_cast<const uint4*>(qr + nqh * RKV_D) + (size_t)b * v.Hq * 32;
  const float* qscale = qr + 2 * nqh * RKV_D + (size_t)b * v.Hq;
  const uint4 ld_h0 = reinterpret_cast<const uint4*>(v.hop)[tid], ld_h1 = reinterpret_cast<const uint4*>(v.hop)[tid + 256];
  uint4 ld_q[QP / 16 * CT];
  const int q_row = tid & (QP - 1), q_piece = QX ? 8 * (q_row >> 2) + (q_row & 3) : q_row;
#pragma unroll
  for (int i = 0; i < QP / 16 * CT; ++i) {           // column 256 / QP i + tid / QP, row tid % QP of the operand
    const int col = 256 / QP * i + tid / QP;
    ld_q[i] = col / G < rsv ? qimg[(size_t)head_of(col) * 32 + q_piece] : make_uint4(0, 0, 0, 0);
  }
  const float2 ld_step = v.rope[16 * 64 + (tid & 63)], ld_cs0 = v.rope[(size_t)(t0 + min(tid, CH - 1)) * 64];
  const int cnt = v.max_sinks > 0 ? v.sink_cnt[b] : 0;
  const int ld_spos = (v.max_sinks > 0 && (tid & 63) < v.max_sinks) ? v.sink_pos[b * v.max_sinks + (tid & 63)] : -1;
  float ks_[4], kz_[4];
  uint32_t vmw[4] = {0, 0, 0, 0};
  if (v.meta8) {
    // G scale bytes, then G zero-point bytes (z + 128) per token
    const size_t mi = ((size_t)(b * v.NRG + rg) * v.Tpad + t0 + min(tid, CH - 1)) * (2 * G);
    auto fetch8 = [&](const uint32_t* m, float (&s)[4], float (&z)[4]) {
      const uint8_t* p8 = reinterpret_cast<const uint8_t*>(m) + mi;
      uint32_t sw, zw;
      if constexpr (G == 4) {
        const uint2 u = rkv_ld_stream(reinterpret_cast<const uint2*>(p8));
        sw = u.x; zw = u.y;
      } else {
        sw = *reinterpret_cast<const uint32_t*>(p8);
        zw = sw >> 16;
      }
      s[0] = __builtin_amdgcn_cvt_f32_fp8((int)sw, 0);
      s[1] = __builtin_amdgcn_cvt_f32_fp8((int)sw, 1);
      s[2] = __builtin_amdgcn_cvt_f32_fp8((int)sw, 2);
      s[3] = __builtin_amdgcn_cvt_f32_fp8((int)sw, 3);
#pragma unroll
      for (int i = 0; i < 4; ++i) z[i] = (float)((zw >> (8 * i)) & 0xffu) - 128.0f;
    };
    float s[4], z[4];
    fetch8(v.km, ks_, kz_);
    fetch8(v.vm, s, z);
#pragma unroll
    for (int i = 0; i < G; ++i) vmw[i] = rkv_pack_meta(s[i], z[i]);
  } else {
    const size_t mi = ((size_t)(b * v.NRG + rg) * v.Tpad + t0 + min(tid, CH - 1)) * G;
    uint32_t km[4] = {0, 0, 0, 0};
    if constexpr (G == 4) {
      const uint4 u = rkv_ld_stream(reinterpret_cast<const uint4*>(v.km + mi));
      km[0] = u.x; km[1] = u.y; km[2] = u.z; km[3] = u.w;
      const uint4 w = rkv_ld_stream(reinterpret_cast<const uint4*>(v.vm + mi));
      vmw[0] = w.x; vmw[1] = w.y; vmw[2] = w.z; vmw[3] = w.w;
    } else {
      const uint2 u = rkv_ld_stream(reinterpret_cast<const uint2*>(v.km + mi));
      km[0] = u.x; km[1] = u.y;
      const uint2 w = rkv_ld_stream(reinterpret_cast<const uint2*>(v.vm + mi));
      vmw[0] = w.x; vmw[1] = w.y;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) rkv_unpack_meta(km[i], ks_[i], kz_[i]);
  }
  // per column of this lane: scale of the score, the query's channel pair 0 for the zero-points, last position attended
  float c_scale[CT], c_w0[CT], c_w1[CT];
  int c_lim[CT];
  const float lane_scale = 2.0f * rsqrtf((float)v.n);   // FP4 nibbles hold code / 2; 1 / sqrt(n) normalises the rotation
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    const int col = 16 * ct + n;
    const bool ok = col / G < rsv;
    const int hv = ok ? head_of(col) : head_of(n % G);  // (any head that exists)
    const float* qn = qr + ((size_t)b * v.Hq + hv) * RKV_D;
    c_scale[ct] = qscale[hv] * lane_scale;
    c_w0[ct] = 64.0f * lane_scale * qn[0];
    c_w1[ct] = 64.0f * lane_scale * qn[v.rope_style ? 1 : 64];
    c_lim[ct] = len - 1;
    if (q_lim) c_lim[ct] = min(c_lim[ct], q_lim[b * nq + (ok ? (rrg * rs + col / G) / (rep / nq) : 0)]);
  }
  const int tw = t0 + wave * (16 * TILES);
  float cc[4][4], ss[4][4];                          // RoPE angles of token n (of the tile), pairs 16 p + 4 q + r
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    // (QX: minus the distance to the query's position; tokens behind it are masked)
    const float4* rp = reinterpret_cast<const float4*>(v.rope + (size_t)(QX ? max(len - 1 - (tw + n), 0) : tw + n) * 64 + 16 * p + 4 * q);
    const float4 x = rp[0], y = rp[1];
    cc[p][0] = x.x; ss[p][0] = x.y; cc[p][1] = x.z; ss[p][1] = x.w;
    cc[p][2] = y.x; ss[p][2] = y.y; cc[p][3] = y.z; ss[p][3] = y.w;
    if constexpr (QX) {
#pragma unroll
      for (int r = 0; r < 4; ++r) ss[p][r] = -ss[p][r];
    }
  }
  const uint4* ktiles = reinterpret_cast<const uint4*>(v.kc + rkv_k_tilebase(v, b, rg, tw >> 4));
  const uint32_t* khtiles = HI ? v.kh + (rkv_k_tilebase(v, b, rg, tw >> 4) >> (HB == 1 ? 1 : 0)) : nullptr;
  uint4 cw[GP], cwh[HI ? GP : 1];
  auto load_tile = [&](int ti) {
#pragma unroll
    for (int pr = 0; pr < GP; ++pr) {
      const size_t li = (size_t)ti * (32 * G) + pr * 64 + lane;
      cw[pr] = rkv_ld_stream(ktiles + li);
      if constexpr (HB == 2) {
        cwh[pr] = rkv_ld_stream(reinterpret_cast<const uint4*>(khtiles) + li);
      } else if constexpr (HB == 1) {
        const uint2 u = rkv_ld_stream(reinterpret_cast<const uint2*>(khtiles) + li);
        cwh[pr] = make_uint4(u.x, u.y, 0, 0);
      }
    }
  };
  load_tile(0);

  // ---- what came back goes to LDS
  (&sh.k.H[0][0])[tid] = ld_h0;
  (&sh.k.H[0][0])[tid + 256] = ld_h1;
#pragma unroll
  for (int i = 0; i < QP / 16 * CT; ++i) sh.k.q[q_row][256 / QP * i + tid / QP] = ld_q[i];
  if (tid < 64) {
    sh.k.step[tid] = ld_step;
    s_sink[tid] = tid < cnt ? ld_spos : -1;
  }
  if (tid < CH) {                                    // thread = token of the chunk
    sh.k.cs0[tid] = ld_cs0;
#pragma unroll
    for (int a = 0; a < G; ++a) {
      float Z = 0.f;
#pragma unroll
      for (int i = 0; i < G; ++i) Z = fmaf((__popc(a & i) & 1) ? -ks_[i] : ks_[i], kz_[i] - MID, Z);
      sh.k.ks[a][tid] = ks_[a];
      sh.k.kz[a][tid] = Z;
    }
#pragma unroll
    for (int i = 0; i < G; ++i) s_vm[i][tid] = vmw[i];
  }
  __syncthreads();
  __builtin_amdgcn_s_setprio(0);

  // ------------------------------------------------------------------ phase K
  uint32_t sink_tiles = 0;                           // the wave's tiles that hold a retained sink token
  for (int i = 0; i < cnt; ++i) {
    const int d = s_sink[i] - tw;
    if (d >= 0 && d < 16 * TILES) sink_tiles |= 1u << (d >> 4);
  }
  sink_tiles = __builtin_amdgcn_readfirstlane(sink_tiles);
  const v4f zero4 = {0.f, 0.f, 0.f, 0.f};
  const v4f centre4 = {q == 0 ? -64.0f * MID : 0.f, 0.f, 0.f, 0.f};   // channel 0 of H_128 of the constant MID / 2

#pragma unroll
  for (int ti = 0; ti < TILES; ++ti) {
    const int tt = tw + ti * 16;
    if (tt >= len) break;                            // wave-uniform
    v8i A[G], Ah[HI ? G : 1];
#pragma unroll
    for (int pr = 0; pr < GP; ++pr) {
      A[2 * pr] = unpack_fp4(cw[pr].x, cw[pr].y);
      A[2 * pr + 1] = unpack_fp4(cw[pr].z, cw[pr].w);
      if constexpr (HB == 2) {
        Ah[2 * pr] = unpack_fp4(cwh[pr].x, cwh[pr].y);
        Ah[2 * pr + 1] = unpack_fp4(cwh[pr].z, cwh[pr].w);
      } else if constexpr (HB == 1) {
        Ah[2 * pr] = unpack_fp4_bits(cwh[pr].x);
        Ah[2 * pr + 1] = unpack_fp4_bits(cwh[pr].y);
      }
    }
    if (ti + 1 < TILES) load_tile(ti + 1);               // prefetch (inside the padded allocation)
    v4f d[G][CT];
#pragma unroll
    for (int blk = 0; blk < G; ++blk)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) d[blk][ct] = zero4;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      v8i Hl = as_fp4(sh.k.H[p][lane]), Hh = as_fp4(sh.k.H[p + 4][lane]);
      v8h bh[CT], bl[CT];
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        bh[ct] = __builtin_bit_cast(v8h, sh.k.q[QP / 4 * p + q][16 * ct + n]);
        if constexpr (!QX) bl[ct] = __builtin_bit_cast(v8h, sh.k.q[8 * p + 4 + q][16 * ct + n]);
      }
      v4f lo[G], hi[G];
#pragma unroll
      for (int blk = 0; blk < G; ++blk) {
        lo[blk] = mfma_fp4(Hl, A[blk], p == 0 ? centre4 : zero4);
        hi[blk] = mfma_fp4(Hh, A[blk], zero4);
      }
      if constexpr (HI) {                            // FP4 +-1 with bit 2 set is +-4
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          Hl[i] |= 0x44444444;
          Hh[i] |= 0x44444444;
        }
#pragma unroll
        for (int blk = 0; blk < G; ++blk) {
          lo[blk] = mfma_fp4(Hl, Ah[blk], lo[blk]);
          hi[blk] = mfma_fp4(Hh, Ah[blk], hi[blk]);
        }
      }
#pragma unroll
      for (int blk = 0; blk < G; ++blk) {
        float x[8];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          x[r] = lo[blk][r] * cc[p][r] - hi[blk][r] * ss[p][r];
          x[4 + r] = lo[blk][r] * ss[p][r] + hi[blk][r] * cc[p][r];
        }
        const Split8 k = split8(x);
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          d[blk][ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(k.lo, bh[ct], d[blk][ct], 0, 0, 0);
          if constexpr (!QX) d[blk][ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(k.hi, bl[ct], d[blk][ct], 0, 0, 0);
          d[blk][ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(k.hi, bh[ct], d[blk][ct], 0, 0, 0);
        }
      }
      // on to the next tile's token
      const float4* st = reinterpret_cast<const float4*>(&sh.k.step[16 * p + 4 * q]);
      const float4 s01 = st[0], s23 = st[1];
      const float sc4[4] = {s01.x, s01.z, s23.x, s23.z}, sn4[4] = {s01.y, s01.w, s23.y, s23.w};
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float c = cc[p][r], s = ss[p][r];
        cc[p][r] = c * sc4[r] - s * sn4[r];
        ss[p][r] = s * sc4[r] + c * sn4[r];
      }
    }
    // scales, butterfly and zero-points of tokens 4q + r; this lane's columns all belong to KV head a = n % G
    const int tl = wave * (16 * TILES) + ti * 16 + 4 * q;
    float s_[G][4], sc[4][CT];
#pragma unroll
    for (int blk = 0; blk < G; ++blk) {
      const float4 f = *reinterpret_cast<const float4*>(&sh.k.ks[blk][tl]);
      const uint32_t sg = (uint32_t)(__popc(n & (G - 1) & blk) & 1) << 31;
      s_[blk][0] = flip(f.x, sg); s_[blk][1] = flip(f.y, sg); s_[blk][2] = flip(f.z, sg); s_[blk][3] = flip(f.w, sg);
    }
    const float4 Z4 = *reinterpret_cast<const float4*>(&sh.k.kz[n & (G - 1)][tl]);
    const float4 e01 = *reinterpret_cast<const float4*>(&sh.k.cs0[tl]), e23 = *reinterpret_cast<const float4*>(&sh.k.cs0[tl + 2]);
    const float Z[4] = {Z4.x, Z4.y, Z4.z, Z4.w}, c0[4] = {e01.x, e01.z, e23.x, e23.z}, s0[4] = {e01.y, e01.w, e23.y, e23.w};
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        float t = 0.f;
#pragma unroll
        for (int blk = 0; blk < G; ++blk) t = blk == 0 ? s_[0][r] * d[0][ct][r] : fmaf(s_[blk][r], d[blk][ct][r], t);
        sc[r][ct] = fmaf(t, c_scale[ct], -Z[r] * fmaf(c0[r], c_w0[ct], s0[r] * c_w1[ct]));
      }
    uint32_t masked = 0;
    if (sink_tiles & (1u << ti))
      for (int i = 0; i < cnt; ++i) {
        const int dd = s_sink[i] - (tt + 4 * q);
        if (dd >= 0 && dd < 4) masked |= 1u << dd;
      }
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      float4 o;
      float* op = &o.x;
#pragma unroll
      for (int r = 0; r < 4; ++r) op[r] = (((masked >> r) & 1u) || tt + 4 * q + r > c_lim[ct]) ? -INFINITY : sc[r][ct];
      *reinterpret_cast<float4*>(&s_sc[16 * ct + n][tl]) = o;
    }
  }
  __builtin_amdgcn_s_setprio(3);

  // ------------------------------------------------------------------ phases S and V
  // wave -> KV head a, channel tiles: all eight (G = 4), or one half of them (G = 2)
  constexpr int NB = G == 4 ? 4 : 2;                 // blocks of 32 channels per wave
  constexpr int NQ = CH / 128;                       // contractions of 128 tokens
  const int a = wave & (G - 1), wb = G == 4 ? 0 : (wave >> 1) * 2;
  const int nslab = min(CH / 32, (len - t0 + 31) >> 5);
  const uint4* vslab = reinterpret_cast<const uint4*>(v.vc + rkv_v_slabbase(v, b, rg, t0 >> 5));
  const uint32_t* vhslab = HI ? v.vh + (rkv_v_slabbase(v, b, rg, t0 >> 5) >> (HB == 1 ? 1 : 0)) : nullptr;
  uint4 vcodes[NQ][NB], vhcodes[HI ? NQ : 1][HI ? NB : 1];
#pragma unroll
  for (int s = 0; s < NQ; ++s)
#pragma unroll
    for (int w = 0; w < NB; ++w) {
      // lane group q holds slab 4 s + q: 32 of the 128 tokens of a contraction (behind the sequence's end: the last one
      // again, their weights are zero)
      const uint32_t li = (uint32_t)(min(4 * s + q, nslab - 1) * (64 * G) + ((wb + w) * G + a) * 16 + n);
      vcodes[s][w] = rkv_ld_stream(vslab + li);
      if constexpr (HB == 2) {
        vhcodes[s][w] = rkv_ld_stream(reinterpret_cast<const uint4*>(vhslab) + li);
      } else if constexpr (HB == 1) {
        const uint2 u = rkv_ld_stream(reinterpret_cast<const uint2*>(vhslab) + li);
        vhcodes[s][w] = make_uint4(u.x, u.y, 0, 0);
      }
    }
  __syncthreads();                                   // all scores are there; the key phase's part of LDS is free

  uint8_t* const dig = sh.dig[wave];
  const int tq = CH == 256 ? 4 * lane : min(4 * lane, CH - 4);   // the lane's tokens 4 lane .. + 3, inside the chunk
  const int left = min(CH, len - t0) - 4 * lane;     // how many of them exist
  float vs[4], vz[4];
  {
    const uint4 m4 = *reinterpret_cast<const uint4*>(&s_vm[a][tq]);
    rkv_unpack_meta(m4.x, vs[0], vz[0]);
    rkv_unpack_meta(m4.y, vs[1], vz[1]);
    rkv_unpack_meta(m4.z, vs[2], vz[2]);
    rkv_unpack_meta(m4.w, vs[3], vz[3]);
  }
  const int groups = NC / G <= 4 ? 1 : (rsv + 3) >> 2;   // (no loop, and no registers kept for one, where four heads are all there can be)
#pragma unroll 1
  for (int g = 0; g < groups; ++g) {
    float hm[4], hl[4], hzs[4], hdown[4];
    uint32_t dg[4][6];
#pragma unroll
    for (int qq = 0; qq < 4; ++qq) {
      hm[qq] = -INFINITY;
      hl[qq] = hzs[qq] = hdown[qq] = 0.f;
#pragma unroll
      for (int k = 0; k < 6; ++k) dg[qq][k] = 0;
      const int rr = 4 * g + qq;
      if (rr < rsv) {                                // wave-uniform
        const float4 s4 = *reinterpret_cast<const float4*>(&s_sc[rr * G + a][tq]);
        const float sv[4] = {left > 0 ? s4.x : -INFINITY, left > 1 ? s4.y : -INFINITY, left > 2 ? s4.z : -INFINITY, left > 3 ? s4.w : -INFINITY};
        const float m = wave_allreduce<true>(fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3])));
        float pe[4], w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          pe[i] = sv[i] > -INFINITY ? __expf(sv[i] - m) : 0.f;
          w[i] = pe[i] > 0.f ? pe[i] * vs[i] : 0.f;
        }
        const float l = wave_allreduce<false>((pe[0] + pe[1]) + (pe[2] + pe[3]));
        const float wmax = wave_allreduce<true>(fmaxf(fmaxf(w[0], w[1]), fmaxf(w[2], w[3])));
        // 24-bit fixed point: the largest weight lands in [2^23, 2^24); six base-16 digits
        int ex = 0;
        if (wmax > 0.f) frexpf(wmax, &ex);
        const float up = ldexpf(1.0f, 24 - ex), down = ldexpf(1.0f, ex - 24);
        uint32_t W[4];
        float zs = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          W[i] = (uint32_t)rintf(w[i] * up);
          if (W[i]) zs = fmaf((float)W[i], vz[i], zs);
        }
        // (the largest weight is a 24-bit integer as it stands, so no digit exceeds 15.)  A byte 0..15 read as
        // E4M3 is that integer times 2^-9 - subnormals and the first binade are one straight line -: the bytes of
        // four tokens' weights are brought together and parted into their nibbles, nothing is converted
        const uint32_t p01 = __builtin_amdgcn_perm(W[1], W[0], 0x05010400u), p23 = __builtin_amdgcn_perm(W[3], W[2], 0x05010400u);
        const uint32_t b2 = __builtin_amdgcn_perm(__builtin_amdgcn_perm(W[3], W[2], 0x0c0c0602u),
                                                  __builtin_amdgcn_perm(W[1], W[0], 0x0c0c0602u), 0x05040100u);
        const uint32_t b0 = __builtin_amdgcn_perm(p23, p01, 0x05040100u), b1 = __builtin_amdgcn_perm(p23, p01, 0x07060302u);
        dg[qq][0] = (b2 >> 4) & 0x0f0f0f0fu; dg[qq][1] = b2 & 0x0f0f0f0fu;
        dg[qq][2] = (b1 >> 4) & 0x0f0f0f0fu; dg[qq][3] = b1 & 0x0f0f0f0fu;
        dg[qq][4] = (b0 >> 4) & 0x0f0f0f0fu; dg[qq][5] = b0 & 0x0f0f0f0fu;
        hm[qq] = m;
        hl[qq] = l;
        hzs[qq] = wave_allreduce<false>(zs) * down;
        hdown[qq] = down;
      }
    }
    v4f acc[2 * NB][2];                              // [channel tile][digit set]
#pragma unroll
    for (int i = 0; i < 2 * NB; ++i) acc[i][0] = acc[i][1] = zero4;
#pragma unroll
    for (int s = 0; s < NQ; ++s) {
      if (4 * s < nslab) {                           // workgroup-uniform
        wave_lds_fence();                            // (the digits of the tokens before have been read)
        if ((lane >> 5) == s) {
          uint8_t* dst = dig + ((4 * lane) & 127);
#pragma unroll
          for (int qq = 0; qq < 4; ++qq)
#pragma unroll
            for (int k = 0; k < 6; ++k)
              *reinterpret_cast<uint32_t*>(dst + (k < 4 ? (4 * qq + k) * DROW : DSET1 + (2 * qq + k - 4) * DROW)) = dg[qq][k];
        }
        wave_lds_fence();
        // FP8 operand: lane group q holds tokens 16 q .. + 15 and 64 + 16 q .. + 15 of the 128.  Rows of set 1
        // whose digit does not exist repeat another one; their results are not used
        v8i D[2];
#pragma unroll
        for (int set = 0; set < 2; ++set) {
          const uint8_t* row = dig + (set == 0 ? n * DROW : DSET1 + (2 * (n >> 2) + (n & 1)) * DROW) + 16 * q;
          const uint4 d0 = *reinterpret_cast<const uint4*>(row), d1 = *reinterpret_cast<const uint4*>(row + 64);
          D[set][0] = (int)d0.x; D[set][1] = (int)d0.y; D[set][2] = (int)d0.z; D[set][3] = (int)d0.w;
          D[set][4] = (int)d1.x; D[set][5] = (int)d1.y; D[set][6] = (int)d1.z; D[set][7] = (int)d1.w;
        }
#pragma unroll
        for (int w = 0; w < NB; ++w)
#pragma unroll
          for (int c2 = 0; c2 < 2; ++c2) {
            const v8i B = c2 ? unpack_fp4(vcodes[s][w].z, vcodes[s][w].w) : unpack_fp4(vcodes[s][w].x, vcodes[s][w].y);
            v8i Bh = B;
            if constexpr (HB == 2) Bh = c2 ? unpack_fp4(vhcodes[s][w].z, vhcodes[s][w].w) : unpack_fp4(vhcodes[s][w].x, vhcodes[s][w].y);
            if constexpr (HB == 1) Bh = unpack_fp4_bits(c2 ? vhcodes[s][w].y : vhcodes[s][w].x);
#pragma unroll
            for (int set = 0; set < 2; ++set) {
              v4f& o = acc[2 * w + c2][set];
              if constexpr (HI) o += 4.0f * mfma_fp8_fp4(D[set], Bh, zero4);   // the upper plane counts fourfold
              o = mfma_fp8_fp4(D[set], B, o);
            }
          }
      }
    }
    // lane group q: query head 4 g + q, channels 16 * tile + n; registers: digits
    const int rr = 4 * g + q;
    auto pick = [&](const float (&x)[4]) { return q == 0 ? x[0] : q == 1 ? x[1] : q == 2 ? x[2] : x[3]; };
    const float wsc = 1024.0f * pick(hdown), zs = pick(hzs), m = pick(hm), l = pick(hl);
    if (rr < rsv) {
      float* dst = part + (((size_t)b * v.Hq + head_of(rr * G + a)) * nch + chunk) * RKV_PART_STRIDE;
#pragma unroll
      for (int i = 0; i < 2 * NB; ++i) {
        const v4f h = acc[i][0], lo = acc[i][1];
        const float sum = ((((h[0] * 16.0f + h[1]) * 16.0f + h[2]) * 16.0f + h[3]) * 16.0f + lo[0]) * 16.0f + lo[1];
        dst[4 + 16 * (2 * wb + i) + n] = sum * wsc - zs;
      }
      if (wb == 0 && n == 0) {
        dst[0] = m;
        dst[1] = l;
      }
    }
  }
}

// More than one (query token, query head) pair per KV head, on a cache whose scores do not come from the scores
// kernel.  (One pair fills 4 of the 16 columns: there k_decode_mfma, which takes the dot product on the vector pipe, has
// about 650 vector instructions per tile of 16 tokens and four heads where this kernel has 840, of one query head or
// of four.  8 sequences x 4096 tokens, 32 heads, one query token through rkv_decode_attention_multi: 38 us there,
// 45.5 here.  From two pairs on this kernel is the faster one: 47.9 us against the 53.2 of a k_decode_mfma with two
// query heads per workgroup.)
bool rkv_shared_decode(const rkv_cache* c, int heads_per_kv_head) {
  return c->decode_path != 3 && !rkv_scores_path(c) && heads_per_kv_head > 1;
}

// Query heads per KV head and workgroup: as many as 32 columns take; fewer, down to four, as long as the workgroups
// that makes are at most one per compute unit (their keys are rotated again by each, but it has fewer query heads to go through one
// after the other, and sixteen columns).  8 heads on each of 8, 1024 tokens: 32 sequences (128 workgroups of eight heads)
// 25.0 us, of four; 48 sequences (192) 31.3 us, 33.7 if split into 384; 64 (256) 33.1 and 35.2.
int rkv_shared_heads(const rkv_cache* c, int heads_per_kv_head, int chunk) {
  const int most = 32 / c->v.g;
  int rs = heads_per_kv_head < most ? heads_per_kv_head : most;
  const size_t load = rkv_mfma_load(c, chunk);
  while (rs > 4 && 2 * load * ((heads_per_kv_head + rs - 1) / rs) <= (size_t)c->n_cu) rs = rs > 8 ? 8 : 4;
  return rs;
}

// v, nq: the (virtual) view of rkv_launch_decode_mfma; chunk: 256 or 128 tokens per workgroup; exact_q: the queries were prepared
// unrotated (rkv_prep_form), each at its sequence's last token
int rkv_launch_decode_shared(const rkv_cache* c, const RkvView& v, const float* qr, float* part, int nch, int chunk, const int* q_lim, int nq, bool exact_q,
                             hipEvent_t ev_start, hipEvent_t ev_stop, hipStream_t s) {
  const int rep = v.Hq / v.Hkv, split = RKV_MFMA_CHUNK / chunk;
  const int rs = rkv_shared_heads(c, rep, chunk), ns = (rep + rs - 1) / rs, ct = rs * v.g <= 16 ? 1 : 2;
  auto recip = [](int d) { return d <= 1 ? 0u : (uint32_t)((((uint64_t)1 << 32) + d - 1) / d); };
  dim3 grid(8 * nch * ns, (v.B * v.NRG + 7) / 8, 1);
  if (c->ragged) {                                          // all sequences' chunks in one dimension
    unsigned total = 0;
    for (int b = 0; b < v.B; ++b) total += (c->hlens[b] + RKV_MFMA_CHUNK - 1) / RKV_MFMA_CHUNK;
    grid = dim3(((total * split + 7) & ~7u) * ns, v.NRG, 1);
  }
  if (grid.y > 65535) return RKV_EINVAL;
#define RKV_SH_Q(G_, C_, H_, T_) (exact_q ? k_decode_shared<G_, C_, H_, T_, true> : k_decode_shared<G_, C_, H_, T_, false>)
#define RKV_SH(G_, C_, T_) (v.hb == 2 ? RKV_SH_Q(G_, C_, 2, T_) : v.hb == 1 ? RKV_SH_Q(G_, C_, 1, T_) : RKV_SH_Q(G_, C_, 0, T_))
#define RKV_SH_C(G_, T_) (ct == 1 ? RKV_SH(G_, 1, T_) : RKV_SH(G_, 2, T_))
  auto fn = split == 1 ? (v.g == 4 ? RKV_SH_C(4, 4) : RKV_SH_C(2, 4)) : (v.g == 4 ? RKV_SH_C(4, 2) : RKV_SH_C(2, 2));
#undef RKV_SH_C
#undef RKV_SH
#undef RKV_SH_Q
  if (ev_start && ev_stop)
    hipExtLaunchKernelGGL(fn, grid, dim3(256), 0, s, ev_start, ev_stop, 0, v, qr, part, nch, q_lim, nq, ns, rs, recip(ns), recip(v.NRG));
  else
    hipLaunchKernelGGL(fn, grid, dim3(256), 0, s, v, qr, part, nch, q_lim, nq, ns, rs, recip(ns), recip(v.NRG));
  return RKV_OK;
}
