// Read half, matrix-core kernel for gfx950.
//
// The inverse rotation of the keys is a dense contraction with a +-1 matrix, and 2-bit codes are
// exactly representable in FP4 (E2M1: a nibble holding the integer c in its two low bits is the
// value c/2), so the per-head Hadamard H_128 of the raw codes runs on
// v_mfma_f32_16x16x128_f8f6f4 with exact small-integer results in fp32.  The rest is linear in
// those results:
//     k^[head a][j] = (1/sqrt(n)) * sum_blk H_g[a][blk] * scale_blk * (H_128 c_blk - 128 zero_blk e_0)[j]
// (H_n = H_g (x) H_128 for the grouped-head rotation of Sec. 4.2; Eq. 7 folded in).  The sum over
// the blocks is a second, tiny matrix product on v_mfma_f32_4x4x4_16b_f16 (16 independent 4x4x4
// products per instruction): rows = the token's fp16 scales signed by a row of H_g, columns = the
// blocks' results, which are exact in fp16.  Codes are centred on their middle value (the big product of channel 0 starts
// at minus its share of it), the zero-points with them: channel 0 is then no larger than the others, which halves the error of
// the scores (30 drawn calls of one query head per KV head: 0.56 times the distance from 64-bit attention).  The
// vector ALU does RoPE - on the query, see the key phase - and the dot with the query (Eq. 5).  p.V runs on the same instruction with the codes as the FP4
// operand and the softmax weights p_t * scale_t as the other: each weight is scaled by a power of
// two per (head, chunk) to a 24-bit integer and split into six base-16 digits, which FP8 (E4M3)
// holds exactly.  All products are then small half-integers of similar size, so the instruction's
// internal accumulation is exact (with weights of mixed magnitude in one dot product it is not:
// small terms are cut ~2^-14 below the largest); zero-points enter as one scalar per head.
//
// One workgroup = (sequence, rotation group, chunk of 256 or 128 tokens), 4 waves.
//   phase K  wave w: four or two tiles of 16 tokens.  A = codes [16 tokens x 128], B = H_128 tile
//            [128 x 16 channels]; lane (n, q) of the result holds channel 16*tile + n of tokens
//            4q..4q+3.  Scores are reduced over the 16 channel lanes with DPP and go to LDS.
//   phase S  wave: softmax statistics of head a = wave mod G over the chunk, weights -> FP8 digits in the wave's own LDS.
//   phase V  the same wave: rows = the head's six digits, contraction over 128 tokens of the head, columns = 16
//            channels: sixteen products per wave, and no workgroup barrier between S and V.  (With rows = 4 heads x 4
//            digits of one 32-token slab, block-diagonal over the heads, there were 32 of 33 cycles each.)
// What an instruction costs on this chip (cycles of a SIMD, four waves on it, measured): 16x16x128 FP4 product 16.6,
// FP8 x FP4 33, 4x4x4 8.3, float multiply-add 2.4, conversion, permute or lane move 4.2; matrix and vector
// instructions add up but for two of the latter per product.
// Covers: reorder that keeps 128-blocks, rot_heads 2 or 4, codes of 2 to 4 bits in groups of 128;
// both RoPE pairings (the Hadamard operand tiles are built so that tiles p and p + 4 yield the two
// channels of a pair); one query head per KV head and one query token.  Several of either are
// k_decode_shared's; here the variants on precomputed scores (PRE) take them.  Everything else takes the
// general kernel.
#include "rkv_internal.h"
#include "rkv_mfma_ops.h"
#include "rkv_append_one.h"
#include "rkv_prep_q.h"
#include <hip/hip_ext.h>

typedef _Float16 v4h __attribute__((ext_vector_type(4)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));

#ifndef MF_TILES
#define MF_TILES 4         // 16-token tiles per wave
#endif
#define MF_CH (64 * MF_TILES)   // tokens per workgroup (4 waves)
static_assert(MF_CH == 256, "the per-sequence chunk table (k_lens) counts chunks of 256 tokens");
static_assert(MF_CH == RKV_MFMA_CHUNK, "the work-space size of a call is worked out from RKV_MFMA_CHUNK");
#define MF_OCC 3           // workgroups per compute unit the register budget is set for
#define MF_OCC_HI 2        // the same for the variants that hold a second plane of codes of four heads over whole chunks (three would spill)

__device__ __forceinline__ v4h as_v4h(uint32_t a, uint32_t b) {
  union { uint32_t u[2]; v4h h; } c;
  c.u[0] = a;
  c.u[1] = b;
  return c.h;
}
// two floats that are exactly representable in fp16 -> packed pair
__device__ __forceinline__ uint32_t pk_f16(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(a, b));
}
// 16 independent 4x4x4 products: block = lane / 4, A row / B column = lane % 4, result column = lane % 4
__device__ __forceinline__ v4f mfma_4x4x4(const v4h& a, const v4h& b, const v4f& c) {
  return __builtin_amdgcn_mfma_f32_4x4x4f16(a, b, c, 0, 0, 0);
}

// Sum NV values over the 16 lanes of a row; lane n ends with the total of value n (NV = 16) or of
// value n & 7 (NV = 8).
// The first two steps of the sixteen-value case, written out: a step's lanes of the upper half keep
// the upper values and those of the lower half the lower ones, which a DPP addition does in one
// instruction per half when it is told to write only that half's banks of four lanes (the other
// lanes keep what the destination holds) - two instructions per result where a select of what to
// keep, a select of what to send and the addition take three.  The compiler does not look into
// the text for the two idle cycles a DPP operand needs after a vector write of it, and it does not
// know of them for the results either: hence the waits at both ends, and the order inside (every
// register is read two or more instructions after it was written).
__device__ __forceinline__ void row_transpose_reduce_16_to_4(const float (&v)[16], float (&k4)[4]) {
  float a0, a1, a2, a3, a4, a5, a6, a7;
  asm("s_nop 1\n\t"
      "v_add_f32_dpp %4, %12, %12 row_mirror row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %5, %13, %13 row_mirror row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %6, %14, %14 row_mirror row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %7, %15, %15 row_mirror row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %8, %16, %16 row_mirror row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %9, %17, %17 row_mirror row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %10, %18, %18 row_mirror row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %11, %19, %19 row_mirror row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %4, %20, %20 row_mirror row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %5, %21, %21 row_mirror row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %6, %22, %22 row_mirror row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %7, %23, %23 row_mirror row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %8, %24, %24 row_mirror row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %9, %25, %25 row_mirror row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %10, %26, %26 row_mirror row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %11, %27, %27 row_mirror row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %0, %4, %4 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
      "v_add_f32_dpp %1, %5, %5 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
      "v_add_f32_dpp %2, %6, %6 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
      "v_add_f32_dpp %3, %7, %7 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
      "v_add_f32_dpp %0, %8, %8 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
      "v_add_f32_dpp %1, %9, %9 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
      "v_add_f32_dpp %2, %10, %10 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
      "v_add_f32_dpp %3, %11, %11 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
      "s_nop 1"
      : "=&v"(k4[0]), "=&v"(k4[1]), "=&v"(k4[2]), "=&v"(k4[3]), "=&v"(a0), "=&v"(a1), "=&v"(a2), "=&v"(a3), "=&v"(a4), "=&v"(a5),
        "=&v"(a6), "=&v"(a7)
      : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "v"(v[4]), "v"(v[5]), "v"(v[6]), "v"(v[7]), "v"(v[8]), "v"(v[9]), "v"(v[10]),
        "v"(v[11]), "v"(v[12]), "v"(v[13]), "v"(v[14]), "v"(v[15]));
}

template <int NV>
__device__ __forceinline__ float row_transpose_reduce(const float (&v)[NV], int n) {
  static_assert(NV == 16 || NV == 8, "");
  float k4[4];
  if constexpr (NV == 16) {
    row_transpose_reduce_16_to_4(v, k4);
  } else {
    float k8[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) k8[i] = v[i] + dpp_f<DPP_ROW_MIRROR>(v[i]);
    const bool hi = (n & 4) != 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float keep = hi ? k8[i + 4] : k8[i], send = hi ? k8[i] : k8[i + 4];
      k4[i] = keep + dpp_f<DPP_ROW_HALF_MIRROR>(send);
    }
  }
  float k2[2];
  {
    const bool hi = (n & 2) != 0;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float keep = hi ? k4[i + 2] : k4[i], send = hi ? k4[i] : k4[i + 2];
      k2[i] = keep + dpp_f<DPP_QUAD_MIRROR>(send);
    }
  }
  const bool hi = (n & 1) != 0;
  const float keep = hi ? k2[1] : k2[0], send = hi ? k2[0] : k2[1];
  return keep + dpp_f<DPP_QUAD_SWAP>(send);
}

// MULTI (with PRE): several query tokens per sequence.  v.Hq then counts virtual heads (nq per real head, see
// rkv_virtual_head) and virtual head hv only attends tokens at positions <= q_lim[b][query token of hv].
// Without PRE q_lim, if set, is the position of the sequence's one query token.
// META8: scales in FP8 E4M3 and zero-points in 8 bits (rkv_load_meta describes the layout); they
// are widened to the fp16 operands of the small matrix products right after loading.
// HB = 2: 4-bit codes, c = c_lo + 4 c_hi.  The plane of the upper two bits has the layout of the lower
// one.  HB = 1: 3-bit codes, the plane of third bits holds one dword per operand (half the size).
// Key phase: it goes through the same unpacking (nibble = c_hi / 2) and meets a copy of the
// Hadamard operand with entries +-4 in place of +-1, accumulating onto the low plane's products,
// so that the big products yield H_128 (c / 2) as before.  Value phase: it accumulates separately
// and is folded in, times 4, once per chunk.  Sums stay exact: |H_128 (c / 2)| <= 960 < 1024.
// SUB = 2 or 4 (with PRE): quantization groups of 64 or 32 channels, reorder inside the heads.  The
// scores come from k_scores_row2 (a key phase of SUB masked passes over the sub-blocks was the
// first design and measured slower); here every value head has SUB (scale, zero-point) pairs per
// token, so the softmax phase makes SUB sets of weight digits and a wave of the value phase takes
// the set of the sub-block its 32 channels lie in.  (HB composes with SUB and PRE: the value phase's plane of
// upper bits does not depend on where the scores and the weights come from.)
// ALU: measurement only.  The same kernel with the cache stream - K codes, K metadata, V codes,
// V metadata - replaced by values made up in registers (from the lane number and a kernel
// argument, so that nothing folds at compile time): what the arithmetic alone costs when no byte
// of the cache has to arrive.  The results mean nothing.
// PRE: the scores of the compressed stream come from a buffer [sequence][query head][token slot]
// (-infinity at retained sink tokens) in place of the key phase - a reorder over the whole token
// row, whose scores k_scores_row computes; qt then points to that buffer.  Softmax, values and
// partial results as in the plain kernel.
// STEP: a whole decode step but for the merge.  The sequences' last token is new: the workgroup whose chunk holds it appends it
// first (rkv_append_one: two round trips and a barrier more for one workgroup in nch), and every workgroup rotates the queries
// of its rotation group itself - one channel pair per thread, two positions -, the first chunk's leaving the plain copy for the
// merge.  That is what the launch in front did, 4 to 7 us of latency: one sequence x 4096 tokens 17.7 -> 15.9 us a step
// (rkv_step_in_decode).
template <int G, int REP, bool MULTI, bool META8, int HB, int SUB = 0, bool ALU = false, bool PRE = false, int TILES = MF_TILES, bool STEP = false>
__global__ void __launch_bounds__(256, (HB && G == 4 && TILES == 4) ? MF_OCC_HI : MF_OCC) k_decode_mfma(RkvView v, const float* __restrict__ qt,
                                                                       float* __restrict__ part, int nch,
                                                                       const int* __restrict__ q_lim, int nq, int ns, uint32_t inv_ns, uint32_t inv_nrg,
                                                                       RkvStepIn step) {
  constexpr bool HI = HB != 0;
  constexpr int CH = 64 * TILES;                 // tokens per workgroup (4 waves)
  constexpr int NH = G * REP;                    // query heads served by this workgroup: REP per KV head
  constexpr float MID = HB == 0 ? 1.5f : HB == 1 ? 3.5f : 7.5f;     // middle code
  __shared__ __attribute__((aligned(16))) float s_sc[NH][CH];
  // Weight digits of phase S for the matrix products of phase V, a part of its own for each wave: [query head][sub-block][digit] rows
  // of a byte per token (rows of a stride that spreads the operand's sixteen-byte pieces over the banks)
  constexpr int NS = SUB ? SUB : 1;              // sub-blocks of a value head (groups of 64 / 32): weights per sub-block
  constexpr int DROW = CH + 16;
  __shared__ __attribute__((aligned(16))) uint8_t s_dig[4][REP * NS * 6 * DROW];
  __shared__ int s_sink[64];
  __shared__ uint4 s_H[8][64];                   // Hadamard operand tiles
  __shared__ float2 s_step[64];                  // RoPE rotation by 16 positions, per channel pair
  __shared__ float s_c2[64];                     // 2 cos of one position's angle, per channel pair
  __shared__ uint4 s_q[2][4][G / 2][16];         // key phase: [r - 1][p][f / 4][n] x 4 floats f % 4, f = 2 * KV head + (lo, hi); version r: at position pos - r
  // Metadata of the chunk's keys and values (plain variants): fetched once, at the start, token by
  // token, and kept in LDS - a tile's worth held in registers a whole tile ahead of its use costs
  // 16 registers.
  // They are stored there in the form their users take: per token the scales of the group's blocks
  // as packed fp16 pairs (s_ks, key phase: the A operand of the small matrix products, up to signs), for the
  // values (scale, zero-point) per head (s_vm) - whatever the storage format was.  The keys'
  // zero-points never reach the key phase: H_128 of a constant block is 128 z e_0, so they only
  // touch channel 0 of every head, k^[a][0] -= (2 / sqrt(n)) * 64 * Z_a(t) with
  // Z_a(t) = sum_blk H_g[a][blk] * scale_blk * (zero_blk - the middle code), and channel 0 is one half of RoPE pair 0,
  // whose angle at token t is t itself.  Their share of the score of (token t, query head h),
  //     - 64 * Z_a(t) * (cos(t) * q~[h][pair 0, first half] + sin(t) * q~[h][pair 0, second half]),
  // is worked out once per token when the metadata are staged and put where the key phase adds
  // its sum (s_sc).
  constexpr bool LM = SUB == 0;
  constexpr int MWL = META8 ? G / 2 : G;             // metadata dwords per token and rotation group as stored
  constexpr int GP = G / 2;                          // packed pairs per token
  __shared__ __attribute__((aligned(16))) uint32_t s_ks[CH * GP], s_vm[LM ? G : 1][LM ? CH : 4];
  static_assert(SUB == 0 || PRE, "groups of 64 / 32 run on precomputed scores");
  static_assert(!ALU || (!META8 && HB == 0 && !MULTI), "the arithmetic-only measurement exists for the plain 2-bit variants");
  static_assert(!PRE || CH == 256, "precomputed scores: a thread per token of the chunk");
  static_assert(PRE || (REP == 1 && !MULTI), "the key phase serves one query head per KV head");
  static_assert(!PRE || !ALU, "precomputed scores: no arithmetic-only measurement");

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = lane & 15, q = lane >> 4;
  // Wave priority: the few instructions before the first barrier, and the short softmax and
  // value phases at the end, go ahead of the key phases of the compute unit's other workgroups
  // (which are dense vector work and fill every gap): a young wave otherwise waits behind them for
  // each of its instructions, and its workgroup's place on the compute unit idles meanwhile.
  __builtin_amdgcn_s_setprio(3);
  // The arguments the first microsecond needs, asked for in one go (left to itself the compiler
  // fetches each where it is first used, one scalar round trip after the other)
  asm volatile("" ::"s"(v.kc), "s"(v.km), "s"(v.vc), "s"(v.vm), "s"(v.rope), "s"(v.hop), "s"(v.sink_pos), "s"(v.sink_cnt), "s"(v.lens),
               "s"(qt), "s"(v.Tpad), "s"(v.NRG), "s"(v.B), "s"(v.len), "s"(v.max_sinks), "s"(nch), "s"(ns), "s"(inv_ns), "s"(inv_nrg));
  // row (n & 3) of H_g as fp16 sign masks for the packed scale pairs (blocks 0,1) and (2,3);
  // rows >= G are zero
  const int hrow = n & 3;
  const uint32_t keep_row = hrow < G ? 0xffffffffu : 0u;
  const uint32_t sm01 = ((__popc(hrow & 1) & 1) ? 0x80000000u : 0u);
  const uint32_t sm23 = ((__popc(hrow & 2) & 1) ? 0x00008000u : 0u) | ((__popc(hrow & 3) & 1) ? 0x80000000u : 0u);

  // On precomputed scores one workgroup serves REP of the `rep` query heads that share a KV head, which read the
  // same V codes; the workgroups of the other query-head groups read the chunk's again.
  // With per-sequence lengths the grid has no sequence dimension: the chunks of all sequences are
  // numbered consecutively (cstart[b] = chunks of the sequences before b), rounded up to 8 in all,
  // so that no workgroup is launched for chunks a shorter sequence does not have.
  // (ns = query-head groups of a KV head = rep / REP; the quotients below are taken with the
  // reciprocals the host passes - inv = ceil(2^32 / d), 0 for d = 1 -: a scalar integer division
  // is some thirty dependent instructions, several of them on the vector pipe that the compute
  // unit's other workgroups keep busy, and there were five of them before the first request)
  const int rep = ns * REP;
  int rg = blockIdx.y;
  int rrg, chunk, b;
  if (v.lens) {
    const int tot8 = gridDim.x / ns;
    rrg = blockIdx.x / tot8;
    constexpr int SPLIT = MF_CH / CH;            // (the table counts chunks of MF_CH tokens)
    const int w_ = blockIdx.x - rrg * tot8, w = w_ / SPLIT;
    if (w >= v.cstart[v.B]) return;
    int lo = 0, hi = v.B;                        // the last sequence whose first chunk is <= w and that has chunks
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (v.cstart[mid] <= w) lo = mid;
      else hi = mid;
    }
    b = lo;
    chunk = (w - v.cstart[b]) * SPLIT + w_ % SPLIT;
  } else {
    // One grid dimension.  Workgroups go to the chip's eight compute dies (each with an L2 of its
    // own) in turn, so id % 8 names the die: a die takes every eighth (sequence, rotation group)
    // and runs all of its chunks, and for each chunk the workgroups of all query-head groups one
    // after the other.  What those workgroups share - the prepared queries, the sink list, and
    // with GQA the chunk's codes themselves - is then fetched into one L2 once.
    // (grid: x = 8 * nch * ns, y = eighths of the (sequence, rotation group) pairs; x runs fastest)
    const int xcd = blockIdx.x & 7, rem = blockIdx.x >> 3;
    chunk = inv_ns ? (int)__umulhi((uint32_t)rem, inv_ns) : rem;
    rrg = rem - chunk * ns;
    // A step's chunk with the append lives the longest: where a die runs several pairs it goes first, so as not to be behind all
    // others (us per step: 16 sequences x 4096, 40 heads 67.3 -> 65.7; 8 x 4096, rotation over two heads 39.3 -> 37.4).  With one pair
    // per die the order stays: one x 32768, 36.1 and in reverse 37.3 to 38.0.
    if constexpr (STEP)
      if (gridDim.y > 1) chunk = nch - 1 - chunk;
    const int br = blockIdx.y * 8 + xcd;
    if (br >= v.B * v.NRG) return;
    b = inv_nrg ? (int)__umulhi((uint32_t)br, inv_nrg) : br;
    rg = br - b * v.NRG;
  }
  int len = rkv_len(v, b);
  if (chunk * CH >= len) return;
  const int t0 = chunk * CH;
  // (on scores of its own: one query token per sequence, which may lie before the sequence's end; a chunk behind it has weights of zero)
  if constexpr (!PRE)
    if (q_lim) len = min(len, q_lim[b] + 1);

  // Everything the workgroup needs before its first tile is requested here, back to back, and put
  // in LDS further down, once - a request that is waited for before the next one goes out costs a
  // round trip to L2 or memory each, and the workgroup's place on the compute unit idles meanwhile
  // (six such round trips were a quarter of a workgroup's life).
  //  - Hadamard operand tiles (the key phase reads two of them per step)
  const uint4 ld_h0 = reinterpret_cast<const uint4*>(v.hop)[tid], ld_h1 = reinterpret_cast<const uint4*>(v.hop)[tid + 256];
  //  - queries of this rotation group, already RoPE'd, scaled and laid out as s_q by k_prep_q
  constexpr int Q16 = 2 * 16 * 4 * 2 * G / 4;            // 16-byte pieces in all
  constexpr int QN = (Q16 + 255) / 256;                  // per thread
  const uint4* q_src = reinterpret_cast<const uint4*>(qt + ((size_t)b * v.NRG + rg) * (2 * 16 * 4 * 2 * G));
  uint4 ld_q[QN];
#pragma unroll
  for (int i = 0; i < QN; ++i) ld_q[i] = !STEP && tid + 256 * i < Q16 ? q_src[tid + 256 * i] : make_uint4(0, 0, 0, 0);
  //  - RoPE angles are kept for the first of a lane's four tokens only; the query's copies at positions 1 and 2 back make
  //    up for it (rkv_prep_q_one).  The next tile follows by
  //    rotating 16 positions (table row 16; used once per tile, read from LDS)
  const float2 ld_step = v.rope[16 * 64 + (tid & 63)];
  const float ld_c2 = 2.0f * v.rope[64 + (tid & 63)].x;
  //  - the sink list: positions unconditionally (the store holds max_sinks of them, unused ones -1), masked by the count below
  const int ld_cnt = v.max_sinks > 0 ? v.sink_cnt[b] : 0;
  const int ld_spos = (v.max_sinks > 0 && (tid & 63) < v.max_sinks) ? v.sink_pos[b * v.max_sinks + (tid & 63)] : -1;
  //  - (a step) channel pair tid mod 64 of query head tid / 64 and its angles at the last three positions; pair 0 of head `lane`
  [[maybe_unused]] float st_x = 0.f, st_y = 0.f, st_x0 = 0.f, st_y0 = 0.f;
  [[maybe_unused]] float2 st_cs[3], st_cs0;
  [[maybe_unused]] const int qa = tid >> 6, qj = tid & 63;
  if constexpr (STEP) {
    const __half* qrow = step.q + ((size_t)b * v.Hq + rg * G) * RKV_D;
    const __half* row = qrow + (qa < G ? qa : 0) * RKV_D;
    st_x = __half2float(row[v.rope_style ? 2 * qj : qj]);
    st_y = __half2float(row[v.rope_style ? 2 * qj + 1 : qj + 64]);
    st_x0 = __half2float(qrow[(lane & (G - 1)) * RKV_D]);
    st_y0 = __half2float(qrow[(lane & (G - 1)) * RKV_D + (v.rope_style ? 1 : 64)]);
#pragma unroll
    for (int r = 0; r < 3; ++r) st_cs[r] = v.rope[(size_t)(len - 1 - r) * 64 + qj];      // (a step of this kind leaves at least three tokens)
    st_cs0 = v.rope[(size_t)(len - 1) * 64];
    if (len - 1 >= t0 && len - 1 < t0 + CH) {                // the chunk of the new token
      __shared__ RkvOneLds one;
      rkv_append_one<G, HB>(v, step.k + (size_t)b * v.E, step.v + (size_t)b * v.E, len - 1, b, rg, one);
      __syncthreads();                                       // (its codes and metadata are read below like any other's)
    }
  }
  //  - (plain variants) the metadata of token t0 + tid of keys and values, its RoPE angle for channel
  //    pair 0 and the queries' entries for that pair: staged below
  uint32_t ld_mk[4] = {0, 0, 0, 0}, ld_mv[4] = {0, 0, 0, 0};
  float2 ld_cs0 = make_float2(0.f, 0.f);
  float ld_q0[G][2];
  if constexpr (!PRE) {
    const size_t mi = ((size_t)(b * v.NRG + rg) * v.Tpad + t0 + tid) * MWL;
    auto fetch = [&](const uint32_t* g, uint32_t (&d)[4]) {
      if constexpr (ALU) return;
      if constexpr (MWL == 4) {
        const uint4 u = rkv_ld_stream(reinterpret_cast<const uint4*>(g));
        d[0] = u.x; d[1] = u.y; d[2] = u.z; d[3] = u.w;
      } else if constexpr (MWL == 2) {
        const uint2 u = rkv_ld_stream(reinterpret_cast<const uint2*>(g));
        d[0] = u.x; d[1] = u.y;
      } else {
        d[0] = *g;
      }
    };
    if (CH == 256 || tid < CH) {
      fetch(v.km + mi, ld_mk);
      fetch(v.vm + mi, ld_mv);
      ld_cs0 = v.rope[(size_t)(t0 + tid) * 64];
    }
    // channel pair 0 of the queries at their own position (the plain copy, in front of the other), scaled like the other
    const float* q_nat = qt - (size_t)v.B * v.Hq * RKV_D + ((size_t)b * v.Hq + rg * G) * RKV_D;
    const float lane_scale = 2.0f * rsqrtf((float)v.n);
    if constexpr (STEP) {
      const int l = __float_as_int(rkv_prep_q_turn(st_x0, st_y0, -1.f, st_cs0.x, st_cs0.y) * lane_scale);
      const int h = __float_as_int(rkv_prep_q_turn(st_y0, st_x0, 1.f, st_cs0.x, st_cs0.y) * lane_scale);
#pragma unroll
      for (int i = 0; i < G; ++i) {
        ld_q0[i][0] = __int_as_float(__builtin_amdgcn_readlane(l, i));
        ld_q0[i][1] = __int_as_float(__builtin_amdgcn_readlane(h, i));
      }
    } else {
#pragma unroll
      for (int i = 0; i < G; ++i) {
        ld_q0[i][0] = q_nat[i * RKV_D] * lane_scale;
        ld_q0[i][1] = q_nat[i * RKV_D + (v.rope_style ? 1 : 64)] * lane_scale;
      }
    }
  }
  //  - the RoPE angles of this lane's first token and the first key tile: in the key phase below
  [[maybe_unused]] int per_query = 1;            // query heads of a KV head per query token
  if constexpr (MULTI) per_query = rep / nq;

  const int cnt = ld_cnt;
  {
    if constexpr (PRE) {
      // thread = token of the chunk: its scores from the buffer, its value metadata to LDS (with
      // groups of 64 / 32 the softmax phase fetches the sub-blocks' metadata itself)
      uint32_t dv[G];
      if constexpr (LM && META8) {
        // G scale bytes, then G zero-point bytes -> (scale, zero-point) fp16 pairs, the form the softmax phase takes
        const uint8_t* vm8 = reinterpret_cast<const uint8_t*>(v.vm) + ((size_t)(b * v.NRG + rg) * v.Tpad + t0 + tid) * (2 * G);
        uint32_t sw, zw;
        if constexpr (G == 4) {
          const uint2 u = rkv_ld_stream(reinterpret_cast<const uint2*>(vm8));
          sw = u.x; zw = u.y;
        } else {
          sw = *reinterpret_cast<const uint32_t*>(vm8);
          zw = sw >> 16;
        }
        dv[0] = rkv_pack_meta(__builtin_amdgcn_cvt_f32_fp8((int)sw, 0), (float)(zw & 0xffu) - 128.0f);
        dv[1] = rkv_pack_meta(__builtin_amdgcn_cvt_f32_fp8((int)sw, 1), (float)((zw >> 8) & 0xffu) - 128.0f);
        if constexpr (G == 4) {
          dv[2] = rkv_pack_meta(__builtin_amdgcn_cvt_f32_fp8((int)sw, 2), (float)((zw >> 16) & 0xffu) - 128.0f);
          dv[3] = rkv_pack_meta(__builtin_amdgcn_cvt_f32_fp8((int)sw, 3), (float)(zw >> 24) - 128.0f);
        }
      } else if constexpr (LM) {
        const size_t mi = ((size_t)(b * v.NRG + rg) * v.Tpad + t0 + tid) * G;
        if constexpr (G == 4) {
          const uint4 u = rkv_ld_stream(reinterpret_cast<const uint4*>(v.vm + mi));
          dv[0] = u.x; dv[1] = u.y; dv[2] = u.z; dv[3] = u.w;
        } else {
          const uint2 u = rkv_ld_stream(reinterpret_cast<const uint2*>(v.vm + mi));
          dv[0] = u.x; dv[1] = u.y;
        }
      }
      float pre[NH];
#pragma unroll
      for (int a = 0; a < G; ++a)
#pragma unroll
        for (int rri = 0; rri < REP; ++rri) {
          const int qh = (rg * G + a) * rep + rrg * REP + rri;
          bool seen = t0 + tid < len;
          // (several query tokens: virtual head rrg * REP + rri of its KV head belongs to query token (that / heads per token))
          if constexpr (MULTI) seen = seen && t0 + tid <= q_lim[b * nq + (rrg * REP + rri) / per_query];
          pre[a * REP + rri] = seen ? qt[((size_t)b * v.Hq + qh) * v.Tpad + t0 + tid] : -INFINITY;
        }
      if (tid < 64) s_sink[tid] = tid < cnt ? ld_spos : -1;
      if constexpr (LM) {
#pragma unroll
        for (int i = 0; i < G; ++i) s_vm[i][tid] = dv[i];
      }
#pragma unroll
      for (int a = 0; a < NH; ++a) s_sc[a][tid] = pre[a];
      __syncthreads();
    } else {
    // ------------------------------------------------------------------ phase K
    {
      const int tw = t0 + wave * (16 * TILES);
      float cs_c[4], cs_s[4];
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const float2 cs = v.rope[(size_t)(tw + 4 * q) * 64 + 16 * p + n];
        cs_c[p] = cs.x;
        cs_s[p] = cs.y;
      }
      const uint4* ktiles = reinterpret_cast<const uint4*>(v.kc + rkv_k_tilebase(v, b, rg, tw >> 4));
      // the plane above the low two bits: 16 bytes per lane and pair of blocks (HB = 2) or 8 (HB = 1)
      const uint32_t* khtiles = HI ? v.kh + (rkv_k_tilebase(v, b, rg, tw >> 4) >> (HB == 1 ? 1 : 0)) : nullptr;

      uint4 cw[G / 2], cwh[HI ? G / 2 : 1];
      auto load_tile = [&](int ti) {
        if constexpr (ALU) {                                 // made-up codes
          const uint32_t x = (uint32_t)lane * 2654435761u ^ (uint32_t)(nq + ti);
#pragma unroll
          for (int pr = 0; pr < G / 2; ++pr) cw[pr] = make_uint4(x, x * 3u, x * 5u, x * 7u + pr);
        }
#pragma unroll
        for (int pr = 0; pr < G / 2; ++pr) if constexpr (!ALU) cw[pr] = rkv_ld_stream(ktiles + (size_t)ti * (32 * G) + pr * 64 + lane);
        if constexpr (HI) {
#pragma unroll
          for (int pr = 0; pr < G / 2; ++pr) {
            const size_t li = (size_t)ti * (32 * G) + pr * 64 + lane;
            if constexpr (HB == 2) {
              cwh[pr] = rkv_ld_stream(reinterpret_cast<const uint4*>(khtiles) + li);
            } else {
              const uint2 u = rkv_ld_stream(reinterpret_cast<const uint2*>(khtiles) + li);
              cwh[pr] = make_uint4(u.x, u.y, 0, 0);
            }
          }
        }
      };
      load_tile(0);
      // (the requests are all out: what came back goes to LDS)
      (&s_H[0][0])[tid] = ld_h0;
      (&s_H[0][0])[tid + 256] = ld_h1;
      if constexpr (STEP) {
        if (qa < G) {
          const float lane_scale = 2.0f * rsqrtf((float)v.n);
          float* const qf = reinterpret_cast<float*>(&s_q[0][0][0][0]);
#pragma unroll
          for (int r = 1; r < 3; ++r) {
            float* const at = qf + ((((r - 1) * 4 + (qj >> 4)) * (G / 2) + (qa >> 1)) * 16 + (qj & 15)) * 4 + 2 * (qa & 1);
            at[0] = rkv_prep_q_turn(st_x, st_y, -1.f, st_cs[r].x, st_cs[r].y) * lane_scale;
            at[1] = rkv_prep_q_turn(st_y, st_x, 1.f, st_cs[r].x, st_cs[r].y) * lane_scale;
          }
          if (chunk == 0) {                                  // the plain copy, which the merge reads
            float* const qn = step.qr + ((size_t)b * v.Hq + rg * G + qa) * RKV_D;
            qn[v.rope_style ? 2 * qj : qj] = rkv_prep_q_turn(st_x, st_y, -1.f, st_cs[0].x, st_cs[0].y);
            qn[v.rope_style ? 2 * qj + 1 : qj + 64] = rkv_prep_q_turn(st_y, st_x, 1.f, st_cs[0].x, st_cs[0].y);
          }
        }
      } else {
#pragma unroll
        for (int i = 0; i < QN; ++i)
          if (tid + 256 * i < Q16) (&s_q[0][0][0][0])[tid + 256 * i] = ld_q[i];
      }
      if (tid < 64) {
        s_step[tid] = ld_step;
        s_c2[tid] = ld_c2;
        s_sink[tid] = tid < cnt ? ld_spos : -1;              // complete after the barrier that precedes the key phase
      }
      if (CH == 256 || tid < CH) {                     // thread = token of the chunk (inside the padded allocation)
        // a token's metadata as stored -> packed fp16 pairs (s01, s23) and (z01, z23)
        auto pairs = [&](const uint32_t* src, uint32_t (&sp)[2], uint32_t (&zp)[2]) {
          sp[1] = zp[1] = 0;
          if constexpr (ALU) {                               // scale 1, zero-point 0
            sp[0] = sp[1] = 0x3C003C00u + (uint32_t)(nq - 1);
            zp[0] = zp[1] = 0;
          } else if constexpr (META8) {
            // G scale bytes, then G zero-point bytes.  FP8 -> fp32 -> fp16 is exact; a zero-point byte
            // u = z + 128 under the high byte 0x64 is the fp16 number 1024 + u
            const uint32_t d0 = src[0], dz = G == 4 ? src[1] : src[0] >> 16;
            const v2h off = {(_Float16)1152.0f, (_Float16)1152.0f};
            const auto f01 = __builtin_amdgcn_cvt_pk_f32_fp8((int)d0, false);
            sp[0] = pk_f16(f01[0], f01[1]);
            zp[0] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(v2h, __builtin_amdgcn_perm(0x64646464u, dz, 0x04010400u)) - off);
            if constexpr (G == 4) {
              const auto f23 = __builtin_amdgcn_cvt_pk_f32_fp8((int)d0, true);
              sp[1] = pk_f16(f23[0], f23[1]);
              zp[1] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(v2h, __builtin_amdgcn_perm(0x64646464u, dz, 0x04030402u)) - off);
            }
          } else {                                           // (scale, zero-point) fp16 pairs per block
            sp[0] = __builtin_amdgcn_perm(src[1], src[0], 0x05040100u);
            zp[0] = __builtin_amdgcn_perm(src[1], src[0], 0x07060302u);
            if constexpr (G == 4) {
              sp[1] = __builtin_amdgcn_perm(src[3], src[2], 0x05040100u);
              zp[1] = __builtin_amdgcn_perm(src[3], src[2], 0x07060302u);
            }
          }
        };
        uint32_t sp[2], zp[2];
        uint32_t (&dk)[4] = ld_mk, (&dv)[4] = ld_mv;
        pairs(dk, sp, zp);
    #pragma unroll
        for (int i = 0; i < GP; ++i) s_ks[tid * GP + i] = sp[i];
        {
          // the zero-points' share of this token's scores (see above); -infinity past the sequence's end,
          // which is what a slot the key phase never writes must hold
          float sf[4], zf[4];
    #pragma unroll
          for (int i = 0; i < 4; ++i) {
            const uint32_t sw = sp[i >> 1], zw = zp[i >> 1];
            sf[i] = i < G ? (float)__builtin_bit_cast(_Float16, (uint16_t)(i & 1 ? sw >> 16 : sw & 0xffffu)) : 0.f;
            zf[i] = i < G ? (float)__builtin_bit_cast(_Float16, (uint16_t)(i & 1 ? zw >> 16 : zw & 0xffffu)) : 0.f;
          }
          const float2 cs0 = ld_cs0;
    #pragma unroll
          for (int a = 0; a < G; ++a) {
            float Z = 0.f;
    #pragma unroll
            for (int i = 0; i < G; ++i) Z = fmaf((__popc(a & i) & 1) ? -sf[i] : sf[i], zf[i] - MID, Z);
            s_sc[a][tid] = t0 + tid < len ? -64.0f * Z * fmaf(cs0.x, ld_q0[a][0], cs0.y * ld_q0[a][1]) : -INFINITY;
          }
        }
        if constexpr (META8 || ALU) {                      // values: (scale, zero-point) per head
          pairs(dv, sp, zp);
          s_vm[0][tid] = __builtin_amdgcn_perm(zp[0], sp[0], 0x05040100u);
          s_vm[1][tid] = __builtin_amdgcn_perm(zp[0], sp[0], 0x07060302u);
          if constexpr (G == 4) {
            s_vm[2][tid] = __builtin_amdgcn_perm(zp[1], sp[1], 0x05040100u);
            s_vm[3][tid] = __builtin_amdgcn_perm(zp[1], sp[1], 0x07060302u);
          }
        } else {
    #pragma unroll
          for (int i = 0; i < G; ++i) s_vm[i][tid] = dv[i];
        }
      }
      __syncthreads();        // LDS copies of the Hadamard operand and the query are complete; first tile already in flight
      __builtin_amdgcn_s_setprio(0);
      // which of the wave's tiles hold a retained sink token (a wave-uniform bit mask): the others
      // skip the comparison with the sink list
      uint32_t sink_tiles = 0;
      for (int i = 0; i < cnt; ++i) {
        const int d = s_sink[i] - tw;
        if (d >= 0 && d < 16 * TILES) sink_tiles |= 1u << (d >> 4);
      }
      sink_tiles = __builtin_amdgcn_readfirstlane(sink_tiles);

#pragma unroll
      for (int ti = 0; ti < TILES; ++ti) {
        const int tt = tw + ti * 16;
        if (tt >= len) break;                              // wave-uniform
        v8i A[G];
#pragma unroll
        for (int pr = 0; pr < G / 2; ++pr) {
          A[2 * pr] = unpack_fp4(cw[pr].x, cw[pr].y);
          A[2 * pr + 1] = unpack_fp4(cw[pr].z, cw[pr].w);
        }
        v8i Ah[HI ? G : 1];
        if constexpr (HI) {
#pragma unroll
          for (int pr = 0; pr < G / 2; ++pr) {
            if constexpr (HB == 2) {
              Ah[2 * pr] = unpack_fp4(cwh[pr].x, cwh[pr].y);
              Ah[2 * pr + 1] = unpack_fp4(cwh[pr].z, cwh[pr].w);
            } else {
              Ah[2 * pr] = unpack_fp4_bits(cwh[pr].x);
              Ah[2 * pr + 1] = unpack_fp4_bits(cwh[pr].y);
            }
          }
        }
        // scale rows of the 4x4 products: (+-s_0, +-s_1, +-s_2, +-s_3) of token 4q + r, signs of H_g row n & 3
        v4h sA[4];
        {
          const uint32_t* sp = &s_ks[(wave * (16 * TILES) + ti * 16 + 4 * q) * GP];
          uint32_t sw[4][2];
          if constexpr (G == 4) {
#pragma unroll
            for (int r = 0; r < 4; r += 2) {
              const uint4 a = *reinterpret_cast<const uint4*>(sp + 2 * r);
              sw[r][0] = a.x; sw[r][1] = a.y; sw[r + 1][0] = a.z; sw[r + 1][1] = a.w;
            }
          } else {
            const uint4 a = *reinterpret_cast<const uint4*>(sp);
            sw[0][0] = a.x; sw[1][0] = a.y; sw[2][0] = a.z; sw[3][0] = a.w;
            sw[0][1] = sw[1][1] = sw[2][1] = sw[3][1] = 0;
          }
#pragma unroll
          for (int r = 0; r < 4; ++r) sA[r] = as_v4h((sw[r][0] ^ sm01) & keep_row, G == 4 ? (sw[r][1] ^ sm23) & keep_row : 0u);
        }
        if (ti + 1 < TILES) load_tile(ti + 1);          // prefetch (inside the padded allocation)

        // (One pass.  Without the loop some variants wait for the value codes before the softmax phase's barrier instead of behind
        // it: one sequence x 8192 tokens, 4-bit codes, half chunks, 21.7 -> 22.3 us a call; 2-bit codes are the same within 1 %.)
#pragma unroll
        for (int pass = 0; pass < 1; ++pass) {
        const float centre = n == 0 ? -64.0f * MID : 0.f;  // channel 0 of H_128 of the constant MID / 2
        const v4f centre4 = {centre, centre, centre, centre};
        float pt[4 * G];                                   // [token of the lane][KV head]
#pragma unroll
        for (int i = 0; i < 4 * G; ++i) pt[i] = 0.f;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          // k^[a] = sum_blk H_g[a][blk] * scale_blk * u_blk for the channels 16p + n and 16p + n + 64 - or the even and the odd
          // channel of pair 16p + n -, u = H_128 of the raw codes: half-integers, exact
          const float c = cs_c[p], s = cs_s[p], cc = s_c2[16 * p + n];  // angles of token 4q
          v4f k[2][4];
#pragma unroll
          for (int half = 0; half < 2; ++half) {
            v4f u[G];
            {
              v8i H;
              const uint4 h0 = s_H[p + 4 * half][lane];
              H[0] = (int)h0.x; H[1] = (int)h0.y; H[2] = (int)h0.z; H[3] = (int)h0.w; H[4] = H[5] = H[6] = H[7] = 0;
              const v4f zero4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
              for (int blk = 0; blk < G; ++blk) u[blk] = mfma_fp4(A[blk], H, p == 0 && half == 0 ? centre4 : zero4);
              if constexpr (HI) {
                // FP4 1.0 (0x2) and -1.0 (0xA) with bit 2 set are 4.0 and -4.0
#pragma unroll
                for (int i = 0; i < 4; ++i) H[i] |= 0x44444444;
#pragma unroll
                for (int blk = 0; blk < G; ++blk) u[blk] = mfma_fp4(Ah[blk], H, u[blk]);
              }
            }
            // The butterfly H_g over the blocks with their scales: 16 independent 4x4x4 products per instruction - block = (token
            // 4q + r, 4 channel lanes), A row a = signed fp16 scales, B = the four blocks' results (exact in fp16), fp32 accumulate
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const v4f z4 = {0.f, 0.f, 0.f, 0.f};
              if constexpr (G == 4) k[half][r] = mfma_4x4x4(sA[r], as_v4h(pk_f16(u[0][r], u[1][r]), pk_f16(u[2][r], u[3][r])), z4);
              else k[half][r] = mfma_4x4x4(sA[r], as_v4h(pk_f16(u[0][r], u[1][r]), 0u), z4);
            }
          }
          // RoPE is put on the query: <R(4q + r) k, q~> = <k, x_r>, x_r the query rotated back to token 4q + r.  Tokens 4q + 1 and
          // 4q + 2 from the query's two copies, their neighbours by x(t + 1) + x(t - 1) = 2 cos(1) x(t), one multiply-add per
          // number: twelve operations for four tokens where rotating each key took sixteen (and eight for the dot products in
          // either form).  16 sequences x 4096 tokens, 40 heads: 76.4 -> 71.4 us a step.
#pragma unroll
          for (int i = 0; i < 2 * G; i += 4) {
            const uint4 w1 = s_q[0][p][i / 4][n], w2 = s_q[1][p][i / 4][n];
            const float q1[4] = {__uint_as_float(w1.x), __uint_as_float(w1.y), __uint_as_float(w1.z), __uint_as_float(w1.w)};
            const float q2[4] = {__uint_as_float(w2.x), __uint_as_float(w2.y), __uint_as_float(w2.z), __uint_as_float(w2.w)};
#pragma unroll
            for (int a2 = 0; a2 < 2; ++a2) {
              const int a = i / 2 + a2;
#pragma unroll
              for (int half = 0; half < 2; ++half) {
                const float x1 = half == 0 ? q1[2 * a2] * c + q1[2 * a2 + 1] * s : q1[2 * a2 + 1] * c - q1[2 * a2] * s;
                const float x2 = half == 0 ? q2[2 * a2] * c + q2[2 * a2 + 1] * s : q2[2 * a2 + 1] * c - q2[2 * a2] * s;
                pt[0 * G + a] = fmaf(k[half][0][a], fmaf(cc, x1, -x2), pt[0 * G + a]);
                pt[1 * G + a] = fmaf(k[half][1][a], x1, pt[1 * G + a]);
                pt[2 * G + a] = fmaf(k[half][2][a], x2, pt[2 * G + a]);
                pt[3 * G + a] = fmaf(k[half][3][a], fmaf(cc, x2, -x1), pt[3 * G + a]);
              }
            }
          }
        }
        // on to the next tile's first token, 16 positions from this tile's
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          const float c = cs_c[p], s = cs_s[p];
          const float2 st = s_step[16 * p + n];
          cs_c[p] = c * st.x - s * st.y;
          cs_s[p] = s * st.x + c * st.y;
        }
        // reduce over the 16 channel lanes: value idx = r * G + a (token 4q + r, head a) ends in lane idx, and is added to the
        // zero-points' share, put there when the metadata were staged
        const float tot = row_transpose_reduce<4 * G>(pt, n);
        const int idx = n & (4 * G - 1), tok = tt + 4 * q + idx / G, a = idx % G;
        bool masked = tok >= len;
        if (sink_tiles & (1u << ti))
          for (int i = 0; i < cnt; ++i) masked |= (s_sink[i] == tok);
        if (n < 4 * G) s_sc[a][tok - t0] = masked ? -INFINITY : tot + s_sc[a][tok - t0];
        }
      }
    }
    }
    __builtin_amdgcn_s_setprio(3);
    // ------------------------------------------------------------------ phases S and V
    // wave -> KV head a, channel tiles: all eight (G = 4), or one half of them (G = 2; the head's two waves make the same digits)
    constexpr int NB = G == 4 ? 4 : 2;             // blocks of 32 channels per wave
    constexpr int NQ = CH / 128;                   // contractions of 128 tokens
    constexpr int NT = CH / 64;                    // tokens of a lane in phase S: consecutive ones
    const int a = wave & (G - 1), wb = G == 4 ? 0 : (wave >> 1) * 2;
    // Groups of 64 / 32: the V metadata of the lane's tokens - otherwise they are in LDS
    [[maybe_unused]] uint32_t vmeta[NS][NT];
    if constexpr (SUB != 0) {
#pragma unroll
      for (int i = 0; i < NT; ++i) {
        const size_t mi = ((size_t)(b * v.NRG + rg) * v.Tpad + t0 + NT * lane + i) * (G * NS);
        if constexpr (META8) {
          // the head's NS scale bytes and NS zero-point bytes, one load each
          const uint8_t* vm8 = reinterpret_cast<const uint8_t*>(v.vm) + 2 * mi + a * NS;
          uint32_t sw, zw;
          if constexpr (NS == 4) {
            sw = *reinterpret_cast<const uint32_t*>(vm8);
            zw = *reinterpret_cast<const uint32_t*>(vm8 + G * NS);
          } else {
            sw = *reinterpret_cast<const uint16_t*>(vm8);
            zw = *reinterpret_cast<const uint16_t*>(vm8 + G * NS);
          }
#pragma unroll
          for (int sb = 0; sb < NS; ++sb) vmeta[sb][i] = __builtin_amdgcn_perm(zw, sw, 0x0c0c0000u | ((4u + sb) << 8) | sb);
        } else {
#pragma unroll
          for (int sb = 0; sb < NS; ++sb) vmeta[sb][i] = v.vm[mi + a * NS + sb];
        }
      }
    }
    const uint4* vslab = reinterpret_cast<const uint4*>(v.vc + rkv_v_slabbase(v, b, rg, t0 >> 5));
    const uint32_t* vhslab = HI ? v.vh + (rkv_v_slabbase(v, b, rg, t0 >> 5) >> (HB == 1 ? 1 : 0)) : nullptr;
    const int nslab = max(1, min(CH / 32, (len - t0 + 31) >> 5));   // (a chunk behind the query's position: weights of zero)
    // all V codes of the chunk's share of the wave: in flight while the softmax phase runs.  Lane group q holds slab 4 s + q, 32 of
    // the 128 tokens of a contraction (behind the sequence's end: the last one again, their weights are zero)
    uint4 vcodes[NQ][NB], vhcodes[HI ? NQ : 1][HI ? NB : 1];
#pragma unroll
    for (int s = 0; s < NQ; ++s)
#pragma unroll
      for (int w = 0; w < NB; ++w) {
        const uint32_t li = (uint32_t)(min(4 * s + q, nslab - 1) * (64 * G) + ((wb + w) * G + a) * 16 + n);
        if constexpr (ALU) {
          const uint32_t x = li * 2654435761u ^ (uint32_t)(nq + s);
          vcodes[s][w] = make_uint4(x, x * 3u, x * 5u, x * 7u);
        } else {
          vcodes[s][w] = rkv_ld_stream(vslab + li);
        }
        if constexpr (HB == 2) {
          vhcodes[s][w] = rkv_ld_stream(reinterpret_cast<const uint4*>(vhslab) + li);
        } else if constexpr (HB == 1) {
          const uint2 u = rkv_ld_stream(reinterpret_cast<const uint2*>(vhslab) + li);
          vhcodes[s][w] = make_uint4(u.x, u.y, 0, 0);
        }
      }
    __syncthreads();                               // all scores are there

    // ---- phase S: the head's statistics over the chunk, its weights as rows of digits in the wave's own part of LDS
    uint8_t* const dig = s_dig[wave];
    float hm[REP], hl[REP], hzs[REP][NS], hdown[REP][NS];
#pragma unroll
    for (int rri = 0; rri < REP; ++rri) {
      float sv[NT], w[NT], zv[NT];
      if constexpr (NT == 4) {
        const float4 x = *reinterpret_cast<const float4*>(&s_sc[a * REP + rri][4 * lane]);
        sv[0] = x.x; sv[1] = x.y; sv[2] = x.z; sv[3] = x.w;
      } else {
        const float2 x = *reinterpret_cast<const float2*>(&s_sc[a * REP + rri][2 * lane]);
        sv[0] = x.x; sv[1] = x.y;
      }
      [[maybe_unused]] uint32_t vmw[NT];
      if constexpr (LM) {
#pragma unroll
        for (int i = 0; i < NT; ++i) vmw[i] = s_vm[a][NT * lane + i];
      }
      float m = -INFINITY;
#pragma unroll
      for (int i = 0; i < NT; ++i) m = fmaxf(m, sv[i]);
      m = wave_allreduce<true>(m);
      float pe[NT], l = 0.f;
#pragma unroll
      for (int i = 0; i < NT; ++i) {
        pe[i] = sv[i] > -INFINITY ? __expf(sv[i] - m) : 0.f;
        l += pe[i];
      }
      hm[rri] = m;
      hl[rri] = wave_allreduce<false>(l);
#pragma unroll
      for (int sb = 0; sb < NS; ++sb) {                     // once, or once per sub-block of the head (its own scales and zero-points)
        float wmax = 0.f;
#pragma unroll
        for (int i = 0; i < NT; ++i) {
          float s_, z_;
          if constexpr (LM) {
            rkv_unpack_meta(vmw[i], s_, z_);
          } else if constexpr (META8) {
            s_ = __builtin_amdgcn_cvt_f32_fp8((int)vmeta[sb][i], 0);
            z_ = (float)((vmeta[sb][i] >> 8) & 0xffu) - 128.0f;
          } else {
            rkv_unpack_meta(vmeta[sb][i], s_, z_);
          }
          w[i] = pe[i] * s_;
          zv[i] = z_;
          wmax = fmaxf(wmax, w[i]);
        }
        wmax = wave_allreduce<true>(wmax);
        // 24-bit fixed point: largest weight lands in [2^23, 2^24); six base-16 digits.  (It is a 24-bit integer as it
        // stands, so no digit exceeds 15.)  A byte 0..15 read as E4M3 is that integer times 2^-9 - subnormals and the
        // first binade are one straight line -: the bytes of the lane's weights are brought together and parted into
        // their nibbles, nothing is converted
        int ex = 0;
        if (wmax > 0.f) frexpf(wmax, &ex);
        const float up = ldexpf(1.0f, 24 - ex), down = ldexpf(1.0f, ex - 24);
        float zs = 0.f;
        uint32_t W[4] = {0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < NT; ++i) {
          W[i] = (uint32_t)rintf(w[i] * up);
          zs += (float)W[i] * zv[i];
        }
        hzs[rri][sb] = wave_allreduce<false>(zs) * down;
        hdown[rri][sb] = down;
        const uint32_t p01 = __builtin_amdgcn_perm(W[1], W[0], 0x05010400u);       // bytes 0 of both, bytes 1 of both
        uint32_t by[3];                                                            // byte j of all the lane's weights
        by[2] = __builtin_amdgcn_perm(W[1], W[0], 0x0c0c0602u);
        if constexpr (NT == 4) {
          const uint32_t p23 = __builtin_amdgcn_perm(W[3], W[2], 0x05010400u);
          by[2] = __builtin_amdgcn_perm(__builtin_amdgcn_perm(W[3], W[2], 0x0c0c0602u), by[2], 0x05040100u);
          by[0] = __builtin_amdgcn_perm(p23, p01, 0x05040100u);
          by[1] = __builtin_amdgcn_perm(p23, p01, 0x07060302u);
        } else {
          by[0] = p01 & 0xffffu;
          by[1] = p01 >> 16;
        }
        uint8_t* const dst = dig + (rri * NS + sb) * (6 * DROW) + NT * lane;
#pragma unroll
        for (int k = 0; k < 6; ++k) {                       // most significant first
          const uint32_t dg = (k & 1) ? by[2 - k / 2] & 0x0f0f0f0fu : (by[2 - k / 2] >> 4) & 0x0f0f0f0fu;
          if constexpr (NT == 4) *reinterpret_cast<uint32_t*>(dst + k * DROW) = dg;
          else *reinterpret_cast<uint16_t*>(dst + k * DROW) = (uint16_t)dg;
        }
      }
    }
    wave_lds_fence();

    // ---- phase V: rows = 8 * query head + digit (the rows of digits that do not exist repeat one that does, their results are
    // not used), contraction over 128 tokens, columns = 16 channels of the head
    {
      const v4f zero4 = {0.f, 0.f, 0.f, 0.f};
      v4f acc[2 * NB], acch[HI ? 2 * NB : 1];
#pragma unroll
      for (int i = 0; i < 2 * NB; ++i) acc[i] = zero4;
      if constexpr (HI) {
#pragma unroll
        for (int i = 0; i < 2 * NB; ++i) acch[i] = zero4;
      }
      const uint8_t* const row = dig + ((REP == 2 ? (n >> 3) * NS * 6 : 0) + min(n & 7, 5)) * DROW + 16 * q;
#pragma unroll
      for (int s = 0; s < NQ; ++s) {
        if (4 * s < nslab) {                                // workgroup-uniform
          v8i D;
#pragma unroll
          for (int w = 0; w < NB; ++w) {
            if (w == 0 || (SUB == 4) || (SUB == 2 && NB == 4 && w == 2)) {
              // FP8 operand: lane group q holds tokens 16 q .. + 15 and 64 + 16 q .. + 15 of the 128
              const int sb = SUB == 4 ? wb + w : SUB == 2 ? (wb + w) >> 1 : 0;      // channels 32 (wb + w) .. + 31 lie in one sub-block
              const uint4 d0 = *reinterpret_cast<const uint4*>(row + sb * 6 * DROW + 128 * s), d1 = *reinterpret_cast<const uint4*>(row + sb * 6 * DROW + 128 * s + 64);
              D[0] = (int)d0.x; D[1] = (int)d0.y; D[2] = (int)d0.z; D[3] = (int)d0.w;
              D[4] = (int)d1.x; D[5] = (int)d1.y; D[6] = (int)d1.z; D[7] = (int)d1.w;
            }
#pragma unroll
            for (int ct = 0; ct < 2; ++ct) {
              const uint4 u = vcodes[s][w];
              acc[2 * w + ct] = mfma_fp8_fp4(D, ct ? unpack_fp4(u.z, u.w) : unpack_fp4(u.x, u.y), acc[2 * w + ct]);
              if constexpr (HI) {
                const uint4 uh = vhcodes[s][w];
                const v8i Bh = HB == 2 ? (ct ? unpack_fp4(uh.z, uh.w) : unpack_fp4(uh.x, uh.y)) : unpack_fp4_bits(ct ? uh.y : uh.x);
                acch[2 * w + ct] = mfma_fp8_fp4(D, Bh, acch[2 * w + ct]);
              }
            }
          }
        }
      }
      // Lane groups 0 and 1 hold the upper four and the lower two digits of the first query head's results (2 and 3: of the
      // second's).  They exchange half of the channel tiles each and put together the other half
      const bool up4 = (q & 1) == 0;
      float part_[2 * NB];
#pragma unroll
      for (int i = 0; i < 2 * NB; ++i) {
        v4f h = acc[i];
        if constexpr (HI) h += acch[i] * 4.0f;              // the upper plane counts fourfold
        const float two = h[0] * 16.0f + h[1];
        part_[i] = up4 ? ((two * 16.0f + h[2]) * 16.0f + h[3]) * 256.0f : two;
      }
      const int rr = q >> 1;
      float* const dst = part + (((size_t)b * v.Hq + (rg * G + a) * rep + rrg * REP + (REP == 2 ? rr : 0)) * nch + chunk) * RKV_PART_STRIDE;
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const float sum = (up4 ? part_[i] : part_[NB + i]) + __shfl_xor(up4 ? part_[NB + i] : part_[i], 16);
        if (rr < REP) {
          const int tile = 2 * wb + (up4 ? i : NB + i);     // 16 channels each
          const int sb = SUB ? tile * SUB / 8 : 0;
          float wsc = hdown[0][0], z = hzs[0][0];
#pragma unroll
          for (int r2 = 0; r2 < REP; ++r2)
#pragma unroll
            for (int s2 = 0; s2 < NS; ++s2)
              if ((r2 || s2) && rr == r2 && sb == s2) { wsc = hdown[r2][s2]; z = hzs[r2][s2]; }
          dst[4 + 16 * tile + n] = sum * (1024.0f * wsc) - z;  // (FP4 nibble = code / 2, digit byte = digit * 2^-9)
        }
      }
      if (rr < REP && up4 && n == 0 && wb == 0) {
        dst[0] = REP == 2 && rr ? hm[REP - 1] : hm[0];
        dst[1] = REP == 2 && rr ? hl[REP - 1] : hl[0];
      }
    }
  }
}



// a reorder across 128-blocks inside the rotation groups, groups of 128: scores from the scores kernel
// (the rotation group's own blocks in its table), softmax and values from this file's kernel
static bool mfma_cross_block(const rkv_cache* c) {
  const RkvView& v = c->v;
  return !c->blocks_aligned && c->in_groups && v.qg == 128 && rkv_scores_local(c);
}

// groups of 64 / 32 (the reorder inside the rotation groups, or over the whole row): the same route
static bool mfma_sub_groups(const rkv_cache* c) {
  const RkvView& v = c->v;
  return v.qg < 128 && rkv_scores_path(c);
}

int rkv_mfma_variant(const rkv_cache* c) {
  return rkv_row_supported(c) ? RKV_KERNEL_MFMA_ROW : mfma_cross_block(c) ? RKV_KERNEL_MFMA_CROSS : mfma_sub_groups(c) ? RKV_KERNEL_MFMA_SUB : RKV_KERNEL_MFMA;
}

bool rkv_mfma_supported(const rkv_cache* c) {
  const RkvView& v = c->v;
  if (mfma_cross_block(c) || mfma_sub_groups(c) || rkv_row_supported(c)) return true;
  // 2-bit codes, or wider ones (a second plane), in groups of 128
  return c->blocks_aligned && v.qg == 128 && (v.g == 2 || v.g == 4);
}

typedef void (*RkvDecodeFn)(RkvView, const float*, float*, int, const int*, int, int, uint32_t, uint32_t, RkvStepIn);

// The variant of the kernel a cache takes.  multi: several query tokens per sequence; share: query
// heads of a KV head per workgroup (1 or 2); alu: the arithmetic-only measurement.
static RkvDecodeFn pick_kernel(const rkv_cache* c, bool multi, int share, bool alu, int chunk, bool step = false) {
  const RkvView& v = c->v;
  // precomputed scores (groups of 64 / 32; a reorder over the whole row): softmax and value phases only
#define RKV_MF_PRE_M(G_, R_, S_, H_, M_) (v.meta8 ? k_decode_mfma<G_, R_, M_, true, H_, S_, false, true> : k_decode_mfma<G_, R_, M_, false, H_, S_, false, true>)
#define RKV_MF_PRE(G_, R_, S_, H_) (multi ? RKV_MF_PRE_M(G_, R_, S_, H_, true) : RKV_MF_PRE_M(G_, R_, S_, H_, false))
#define RKV_MF_PRE_SUB(G_, H_) (sub == 4 ? RKV_MF_PRE(G_, 1, 4, H_) : RKV_MF_PRE(G_, 1, 2, H_))
  if (v.qg < 128 && rkv_scores_path(c)) {                   // (groups of 64 / 32: codes of 2, 3 or 4 bits)
    const int sub = 128 / v.qg;
    if (v.g == 4) return v.hb == 2 ? RKV_MF_PRE_SUB(4, 2) : v.hb == 1 ? RKV_MF_PRE_SUB(4, 1) : RKV_MF_PRE_SUB(4, 0);
    return v.hb == 2 ? RKV_MF_PRE_SUB(2, 2) : v.hb == 1 ? RKV_MF_PRE_SUB(2, 1) : RKV_MF_PRE_SUB(2, 0);
  }
  if (rkv_scores_path(c)) {                                 // (a reorder over the whole row, or across blocks inside the rotation groups)
#define RKV_MF_PRE_X(G_, R_) (v.hb == 2 ? RKV_MF_PRE(G_, R_, 0, 2) : v.hb == 1 ? RKV_MF_PRE(G_, R_, 0, 1) : RKV_MF_PRE(G_, R_, 0, 0))
    if (v.g == 4) return share == 1 ? RKV_MF_PRE_X(4, 1) : RKV_MF_PRE_X(4, 2);
    return share == 1 ? RKV_MF_PRE_X(2, 1) : RKV_MF_PRE_X(2, 2);
#undef RKV_MF_PRE_X
  }
#undef RKV_MF_PRE_SUB
#undef RKV_MF_PRE
#undef RKV_MF_PRE_M
  if (alu) return v.g == 4 ? k_decode_mfma<4, 1, false, false, 0, 0, true> : k_decode_mfma<2, 1, false, false, 0, 0, true>;
#define RKV_MF_PICK_S(G_, M_, H_, T_) (step ? k_decode_mfma<G_, 1, false, M_, H_, 0, false, false, T_, true> : k_decode_mfma<G_, 1, false, M_, H_, 0, false, false, T_>)
#define RKV_MF_PICK_H(G_, H_, T_) (v.meta8 ? RKV_MF_PICK_S(G_, true, H_, T_) : RKV_MF_PICK_S(G_, false, H_, T_))
#define RKV_MF_PICK(G_, T_) (v.hb == 2 ? RKV_MF_PICK_H(G_, 2, T_) : v.hb == 1 ? RKV_MF_PICK_H(G_, 1, T_) : RKV_MF_PICK_H(G_, 0, T_))
  if (chunk == MF_CH) return v.g == 4 ? RKV_MF_PICK(4, MF_TILES) : RKV_MF_PICK(2, MF_TILES);
  return v.g == 4 ? RKV_MF_PICK(4, MF_TILES / 2) : RKV_MF_PICK(2, MF_TILES / 2);
#undef RKV_MF_PICK_H
#undef RKV_MF_PICK_S
#undef RKV_MF_PICK
}

// Workgroups of `chunk` tokens of a call, per group of query heads, on the busiest of the eight dies, times eight: what
// counts against the chip's compute units.  A die takes every eighth (sequence, rotation group) pair with all its
// chunks, so that a single sequence with two rotation groups keeps two dies busy; with per-sequence
// lengths the chunks of all sequences go to the dies in turn.
size_t rkv_mfma_load(const rkv_cache* c, int chunk) {
  const RkvView& v = c->v;
  if (!c->ragged) return ((size_t)v.B * v.NRG + 7) / 8 * 8 * ((v.len + chunk - 1) / chunk);
  size_t total = 0;
  for (int b = 0; b < v.B; ++b) total += (c->hlens[b] + MF_CH - 1) / MF_CH;
  return total * (MF_CH / chunk) * v.NRG;
}

// Tokens per workgroup.  Half chunks are half the tiles in turn, at the price of setting up twice as many
// workgroups, and they leave a last round of half its size.  Up to half a workgroup per compute unit they make a call 1.2 times
// as fast; up to one and a half (two rounds of whole chunks on some units become three half ones on all) 1.05 to
// 1.1 times, except where a workgroup has two column tiles (two fit a compute unit, not three) or the query heads
// have been given to several workgroups already (which half chunks would take back): there they lose.  Above that they
// lose.  Wider codes on k_decode_mfma with four heads in a rotation group, of whose whole chunks two fit a
// compute unit and of half ones three, take them a quarter of a workgroup further.  (k_decode_shared with one column tile: 1.2 times
// as fast up to half a workgroup, 1.02 to 1.05 above one and up to one and a half; at one workgroup per unit whole chunks are the
// faster ones by 1 to 7 %, which the rule does not use.)
// us a step (k_decode_mfma) or a call, whole / half chunks, at 0.5, 1, 2, 3 and 8 workgroups per unit:
//   k_decode_mfma, 2-bit codes             17.6 / 14.8, 17.6 / 17.1, 21.7 / 25.4, 28.0 / 32.5, 56.6 / 60.3
//   ... 3-bit                              19.3 / 16.2, 19.9 / 19.2, 24.4 / 28.4, 37.2 / 36.6, 77.1 / 78.7
//   ... 4-bit                              19.3 / 16.8, 19.9 / 19.3, 24.9 / 29.5, 38.7 / 39.5, 80.2 / 81.5
//   ... 2-bit, two heads per group                      15.5 / 15.5, 17.0 / 20.2,              41.3 / 49.0
//   ... 4-bit, two heads per group                      16.6 / 16.5, 19.1 / 23.0,              51.1 / 58.2
// and at 0.5, 1, 1.5, 1.75, 3 and 10:
//   k_decode_shared, 4 heads on each of 8  23.1 / 19.9, 23.6 / 25.2, 30.9 / 30.2, 31.1 / 34.6, 39.7 / 44.6, 97.0 / 114
//   ... 3-bit                              24.6 / 20.8, 25.8 / 26.7, 33.8 / 32.6, 34.2 / 37.5, 46.9 / 48.2, 124 / 135
//   ... 4-bit                              25.2 / 21.2, 26.2 / 27.0, 33.9 / 32.4, 35.0 / 38.0, 48.3 / 50.1, 130 / 142
//   ... two column tiles, 8 on each of 8   23.8 / 23.8, 29.3 / 31.7, 38.6 / 41.0, 40.8 / 49.7, 54.6 / 66.7, 145 / 195
// (The work space: partial results of half chunks are within what a caller brings.  The one built in for
// rkv_decode_attention_static, a single query's, may hold those of whole chunks only; the usual step then takes these, with it or without.)
int rkv_mfma_chunk(const rkv_cache* c, int nq) {
  const RkvView& v = c->v;
  if (rkv_scores_path(c) || c->decode_path == 3) return MF_CH;
  if (c->decode_chunk) return c->decode_chunk;
  const int rep = v.Hq / v.Hkv * (nq > 0 ? nq : 1);
  const bool shared = rkv_shared_decode(c, rep);
  size_t load = rkv_mfma_load(c, MF_CH);
  int quarters = v.hb && v.g == 4 ? 7 : 6;                  // of a workgroup per compute unit
  if (shared) {
    const int rs = rkv_shared_heads(c, rep, MF_CH), ns = (rep + rs - 1) / rs;
    load *= ns;
    quarters = ns > 1 || rs * v.g > 16 ? 2 : 6;
  }
  if (4 * load > quarters * (size_t)c->n_cu) return MF_CH;
  if (nq > 0) return MF_CH / 2;
  auto fits = [&](int chunk) {
    const size_t nch = ((size_t)v.len + chunk - 1) / chunk;
    return rkv_query_scratch_bytes(v.B, v.Hq) + (size_t)v.B * v.Hq * nch * RKV_PART_STRIDE * 4 + 256 <= RKV_STATIC_SCRATCH_BYTES;
  };
  return fits(MF_CH / 2) || !fits(MF_CH) ? MF_CH / 2 : MF_CH;
}

// Query heads of a KV head (virtual ones: times the query tokens) served by one workgroup: two on precomputed scores where
// their number is even (they read the same V codes), else one.  0: k_decode_shared, which serves them all.
int rkv_mfma_share(const rkv_cache* c, int heads_per_kv_head) {
  if (rkv_shared_decode(c, heads_per_kv_head)) return 0;    // all query heads of a KV head together: a query layout of its own
  if (c->v.qg < 128) return 1;                              // groups of 64 / 32: one query head per workgroup
  return heads_per_kv_head % 2 == 0 ? 2 : 1;
}

// The form of the prepared queries (rkv_prep_q_one): 0 k_decode_shared's, 2 the same unrotated, 1 k_decode_mfma's, -1 the plain copy alone.
// at_end: one query token per sequence, at the sequence's last token.
int rkv_prep_form(const rkv_cache* c, int heads_per_kv_head, bool at_end) {
  const int share = rkv_mfma_share(c, heads_per_kv_head);
  return share == 0 ? (at_end ? 2 : 0) : heads_per_kv_head == 1 && !rkv_scores_path(c) ? 1 : -1;
}

// Whether a decode step's token is appended, and its queries prepared, by k_decode_mfma itself (STEP): one query head per KV head,
// its own key phase, one length for all - with per-sequence lengths the step's launch in front sets the new ones -, at
// least two tokens before this one, so that the query's copies lie at positions the angle table has, and at most sixteen workgroups per
// compute unit: every one of them prepares the queries again.  us per step, with a launch in front and without: 1 workgroup
// per unit (one sequence x 4096, 32 heads) 17.7 / 15.9, 4 (x 32768) 38.1 / 35.2, 8 (64 x 1024) 59.9 / 57.1, 12 (16 x 4096, 48 heads) 80.5 /
// 79.4, 16 (16 x 8192) 101.6 / 99.2, 32 (16 x 16384) 192.4 / 192.3, 64 (32 x 8192, rotation over two heads) 238.2 / 242.2.
bool rkv_step_in_decode(const rkv_cache* c) {
  const RkvView& v = c->v;
  return rkv_mfma_variant(c) == RKV_KERNEL_MFMA && v.Hq == v.Hkv && c->decode_path != 3 && !c->ragged && v.len >= 2 &&
         rkv_mfma_load(c, rkv_mfma_chunk(c, 0)) <= 16 * (size_t)c->n_cu;
}

// nq == 0: the usual step, one query token that attends the whole cache (and, if set, the current
// token's exact row).  nq >= 1: nq query tokens per sequence, token i at position q_pos[b][i] and
// blind to cached tokens behind it; q, out and lse are then [batch][nq][heads][...] and the scratch
// buffer holds nq times the single-query size.
// q_prepared: the queries are already in the scratch block (rkv_launch_step_mfma put them there)
// step: the last token's rows and the raw queries, where the launch is the step itself (rkv_step_in_decode); *appended
// then says whether it went out, whatever becomes of the merge behind it
int rkv_launch_decode_mfma(rkv_cache* c, const __half* q, const int* q_pos, int nq, float* out, float* lse, void* scratch,
                           bool q_prepared, const RkvStepIn& step, bool* appended, hipStream_t s) {
  if (!rkv_mfma_supported(c)) return RKV_EINVAL;
  const bool multi = nq > 0;
  if (multi && (c->cur_k || !q_pos)) return RKV_EINVAL;
  if (!multi) nq = 1;
  RkvView v = c->v;
  v.Hq *= nq;                                               // virtual heads
  float* qr = (float*)scratch;
  const size_t qbytes = rkv_query_scratch_bytes(v.B, v.Hq);
  float* part = (float*)((char*)scratch + qbytes);
  const int rep = v.Hq / v.Hkv;
  const bool sg = mfma_sub_groups(c);
  const bool xb = mfma_cross_block(c) || sg;
  const bool row = rkv_scores_path(c);
  if (row && multi && !rkv_scores_multi_ok(c, nq)) return RKV_EINVAL;   // (the scores kernel serves 8 rows per KV head)
  const int share = rkv_mfma_share(c, rep);
  const bool at_end = !multi && !q_pos && !c->cur_k;
  if (!q_prepared && !step.q) rkv_launch_prep_q(v, q, q_pos, c->cur_k ? 1 : 0, qr, rkv_prep_form(c, rep, at_end), nq, s);
  float* qt = qr + (size_t)v.B * v.Hq * RKV_D;              // lane-ordered copy written by k_prep_q
  const int chunk = rkv_mfma_chunk(c, multi ? nq : 0), split = MF_CH / chunk;
  const int nch = (v.len + chunk - 1) / chunk;
  if (share == 0) {
    const bool timed = c->ev_start && c->ev_stop;
    if (nch > 0) {
      const int rc = rkv_launch_decode_shared(c, v, qr, part, nch, chunk, multi ? q_pos : nullptr, nq, at_end, timed ? c->ev_start : nullptr,
                                              timed ? c->ev_stop : nullptr, s);
      if (rc != RKV_OK) return rc;
    } else if (timed) {
      RKV_HIP_CHECK(hipEventRecord(c->ev_start, s));
      RKV_HIP_CHECK(hipEventRecord(c->ev_stop, s));
    }
    rkv_launch_merge(v, qr, part, nch, chunk, c->cur_k, c->cur_v, multi ? q_pos : nullptr, nq, out, lse, s);
    return rkv_check_launch();
  }
  const int ns = rep / share;
  // reciprocals for the kernel's index arithmetic: ceil(2^32 / d) gives exact quotients n / d for n * d < 2^32
  auto recip = [](int d) { return d <= 1 ? 0u : (uint32_t)((((uint64_t)1 << 32) + d - 1) / d); };
  dim3 grid(8 * nch * ns, (v.B * v.NRG + 7) / 8, 1);        // see the kernel for the mapping
  if (c->ragged) {                                          // all sequences' chunks in one dimension
    int total = 0;
    for (int b = 0; b < v.B; ++b) total += (c->hlens[b] + MF_CH - 1) / MF_CH;
    grid = dim3(((total * split + 7) & ~7) * ns, v.NRG, 1);
  }
  if (grid.y > 65535) return RKV_EINVAL;
  if (c->decode_path == 3 && (multi || xb || v.hb || v.meta8 || share != 1)) return RKV_EINVAL;   // arithmetic-only measurement: plain variants
  // The measurement events, if set, are tied to the kernel's own dispatch (its begin and end time
  // stamps): events recorded as separate commands before and after it also count the gaps between
  // commands on the stream, some 4 us per launch.
  const bool timed = c->ev_start && c->ev_stop;
  if (row) {
    // a reorder over the whole row: the scores come from a kernel of their own, into a buffer behind
    // the partial results (rkv_decode_scratch_bytes reserves it); the events span both kernels
    if (c->decode_path == 3) return RKV_EINVAL;
    float* sc = (float*)((char*)part + rkv_partial_bytes(v.B, v.Hq, (int)v.Tpad));
    if (timed) RKV_HIP_CHECK(hipEventRecord(c->ev_start, s));
    const int rc = rkv_launch_scores_row(c, v, qr, sc, s);
    if (rc != RKV_OK) return rc;
    if (nch > 0)
      hipLaunchKernelGGL(pick_kernel(c, multi, share, false, MF_CH), grid, dim3(256), 0, s, v, (const float*)sc, part, nch,
                         multi ? q_pos : (const int*)nullptr, nq, ns, recip(ns), recip(v.NRG), RkvStepIn());
    if (timed) RKV_HIP_CHECK(hipEventRecord(c->ev_stop, s));
    rkv_launch_merge(v, qr, part, nch, MF_CH, c->cur_k, c->cur_v, multi ? q_pos : nullptr, nq, out, lse, s);
    return rkv_check_launch();
  }
  RkvStepIn in = step;
  in.qr = qr;
  if (nch > 0) {                                            // (an empty cache has only the current token)
    if (timed)
      hipExtLaunchKernelGGL(pick_kernel(c, multi, share, c->decode_path == 3, chunk, step.q != nullptr), grid, dim3(256), 0, s, c->ev_start, c->ev_stop, 0, v,
                            qt, part, nch, multi ? q_pos : nullptr, nq, ns, recip(ns), recip(v.NRG), in);
    else
      hipLaunchKernelGGL(pick_kernel(c, multi, share, c->decode_path == 3, chunk, step.q != nullptr), grid, dim3(256), 0, s, v, qt, part, nch,
                         multi ? q_pos : nullptr, nq, ns, recip(ns), recip(v.NRG), in);
  } else if (timed) {
    RKV_HIP_CHECK(hipEventRecord(c->ev_start, s));
    RKV_HIP_CHECK(hipEventRecord(c->ev_stop, s));
  }
  if (step.q) {
    const int rc = rkv_check_launch();
    if (rc != RKV_OK) return rc;
    *appended = true;
  }
  rkv_launch_merge(v, qr, part, nch, chunk, c->cur_k, c->cur_v, multi ? q_pos : nullptr, nq, out, lse, s);
  return rkv_check_launch();
}
