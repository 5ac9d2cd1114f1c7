// Attention-sink identification (Sec. 4.3): the tokens with the most massive activations in the
// output of the previous decoder block are the ones kept in fp16.  A token's score is its largest
// |activation|; the k highest scores win, ties go to the lower token index, indices are returned in
// ascending order.  fp16 maxima are exact, so the result equals the definition bit for bit.
#include "rkv_internal.h"
#include <type_traits>

// score[b][t] = max_c |x[b][t][c]|; one wave per token row, 16-byte loads, packed fp16 maxima
__global__ void __launch_bounds__(256) k_token_maxabs(const __half* __restrict__ x, int n_tok, int width, float* __restrict__ score) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int t = blockIdx.x * 4 + wave, b = blockIdx.y;
  if (t >= n_tok) return;
  const __half* row = x + ((size_t)b * n_tok + t) * width;
  typedef _Float16 h2 __attribute__((ext_vector_type(2)));
  h2 m = {(_Float16)0, (_Float16)0};
  const int n16 = width >> 3;                                  // 16-byte pieces (width is a multiple of 8)
#pragma unroll 4
  for (int i = lane; i < n16; i += 64) {
    const uint4 u = rkv_ld_stream(reinterpret_cast<const uint4*>(row) + i);
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) m = __builtin_elementwise_max(m, __builtin_bit_cast(h2, w[k] & 0x7fff7fffu));
  }
  float s = fmaxf((float)m[0], (float)m[1]);
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) s = fmaxf(s, __shfl_xor(s, o));
  if (lane == 0) score[(size_t)b * n_tok + t] = s;
}

// largest of the 64 lanes' values, in every lane: four steps inside each row of 16, then the four rows
__device__ __forceinline__ uint32_t wave_umax(uint32_t x) {
  auto step = [&](auto ctrl) {
    const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, decltype(ctrl)::value, 0xf, 0xf, true);
    x = o > x ? o : x;
  };
  step(std::integral_constant<int, 0xB1>());                   // quad_perm [1,0,3,2]
  step(std::integral_constant<int, 0x4E>());                   // quad_perm [2,3,0,1]
  step(std::integral_constant<int, 0x141>());                  // row_half_mirror
  step(std::integral_constant<int, 0x140>());                  // row_mirror
  const uint32_t r0 = __builtin_amdgcn_readlane(x, 0), r1 = __builtin_amdgcn_readlane(x, 16);
  const uint32_t r2 = __builtin_amdgcn_readlane(x, 32), r3 = __builtin_amdgcn_readlane(x, 48);
  const uint32_t a = r0 > r1 ? r0 : r1, c = r2 > r3 ? r2 : r3;
  return a > c ? a : c;
}

// k rounds of "largest remaining score, lowest index"; one workgroup per sequence.  Scores are >= 0, so
// their bit patterns order like the values; 1 + pattern (0: none left) and the complemented index are
// compared one after the other, each with a reduction on the vector pipe.
// What bounds this kernel is latency (a few KB of scores, k dependent rounds).  Every thread owns the
// tokens t = tid, tid + 1024, ..., holds the scores of the first TOPK_HELD of them in registers (8192 tokens in all;
// a longer prompt's further ones are read again from memory by the owner of a pick) and knows its best,
// so a round is one reduction over the workgroup and a new choice by one thread.  4 sequences of 4096 tokens, k = 4:
// 6.0 us, against 13.6 us with 256 threads that read all scores in every round.
#define TOPK_THREADS 1024
#define TOPK_HELD 8
__global__ void __launch_bounds__(TOPK_THREADS) k_topk_tokens(float* __restrict__ score, int n_tok, int k, int32_t* __restrict__ idx_out,
                                                              uint8_t* __restrict__ mask_out) {
  constexpr int NW = TOPK_THREADS / 64;
  __shared__ uint32_t s_hi[2][NW], s_lo[2][NW];
  __shared__ int s_pick[64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, b = blockIdx.x;
  float* sc = score + (size_t)b * n_tok;
  uint32_t held[TOPK_HELD];
#pragma unroll
  for (int i = 0; i < TOPK_HELD; ++i) {
    const int t = tid + i * TOPK_THREADS;
    held[i] = t < n_tok ? 1u + __float_as_uint(sc[t]) : 0u;
  }
  if (mask_out)
    for (int t = tid; t < n_tok; t += TOPK_THREADS) mask_out[(size_t)b * n_tok + t] = 0;
  uint32_t hi, lo;                                             // this thread's best: 1 + score bits, complemented index
  auto choose = [&]() {
    hi = 0;
    lo = 0;
#pragma unroll
    for (int i = 0; i < TOPK_HELD; ++i)
      if (held[i] > hi) {                                      // (ties: the earlier token stays)
        hi = held[i];
        lo = ~(uint32_t)(tid + i * TOPK_THREADS);
      }
    for (int t = tid + TOPK_HELD * TOPK_THREADS; t < n_tok; t += TOPK_THREADS) {
      const float s = sc[t];
      if (s >= 0.0f && 1u + __float_as_uint(s) > hi) {         // picked tokens are marked with -1
        hi = 1u + __float_as_uint(s);
        lo = ~(uint32_t)t;
      }
    }
  };
  choose();
  for (int round = 0; round < k; ++round) {
    const int buf = round & 1;                                 // (two sets of slots in turn: a wave already in the next round writes the other)
    {
      const uint32_t mh = wave_umax(hi), ml = wave_umax(hi == mh ? lo : 0u);
      if (lane == 0) {
        s_hi[buf][wave] = mh;
        s_lo[buf][wave] = ml;
      }
    }
    __syncthreads();
    const uint32_t wh = lane < NW ? s_hi[buf][lane] : 0u, wl = lane < NW ? s_lo[buf][lane] : 0u;
    const uint32_t mh = wave_umax(wh), ml = wave_umax(wh == mh ? wl : 0u);
    if (hi == mh && lo == ml) {                                // the token's owner (k <= n_tok, so one is left in every round)
      const int t = (int)~ml;
      s_pick[round] = t;
      if (mask_out) mask_out[(size_t)b * n_tok + t] = 1;       // (this thread cleared the byte above)
#pragma unroll
      for (int i = 0; i < TOPK_HELD; ++i)
        if (t == tid + i * TOPK_THREADS) held[i] = 0;
      if (t >= TOPK_HELD * TOPK_THREADS) sc[t] = -1.0f;
      choose();
    }
  }
  __syncthreads();
  if (tid < k) {                                               // ascending order: the place of a pick is how many are below it
    const int mine = s_pick[tid];
    int place = 0;
    for (int i = 0; i < k; ++i) place += s_pick[i] < mine;
    idx_out[(size_t)b * k + place] = mine;
  }
}

int rkv_launch_select_sinks(const __half* x, int batch, int n_tok, int width, int k, int32_t* idx_out, uint8_t* mask_out,
                            float* scratch, hipStream_t s) {
  hipLaunchKernelGGL(k_token_maxabs, dim3((n_tok + 3) / 4, batch), dim3(256), 0, s, x, n_tok, width, scratch);
  hipLaunchKernelGGL(k_topk_tokens, dim3(batch), dim3(TOPK_THREADS), 0, s, scratch, n_tok, k, idx_out, mask_out);
  return rkv_check_launch();
}

// ---------------------------------------------------------------------------------------------
// Offline folding of rotation and reorder into a projection (Sec. 4.2, Sec. 4.4): each row of the
// matrix is rotated group by group (butterflies in LDS, fp32) and gathered through the reorder
// indices.  One workgroup per row; cold path.
// ---------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_fold_rotation(const float* __restrict__ w, const int* __restrict__ perm, float* __restrict__ out,
                                                       int E, int n) {
  extern __shared__ float row[];
  const size_t base = (size_t)blockIdx.x * E;
  for (int c = threadIdx.x; c < E; c += 256) row[c] = w[base + c];
  __syncthreads();
  for (int h = 1; h < n; h <<= 1) {                 // Eq. 10 without the 1/sqrt(2) factors; h < n keeps a pair inside its group
    for (int i = threadIdx.x; i < E / 2; i += 256) {
      const int lo = ((i / h) * 2 * h) + (i % h), hi = lo + h;
      const float a = row[lo], b = row[hi];
      row[lo] = a + b;
      row[hi] = a - b;
    }
    __syncthreads();
  }
  const float rs = rsqrtf((float)n);
  for (int c = threadIdx.x; c < E; c += 256) out[base + c] = row[perm ? perm[c] : c] * rs;
}

int rkv_launch_fold_rotation(const rkv_config* cfg, const float* w, int rows, const int* perm, float* out, hipStream_t s) {
  const int E = cfg->n_kv_heads * RKV_D, n = cfg->rot_heads * RKV_D;
  const size_t lds = (size_t)E * 4;
  if (lds > 64 * 1024) return RKV_EINVAL;
  if (lds > 48 * 1024)
    RKV_HIP_CHECK(hipFuncSetAttribute((const void*)k_fold_rotation, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  hipLaunchKernelGGL(k_fold_rotation, dim3(rows), dim3(256), lds, s, w, perm, out, E, n);
  return rkv_check_launch();
}
