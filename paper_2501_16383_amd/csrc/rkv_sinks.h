// Retention of the sink rows of an append (Sec. 4.3): keep the original fp16 rows of flagged tokens, first come first kept.
// One workgroup per sequence.  Latency bounds it: the flags of 4096 tokens are 4 KB and the rows kept a few tens of KB.
// Flags are read in coalesced passes (thread = token, all of a block's loads in flight together) and turned into wave
// ballots; the first wave places the flagged tokens with a prefix sum over the ballots of a block, and the rows are copied
// piece by piece over all retained rows at once, so that a copy is one round trip.  In a launch of its own (1024 threads)
// 4 sequences of 4096 tokens, 4 rows of 5120 channels each, take 9.9 us; the matrix-core append does it beside its own
// work, in workgroups of the same launch (256 threads).
#pragma once
#include "rkv_internal.h"

struct RkvSinkLds {
  unsigned long long ball[64];
  int tok[64];
  int n_new;
  float row[512];
};
// n_new: rows per sequence in k, vv and mask; sequence b uses the first n_b of them
template <int THREADS>
__device__ __forceinline__ void rkv_sinks_of(const RkvView& v, const __half* __restrict__ k, const __half* __restrict__ vv,
                                             const uint8_t* __restrict__ mask, int n_new, int n_b, int b, RkvSinkLds& lds) {
  constexpr int PASSES = 64 * 64 / THREADS;                 // passes of THREADS tokens per block: 64 ballots, one per lane of the first wave
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int cnt0 = v.sink_cnt[b];
  const int room = v.max_sinks - cnt0;
  const uint8_t* mb = mask + (size_t)b * n_new;
  int run = 0;                                              // flagged tokens of the blocks before this one
  for (int base = 0; base < n_b && run < room; base += 64 * 64) {
    uint8_t f[PASSES];
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
      const int t = base + p * THREADS + tid;
      f[p] = t < n_b ? mb[t] : (uint8_t)0;
    }
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
      const unsigned long long bal = __ballot(f[p] != 0);
      if (lane == 0) lds.ball[p * (THREADS / 64) + wave] = bal;
    }
    __syncthreads();
    if (wave == 0) {
      unsigned long long bal = lds.ball[lane];                // tokens base + 64 lane .. + 63
      int upto = __popcll(bal);
      const int own = upto;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int below = __shfl_up(upto, o);
        if (lane >= o) upto += below;
      }
      int slot = run + upto - own;
      while (bal && slot < room) {                          // (room <= 64: at most as many slots as lds.tok holds)
        lds.tok[slot++] = base + 64 * lane + (int)__ffsll((unsigned long long)bal) - 1;
        bal &= bal - 1;
      }
      if (lane == 63) lds.n_new = run + upto;
    }
    __syncthreads();
    run = lds.n_new;
  }
  const int nn = min(run, max(room, 0));
  // whole rows, 16 bytes per thread, all retained rows together and every load of a round issued before
  // its stores (rows are 256-byte multiples and 16-byte aligned: E is a multiple of 128 halves)
  {
    // (vector types and addresses that always exist: anything else puts the pieces in scratch memory)
    const rkv_u4v* k4 = reinterpret_cast<const rkv_u4v*>(k) + (size_t)b * n_new * (v.E / 8);
    const rkv_u4v* v4 = reinterpret_cast<const rkv_u4v*>(vv) + (size_t)b * n_new * (v.E / 8);
    rkv_u4v* dk4 = reinterpret_cast<rkv_u4v*>(v.sink_k) + ((size_t)b * v.max_sinks + cnt0) * (v.E / 8);
    rkv_u4v* dv4 = reinterpret_cast<rkv_u4v*>(v.sink_v) + ((size_t)b * v.max_sinks + cnt0) * (v.E / 8);
    const int n16 = v.E / 8, all = nn * n16;
    for (int e0 = 0; e0 < all; e0 += 4 * THREADS) {
      rkv_u4v a0, a1, a2, a3, c0, c1, c2, c3;
      auto get = [&](int u, rkv_u4v& x, rkv_u4v& y) __attribute__((always_inline)) {
        const int e = min(e0 + u * THREADS + tid, all - 1), i = e / n16;
        const size_t src = (size_t)lds.tok[i] * n16 + (e - i * n16);
        x = k4[src];
        y = v4[src];
      };
      auto put = [&](int u, const rkv_u4v& x, const rkv_u4v& y) __attribute__((always_inline)) {
        const int e = e0 + u * THREADS + tid;
        if (e < all) {
          if (!v.keys_rotated) dk4[e] = x;
          dv4[e] = y;
        }
      };
      get(0, a0, c0); get(1, a1, c1); get(2, a2, c2); get(3, a3, c3);
      put(0, a0, c0); put(1, a1, c1); put(2, a2, c2); put(3, a3, c3);
    }
  }
  if (tid < nn) v.sink_pos[b * v.max_sinks + cnt0 + tid] = rkv_len(v, b) + lds.tok[tid];
  if (tid == 0) v.sink_cnt[b] = cnt0 + nn;
  if (!v.keys_rotated) return;
  for (int i = 0; i < nn; ++i) {
    const size_t src = ((size_t)b * n_new + lds.tok[i]) * v.E, dst = ((size_t)b * v.max_sinks + cnt0 + i) * v.E;
    // the keys arrived rotated and reordered: undo the reorder, rotate again (H is its own
    // inverse), round to fp16 - group by group, butterflies in LDS (n <= 512 in this mode)
    for (int rg = 0; rg < v.NRG; ++rg) {
      const int gb = rg * v.n;
      for (int c = tid; c < v.n; c += THREADS) lds.row[c] = __half2float(k[src + v.pinv[gb + c]]);
      __syncthreads();
      for (int h = 1; h < v.n; h <<= 1) {
        for (int j = tid; j < v.n / 2; j += THREADS) {
          const int lo = ((j / h) * 2 * h) + (j % h), hi = lo + h;
          const float a = lds.row[lo], c2 = lds.row[hi];
          lds.row[lo] = a + c2;
          lds.row[hi] = a - c2;
        }
        __syncthreads();
      }
      const float rs = rsqrtf((float)v.n);
      for (int c = tid; c < v.n; c += THREADS) v.sink_k[dst + gb + c] = __float2half_rn(lds.row[c] * rs);
      __syncthreads();
    }
  }
}
