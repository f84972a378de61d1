// What both selections of pfc_sample share on the device: the scores and sums over a workgroup.
#pragma once

#include "pfc_common.h"

namespace pfc {

struct PhiloxKey {
  uint32_t k0, k1;   // lo32(seed), hi32(seed)
  uint32_t c2, c3;   // lo32(step), hi32(step)
  uint32_t mask;     // ANDed onto every score
};

// Scores of classes 4q .. 4q+3.
__device__ __forceinline__ void philox_block(uint32_t q, const PhiloxKey& key, uint32_t out[4]) {
  uint32_t c0 = q, c1 = 0u, c2 = key.c2, c3 = key.c3;   // class ids are < 2^31, so hi32(j/4) = 0
  uint32_t k0 = key.k0, k1 = key.k1;
#pragma unroll
  for (int round = 0; round < 10; ++round) {
    const uint32_t hi0 = __umulhi(0xD2511F53u, c0), lo0 = 0xD2511F53u * c0;
    const uint32_t hi1 = __umulhi(0xCD9E8D57u, c2), lo1 = 0xCD9E8D57u * c2;
    const uint32_t n0 = hi1 ^ c1 ^ k0;
    const uint32_t n2 = hi0 ^ c3 ^ k1;
    c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  out[0] = c0 & key.mask; out[1] = c1 & key.mask; out[2] = c2 & key.mask; out[3] = c3 & key.mask;
}

// Sum over the NT threads of a block, to every thread; sm: NT / 64 words.
template <int NT>
__device__ __forceinline__ uint32_t block_sum(uint32_t v, uint32_t* sm) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = v;
  __syncthreads();
  uint32_t r = 0;
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) r += sm[i];
  __syncthreads();
  return r;
}

// exclusive scan over the NT threads of a block; also returns the block total
template <int NT>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* sm, uint32_t& total) {
  uint32_t inc = v;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t n = __shfl_up(inc, o, 64);
    if (lane >= o) inc += n;
  }
  if (lane == 63) sm[w] = inc;
  __syncthreads();
  uint32_t base = 0;
  total = 0;
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) {
    const uint32_t x = sm[i];
    if (i < w) base += x;
    total += x;
  }
  __syncthreads();
  return base + inc - v;
}

// All NT threads: walk a histogram of NB bins from the largest bin downwards until `need`
// (>= 1) entries are covered.  Returns the bin that holds the last of them and how many are to be
// taken from inside it (bin 0 and 0 if the histogram holds fewer than `need`).
template <int NT, int NB>
__device__ __forceinline__ void find_bin(const uint32_t* hist, uint32_t need, uint32_t* sm,
                                         uint32_t& bin, uint32_t& need_inside) {
  __shared__ uint32_t s_bin, s_need;
  constexpr int kPer = NB / NT;
  const int t = threadIdx.x;
  uint32_t own[kPer], mine = 0, total;
#pragma unroll
  for (int e = 0; e < kPer; ++e) {   // thread t owns bins NB-1-t*kPer downwards
    own[e] = hist[NB - 1 - (t * kPer + e)];
    mine += own[e];
  }
  if (t == 0) {
    s_bin = 0u;
    s_need = 0u;
  }
  const uint32_t exc = block_excl_scan<NT>(mine, sm, total);
  if (exc < need && need <= exc + mine) {   // exactly one thread
    uint32_t cum = exc;
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      if (cum < need && need <= cum + own[e]) {
        s_bin = (uint32_t)(NB - 1 - (t * kPer + e));
        s_need = need - cum;
      }
      cum += own[e];
    }
  }
  __syncthreads();
  bin = s_bin;
  need_inside = s_need;
}

// One lane per distinct label of the wavefront: with long-tailed labels a frequent class would otherwise
// bring thousands of atomics onto one word.
__device__ __forceinline__ bool first_of_label(int64_t y, bool valid) {
  bool lead = false;
  unsigned long long todo = __ballot(valid);
  while (todo) {   // wave-uniform loop over the distinct labels
    const int src = __ffsll(todo) - 1;
    const int64_t y0 = __shfl(y, src, 64);
    lead = lead || (int)(threadIdx.x & 63) == src;
    todo &= ~__ballot(valid && y == y0);
  }
  return lead;
}

// The radix selection (pfc_sample_radix.hip); k is left in sc.st->k.
int sample_radix(pfc_ctx* ctx, const int64_t* labels, int32_t B, uint32_t ceil_rN, int64_t cap,
                 const PhiloxKey& key, int32_t* idx_out, int32_t* yl_out);

}  // namespace pfc
