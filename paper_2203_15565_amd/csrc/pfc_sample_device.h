// What both selections of pfc_sample share on the device: the scores and sums over a workgroup.
#pragma once

#include "pfc_common.h"

namespace pfc {

struct PhiloxKey {
  uint32_t k0, k1;   // lo32(seed), hi32(seed)
  uint32_t c2, c3;   // lo32(step), hi32(step)
  uint32_t mask;     // ANDed onto every score
};

// To pinned host memory, for a host that waits for the stream before it reads.
__device__ __forceinline__ void store_to_host(uint32_t* p, uint32_t x) {
  __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

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

// Sum over the 64 lanes of a wavefront, to every lane: through the cross-lane modifiers of the vector
// ALU (as wave_sum), where a shuffle a step is a round trip to LDS.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_uadd(uint32_t v) {
  return v + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}
__device__ __forceinline__ uint32_t wave_usum(uint32_t v) {
  v = dpp_uadd<0xB1>(v);    // quad_perm [1,0,3,2]
  v = dpp_uadd<0x4E>(v);    // quad_perm [2,3,0,1]
  v = dpp_uadd<0x141>(v);   // row_half_mirror
  v = dpp_uadd<0x140>(v);   // row_mirror
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 0) + (uint32_t)__builtin_amdgcn_readlane((int)v, 16) +
         (uint32_t)__builtin_amdgcn_readlane((int)v, 32) + (uint32_t)__builtin_amdgcn_readlane((int)v, 48);
}
// Inclusive sums over the lanes.
__device__ __forceinline__ uint32_t wave_uscan(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, true);   // row_shr 1, 2, 4, 8
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, true);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, true);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, true);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);  // last lane of rows 0 and 2 to the next
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);  // lane 31 to rows 2 and 3
  return v;
}

// Sums of M values over the NT threads of a block, to every thread; sm: M * NT / 64 words, not in use
// again before the block has met once more.
template <int NT, int M>
__device__ __forceinline__ void block_sums(uint32_t (&v)[M], uint32_t* sm) {
#pragma unroll
  for (int m = 0; m < M; ++m) {
    v[m] = wave_usum(v[m]);
    if ((threadIdx.x & 63) == 0) sm[m * (NT / 64) + (threadIdx.x >> 6)] = v[m];
  }
  __syncthreads();
#pragma unroll
  for (int m = 0; m < M; ++m) {
    v[m] = 0;
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) v[m] += sm[m * (NT / 64) + i];
  }
}
// One value; sm may be used again at once.
template <int NT>
__device__ __forceinline__ uint32_t block_sum(uint32_t v, uint32_t* sm) {
  uint32_t one[1] = {v};
  block_sums<NT, 1>(one, sm);
  __syncthreads();
  return one[0];
}

// exclusive scan over the NT threads of a block; also returns the block total.  sm: NT / 64 words, not
// in use again before the block has met once more.
template <int NT>
__device__ __forceinline__ uint32_t block_excl_scan_once(uint32_t v, uint32_t* sm, uint32_t& total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint32_t inc = wave_uscan(v);
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
  return base + inc - v;
}
// sm may be used again at once.
template <int NT>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* sm, uint32_t& total) {
  const uint32_t r = block_excl_scan_once<NT>(v, sm, total);
  __syncthreads();
  return r;
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
  const uint32_t exc = block_excl_scan_once<NT>(mine, sm, total);   // a barrier behind the lines above
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

// Marks the classes of a workgroup's labels, PER of them to a thread, in pos_bits; first[c]: no label in
// front has marked class y[c], in this workgroup or another.  An LDS hash table of the bitmap's 64-bit
// words gathers their bits, then one atomic sets those of a word: with long-tailed labels a frequent
// class would bring thousands of atomics onto one word, with ids in the order of frequency a few lines
// of memory those of all frequent classes.  (Before, a loop over the distinct labels of a wavefront,
// one after the other: 2.5 us where all 64 differ.)  alone: no other workgroup marks.  pos_bits: 8-byte
// aligned, whole 64-bit words.
constexpr int kMarkSlots = 2048;   // at least twice the labels of a workgroup (512 or 1024; radix passes 256)
struct MarkLds {
  unsigned long long bits[kMarkSlots];
  int32_t key[kMarkSlots];         // word
};
template <int NT, int PER>
__device__ __forceinline__ void mark_labels(const int64_t (&y)[PER], const bool (&valid)[PER], bool (&first)[PER],
                                            MarkLds& lds, uint32_t* pos_bits, bool alone) {
  static_assert(kMarkSlots >= 2 * NT * PER && kMarkSlots % NT == 0, "room for every label");
  constexpr int OWN = kMarkSlots / NT;
  unsigned long long* words = reinterpret_cast<unsigned long long*>(pos_bits);
#pragma unroll
  for (int s = 0; s < OWN; ++s) {
    lds.key[s * NT + threadIdx.x] = -1;
    lds.bits[s * NT + threadIdx.x] = 0u;
  }
  __syncthreads();
  unsigned at[PER];
#pragma unroll
  for (int c = 0; c < PER; ++c) {
    first[c] = false;
    at[c] = 0u;
    if (!valid[c]) continue;
    const int32_t w = (int32_t)(y[c] >> 6);   // classes: below 2^31
    unsigned slot = ((unsigned)w * 2654435761u) >> 8;
    for (;;) {   // ends: there are more slots than labels
      slot %= kMarkSlots;
      const int32_t seen = atomicCAS(&lds.key[slot], -1, w);
      if (seen == -1 || seen == w) break;
      ++slot;
    }
    at[c] = slot;
    const unsigned long long bit = 1ull << (y[c] & 63);
    first[c] = !(atomicOr(&lds.bits[slot], bit) & bit);
  }
  __syncthreads();
  unsigned long long old[OWN];
#pragma unroll
  for (int s = 0; s < OWN; ++s) {
    const int32_t w = lds.key[s * NT + threadIdx.x];
    old[s] = 0u;
    if (w < 0) continue;
    const unsigned long long bits = lds.bits[s * NT + threadIdx.x];
    if (alone) words[w] = bits;
    else old[s] = atomicOr(&words[w], bits);
  }
  if (alone) return;
#pragma unroll
  for (int s = 0; s < OWN; ++s) lds.bits[s * NT + threadIdx.x] = old[s];
  __syncthreads();
#pragma unroll
  for (int c = 0; c < PER; ++c) first[c] = first[c] && !((lds.bits[at[c]] >> (y[c] & 63)) & 1u);
}

// The radix selection (pfc_sample_radix.hip).
int sample_radix(pfc_ctx* ctx, const int64_t* labels, int32_t B, uint32_t ceil_rN, int64_t cap,
                 const PhiloxKey& key, int32_t* idx_out, int32_t* yl_out);

}  // namespace pfc
