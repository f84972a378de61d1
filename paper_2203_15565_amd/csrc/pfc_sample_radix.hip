// The radix selection of pfc_sample: the general one, taken where the window of pfc_sample.hip is not
// the better way (window_select in pfc_sample_plan.h: large batches, masks that move the scores).
//
// The k - U negatives with the largest scores are found by a three-pass radix select (8 + 12 + 12
// bits), equal scores going to the smaller class id; an index-ordered compaction then writes S in
// ascending class id, and a binary search finds the labels in it.  Scores are recomputed wherever
// they are needed (about 60 integer operations per four classes).  Its six launches do the same work
// whatever the scores are; the batch costs them only its marking and its searches: 60 / 68 / 120 /
// 187 us with 16 / 32 / 131 / 262 thousand samples at N = 2,059,906, 107 us with few at 10 million.
#include "pfc_common.h"
#include "pfc_sample_device.h"

namespace pfc {

namespace {

constexpr int kThreads = 256;
constexpr int kItersPerBlock = kRadixClasses / (kThreads * 4);   // ordered passes

// Radix passes over the 32-bit score: bits [31:24], [23:12], [11:0].  The first pass sees every
// class, so it is kept narrow (256 bins: few global atomics per block); the later passes see
// only the classes inside the chosen bin, so their 4096-bin histograms are almost empty.
constexpr int kHistStride = 4096;
static_assert(kRadixHistWords == 3 * kHistStride, "histograms of the three passes");
template <int P> struct Pass;
template <> struct Pass<0> { static constexpr int kBins = 256, kShift = 24; };
template <> struct Pass<1> { static constexpr int kBins = 4096, kShift = 12; };
template <> struct Pass<2> { static constexpr int kBins = 4096, kShift = 0; };

// The batch classes are marked in the bitmap that the next window selection would use: it is clear
// before a call, and the label remap clears the words it knows to be set again, so that it stays the
// next one's.  Histograms and the count of positives are all zero between calls in the same way: the
// last reader of each piece clears it.  The batch classes are marked inside the launch of the first
// radix pass (see sample_hist_kernel), not by a launch of their own.
__device__ __forceinline__ uint32_t* batch_bits(const SampleScratch& sc) {
  return sc.st->next & 1u ? sc.pos_bits[1] : sc.pos_bits[0];
}

// The four "is positive" bits of classes 4q..4q+3 (bit e = class 4q+e).
__device__ __forceinline__ uint32_t pos_nibble(const uint32_t* __restrict__ pos_bits, uint32_t q) {
  return (pos_bits[q >> 3] >> ((q & 7u) * 4u)) & 0xFu;
}

// State of the select after pass P-1, found by every workgroup of the launch of pass P (or of the
// count launch, P = 3) from the histogram of pass P-1 and what workgroup 0 of the launch before left
// in `sel` -- the same integers everywhere, instead of a one-workgroup launch in between.
// Workgroup 0 records the new state for the next launch and clears what nobody reads any more (the
// histogram of pass P-2, the count of positives).
template <int P>
__device__ __forceinline__ void select_state(const SampleScratch& sc, uint32_t ceil_rN, uint32_t* sm,
                                             uint32_t& prefix, uint32_t& need, uint32_t& none) {
  static_assert(P >= 1 && P <= 3, "state after pass P-1");
  RadixState* sel = &sc.st->radix;
  uint32_t need_in, prefix_in;
  if constexpr (P == 1) {
    const uint32_t U = sel->U;
    const uint32_t k = U > ceil_rN ? U : ceil_rN;
    none = (k == U) ? 1u : 0u;
    need_in = k - U;
    prefix_in = 0u;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      if (sc.k_host) store_to_host(sc.k_host, k);
      sel->none = none;
    }
  } else {
    none = sel->none;
    need_in = sel->need[P - 2];
    prefix_in = sel->prefix[P - 2];
  }
  uint32_t bin = 0u;
  need = 0u;
  if (!none)
    find_bin<kThreads, Pass<P - 1>::kBins>(sc.hist + (P - 1) * kHistStride, need_in, sm, bin, need);
  prefix = prefix_in | (bin << Pass<P - 1>::kShift);
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) {
      sel->need[P - 1] = need;
      sel->prefix[P - 1] = prefix;
      if (P == 2) sel->U = 0u;
    }
    if constexpr (P >= 2) {
      constexpr int kOld = Pass<P - 2>::kBins;
      for (int b = threadIdx.x; b < kOld; b += kThreads) sc.hist[(P - 2) * kHistStride + b] = 0u;
    }
  }
}

// Radix pass P over the classes whose score agrees with the prefix found so far.
// Passes 1 and 2 skip the classes of the batch (their bits are complete by then).  Pass 0 runs in
// the same launch as the marking of the batch classes, so it cannot know them yet: it counts EVERY
// class, and the workgroups behind the first `hist_blocks` mark the labels -- the one thread that
// sets a class's bit first takes that class's score out of the merged histogram again and counts
// the class as a positive.  Integer atomics only, so the histogram after the launch is the same
// whatever the order.
template <int P>
__global__ __launch_bounds__(kThreads) void sample_hist_kernel(
    int64_t N, PhiloxKey key, SampleScratch sc, uint32_t ceil_rN, const int64_t* __restrict__ labels,
    int B, int hist_blocks, int32_t* __restrict__ err_flag) {
  constexpr int kBins = Pass<P>::kBins, kShift = Pass<P>::kShift;
  uint32_t* pos_bits = batch_bits(sc);
  if constexpr (P == 0) {
    if ((int)blockIdx.x >= hist_blocks) {   // marking part of the launch
      const int i = ((int)blockIdx.x - hist_blocks) * kThreads + threadIdx.x;
      const int64_t y = i < B ? labels[i] : 0;
      const bool valid = i < B && y >= 0 && y < N;
      if (i < B && !valid) atomicOr(err_flag, 1);
      __shared__ MarkLds marks;
      const int64_t ys[1] = {y};
      const bool valids[1] = {valid};
      bool first[1];
      mark_labels<kThreads, 1>(ys, valids, first, marks, pos_bits, false);
      if (first[0]) {   // first to mark class y
        uint32_t u[4];
        philox_block((uint32_t)(y >> 2), key, u);
        atomicSub(&sc.hist[u[y & 3] >> kShift], 1u);
      }
      const uint32_t nf = __popcll(__ballot(first[0]));
      if (nf && (threadIdx.x & 63) == 0) atomicAdd(&sc.st->radix.U, nf);
      return;
    }
  }
  __shared__ uint32_t lh[kBins], sm[kThreads / 64];
  for (int b = threadIdx.x; b < kBins; b += blockDim.x) lh[b] = 0u;
  uint32_t prefix = 0u, need = 0u, none = 0u;
  if constexpr (P > 0) select_state<P>(sc, ceil_rN, sm, prefix, need, none);
  __syncthreads();
  if (!(P > 0 && none)) {
    const uint32_t nq = (uint32_t)((N + 3) >> 2);
    const uint32_t stride = (uint32_t)hist_blocks * blockDim.x;
    for (uint32_t q = blockIdx.x * blockDim.x + threadIdx.x; q < nq; q += stride) {
      uint32_t u[4];
      philox_block(q, key, u);
      uint32_t pb = 0u;
      if constexpr (P > 0) pb = pos_nibble(pos_bits, q);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t j = (int64_t)q * 4 + e;
        if (j >= N || ((pb >> e) & 1u)) continue;
        if (P == 0) {
          atomicAdd(&lh[u[e] >> kShift], 1u);
        } else {
          // bits above this pass's field must equal the prefix
          constexpr int kAbove = kShift + 12;
          if ((u[e] >> kAbove) == (prefix >> kAbove))
            atomicAdd(&lh[(u[e] >> kShift) & (kBins - 1)], 1u);
        }
      }
    }
  }
  __syncthreads();
  for (int b = threadIdx.x; b < kBins; b += blockDim.x) {
    const uint32_t c = lh[b];
    if (c) atomicAdd(&sc.hist[P * kHistStride + b], c);
  }
}

// Selection predicate pieces for classes 4q..4q+3: bit e of `sure` = positive or score above the
// threshold; bit e of `eq` = non-positive and score equal to the threshold.
__device__ __forceinline__ void classify(uint32_t q, int64_t N, const PhiloxKey& key,
                                         const uint32_t* __restrict__ pos_bits, uint32_t T,
                                         uint32_t none, uint32_t& sure, uint32_t& eq) {
  sure = 0u;
  eq = 0u;
  const uint32_t nq = (uint32_t)((N + 3) >> 2);
  if (q >= nq) return;
  uint32_t u[4];
  philox_block(q, key, u);
  const uint32_t pb = pos_nibble(pos_bits, q);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int64_t j = (int64_t)q * 4 + e;
    if (j >= N) continue;
    if ((pb >> e) & 1u) {
      sure |= 1u << e;
    } else if (!none) {
      if (u[e] > T) sure |= 1u << e;
      else if (u[e] == T) eq |= 1u << e;
    }
  }
}

__global__ __launch_bounds__(kThreads) void sample_count_kernel(int64_t N, PhiloxKey key,
                                                                SampleScratch sc, uint32_t ceil_rN) {
  __shared__ uint32_t sm[kThreads / 64];
  const uint32_t* pos_bits = batch_bits(sc);
  uint32_t T, need, none;
  select_state<3>(sc, ceil_rN, sm, T, need, none);   // the full 32-bit threshold
  uint32_t nsure = 0, neq = 0;
#pragma unroll
  for (int it = 0; it < kItersPerBlock; ++it) {
    const uint32_t q = blockIdx.x * (kRadixClasses / 4) + it * kThreads + threadIdx.x;
    uint32_t sure, eq;
    classify(q, N, key, pos_bits, T, none, sure, eq);
    nsure += __popc(sure);
    neq += __popc(eq);
  }
  const uint32_t bs = block_sum<kThreads>(nsure, sm);
  const uint32_t be = block_sum<kThreads>(neq, sm);
  if (threadIdx.x == 0) {
    sc.radix_cnt[2 * blockIdx.x] = bs;
    sc.radix_cnt[2 * blockIdx.x + 1] = be;
  }
}

// Ordered write of S.  Every block first adds up the counts of the blocks in front of it: its
// output offset is their "sure" classes plus the equal-to-threshold ones they were allowed to
// keep -- the quota need[2] is used up in ascending class id, so that is min(quota, number of
// equal classes in front).  The last block also leaves the total.
__global__ __launch_bounds__(kThreads) void sample_compact_kernel(int64_t N, PhiloxKey key,
                                                                  SampleScratch sc, int64_t cap,
                                                                  int32_t* __restrict__ idx_out) {
  __shared__ uint32_t sm[kThreads / 64];
  RadixState* sel = &sc.st->radix;
  const uint32_t* pos_bits = batch_bits(sc);
  const uint32_t T = sel->prefix[2], none = sel->none;
  const uint32_t need_eq = none ? 0u : sel->need[2];
  if (blockIdx.x == 0)   // nobody reads the last pass's histogram any more
    for (int b = threadIdx.x; b < Pass<2>::kBins; b += kThreads) sc.hist[2 * kHistStride + b] = 0u;
  uint32_t front_sure = 0, front_eq = 0;
  for (uint32_t b = threadIdx.x; b < blockIdx.x; b += kThreads) {
    front_sure += sc.radix_cnt[2 * b];
    front_eq += sc.radix_cnt[2 * b + 1];
  }
  front_sure = block_sum<kThreads>(front_sure, sm);
  front_eq = block_sum<kThreads>(front_eq, sm);
  uint32_t out = front_sure + (front_eq < need_eq ? front_eq : need_eq);
  uint32_t eq_run = front_eq;
#pragma unroll
  for (int it = 0; it < kItersPerBlock; ++it) {
    const uint32_t q = blockIdx.x * (kRadixClasses / 4) + it * kThreads + threadIdx.x;
    uint32_t sure, eq;
    classify(q, N, key, pos_bits, T, none, sure, eq);
    uint32_t tot_e, tot_s;
    uint32_t eq_rank = eq_run + block_excl_scan<kThreads>(__popc(eq), sm, tot_e);
    // keep an equal-score class only while the quota lasts (ascending class id)
    uint32_t chosen = sure;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if ((eq >> e) & 1u) {
        if (eq_rank < need_eq) chosen |= 1u << e;
        ++eq_rank;
      }
    }
    uint32_t pos = out + block_excl_scan<kThreads>(__popc(chosen), sm, tot_s);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if ((chosen >> e) & 1u) {
        if ((int64_t)pos < cap) idx_out[pos] = (int32_t)(q * 4u + e);
        ++pos;
      }
    }
    eq_run += tot_e;
    out += tot_s;
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) sel->total = out;
}

// labels_local[i] = position of labels[i] in the ascending idx (binary search), -1 if absent.
__global__ __launch_bounds__(kThreads) void sample_remap_kernel(
    const int64_t* __restrict__ labels, int B, int64_t N, const int32_t* __restrict__ idx,
    SampleScratch sc, int64_t cap, int32_t* __restrict__ yl_out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= B) return;
  const int64_t y = labels[i];
  int64_t k = sc.st->radix.total;
  if (k > cap) k = cap;
  int32_t res = -1;
  if (y >= 0 && y < N) {
    int64_t lo = 0, hi = k;
    while (lo < hi) {
      const int64_t mid = (lo + hi) >> 1;
      if (idx[mid] < (int32_t)y) lo = mid + 1; else hi = mid;
    }
    if (lo < k && idx[lo] == (int32_t)y) res = (int32_t)lo;
  }
  yl_out[i] = res;
  // last user of the "is in the batch" bits: clear this label's word again
  if (y >= 0 && y < N) batch_bits(sc)[y >> 5] = 0u;
}

}  // namespace

int sample_radix(pfc_ctx* c, const int64_t* labels, int32_t B, uint32_t ceil_rN, int64_t cap,
                 const PhiloxKey& key, int32_t* idx_out, int32_t* yl_out) {
  const int64_t N = c->N;
  const SampleScratch& sc = c->samp;
  const unsigned nblk = (unsigned)((N + kRadixClasses - 1) / kRadixClasses);
  const int64_t nq = (N + 3) / 4;
  int hist_blocks = (int)((nq + kThreads * 4 - 1) / (kThreads * 4));
  if (hist_blocks > 512) hist_blocks = 512;
  const int mark_blocks = (B + kThreads - 1) / kThreads;
  PFC_LAUNCH(c, KID_SAMPLE_HIST0, sample_hist_kernel<0>, dim3(hist_blocks + mark_blocks),
             dim3(kThreads), 0, N, key, sc, ceil_rN, labels, B, hist_blocks, c->err_flag);
  PFC_LAUNCH(c, KID_SAMPLE_HIST1, sample_hist_kernel<1>, dim3(hist_blocks), dim3(kThreads), 0, N,
             key, sc, ceil_rN, labels, B, hist_blocks, c->err_flag);
  PFC_LAUNCH(c, KID_SAMPLE_HIST2, sample_hist_kernel<2>, dim3(hist_blocks), dim3(kThreads), 0, N,
             key, sc, ceil_rN, labels, B, hist_blocks, c->err_flag);
  PFC_LAUNCH(c, KID_SAMPLE_COUNT, sample_count_kernel, dim3(nblk), dim3(kThreads), 0, N, key, sc,
             ceil_rN);
  PFC_LAUNCH(c, KID_SAMPLE_COMPACT, sample_compact_kernel, dim3(nblk), dim3(kThreads), 0, N, key, sc,
             cap, idx_out);
  PFC_LAUNCH(c, KID_SAMPLE_REMAP, sample_remap_kernel, dim3(mark_blocks), dim3(kThreads), 0, labels,
             B, N, idx_out, sc, cap, yl_out);
  return PFC_OK;
}

}  // namespace pfc
