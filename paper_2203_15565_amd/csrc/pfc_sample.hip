// pfc_sample: the sampled class set S of one iteration (arXiv 2203.15565, Sec. 3.2 / Fig. 4:
// the classes present in the batch go in first, random negatives fill the buffer up to r*N).
//
// Integer work only.  Every class gets a 32-bit Philox4x32-10 score (Salmon et al., SC'11); the
// k - U negatives with the largest scores are taken, equal scores going to the smaller class id,
// and S is written in ascending class id.
//
// The scores are independent and uniform, so the score at which the selection ends is known
// beforehand up to a few standard deviations: the number of classes at or above a score is
// binomial.  The host hands the kernels a window of scores that holds it (about 6.5 standard
// deviations and the batch size wide, select_window), and two launches do the rest:
//
//   sample_scan   every score once: one bit per class that lies above the window, and a list of
//                 the classes inside it (a few thousand of millions); marks the batch classes
//   sample_write  every workgroup finds the exact end of the selection in the list, its own output
//                 offset from the counts of the workgroups in front, and writes its part of S and
//                 the positions of the labels that fall into it
//
// A window that misses (about once in 10^10 calls; or because a score mask has moved the scores) is
// seen by sample_write from the counts, and its workgroups then run a full radix select each for
// themselves: the same result, slowly.  Where the window is not the better way -- it is at least the
// batch wide, so with large batches -- or known to miss, the call takes the radix passes of
// pfc_sample_radix.hip instead (window_select in pfc_sample_plan.h).
//
// What bounds it: latency (a launch takes 2.8 us whatever it does; sample_write is a chain of one read
// of memory and nine meetings of a workgroup), for many classes the one Philox block per four of them
// (13 us of integer work at 10 million) and the list, which every workgroup of sample_write reads (33
// GB/s a compute unit).  Measured with rocprofv3, sum of the sampler's kernels, at N = 93,431 /
// 2,059,906 / 10,000,000: three radix passes, count, write and label remap, which recomputed the
// scores in five of six launches, 38 / 57 / 120 us; two launches 15 / 25 / 56; with the labels marked
// through a hash table, the list in parts and without dependent reads in sample_write 11.9 / 20 / 44.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <mutex>

#include "pfc_common.h"
#include "pfc_sample_device.h"
#include "pfc_sample_plan.h"

namespace pfc {

namespace {

constexpr int kThreads = 256;
constexpr int kWriteThreads = 512;   // of sample_write
constexpr int kWriteLabels = 2;      // labels of a thread of sample_write that it requests first

// The window: scores lo .. lo + width (both inside).  Scores above it are taken, below it not.
struct Window {
  uint32_t lo, width;
  int shift;        // bin of a score inside: (score - lo) >> shift, below kWindowBins
  __device__ __forceinline__ bool inside(uint32_t u) const { return u - lo <= width; }
  __device__ __forceinline__ bool above(uint32_t u) const { return u > lo + width; }
};

// Ascending order of keys = order of preference: larger score first, then smaller class id.
__device__ __forceinline__ uint64_t select_key(uint32_t score, uint32_t id) {
  return ((uint64_t)(~score) << 32) | id;
}

// Everything that carries counts or marks of one call exists twice (SampleState::hdr, pos_bits,
// blk_pos, pos_list).  A call works on one set and, in its second launch, clears what the call
// before left in the other, so no call starts with a clearing pass; which set is next is kept on
// the device, so that a captured and replayed call alternates as well.

// ---------------------------------------------------------------------------------------------
// sample_scan.  The classes [b << cls_log2, (b + 1) << cls_log2) of workgroup b < nblk of sample_write
// are scored by 1 << scan_split workgroups; the workgroups behind those mark the batch classes in the same launch: the one thread that sets a
// class's bit first counts the class, as one that the bits of the first part hold already or not,
// and lists its key if its score lies in the window (the first part lists it too, not knowing the
// batch).  Integer atomics only: the counts do not depend on the order, and the lists are read as
// sets.
// The counts of the workgroups' classes are added up in LDS first: with ids in the order of the classes'
// frequency one range of them owns thousands of the batch's classes, whose atomics on its one count queue
// up (2,059,906 classes without negatives, labels dense in the low ids: 16,384 samples 52 -> 39 us,
// 65,536 114 -> 78; spread evenly 38 -> 36 and 75 -> 66).  Likewise the counts of the whole batch, which a
// marking workgroup that is alone just writes.  This launch, us, a loop over the distinct labels of
// every wavefront and one count of the list -> now: 128 labels, 10,000 classes 8.0 -> 4.5; 512, 93,431
// 7.0 -> 4.7; 1024, 2,059,906 11.5 -> 7.1.
// ---------------------------------------------------------------------------------------------
// LABELS: of a thread of the marking part.
template <int LABELS>
__global__ __launch_bounds__(kThreads) void sample_scan_kernel(
    int64_t N, PhiloxKey key, Window win, SampleScratch sc, int cls_log2, int nblk, int scan_split,
    uint32_t part_mask, const int64_t* __restrict__ labels, int B, int32_t* __restrict__ err_flag) {
  const uint32_t par = sc.st->next & 1u;
  SampleHdr* hdr = &sc.st->hdr[par];
  const int lane = threadIdx.x & 63;
  __shared__ union ScanLds {
    uint64_t list[kLocalList];
    struct {
      uint32_t pos[kMaxBlocks];
      MarkLds marks;
      uint64_t list[kThreads * LABELS];
      uint32_t n[3];   // entries of list; batch classes; of these, above the window
    } mark;
  } lds;
  __shared__ uint32_t s_n, s_base, sm[4];
  const int nscan = nblk << scan_split;
  if ((int)blockIdx.x >= nscan) {   // marking part of the launch
    auto& m = lds.mark;
    const bool alone = B <= kThreads * LABELS, gather = nblk <= kMaxBlocks;
    int64_t y[LABELS];
    bool valid[LABELS], lead[LABELS];
    const int i0 = ((int)blockIdx.x - nscan) * kThreads * LABELS + threadIdx.x;
#pragma unroll
    for (int c = 0; c < LABELS; ++c) y[c] = i0 + c * kThreads < B ? labels[i0 + c * kThreads] : 0;
    if (gather)
      for (int b = threadIdx.x; b < nblk; b += kThreads) m.pos[b] = 0u;
    if (threadIdx.x < 3) m.n[threadIdx.x] = 0u;
#pragma unroll
    for (int c = 0; c < LABELS; ++c) {
      valid[c] = i0 + c * kThreads < B && y[c] >= 0 && y[c] < N;
      if (i0 + c * kThreads < B && !valid[c]) atomicOr(err_flag, 1);
    }
    mark_labels<kThreads, LABELS>(y, valid, lead, m.marks, sc.pos_bits[par], alone);
    uint32_t na = 0, nf = 0;
#pragma unroll
    for (int c = 0; c < LABELS; ++c) {
      if (!lead[c]) continue;   // first to mark class y
      uint32_t u[4];
      philox_block((uint32_t)(y[c] >> 2), key, u);
      const uint32_t uy = u[y[c] & 3];
      const bool above = win.above(uy);
      ++nf;
      na += above;
      atomicAdd(gather ? &m.pos[y[c] >> cls_log2] : &sc.blk_pos[par][y[c] >> cls_log2], above ? 0x10000u : 1u);
      if (win.inside(uy)) m.list[atomicAdd(&m.n[0], 1u)] = select_key(uy, (uint32_t)y[c]);
    }
    nf = wave_usum(nf);
    na = wave_usum(na);
    if (lane == 0) {
      if (nf) atomicAdd(&m.n[1], nf);
      if (na) atomicAdd(&m.n[2], na);
    }
    __syncthreads();
    const uint32_t n = m.n[0];
    if (threadIdx.x == 0) {
      if (alone) {
        hdr->U = m.n[1];
        hdr->pos_above = m.n[2];
        hdr->npos = n;
        s_base = 0u;
      } else {
        s_base = n ? atomicAdd(&hdr->npos, n) : 0u;
        if (m.n[1]) atomicAdd(&hdr->U, m.n[1]);
        if (m.n[2]) atomicAdd(&hdr->pos_above, m.n[2]);
      }
    }
    if (gather) {
      for (int b = threadIdx.x; b < nblk; b += kThreads) {
        if (alone) sc.blk_pos[par][b] = m.pos[b];
        else if (m.pos[b]) atomicAdd(&sc.blk_pos[par][b], m.pos[b]);
      }
    }
    __syncthreads();
    for (uint32_t e = threadIdx.x; e < n; e += kThreads)
      if (s_base + e < sc.pos_cap) sc.pos_list[par][s_base + e] = m.list[e];
    return;
  }
  uint64_t* s_list = lds.list;
  if (threadIdx.x == 0) s_n = 0u;
  __syncthreads();
  const uint32_t nq = (uint32_t)((N + 3) >> 2);
  const uint32_t q0 = blockIdx.x << (cls_log2 - scan_split - 2);
  const int iters = 1 << (cls_log2 - scan_split - 10);
  uint32_t cnt = 0;
  for (int it = 0; it < iters; ++it) {
    const uint32_t q = q0 + it * kThreads + threadIdx.x;
    uint32_t nib = 0u;
    if (q < nq) {
      uint32_t u[4];
      philox_block(q, key, u);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t j = q * 4u + e;
        if ((int64_t)j >= N) continue;
        if (win.above(u[e])) nib |= 1u << e;
        if (win.inside(u[e])) {
          const uint32_t p = atomicAdd(&s_n, 1u);
          if (p < (uint32_t)kLocalList) s_list[p] = select_key(u[e], j);
        }
      }
    }
    cnt += __popc(nib);
    // eight neighbouring lanes hold one word of bits: combine them through the vector ALU
    uint32_t v = nib << ((lane & 7) * 4);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, true);    // lane ^ 1
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xf, 0xf, true);    // lane ^ 2
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xf, 0xf, true);   // 7 - lane
    if ((lane & 7) == 0 && q < nq) sc.above_bits[q >> 3] = v;
  }
  const uint32_t total = block_sum<kThreads>(cnt, sm);   // also a barrier behind the list
  const uint32_t n = s_n;
  if (threadIdx.x == 0) {
    sc.above_cnt[blockIdx.x] = total;
    if (n) s_base = atomicAdd(&hdr->listed[blockIdx.x & part_mask][0], n);
    if (n > (uint32_t)kLocalList) atomicOr(&hdr->overflow, 1u);
    if (blockIdx.x == 0) {
      sc.st->cur = par;
      hdr->nblk = (uint32_t)nblk;
      hdr->nwords = (uint32_t)((N + 31) >> 5);
    }
  }
  if (n == 0) return;
  __syncthreads();
  const uint32_t base = s_base, part_cap = sc.list_cap / (part_mask + 1);
  uint64_t* list = sc.list + (blockIdx.x & part_mask) * part_cap;
  for (uint32_t e = threadIdx.x; e < n && e < (uint32_t)kLocalList; e += kThreads)
    if (base + e < part_cap) list[base + e] = s_list[e];
}

// ---------------------------------------------------------------------------------------------
// sample_write.
// ---------------------------------------------------------------------------------------------
// Its time, us, with two reads that waited for others (bits of the batch classes of the end bin,
// labels) and 16 meetings of the workgroup -> now: 10,000 classes, 128 labels 7.4 -> 6.4; 93,431, 512
// 8.4 -> 7.1; 2,059,906, 1024 13.4 -> 12.6; 10,000,000, 2048 (half the workgroups) 36 -> 25.
struct WriteShared {
  uint32_t sm[kWriteThreads / 64];          // sums and scans in turn
  uint32_t sm2[3 * kWriteThreads / 64];
  uint32_t hist[4096];                      // window bins, or radix bins of the slow select
  uint32_t word[1 << (kMaxClsLog2 - 5)];    // chosen classes of this workgroup
  uint32_t pre[1 << (kMaxClsLog2 - 5)];     // chosen classes in front of each word
  uint64_t bin_list[kBinList];              // keys in the bin in which the selection ends,
  uint64_t bin_pos[kBinList];               // those of batch classes once more
  uint32_t bin_n, bin_npos;
  uint64_t key_end;
};

// The window missed: a radix select over all scores (bits 31..24, 23..12, 11..0), run by every
// workgroup for itself.  Leaves this workgroup's chosen classes in s.word and returns how many
// chosen classes lie in front.
__device__ __forceinline__ uint32_t slow_select(int64_t N, const PhiloxKey& key,
                                             const uint32_t* pos_bits, uint32_t need, int cls_log2,
                                             WriteShared& s) {
  const uint32_t nq = (uint32_t)((N + 3) >> 2);
  const uint32_t q0 = blockIdx.x << (cls_log2 - 2), q1 = q0 + (1u << (cls_log2 - 2));
  uint32_t prefix = 0u;
#pragma unroll 1
  for (int pass = 0; pass < 3; ++pass) {
    const int sh = pass == 0 ? 24 : pass == 1 ? 12 : 0;
    const int above = pass == 0 ? 32 : sh + 12;   // bits that are fixed already start here
    for (int b = threadIdx.x; b < 4096; b += kWriteThreads) s.hist[b] = 0u;
    __syncthreads();
#pragma unroll 1
    for (uint32_t q = threadIdx.x; q < nq; q += kWriteThreads) {
      uint32_t u[4];
      philox_block(q, key, u);
      const uint32_t pb = pos_bits[q >> 3] >> ((q & 7u) * 4u);
      for (int e = 0; e < 4; ++e) {
        if ((int64_t)q * 4 + e >= N || ((pb >> e) & 1u)) continue;
        if (above < 32 && (u[e] >> above) != (prefix >> above)) continue;
        atomicAdd(&s.hist[(u[e] >> sh) & 0xFFFu], 1u);
      }
    }
    __syncthreads();
    uint32_t bin, inside;
    find_bin<kWriteThreads, 4096>(s.hist, need, s.sm, bin, inside);
    prefix |= bin << sh;
    need = inside;
    __syncthreads();
  }
  // scores above `prefix` are taken, and the first `need` classes (ascending id) that equal it
  uint32_t sure = 0, eq = 0;
#pragma unroll 1
  for (uint32_t q = threadIdx.x; q < nq && q < q0; q += kWriteThreads) {
    uint32_t u[4];
    philox_block(q, key, u);
    const uint32_t pb = pos_bits[q >> 3] >> ((q & 7u) * 4u);
    for (int e = 0; e < 4; ++e) {
      if ((pb >> e) & 1u) ++sure;
      else if (u[e] > prefix) ++sure;
      else if (u[e] == prefix) ++eq;
    }
  }
  sure = block_sum<kWriteThreads>(sure, s.sm);
  eq = block_sum<kWriteThreads>(eq, s.sm);
  const uint32_t front = sure + (eq < need ? eq : need);
  for (uint32_t w = threadIdx.x; w < (1u << (cls_log2 - 5)); w += kWriteThreads) s.word[w] = 0u;
  __syncthreads();
  uint32_t eq_run = eq;
#pragma unroll 1
  for (uint32_t qb = q0; qb < q1; qb += kWriteThreads) {
    const uint32_t q = qb + threadIdx.x;
    uint32_t chosen = 0u, same = 0u, tot;
    if (q < nq && q < q1) {
      uint32_t u[4];
      philox_block(q, key, u);
      const uint32_t pb = pos_bits[q >> 3] >> ((q & 7u) * 4u);
      for (int e = 0; e < 4; ++e) {
        if ((int64_t)q * 4 + e >= N) continue;
        if (((pb >> e) & 1u) || u[e] > prefix) chosen |= 1u << e;
        else if (u[e] == prefix) same |= 1u << e;
      }
    }
    uint32_t rank = eq_run + block_excl_scan<kWriteThreads>(__popc(same), s.sm, tot);
    for (int e = 0; e < 4; ++e) {
      if (!((same >> e) & 1u)) continue;
      if (rank < need) chosen |= 1u << e;
      ++rank;
    }
    eq_run += tot;
    if (chosen) atomicOr(&s.word[(q - q0) >> 3], chosen << ((q & 7u) * 4u));
  }
  __syncthreads();
  return front;
}

// NE: list entries that every thread keeps in registers over the three looks at the list.  The host
// picks it so that the usual list fits (few registers where the list is short); the rest of a
// longer one is read again each time.  512 threads: with 1024 the 64 registers of two resident
// workgroups spill (2 million classes: 38 us instead of 13).
template <int NE>
__global__ __launch_bounds__(kWriteThreads, 4) void sample_write_kernel(
    int64_t N, PhiloxKey key, Window win, SampleScratch sc, int cls_log2, int nblk, int scan_split,
    uint32_t part_mask, uint32_t keep, uint32_t ceil_rN, const int64_t* __restrict__ labels, int B, int64_t cap,
    int32_t* __restrict__ idx_out, int32_t* __restrict__ yl_out) {
  constexpr int NT = kWriteThreads;
  __shared__ WriteShared s;
  const int t = threadIdx.x;
  const uint32_t me = blockIdx.x;
  const uint32_t word0 = me << (cls_log2 - 5), nwords = (uint32_t)((N + 31) >> 5);
  const int own_words = 1 << (cls_log2 - 5);

  // Everything that is certain to be needed is requested before anything is waited for, from both
  // sets where the set at hand decides (it is one load away itself), the list up to its usual
  // length whatever it holds.
  uint64_t x[NE];
  // this thread's part of the list, and its place among the threads that share the part
  const uint32_t part_threads = NT / (part_mask + 1), part_cap = sc.list_cap / (part_mask + 1);
  const uint32_t part = t / part_threads, part_t = t % part_threads;
  const uint64_t* list = sc.list + part * part_cap;
  const uint32_t kept = keep * part_threads;   // entries of the part that are requested now (keep <= NE)
#pragma unroll
  for (int c = 0; c < NE; ++c) {
    const uint32_t e = c * part_threads + part_t;
    x[c] = e < kept ? list[e] : 0ull;
  }
  const uint64_t first_pos0 = (uint32_t)t < sc.pos_cap ? sc.pos_list[0][t] : 0ull,
                 first_pos1 = (uint32_t)t < sc.pos_cap ? sc.pos_list[1][t] : 0ull;
  int64_t ys[kWriteLabels];
#pragma unroll
  for (int c = 0; c < kWriteLabels; ++c) ys[c] = c * NT + t < B ? labels[c * NT + t] : -1;
  const uint32_t above0 = (uint32_t)t < (uint32_t)nblk << scan_split ? sc.above_cnt[t] : 0u;
  const uint32_t blk0 = t < nblk ? sc.blk_pos[0][t] : 0u, blk1 = t < nblk ? sc.blk_pos[1][t] : 0u;
  const uint32_t par = sc.st->cur & 1u;
  const SampleHdr *hp0 = &sc.st->hdr[0], *hp1 = &sc.st->hdr[1];
  auto pick = [&](uint32_t SampleHdr::*f) {
    const uint32_t a = hp0->*f, b = hp1->*f;
    return par ? b : a;
  };
  const uint32_t U = pick(&SampleHdr::U), pos_above = pick(&SampleHdr::pos_above),
                 npos = pick(&SampleHdr::npos), overflow = pick(&SampleHdr::overflow);
  uint32_t n = 0, part_n = 0, most = 0;   // entries of the list, of this thread's part, of the longest part
#pragma unroll
  for (int p = 0; p < kListParts; ++p) {
    const uint32_t a = hp0->listed[p][0], b = hp1->listed[p][0], m = par ? b : a;
    n += m;
    most = m > most ? m : most;
    part_n = (uint32_t)p == part ? m : part_n;
  }
  const uint32_t old_words = par ? hp0->nwords : hp1->nwords,
                 old_blk = par ? hp0->nblk : hp1->nblk;
  // counts: of every workgroup (does the window hold the end of the selection?) and of those in
  // front (where does this one's output start?)
  const uint32_t nscan = (uint32_t)nblk << scan_split;
  uint32_t tot_above = 0, front = 0, front_pos = 0;
  auto add_above = [&](uint32_t b, uint32_t a) {
    tot_above += a;
    if ((b >> scan_split) < me) front += a;
  };
  auto add_pos = [&](uint32_t b, uint32_t p0, uint32_t p1) {
    const uint32_t p = par ? p1 : p0;
    if (b < me) {
      front += p & 0xFFFFu;
      front_pos += (p & 0xFFFFu) + (p >> 16);
    }
  };
  add_above(t, above0);
  add_pos(t, blk0, blk1);
  for (uint32_t b = NT + t; b < nscan; b += NT) add_above(b, sc.above_cnt[b]);
  for (uint32_t b = NT + t; b < (uint32_t)nblk; b += NT) add_pos(b, sc.blk_pos[0][b], sc.blk_pos[1][b]);
  const uint32_t k = U > ceil_rN ? U : ceil_rN;
  const uint32_t R = k - U;   // negatives to take
  const uint32_t* pos_bits = par ? sc.pos_bits[1] : sc.pos_bits[0];
  for (int b = t; b < kWindowBins; b += NT) s.hist[b] = 0u;
  for (int w = t; w < own_words; w += NT) {
    uint32_t v = 0u;
    if (word0 + w < nwords) {
      // (not waiting for R, which is two loads away)
      const uint32_t p0 = sc.pos_bits[0][word0 + w], p1 = sc.pos_bits[1][word0 + w], a = sc.above_bits[word0 + w];
      v = (par ? p1 : p0) | (R ? a : 0u);
    }
    s.word[w] = v;
  }
  if (t == 0) {
    s.bin_n = s.bin_npos = 0u;
    s.key_end = 0ull;
  }
  uint32_t sums[2] = {tot_above, R ? front : front_pos};
  block_sums<NT, 2>(sums, s.sm2);
  tot_above = sums[0];
  uint32_t out = sums[1];
  if (R != 0) {
    const uint32_t neg_above = tot_above - pos_above;
    const uint32_t need = R - neg_above;
    bool ok = overflow == 0u && npos <= sc.pos_cap && most <= part_cap && neg_above <= R &&
              R <= neg_above + (n - npos);
    auto each = [&](auto fn) {   // fn(key) for every entry of the list
#pragma unroll
      for (int c = 0; c < NE; ++c)
        if (c * part_threads + part_t < (part_n < kept ? part_n : kept)) fn(x[c]);
      for (uint32_t e = kept + part_t; e < part_n; e += part_threads) fn(list[e]);
    };
    auto bin_of = [&](uint64_t y) { return (~(uint32_t)(y >> 32) - win.lo) >> win.shift; };
    const uint64_t* pl = par ? sc.pos_list[1] : sc.pos_list[0];
    const uint64_t first_pos = par ? first_pos1 : first_pos0;
    auto each_pos = [&](auto fn) {   // likewise of the list of the batch classes
      if ((uint32_t)t < npos) fn(first_pos);
      for (uint32_t e = NT + t; e < npos; e += NT) fn(pl[e]);
    };
    if (ok && need) {
      // negatives of the window by bin (the list holds batch classes too: taken out again)
      each([&](uint64_t y) { atomicAdd(&s.hist[bin_of(y)], 1u); });
      each_pos([&](uint64_t y) { atomicSub(&s.hist[bin_of(y)], 1u); });
      __syncthreads();
      uint32_t bin, inside;
      find_bin<NT, kWindowBins>(s.hist, need, s.sm, bin, inside);
      auto to = [&](uint64_t* list, uint32_t* n, uint64_t y) {
        if (bin_of(y) != bin) return;
        const uint32_t p = atomicAdd(n, 1u);
        if (p < (uint32_t)kBinList) list[p] = y;
      };
      each([&](uint64_t y) { to(s.bin_list, &s.bin_n, y); });
      each_pos([&](uint64_t y) { to(s.bin_pos, &s.bin_npos, y); });
      __syncthreads();
      const uint32_t nb = s.bin_n, np = s.bin_npos;   // np <= nb
      ok = nb <= (uint32_t)kBinList;
      if (ok && (uint32_t)t < nb) {
        const uint64_t mine = s.bin_list[t];
        uint32_t rank = 0;   // negatives in front
        bool negative = true;
        for (uint32_t e = 0; e < nb; ++e) rank += s.bin_list[e] < mine ? 1u : 0u;
        for (uint32_t e = 0; e < np; ++e) {
          const uint64_t p = s.bin_pos[e];
          rank -= p < mine ? 1u : 0u;
          negative = negative && p != mine;
        }
        if (negative && rank == inside - 1u) s.key_end = mine + 1ull;   // keys below this are taken
      }
      __syncthreads();
    }
    if (ok) {
      if (need) {
        const uint64_t end = s.key_end;
        uint32_t c[1] = {0};
        each([&](uint64_t y) {
          if (y >= end) return;
          const uint32_t j = (uint32_t)y, b = j >> cls_log2;
          if (b < me) ++c[0];
          else if (b == me) atomicOr(&s.word[(j >> 5) - word0], 1u << (j & 31u));
        });
        // a batch class in the window was counted as one already
        each_pos([&](uint64_t y) {
          if (y < end && ((uint32_t)y >> cls_log2) < me) --c[0];
        });
        block_sums<NT, 1>(c, s.sm2);
        out += c[0];
      }
    } else {
      __syncthreads();
      out = slow_select(N, key, pos_bits, R, cls_log2, s);
      __syncthreads();
    }
  }

  // number of chosen classes in front of every word, then the ids, four classes per thread
  const uint32_t out0 = out;
  uint32_t run = 0;
  for (int w0 = 0; w0 < own_words; w0 += NT) {
    const int w = w0 + t;
    uint32_t tot;
    const uint32_t p =
        run + block_excl_scan<NT>(w < own_words ? __popc(s.word[w]) : 0u, s.sm, tot);
    if (w < own_words) s.pre[w] = p;
    run += tot;
  }
  __syncthreads();
  for (int b = t; b < own_words * 8; b += NT) {
    const uint32_t word = s.word[b >> 3], sh = (b & 7) * 4, c4 = (word >> sh) & 0xFu;
    uint32_t pos = out0 + s.pre[b >> 3] + __popc(word & ((1u << sh) - 1u));
    const uint32_t id0 = (me << cls_log2) + (uint32_t)b * 4u;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if ((c4 >> e) & 1u) {
        if ((int64_t)pos < cap) idx_out[pos] = (int32_t)(id0 + e);
        ++pos;
      }
    }
  }
  // positions of the labels that lie here (-1 for a bad label)
  auto place = [&](int i, int64_t y) {
    if (y < 0 || y >= N) {
      if (me == 0) yl_out[i] = -1;
    } else if ((uint32_t)(y >> cls_log2) == me) {
      const uint32_t w = (uint32_t)(y >> 5) - word0;
      const uint32_t pos = out0 + s.pre[w] + __popc(s.word[w] & ((1u << (y & 31)) - 1u));
      yl_out[i] = (int64_t)pos < cap ? (int32_t)pos : -1;
    }
  };
#pragma unroll
  for (int c = 0; c < kWriteLabels; ++c)
    if (c * NT + t < B) place(c * NT + t, ys[c]);
  for (int i0 = kWriteLabels * NT + t; i0 < B; i0 += 4 * NT) {   // four loads in flight
    int64_t more[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) more[c] = i0 + c * NT < B ? labels[i0 + c * NT] : 0;
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (i0 + c * NT < B) place(i0 + c * NT, more[c]);
  }
  // clear the other set for the next call (this launch uses none of it but the two sizes, and
  // those stay)
  uint32_t* old_bits = par ? sc.pos_bits[0] : sc.pos_bits[1];
  uint32_t* old_pos = par ? sc.blk_pos[0] : sc.blk_pos[1];
  for (uint32_t w = me * NT + t; w < old_words; w += (uint32_t)nblk * NT)
    old_bits[w] = 0u;
  for (uint32_t b = me * NT + t; b < old_blk; b += (uint32_t)nblk * NT)
    old_pos[b] = 0u;
  if (me == 0 && t < kListParts) (par ? sc.st->hdr[0] : sc.st->hdr[1]).listed[t][0] = 0u;
  if (me == 0 && t == 0) {
    SampleHdr* old = par ? &sc.st->hdr[0] : &sc.st->hdr[1];
    old->U = 0u;
    old->pos_above = 0u;
    old->npos = 0u;
    old->overflow = 0u;
    if (sc.k_host) store_to_host(sc.k_host, k);
    sc.st->next = par ^ 1u;
  }
}

}  // namespace

size_t sample_layout(int64_t N, int64_t B, char* base, SampleScratch* out) {
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char* p = base + off;
    off += (bytes + 255) / 256 * 256;
    return p;
  };
  const size_t words = (size_t)(N + 31) / 32;
  const size_t blk = (size_t)sample_count_cap(N);
  const size_t list = (size_t)window_list_cap(N, B), pos = (size_t)window_pos_cap(B);
  out->st = (SampleState*)take(sizeof(SampleState));
  for (int i = 0; i < 2; ++i) {
    out->pos_bits[i] = (uint32_t*)take(words * 4);
    out->blk_pos[i] = (uint32_t*)take(blk * 4);
    out->pos_list[i] = (uint64_t*)take(pos * 8);
  }
  out->above_bits = (uint32_t*)take(words * 4);
  out->above_cnt = (uint32_t*)take(blk * 4);
  out->list = (uint64_t*)take(list * 8);
  out->list_cap = (uint32_t)list;
  out->pos_cap = (uint32_t)pos;
  out->hist = (uint32_t*)take(kRadixHistWords * 4);
  out->radix_cnt = (uint32_t*)take((size_t)((N + kRadixClasses - 1) / kRadixClasses) * 8);
  return off;
}

int sample_impl(pfc_ctx* c, const int64_t* labels, int32_t B, double r, uint64_t seed,
                uint64_t step, uint32_t score_mask, int32_t* idx_out, int32_t* yl_out,
                int64_t* k_out) {
  const int64_t N = c->N;
  int64_t crn = (int64_t)ceil(r * (double)N);
  if (crn > N) crn = N;
  if (crn < 1) crn = 1;
  const int64_t cap = pfc_num_sampled(N, B, r);
  PhiloxKey key;
  key.k0 = (uint32_t)(seed & 0xFFFFFFFFu);
  key.k1 = (uint32_t)(seed >> 32);
  key.c2 = (uint32_t)(step & 0xFFFFFFFFu);
  key.c3 = (uint32_t)(step >> 32);
  key.mask = score_mask;

  const SelectWindow sw = select_window(N, crn, B);
  c->samp.k_host = crn < (int64_t)B ? c->host_pin : nullptr;   // (otherwise U <= B <= ceil(r*N))
  const SampleScratch& sc = c->samp;
  // the timing hooks report the launches of this call, not those of an earlier one on the other way
  for (int id = KID_SAMPLE_SCAN; id <= KID_SAMPLE_REMAP; ++id) c->ev_used[id] = 0;
  if (window_select(N, crn, B, score_mask, sw)) {
    const int cls_log2 = sample_write_log2(N), nblk = (int)sample_write_blocks(N);
    const int split = cls_log2 - sample_cls_log2(N), nscan = nblk << split;
    const uint32_t part_mask = list_parts(nscan) - 1;
    const Window win{sw.lo, sw.width, sw.shift};
    // few labels: more workgroups of fewer each, whose chains are shorter; many: fewer atomics on a word
    const int labels_per = B <= 1024 ? 2 : 4, mark_blocks = (B + kThreads * labels_per - 1) / (kThreads * labels_per);
    auto scan_kernel = labels_per == 2 ? sample_scan_kernel<2> : sample_scan_kernel<4>;
    PFC_LAUNCH(c, KID_SAMPLE_SCAN, scan_kernel, dim3(nscan + mark_blocks), dim3(kThreads),
               0, N, key, win, sc, cls_log2, nblk, split, part_mask, labels, B, c->err_flag);
    // entries that a thread keeps: what a longer part has to its usual length, within the list
    const double part = sw.expected * ((nscan + part_mask) / (part_mask + 1)) / nscan;
    const uint32_t threads = kWriteThreads / (part_mask + 1), cap_each = sc.list_cap / (part_mask + 1) / threads;
    const uint32_t keep = std::min({24u, cap_each, (uint32_t)ceil((part + 4.0 * sqrt(part)) / threads)});
    auto write_kernel = keep <= 2    ? sample_write_kernel<2>
                        : keep <= 6  ? sample_write_kernel<6>
                        : keep <= 16 ? sample_write_kernel<16>
                                     : sample_write_kernel<24>;
    PFC_LAUNCH(c, KID_SAMPLE_WRITE, write_kernel, dim3(nblk), dim3(kWriteThreads), 0, N, key, win, sc,
               cls_log2, nblk, split, part_mask, keep, (uint32_t)crn, labels, B, cap, idx_out, yl_out);
  } else {
    const int rc = sample_radix(c, labels, B, (uint32_t)crn, cap, key, idx_out, yl_out);
    if (rc != PFC_OK) return rc;
  }

  if (!sc.k_host) {
    *k_out = crn;
  } else {
    PFC_HIP(hipStreamSynchronize(c->stream));
    *k_out = (int64_t)*(volatile const uint32_t*)sc.k_host;
  }
  return PFC_OK;
}

}  // namespace pfc

// ---------------------------------------------------------------------------------------------
// pfc_sample_noalloc: pfc_sample for callers that cannot allocate.  The sampler's scratch lives in
// ONE file-scope device array per GPU instead of a context's hipMalloc'ed buffer; the kernels are
// those of pfc_sample and take its pieces as pointers.
// ---------------------------------------------------------------------------------------------
namespace {

constexpr int64_t kNoallocMaxN = (int64_t)1 << 24;                               // 16,777,216 classes
constexpr int64_t kNoallocMaxB = (int64_t)1 << 20;
// what sample_layout asks for at (kNoallocMaxN, kNoallocMaxB), checked on every call
constexpr size_t kNaBytes = (size_t)9 << 20;

// Zero when the code object is loaded; afterwards every call leaves it so that the next one finds
// its set cleared (see above), except the error word, which only ever gains bits.
static __device__ __align__(256) uint32_t scratch[kNaBytes / 4];

constexpr int kNaMaxDevices = 64;
std::mutex g_na_mutex;
uint32_t* g_na_ptr[kNaMaxDevices];   // device address of `scratch` on each GPU, once looked up

// The array's name is only a host-side handle: its address on the current device comes from the
// runtime, once per device, and is what the kernels are given.
int noalloc_scratch(uint32_t** out) {
  int dev = -1;
  PFC_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kNaMaxDevices) return PFC_EINVAL;
  std::lock_guard<std::mutex> lock(g_na_mutex);
  if (!g_na_ptr[dev]) {
    uint32_t* p = nullptr;
    PFC_HIP(hipGetSymbolAddress((void**)&p, HIP_SYMBOL(scratch)));
    if (!p) return PFC_EHIP;
    g_na_ptr[dev] = p;
  }
  *out = g_na_ptr[dev];
  return PFC_OK;
}

}  // namespace

extern "C" int pfc_sample_noalloc(const int64_t* labels, int32_t B, int64_t N, double r,
                                  uint64_t seed, uint64_t step, int32_t* idx_out,
                                  int32_t* labels_local_out, int64_t* k_out, void* hip_stream) {
  if (!labels || !idx_out || !labels_local_out || !k_out) return PFC_EINVAL;
  if (N < 1 || N > kNoallocMaxN) return PFC_EINVAL;
  if (B < 1 || B > (1 << 20)) return PFC_EINVAL;
  if (!(r > 0.0) || !(r <= 1.0)) return PFC_EINVAL;
  // k must be known without reading anything back: no waiting, no pinned buffer
  if ((int64_t)ceil(r * (double)N) < (int64_t)B) return PFC_EINVAL;
  uint32_t* base = nullptr;
  const int rc = noalloc_scratch(&base);
  if (rc != PFC_OK) return rc;
  pfc_ctx c;   // a view of the static scratch on the stack: nothing is allocated, nothing kept
  memset(&c, 0, sizeof(c));
  c.N = N;
  c.stream = (hipStream_t)hip_stream;
  // the layout of the largest call, so that every call finds the sets of the one before
  const size_t need = pfc::sample_layout(kNoallocMaxN, kNoallocMaxB, (char*)base, &c.samp);
  if (need > kNaBytes) return PFC_EINVAL;
  c.err_flag = reinterpret_cast<int32_t*>(&c.samp.st->spare[0]);
  return pfc::sample_impl(&c, labels, B, r, seed, step, 0xFFFFFFFFu, idx_out, labels_local_out,
                          k_out);
}
