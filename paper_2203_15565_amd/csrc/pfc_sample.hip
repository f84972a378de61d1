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
// What bounds it: latency (a launch takes 5 us whatever it does; sample_write is a chain of four
// dependent reads) and, for many classes, the one Philox block per four of them (13 us of integer
// work at 10 million).  Measured with rocprofv3, sum of the sampler's kernels, at N = 93,431 /
// 2,059,906 / 10,000,000: three radix passes, count, write and label remap, which recomputed the
// scores in five of six launches, 38 / 57 / 120 us; these two 15 / 25 / 52 us.
#include <math.h>
#include <string.h>

#include <mutex>

#include "pfc_common.h"
#include "pfc_sample_device.h"
#include "pfc_sample_plan.h"

namespace pfc {

namespace {

constexpr int kThreads = 256;
constexpr int kWriteThreads = 512;   // of sample_write

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
// sample_scan.  Workgroup b < nblk scores the classes [b << cls_log2, (b + 1) << cls_log2); the
// workgroups behind those mark the batch classes in the same launch: the one thread that sets a
// class's bit first counts the class, as one that the bits of the first part hold already or not,
// and lists its key if its score lies in the window (the first part lists it too, not knowing the
// batch).  Integer atomics only: the counts do not depend on the order, and the lists are read as
// sets.
// The counts of the workgroups' classes are added up in LDS first: with ids in the order of the classes'
// frequency one range of them owns thousands of the batch's classes, whose atomics on its one count queue
// up (2,059,906 classes without negatives, labels dense in the low ids: 16,384 samples 52 -> 39 us,
// 65,536 114 -> 78; spread evenly 38 -> 36 and 75 -> 66).
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void sample_scan_kernel(
    int64_t N, PhiloxKey key, Window win, SampleScratch sc, int cls_log2, int nblk,
    const int64_t* __restrict__ labels, int B, int32_t* __restrict__ err_flag) {
  const uint32_t par = sc.st->next & 1u;
  SampleHdr* hdr = &sc.st->hdr[par];
  const int lane = threadIdx.x & 63;
  __shared__ uint64_t s_list[kLocalList];
  if ((int)blockIdx.x >= nblk) {   // marking part of the launch
    uint32_t* s_pos = reinterpret_cast<uint32_t*>(s_list);
    const bool gather = nblk <= kMaxBlocks;
    if (gather) {
      for (int b = threadIdx.x; b < nblk; b += kThreads) s_pos[b] = 0u;
      __syncthreads();
    }
    const int i = ((int)blockIdx.x - nblk) * kThreads + threadIdx.x;
    const int64_t y = i < B ? labels[i] : 0;
    const bool valid = i < B && y >= 0 && y < N;
    if (i < B && !valid) atomicOr(err_flag, 1);
    const bool lead = first_of_label(y, valid);
    bool first = false, above = false;
    if (lead) {
      const uint32_t bit = 1u << (y & 31);
      first = !(atomicOr(&sc.pos_bits[par][y >> 5], bit) & bit);
      if (first) {   // first to mark class y
        uint32_t u[4];
        philox_block((uint32_t)(y >> 2), key, u);
        const uint32_t uy = u[y & 3];
        above = win.above(uy);
        atomicAdd(gather ? &s_pos[y >> cls_log2] : &sc.blk_pos[par][y >> cls_log2], above ? 0x10000u : 1u);
        if (win.inside(uy)) {
          const uint32_t p = atomicAdd(&hdr->npos, 1u);
          if (p < sc.pos_cap) sc.pos_list[par][p] = select_key(uy, (uint32_t)y);
        }
      }
    }
    const uint32_t nf = __popcll(__ballot(first)), na = __popcll(__ballot(above));
    if (lane == 0) {
      if (nf) atomicAdd(&hdr->U, nf);
      if (na) atomicAdd(&hdr->pos_above, na);
    }
    if (gather) {
      __syncthreads();
      for (int b = threadIdx.x; b < nblk; b += kThreads)
        if (s_pos[b]) atomicAdd(&sc.blk_pos[par][b], s_pos[b]);
    }
    return;
  }
  __shared__ uint32_t s_n, s_base, sm[4];
  if (threadIdx.x == 0) s_n = 0u;
  __syncthreads();
  const uint32_t nq = (uint32_t)((N + 3) >> 2);
  const uint32_t q0 = blockIdx.x << (cls_log2 - 2);
  const int iters = 1 << (cls_log2 - 10);
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
    if (n) s_base = atomicAdd(&hdr->listed, n);
    if (n > (uint32_t)kLocalList) atomicOr(&hdr->overflow, 1u);
    if (blockIdx.x == 0) {
      sc.st->cur = par;
      hdr->nblk = (uint32_t)nblk;
      hdr->nwords = (uint32_t)((N + 31) >> 5);
    }
  }
  if (n == 0) return;
  __syncthreads();
  const uint32_t base = s_base;
  for (uint32_t e = threadIdx.x; e < n && e < (uint32_t)kLocalList; e += kThreads)
    if (base + e < sc.list_cap) sc.list[base + e] = s_list[e];
}

// ---------------------------------------------------------------------------------------------
// sample_write.
// ---------------------------------------------------------------------------------------------
struct WriteShared {
  uint32_t sm[kWriteThreads / 64];
  uint32_t hist[4096];                      // window bins, or radix bins of the slow select
  uint32_t word[1 << (kMaxClsLog2 - 5)];    // chosen classes of this workgroup
  uint32_t pre[1 << (kMaxClsLog2 - 5)];     // chosen classes in front of each word
  uint64_t bin_list[kBinList];
  uint32_t bin_n;
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
    int64_t N, PhiloxKey key, Window win, SampleScratch sc, int cls_log2, int nblk,
    uint32_t ceil_rN, const int64_t* __restrict__ labels, int B, int64_t cap,
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
#pragma unroll
  for (int c = 0; c < NE; ++c) {
    const uint32_t e = c * NT + t;
    x[c] = e < sc.list_cap ? sc.list[e] : 0ull;
  }
  const uint32_t par = sc.st->cur & 1u;
  const SampleHdr *hp0 = &sc.st->hdr[0], *hp1 = &sc.st->hdr[1];
  auto pick = [&](uint32_t SampleHdr::*f) {
    const uint32_t a = hp0->*f, b = hp1->*f;
    return par ? b : a;
  };
  const uint32_t U = pick(&SampleHdr::U), pos_above = pick(&SampleHdr::pos_above),
                 npos = pick(&SampleHdr::npos), overflow = pick(&SampleHdr::overflow),
                 listed = pick(&SampleHdr::listed);
  const uint32_t old_words = par ? hp0->nwords : hp1->nwords,
                 old_blk = par ? hp0->nblk : hp1->nblk;
  // counts: of every workgroup (does the window hold the end of the selection?) and of those in
  // front (where does this one's output start?)
  uint32_t tot_above = 0, front = 0, front_pos = 0;
  for (uint32_t b = t; b < (uint32_t)nblk; b += NT) {
    const uint32_t a = sc.above_cnt[b], p0 = sc.blk_pos[0][b], p1 = sc.blk_pos[1][b];
    const uint32_t p = par ? p1 : p0;
    tot_above += a;
    if (b < me) {
      front += a + (p & 0xFFFFu);
      front_pos += (p & 0xFFFFu) + (p >> 16);
    }
  }
  const uint32_t k = U > ceil_rN ? U : ceil_rN;
  const uint32_t R = k - U;   // negatives to take
  const uint32_t* pos_bits = par ? sc.pos_bits[1] : sc.pos_bits[0];
  for (int b = t; b < kWindowBins; b += NT) s.hist[b] = 0u;
  for (int w = t; w < own_words; w += NT) {
    uint32_t v = 0u;
    if (word0 + w < nwords) {
      const uint32_t p0 = sc.pos_bits[0][word0 + w], p1 = sc.pos_bits[1][word0 + w];
      v = (par ? p1 : p0) | (R ? sc.above_bits[word0 + w] : 0u);
    }
    s.word[w] = v;
  }
  if (t == 0) {
    s.bin_n = 0u;
    s.key_end = 0ull;
  }
  tot_above = block_sum<NT>(tot_above, s.sm);
  front = block_sum<NT>(R ? front : front_pos, s.sm);
  uint32_t out = front;
  if (R != 0) {
    const uint32_t n = listed;
    const uint32_t neg_above = tot_above - pos_above;
    const uint32_t need = R - neg_above;
    bool ok = overflow == 0u && npos <= sc.pos_cap && n <= sc.list_cap && neg_above <= R &&
              R <= neg_above + (n - npos);
    auto each = [&](auto fn) {   // fn(key) for every entry of the list
#pragma unroll
      for (int c = 0; c < NE; ++c)
        if ((uint32_t)(c * NT + t) < n) fn(x[c]);
      for (uint32_t e = NE * NT + t; e < n; e += NT) fn(sc.list[e]);
    };
    auto bin_of = [&](uint64_t y) { return (~(uint32_t)(y >> 32) - win.lo) >> win.shift; };
    const uint64_t* pl = par ? sc.pos_list[1] : sc.pos_list[0];
    if (ok && need) {
      // negatives of the window by bin (the list holds batch classes too: taken out again)
      each([&](uint64_t y) { atomicAdd(&s.hist[bin_of(y)], 1u); });
      for (uint32_t e = t; e < npos; e += NT) atomicSub(&s.hist[bin_of(pl[e])], 1u);
      __syncthreads();
      uint32_t bin, inside;
      find_bin<NT, kWindowBins>(s.hist, need, s.sm, bin, inside);
      each([&](uint64_t y) {
        const uint32_t j = (uint32_t)y;
        if (bin_of(y) == bin && !((pos_bits[j >> 5] >> (j & 31u)) & 1u)) {
          const uint32_t p = atomicAdd(&s.bin_n, 1u);
          if (p < (uint32_t)kBinList) s.bin_list[p] = y;
        }
      });
      __syncthreads();
      const uint32_t nb = s.bin_n;
      ok = nb <= (uint32_t)kBinList;
      if (ok && (uint32_t)t < nb) {
        const uint64_t mine = s.bin_list[t];
        uint32_t rank = 0;
        for (uint32_t e = 0; e < nb; ++e) rank += s.bin_list[e] < mine ? 1u : 0u;
        if (rank == inside - 1u) s.key_end = mine + 1ull;   // keys below this are taken
      }
      __syncthreads();
    }
    if (ok) {
      if (need) {
        const uint64_t end = s.key_end;
        uint32_t c = 0;
        each([&](uint64_t y) {
          if (y >= end) return;
          const uint32_t j = (uint32_t)y, b = j >> cls_log2;
          if (b < me) ++c;
          else if (b == me) atomicOr(&s.word[(j >> 5) - word0], 1u << (j & 31u));
        });
        // a batch class in the window was counted as one already
        for (uint32_t e = t; e < npos; e += NT) {
          const uint64_t y = pl[e];
          if (y < end && ((uint32_t)y >> cls_log2) < me) --c;
        }
        out += block_sum<NT>(c, s.sm);
      }
    } else {
      out = slow_select(N, key, pos_bits, R, cls_log2, s);
    }
  }
  __syncthreads();

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
  // positions of the labels that lie here (-1 for a bad label), four loads in flight
  for (int i0 = t; i0 < B; i0 += 4 * NT) {
    int64_t ys[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) ys[c] = i0 + c * NT < B ? labels[i0 + c * NT] : 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int i = i0 + c * NT;
      const int64_t y = ys[c];
      if (i >= B) break;
      if (y < 0 || y >= N) {
        if (me == 0) yl_out[i] = -1;
      } else if ((uint32_t)(y >> cls_log2) == me) {
        const uint32_t w = (uint32_t)(y >> 5) - word0;
        const uint32_t pos = out0 + s.pre[w] + __popc(s.word[w] & ((1u << (y & 31)) - 1u));
        yl_out[i] = (int64_t)pos < cap ? (int32_t)pos : -1;
      }
    }
  }
  // clear the other set for the next call (this launch uses none of it but the two sizes, and
  // those stay)
  uint32_t* old_bits = par ? sc.pos_bits[0] : sc.pos_bits[1];
  uint32_t* old_pos = par ? sc.blk_pos[0] : sc.blk_pos[1];
  for (uint32_t w = me * NT + t; w < old_words; w += (uint32_t)nblk * NT)
    old_bits[w] = 0u;
  for (uint32_t b = me * NT + t; b < old_blk; b += (uint32_t)nblk * NT)
    old_pos[b] = 0u;
  if (me == 0 && t == 0) {
    SampleHdr* old = par ? &sc.st->hdr[0] : &sc.st->hdr[1];
    old->U = 0u;
    old->pos_above = 0u;
    old->npos = 0u;
    old->overflow = 0u;
    old->listed = 0u;
    sc.st->k = k;
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
  const int64_t nb = sample_blocks(N);
  const size_t blk = (size_t)(nb > kMaxBlocks ? nb : kMaxBlocks);   // smaller N may have more blocks
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
  const SampleScratch& sc = c->samp;
  // the timing hooks report the launches of this call, not those of an earlier one on the other way
  for (int id = KID_SAMPLE_SCAN; id <= KID_SAMPLE_REMAP; ++id) c->ev_used[id] = 0;
  if (window_select(N, crn, B, score_mask, sw)) {
    const int cls_log2 = sample_cls_log2(N), nblk = (int)sample_blocks(N);
    const Window win{sw.lo, sw.width, sw.shift};
    const int mark_blocks = (B + kThreads - 1) / kThreads;
    PFC_LAUNCH(c, KID_SAMPLE_SCAN, sample_scan_kernel, dim3(nblk + mark_blocks), dim3(kThreads), 0, N,
               key, win, sc, cls_log2, nblk, labels, B, c->err_flag);
    const double usual = sw.expected + 4.0 * sqrt(sw.expected);
    auto write_kernel = usual <= 2.0 * kWriteThreads   ? sample_write_kernel<2>
                        : usual <= 6.0 * kWriteThreads ? sample_write_kernel<6>
                        : usual <= 16. * kWriteThreads ? sample_write_kernel<16>
                                                       : sample_write_kernel<24>;
    PFC_LAUNCH(c, KID_SAMPLE_WRITE, write_kernel, dim3(nblk), dim3(kWriteThreads), 0, N, key, win, sc,
               cls_log2, nblk, (uint32_t)crn, labels, B, cap, idx_out, yl_out);
  } else {
    const int rc = sample_radix(c, labels, B, (uint32_t)crn, cap, key, idx_out, yl_out);
    if (rc != PFC_OK) return rc;
  }

  if (crn >= (int64_t)B) {
    // U <= B <= ceil(r*N): k is known without the labels.
    *k_out = crn;
  } else {
    PFC_HIP(hipMemcpyAsync(c->host_pin, &sc.st->k, 4, hipMemcpyDeviceToHost, c->stream));
    PFC_HIP(hipStreamSynchronize(c->stream));
    *k_out = (int64_t)c->host_pin[0];
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
