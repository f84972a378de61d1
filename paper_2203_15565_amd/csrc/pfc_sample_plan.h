// Host-side rules of pfc_sample: how the classes are dealt to workgroups, the window of scores in
// which the selection ends, and which of the two selections a call takes.  Plain C++, so that the
// rules can be checked on the CPU over everything that the entry points accept.
#pragma once

#include <math.h>
#include <stdint.h>

namespace pfc {

constexpr int kWindowBins = 1024;      // histogram of the window (LDS)
constexpr int kLocalList = 4096;       // classes of one workgroup that may lie in the window
constexpr int kBinList = 256;          // classes that may share the bin in which the selection ends
constexpr int kListParts = 8;          // parts of the list of the window
constexpr int kMinClsLog2 = 10, kMaxClsLog2 = 15;   // classes per workgroup: 2^10 .. 2^15
constexpr int kMaxBlocks = 640;        // workgroups, as long as 2^15 classes each suffice for that
                                       // (up to 20,971,520 classes; beyond, one per 2^15 classes)
constexpr int64_t kWindowBatch = 1 << 16;     // largest batch of the window selection
constexpr int64_t kMissClasses = 10 * 1024;   // classes up to which a missed window costs little

// Classes per workgroup of sample_scan (log2): few enough workgroups that the parts every one of them repeats
// (the list, the counts, the labels) stay small, enough of them to use the GPU (up to 2.5 per
// compute unit).
inline int sample_cls_log2(int64_t N) {
  int l = kMinClsLog2;
  while (l < kMaxClsLog2 && ((N + ((int64_t)1 << l) - 1) >> l) > kMaxBlocks) ++l;
  return l;
}

inline int64_t sample_blocks(int64_t N) {
  const int l = sample_cls_log2(N);
  return (N + ((int64_t)1 << l) - 1) >> l;
}

// Of sample_write: no more workgroups than the compute units hold at a time (two each), because each
// goes through the whole list (10 million classes: 611 workgroups, which are two rounds, 35 us, 306 of
// twice the classes 24; the scores, which are work, stay with 611: 20 us there).
inline int sample_write_log2(int64_t N) {
  const int l = sample_cls_log2(N);
  return l < kMaxClsLog2 && sample_blocks(N) > 512 ? l + 1 : l;
}

// Parts of the list of the window, one count each: the workgroups of sample_scan queue up on a count
// (503 on one count: 5 us of a launch of 11).  Few workgroups would fill the parts unevenly.
inline int list_parts(int scan_blocks) { return scan_blocks >= 64 ? kListParts : 1; }

// Half width of the window in classes at rank n q of N (two thirds of it are never used up).
inline double window_margin(double n, double q) { return 6.5 * sqrt(n * q * (1.0 - q)) + 40.0; }

struct SelectWindow {
  uint32_t lo, width;   // scores lo .. lo + width, both inside
  int shift;            // bin of a score inside: (score - lo) >> shift, below kWindowBins
  double expected;      // classes inside, on average
};

// The window of scores in which the selection of k - U negatives ends.  Counted over ALL classes,
// the last class taken is number n0 = k - U + (batch classes above it) from the top, between
// ceil_rN - B and ceil_rN whatever the batch holds.  The number of classes at or above the score
// 2^32 (1 - q) is binomial(N, q): 6.5 standard deviations and a constant for small counts.
inline SelectWindow select_window(int64_t N, int64_t ceil_rN, int64_t B) {
  const double n = (double)N;
  auto margin = [&](double rank) {
    const double q = rank < 0 ? 0 : rank > n ? 1 : rank / n;
    return window_margin(n, q);
  };
  const double hi_rank = (double)ceil_rN, lo_rank = (double)ceil_rN - (double)B;
  double top = lo_rank - margin(lo_rank < 0 ? 0 : lo_rank), bot = hi_rank + margin(hi_rank);
  if (top < 0) top = 0;
  if (bot > n) bot = n;
  const double two32 = 4294967296.0;
  double lo = floor(two32 * (1.0 - bot / n)), hi = ceil(two32 * (1.0 - top / n)) - 1.0;
  if (bot >= n) lo = 0;
  if (top <= 0 || hi > two32 - 1.0) hi = two32 - 1.0;
  if (lo > hi) lo = hi;
  SelectWindow w;
  w.lo = (uint32_t)lo;
  w.width = (uint32_t)hi - w.lo;
  w.shift = 0;
  while ((w.width >> w.shift) >= (uint32_t)kWindowBins) ++w.shift;
  w.expected = bot - top;
  return w;
}

// Entries that the list of the window needs: twice what the widest window of a call holds on average,
// and room for small numbers.
inline int64_t window_list_cap(int64_t N, int64_t B) {
  int64_t b = B < N ? B : N;
  if (b > kWindowBatch) b = kWindowBatch;
  return (int64_t)(2.0 * ((double)b + 2.0 * window_margin((double)N, 0.5))) + 4096;
}

// Entries that the list of the batch classes inside the window needs: all of them may lie there.  Larger
// batches never take the window.
inline int64_t window_pos_cap(int64_t B) { return B < kWindowBatch ? B : kWindowBatch; }

// Whether a mask leaves the scores where the window expects them: it only clears low bits, and there
// is no more than one class to a step of what is left, on average.
inline bool mask_keeps_window(int64_t N, uint32_t mask) {
  const uint32_t cleared = ~mask;
  return (cleared & (cleared + 1u)) == 0u && (uint64_t)N * ((uint64_t)cleared + 1u) <= ((uint64_t)1 << 32);
}

// Mean number of classes in a bin of the window's histogram.
inline double window_bin_classes(int64_t N, const SelectWindow& w) {
  return (double)N * (double)((uint64_t)1 << w.shift) / 4294967296.0;
}

// Which selection: the window (two launches), or the radix passes (six), whose cost does not depend
// on where the scores lie and on the batch only through its marking.
//
// The window is at least the batch wide, and each of its workgroups goes through the whole list of
// the window and all labels, so it loses where the batch is large; a mask that moves the scores away
// from the window makes every workgroup select for itself.  The end bin has to hold the classes that
// fall into it (8 standard deviations kept).
//
// The line between them is an estimate of both in us, fitted to 306 forms of 8 thousand .. 16.7 million classes
// and batches of 2,048 .. 65,536 on 256 compute units (beyond, up to 200 million classes and batches from
// 4,096); the way it picks is 0.1 % behind the other on average, 13 % at most (65,536 samples of 8,000
// classes).  Measured, window / radix:
//   N = 93,431, r = 0.1:      B = 8,192 25.8 / 42.0;  no negatives: 32,768 44 / 57, 65,536 64 / 74
//   N = 2,059,906, r = 0.1:   B = 16,384 51 / 60, 32,768 89 / 68, 65,536 165 / 84, 262,144 3,869 / 187
//   N = 2,059,906, no negatives: B = 16,384 37 / 60, 65,536 67 / 85
//   N = 6,000,000, r = 0.1:   B = 16,384 62 / 86, 32,768 93 / 95
//   N = 16,700,000, r = 0.5:  B = 49,152 169 / 184, 65,536 204 / 194
//   N = 2,059,906, mask 0x3FF: 8,168 / 69; N = 10,000 41 / 42; N = 15,000 51 / 44
inline bool window_select(int64_t N, int64_t ceil_rN, int64_t B, uint32_t mask, const SelectWindow& w) {
  if (B > kWindowBatch) return false;
  if (!mask_keeps_window(N, mask)) return N <= kMissClasses;
  const double bin = window_bin_classes(N, w);
  if (bin + 8.0 * sqrt(bin) + 8.0 > (double)kBinList) return false;
  // in millions of classes, thousands of samples, list entries and distinct labels
  const double n = (double)N, classes = n * 1e-6, b = (double)B * 1e-3;
  const double list = ceil_rN > 1 ? w.expected * 1e-3 : 0.0;   // no negatives: nothing to look for
  const double distinct = n * (1.0 - exp(-(double)B / n)) * 1e-3;
  const double blocks = (double)sample_blocks(N);
  // more workgroups than the compute units hold at a time (two each) repeat the common part later
  const double rounds = 1.0 + 0.75 * floor((blocks - 1.0) / 512.0);
  // every workgroup: its classes, the list, all labels; and atomics on the counts of a workgroup and
  // on the list of the batch classes inside the window
  const double window_us = 7.0 + 1.4 * classes + rounds * (1.1 * list + b) + 2.5 * distinct / blocks +
                           1.05 * distinct * fmin(1.0, w.expected / n);
  // the passes over the classes, the counts in front of each workgroup (their square), the labels
  const double far = fmax(0.0, classes - 20.0);
  const double radix_us = 31.0 + 6.9 * classes + 0.035 * far * far + 0.68 * b;
  return window_us <= radix_us;
}

}  // namespace pfc
