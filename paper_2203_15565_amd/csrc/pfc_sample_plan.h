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

inline int64_t sample_write_blocks(int64_t N) {
  const int l = sample_write_log2(N);
  return (N + ((int64_t)1 << l) - 1) >> l;
}

// Counts that the scratch has room for: of sample_write's workgroups, and of sample_scan's, which are whole
// ones of those.  (Smaller N may have more of either.)
inline int64_t sample_count_cap(int64_t N) {
  const int64_t n = sample_blocks(N);
  return n > kMaxBlocks ? n : kMaxBlocks;
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
// The line between them is an estimate of both in us, fitted to 369 forms of 8 thousand .. 200 million
// classes and batches of 2,048 .. 65,536 on 256 compute units; over these the way it picks is 0.3 %
// behind the other on average and 5 % at most, but for batches whose distinct labels leave no negative
// to look for, which the rule cannot know (40,000 classes, r = 0.5, 32,768 samples: 40.6 / 52.1, and it
// picks the second).  The workgroups that count are those of sample_write.  (With those of sample_scan,
// and weights of kernels that marked label by label, grids that sample_write halves took the radix
// passes too early: 1,187,840 classes, r = 0.1, 8,192 samples 46.9 us instead of 28.0; 8,437,760 and
// 16,384 97.7 instead of 61.2.)  Measured, window / radix, calls back to back (without negatives the
// wait for k is in it; the masked ones were measured on kernels that marked label by label):
//   N = 527,360, r = 0.1:     B = 8,192 26.3 / 39.7, 16,384 38 / 43, 24,576 53 / 47
//   N = 2,109,440, r = 0.1:   B = 16,384 44 / 58, 24,576 57 / 63, 32,768 72 / 67, 65,536 130 / 83
//   N = 2,059,906, no negatives: B = 16,384 34 / 57, 65,536 55 / 82
//   N = 6,553,600, r = 0.1:   B = 16,384 55 / 85, 32,768 82 / 94, 65,536 139 / 110
//   N = 10,469,376, r = 0.1:  B = 32,768 93 / 118, 49,152 120 / 126, 65,536 147 / 134
//   N = 20,000,000, r = 0.01: B = 32,768 136 / 166, 49,152 183 / 175;  60,000,000: 65,536 490 / 501
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
  const double blocks = (double)sample_write_blocks(N);
  // more workgroups than the compute units hold at a time (two each) repeat the common part later
  const double rounds = 1.0 + 0.75 * floor((blocks - 1.0) / 512.0);
  // every workgroup: its classes, the list, all labels; and atomics on the counts of a workgroup and
  // on the list of the batch classes inside the window
  const double window_us = 10.0 + 1.3 * classes + rounds * (list + 0.6 * b) + distinct / blocks +
                           0.5 * distinct * fmin(1.0, w.expected / n);
  // the passes over the classes, the counts in front of each workgroup (their square), the labels
  const double far = fmax(0.0, classes - 20.0);
  const double radix_us = 32.0 + 6.9 * classes + 0.035 * far * far + 0.55 * b;
  return window_us <= radix_us;
}

}  // namespace pfc
