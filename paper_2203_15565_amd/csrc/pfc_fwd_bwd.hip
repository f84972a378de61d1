// pfc_forward_backward: margin-softmax loss over the sampled centers and its gradients
// (arXiv 2203.15565: Eq. 1 restricted to the sampled set S as in Eq. 4; Eq. 2 / Eq. 4 for the
// feature gradient, the bracket of Eq. 3 for the center gradient).
//
// Pipeline (one stream, no host synchronisation):
//   gather_normalize   Xn = x/|x|, Wn = W[idx]/|W[idx]|             (HBM bound)
//   gemm_logits        c = Wn Xn^T, margin, e = exp(s c) -> E and per-tile row sums (MFMA)
//   row_combine        l_i, lse_i, per-row loss, s/(B l_i), label-column coefficient,
//                      Xs = (s/(B l_i)) xn_i
//   gemm_backward      both backward products in one launch (MFMA): partial sums of E Wn over
//                      slices of S, and dWn = E^T Xs (off-label part)
//   gradients_final    adds the label-column term to the dWn rows of positive classes (fp32); features:
//                      reduce slices, scale, label term, project through x -> x/|x|; mean loss
// In the fused call the label-column term (dweight_label, into a side buffer) comes before
// gemm_backward_update, whose dweight tiles end in the update of their rows.
//
// Cosines lie in [-1,1]: up to s = 64, exp(s c) lies in [e^-64, e^64] and a row sum over at most
// 2^31 classes stays below 3.4e38, so exp needs no running maximum and one fixed reference (zero)
// serves every tile, p_ij = E_ij / l_i with l_i known only after the GEMM.  Above s = 64 one more
// pass of the logit GEMM (gemm_rowmax, row_ref) finds each sample's largest logit first and the
// softmax runs relative to it.
// The label column is kept out of E (stored as zero) and handled in fp32 on the side, where
// (p - 1) and the margin derivative are formed without bf16 rounding.
#include <limits.h>
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "pfc_common.h"
#include "pfc_gemm.h"
#include "pfc_step_plan.h"

// Phase clocks for tuning, compiled in only with -DPFC_PHASES (never in the shipped library):
// thread 0 of every workgroup of the selected kernel stores the constant-rate clock at up to 8
// points.  Kernel tags: 1 logits, 2 dweight, 3 dweight+update.
#ifdef PFC_PHASES
__device__ unsigned long long pfc_phase_buf[32768 * 8];
__device__ int pfc_phase_sel;
#define PFC_PHASE(tag, slot)                                                               \
  do {                                                                                     \
    if (threadIdx.x == 0 && blockIdx.x < 32768 && pfc_phase_sel == (tag))                  \
      pfc_phase_buf[blockIdx.x * 8 + (slot)] = __builtin_amdgcn_s_memrealtime();               \
  } while (0)
extern "C" int pfc_debug_phases(unsigned long long* host_out, int n) {
  return (int)hipMemcpyFromSymbol(host_out, HIP_SYMBOL(pfc_phase_buf), (size_t)n * 8);
}
extern "C" int pfc_debug_select(int tag) {
  void* p = nullptr;
  if (hipGetSymbolAddress(&p, HIP_SYMBOL(pfc_phase_buf)) != hipSuccess) return -1;
  if (hipMemset(p, 0, sizeof(unsigned long long) * 32768 * 8) != hipSuccess) return -2;
  return (int)hipMemcpyToSymbol(HIP_SYMBOL(pfc_phase_sel), &tag, sizeof(int));
}
#else
#define PFC_PHASE(tag, slot)
#endif

namespace pfc {

namespace {

constexpr float kEpsNorm = 1e-12f;
constexpr float kEpsSin2 = 1e-12f;

// ---------------------------------------------------------------------------------------------
// normalize_x_row: one wavefront per (padded) feature row.
//
// Row length: the caller's arrays (X, W, v, dX, dWn) have rows of D floats, D a multiple of 64.
// The library's own GEMM operands (Xn, Xs, Wn and the dfeatures partial sums) have rows of
// Dp >= D elements, D rounded up to 128 (to 256 where the backward launch takes 256-tiles), the
// columns from D on being zero, so that the GEMMs only ever see whole tiles; a wavefront walks a
// row in NC chunks of 256 columns, and kernels that touch the caller's rows skip the columns from
// D on.
// ---------------------------------------------------------------------------------------------
template <typename T, int NC>
__device__ __forceinline__ void normalize_x_row(int i, const float* __restrict__ X, int B, int D,
                                                int Dp, const int32_t* __restrict__ yl, int64_t k,
                                                T* __restrict__ Xn, float* __restrict__ rnormX,
                                                float* __restrict__ clabel,
                                                int32_t* __restrict__ err_flag) {
  const int lane = threadIdx.x & 63;
  constexpr int nchunk = NC;   // float4 chunks per lane
  float4 v[NC];
  float ss = 0.f;
#pragma unroll
  for (int c = 0; c < nchunk; ++c) {
    const int d = c * 256 + lane * 4;
    v[c] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (i < B && d < D) v[c] = *reinterpret_cast<const float4*>(X + (int64_t)i * D + d);
    ss += v[c].x * v[c].x + v[c].y * v[c].y + v[c].z * v[c].z + v[c].w * v[c].w;
  }
  ss = wave_sum(ss);
  const float rn = (i < B) ? 1.f / fmaxf(sqrtf(ss), kEpsNorm) : 0.f;
#pragma unroll
  for (int c = 0; c < nchunk; ++c) {
    if (c * 256 + lane * 4 >= Dp) continue;
    // rn == 0 for padded rows
    const T o[4] = {from_float<T>(v[c].x * rn), from_float<T>(v[c].y * rn),
                    from_float<T>(v[c].z * rn), from_float<T>(v[c].w * rn)};
    __builtin_memcpy(__builtin_assume_aligned(Xn + (int64_t)i * Dp + c * 256 + lane * 4, sizeof(o)),
                     o, sizeof(o));
  }
  if (lane == 0) {
    rnormX[i] = rn;
    clabel[i] = 0.f;
    if (i < B) {
      const int32_t y = yl[i];
      if (y < 0 || (int64_t)y >= k) atomicOr(err_flag, 2);
    }
  }
}

// ---------------------------------------------------------------------------------------------
// order_labels (in gather_normalize, batches of several label windows): the samples of window w
// ordered by class and, inside a class, by number, and where each class begins; samples without a
// class of S are left out.  A bitonic sort of (class, sample) in LDS, 55 passes for 1024 samples,
// beside the other workgroups of the launch.
// ---------------------------------------------------------------------------------------------
constexpr int kNormWaves = 4;   // wavefronts per workgroup
struct OrderLds {
  uint64_t key[kLabelWindow];
  int runs[kNormWaves], samples;
};
__device__ __forceinline__ void order_labels(int w, OrderLds& lds, int B, const int32_t* __restrict__ yl,
                                             int64_t k, int32_t* __restrict__ order,
                                             int32_t* __restrict__ runs) {
  constexpr int THREADS = kNormWaves * 64, PER = kLabelWindow / THREADS;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int i0 = w * kLabelWindow;
  for (int e = t; e < kLabelWindow; e += THREADS) {
    const int32_t y = i0 + e < B ? yl[i0 + e] : -1;
    lds.key[e] = y >= 0 && (int64_t)y < k ? (uint64_t)(uint32_t)y << 32 | (uint32_t)(i0 + e) : ~0ull;
  }
  if (t == 0) lds.samples = 0;
  __syncthreads();
  // A wavefront's pairs lie in its own 256 places as long as partners are at most 128 apart: only
  // the three wider passes need the workgroup to meet, before and behind them.
  static_assert(PER == 4 && kNormWaves == 4, "128 pairs to a wavefront");
  for (int size = 2; size <= kLabelWindow; size *= 2)
    for (int j = size / 2; j > 0; j /= 2) {
#pragma unroll
      for (int u = 0; u < PER / 2; ++u) {
        const int q = wave * 128 + u * 64 + lane, a = (q & ~(j - 1)) * 2 + (q & (j - 1)), b = a + j;
        const uint64_t ka = lds.key[a], kb = lds.key[b];
        if ((ka > kb) == ((a & size) == 0)) {
          lds.key[a] = kb;
          lds.key[b] = ka;
        }
      }
      if (j > 128 || (j == 1 && size >= 256)) {
        __syncthreads();
      } else {   // this wavefront's LDS accesses stay in order
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      }
    }
  // thread t: PER neighbouring places
  bool first[PER];
  int n = 0;
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int at = t * PER + e;
    const uint64_t key = lds.key[at];
    const bool valid = key != ~0ull;
    first[e] = valid && (at == 0 || (lds.key[at - 1] >> 32) != (key >> 32));
    n += first[e];
    if (valid) order[i0 + at] = (int32_t)(uint32_t)key;
    if (valid && (at == kLabelWindow - 1 || lds.key[at + 1] == ~0ull)) lds.samples = at + 1;
  }
  int upto = n;   // classes that begin up to this thread's places, in its wavefront
#pragma unroll
  for (int o = 1; o < 64; o *= 2) {
    const int v = __shfl_up(upto, o, 64);
    if (lane >= o) upto += v;
  }
  if (lane == 63) lds.runs[wave] = upto;
  __syncthreads();
  int before = upto - n, total = 0;
#pragma unroll
  for (int v = 0; v < kNormWaves; ++v) {
    if (v < wave) before += lds.runs[v];
    total += lds.runs[v];
  }
  runs += (int64_t)w * kWindowRuns;
#pragma unroll
  for (int e = 0; e < PER; ++e)
    if (first[e]) runs[1 + before++] = t * PER + e;
  if (t == 0) {
    runs[0] = total;
    runs[1 + total] = lds.samples;
  }
}

// ---------------------------------------------------------------------------------------------
// gather_normalize: the first x_blocks workgroups normalise the features (normalize_x_row), the
// others the sampled centers: the two need nothing of each other, and a launch of its own for a few
// hundred rows of features is 3-5 us that nothing runs beside (step, 128 x 1,000 x 512 fp32 62.2 ->
// 59.8 us, 512 x 9,344 x 512 104.4 -> 102.5).  Centers: one wavefront per group of NB consecutive
// sampled rows, all NB row reads (2 KB each at D = 512, ascending row ids) in flight before the
// first is reduced.  Rows k..kp-1 of Wn are written as zeros.
// ---------------------------------------------------------------------------------------------
// SHORT (rows of at most 128 floats): half a wavefront to a center, twice the centers in flight.
// Step, us, before -> now: 256 samples x 25,723 classes x 128 69.4 -> 67.9, 256 x 40,000 x 64 76.9
// -> 73.7, 300 x 300,000 x 64 368 -> 348.  (In front of either: one workgroup for every label
// window of a large batch, order_labels.)
// PLAIN: the rows of W are to stay in the memory-side cache (row_policy); otherwise they are loaded
// nontemporally, which keeps them from displacing what the GEMMs that follow want (0.145 -> 0.121 ms
// at the headline workload).
template <bool PLAIN>
__device__ __forceinline__ f32x4 load_w(const float* p) {
  if constexpr (PLAIN) return *reinterpret_cast<const f32x4*>(p);
  else return __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p));
}
template <typename T, int NC, bool SHORT, bool PLAIN>
__global__ __launch_bounds__(kNormWaves * 64) void gather_normalize_kernel(
    int x_blocks, const float* __restrict__ X, int B, int Bp, const int32_t* __restrict__ yl,
    T* __restrict__ Xn, float* __restrict__ rnormX, float* __restrict__ clabel,
    const float* __restrict__ W, int64_t N, const int32_t* __restrict__ idx, int64_t k, int64_t kp,
    int D, int Dp, T* __restrict__ Wn, float* __restrict__ rnormW, int32_t* __restrict__ head,
    int nwin, int32_t* __restrict__ order, int32_t* __restrict__ runs, int32_t* __restrict__ err_flag) {
  if ((int)blockIdx.x < nwin) {
    __shared__ OrderLds lds;
    order_labels(blockIdx.x, lds, B, yl, k, order, runs);
    return;
  }
  const int block = (int)blockIdx.x - nwin;
  if (block < x_blocks) {
    const int i = block * kNormWaves + (threadIdx.x >> 6);
    if (i < Bp) normalize_x_row<T, NC>(i, X, B, D, Dp, yl, k, Xn, rnormX, clabel, err_flag);
    return;
  }
  constexpr int NB = 4;
  const int lane = threadIdx.x & 63;
  if constexpr (SHORT) {   // Dp == 128
    const int l = lane & 31, d = l * 4;
    const int64_t js = ((int64_t)(block - x_blocks) * kNormWaves + (threadIdx.x >> 6)) * (2 * NB) + (lane >> 5);
    f32x4 v[NB];
    bool ok[NB];
#pragma unroll
    for (int u = 0; u < NB; ++u) {   // centers js, js + 2, ..
      const int64_t j = js + 2 * u;
      const int64_t row = j < k ? idx[j] : -1;
      ok[u] = row >= 0 && row < N;
      if (j < k && !ok[u] && l == 0) atomicOr(err_flag, 4);
      v[u] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (ok[u] && d < D) v[u] = load_w<PLAIN>(W + row * D + d);
    }
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const int64_t j = js + 2 * u;
      if (j >= kp) break;
      const float ss =
          lane_group_sum<32>(v[u][0] * v[u][0] + v[u][1] * v[u][1] + v[u][2] * v[u][2] + v[u][3] * v[u][3]);
      const float rn = ok[u] ? 1.f / fmaxf(sqrtf(ss), kEpsNorm) : 0.f;
      if (l == 0) {
        rnormW[j] = rn;
        head[j] = 0x7fffffff;
      }
      for (int w = l; w < nwin; w += 32) head[(int64_t)(1 + w) * kp + j] = 0x7fffffff;
      const T o[4] = {from_float<T>(ok[u] ? v[u][0] * rn : 0.f), from_float<T>(ok[u] ? v[u][1] * rn : 0.f),
                      from_float<T>(ok[u] ? v[u][2] * rn : 0.f), from_float<T>(ok[u] ? v[u][3] * rn : 0.f)};
      __builtin_memcpy(__builtin_assume_aligned(Wn + j * Dp + d, sizeof(o)), o, sizeof(o));
    }
    return;
  }
  const int64_t jb = ((int64_t)(block - x_blocks) * kNormWaves + (threadIdx.x >> 6)) * NB;
  if (jb >= kp) return;
  float4 v[NB][NC];
  bool ok[NB];
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    const int64_t j = jb + u;
    ok[u] = false;
    if (j < k) {
      const int64_t row = idx[j];
      ok[u] = (row >= 0 && row < N);
      if (!ok[u] && lane == 0) atomicOr(err_flag, 4);
      if (ok[u]) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          const int d = c * 256 + lane * 4;
          v[u][c] = make_float4(0.f, 0.f, 0.f, 0.f);
          if (d < D) {
            const f32x4 t = load_w<PLAIN>(W + row * D + d);
            v[u][c] = make_float4(t[0], t[1], t[2], t[3]);
          }
        }
      }
    }
  }
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    const int64_t j = jb + u;
    if (j >= kp) break;
    float ss = 0.f;
    if (ok[u]) {
#pragma unroll
      for (int c = 0; c < NC; ++c)
        ss += v[u][c].x * v[u][c].x + v[u][c].y * v[u][c].y + v[u][c].z * v[u][c].z +
              v[u][c].w * v[u][c].w;
    }
    ss = wave_sum(ss);
    const float rn = ok[u] ? 1.f / fmaxf(sqrtf(ss), kEpsNorm) : 0.f;
    if (lane == 0) {
      rnormW[j] = rn;
      head[j] = 0x7fffffff;   // first sample carrying this class: filled in by row_combine
    }
    // likewise the first sample of every window of kLabelWindow samples (large batches only)
    if (lane < nwin) head[(int64_t)(1 + lane) * kp + j] = 0x7fffffff;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      if (c * 256 + lane * 4 >= Dp) continue;
      T o[4];
      if (ok[u]) {
        o[0] = from_float<T>(v[u][c].x * rn);
        o[1] = from_float<T>(v[u][c].y * rn);
        o[2] = from_float<T>(v[u][c].z * rn);
        o[3] = from_float<T>(v[u][c].w * rn);
      } else {
        o[0] = o[1] = o[2] = o[3] = from_float<T>(0.f);
      }
      T* g = Wn + j * Dp + c * 256 + lane * 4;
      if constexpr (sizeof(T) == 2) {
        uint2 pk;
        __builtin_memcpy(&pk, o, 8);
        *reinterpret_cast<uint2*>(g) = pk;
      } else {
        float4 f4;
        f4.x = (float)o[0]; f4.y = (float)o[1]; f4.z = (float)o[2]; f4.w = (float)o[3];
        *reinterpret_cast<float4*>(g) = f4;
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// gemm_logits: tile of c[j][i] (rows = sampled classes, columns = samples), fused epilogue:
// clamp, margin on the label entry, e = exp(s*c), per-tile column sums, and E[i][j] = e (label
// entry and padding stored as zero).  A lane holds one sample i and runs of 4 consecutive
// classes j, so the sums over j are in-lane; in bf16 E lies in octets of classes (OctetLds), which
// a wavefront writes straight from its registers, 512 bytes in one piece.
//
// The element-wise part exists in four versions.  GUARDED: the wavefront's part of the tile holds
// a label entry or padding (few wavefronts do); the plain version costs 5 VALU instructions per
// entry.  EXTRAS: the options are on -- negatives whose cosine exceeds `tau` are left out of the
// softmax (the PFC* filter, Sec. 3.3 / Fig. 4 caption) and the largest non-label cosine of every
// sample is tracked (for AMNCS, Sec. 3.3).
// ---------------------------------------------------------------------------------------------
struct LossParams {
  float s, s_log2e;
  float m, cos_m, sin_m;
  int32_t cosface;   // 0: label logit s*cos(theta+m); 1: s*(cos(theta) - m)
  float tau;         // filter threshold (entries with cosine > tau are dropped); >= 1: off
  int32_t extras;    // filter, column maxima and/or a per-sample reference requested
  const float* rowref;   // [Bp] largest logit of every sample, or null: exp(z - rowref_i) instead
                         // of exp(z) (scales above 64, where exp(z) could leave the fp32 range)
};

__device__ __forceinline__ float label_logit(const LossParams& lp, float c) {
  if (lp.cosface) return lp.s * (c - lp.m);
  return lp.s * (c * lp.cos_m - sqrtf(fmaxf(1.f - c * c, 0.f)) * lp.sin_m);
}

// The row sum of exp(z) enters the gradient through p - 1, which for a confident sample is nothing
// but its rounding: its additions therefore keep one order whether a tile has 128 classes or 64.  A
// wavefront of a 128-tile chains the 32 values a lane holds of 64 classes; a 64-tile, whose
// wavefronts hold 32 classes each, chains the two of them, and row_combine adds the tiles in pairs.
template <class Cfg>
constexpr bool logits_chained() { return Cfg::BM == 64; }

template <class Cfg, bool GUARDED, bool EXTRAS>
__device__ __forceinline__ void logits_epilogue_columns(
    const f32x16 (&acc)[Cfg::TM][Cfg::TN], int64_t j0, int i0, int B, int klim, int64_t kp,
    int Bp, const int (&ylane)[Cfg::TN], const LossParams& lp,
    typename Cfg::elem* __restrict__ E, float* __restrict__ clabel, float (&colsum)[Cfg::TN],
    float (&collab)[Cfg::TN], float (&colmax)[Cfg::TN]) {
  using T = typename Cfg::elem;
  constexpr bool kOctets = sizeof(T) == 2, kChain = logits_chained<Cfg>();
#pragma unroll
  for (int bn = 0; bn < Cfg::TN; ++bn) {
    const int il = acc_col<Cfg>(bn);
    const int i = i0 + il;
    const bool vi = i < B;
    const int yloc = ylane[bn];
    float sum = kChain ? colsum[bn] : 0.f, clab = 0.f, cmax = -2.f;
    float ref = 0.f;
    if constexpr (EXTRAS) ref = lp.rowref ? lp.rowref[i] : 0.f;   // i < Bp: padded entries are 0
    const float ref2 = ref * 1.44269504088896340736f;
#pragma unroll
    for (int bm = 0; bm < Cfg::TM; ++bm) {
      uint32_t w[4][2];
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        T pack[4];
        const int jl = acc_row<Cfg>(bm, g4 * 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float c = __builtin_amdgcn_fmed3f(acc[bm][bn][g4 * 4 + e], -1.f, 1.f);
          // exp(s*c), |s*c*log2(e)| <= 93 without a reference; exp(s*c - ref) <= 1 with one
          float ev = EXTRAS ? __builtin_amdgcn_exp2f(fmaf(c, lp.s_log2e, -ref2))
                            : __builtin_amdgcn_exp2f(c * lp.s_log2e);
          if constexpr (GUARDED) {
            const bool lab = (jl + e == yloc);
            const bool neg = vi && jl + e < klim && !lab;      // a real, non-label entry
            ev = neg ? ev : 0.f;
            clab = lab ? c : clab;
            if constexpr (EXTRAS) {
              cmax = neg ? fmaxf(cmax, c) : cmax;
              ev = (c > lp.tau) ? 0.f : ev;
            }
          } else if constexpr (EXTRAS) {
            cmax = fmaxf(cmax, c);
            ev = (c > lp.tau) ? 0.f : ev;
          }
          sum += ev;
          pack[e] = from_float<T>(ev);
        }
        if constexpr (kOctets) {
          __builtin_memcpy(w[g4], pack, 8);
        } else {
          uint4 pk;
          __builtin_memcpy(&pk, pack, 16);
          *reinterpret_cast<uint4*>(E + (int64_t)i * kp + j0 + jl) = pk;
        }
      }
      if constexpr (kOctets) {
        // The lane halves hold classes 0..3 and 4..7 of every eight: exchanged, a lane has an octet, the
        // second half of the wavefront the next one.
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const auto lo = __builtin_amdgcn_permlane32_swap(w[2 * h][0], w[2 * h + 1][0], false, false);
          const auto hi = __builtin_amdgcn_permlane32_swap(w[2 * h][1], w[2 * h + 1][1], false, false);
          const int64_t octet = ((j0 + acc_row<Cfg>(bm, 0)) >> 3) + 2 * h + ((threadIdx.x >> 5) & 1);
          // E is far larger than the L2 and next read by another kernel: store it nontemporally
          __builtin_nontemporal_store(u32x4{lo[0], hi[0], lo[1], hi[1]},
                                      reinterpret_cast<u32x4*>(E + (octet * Bp + i) * 8));
        }
      }
    }
    if constexpr (GUARDED) {
      if (yloc >= 0) {   // this lane holds sample i's label entry: it was left out of `sum`
        clabel[i] = clab;
        const float el = __expf(label_logit(lp, clab) - ref);
        if constexpr (kChain) collab[bn] = el;
        else sum += el;
      }
    }
    if constexpr (!kChain) sum += __shfl_xor(sum, 32, 64);
    colsum[bn] = sum;
    if constexpr (EXTRAS) colmax[bn] = fmaxf(cmax, __shfl_xor(cmax, 32, 64));
  }
}

template <class Cfg, bool EXTRAS>
__global__ __launch_bounds__(Cfg::THREADS) void gemm_logits_kernel(
    const typename Cfg::elem* __restrict__ Wn, const typename Cfg::elem* __restrict__ Xn, int D,
    int Dp, int64_t k, int B, int Bp, int64_t kp, const int32_t* __restrict__ yl, LossParams lp,
    typename Cfg::elem* __restrict__ E, float* __restrict__ rowpart,
    float* __restrict__ rowmaxpart, float* __restrict__ clabel, int tiles_j, int tiles_i,
    int ahead) {
  using T = typename Cfg::elem;
  extern __shared__ __align__(16) char smem[];
  int tj, ti;
  if (!xcd_tile(blockIdx.x, tiles_i, tiles_j, tj, ti)) return;
  // From the last class down: Wn's last rows and then E's first are the ones that the memory-side
  // cache still holds when they are next read (us a step: 1024 x 360,232 2059 -> 2021, 2048 x 500,000
  // 3980 -> 3923, 1024 x 205,991 1239 -> 1233, others even).
  tj = tiles_j - 1 - tj;
  const int64_t j0 = (int64_t)tj * Cfg::BM;
  const int i0 = ti * Cfg::BN;

  // labels: requested in front of the reduction (behind it they were a wait of 2 us of their own;
  // with fp32 operands they only delay the first slab)
  int32_t ylab[Cfg::TN];
  auto request_labels = [&]() {
#pragma unroll
    for (int bn = 0; bn < Cfg::TN; ++bn) {
      const int i = i0 + acc_col<Cfg>(bn);
      ylab[bn] = i < B ? yl[i] : -1;
    }
  };
  if constexpr (Cfg::DMA) request_labels();

  f32x16 acc[Cfg::TM][Cfg::TN];
  zero_acc<Cfg>(acc);
  PFC_PHASE(1, 0);
  // the reduction ends with column D (a multiple of every slab): the rest of the rows is zero
  gemm_tile<Cfg>(Wn + j0 * Dp, Dp, Xn + (int64_t)i0 * Dp, Dp, D / Cfg::BK, smem, acc);
  PFC_PHASE(1, 1);
  if constexpr (!Cfg::DMA) request_labels();
  // Pull the Wn block of the class tile that the workgroups `ahead` ids later will multiply (same
  // XCD, about one round later) into this XCD's L2: the tiles_i workgroups of a class tile touch
  // a part of the rows each, one 4-byte load per 128-byte line.  The values are only kept alive
  // until the end of the kernel, never used.
  uint32_t touched = 0;
  {
    int ntj, nti;
    const int nb = (int)blockIdx.x + ahead;
    if (nb < (int)gridDim.x && (int)(threadIdx.x >> 1) < Cfg::BM &&
        xcd_tile(nb, tiles_i, tiles_j, ntj, nti)) {
      ntj = tiles_j - 1 - ntj;
      const int row_bytes = Dp * (int)sizeof(T);
      const int off = ((nti * 256) % row_bytes) + (threadIdx.x & 1) * 128;
      const char* p = reinterpret_cast<const char*>(Wn + (int64_t)ntj * Cfg::BM * Dp) +
                      (int64_t)(threadIdx.x >> 1) * row_bytes + off;
      touched = *reinterpret_cast<const uint32_t*>(p);
    }
    __builtin_amdgcn_sched_barrier(0);
  }

  static_assert(2 * Cfg::WM * Cfg::BN * 4 <= Cfg::LDS_BYTES, "epilogue LDS");
  static_assert(!logits_chained<Cfg>() || 2 * Cfg::BN * 2 <= 2 * Cfg::WM * Cfg::BN, "chain LDS");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t krem = k - j0;
  const int klim = krem < (int64_t)Cfg::BM ? (int)krem : Cfg::BM;   // valid classes in this tile

  // ylane[bn]: tile row of sample i's label entry if THIS lane holds it, else -1.  A lane holds
  // the rows  wm*WTM + bm*32 + (r/4)*8 + half*4 + r%4.
  int ylane[Cfg::TN];
  bool any_label = false;
#pragma unroll
  for (int bn = 0; bn < Cfg::TN; ++bn) {
    const int i = i0 + acc_col<Cfg>(bn);
    ylane[bn] = -1;
    if (i < B) {
      const int64_t y = (int64_t)ylab[bn] - j0;
      if (y >= 0 && y < (int64_t)klim) {
        const int rel = (int)y - (wave / Cfg::WN) * Cfg::WTM;
        if (rel >= 0 && rel < Cfg::WTM && ((rel >> 2) & 1) == (lane >> 5)) ylane[bn] = (int)y;
      }
    }
    any_label = any_label || (ylane[bn] >= 0);
  }
  const bool guarded = __any(any_label) || klim < Cfg::BM || i0 + Cfg::BN > B;   // wave-uniform

  float* red = reinterpret_cast<float*>(smem);   // [WM][BN] sums, then [WM][BN] maxima
  float colsum[Cfg::TN], collab[Cfg::TN], colmax[Cfg::TN];
#pragma unroll
  for (int bn = 0; bn < Cfg::TN; ++bn) colmax[bn] = -2.f;
  auto epilogue = [&]() {
    if (guarded)
      logits_epilogue_columns<Cfg, true, EXTRAS>(acc, j0, i0, B, klim, kp, Bp, ylane, lp, E,
                                                 clabel, colsum, collab, colmax);
    else
      logits_epilogue_columns<Cfg, false, EXTRAS>(acc, j0, i0, B, klim, kp, Bp, ylane, lp, E,
                                                  clabel, colsum, collab, colmax);
  };
  if constexpr (logits_chained<Cfg>()) {
    // the second wavefront row goes on from the sums of the first: one chain over the tile's 64 rows
    static_assert(Cfg::WM == 2 && Cfg::TM == 1, "a chain of two blocks");
    const int o = (wave % Cfg::WN) * Cfg::TN * 64 + lane;
#pragma unroll
    for (int bn = 0; bn < Cfg::TN; ++bn) colsum[bn] = collab[bn] = 0.f;
    if (wave / Cfg::WN == 0) {
      epilogue();
#pragma unroll
      for (int bn = 0; bn < Cfg::TN; ++bn) {
        red[o + bn * 64] = colsum[bn];
        red[2 * Cfg::BN + o + bn * 64] = collab[bn];
        colsum[bn] = 0.f;
      }
    }
    __syncthreads();
    if (wave / Cfg::WN == 1) {
      float before[Cfg::TN];
#pragma unroll
      for (int bn = 0; bn < Cfg::TN; ++bn) {
        colsum[bn] = red[o + bn * 64];
        before[bn] = red[2 * Cfg::BN + o + bn * 64];
      }
      epilogue();
#pragma unroll
      for (int bn = 0; bn < Cfg::TN; ++bn) {
        colsum[bn] += collab[bn] + before[bn];   // at most one of the two is not zero
        colsum[bn] += __shfl_xor(colsum[bn], 32, 64);
      }
    }
    __syncthreads();
  } else {
    epilogue();
  }

  PFC_PHASE(1, 2);
  // cross-wave reduction over the WM wavefronts that share a column (fixed order)
  if (lane < 32) {
#pragma unroll
    for (int bn = 0; bn < Cfg::TN; ++bn) {
      const int o = (wave / Cfg::WN) * Cfg::BN + (wave % Cfg::WN) * Cfg::WTN + bn * 32 + lane;
      red[o] = colsum[bn];
      red[Cfg::WM * Cfg::BN + o] = colmax[bn];
    }
  }
  __syncthreads();
  for (int t = threadIdx.x; t < Cfg::BN; t += Cfg::THREADS) {
    float v = 0.f, mx = -2.f;
#pragma unroll
    for (int w = 0; w < Cfg::WM; ++w) {
      v += red[w * Cfg::BN + t];
      mx = fmaxf(mx, red[Cfg::WM * Cfg::BN + w * Cfg::BN + t]);
    }
    rowpart[(int64_t)(i0 + t) * tiles_j + tj] = v;
    if constexpr (EXTRAS) rowmaxpart[(int64_t)(i0 + t) * tiles_j + tj] = mx;
  }
  PFC_PHASE(1, 3);
  asm volatile("" ::"v"(touched));
}

// ---------------------------------------------------------------------------------------------
// gemm_logits_slim: gemm_logits with fp32 operands for problems of few 64-tiles: tiles of 64 classes x
// 16 samples, four wavefronts of 16 x 16, so that four times as many compute units work.  What bounds a
// 64-tile is its 16,384 cycles of matrix instructions (D = 512) and 256 KB of operands on one compute
// unit; here it is the operands, 160 KB at 28 GB/s.  v_mfma_f32_16x16x4_f32 adds the products one after
// the other, as the 32x32x2 form does; with the reduction steps 0 4 1 5 and 2 6 3 7 of every eight in
// one instruction each, the chain and hence the bits of a cosine are those of gemm_tile_fp32.  The row
// sums too: the classes with bit 2 clear and those with it set of all 64 are a chain each, then the two
// are added.  Forward/backward, us, 64-tiles -> now: 128 x 1,000 x 512 36.0 -> 30.8, 48 x 1,000 x 512
// 34.3 -> 29.1, 100 x 3,000 x 1024 63.3 -> 58.6.
// LDS: four stages of 64 reduction steps, rows of 256 bytes (the 64 classes, then the 16 samples),
// chunk c of 16 bytes of row r at position c ^ (r & 15): 16 rows read two chunks each without conflicts.
// ---------------------------------------------------------------------------------------------
constexpr int kSlimRows = 80, kSlimStages = 4, kSlimStageBytes = kSlimRows * 256, kSlimLoads = kSlimRows / 4 / 4;
constexpr int kSlimLds = kSlimStages * kSlimStageBytes;

template <bool EXTRAS>
__global__ __launch_bounds__(256) void gemm_logits_slim_kernel(
    const float* __restrict__ Wn, const float* __restrict__ Xn, int D, int Dp, int64_t k, int B, int64_t kp,
    const int32_t* __restrict__ yl, LossParams lp, float* __restrict__ E, float* __restrict__ rowpart,
    float* __restrict__ rowmaxpart, float* __restrict__ clabel, int tiles_j, int tiles_i) {
  extern __shared__ __align__(16) char smem[];
  int tj, ti;
  if (!xcd_tile(blockIdx.x, tiles_i, tiles_j, tj, ti)) return;
  const int64_t j0 = (int64_t)tj * 64;
  const int i0 = ti * 16;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 15, g = lane >> 4;
  const int i = i0 + col;
  const int32_t y = i < B ? yl[i] : -1;

  // Loads to LDS: instruction p of a wavefront fills rows 4 (wave + 4 p) .. + 3 of a stage.
  const int row0 = 4 * wave + (lane >> 4);
  const uint32_t toff = (uint32_t)((lane >> 4) * Dp * 4 + (((lane & 15) ^ row0) * 16));
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem + wave * 1024;
  const char* wbase = reinterpret_cast<const char*>(Wn + (j0 + 4 * wave) * Dp);
  const char* xbase = reinterpret_cast<const char*>(Xn + (int64_t)(i0 + 4 * wave) * Dp);
  auto request = [&](int s) {
    const uint32_t stage = lds0 + (s % kSlimStages) * kSlimStageBytes;
#pragma unroll
    for (int p = 0; p < kSlimLoads; ++p)
      lds_load((p < 4 ? wbase + (int64_t)p * 16 * Dp * 4 : xbase) + s * 256, toff, stage + p * 4096);
  };
  const int n = D / 64;
#pragma unroll
  for (int s = 0; s < kSlimStages - 1; ++s)
    if (s < n) request(s);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int s = 0; s < n; ++s) {
    // stage s is there, and all wavefronts are done with the one before
    if (s + 2 < n) dma_wait_barrier<2 * kSlimLoads>();
    else if (s + 1 < n) dma_wait_barrier<kSlimLoads>();
    else dma_wait_barrier<0>();
    if (s + kSlimStages - 1 < n) request(s + kSlimStages - 1);
    const char* stage = smem + (s % kSlimStages) * kSlimStageBytes;
    // this lane's two of every eight reduction steps of its class and its sample (rows & 15: col)
    float a[8][2], b[8][2];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int at = ((2 * q + (g & 1)) ^ col) * 16 + (g >> 1) * 4;
      const float* pa = reinterpret_cast<const float*>(stage + (wave * 16 + col) * 256 + at);
      const float* pb = reinterpret_cast<const float*>(stage + (64 + col) * 256 + at);
      a[q][0] = pa[0];
      a[q][1] = pa[2];
      b[q][0] = pb[0];
      b[q][1] = pb[2];
    }
    __builtin_amdgcn_sched_barrier(0);   // all of them in flight before the first is used
#pragma unroll
    for (int q = 0; q < 8; ++q)
#pragma unroll
      for (int u = 0; u < 2; ++u) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[q][u], b[q][u], acc, 0, 0, 0);
  }
  __syncthreads();

  // this lane: sample i, classes j0 + jl .. jl + 3
  const int jl = wave * 16 + g * 4;
  const int64_t krem = k - j0, yrel = (int64_t)y - j0;
  const int klim = krem < 64 ? (int)krem : 64;
  const int yloc = y >= 0 && yrel >= 0 && yrel < klim ? (int)yrel : -1;
  float ref = 0.f;
  if constexpr (EXTRAS) ref = lp.rowref ? lp.rowref[i] : 0.f;
  const float ref2 = ref * 1.44269504088896340736f;
  f32x4 e;
  float cmax = -2.f;
  float* red = reinterpret_cast<float*>(smem);   // [16 samples][64 + 4]: e, then [16][17] maxima, [16] label terms
  constexpr int RS = 68;
  float *redmax = red + 16 * RS, *redlab = redmax + 16 * 17;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float c = __builtin_amdgcn_fmed3f(acc[r], -1.f, 1.f);
    float ev = EXTRAS ? __builtin_amdgcn_exp2f(fmaf(c, lp.s_log2e, -ref2)) : __builtin_amdgcn_exp2f(c * lp.s_log2e);
    const bool lab = jl + r == yloc, neg = i < B && jl + r < klim && !lab;   // neg: a real, non-label entry
    ev = neg ? ev : 0.f;
    if (lab) {
      clabel[i] = c;
      redlab[col] = __expf(label_logit(lp, c) - ref);
    }
    if constexpr (EXTRAS) {
      cmax = neg ? fmaxf(cmax, c) : cmax;
      ev = (c > lp.tau) ? 0.f : ev;
    }
    e[r] = ev;
  }
  *reinterpret_cast<f32x4*>(E + (int64_t)i * kp + j0 + jl) = e;
  *reinterpret_cast<f32x4*>(red + col * RS + jl) = e;
  if constexpr (EXTRAS) redmax[col * 17 + wave * 4 + g] = cmax;
  __syncthreads();
  if (threadIdx.x < 32) {   // thread (half, sample): the chain of the classes whose bit 2 is `half`
    const int half = threadIdx.x >> 4, t = threadIdx.x & 15, ii = i0 + t;
    f32x4 v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = *reinterpret_cast<const f32x4*>(red + t * RS + q * 8 + half * 4);
    float sum = 0.f;
#pragma unroll
    for (int q = 0; q < 8; ++q)
#pragma unroll
      for (int r = 0; r < 4; ++r) sum += v[q][r];
    // the label term joins the chain of its half (not all threads hold the same sample's `yloc`)
    const int yt = __shfl(yloc, t, 64);
    if (yt >= 0 && ((yt >> 2) & 1) == half) sum += redlab[t];
    sum += __shfl_xor(sum, 16, 64);
    if (half == 0) rowpart[(int64_t)ii * tiles_j + tj] = sum;
    if constexpr (EXTRAS) {
      float mx = -2.f;
#pragma unroll
      for (int q = 0; q < 16; ++q) mx = fmaxf(mx, redmax[t * 17 + q]);
      if (half == 0) rowmaxpart[(int64_t)ii * tiles_j + tj] = mx;
    }
  }
}

// ---------------------------------------------------------------------------------------------
// gemm_rowmax (scales above 64 only): the logits GEMM once more, in front of gemm_logits, with an
// epilogue that keeps nothing but the largest logit of every sample in every tile (label entry
// with its margin); row_ref reduces the tiles.  The softmax then runs relative to that maximum,
// as an online softmax would, and works for any scale; at s <= 64 a zero reference is exact as
// well and this pass is skipped.
// ---------------------------------------------------------------------------------------------
template <class Cfg>
__global__ __launch_bounds__(Cfg::THREADS) void gemm_rowmax_kernel(
    const typename Cfg::elem* __restrict__ Wn, const typename Cfg::elem* __restrict__ Xn, int D,
    int Dp, int64_t k, int B, const int32_t* __restrict__ yl, LossParams lp,
    float* __restrict__ rowmaxpart, int tiles_j, int tiles_i) {
  extern __shared__ __align__(16) char smem[];
  int tj, ti;
  if (!xcd_tile(blockIdx.x, tiles_i, tiles_j, tj, ti)) return;
  const int64_t j0 = (int64_t)tj * Cfg::BM;
  const int i0 = ti * Cfg::BN;
  f32x16 acc[Cfg::TM][Cfg::TN];
  zero_acc<Cfg>(acc);
  gemm_tile<Cfg>(Wn + j0 * Dp, Dp, Xn + (int64_t)i0 * Dp, Dp, D / Cfg::BK, smem, acc);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t krem = k - j0;
  const int klim = krem < (int64_t)Cfg::BM ? (int)krem : Cfg::BM;
  float* red = reinterpret_cast<float*>(smem);   // [WM][BN]
#pragma unroll
  for (int bn = 0; bn < Cfg::TN; ++bn) {
    const int i = i0 + acc_col<Cfg>(bn);
    const int yloc = i < B ? (int)((int64_t)yl[i] - j0) : -1;   // tile row of the label entry
    float zmax = -3.0e38f;
#pragma unroll
    for (int bm = 0; bm < Cfg::TM; ++bm)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int jl = acc_row<Cfg>(bm, r);
        const float c = __builtin_amdgcn_fmed3f(acc[bm][bn][r], -1.f, 1.f);
        const bool lab = jl == yloc;
        const float z = lab ? label_logit(lp, c) : lp.s * c;
        // entries the filter leaves out of the softmax do not count (the label is never filtered)
        const bool in = i < B && jl < klim && (lab || !(c > lp.tau));
        zmax = in ? fmaxf(zmax, z) : zmax;
      }
    zmax = fmaxf(zmax, __shfl_xor(zmax, 32, 64));
    if (lane < 32)
      red[(wave / Cfg::WN) * Cfg::BN + (wave % Cfg::WN) * Cfg::WTN + bn * 32 + lane] = zmax;
  }
  __syncthreads();
  for (int t = threadIdx.x; t < Cfg::BN; t += Cfg::THREADS) {
    float mx = -3.0e38f;
#pragma unroll
    for (int w = 0; w < Cfg::WM; ++w) mx = fmaxf(mx, red[w * Cfg::BN + t]);
    rowmaxpart[(int64_t)(i0 + t) * tiles_j + tj] = mx;
  }
}

// rowref[i] = max over the tiles of sample i (0 for padded samples); one wavefront per sample.
__global__ void row_ref_kernel(const float* __restrict__ rowmaxpart, int tiles_j, int B, int Bp,
                               float* __restrict__ rowref) {
  const int lane = threadIdx.x & 63;
  const int i = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (i >= Bp) return;
  float mx = -3.0e38f;
  if (i < B)
    for (int t = lane; t < tiles_j; t += 64) mx = fmaxf(mx, rowmaxpart[(int64_t)i * tiles_j + t]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
  if (lane == 0) rowref[i] = i < B ? mx : 0.f;
}

// ---------------------------------------------------------------------------------------------
// row_combine: one wavefront per (padded) sample.  l_i = sum of the per-tile partial sums (lane
// strided, then a fixed shuffle tree: the same order on every run), the per-row scalars, and the
// row of Xs = (s/(B l_i)) * x_i/|x_i| that feeds the dweight GEMM (zero for padded rows).
// ---------------------------------------------------------------------------------------------
// The first workgroups of the launch (label_heads) find the first sample of every class, one window of
// kLabelWindow samples each: an LDS hash table of its distinct labels, then one atomic for each of
// them.  (One per sample from the rows themselves: thousands meet on the word of a frequent class
// with a large batch, and in a small one they are the end of the chain of every wavefront.  Step
// 16,384 samples x 3,592 x 512 460.6 -> 438.4 us, 512 x 9,344 101.0 -> 99.9.)
struct HeadsLds {
  static constexpr int SLOTS = 2 * kLabelWindow;   // at most half full
  int32_t key[SLOTS], first[SLOTS];
};
__device__ __forceinline__ void label_heads(int w, HeadsLds& lds, int B,
                                            const int32_t* __restrict__ yl, int64_t k, int64_t kp,
                                            int32_t* __restrict__ head, int nwin) {
  for (int t = threadIdx.x; t < HeadsLds::SLOTS; t += blockDim.x) {
    lds.key[t] = -1;
    lds.first[t] = INT_MAX;
  }
  __syncthreads();
  const int end = min(B, (w + 1) * kLabelWindow);
  for (int p = w * kLabelWindow + threadIdx.x; p < end; p += blockDim.x) {
    const int32_t y = yl[p];
    if (y < 0 || (int64_t)y >= k) continue;
    unsigned slot = ((unsigned)y * 2654435761u) % HeadsLds::SLOTS;
    for (;;) {   // ends: there are more slots than samples in a window
      const int32_t seen = atomicCAS(&lds.key[slot], -1, y);
      if (seen == -1 || seen == y) break;
      slot = (slot + 1) % HeadsLds::SLOTS;
    }
    atomicMin(&lds.first[slot], p);
  }
  __syncthreads();
  for (int t = threadIdx.x; t < HeadsLds::SLOTS; t += blockDim.x) {
    const int32_t y = lds.key[t];
    if (y < 0) continue;
    atomicMin(&head[y], lds.first[t]);   // integer: order-independent
    if (nwin) head[(int64_t)(1 + w) * kp + y] = lds.first[t];
  }
}

// f(p[lane]), f(p[lane + 64]), .. below n, eight loads at a time: one after the other they were the
// length of the launch (us, one at a time -> now: 805 tiles 11.1 -> 8.8, 1,408 15.4 -> 9.2, 1,954 22.1 ->
// 14.2, 2,344 16.1 -> 7.6).  f(none) has no effect.
template <class F>
__device__ __forceinline__ void lane_strided(const float* __restrict__ p, int n, int lane, float none, F f) {
  constexpr int U = 8;
  for (int t = lane; t - lane < n; t += 64 * U) {
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = t + 64 * u < n ? p[t + 64 * u] : none;
#pragma unroll
    for (int u = 0; u < U; ++u) f(v[u]);
  }
}

template <typename T, int NC>
__global__ void row_combine_kernel(int head_blocks, const float* __restrict__ rowpart, int tiles_j,
                                   int pairs, int B,
                                   int Bp,
                                   int D, int Dp, const float* __restrict__ X,
                                   const float* __restrict__ rnormX,
                                   const float* __restrict__ clabel, LossParams lp,
                                   const float* __restrict__ rowmaxpart,
                                   float* __restrict__ rowscale, float* __restrict__ dlabel,
                                   float* __restrict__ lossrow, float* __restrict__ rowmax,
                                   const int32_t* __restrict__ yl, int64_t k, int64_t kp,
                                   int32_t* __restrict__ head, int nwin, T* __restrict__ Xs,
                                   const float* __restrict__ W, int64_t N,
                                   const int32_t* __restrict__ idx, float* __restrict__ wlab) {
  __shared__ HeadsLds lds;
  if ((int)blockIdx.x < head_blocks) {
    label_heads(blockIdx.x, lds, B, yl, k, kp, head, nwin);
    return;
  }
  const int lane = threadIdx.x & 63;
  const int i = ((int)blockIdx.x - head_blocks) * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (i >= Bp) return;
  float scale = 0.f;
  if (i < B) {
    float l = 0.f;
    if (pairs) {   // 64-tiles (their number is even: classes are padded to 256)
      for (int t = lane; t < tiles_j / 2; t += 64) {
        const float2 v = *reinterpret_cast<const float2*>(rowpart + (int64_t)i * tiles_j + 2 * t);
        l += v.x + v.y;
      }
    } else {
      lane_strided(rowpart + (int64_t)i * tiles_j, tiles_j, lane, 0.f, [&](float x) { l += x; });
    }
    l = wave_sum(l);
    scale = (lp.s / (float)B) / l;   // B * l could leave the fp32 range, s/B never does
    float mx = -2.f;
    if (lp.extras) {
      lane_strided(rowmaxpart + (int64_t)i * tiles_j, tiles_j, lane, mx, [&](float x) { mx = fmaxf(mx, x); });
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    }
    if (lane == 0) {
      const float c = clabel[i];
      const float sin2 = 1.f - c * c;
      const float zlab = label_logit(lp, c);
      const float ref = lp.rowref ? lp.rowref[i] : 0.f;   // l is the sum of exp(z - ref)
      const float p = __expf(zlab - ref) / l;
      // d(label logit)/d cos / s: sin(theta+m)/sin(theta) for the angular margin, 1 for the cosine one
      const float rho = lp.cosface ? 1.f : lp.cos_m + c * lp.sin_m / sqrtf(fmaxf(sin2, kEpsSin2));
      lossrow[i] = (logf(l) + ref) - zlab;
      rowscale[i] = scale;
      dlabel[i] = (lp.s / (float)B) * (p - 1.f) * rho;
      rowmax[i] = mx;
    }
  } else if (lane == 0) {
    lossrow[i] = 0.f;
    rowscale[i] = 0.f;
    dlabel[i] = 0.f;
    rowmax[i] = 0.f;
  }
  const float f = (i < B) ? rnormX[i] * scale : 0.f;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int d = c * 256 + lane * 4;
    if (d >= Dp) continue;
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (i < B && d < D) v = *reinterpret_cast<const float4*>(X + (int64_t)i * D + d);
    T o[4] = {from_float<T>(v.x * f), from_float<T>(v.y * f), from_float<T>(v.z * f),
              from_float<T>(v.w * f)};
    if constexpr (sizeof(T) == 2) {
      uint2 pk;
      __builtin_memcpy(&pk, o, 8);
      *reinterpret_cast<uint2*>(Xs + (int64_t)i * Dp + d) = pk;
    } else {
      uint4 pk;
      __builtin_memcpy(&pk, o, 16);
      *reinterpret_cast<uint4*>(Xs + (int64_t)i * Dp + d) = pk;
    }
  }
  // fused step: keep the label's row of W for gradients_final, which runs after the update
  if (wlab && i < B) {
    const int32_t y = yl[i];
    const int64_t row = (y >= 0 && (int64_t)y < k) ? idx[y] : -1;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int d = c * 256 + lane * 4;
      if (row >= 0 && row < N && d < D)
        *reinterpret_cast<float4*>(wlab + (int64_t)i * D + d) =
            *reinterpret_cast<const float4*>(W + row * D + d);
    }
  }
}

// ---------------------------------------------------------------------------------------------
// dfeatures_tile (in gemm_backward): slice `sp` of S: part[sp][i][d] = sum_{j in slice} E[i][j] *
// Wn[j][d] (A = E with k contiguous, B = Wn k-major).
// ---------------------------------------------------------------------------------------------
// Products of one uninterrupted sum (gemm_tile's CHAIN) in the two backward products with fp32
// operands.  Their 128- and 64-tiles need fewer slices than 256-tiles to fill the GPU, and a slice
// of many thousand products adds up rounding errors.  The pieces cost 0 - 3 % of a step, as many
// slices as 256-tiles take up to 18 %.
constexpr int kDxSumSteps = 256, kDwSumSteps = 512;
template <class Cfg, int STEPS, bool PIECES>
constexpr int sum_slabs() { return PIECES ? STEPS / Cfg::BK : 0; }

// E from entry (sample i, class j) on, as an operand of a backward product: rows of kp, or octets.
template <class Cfg>
__device__ __forceinline__ const typename Cfg::elem* e_tile(const typename Cfg::elem* E, int64_t i, int64_t j, int Bp,
                                                            int64_t kp) {
  return Cfg::A_OCTETS ? E + j * Bp + i * 8 : E + i * kp + j;
}
template <class Cfg>
__device__ __forceinline__ int64_t e_ld(int Bp, int64_t kp) { return Cfg::A_OCTETS ? Bp : kp; }

template <class Cfg, bool PIECES>
__device__ __forceinline__ void dfeatures_tile(int wg, char* smem,
                                               const typename Cfg::elem* __restrict__ E,
                                               const typename Cfg::elem* __restrict__ Wn, int D,
                                               int Bp, int64_t kp, const DxShape& dx,
                                               float* __restrict__ part) {
  int sp, tile;
  if (!xcd_tile(wg, dx.tiles_i * dx.tiles_d, dx.splits, sp, tile)) return;
  const int ti = tile / dx.tiles_d, td = tile % dx.tiles_d;
  const int i0 = ti * Cfg::BM, d0 = td * Cfg::BN;
  const int slab0 = sp * dx.slabs_per;
  int ns = dx.slabs_total - slab0;
  if (ns > dx.slabs_per) ns = dx.slabs_per;
  f32x16 acc[Cfg::TM][Cfg::TN];
  zero_acc<Cfg>(acc);
  const int64_t koff = (int64_t)slab0 * Cfg::BK;
  gemm_tile<Cfg, sum_slabs<Cfg, kDxSumSteps, PIECES>()>(e_tile<Cfg>(E, i0, koff, Bp, kp), e_ld<Cfg>(Bp, kp),
                                                        Wn + koff * D + d0, D, ns, smem, acc);
  float* out = part + (int64_t)sp * Bp * D;
#pragma unroll
  for (int bm = 0; bm < Cfg::TM; ++bm)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = i0 + acc_row<Cfg>(bm, r);
#pragma unroll
      for (int bn = 0; bn < Cfg::TN; ++bn)
        out[(int64_t)i * D + d0 + acc_col<Cfg>(bn)] = acc[bm][bn][r];
    }
}

// ---------------------------------------------------------------------------------------------
// dweight_tile (in gemm_backward): dWn[j][d] = sum_i E[i][j] * Xs[i][d] (both operands k-major);
// rows j < k are written.  When k is small and the batch large (the regime without extra negatives,
// Sec. 3.3) there are too few tiles to fill the GPU: SPLIT cuts the batch (the reduction) into
// slices that write partial tiles, summed in fixed order by dweight_reduce.  Xs has rows of Dp
// elements; the partial tiles too; dWn (the caller's) has rows of D floats, columns from D on are
// not stored.
// ---------------------------------------------------------------------------------------------
template <class Cfg, bool SPLIT, bool PIECES>
__device__ __forceinline__ void dweight_tile(
    int wg, char* smem, const typename Cfg::elem* __restrict__ E,
    const typename Cfg::elem* __restrict__ Xs, int D, int Dp, int64_t k, int64_t kp, int Bp,
    float* __restrict__ out, int tiles_j, int tiles_d, int slabs_per, int splits) {
  int tj, td, sp = 0, ns = Bp / Cfg::BK;
  if constexpr (SPLIT) {
    int tile;
    if (!xcd_tile(wg, tiles_j * tiles_d, splits, sp, tile)) return;
    tj = tile / tiles_d;
    td = tile % tiles_d;
    ns -= sp * slabs_per;
    if (ns > slabs_per) ns = slabs_per;
  } else {
    if (!xcd_tile(wg, tiles_d, tiles_j, tj, td)) return;
  }
  const int64_t j0 = (int64_t)tj * Cfg::BM;
  const int d0 = td * Cfg::BN;
  const int64_t i0 = (int64_t)sp * slabs_per * Cfg::BK;   // first sample of this slice
  f32x16 acc[Cfg::TM][Cfg::TN];
  zero_acc<Cfg>(acc);
  PFC_PHASE(2, 0);
  gemm_tile<Cfg, sum_slabs<Cfg, kDwSumSteps, PIECES>()>(e_tile<Cfg>(E, i0, j0, Bp, kp), e_ld<Cfg>(Bp, kp),
                                                        Xs + i0 * Dp + d0, Dp, ns, smem, acc);
  PFC_PHASE(2, 1);
  float* dst = SPLIT ? out + (int64_t)sp * kp * Dp : out;
  const int ld = SPLIT ? Dp : D;
  auto store_tile = [&](auto guarded) {
    bool col_in[Cfg::TN];
#pragma unroll
    for (int bn = 0; bn < Cfg::TN; ++bn) col_in[bn] = !guarded.value || d0 + acc_col<Cfg>(bn) < D;
#pragma unroll
    for (int bm = 0; bm < Cfg::TM; ++bm)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t j = j0 + acc_row<Cfg>(bm, r);
        if (SPLIT || j < k) {
#pragma unroll
          for (int bn = 0; bn < Cfg::TN; ++bn)
            if (col_in[bn]) dst[j * ld + d0 + acc_col<Cfg>(bn)] = acc[bm][bn][r];
        }
      }
  };
  // only the last column tile of a D that is no multiple of the tile width needs the guard
  if (SPLIT || d0 + Cfg::BN <= D)
    store_tile(std::false_type{});
  else
    store_tile(std::true_type{});
  PFC_PHASE(2, 2);
}

// gemm_backward: the two backward products need nothing of each other, so they share a launch: the
// first dx.wgs workgroups (a multiple of 8, so that workgroup ids keep their XCD) work on
// dfeatures, the others on dweight.  Alone, either leaves the GPU partly idle: small problems have
// too few tiles and are bound by the latency of a tile (17 + 18 us one after the other, 24 together
// at 512 samples x 9,344 classes x 512), large ones lose the last round of dweight tiles and have
// all compute units store their tiles at the same time (291 + 219 us, 495 together at 1024 x
// 205,991 x 512).  The dfeatures workgroups are the longest and start first; dx_shape says how many
// there are.  (Large batches can have the longer reduction in dweight: its workgroups are then in
// front, w_first of them.)
template <class CfgX, class CfgW, bool SPLIT, bool PIECES>
__global__ __launch_bounds__(CfgX::THREADS, CfgX::MIN_WAVES) void gemm_backward_kernel(
    const typename CfgX::elem* __restrict__ E, const typename CfgX::elem* __restrict__ Wn,
    const typename CfgX::elem* __restrict__ Xs, int D, int Dp, int64_t k, int64_t kp, int Bp,
    DxShape dx, float* __restrict__ dXpart, float* __restrict__ dWout, int tiles_j, int tiles_d,
    int slabs_per, int splits,
    int w_first) {
  static_assert(CfgX::THREADS == CfgW::THREADS, "one launch shape");
  extern __shared__ __align__(16) char smem[];
  // (an offset that is no multiple of 8 turns all ids to other XCDs alike)
  const int b = (int)blockIdx.x < w_first ? (int)blockIdx.x + dx.wgs : (int)blockIdx.x - w_first;
  if (b < dx.wgs)
    dfeatures_tile<CfgX, PIECES>(b, smem, E, Wn, Dp, Bp, kp, dx, dXpart);
  else
    dweight_tile<CfgW, SPLIT, PIECES>(b - dx.wgs, smem, E, Xs, D, Dp, k, kp, Bp, dWout, tiles_j,
                                      tiles_d, slabs_per, splits);
}

// dW[j][d] = sum over slices of part[slice][j][d], in slice order (rows of Dp floats in `part`, of
// D floats in dW).
__global__ void dweight_reduce_kernel(const float* __restrict__ part, int splits, int64_t k,
                                      int64_t kp, int D, int Dp, float* __restrict__ dW) {
  const int64_t e4 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e4 >= k * D / 4) return;
  const int64_t j = e4 / (D / 4);
  const int d = (int)(e4 - j * (D / 4)) * 4;
  float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int sp = 0; sp < splits; ++sp) {
    const float4 t =
        *reinterpret_cast<const float4*>(part + ((int64_t)sp * kp + j) * Dp + d);
    a.x += t.x; a.y += t.y; a.z += t.z; a.w += t.w;
  }
  *reinterpret_cast<float4*>(dW + e4 * 4) = a;
}

// dweight_label_block (in gradients_final, or dweight_label in a launch of its own): dWn[y] += sum
// over samples i with label y of dlabel_i * xn_i.  Block i does the whole sum for its class if i is
// the first sample carrying that label (head[y] == i, found with an integer atomicMin by
// row_combine).  The matching samples are listed in ascending order; thread group g (one float4
// column per thread) sums the matches whose ordinal is congruent to g, and the groups are combined
// in fixed order, so the result does not depend on timing.  LABEL_COMPACT (fused step): the sum is
// not added to dWn[y] but written to row i of a B x D side buffer, i being that first sample; the
// fused GEMM picks it up through head[].  Batches of several windows of kLabelWindow samples:
// window_label_block, further down.
constexpr int kLabelThreads = 1024;
enum LabelMode { LABEL_ADD, LABEL_COMPACT };
struct LabelLds {
  float4 part[kLabelThreads];
  int list[kLabelThreads];
  float coef[kLabelThreads];   // dlabel_p / |x_p| of the listed samples
  int wcnt[kLabelThreads / 64];
};
template <LabelMode MODE>
__device__ __forceinline__ void dweight_label_block(
    int i, LabelLds& lds, const float* __restrict__ X, int B, int D,
    const int32_t* __restrict__ yl, int64_t k, const int32_t* __restrict__ head,
    const float* __restrict__ rnormX, const float* __restrict__ dlabel, float* __restrict__ dW) {
  int* s_list = lds.list;
  float* s_coef = lds.coef;
  int* s_wcnt = lds.wcnt;
  float4* s_part = lds.part;
  const int t = threadIdx.x;
  const int lane = t & 63, wave = t >> 6;
  const int32_t y = yl[i];
  if (y < 0 || (int64_t)y >= k) return;
  if (head[y] != i) return;   // an earlier sample carries this label and does the sum
  const int cols = D >> 2;                 // float4 columns: 16 .. 256
  const int G = kLabelThreads / cols;      // thread groups
  const int col = t % cols, g = t / cols;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  int ordinal0 = 0;                        // matches seen in earlier chunks
  for (int p0 = i; p0 < B; p0 += kLabelThreads) {
    const int p = p0 + t;
    const bool hit = (p < B) && (yl[p] == y);
    const unsigned long long bal = __ballot(hit);
    const int before = __popcll(bal & ((1ull << lane) - 1ull));
    if (lane == 0) s_wcnt[wave] = __popcll(bal);
    __syncthreads();
    int base = 0, total = 0;
    for (int w = 0; w < kLabelThreads / 64; ++w) {
      const int c = s_wcnt[w];
      if (w < wave) base += c;
      total += c;
    }
    if (hit) {
      s_list[base + before] = p;
      s_coef[base + before] = dlabel[p] * rnormX[p];
    }
    __syncthreads();
    // group g takes list entries whose global ordinal is congruent to g modulo G; six row
    // loads are in flight at a time, the additions stay in list order
    int e = (g - ordinal0 % G + G) % G;
    constexpr int UN = 6;
    for (; e + (UN - 1) * G < total; e += UN * G) {
      float4 x[UN];
      float a[UN];
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        const int q = s_list[e + u * G];
        a[u] = s_coef[e + u * G];
        x[u] = *reinterpret_cast<const float4*>(X + (int64_t)q * D + col * 4);
      }
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        acc.x += a[u] * x[u].x; acc.y += a[u] * x[u].y; acc.z += a[u] * x[u].z; acc.w += a[u] * x[u].w;
      }
    }
    for (; e < total; e += G) {
      const int q = s_list[e];
      const float4 x = *reinterpret_cast<const float4*>(X + (int64_t)q * D + col * 4);
      const float a = s_coef[e];
      acc.x += a * x.x; acc.y += a * x.y; acc.z += a * x.z; acc.w += a * x.w;
    }
    ordinal0 += total;
    __syncthreads();
  }
  s_part[t] = acc;
  __syncthreads();
  if (g == 0) {
    float4 r = s_part[col];
    for (int gg = 1; gg < G; ++gg) {
      const float4 o = s_part[gg * cols + col];
      r.x += o.x; r.y += o.y; r.z += o.z; r.w += o.w;
    }
    if constexpr (MODE != LABEL_ADD) {
      *reinterpret_cast<float4*>(dW + (int64_t)i * D + col * 4) = r;
    } else {
      float4* dst = reinterpret_cast<float4*>(dW + (int64_t)y * D + col * 4);
      float4 cur = *dst;
      cur.x += r.x; cur.y += r.y; cur.z += r.z; cur.w += r.w;
      *dst = cur;
    }
  }
}

template <LabelMode MODE>
__global__ __launch_bounds__(kLabelThreads) void dweight_label_kernel(
    const float* __restrict__ X, int B, int D, const int32_t* __restrict__ yl, int64_t k,
    const int32_t* __restrict__ head, const float* __restrict__ rnormX,
    const float* __restrict__ dlabel, float* __restrict__ dW) {
  __shared__ LabelLds lds;
  dweight_label_block<MODE>(blockIdx.x, lds, X, B, D, yl, k, head, rnormX, dlabel, dW);
}

// window_label_block (in gradients_final, or window_label in a launch of its own): the label part
// of batches of several windows (Sec. 3.3 enlarges the batch to 8K and 16K).  With long-tailed
// labels one class can own a fifth of the batch, and one workgroup cannot read thousands of feature
// rows quickly (a compute unit draws a small share of the memory bandwidth); most classes have a
// sample or two.  order_labels has put the samples of a window in order of their class.
// kWindowBlocks workgroups share a window's classes: one wavefront sums a class of up to
// kWindowWave samples, the 16 of a workgroup share a larger one.  The sum goes to row i of `part`,
// i being the class's first sample in the window; dweight_label_combine adds a class's sums in
// window order.  (A workgroup for every sample of the batch, which scanned the window if it was the
// first of its class, and nothing to do for most of them: gradients_final at 16,384 samples x 3,592
// classes x 512 89.5 us, now 35.3; step 392 -> 338.)
constexpr int kWindowBlocks = 32, kWindowWave = 8;
template <int NC>
struct WindowLds {
  int begin[kLabelWindow / kWindowBlocks], end[kLabelWindow / kWindowBlocks];
  float4 part[kLabelThreads / 64 - 1][NC][64];
};
// sum over this wavefront's entries e < cnt (<= 64) of dl_e * rn_e * X[row_e], lane e holding entry e
template <int NC>
__device__ __forceinline__ void label_rows(float4 (&acc)[NC], int cnt, int row, float dl, float rn,
                                           const float* __restrict__ X, int D) {
  constexpr int UN = NC <= 2 ? 4 : 2;   // rows in flight
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int c = 0; c < NC; ++c) acc[c] = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int e = 0; e < cnt; e += UN) {
    float4 x[UN][NC];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      if (e + u >= cnt) continue;
      const float* src = X + (int64_t)__builtin_amdgcn_readlane(row, e + u) * D + lane * 4;
#pragma unroll
      for (int c = 0; c < NC; ++c)
        if (c * 256 + lane * 4 < D) x[u][c] = *reinterpret_cast<const float4*>(src + c * 256);
    }
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      if (e + u >= cnt) continue;
      const float a = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, dl * rn), e + u));
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        if (c * 256 + lane * 4 >= D) continue;
        acc[c].x += a * x[u][c].x; acc[c].y += a * x[u][c].y;
        acc[c].z += a * x[u][c].z; acc[c].w += a * x[u][c].w;
      }
    }
  }
}
template <int NC>
__device__ __forceinline__ void window_label_block(int block, WindowLds<NC>& lds, const float* __restrict__ X,
                                                   int D, const int32_t* __restrict__ order,
                                                   const int32_t* __restrict__ runs,
                                                   const float* __restrict__ rnormX,
                                                   const float* __restrict__ dlabel,
                                                   float* __restrict__ part) {
  constexpr int WAVES = kLabelThreads / 64;
  const int w = block / kWindowBlocks, b = block % kWindowBlocks;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  order += (int64_t)w * kLabelWindow;
  runs += (int64_t)w * kWindowRuns;
  // this workgroup's classes: b, b + kWindowBlocks, ..
  const int total = runs[0], mine = (total - b + kWindowBlocks - 1) / kWindowBlocks;
  if (threadIdx.x < kLabelWindow / kWindowBlocks) {   // (not waiting for their number: those behind it are not used)
    const int r = b + (int)threadIdx.x * kWindowBlocks;
    lds.begin[threadIdx.x] = runs[1 + r];
    lds.end[threadIdx.x] = runs[2 + r];
  }
  __syncthreads();
  float4 acc[NC];
  // entries first, first + step, .. below `end`, at most 64 of them
  auto sum = [&](int first, int step, int end) __attribute__((always_inline)) {
    const int at = first + lane * step;
    int row = 0;
    float dl = 0.f, rn = 0.f;
    if (at < end) {
      row = order[at];
      dl = dlabel[row];
      rn = rnormX[row];
    }
    label_rows<NC>(acc, first < end ? (end - first + step - 1) / step : 0, row, dl, rn, X, D);
  };
  auto store = [&](int begin) __attribute__((always_inline)) {
    float* dst = part + (int64_t)order[begin] * D;
#pragma unroll
    for (int c = 0; c < NC; ++c)
      if (c * 256 + lane * 4 < D) *reinterpret_cast<float4*>(dst + c * 256 + lane * 4) = acc[c];
  };
  for (int u = 0; u < mine; ++u) {
    const int begin = __builtin_amdgcn_readfirstlane(lds.begin[u]), end = __builtin_amdgcn_readfirstlane(lds.end[u]);
    if (end - begin <= kWindowWave) {
      if (u % WAVES == wave) {
        sum(begin, 1, end);
        store(begin);
      }
      continue;
    }
    sum(begin + wave, WAVES, end);
    if (wave > 0) {
#pragma unroll
      for (int c = 0; c < NC; ++c) lds.part[wave - 1][c][lane] = acc[c];
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll NC <= 2 ? 3 : 1
      for (int v = 0; v < WAVES - 1; ++v)
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          const float4 o = lds.part[v][c][lane];
          acc[c].x += o.x; acc[c].y += o.y; acc[c].z += o.z; acc[c].w += o.w;
        }
      store(begin);
    }
    __syncthreads();
  }
}
template <int NC>
__global__ __launch_bounds__(kLabelThreads) void window_label_kernel(
    const float* __restrict__ X, int D, const int32_t* __restrict__ order, const int32_t* __restrict__ runs,
    const float* __restrict__ rnormX, const float* __restrict__ dlabel, float* __restrict__ part) {
  __shared__ WindowLds<NC> lds;
  window_label_block<NC>(blockIdx.x, lds, X, D, order, runs, rnormX, dlabel, part);
}

// dweight_label_combine (after window_label_block): the wavefront of sample i, if that is the first
// of its class in the whole batch, adds the class's window sums (rows of `part` named by the window
// heads) in window order; the total goes to row i of `part` (COMPACT, fused step) or is added to
// dWn[y].
template <bool COMPACT>
__global__ void dweight_label_combine_kernel(int B, int D, const int32_t* __restrict__ yl, int64_t k,
                                        const int32_t* __restrict__ head, int64_t kp, int nwin,
                                        float* __restrict__ part, float* __restrict__ dW) {
  const int lane = threadIdx.x & 63;
  const int i = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (i >= B) return;
  const int32_t y = __builtin_amdgcn_readfirstlane(yl[i]);
  if (y < 0 || (int64_t)y >= k) return;
  if (head[y] != i) return;
  const int32_t h = lane < nwin ? head[(int64_t)(1 + lane) * kp + y] : INT_MAX;
  const unsigned long long in = __ballot(h != INT_MAX);   // the windows that have the class
  for (int d = lane * 4; d < D; d += 256) {
    float4* dst = reinterpret_cast<float4*>((COMPACT ? part + (int64_t)i * D : dW + (int64_t)y * D) + d);
    float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
    for (unsigned long long m = in; m;) {
      constexpr int UN = 4;   // rows in flight
      float4 o[UN];
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        o[u] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (!m) continue;
        o[u] = *reinterpret_cast<const float4*>(part + (int64_t)__builtin_amdgcn_readlane(h, __builtin_ctzll(m)) * D + d);
        m &= m - 1;
      }
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        r.x += o[u].x; r.y += o[u].y; r.z += o[u].z; r.w += o[u].w;
      }
    }
    if constexpr (!COMPACT) {
      const float4 cur = *dst;
      r.x += cur.x; r.y += cur.y; r.z += cur.z; r.w += cur.w;
    }
    *dst = r;
  }
}

// ---------------------------------------------------------------------------------------------
// fused_update_tile (in gemm_backward_update, fused step): the dweight product on tiles that span all D
// columns, followed
// in the same workgroup by the SGD-momentum update of the tile's rows (Eq. 3; text after Eq. 4),
// so dWn is never written to memory: dWn_j = GEMM row + label part, g = (dWn - <dWn,wn> wn)/|w|,
// v <- mu v + g, W <- W - lr v, with the arithmetic of update_kernel in the same order.
// The accumulators go through LDS one half of the tile at a time (the rows of the wavefronts
// with the same wm); then every wavefront takes whole rows, 16 bytes per lane and column chunk,
// RB rows in flight.
// ---------------------------------------------------------------------------------------------
template <class Cfg>
struct FusedUpdateLds {
  static constexpr int HR = Cfg::WTM;               // rows per half
  static constexpr int SROW = Cfg::BN + 4;          // floats per staged row (+4: the two rows a
                                                    // store instruction touches fall 16 banks apart)
  static constexpr int BYTES = HR * SROW * 4;
  static constexpr int LDS = BYTES > Cfg::LDS_BYTES ? BYTES : Cfg::LDS_BYTES;
};

template <class Cfg>
__device__ __forceinline__ void fused_update_tile(
    int64_t j0, char* smem, const typename Cfg::elem* __restrict__ E,
    const typename Cfg::elem* __restrict__ Xs, int64_t k, int64_t kp, int Bp,
    const int32_t* __restrict__ idx, const int32_t* __restrict__ head,
    const float* __restrict__ lab, float* spare, float* __restrict__ W, float* __restrict__ V,
    int64_t N, float lr, float mu, int32_t* __restrict__ err_flag) {
  using FL = FusedUpdateLds<Cfg>;
  constexpr int D = Cfg::BN, NC = D / 256, HR = FL::HR, SROW = FL::SROW;
  constexpr int WAVES = Cfg::THREADS / 64, RPW = HR / WAVES;   // rows per wavefront and half
  constexpr int ROWS = Cfg::WM * RPW;                           // rows per wavefront and tile
  constexpr int WIN = 5;   // rows of W and v in flight (3 rows and the label part of each: 1024 x 205,991 with the
                           // update 1099 us a step, 3 rows 1089, 5 rows 1083)
  static_assert(D % 256 == 0 && HR % WAVES == 0 && ROWS <= 64 && WIN <= ROWS, "fused update geometry");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // Two spare rows of D floats: the first holds zeros (never written) and is what a padding row of
  // the last tile reads instead of W and v; the second takes the stores of the padding rows and is
  // never read.  Every row thus issues the same loads of W and v and the same stores in the same
  // order with no branch in between, which is what lets the wait for row n's operands leave the
  // younger requests of rows n+1 .. n+WIN in flight.  The few centers that are the label of a
  // sample read their label part when they are at it: as part of the window it was a third of all
  // loads, of a row of zeros for nearly every center.
  const float* zero_row = spare;
  float* trash_row = spare + D;

  // Row n of this wavefront (n = h*RPW + q) is tile row h*HR + q*WAVES + wave: neighbouring
  // wavefronts take neighbouring rows.  Lane n fetches its class id and label head now, so that
  // the epilogue starts its row loads without a dependent index load in front.
  int32_t idxv = -1, headv = INT_MAX;
  if (lane < ROWS) {
    const int64_t j = j0 + (lane / RPW) * HR + (lane % RPW) * WAVES + wave;
    if (j < k) {
      idxv = idx[j];
      headv = head[j];
      if (idxv < 0 || (int64_t)idxv >= N) {
        atomicOr(err_flag, 8);
        idxv = -1;
      }
    }
  }

  f32x16 acc[Cfg::TM][Cfg::TN];
  zero_acc<Cfg>(acc);
  PFC_PHASE(3, 0);
  gemm_tile<Cfg>(e_tile<Cfg>(E, 0, j0, Bp, kp), e_ld<Cfg>(Bp, kp), Xs, D, Bp / Cfg::BK, smem, acc);
  PFC_PHASE(3, 1);

  // A window of WIN rows of W and v is kept in flight: the loads of row n+WIN
  // are issued as soon as row n has been used, across the two halves.  (Native vector types:
  // arrays of them stay in registers.)
  f32x4 w[WIN][NC], v[WIN][NC];
  auto request = [&](int n) {
    const int64_t row = __builtin_amdgcn_readlane(idxv, n);   // wave-uniform
    const float* wsrc = row >= 0 ? W + row * D : zero_row;    // scalar selects, no branch
    const float* vsrc = row >= 0 ? V + row * D : zero_row;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      // nontemporal: rows loaded plainly would be written back to the memory-side cache and leave it
      // while the next kernels run (us a step: 1024 x 36,024 249 -> 242, 1024 x 70,000 406 -> 386, 1024 x
      // 205,991 1023 -> 1004, 2048 x 500,000 3980 -> 3927)
      w[n % WIN][c] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(wsrc + c * 256 + lane * 4));
      v[n % WIN][c] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(vsrc + c * 256 + lane * 4));
    }
  };
#pragma unroll
  for (int n = 0; n < WIN; ++n) request(n);

  float* stage = reinterpret_cast<float*>(smem);
  const int wm = wave / Cfg::WN, wn = wave % Cfg::WN;
#pragma unroll
  for (int h = 0; h < Cfg::WM; ++h) {
    if (wm == h) {
#pragma unroll
      for (int bm = 0; bm < Cfg::TM; ++bm)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = bm * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
#pragma unroll
          for (int bn = 0; bn < Cfg::TN; ++bn)
            stage[row * SROW + wn * Cfg::WTN + bn * 32 + (lane & 31)] = acc[bm][bn][r];
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < RPW; ++q) {
      const int n = h * RPW + q;
      const int64_t row = __builtin_amdgcn_readlane(idxv, n);
      const int r = q * WAVES + wave;
      float* wdst = row >= 0 ? W + row * D : trash_row;
      float* vdst = row >= 0 ? V + row * D : trash_row;
      f32x4 g[NC];
      float ww = 0.f, gw = 0.f;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int d = c * 256 + lane * 4;
        g[c] = *reinterpret_cast<const f32x4*>(stage + r * SROW + d);
      }
      // the label part of a center that is the label of a sample
      const int hd = __builtin_amdgcn_readlane(headv, n);
      if (hd != INT_MAX) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
          g[c] += *reinterpret_cast<const f32x4*>(lab + (int64_t)hd * D + c * 256 + lane * 4);
      }
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const f32x4 wc = w[n % WIN][c];
        ww += wc[0] * wc[0] + wc[1] * wc[1] + wc[2] * wc[2] + wc[3] * wc[3];
        gw += g[c][0] * wc[0] + g[c][1] * wc[1] + g[c][2] * wc[2] + g[c][3] * wc[3];
      }
      ww = wave_sum(ww);
      gw = wave_sum(gw);
      const float rn = 1.f / fmaxf(sqrtf(ww), 1e-12f);
      const float t = gw * rn * rn;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int d = c * 256 + lane * 4;
        const f32x4 wc = w[n % WIN][c], vc = v[n % WIN][c];
        f32x4 vn, wq;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          vn[e] = mu * vc[e] + (g[c][e] - t * wc[e]) * rn;
          wq[e] = wc[e] - lr * vn[e];
        }
        // not read again before the next step's gather: nontemporal, so that the rows do not
        // sit dirty in the L2 while the next kernels run
        __builtin_nontemporal_store(vn, reinterpret_cast<f32x4*>(vdst + d));
        __builtin_nontemporal_store(wq, reinterpret_cast<f32x4*>(wdst + d));
      }
      if (n + WIN < ROWS) request(n + WIN);
    }
    __syncthreads();   // the next half overwrites the staged rows
    PFC_PHASE(3, 2 + h);
  }
}

// gemm_backward_update: as gemm_backward, the dfeatures product (MFMA bound) shares the launch with
// the dweight product that ends in the update (HBM bound more than half of its time): 715 us one
// after the other, 698 together at 1024 samples x 205,991 classes x 512, 162 -> 137 at 36,024
// classes.  Behind the dfeatures workgroups, n_big workgroups take tiles of CfgB::BM rows; the rows
// left over when those no longer fill a whole round of workgroups on the GPU go to the following
// workgroups in tiles of CfgS::BM rows, so that the last, partly filled round is short.
template <class CfgX, class CfgB, class CfgS>
__global__ __launch_bounds__(CfgB::THREADS) void gemm_backward_update_kernel(
    const typename CfgB::elem* __restrict__ E, const typename CfgB::elem* __restrict__ Wn,
    const typename CfgB::elem* __restrict__ Xs, DxShape dx, float* __restrict__ dXpart, int64_t k, int64_t kp, int Bp, const int32_t* __restrict__ idx,
    const int32_t* __restrict__ head, const float* __restrict__ lab, float* spare,
    float* __restrict__ W, float* __restrict__ V, int64_t N, float lr, float mu,
    int32_t* __restrict__ err_flag, int n_big) {
  static_assert(CfgB::THREADS == CfgS::THREADS && CfgB::THREADS == CfgX::THREADS &&
                CfgB::BN == CfgS::BN, "one launch shape");
  extern __shared__ __align__(16) char smem[];
  if ((int)blockIdx.x < dx.wgs) {
    dfeatures_tile<CfgX, false>(blockIdx.x, smem, E, Wn, CfgB::BN, Bp, kp, dx, dXpart);
    return;
  }
  const int b = (int)blockIdx.x - dx.wgs;
  if (b < n_big)
    fused_update_tile<CfgB>((int64_t)b * CfgB::BM, smem, E, Xs, k, kp, Bp, idx, head, lab, spare,
                            W, V, N, lr, mu, err_flag);
  else
    fused_update_tile<CfgS>((int64_t)n_big * CfgB::BM + (int64_t)(b - n_big) * CfgS::BM, smem, E,
                            Xs, k, kp, Bp, idx, head, lab, spare, W, V, N, lr, mu, err_flag);
}

// dfeatures_final_block (in gradients_final): WPS wavefronts per sample.
//   g  = (s/(B l_i)) * sum_slices part + dlabel_i * wn_{y_i}        (dL/d xn_i)
//   dx = (g - <g, xn_i> xn_i) / |x_i|
template <int NC, int WPS>
struct FinalLds {
  float4 part[kLabelThreads / 64 / WPS][WPS > 1 ? WPS - 1 : 1][WPS > 1 ? NC : 1][64];
};
struct FinalArgs {
  const float* part;
  int splits, B, Bp, D, Dp;
  const float* X;
  const float* W;
  int64_t N;
  const int32_t* idx;
  const int32_t* yl;
  int64_t k;
  const float *rnormX, *rnormW, *wlab, *rowscale, *dlabel;
  float* dX;
  const float* lossrow;
  float* loss_out;
  const float *clabel, *rowmax;
  float* stats_out;
};

// Mean loss (and, on request, mean label cosine = APCS and mean largest non-label cosine = AMNCS),
// each summed in a fixed order (256 strided partials, then a tree).
__device__ __forceinline__ void mean_loss_block(float* sm, const FinalArgs& a) {
  const int nq = a.stats_out ? 3 : 1;
  for (int q = 0; q < nq; ++q) {
    const float* src = q == 0 ? a.lossrow : q == 1 ? a.clabel : a.rowmax;
    float v = 0.f;
    if (threadIdx.x < 256) {
      for (int r = threadIdx.x; r < a.B; r += 256) v += src[r];
      sm[threadIdx.x] = v;
    }
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
      if ((int)threadIdx.x < o) sm[threadIdx.x] += sm[threadIdx.x + o];
      __syncthreads();
    }
    if (threadIdx.x == 0) (q == 0 ? a.loss_out : a.stats_out + (q - 1))[0] = sm[0] / (float)a.B;
    __syncthreads();
  }
}

template <int NC, int WPS>
__device__ __forceinline__ void dfeatures_final_block(int block, FinalLds<NC, WPS>& lds,
                                                      const FinalArgs& a) {
  constexpr int SPB = kLabelThreads / 64 / WPS;   // samples per workgroup
  const int lane = threadIdx.x & 63;
  const int grp = (threadIdx.x >> 6) / WPS, wave = (threadIdx.x >> 6) % WPS;
  const int i = block * SPB + grp;
  const int D = a.D;
  // The wavefronts of a sample share the slices of S (wavefront w takes slices w, w + WPS, ...:
  // several independent loads in flight each); their partial rows are added in wavefront order by
  // wavefront 0, which then finishes the row: the same order on every run.  What the last step
  // needs is requested before the slices and in front of the barrier: the chain label -> class id
  // -> row of W behind them was most of a small launch.
  const bool ends = wave == 0 && i < a.B;
  float rs = 0.f, rnx = 0.f, dl = 0.f, rnw = 0.f;
  int32_t y = -1;
  float4 x[NC], w[NC], sum[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) x[c] = w[c] = sum[c] = make_float4(0.f, 0.f, 0.f, 0.f);
  if (ends) {
    y = a.yl[i];
    rs = a.rowscale[i];
    rnx = a.rnormX[i];
    dl = a.dlabel[i];
#pragma unroll
    for (int c = 0; c < NC; ++c)
      if (c * 256 + lane * 4 < D) x[c] = *reinterpret_cast<const float4*>(a.X + (int64_t)i * D + c * 256 + lane * 4);
  }
  if (i < a.B) {
    // U slices requested before the first is added (longer rows have no registers for it)
    constexpr int U = NC <= 2 ? 2 : 1;
    for (int sp = wave; sp < a.splits; sp += U * WPS) {
      float4 t[U][NC];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          t[u][c] = make_float4(0.f, 0.f, 0.f, 0.f);   // columns from D on are zero
          if (sp + u * WPS < a.splits && c * 256 + lane * 4 < D)
            t[u][c] = *reinterpret_cast<const float4*>(a.part + ((int64_t)(sp + u * WPS) * a.Bp + i) * a.Dp + c * 256 +
                                                       lane * 4);
        }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          sum[c].x += t[u][c].x; sum[c].y += t[u][c].y; sum[c].z += t[u][c].z; sum[c].w += t[u][c].w;
        }
    }
  }
  if (ends && y >= 0 && (int64_t)y < a.k) {
    const int64_t row = a.idx[y];
    rnw = a.rnormW[y];
    if (row >= 0 && row < a.N) {
      // (a.wlab: W has been updated already, the label's row as it was)
      const float* src = a.wlab ? a.wlab + (int64_t)i * D : a.W + row * D;
#pragma unroll
      for (int c = 0; c < NC; ++c)
        if (c * 256 + lane * 4 < D) w[c] = *reinterpret_cast<const float4*>(src + c * 256 + lane * 4);
    }
  }
  if constexpr (WPS > 1) {
    if (wave > 0) {
#pragma unroll
      for (int c = 0; c < NC; ++c) lds.part[grp][wave - 1][c][lane] = sum[c];
    }
    __syncthreads();
    if (!ends) return;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
#pragma unroll
      for (int v = 0; v < WPS - 1; ++v) {
        if (v + 1 >= a.splits) break;   // those wavefronts had no slice
        const float4 t = lds.part[grp][v][c][lane];
        sum[c].x += t.x; sum[c].y += t.y; sum[c].z += t.z; sum[c].w += t.w;
      }
    }
  } else if (!ends) {
    return;
  }
  float* dX = a.dX;
  float4 g[NC], xn[NC];
  float u = 0.f;
#pragma unroll
  for (int c = 0; c < NC; ++c) {   // (all are zero from column D on)
    float4 t = sum[c], v = x[c];
    const float f = dl * rnw;
    t.x *= rs; t.y *= rs; t.z *= rs; t.w *= rs;
    t.x += f * w[c].x; t.y += f * w[c].y; t.z += f * w[c].z; t.w += f * w[c].w;
    v.x *= rnx; v.y *= rnx; v.z *= rnx; v.w *= rnx;
    g[c] = t;
    xn[c] = v;
    u += t.x * v.x + t.y * v.y + t.z * v.z + t.w * v.w;
  }
  u = wave_sum(u);
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    float4 o;
    o.x = (g[c].x - u * xn[c].x) * rnx;
    o.y = (g[c].y - u * xn[c].y) * rnx;
    o.z = (g[c].z - u * xn[c].z) * rnx;
    o.w = (g[c].w - u * xn[c].w) * rnx;
    if (c * 256 + lane * 4 < D)
      *reinterpret_cast<float4*>(dX + (int64_t)i * D + c * 256 + lane * 4) = o;
  }
}

// gradients_final: what is left after the backward products, in one launch: the label part of dWn
// (`label_blocks` workgroups), the finished rows of dX and the mean loss (workgroup 0: the longest
// with a large batch).  None needs anything of the others; one after the other they are two chains
// of dependent loads that leave the GPU idle, and with a large batch the mean loss runs alone at
// the end.  64 registers: two workgroups on a compute unit.  Step, two launches -> one: 128 x 1,000
// x 512 fp32 59.9 -> 56.1 us, 512 x 9,344 x 512 104.4 -> 101.0, 256 x 25,723 x 128 79.5 -> 74.1,
// 768 x 20,599 x 1024 277 -> 271, 16,384 samples x 3,592 476 -> 462.  A sample gets four wavefronts; up
// to kFinalOneSplits slices one: three of four would have none; from kFinalWideSplits on 16, below
// which a third of them would have none, if there is a compute unit for every sample.  (This launch,
// us, 16 wavefronts / 4: 1024 x 205,991 x 512 20.8 / 17.7, fused 16.9 / 12.6, fused 1024 x 36,024 13.8 /
// 10.0, 1024 x 40,000 x 256 14.8 / 12.2, 400 x 40,000 x 1024 14.7 / 12.3; 200 x 60,000 x 768 11.2 /
// 12.8, 64 x 200,000 x 512 in fp32 12.3 / 16.0.  Behind the line: 260 x 60,000 x 512 9.1 / 9.9, in fp32 10.8 /
// 12.3, 260 x 40,000 x 1024 12.0 / 11.9, 320 x 60,000 x 512 10.8 / 9.9, 400 12.6 / 10.3.)
constexpr int kFinalWideSplits = 12, kFinalOneSplits = 2;
template <int NC, int WPS, bool WINDOWS>
__global__ __launch_bounds__(kLabelThreads, 8) void gradients_final_kernel(
    FinalArgs a, int label_blocks, const int32_t* __restrict__ head, const int32_t* __restrict__ order,
    const int32_t* __restrict__ runs, float* __restrict__ label_out) {
  __shared__ union Lds {
    std::conditional_t<WINDOWS, WindowLds<NC>, LabelLds> label;
    FinalLds<NC, WPS> final;
    float sum[256];
  } lds;
  const int b = (int)blockIdx.x - 1;
  if (b < 0)
    mean_loss_block(lds.sum, a);
  else if (b >= label_blocks)
    dfeatures_final_block<NC, WPS>(b - label_blocks, lds.final, a);
  else if constexpr (WINDOWS)
    window_label_block<NC>(b, lds.label, a.X, a.D, order, runs, a.rnormX, a.dlabel, label_out);
  else
    dweight_label_block<LABEL_ADD>(b, lds.label, a.X, a.B, a.D, a.yl, a.k, head, a.rnormX, a.dlabel, label_out);
}

// ---------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------
// One size of GEMM tiles: the tile of every product (BM x BN of its output, WM x WN wavefronts).
template <typename T, int BM, int BN, int WM, int WN>
struct Tiles {
  using F = TileCfg<T, BM, BN, WM, WN, false, false>;   // logits: classes x samples
  using W = TileCfg<T, BM, BN, WM, WN, true, true>;     // dweight: classes x columns
  using X = TileCfg<T, BM, BN, WM, WN, false, true>;    // dfeatures: samples x columns
  static constexpr int BACK_LDS = X::LDS_BYTES > W::LDS_BYTES ? X::LDS_BYTES : W::LDS_BYTES;
  // sums in pieces (kDxSumSteps); a 256-tile has no registers for them
  static constexpr bool PIECES = sizeof(T) == 4 && BM < 256;
};

template <class S>
int set_lds_limits_logits(S) {
  using F = typename S::F;
  const void* f[] = {(const void*)gemm_logits_kernel<F, false>, (const void*)gemm_logits_kernel<F, true>,
                     (const void*)gemm_rowmax_kernel<F>};
  for (const void* p : f)
    PFC_HIP(hipFuncSetAttribute(p, hipFuncAttributeMaxDynamicSharedMemorySize, F::LDS_BYTES));
  if constexpr (std::is_same_v<typename F::elem, float> && F::BM == 64) {
    const void* slim[] = {(const void*)gemm_logits_slim_kernel<false>, (const void*)gemm_logits_slim_kernel<true>};
    for (const void* p : slim) PFC_HIP(hipFuncSetAttribute(p, hipFuncAttributeMaxDynamicSharedMemorySize, kSlimLds));
  }
  return PFC_OK;
}
template <class S>
int set_lds_limits_backward(S) {
  using X = typename S::X;
  using W = typename S::W;
  constexpr bool kPieces = S::PIECES;
  const void* b[] = {(const void*)(gemm_backward_kernel<X, W, false, false>),
                     (const void*)(gemm_backward_kernel<X, W, false, kPieces>),
                     (const void*)(gemm_backward_kernel<X, W, true, kPieces>)};
  for (const void* p : b)
    PFC_HIP(hipFuncSetAttribute(p, hipFuncAttributeMaxDynamicSharedMemorySize, S::BACK_LDS));
  return PFC_OK;
}

template <typename T, int NC>
int run(pfc_ctx* c, const float* X, const float* W, const int32_t* idx, int64_t k,
        const int32_t* yl, int32_t B, const LossParams& lp, float* loss_out, float* dX_out,
        float* dW_out, float* stats_out, const UpdateArgs* upd) {
  // fused dweight + update: 128 classes x all 512 columns, half-size slabs so that the wide
  // operand fits; this one-kernel form exists for D == 512 only
  using CfgU = TileCfg<T, 128, 512, 2, 4, true, true, 64, 4, 4>;
  using CfgUS = TileCfg<T, 64, 512, 1, 8, true, true, 128>;   // its tiles for the last round
  using Big = Tiles<T, 256, 256, 2, 4>;
  using Mid = Tiles<T, 128, 128, 2, 4>;
  using Small = Tiles<T, 64, 64, 2, 2>;
  constexpr int kFusedLds =
      std::max({FusedUpdateLds<CfgU>::LDS, FusedUpdateLds<CfgUS>::LDS, Big::X::LDS_BYTES});
  static_assert(kFusedLds <= 160 * 1024, "LDS of one compute unit");
  const int D = c->D;
  const int64_t kp = round_up(k, kPadK);
  const TileSize size_f = logits_tiles(c->num_cu, sizeof(T), B, kp, D),
                 size_b = backward_tiles(c->num_cu, sizeof(T), B, kp, D);
  const int Bp = (int)round_up(B, std::max<int>(size_f, size_b));
  // row length of the library's own GEMM operands
  const int Dp = (int)round_up(D, size_b == TILES_256 ? 256 : kPadD);
  T* Xn = (T*)c->Xn; T* Xs = (T*)c->Xs; T* Wn = (T*)c->Wn; T* E = (T*)c->E;
  // windows of the label part (0: the batch fits one window, or the context has no room for them)
  const int nwin = (B > kLabelWindow && c->label_windows) ? (B + kLabelWindow - 1) / kLabelWindow : 0;

  // fused call: one kernel for dweight and update only if D fits its tile and there is at least one
  // tile per CU
  static_assert(CfgU::BM == 128 && CfgU::BN == 512, "fits_one_kernel");
  const bool plain_sums = fits_one_kernel(c->num_cu, D, kp), one_kernel = upd && plain_sums;

  const bool short_rows = Dp == 128;
  const bool plain = !one_kernel && row_policy(c->esize, c->N, D, c->B_max, k).gather_plain;
  auto norm_kernel = plain ? gather_normalize_kernel<T, NC, false, true> : gather_normalize_kernel<T, NC, false, false>;
  if constexpr (NC == 1)
    if (short_rows)
      norm_kernel = plain ? gather_normalize_kernel<T, NC, true, true> : gather_normalize_kernel<T, NC, true, false>;
  const int64_t rows_per_block = (short_rows ? 8 : 4) * kNormWaves;   // (a divisor of kPadK)
  const int x_blocks = (Bp + kNormWaves - 1) / kNormWaves;
  PFC_LAUNCH(c, KID_GATHER_W, norm_kernel,
             dim3((unsigned)(nwin + x_blocks + kp / rows_per_block)),
             dim3(kNormWaves * 64), 0, x_blocks, X, B, Bp, yl, Xn, c->rnormX, c->clabel, W, c->N,
             idx, k, kp, D, Dp, Wn, c->rnormW, c->head, nwin, c->label_order, c->label_runs, c->err_flag);

  // raise the dynamic LDS limit of this context's kernels once (a context has one precision and
  // one D, hence one instantiation of run)
  if (!c->lds_attr_set) {
    int rc = set_lds_limits_logits(Big{});
    if (rc == PFC_OK) rc = set_lds_limits_logits(Mid{});
    if (rc == PFC_OK) rc = set_lds_limits_logits(Small{});
    if (rc == PFC_OK) rc = set_lds_limits_backward(Big{});
    if (rc == PFC_OK) rc = set_lds_limits_backward(Mid{});
    if (rc == PFC_OK) rc = set_lds_limits_backward(Small{});
    if (rc != PFC_OK) return rc;
    PFC_HIP(hipFuncSetAttribute((const void*)(gemm_backward_update_kernel<typename Big::X, CfgU, CfgUS>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, kFusedLds));
    PFC_HIP(hipFuncSetAttribute((const void*)(gemm_backward_update_kernel<typename Mid::X, CfgU, CfgUS>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, kFusedLds));
    c->lds_attr_set = 1;
  }
  auto launch_logits = [&](auto tiles) -> int {
    using Cfg = typename decltype(tiles)::F;
    const int tiles_j = (int)(kp / Cfg::BM), tiles_i = Bp / Cfg::BN;
    if (lp.rowref) {   // scale above 64: the largest logit of every sample first
      PFC_LAUNCH(c, KID_GEMM_ROWMAX, gemm_rowmax_kernel<Cfg>, dim3(xcd_grid(tiles_i, tiles_j)),
                 dim3(Cfg::THREADS), Cfg::LDS_BYTES, Wn, Xn, D, Dp, k, B, yl, lp, c->rowmaxpart,
                 tiles_j, tiles_i);
      PFC_LAUNCH(c, KID_ROW_REF, row_ref_kernel, dim3((Bp + 3) / 4), dim3(256), 0, c->rowmaxpart,
                 tiles_j, B, Bp, c->rowref);
    }
    // the options (filter, column maxima, reference) have a kernel of their own: the plain one
    // stays lean
    bool slim = false;
    if constexpr (sizeof(T) == 4 && Cfg::BM == 64) slim = logits_slim(c->num_cu, B, kp);
    if constexpr (sizeof(T) == 4 && Cfg::BM == 64) {
      if (slim) {
        auto slim_kernel = lp.extras ? gemm_logits_slim_kernel<true> : gemm_logits_slim_kernel<false>;
        PFC_LAUNCH(c, KID_GEMM_LOGITS, slim_kernel, dim3(xcd_grid(Bp / 16, tiles_j)), dim3(256), kSlimLds,
                   (const float*)Wn, (const float*)Xn, D,
                   Dp, k, B, kp, yl, lp, (float*)E, c->rowpart, c->rowmaxpart, c->clabel, tiles_j, Bp / 16);
      }
    }
    if (!slim) {
      auto logits_kernel = lp.extras ? gemm_logits_kernel<Cfg, true> : gemm_logits_kernel<Cfg, false>;
      PFC_LAUNCH(c, KID_GEMM_LOGITS, logits_kernel, dim3(xcd_grid(tiles_i, tiles_j)),
                 dim3(Cfg::THREADS), Cfg::LDS_BYTES, Wn, Xn, D, Dp, k, B, Bp, kp, yl, lp, E, c->rowpart,
                 c->rowmaxpart, c->clabel, tiles_j, tiles_i, c->num_cu / 8 * 8);
    }
    auto combine_kernel = row_combine_kernel<T, NC>;
    const int head_blocks = (B + kLabelWindow - 1) / kLabelWindow;
    PFC_LAUNCH(c, KID_ROW_COMBINE, combine_kernel, dim3(head_blocks + (Bp + 3) / 4), dim3(256), 0,
               head_blocks, c->rowpart,
               tiles_j, logits_chained<Cfg>() ? 1 : 0, B, Bp, D, Dp, X, c->rnormX, c->clabel, lp, c->rowmaxpart, c->rowscale,
               c->dlabel, c->lossrow, c->rowmax, yl, k, kp, c->head, nwin, Xs, W, c->N, idx,
               one_kernel ? c->wlab : nullptr);
    return PFC_OK;
  };
  {
    const int rc = size_f == TILES_256   ? launch_logits(Big{})
                   : size_f == TILES_128 ? launch_logits(Mid{})
                                         : launch_logits(Small{});
    if (rc != PFC_OK) return rc;
  }
  // window sums of the label part, added up: to dW_out, or (compact) in the side buffer
  auto launch_label_sum = [&](auto compact) -> int {
    PFC_LAUNCH(c, KID_DW_LABEL_SUM, dweight_label_combine_kernel<compact.value>, dim3((B + 3) / 4), dim3(256),
               0, B, D, yl, k, c->head, kp, nwin, c->dlab, dW_out);
    return PFC_OK;
  };
  // label part of dWn in a launch of its own: added to dW_out, or (compact) left in the side buffer
  auto launch_label = [&](auto compact) -> int {
    if (nwin) {
      PFC_LAUNCH(c, KID_DW_LABEL, window_label_kernel<NC>, dim3(nwin * kWindowBlocks), dim3(kLabelThreads), 0,
                 X, D, c->label_order, c->label_runs, c->rnormX, c->dlabel, c->dlab);
      return launch_label_sum(compact);
    }
    auto kernel = dweight_label_kernel<compact.value ? LABEL_COMPACT : LABEL_ADD>;
    PFC_LAUNCH(c, KID_DW_LABEL, kernel, dim3(B), dim3(kLabelThreads), 0, X, B, D, yl, k, c->head,
               c->rnormX, c->dlabel, compact.value ? c->dlab : dW_out);
    return PFC_OK;
  };
  // The rest of both gradients; with_label: the label part of dWn is still to be added to dW_out.
  // (One thing keeps them apart: dX written over the features that the label part reads.)
  auto launch_final = [&](const DxShape& dx, bool with_label, const float* wlab) -> int {
    const uintptr_t x0 = (uintptr_t)X, dx0 = (uintptr_t)dX_out, bytes = (uintptr_t)B * D * 4;
    if (with_label && x0 < dx0 + bytes && dx0 < x0 + bytes) {
      const int rc = launch_label(std::false_type{});
      if (rc != PFC_OK) return rc;
      with_label = false;
    }
    const FinalArgs fa{c->dXpart, dx.splits, B, Bp, D, Dp, X, W, c->N, idx, yl, k, c->rnormX,
                       c->rnormW, wlab, c->rowscale, c->dlabel, dX_out, c->lossrow, loss_out,
                       c->clabel, c->rowmax, stats_out};
    const int label_blocks = !with_label ? 0 : nwin ? nwin * kWindowBlocks : B;
    const bool wide = dx.splits >= kFinalWideSplits && B <= c->num_cu && !nwin, one = dx.splits <= kFinalOneSplits;
    const int spb = kLabelThreads / 64 / (wide ? 16 : one ? 1 : 4);
    // (windows: batches above one window, many samples)
    auto kernel = nwin   ? (one ? gradients_final_kernel<NC, 1, true> : gradients_final_kernel<NC, 4, true>)
                  : wide ? gradients_final_kernel<NC, 16, false>
                  : one  ? gradients_final_kernel<NC, 1, false>
                         : gradients_final_kernel<NC, 4, false>;
    PFC_LAUNCH(c, KID_GRAD_FINAL, kernel, dim3((unsigned)(1 + label_blocks + (B + spb - 1) / spb)),
               dim3(kLabelThreads), 0, fa, label_blocks, c->head, c->label_order, c->label_runs,
               nwin ? c->dlab : dW_out);
    return with_label && nwin ? launch_label_sum(std::false_type{}) : PFC_OK;
  };
  const BackwardShape shape = backward_shape(c->num_cu, sizeof(T), size_b, Bp, Dp, D, kp);
  // both backward products in one launch; dW_out and the partial sums of dX are written
  auto launch_backward = [&](auto tiles, DxShape& dx) -> int {
    using CX = typename decltype(tiles)::X;
    using CW = typename decltype(tiles)::W;
    constexpr int lds = decltype(tiles)::BACK_LDS;
    const int tiles_j = (int)(kp / CW::BM), tiles_d = Dp / CW::BN;
    dx = shape.dx;
    const int slabs_per = shape.slabs_per, nsp = shape.splits;
    float* dst = nsp > 1 ? c->dXpart + (int64_t)dx.splits * Bp * Dp : dW_out;
    // a class set that the one-kernel form takes: the sums of that form (which has no registers for a
    // second set of accumulators), so that dX has the same bits in either call
    constexpr bool kPieces = decltype(tiles)::PIECES;
    auto kernel = nsp > 1      ? gemm_backward_kernel<CX, CW, true, kPieces>
                  : plain_sums ? gemm_backward_kernel<CX, CW, false, false>
                               : gemm_backward_kernel<CX, CW, false, kPieces>;
    const int wgs_w = tiles_j * tiles_d * nsp;
    PFC_LAUNCH(c, KID_GEMM_BACKWARD, kernel, dim3((unsigned)(dx.wgs + wgs_w)), dim3(CX::THREADS), lds, E,
               Wn, Xs, D, Dp, k, kp, Bp, dx, c->dXpart, dst, tiles_j, tiles_d, slabs_per, nsp,
               shape.dw_first ? wgs_w : 0);
    if (nsp > 1) {
      PFC_LAUNCH(c, KID_DW_REDUCE, dweight_reduce_kernel,
                 dim3((unsigned)((k * D / 4 + 255) / 256)), dim3(256), 0, dst, nsp, k, kp, D, Dp,
                 dW_out);
    }
    return PFC_OK;
  };
  // tiles: those of the dfeatures product.  Its slices are the ones that gemm_backward would take
  // (size_b), whatever the tiles: dX has the same bits in either call.
  auto launch_backward_update = [&](auto tiles, DxShape& dx) -> int {
    using CX = typename decltype(tiles)::X;
    dx = shape.dx;
    dx.tiles_i = Bp / CX::BM;
    dx.tiles_d = Dp / CX::BN;
    dx.wgs = (int)round_up(xcd_grid(dx.tiles_i * dx.tiles_d, dx.splits), 8);
    const int tiles_big = (int)(kp / CfgU::BM);
    const int n_big = tiles_big / c->num_cu * c->num_cu;          // whole rounds
    const int n_small = (tiles_big - n_big) * (CfgU::BM / CfgUS::BM);
    PFC_LAUNCH(c, KID_GEMM_BACKWARD_UPDATE, (gemm_backward_update_kernel<CX, CfgU, CfgUS>),
               dim3((unsigned)(dx.wgs + n_big + n_small)), dim3(CfgU::THREADS), kFusedLds, E, Wn, Xs,
               dx, c->dXpart, k, kp, Bp, idx, c->head, c->dlab, c->spare, upd->W, upd->v, c->N,
               upd->lr, upd->mu, c->err_flag, n_big);
    return PFC_OK;
  };

  DxShape dx;
  int rc;
  if (!one_kernel) {
    rc = size_b == TILES_256   ? launch_backward(Big{}, dx)
         : size_b == TILES_128 ? launch_backward(Mid{}, dx)
                               : launch_backward(Small{}, dx);
    if (rc == PFC_OK) rc = launch_final(dx, true, nullptr);
    // fused call: dWn went through memory (dW_out is the context's own buffer here)
    if (rc == PFC_OK && upd) rc = update_impl(c, upd->W, upd->v, idx, k, dW_out, upd->lr, upd->mu);
    return rc;
  }
  rc = launch_label(std::true_type{});
  if (rc == PFC_OK) {
    // (never 64-tiles: D == 512 and a 128-row tile per compute unit are many 128-tiles)
    // One workgroup per compute unit whatever the dfeatures tile, so the big one where it fits
    rc = Bp % 256 == 0 ? launch_backward_update(Big{}, dx) : launch_backward_update(Mid{}, dx);
  }
  return rc == PFC_OK ? launch_final(dx, false, c->wlab) : rc;
}

}  // namespace

int forward_backward_impl(pfc_ctx* c, const float* X, const float* W, const int32_t* idx,
                          int64_t k, const int32_t* yl, int32_t B, float s, float m,
                          int32_t margin_type, float filter_threshold, float* loss_out,
                          float* dX_out, float* dW_out, float* stats_out,
                          const UpdateArgs* upd) {
  LossParams lp;
  lp.s = s;
  lp.s_log2e = s * 1.44269504088896340736f;
  lp.m = m;
  lp.cos_m = cosf(m);
  lp.sin_m = sinf(m);
  lp.cosface = margin_type == PFC_MARGIN_COSFACE ? 1 : 0;
  lp.tau = filter_threshold;
  // cosines lie in [-1, 1]: up to s = 64 exp(s*cos) and its row sums stay inside the fp32 (and
  // bf16) range without a reference; above, the softmax runs relative to each sample's maximum
  lp.rowref = s > 64.f ? c->rowref : nullptr;
  lp.extras = (filter_threshold < 1.f || stats_out != nullptr || lp.rowref) ? 1 : 0;
#define PFC_RUN(T, NC) \
  return run<T, NC>(c, X, W, idx, k, yl, B, lp, loss_out, dX_out, dW_out, stats_out, upd)
  const int nc = (c->D + 255) / 256;
  if (c->precision == PFC_PRECISION_BF16) {
    switch (nc) {
      case 1: PFC_RUN(__bf16, 1);
      case 2: PFC_RUN(__bf16, 2);
      case 3: PFC_RUN(__bf16, 3);
      case 4: PFC_RUN(__bf16, 4);
    }
  } else {
    switch (nc) {
      case 1: PFC_RUN(float, 1);
      case 2: PFC_RUN(float, 2);
      case 3: PFC_RUN(float, 3);
      case 4: PFC_RUN(float, 4);
    }
  }
#undef PFC_RUN
  return PFC_EINVAL;
}

}  // namespace pfc
