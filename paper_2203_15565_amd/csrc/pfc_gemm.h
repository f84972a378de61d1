// MFMA tile engine for the three GEMMs of the PFC step (gfx950).
//
//   logits    C[j][i] = sum_d Wn[j][d] * Xn[i][d]        A = Wn  (k contiguous), B = Xn (k contiguous)
//   dweight   C[j][d] = sum_i E[i][j]  * Xs[i][d]        A = E   (k-major),      B = Xs (k-major)
//   dfeatures C[i][d] = sum_j E[i][j]  * Wn[j][d]        A = E   (k contiguous), B = Wn (k-major)
//
// Every matrix but E in bf16 (OctetLds) stays in its one natural row-major layout in HBM; an operand whose reduction
// index is its ROW index ("k-major") is staged in LDS as it is and transposed on the way into
// the MFMA registers by the LDS transpose read of gfx950 (ds_read_b64_tr_b16), so no transposed
// copy of E, Wn or Xs is ever written.  Operands are padded with zeros to whole tiles by their
// producers: the main loop has no bounds checks.
//
// A workgroup of WM x WN wavefronts (64 lanes each) owns a BM x BN tile of C.  K is walked in slabs
// of BK = 64 (bf16) or 32 (fp32) reduction steps.  bf16 operands go from global memory to LDS
// without registers (gemm_tile_dma).  The fp32 operands of the backward products are split into
// planes of 16 bits on the way (gemm_tile_split): three bf16 planes and six products; those of the
// logits are multiplied as they are (gemm_tile_fp32).
//
// Fragment convention (the same for A and B, which is all a dot product needs): a group of 16 reduction
// steps is split between the lane halves, lanes 0..31 taking the first half and lanes 32..63 the
// second; one v_mfma_f32_32x32x16 per group.
//
// Accumulator layout of a 32x32 block (16 floats per lane): register r of lane l holds
//   row = (r / 4) * 8 + (l / 32) * 4 + (r % 4),  col = l % 32.
#pragma once

#include <type_traits>
#include <utility>

#include "pfc_common.h"

namespace pfc {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));


template <typename T, int BM_, int BN_, int WM_, int WN_, bool AKM, bool BKM, int SLAB = 128, int ABUF_ = 3,
          int BBUF_ = 2>
struct TileCfg {
  using elem = T;
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_;
  static constexpr bool A_KMAJOR = AKM, B_KMAJOR = BKM;
  static constexpr int BK = SLAB / (int)sizeof(T);   // reduction steps per slab
  static constexpr int GROUPS = SLAB / 32;           // reduction groups (fragment reads) per slab
  static constexpr int SLAB_BYTES = SLAB, ABUF = ABUF_, BBUF = BBUF_;   // slabs of A and B in LDS (bf16)
  static constexpr int THREADS = WM * WN * 64;
  // two workgroups of 128-tiles on a compute unit: at most 128 registers
  static constexpr int MIN_WAVES = BM == 128 && BN == 128 ? 4 : 1;
  static constexpr int WTM = BM / WM, WTN = BN / WN;       // tile of one wavefront
  static constexpr int TM = WTM / 32, TN = WTN / 32;       // 32x32 blocks per wavefront
  static constexpr bool DMA = sizeof(T) == 2;
  static constexpr bool A_OCTETS = DMA && BKM;   // A is E in both backward products
  static constexpr bool SPLIT = !DMA && (AKM || BKM);   // fp32: all but the logits (both k contiguous)
  static constexpr int LDS_BYTES = DMA     ? (ABUF * BM + BBUF * BN) * SLAB
                                   : SPLIT ? 2 * 3 * 32 * (BM + BN)
                                           : 2 * (SLAB + 16) * (BM + BN);
  static_assert(WTM % 32 == 0 && WTN % 32 == 0, "wave tile must be whole 32x32 blocks");
};

__device__ __forceinline__ void mfma_bf16(const u32x4& a, const u32x4& b, f32x16& c) {
  c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                              0, 0);
}

// The MFMA fragments of one reduction group for a whole wavefront tile.
template <class Cfg>
struct Frags {
  u32x4 a[Cfg::TM];
  u32x4 b[Cfg::TN];
};

template <class Cfg>
__device__ __forceinline__ void zero_acc(f32x16 (&acc)[Cfg::TM][Cfg::TN]) {
#pragma unroll
  for (int a = 0; a < Cfg::TM; ++a)
#pragma unroll
    for (int b = 0; b < Cfg::TN; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;
}

template <class Cfg>
__device__ __forceinline__ void add_acc(f32x16 (&to)[Cfg::TM][Cfg::TN],
                                        const f32x16 (&acc)[Cfg::TM][Cfg::TN]) {
#pragma unroll
  for (int a = 0; a < Cfg::TM; ++a)
#pragma unroll
    for (int b = 0; b < Cfg::TN; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) to[a][b][r] += acc[a][b][r];
}

// ---------------------------------------------------------------------------------------------
// bf16 operands: global memory -> LDS without registers (global_load_lds_dwordx4).
// ---------------------------------------------------------------------------------------------
// A wavefront's load fills 1 KB of consecutive LDS (16 bytes a lane), so rows cannot be padded;
// what keeps the fragment reads off each other's banks is the order of the 16-byte chunks inside a
// row, chosen by the lane's global address:
//   k contiguous: chunk c of row r lies at position c ^ (r/2 % 8): a fragment read by 16
//                 consecutive rows touches every bank once.
//   k-major:      likewise for units of 64 bytes, so that the four k-rows of one transpose read
//                 fall into different banks.
template <typename T, int R, bool KMAJOR, int SLAB>
struct DmaLds {
  static constexpr int BK = SLAB / (int)sizeof(T);
  static constexpr int ROW_BYTES = KMAJOR ? R * (int)sizeof(T) : SLAB;
  static constexpr int BYTES = (KMAJOR ? BK : R) * ROW_BYTES;
  static constexpr int CPR = ROW_BYTES / 16;
  static_assert(KMAJOR ? ROW_BYTES >= 128 : ROW_BYTES == 128 || ROW_BYTES == 32, "what the order of the chunks is made for");
  // what the position of a chunk of row r is xor-ed with
  static __device__ __forceinline__ int turn(int r) {
    if constexpr (!KMAJOR) return ROW_BYTES == 32 ? (r >> 3) & 1 : (r >> 1) & 7;
    else return (ROW_BYTES >= 256 ? r & 3 : (r >> 1) & 1) * 4;
  }
};

// 16 bytes a lane from `base` (wave-uniform) + toff to 1 KB of LDS at byte `lds`.
// Assembly, because the compiler makes every LDS read that follows the builtin wait for all loads
// in flight.  The load has no output register.  Its write to LDS is done when dma_wait_barrier is
// behind it: whoever reads the region waits there first.  The scalar copy of the base: it may come
// straight from v_readfirstlane, and a vector memory instruction that reads an SGPR has to stay
// five wait states behind a VALU write of it, a scalar one none (nor does the load behind that).
// It is also the wait state that M0, which the compiler sets, needs; the compiler does not look
// into assembly for either.  (s_nop 4 in its place: 1024 x 36,024 fused 248 -> 252 us, 2048 x
// 500,000 4022 -> 4053; with the copy even.)
__device__ __forceinline__ void lds_load(const char* base, uint32_t toff, uint32_t lds) {
  const uint64_t at = (uint64_t)base;
  const uint64_t g = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) |
                     (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(at >> 32)) << 32;
  uint64_t at_s;
  asm volatile("s_mov_b64 %0, %3\n\tglobal_load_lds_dwordx4 %2, %0"
               : "=&s"(at_s)
               : "{m0}"(__builtin_amdgcn_readfirstlane(lds)), "v"(toff), "s"(g)
               : "memory");
}

// E (bf16) lies in octets of classes: entry (sample i, class j) at (j / 8 * Bp + i) * 8 + j % 8, Bp
// samples to a panel.  What a wavefront of the logits holds is 8 classes of 32 samples each, 512 bytes
// that go out in one piece without a way through LDS (gemm_logits).  An operand slab of it is cut
// into panels likewise, each a run of 16-byte entries (fragment reads and loads touch whole lines):
//   k contiguous (dfeatures): the BK / 8 octets of the slab, each R samples;
//   k-major (dweight): the octets of the slab's R classes, each BK samples; sample k of panel o lies at
//                      position k ^ (o % 4 * 4), so that a transpose read finds the four panels and the
//                      four samples of every 32 lanes in different banks.
// Against rows of classes, written through LDS (us): logits 1024 x 205,991 x 512 280 -> 260, 1024 x
// 360,232 494 -> 463, 1024 x 36,024 55.8 -> 50.8, 16,384 x 3,592 104 -> 95; both backward products
// 413 -> 409, 715 -> 684, fused 1024 x 36,024 133.9 -> 131.2, 16,384 x 3,592 115 -> 117: they read more
// (1024 x 205,991 1,272 -> 1,371 MB), which is not for the panels' beginning at the same place of every
// cache (with Bp + 16 samples to a panel 1,361).  (Reading dfeatures' slabs into LDS rows of 8 octets, a
// line for 8 samples from each of 8 panels in one load: both products of 512 x 9,344 20.4 -> 22.9.)
template <typename T, int R, bool KMAJOR, int SLAB>
struct OctetLds {
  static constexpr int BK = SLAB / (int)sizeof(T), SAMPLES = KMAJOR ? BK : R, PANEL = SAMPLES * 16;
  static constexpr int BYTES = (KMAJOR ? R : BK) / 8 * PANEL;
  static_assert(BK % 16 == 0 && R % 32 == 0, "order of the samples");
  static __device__ __forceinline__ int turn(int o) { return KMAJOR ? (o & 3) * 4 : 0; }
};

template <typename T, class L, int THREADS, bool KMAJOR, bool OCTETS>
struct DmaStager {
  static constexpr int NCH = L::BYTES / 16 / THREADS;        // loads per wavefront and slab
  static_assert(NCH >= 1 && L::BYTES % (THREADS * 16) == 0, "slab must divide evenly");
  const char* base;   // wave-uniform: first byte of the operand tile at the first k of the range
  uint32_t toff;      // this lane's byte offset from there
  int64_t pass, slab; // global byte steps between a lane's loads of one slab / between slabs (uniform)

  // ld: elements from row to row; OCTETS: samples to a panel
  __device__ __forceinline__ void init(const T* tile, int64_t ld) {
    const int t = threadIdx.x;
    base = reinterpret_cast<const char*>(tile);
    if constexpr (OCTETS) {
      constexpr int PPP = THREADS / L::SAMPLES;   // panels that one load of every wavefront fills
      static_assert(PPP >= 1 && THREADS % L::SAMPLES == 0 && (!KMAJOR || PPP % 4 == 0),
                    "one order of the samples for all loads of a lane");
      const int o = t / L::SAMPLES, k = (t % L::SAMPLES) ^ L::turn(o);
      toff = (uint32_t)(((int64_t)o * ld + k) * 16);
      pass = PPP * ld * 16;
      slab = KMAJOR ? (int64_t)L::BK * 16 : L::BK / 8 * ld * 16;
    } else {
      constexpr int RPP = THREADS * 16 / L::ROW_BYTES;    // LDS rows that one load of every wavefront fills
      static_assert(RPP % (KMAJOR ? 4 : 16) == 0, "one order of the chunks for all loads of a lane");
      const int row = t / L::CPR, ch = (t % L::CPR) ^ L::turn(row);
      toff = (uint32_t)((int64_t)row * ld * (int64_t)sizeof(T) + ch * 16);
      pass = (int64_t)RPP * ld * (int64_t)sizeof(T);
      slab = KMAJOR ? (int64_t)L::BK * ld * (int64_t)sizeof(T) : (int64_t)L::BK * (int64_t)sizeof(T);
    }
  }
  // Load p of slab s into the LDS region at byte `lds` (this wavefront's first byte there).
  __device__ __forceinline__ void load(int s, int p, uint32_t lds) const {
    lds_load(base + (int64_t)s * slab + p * pass, toff, lds + p * THREADS * 16);
  }
};

// Waits until at most N of this wavefront's loads are in flight and its LDS reads are back, then
// meets the workgroup: what all wavefronts have loaded before is in LDS, what they have read may be
// overwritten.
template <int N>
__device__ __forceinline__ void dma_wait_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// Byte offsets of this lane's fragment reads in an operand slab.
template <class L, bool KMAJOR, bool OCTETS, int GROUPS, int NB>
struct FragAddr;
template <class L, int GROUPS, int NB>
struct FragAddr<L, false, false, GROUPS, NB> {
  uint32_t a[GROUPS];   // of each reduction group; blocks of 32 rows follow at constant distances
  __device__ __forceinline__ void init(int r0) {
    const int lane = threadIdx.x & 63, row = r0 + (lane & 31);
#pragma unroll
    for (int g = 0; g < GROUPS; ++g) a[g] = row * L::ROW_BYTES + (((g * 2 + (lane >> 5)) ^ L::turn(row)) * 16);
  }
  __device__ __forceinline__ u32x4 read(const char* region, int b, int g) const {
    return *reinterpret_cast<const u32x4*>(region + a[g] + b * 32 * L::ROW_BYTES);
  }
};
template <class L, int GROUPS, int NB>
struct FragAddr<L, true, false, GROUPS, NB> {
  uint32_t a[NB];       // of each block of 32 rows; groups follow at constant distances
  __device__ __forceinline__ void init(int r0) {
    // ds_read_b64_tr_b16: inside each group of 16 lanes, lane s addresses the 4 consecutive tile
    // rows r0' + 4*(s%4).. of reduction step k0 + s/4, and lane i receives tile row r0' + i for
    // the 4 steps k0..k0+3.  Lane groups: (rows 0..15 | 16..31) x (first | second half of the group).
    const int lane = threadIdx.x & 63, grp = lane >> 4, s = lane & 15;
    const int k0 = (grp >> 1) * 8 + (s >> 2);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int byte = (r0 + b * 32 + (grp & 1) * 16 + (s & 3) * 4) * 2;
      a[b] = k0 * L::ROW_BYTES + (((byte >> 4) ^ L::turn(k0)) << 4) + (byte & 15);
    }
  }
  __device__ __forceinline__ u32x4 read(const char* region, int b, int g) const {
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    const char* p = region + a[b] + g * 16 * L::ROW_BYTES;
    // (four k-rows further the order of the chunks is the same)
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * L::ROW_BYTES));
    const u32x2 l2 = __builtin_bit_cast(u32x2, lo), h2 = __builtin_bit_cast(u32x2, hi);
    u32x4 r;
    r[0] = l2[0]; r[1] = l2[1]; r[2] = h2[0]; r[3] = h2[1];
    return r;
  }
};

template <class L, int GROUPS, int NB>
struct FragAddr<L, false, true, GROUPS, NB> {
  uint32_t a;   // groups and blocks of 32 rows follow at constant distances
  __device__ __forceinline__ void init(int r0) {
    const int lane = threadIdx.x & 63;
    a = (lane >> 5) * L::PANEL + (r0 + (lane & 31)) * 16;
  }
  __device__ __forceinline__ u32x4 read(const char* region, int b, int g) const {
    return *reinterpret_cast<const u32x4*>(region + a + g * 2 * L::PANEL + b * 512);
  }
};
template <class L, int GROUPS, int NB>
struct FragAddr<L, true, true, GROUPS, NB> {
  uint32_t a[2];   // of the four steps of either read; groups and blocks of 32 rows follow at constant distances
  __device__ __forceinline__ void init(int r0) {
    // lanes as above
    const int lane = threadIdx.x & 63, grp = lane >> 4, s = lane & 15;
    const int k0 = (grp >> 1) * 8 + (s >> 2), r = r0 + (grp & 1) * 16 + (s & 3) * 4, o = r >> 3;
#pragma unroll
    for (int u = 0; u < 2; ++u) a[u] = o * L::PANEL + ((k0 + 4 * u) ^ L::turn(o)) * 16 + (r & 4) * 2;
  }
  __device__ __forceinline__ u32x4 read(const char* region, int b, int g) const {
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    const char* p = region + b * 4 * L::PANEL + g * 256;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + a[0]));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + a[1]));
    const u32x2 l2 = __builtin_bit_cast(u32x2, lo), h2 = __builtin_bit_cast(u32x2, hi);
    u32x4 r;
    r[0] = l2[0]; r[1] = l2[1]; r[2] = h2[0]; r[3] = h2[1];
    return r;
  }
};

// gemm_tile (below) for bf16 operands.  LDS holds ABUF slabs of A and BBUF of B:
//   * the barrier in front of the last group of slab s frees its buffers (all fragments are read by
//     then) and publishes slab s+1; behind it B of slab s+BBUF and A of slab s+ABUF are requested,
//     one load between two MFMAs, so a load has BBUF - 1 (A: ABUF - 1) whole slabs of MFMAs to
//     arrive;
//   * fragments are read one group ahead, the last group is multiplied behind the barrier.
// Against staging through registers (two stages of 64 steps, 8 ds_write_b128 a wavefront and slab),
// both in turn, us: logits 1024 x 205,991 x 512 296 -> 276, both backward products there 450 ->
// 401, 1024 x 360,232 766 -> 690, 16,384 x 3,592 125 -> 113; products alone, 256 tiles of 256 x 256
// over 6,400 steps, 1.00 - 1.17 -> 1.28 - 1.36 PFLOP/s (both k contiguous), 1.03 -> 1.21 (both
// k-major), 0.97 -> 1.07 (dfeatures).  What bounds it now, by counters and variants of the loop:
// both k contiguous, the matrix cores are busy 82 % of the cycles at 1.46 GHz, the clock that the
// power leaves; with operands from HBM (dfeatures: 57 % at 1.76 GHz) the loads are: when all compute
// units read, one's share of the fabric is 23 - 29 GB/s (requesting lines of later slabs by one of
// the workgroups that share them: 17 % slower).  Without loads and fragment reads in the loop both
// products of 1024 x 205,991 x 512 take 317 us instead of 415.
template <class Cfg>
__device__ __forceinline__ void gemm_tile_dma(const typename Cfg::elem* __restrict__ A, int64_t lda,
                                              const typename Cfg::elem* __restrict__ B, int64_t ldb, int nslabs,
                                              char* smem, f32x16 (&acc)[Cfg::TM][Cfg::TN]) {
  using T = typename Cfg::elem;
  typedef std::conditional_t<Cfg::A_OCTETS, OctetLds<T, Cfg::BM, Cfg::A_KMAJOR, Cfg::SLAB_BYTES>,
                             DmaLds<T, Cfg::BM, Cfg::A_KMAJOR, Cfg::SLAB_BYTES>> LA;
  typedef DmaLds<T, Cfg::BN, Cfg::B_KMAJOR, Cfg::SLAB_BYTES> LB;
  constexpr int ABUF = Cfg::ABUF, BBUF = Cfg::BBUF;
  static_assert(ABUF == BBUF || ABUF == BBUF + 1, "the counts of loads in flight");
  typedef DmaStager<T, LA, Cfg::THREADS, Cfg::A_KMAJOR, Cfg::A_OCTETS> SA;
  typedef DmaStager<T, LB, Cfg::THREADS, Cfg::B_KMAJOR, false> SB;
  constexpr int NA = SA::NCH, NB = SB::NCH, MM = Cfg::TM * Cfg::TN, HEAD = Cfg::GROUPS - 1;
  // loads that may be in flight when slab s+1 (or slab 0) has to be there, nothing being left out
  // at the end
  constexpr int FLY = ABUF == BBUF ? (BBUF - 2) * (NA + NB) : (BBUF - 1) * NA + (BBUF - 2) * NB;
  constexpr int FLY0 = (BBUF - 1) * (NA + NB) + (ABUF - BBUF) * NA;
  const int wave = threadIdx.x >> 6;
  const int wm = wave / Cfg::WN, wn = wave % Cfg::WN;
  SA sa;
  SB sb;
  sa.init(A, lda);
  sb.init(B, ldb);
  FragAddr<LA, Cfg::A_KMAJOR, Cfg::A_OCTETS, Cfg::GROUPS, Cfg::TM> ra;
  FragAddr<LB, Cfg::B_KMAJOR, false, Cfg::GROUPS, Cfg::TN> rb;
  ra.init(wm * Cfg::WTM);
  rb.init(wn * Cfg::WTN);
  constexpr uint32_t B0 = ABUF * LA::BYTES;   // the B buffers lie behind those of A
  const uint32_t lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem +
                       __builtin_amdgcn_readfirstlane(wave) * 1024;
  const int last = nslabs - 1;
  auto load_a = [&](int s, int p, uint32_t buf) { sa.load(s, p, lds + buf); };
  auto load_b = [&](int s, int p, uint32_t buf) { sb.load(s, p, lds + B0 + buf); };
#pragma unroll
  for (int u = 0; u < ABUF; ++u) {
    if (u > last) break;
    if (u < BBUF) {
#pragma unroll
      for (int p = 0; p < NB; ++p) load_b(u, p, u * LB::BYTES);
    }
#pragma unroll
    for (int p = 0; p < NA; ++p) load_a(u, p, u * LA::BYTES);
  }
  if (last >= ABUF - 1) dma_wait_barrier<FLY0>();
  else dma_wait_barrier<0>();

  Frags<Cfg> fc;
  auto read = [&](uint32_t abuf, uint32_t bbuf, int g, Frags<Cfg>& f) {
#pragma unroll
    for (int b = 0; b < Cfg::TM; ++b) f.a[b] = ra.read(smem + abuf, b, g);
#pragma unroll
    for (int b = 0; b < Cfg::TN; ++b) f.b[b] = rb.read(smem + B0 + bbuf, b, g);
  };
  read(0, 0, 0, fc);
  uint32_t ab = 0, bb = 0, ab_before = 0;   // buffers of slab s; that of A of slab s-1
  for (int s = 0; s <= last; ++s) {
    const bool more_a = s > 0 && s - 1 + ABUF <= last, more_b = s + BBUF <= last;
#pragma unroll
    for (int g = 0; g < HEAD; ++g) {
      Frags<Cfg> fn;
      read(ab, bb, g + 1, fn);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < MM; ++q) {
        if (g == 0) {
#pragma unroll
          for (int c = 0; c < NA; ++c)
            if (c * MM / NA == q && more_a) load_a(s - 1 + ABUF, c, ab_before);
        }
        mfma_bf16(fc.a[q / Cfg::TN], fc.b[q % Cfg::TN], acc[q / Cfg::TN][q % Cfg::TN]);
      }
      __builtin_amdgcn_sched_barrier(0);
      fc = fn;
    }
    if (s - 1 + ABUF <= last) dma_wait_barrier<FLY>();
    else dma_wait_barrier<0>();
    ab_before = ab;
    const uint32_t bb_before = bb;
    ab = ab == (ABUF - 1) * LA::BYTES ? 0 : ab + LA::BYTES;
    bb = bb == (BBUF - 1) * LB::BYTES ? 0 : bb + LB::BYTES;
    Frags<Cfg> fn;
    read(ab, bb, 0, fn);   // (behind the last slab: a buffer's old contents, not used)
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < MM; ++q) {
#pragma unroll
      for (int c = 0; c < NB; ++c)
        if (c * MM / NB == q && more_b) load_b(s + BBUF, c, bb_before);
      mfma_bf16(fc.a[q / Cfg::TN], fc.b[q % Cfg::TN], acc[q / Cfg::TN][q % Cfg::TN]);
    }
    __builtin_amdgcn_sched_barrier(0);
    fc = fn;
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------------------------
// fp32 operands, split into planes of 16 bits.
// ---------------------------------------------------------------------------------------------
// x = h + m + l in bf16, each rounded to nearest, so that a plane is at most 2^-9 of the one above.
// That is exact for |x| from 2^-109 to the largest bf16; below, where l gets to the last place of
// bf16's subnormal numbers (which the conversion, the dot and the matrix instruction keep), it is
// off by at most 2^-134.  The operands: normalised rows, exp(z) <= e^64, and Xs = (s / (B l)) xn,
// whose components come to 2^-119 when all of 60,000 centers are next to all of 4096 samples (dWn
// then 2.7e-6 off 64 bits, 2.8e-6 with fp32 MFMAs).  Of the nine products of two values six are
// added up; those left out (m l, l m, l l) come to at most 2^-26.
struct SplitBf16 {
  static constexpr int PLANES = 3, PRODUCTS = 6;
  // h h last: where one product dominates a sum, the accumulator is as large for one rounding of
  // six.  (A product alone off by, rms: 3.1e-8; h h first 5.2e-8; fp32 MFMA 2.5e-8.)
  static constexpr int A[PRODUCTS] = {1, 1, 0, 2, 0, 0}, B[PRODUCTS] = {1, 0, 1, 0, 2, 0};
  // words of one pair of neighbours in the planes; the remainders are exact, the dot instruction
  // takes a plane off without widening it first (x - 1 * h + 0 * h')
  static __device__ __forceinline__ void pair(float a, float b, uint32_t (&w)[PLANES]) {
    // (the constants come from registers: as an inline constant of the instruction, (-1, 0) reads
    // (0, -1))
    uint32_t c_lo = 0x0000bf80u, c_hi = 0xbf800000u;
    asm("" : "+s"(c_lo), "+s"(c_hi));
    const bf16x2 lo = __builtin_bit_cast(bf16x2, c_lo), hi = __builtin_bit_cast(bf16x2, c_hi);
#pragma unroll
    for (int q = 0; q < PLANES; ++q) {
      const bf16x2 v = __builtin_convertvector(f32x2{a, b}, bf16x2);
      w[q] = __builtin_bit_cast(uint32_t, v);
      if (q + 1 < PLANES) {
        a = __builtin_amdgcn_fdot2_f32_bf16(v, lo, a, false);
        b = __builtin_amdgcn_fdot2_f32_bf16(v, hi, b, false);
      }
    }
  }
  static __device__ __forceinline__ void mfma(const u32x4& a, const u32x4& b, f32x16& c) { mfma_bf16(a, b, c); }
};

// f(0th), .., f(last) with the index as a type: the bodies are whole before any loop optimisation.
template <int FROM, class F, int... I>
__device__ __forceinline__ void static_for_seq(std::integer_sequence<int, I...>, F f) {
  (f(std::integral_constant<int, FROM + I>{}), ...);
}
template <int FROM, int TO, class F>
__device__ __forceinline__ void static_for(F f) {
  static_for_seq<FROM>(std::make_integer_sequence<int, TO - FROM>{}, f);
}
// Pieces in front of product q when n of them are spread over `span` products from q0 on.
constexpr int pieces_before(int q, int q0, int span, int n) {
  const int p = q <= q0 ? 0 : ((q - q0) * n + span - 1) / span;
  return p < n ? p : n;
}

// 8 neighbouring values of an operand that a thread splits in every slab.
struct SplitChunk {
  const float* src;     // at slab 0
  int64_t step;         // floats from slab to slab
  uint32_t dst, plane;  // LDS byte offset in a stage, and from plane to plane
};
template <class L, bool KMAJOR>
__device__ __forceinline__ SplitChunk split_chunk(int c, const float* base, int64_t ld, uint32_t region) {
  const int row = c / L::CPR, ch = c % L::CPR;
  return {base + row * ld + ch * 8, KMAJOR ? 16 * ld : 16, region + row * L::ROW_BYTES + ((ch ^ L::turn(row)) * 16),
          L::BYTES};
}

// gemm_tile (below) for the fp32 operands of the backward products.  LDS holds two stages of 16
// reduction steps, each the planes of both operands (layout: DmaLds).  Every thread loads 8
// neighbouring values of an operand, one slab or more ahead, splits them between the MFMAs of the
// slab at hand and stores one 16-byte chunk to each plane of the other stage; the last product of a
// slab is added up behind the barrier, under the first fragment reads of the next one.  What it
// replaces: v_mfma_f32_32x32x2_f32, whose rate (157 TFLOP/s nominal) was the bound at any tile
// size; six bf16 products are 2.7 times that.  Step, us, before -> now: 512 x 9,344 x 512 199 ->
// 181, 300 x 40,000 x 512 736 -> 608, 1024 x 36,024 x 512 with the update 1211 -> 1003, 500 x 4,000
// x 1024 173 -> 154, 128 x 1,000 x 512 even (latency).  Error against 64 bits (2-norm, features |
// centers off the labels), fp32 products -> now.  Scale 64, most of it the logits': 512 x 9,344 x
// 512 6.43e-7 -> 6.41e-7 | 3.07e-6 -> 3.06e-6, 2048 x 16,000 x 512 5.76e-7 -> 5.75e-7 | 3.05e-6 ->
// 3.04e-6, 4096 x 20,000 x 512 5.69e-7 -> 5.60e-7 | 3.01e-6 -> 2.98e-6.  Scale 1, centers, most of
// it the sums': 4.2e-7 -> 3.4e-7, 4.2e-7 -> 3.5e-7, 5.9e-7 -> 5.0e-7: an accumulator takes 6
// roundings for 16 products instead of 8.  What bounds it: large problems the clock that the power
// leaves (1.1 PFLOP/s of 16-bit products), small ones the way from global memory through registers
// and LDS to the fragments in every slab.
template <class Cfg, int CHAIN>
__device__ __forceinline__ void gemm_tile_split(const float* __restrict__ A, int64_t lda,
                                                const float* __restrict__ B, int64_t ldb, int nslabs, char* smem,
                                                f32x16 (&acc)[Cfg::TM][Cfg::TN]) {
  typedef DmaLds<__bf16, Cfg::BM, Cfg::A_KMAJOR, 32> LA;   // a plane of 16 reduction steps
  typedef DmaLds<__bf16, Cfg::BN, Cfg::B_KMAJOR, 32> LB;
  typedef SplitBf16 S;
  constexpr int NP = S::PLANES, NPR = S::PRODUCTS;
  constexpr int STAGE = NP * (LA::BYTES + LB::BYTES), B0 = NP * LA::BYTES;
  constexpr int CA = LA::BYTES / 16, CB = LB::BYTES / 16, THREADS = Cfg::THREADS;
  constexpr int NPT = (CA + CB + THREADS - 1) / THREADS;   // chunks of 8 values per thread and slab
  static_assert(CA % 64 == 0 && CB % 64 == 0, "a wavefront's chunks are of one operand");
  constexpr int MM = Cfg::TM * Cfg::TN;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / Cfg::WN, wn = wave % Cfg::WN;
  FragAddr<LA, Cfg::A_KMAJOR, false, 1, Cfg::TM> ra;
  FragAddr<LB, Cfg::B_KMAJOR, false, 1, Cfg::TN> rb;
  ra.init(wm * Cfg::WTM);
  rb.init(wn * Cfg::WTN);
  // this thread's chunks: those of A first
  SplitChunk ch[NPT];
  bool has[NPT];
#pragma unroll
  for (int p = 0; p < NPT; ++p) {
    const int first = wave * 64 + p * THREADS, id = first + (threadIdx.x & 63);
    has[p] = first < CA + CB;
    if (first < CA) ch[p] = split_chunk<LA, Cfg::A_KMAJOR>(id, A, lda, 0);
    else ch[p] = split_chunk<LB, Cfg::B_KMAJOR>(has[p] ? id - CA : 0, B, ldb, B0);
  }
  const int last = nslabs * (Cfg::BK / 16) - 1;
  // values of the next DEPTH slabs, requested as soon as those before them are split
  constexpr int DEPTH = THREADS == 256 ? 4 : 1;   // (128-tiles: the registers of a second workgroup)
  f32x4 x[DEPTH][NPT][2];
  auto load = [&](int s, int u) __attribute__((always_inline)) {
#pragma unroll
    for (int p = 0; p < NPT; ++p) {
      if (NPT * THREADS > CA + CB && !has[p]) continue;
      x[u][p][0] = *reinterpret_cast<const f32x4*>(ch[p].src + s * ch[p].step);
      x[u][p][1] = *reinterpret_cast<const f32x4*>(ch[p].src + s * ch[p].step + 4);
    }
  };
  u32x4 w[NPT][NP];
  // pair i of this thread's chunks; the last of a chunk stores it to the stage
  auto split = [&](int i, int u, char* stage) __attribute__((always_inline)) {
    const int p = i / 4, e = i % 4;
    uint32_t v[NP];
    S::pair(x[u][p][e / 2][e % 2 * 2], x[u][p][e / 2][e % 2 * 2 + 1], v);
#pragma unroll
    for (int q = 0; q < NP; ++q) w[p][q][e] = v[q];
    if (e == 3) {
      if (NPT * THREADS > CA + CB && !has[p]) return;
#pragma unroll
      for (int q = 0; q < NP; ++q) *reinterpret_cast<u32x4*>(stage + ch[p].dst + q * ch[p].plane) = w[p][q];
    }
  };
  u32x4 a[NP][Cfg::TM], b[NP][Cfg::TN];
  auto read_a = [&](const char* stage, int q, u32x4 (&f)[Cfg::TM]) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < Cfg::TM; ++t) f[t] = ra.read(stage + q * LA::BYTES, t, 0);
  };
  auto read_b = [&](const char* stage, int q, u32x4 (&f)[Cfg::TN]) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < Cfg::TN; ++t) f[t] = rb.read(stage + B0 + q * LB::BYTES, t, 0);
  };
  load(0, 0);
#pragma unroll
  for (int u = 1; u < DEPTH; ++u) load(u < last ? u : last, u);
#pragma unroll
  for (int i = 0; i < 4 * NPT; ++i) split(i, 0, smem);
  load(DEPTH < last ? DEPTH : last, 0);
  __syncthreads();
  read_a(smem, 1, a[1]);
  read_b(smem, 1, b[1]);
  f32x16 sums[Cfg::TM][Cfg::TN];
  if constexpr (CHAIN > 0) zero_acc<Cfg>(sums);
  for (int s0 = 0; s0 <= last; s0 += DEPTH) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
      const int s = s0 + d, u = (d + 1) % DEPTH;   // set of slab s+1
      if (s > last) break;
      char* cur = smem + (s & 1) * STAGE;
      char* nxt = smem + (~s & 1) * STAGE;
      read_b(cur, 0, b[0]);   // in the order that the products need them
      read_a(cur, 0, a[0]);
      read_a(cur, 2, a[2]);
      read_b(cur, 2, b[2]);
      __builtin_amdgcn_sched_barrier(0);
      // between the products of this slab the values of the next one are split, from the second on
      constexpr int Q = (NPR - 1) * MM, Q0 = MM, SPAN = 3 * MM;
      static_for<0, Q>([&](auto qc) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value, t = q % MM, o = q / MM;
        constexpr int from = pieces_before(q, Q0, SPAN, 4 * NPT), to = pieces_before(q + 1, Q0, SPAN, 4 * NPT);
        static_for<from, to>([&](auto i) __attribute__((always_inline)) { split(decltype(i)::value, u, nxt); });
        if constexpr (q == Q0 + SPAN) load(s + 1 + DEPTH < last ? s + 1 + DEPTH : last, u);
        S::mfma(a[S::A[o]][t / Cfg::TN], b[S::B[o]][t % Cfg::TN], acc[t / Cfg::TN][t % Cfg::TN]);
        __builtin_amdgcn_sched_barrier(0);
      });
      __syncthreads();
      u32x4 an[Cfg::TM], bn[Cfg::TN];
      read_a(nxt, 1, an);
      read_b(nxt, 1, bn);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int t = 0; t < MM; ++t)
        S::mfma(a[S::A[NPR - 1]][t / Cfg::TN], b[S::B[NPR - 1]][t % Cfg::TN], acc[t / Cfg::TN][t % Cfg::TN]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int t = 0; t < Cfg::TM; ++t) a[1][t] = an[t];
#pragma unroll
      for (int t = 0; t < Cfg::TN; ++t) b[1][t] = bn[t];
      if constexpr (CHAIN > 0) {
        if ((s + 1) % (CHAIN * Cfg::BK / 16) == 0 && s < last) {
          add_acc<Cfg>(sums, acc);
          zero_acc<Cfg>(acc);
        }
      }
    }
  }
  if constexpr (CHAIN > 0) add_acc<Cfg>(acc, sums);
  __syncthreads();
}

// ---------------------------------------------------------------------------------------------
// fp32 operands of the logits: both k contiguous, multiplied by v_mfma_f32_32x32x2_f32.
// ---------------------------------------------------------------------------------------------
// Operand slab in LDS: R rows of SLAB bytes, padded so that the fragment reads of 32 rows miss each
// other's banks.
template <int R, int SLAB>
struct PlainLds {
  static constexpr int STRIDE = SLAB + 16, BYTES = R * STRIDE;
  static constexpr int CPR = SLAB / 16, CHUNKS = R * CPR;
};

// Global -> register -> LDS staging of one slab.  Thread t owns chunk t % CPR of rows t / CPR + p *
// RPP, p = 0 .. NCH-1.  A wave-uniform base (tile, slab, pass) and one 32-bit offset per thread
// keep addresses out of the vector registers.
template <class L, int THREADS, int SLAB>
struct PlainStager {
  static constexpr int RPP = THREADS / L::CPR, NCH = L::CHUNKS / THREADS;
  static_assert(L::CHUNKS % THREADS == 0 && THREADS % L::CPR == 0, "whole rows in every pass");
  const char* base;
  uint32_t toff;
  int64_t pass;
  int lds;
  // one vector value, so that they are registers whatever the control flow around the loads
  typedef uint32_t Regs __attribute__((ext_vector_type(NCH * 4)));
  __device__ __forceinline__ void init(const float* tile, int64_t ld) {
    const int row = threadIdx.x / L::CPR, ch = threadIdx.x % L::CPR;
    base = reinterpret_cast<const char*>(tile);
    toff = (uint32_t)((int64_t)row * ld * 4 + ch * 16);
    pass = (int64_t)RPP * ld * 4;
    lds = row * L::STRIDE + ch * 16;
  }
  __device__ __forceinline__ void load(int s, int p, Regs& r) const {
    const u32x4 t = *reinterpret_cast<const u32x4*>(base + (int64_t)s * SLAB + p * pass + toff);
#pragma unroll
    for (int e = 0; e < 4; ++e) r[4 * p + e] = t[e];
  }
  __device__ __forceinline__ void store(char* region, const Regs& r) const {
#pragma unroll
    for (int p = 0; p < NCH; ++p) {
      u32x4 t;
#pragma unroll
      for (int e = 0; e < 4; ++e) t[e] = r[4 * p + e];
      *reinterpret_cast<u32x4*>(region + lds + p * RPP * L::STRIDE) = t;
    }
  }
};

// gemm_tile (below) for the fp32 operands of the logits: two stages in LDS, one set of registers,
// loads two slabs ahead, issued one at a time between the MFMAs of the first groups; fragments are
// read a group ahead; the last group of a slab is multiplied behind the barrier.  Slab numbers past
// the end are clamped: such loads and stores are redundant.  Why not in 16-bit planes, as the
// backward products: two fp16 planes and three products are as close to 64 bits (a cosine 6e-8 off
// instead of 2e-7) and take 22 of 60 us less at 512 x 9,344 x 512, but what a confident sample
// passes on is p - 1, the rounding of a sum and a quotient next to 1 multiplied by the scale: with
// other roundings of its cosines the gradients of samples aligned to their centers move by 1e-5 ..
// 1e-4 of their 2-norm, as far as they are off from 64 bits either way, and more than a change of
// the summation order may move them.
template <class Cfg>
__device__ __forceinline__ void gemm_tile_fp32(const float* __restrict__ A, int64_t lda, const float* __restrict__ B,
                                               int64_t ldb, int nslabs, char* smem,
                                               f32x16 (&acc)[Cfg::TM][Cfg::TN]) {
  constexpr int SLAB = Cfg::SLAB_BYTES;
  typedef PlainLds<Cfg::BM, SLAB> LA;
  typedef PlainLds<Cfg::BN, SLAB> LB;
  typedef PlainStager<LA, Cfg::THREADS, SLAB> SA;
  typedef PlainStager<LB, Cfg::THREADS, SLAB> SB;
  constexpr int STAGE = LA::BYTES + LB::BYTES;
  constexpr int NA = SA::NCH, NB = SB::NCH, NL = NA + NB, MM = Cfg::TM * Cfg::TN, HEAD = Cfg::GROUPS - 1;
  // the loads of a slab are placed in front of the MFMAs of the first one or two groups (of all
  // groups before the barrier if two do not have an MFMA for each load)
  constexpr int SPAN = (NL <= 2 * MM ? (HEAD < 2 ? HEAD : 2) : HEAD) * MM;
  static_assert(HEAD >= 1, "the last group is multiplied behind the barrier");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int ra = ((wave / Cfg::WN) * Cfg::WTM + (lane & 31)) * LA::STRIDE + (lane >> 5) * 16;
  const int rb = LA::BYTES + ((wave % Cfg::WN) * Cfg::WTN + (lane & 31)) * LB::STRIDE + (lane >> 5) * 16;
  auto read = [&](const char* stage, int g, Frags<Cfg>& f) __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < Cfg::TM; ++b)
      f.a[b] = *reinterpret_cast<const u32x4*>(stage + ra + b * 32 * LA::STRIDE + g * 32);
#pragma unroll
    for (int b = 0; b < Cfg::TN; ++b)
      f.b[b] = *reinterpret_cast<const u32x4*>(stage + rb + b * 32 * LB::STRIDE + g * 32);
  };
  // 8 reduction steps: four instructions, the t-th of which pairs element t of every lane
  auto multiply = [&](const Frags<Cfg>& f, int q) __attribute__((always_inline)) {
    // whole-vector casts: a bit_cast applied to a single vector element reads element 0
    const f32x4 a = __builtin_bit_cast(f32x4, f.a[q / Cfg::TN]), b = __builtin_bit_cast(f32x4, f.b[q % Cfg::TN]);
    f32x16& c = acc[q / Cfg::TN][q % Cfg::TN];
#pragma unroll
    for (int t = 0; t < 4; ++t) c = __builtin_amdgcn_mfma_f32_32x32x2f32(a[t], b[t], c, 0, 0, 0);
  };
  SA sa;
  SB sb;
  sa.init(A, lda);
  sb.init(B, ldb);
  const int last = nslabs - 1;
  typename SA::Regs a0 = {};
  typename SB::Regs b0 = {};
  {
    typename SA::Regs af = {};
    typename SB::Regs bf = {};
    const int next = last < 1 ? last : 1;
#pragma unroll
    for (int p = 0; p < NA; ++p) sa.load(0, p, af);
#pragma unroll
    for (int p = 0; p < NB; ++p) sb.load(0, p, bf);
#pragma unroll
    for (int p = 0; p < NA; ++p) sa.load(next, p, a0);
#pragma unroll
    for (int p = 0; p < NB; ++p) sb.load(next, p, b0);
    sa.store(smem, af);
    sb.store(smem + LA::BYTES, bf);
  }
  __syncthreads();
  Frags<Cfg> fc;
  read(smem, 0, fc);
  for (int s = 0; s < nslabs; ++s) {
    char* cur = smem + (s & 1) * STAGE;
    char* nxt = smem + (~s & 1) * STAGE;
    const int s2 = s + 2 < last ? s + 2 : last;
    sa.store(nxt, a0);
    sb.store(nxt + LA::BYTES, b0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int g = 0; g < HEAD; ++g) {
      Frags<Cfg> fn;
      read(cur, g + 1, fn);
      __builtin_amdgcn_sched_barrier(0);   // keep the reads ahead of the MFMAs they do not feed
#pragma unroll
      for (int q = 0; q < MM; ++q) {
#pragma unroll
        for (int c = 0; c < NL; ++c)       // chunk c is requested in front of block c * SPAN / NL
          if (c * SPAN / NL == g * MM + q) {
            if (c < NA) sa.load(s2, c, a0);
            else sb.load(s2, c - NA, b0);
          }
        multiply(fc, q);
      }
      __builtin_amdgcn_sched_barrier(0);
      fc = fn;
    }
    __syncthreads();
    Frags<Cfg> fn;
    read(nxt, 0, fn);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < MM; ++q) multiply(fc, q);
    __builtin_amdgcn_sched_barrier(0);
    fc = fn;
  }
  __syncthreads();
}

// Accumulate acc += A_tile * B_tile^T over `nslabs` slabs of K.
//   A: element (first of this workgroup's BM tile rows, first reduction step of its range)
//   B: likewise for its BN tile rows;  lda / ldb in elements (A in octets: lda samples to a panel).
//   smem: Cfg::LDS_BYTES bytes, 16-byte aligned.  Ends with a barrier (smem may be reused).
// CHAIN > 0 (fp32): every CHAIN slabs the accumulators are added to a second set and start again from
// zero, so that no sum is a chain of more than CHAIN * BK products.
template <class Cfg, int CHAIN = 0>
__device__ __forceinline__ void gemm_tile(const typename Cfg::elem* __restrict__ A, int64_t lda,
                                          const typename Cfg::elem* __restrict__ B, int64_t ldb,
                                          int nslabs, char* smem,
                                          f32x16 (&acc)[Cfg::TM][Cfg::TN]) {
  static_assert(CHAIN == 0 || !Cfg::DMA, "bf16 operands: their rounding is what counts");
  if constexpr (Cfg::DMA) gemm_tile_dma<Cfg>(A, lda, B, ldb, nslabs, smem, acc);
  else if constexpr (Cfg::SPLIT) gemm_tile_split<Cfg, CHAIN>(A, lda, B, ldb, nslabs, smem, acc);
  else gemm_tile_fp32<Cfg>(A, lda, B, ldb, nslabs, smem, acc);
}

// Row / column of accumulator register r of block (bm, bn) inside the workgroup tile.
template <class Cfg>
__device__ __forceinline__ int acc_row(int bm, int r) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  return (wave / Cfg::WN) * Cfg::WTM + bm * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
}
template <class Cfg>
__device__ __forceinline__ int acc_col(int bn) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  return (wave % Cfg::WN) * Cfg::WTN + bn * 32 + (lane & 31);
}

// XCD-aware order of workgroups: consecutive workgroup ids are dealt round-robin to the 8 XCDs
// (each with its own L2), so the `inner` workgroups that share an operand tile are given ids
// that land on one XCD.  This is done for the outer indices that form whole groups of 8; the
// remaining outer % 8 (all of them when outer < 8) are laid out plainly, inner index fastest, so
// that their workgroups spread over all XCDs instead of filling outer % 8 of them.  The grid is
// exactly inner * outer workgroups; returns false for ids beyond it.
__device__ __forceinline__ bool xcd_tile(int wg, int inner, int outer, int& o, int& i) {
  const int full = outer & ~7;
  if (wg < full * inner) {
    const int xcd = wg & 7, local = wg >> 3;
    o = (local / inner) * 8 + xcd;
    i = local % inner;
  } else {
    const int t = wg - full * inner;
    o = full + t / inner;
    i = t % inner;
  }
  return o < outer;
}
inline int xcd_grid(int inner, int outer) { return inner * outer; }

}  // namespace pfc
