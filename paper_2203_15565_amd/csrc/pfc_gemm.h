// MFMA tile engine for the three GEMMs of the PFC step (gfx950).
//
//   logits    C[j][i] = sum_d Wn[j][d] * Xn[i][d]        A = Wn  (k contiguous), B = Xn (k contiguous)
//   dweight   C[j][d] = sum_i E[i][j]  * Xs[i][d]        A = E   (k-major),      B = Xs (k-major)
//   dfeatures C[i][d] = sum_j E[i][j]  * Wn[j][d]        A = E   (k contiguous), B = Wn (k-major)
//
// Every matrix stays in its one natural row-major layout in HBM; an operand whose reduction
// index is its ROW index ("k-major") is staged in LDS as it is and transposed on the way into
// the MFMA registers by the LDS transpose read of gfx950 (ds_read_b64_tr_b16), so no transposed
// copy of E, Wn or Xs is ever written.  Operands are padded with zeros to whole tiles by their
// producers: the main loop has no bounds checks.
//
// A workgroup of WM x WN wavefronts (64 lanes each) owns a BM x BN tile of C.  K is walked in
// slabs of BK = 64 (bf16) or 32 (fp32) reduction steps.  bf16 operands go from global memory to LDS
// without registers (gemm_tile_dma); fp32 operands through registers, double buffered in LDS, slab s+1
// waiting in the second LDS stage and the global loads of slab s+2 in flight while slab s is multiplied.
//
// LDS layouts of one fp32 operand slab (R = BM or BN rows of the operand tile; bf16: DmaLds):
//   k contiguous: R rows of 128 bytes, row stride 144: a 16-byte fragment read by 16 consecutive
//                 rows touches every bank once.
//   k-major:      BK rows of R*sizeof(T) bytes, row stride + 64.
//
// Fragment convention (the same for A and B, which is all a dot product needs): a group of 16
// (bf16) or 8 (fp32) reduction steps is split between the lane halves, lanes 0..31 taking the
// first half and lanes 32..63 the second; for bf16 that is one v_mfma_f32_32x32x16_bf16 per
// group, for fp32 four v_mfma_f32_32x32x2_f32, the t-th of which pairs element t of every lane.
//
// Accumulator layout of a 32x32 block (16 floats per lane): register r of lane l holds
//   row = (r / 4) * 8 + (l / 32) * 4 + (r % 4),  col = l % 32.
#pragma once

#include "pfc_common.h"

namespace pfc {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));


// Geometry of one operand slab in LDS.
// SLAB: bytes of K per operand row per slab (128, or 64 for tiles whose wide operand would not fit).
template <typename T, int R, bool KMAJOR, int SLAB>
struct OperandLds {
  static constexpr int SLAB_BYTES = SLAB;
  static constexpr int BK = SLAB / (int)sizeof(T);
  static constexpr int ROWS = KMAJOR ? BK : R;                                   // LDS rows
  static constexpr int ROW_BYTES = KMAJOR ? R * (int)sizeof(T) : SLAB;     // payload
  static constexpr int STRIDE = ROW_BYTES + (KMAJOR ? 64 : 16);                  // padded
  static constexpr int BYTES = ROWS * STRIDE;
  static constexpr int CHUNKS_PER_ROW = ROW_BYTES / 16;
  static constexpr int CHUNKS = ROWS * CHUNKS_PER_ROW;                           // 16-byte chunks
};

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
  static constexpr int WTM = BM / WM, WTN = BN / WN;       // tile of one wavefront
  static constexpr int TM = WTM / 32, TN = WTN / 32;       // 32x32 blocks per wavefront
  using LA = OperandLds<T, BM, AKM, SLAB>;
  using LB = OperandLds<T, BN, BKM, SLAB>;
  static constexpr int A_BYTES = LA::BYTES, B_BYTES = LB::BYTES;
  static constexpr int STAGE_BYTES = A_BYTES + B_BYTES;
  static constexpr bool DMA = sizeof(T) == 2;
  static constexpr int LDS_BYTES = DMA ? (ABUF * BM + BBUF * BN) * SLAB : 2 * STAGE_BYTES;
  static constexpr int A_CHUNKS = LA::CHUNKS / THREADS;    // 16-byte chunks per thread per slab
  static constexpr int B_CHUNKS = LB::CHUNKS / THREADS;
  static_assert(WTM % 32 == 0 && WTN % 32 == 0, "wave tile must be whole 32x32 blocks");
  static_assert(LA::CHUNKS % THREADS == 0 && LB::CHUNKS % THREADS == 0, "slab must divide evenly");
  static_assert(THREADS % LA::CHUNKS_PER_ROW == 0 && THREADS % LB::CHUNKS_PER_ROW == 0,
                "a staging pass must cover whole LDS rows");
};

template <typename T>
__device__ __forceinline__ void mfma_group(const u32x4& a, const u32x4& b, f32x16& c);

template <>
__device__ __forceinline__ void mfma_group<__bf16>(const u32x4& a, const u32x4& b, f32x16& c) {
  c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                              __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// fp32: elements 2 * HALF and 2 * HALF + 1 of the group.
template <int HALF>
__device__ __forceinline__ void mfma_half(const u32x4& a, const u32x4& b, f32x16& c) {
  // whole-vector casts: a bit_cast applied to a single vector element reads element 0
  const f32x4 af = __builtin_bit_cast(f32x4, a);
  const f32x4 bf = __builtin_bit_cast(f32x4, b);
  c = __builtin_amdgcn_mfma_f32_32x32x2f32(af[2 * HALF], bf[2 * HALF], c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_32x32x2f32(af[2 * HALF + 1], bf[2 * HALF + 1], c, 0, 0, 0);
}

template <>
__device__ __forceinline__ void mfma_group<float>(const u32x4& a, const u32x4& b, f32x16& c) {
  mfma_half<0>(a, b, c);
  mfma_half<1>(a, b, c);
}

// Global -> register -> LDS staging of one operand slab.  Thread t owns chunk (t % CPR) of LDS
// rows (t / CPR) + p * (THREADS / CPR), p = 0 .. NCH-1.  Addresses are a wave-uniform 64-bit
// base (tile, slab, pass) plus one 32-bit per-thread offset, which lets the loads use the
// scalar-base addressing form and keeps address registers out of the vector register budget.
template <typename T, class L, int THREADS, int NCH, bool KMAJOR>
struct Stager {
  const char* base;   // wave-uniform: first byte of the operand tile at the first k of the range
  uint32_t toff;      // this thread's byte offset from the pass base
  int64_t pass;       // global byte step between passes (uniform)
  int64_t slab;       // global byte step between slabs (uniform)
  int lds;            // this thread's first LDS byte offset inside the operand region
  static constexpr int RPP = THREADS / L::CHUNKS_PER_ROW;   // LDS rows per pass

  // tile: element (row 0 of the operand tile, first k of the range); ld in elements.
  __device__ __forceinline__ void init(const T* tile, int64_t ld) {
    const int t = threadIdx.x;
    const int row = t / L::CHUNKS_PER_ROW, ch = t % L::CHUNKS_PER_ROW;
    // k contiguous: LDS row = tile row, advancing a slab moves 128 bytes along the row.
    // k-major:      LDS row = reduction step, advancing a slab moves BK rows down.
    base = reinterpret_cast<const char*>(tile);
    toff = (uint32_t)((int64_t)row * ld * (int64_t)sizeof(T) + ch * 16);
    pass = (int64_t)RPP * ld * (int64_t)sizeof(T);
    slab = KMAJOR ? (int64_t)L::BK * ld * (int64_t)sizeof(T) : (int64_t)L::SLAB_BYTES;
    lds = row * L::STRIDE + ch * 16;
  }
  // The chunks of one slab live in ONE vector value (not an array), so they are registers by
  // construction whatever the control flow around the loads.
  typedef uint32_t Regs __attribute__((ext_vector_type(NCH * 4)));
  __device__ __forceinline__ Regs load(int s) const {
    const char* sb = base + (int64_t)s * slab;
    Regs r;
#pragma unroll
    for (int p = 0; p < NCH; ++p) {
      const u32x4 t = *reinterpret_cast<const u32x4*>(sb + p * pass + toff);
      r[4 * p + 0] = t[0]; r[4 * p + 1] = t[1]; r[4 * p + 2] = t[2]; r[4 * p + 3] = t[3];
    }
    return r;
  }
  // chunk p of slab s alone (lets the caller spread the loads of a slab between its MFMAs)
  __device__ __forceinline__ void load_chunk(int s, int p, Regs& r) const {
    const u32x4 t = *reinterpret_cast<const u32x4*>(base + (int64_t)s * slab + p * pass + toff);
    r[4 * p + 0] = t[0]; r[4 * p + 1] = t[1]; r[4 * p + 2] = t[2]; r[4 * p + 3] = t[3];
  }
  __device__ __forceinline__ void store(char* region, const Regs& r) const {
#pragma unroll
    for (int p = 0; p < NCH; ++p) {
      u32x4 t;
      t[0] = r[4 * p + 0]; t[1] = r[4 * p + 1]; t[2] = r[4 * p + 2]; t[3] = r[4 * p + 3];
      *reinterpret_cast<u32x4*>(region + lds + p * RPP * L::STRIDE) = t;
    }
  }
};

// One 16-byte MFMA fragment of 32 tile rows starting at row `r0`, reduction group `g` (8 steps), from an
// fp32 operand slab in LDS.
template <typename T, class L, bool KMAJOR>
__device__ __forceinline__ u32x4 read_frag(const char* region, int r0, int g) {
  const int lane = threadIdx.x & 63;
  if constexpr (!KMAJOR) {
    return *reinterpret_cast<const u32x4*>(region + (r0 + (lane & 31)) * L::STRIDE + g * 32 +
                                           (lane >> 5) * 16);
  } else {
    // four scalar reads, reduction steps g*8 + half*4 + 0..3 of tile row r0 + lane%32
    const char* p = region + (g * 8 + (lane >> 5) * 4) * L::STRIDE + (r0 + (lane & 31)) * 4;
    u32x4 r;
    r[0] = *reinterpret_cast<const uint32_t*>(p);
    r[1] = *reinterpret_cast<const uint32_t*>(p + L::STRIDE);
    r[2] = *reinterpret_cast<const uint32_t*>(p + 2 * L::STRIDE);
    r[3] = *reinterpret_cast<const uint32_t*>(p + 3 * L::STRIDE);
    return r;
  }
}

// The MFMA fragments of one reduction group for a whole wavefront tile.
template <class Cfg>
struct Frags {
  u32x4 a[Cfg::TM];
  u32x4 b[Cfg::TN];
};

template <class Cfg>
__device__ __forceinline__ void read_group(const char* stage, int g, int wm, int wn,
                                           Frags<Cfg>& f) {
  using T = typename Cfg::elem;
#pragma unroll
  for (int bm = 0; bm < Cfg::TM; ++bm)
    f.a[bm] = read_frag<T, typename Cfg::LA, Cfg::A_KMAJOR>(stage, wm * Cfg::WTM + bm * 32, g);
#pragma unroll
  for (int bn = 0; bn < Cfg::TN; ++bn)
    f.b[bn] = read_frag<T, typename Cfg::LB, Cfg::B_KMAJOR>(stage + Cfg::A_BYTES,
                                                            wn * Cfg::WTN + bn * 32, g);
}

template <class Cfg>
__device__ __forceinline__ void mma_group(const Frags<Cfg>& f, f32x16 (&acc)[Cfg::TM][Cfg::TN]) {
  using T = typename Cfg::elem;
#pragma unroll
  for (int bm = 0; bm < Cfg::TM; ++bm)
#pragma unroll
    for (int bn = 0; bn < Cfg::TN; ++bn) mfma_group<T>(f.a[bm], f.b[bn], acc[bm][bn]);
}

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
// A wavefront's load fills 1 KB of consecutive LDS (16 bytes a lane), so rows cannot be padded; what keeps
// the fragment reads off each other's banks is the order of the 16-byte chunks inside a row, chosen by the
// lane's global address:
//   k contiguous: chunk c of row r lies at position c ^ (r/2 % 8): a fragment read by 16 consecutive rows
//                 touches every bank once.
//   k-major:      likewise for units of 64 bytes, so that the four k-rows of one transpose read fall into
//                 different banks.
template <typename T, int R, bool KMAJOR, int SLAB>
struct DmaLds {
  static constexpr int BK = SLAB / (int)sizeof(T);
  static constexpr int ROW_BYTES = KMAJOR ? R * (int)sizeof(T) : SLAB;
  static constexpr int BYTES = (KMAJOR ? BK : R) * ROW_BYTES;
  static constexpr int CPR = ROW_BYTES / 16;
  static_assert(KMAJOR ? ROW_BYTES >= 128 : ROW_BYTES == 128, "what the order of the chunks is made for");
  // what the position of a chunk of row r is xor-ed with
  static __device__ __forceinline__ int turn(int r) {
    if constexpr (!KMAJOR) return (r >> 1) & 7;
    else return (ROW_BYTES >= 256 ? r & 3 : (r >> 1) & 1) * 4;
  }
};

template <typename T, class L, int THREADS, bool KMAJOR>
struct DmaStager {
  static constexpr int NCH = L::BYTES / 16 / THREADS;        // loads per wavefront and slab
  static constexpr int RPP = THREADS * 16 / L::ROW_BYTES;    // LDS rows that one load of every wavefront fills
  static_assert(NCH >= 1 && L::BYTES % (THREADS * 16) == 0, "slab must divide evenly");
  static_assert(RPP % (KMAJOR ? 4 : 16) == 0, "one order of the chunks for all loads of a lane");
  const char* base;   // wave-uniform: first byte of the operand tile at the first k of the range
  uint32_t toff;      // this lane's byte offset from there
  int64_t pass, slab; // global byte steps between a lane's loads of one slab / between slabs (uniform)

  __device__ __forceinline__ void init(const T* tile, int64_t ld) {
    const int t = threadIdx.x;
    const int row = t / L::CPR, ch = (t % L::CPR) ^ L::turn(row);
    base = reinterpret_cast<const char*>(tile);
    toff = (uint32_t)((int64_t)row * ld * (int64_t)sizeof(T) + ch * 16);
    pass = (int64_t)RPP * ld * (int64_t)sizeof(T);
    slab = KMAJOR ? (int64_t)L::BK * ld * (int64_t)sizeof(T) : (int64_t)L::BK * (int64_t)sizeof(T);
  }
  // Load p of slab s into the LDS region at byte `lds` (this wavefront's first byte there).
  // Assembly, because the compiler makes every LDS read that follows the builtin wait for all loads in
  // flight.  The load has no output register; who reads the region waits for it (dma_wait).  M0 needs a
  // wait state before it is used.
  __device__ __forceinline__ void load(int s, int p, uint32_t lds) const {
    const uint64_t at = (uint64_t)(base + (int64_t)s * slab + p * pass);
    const uint64_t g = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) |
                       (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(at >> 32)) << 32;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(__builtin_amdgcn_readfirstlane(lds + p * THREADS * 16)), "v"(toff), "s"(g));
  }
};

// Waits until at most N of this wavefront's loads are in flight and its LDS reads are back, then meets the
// workgroup: what all wavefronts have loaded before is in LDS, what they have read may be overwritten.
template <int N>
__device__ __forceinline__ void dma_wait_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// Byte offsets of this lane's fragment reads in an operand slab.
template <class L, bool KMAJOR, int GROUPS, int NB>
struct FragAddr;
template <class L, int GROUPS, int NB>
struct FragAddr<L, false, GROUPS, NB> {
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
struct FragAddr<L, true, GROUPS, NB> {
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

// gemm_tile (below) for bf16 operands.  LDS holds ABUF slabs of A and BBUF of B:
//   * the barrier in front of the last group of slab s frees its buffers (all fragments are read by then)
//     and publishes slab s+1; behind it B of slab s+BBUF and A of slab s+ABUF are requested, one load
//     between two MFMAs, so a load has BBUF - 1 (A: ABUF - 1) whole slabs of MFMAs to arrive;
//   * fragments are read one group ahead, the last group is multiplied behind the barrier.
// Against staging through registers (two stages of 64 steps, 8 ds_write_b128 a wavefront and slab), both in
// turn, us: logits 1024 x 205,991 x 512 296 -> 276, both backward products there 450 -> 401, 1024 x
// 360,232 766 -> 690, 16,384 x 3,592 125 -> 113; products alone, 256 tiles of 256 x 256 over 6,400 steps,
// 1.00 - 1.17 -> 1.28 - 1.36 PFLOP/s (both k contiguous), 1.03 -> 1.21 (both k-major), 0.97 -> 1.07 (dfeatures).
// What bounds it now, by counters and variants of the loop: both k contiguous, the matrix cores are busy 82 %
// of the cycles at 1.46 GHz, the clock that the power leaves; with operands from HBM (dfeatures: 57 % at
// 1.76 GHz) the loads are: a compute unit's misses return in order, at about 33 GB/s whatever is
// requested earlier (waits taken out: the same; requesting lines of later slabs by one of the workgroups that
// share them: 17 % slower; rows of E stored in blocks of 64 classes: the same).
template <class Cfg>
__device__ __forceinline__ void gemm_tile_dma(const typename Cfg::elem* __restrict__ A, int64_t lda,
                                              const typename Cfg::elem* __restrict__ B, int64_t ldb, int nslabs,
                                              char* smem, f32x16 (&acc)[Cfg::TM][Cfg::TN]) {
  using T = typename Cfg::elem;
  typedef DmaLds<T, Cfg::BM, Cfg::A_KMAJOR, Cfg::SLAB_BYTES> LA;
  typedef DmaLds<T, Cfg::BN, Cfg::B_KMAJOR, Cfg::SLAB_BYTES> LB;
  constexpr int ABUF = Cfg::ABUF, BBUF = Cfg::BBUF;
  static_assert(ABUF == BBUF || ABUF == BBUF + 1, "the counts of loads in flight");
  typedef DmaStager<T, LA, Cfg::THREADS, Cfg::A_KMAJOR> SA;
  typedef DmaStager<T, LB, Cfg::THREADS, Cfg::B_KMAJOR> SB;
  constexpr int NA = SA::NCH, NB = SB::NCH, MM = Cfg::TM * Cfg::TN, HEAD = Cfg::GROUPS - 1;
  // loads that may be in flight when slab s+1 (or slab 0) has to be there, nothing being left out at the end
  constexpr int FLY = ABUF == BBUF ? (BBUF - 2) * (NA + NB) : (BBUF - 1) * NA + (BBUF - 2) * NB;
  constexpr int FLY0 = (BBUF - 1) * (NA + NB) + (ABUF - BBUF) * NA;
  const int wave = threadIdx.x >> 6;
  const int wm = wave / Cfg::WN, wn = wave % Cfg::WN;
  SA sa;
  SB sb;
  sa.init(A, lda);
  sb.init(B, ldb);
  FragAddr<LA, Cfg::A_KMAJOR, Cfg::GROUPS, Cfg::TM> ra;
  FragAddr<LB, Cfg::B_KMAJOR, Cfg::GROUPS, Cfg::TN> rb;
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
        mfma_group<T>(fc.a[q / Cfg::TN], fc.b[q % Cfg::TN], acc[q / Cfg::TN][q % Cfg::TN]);
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
      mfma_group<T>(fc.a[q / Cfg::TN], fc.b[q % Cfg::TN], acc[q / Cfg::TN][q % Cfg::TN]);
    }
    __builtin_amdgcn_sched_barrier(0);
    fc = fn;
  }
  __syncthreads();
}

// Accumulate acc += A_tile * B_tile^T over `nslabs` slabs of K.
//   A: element (first of this workgroup's BM tile rows, first reduction step of its range)
//   B: likewise for its BN tile rows;  lda / ldb in elements.
//   smem: Cfg::LDS_BYTES bytes, 16-byte aligned.  Ends with a barrier (smem may be reused).
// Software pipeline with fp32 operands (two LDS stages, one register set, global loads two slabs ahead):
//   * at the top of iteration s the registers hold slab s+1, loaded during iteration s-1, so it
//     has had a whole iteration to arrive; it goes to the idle LDS stage at once, and the barrier
//     at the end of the iteration publishes it;
//   * the loads of slab s+2 then refill the registers, issued one at a time between the MFMAs of
//     the first groups: a wavefront that issues a whole slab in one burst queues up at the
//     memory pipe (measured: up to 1400 cycles) with its MFMAs stuck behind the loads;
//   * inside a slab the fragments of group g+1 are read from LDS while group g is multiplied;
//   * the last group of a slab is multiplied AFTER the barrier, behind the first fragment reads
//     of the next slab, so the LDS latency at the slab boundary is covered as well.
// Slab numbers past the end are clamped to the last slab: such loads and LDS stores are
// redundant but in bounds, and keep the loop body free of branches.
// CHAIN > 0 (fp32): every CHAIN slabs the accumulators are added to a second set and start again from
// zero, so that no sum is a chain of more than CHAIN * BK additions.
template <class Cfg, int CHAIN = 0>
__device__ __forceinline__ void gemm_tile(const typename Cfg::elem* __restrict__ A, int64_t lda,
                                          const typename Cfg::elem* __restrict__ B, int64_t ldb,
                                          int nslabs, char* smem,
                                          f32x16 (&acc)[Cfg::TM][Cfg::TN]) {
  using T = typename Cfg::elem;
  using LA = typename Cfg::LA;
  using LB = typename Cfg::LB;
  if constexpr (Cfg::DMA) {
    gemm_tile_dma<Cfg>(A, lda, B, ldb, nslabs, smem, acc);
    return;
  }
  const int wave = threadIdx.x >> 6;
  const int wm = wave / Cfg::WN, wn = wave % Cfg::WN;

  typedef Stager<T, LA, Cfg::THREADS, Cfg::A_CHUNKS, Cfg::A_KMAJOR> SA;
  typedef Stager<T, LB, Cfg::THREADS, Cfg::B_CHUNKS, Cfg::B_KMAJOR> SB;
  SA sa;
  SB sb;
  sa.init(A, lda);
  sb.init(B, ldb);
  char* st0 = smem;
  char* st1 = smem + Cfg::STAGE_BYTES;
  const int last = nslabs - 1;
  constexpr int NA = Cfg::A_CHUNKS, NL = Cfg::A_CHUNKS + Cfg::B_CHUNKS;
  constexpr int MM = Cfg::TM * Cfg::TN;            // MFMAs per group
  constexpr int HEAD = Cfg::GROUPS - 1;            // groups multiplied before the barrier
  // the loads of a slab are placed in front of the MFMAs of the first one or two groups (of all
  // groups before the barrier if two do not have an MFMA for each load)
  constexpr int SPAN = (NL <= 2 * MM ? (HEAD < 2 ? HEAD : 2) : HEAD) * MM;
  static_assert(HEAD >= 1, "the last group is multiplied behind the barrier");
  static_assert(CHAIN == 0 || sizeof(T) == 4, "bf16 operands: their rounding is what counts");

  // prologue: slabs 0 and 1 are requested back to back; slab 0 goes to stage 0
  typename SA::Regs a0 = {};
  typename SB::Regs b0 = {};
  {
    typename SA::Regs af = sa.load(0);
    typename SB::Regs bf = sb.load(0);
    a0 = sa.load(last < 1 ? last : 1);
    b0 = sb.load(last < 1 ? last : 1);
    sa.store(st0, af);
    sb.store(st0 + Cfg::A_BYTES, bf);
  }
  __syncthreads();
  Frags<Cfg> fc;
  read_group<Cfg>(st0, 0, wm, wn, fc);
  f32x16 sums[Cfg::TM][Cfg::TN];
  if constexpr (CHAIN > 0) zero_acc<Cfg>(sums);
  for (int s = 0; s < nslabs; ++s) {
    char* cur = (s & 1) ? st1 : st0;
    char* nxt = (s & 1) ? st0 : st1;
    const int s2 = s + 2 < last ? s + 2 : last;
    sa.store(nxt, a0);
    sb.store(nxt + Cfg::A_BYTES, b0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int g = 0; g < HEAD; ++g) {
      Frags<Cfg> fn;
      read_group<Cfg>(cur, g + 1, wm, wn, fn);
      __builtin_amdgcn_sched_barrier(0);   // keep the reads ahead of the MFMAs they do not feed
#pragma unroll
      for (int q = 0; q < MM; ++q) {
        // one block to a wavefront, sums in pieces: the loads go between the MFMAs of the group, and stay
        // there (left to the compiler they end up in front of all four: 512 samples x 9,344 classes x 512
        // 168 us, so 163; larger tiles lose 2 % by it)
        constexpr bool kBetween = CHAIN > 0 && MM == 1;
        if constexpr (kBetween) {
          mfma_half<0>(fc.a[0], fc.b[0], acc[0][0]);
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int c = 0; c < NL; ++c) {     // chunk c is requested in front of MFMA c*SPAN/NL
          if (c * SPAN / NL == g * MM + q) {
            if (c < NA) sa.load_chunk(s2, c, a0);
            else sb.load_chunk(s2, c - NA, b0);
          }
        }
        if constexpr (kBetween) {
          __builtin_amdgcn_sched_barrier(0);
          mfma_half<1>(fc.a[0], fc.b[0], acc[0][0]);
        } else {
          mfma_group<T>(fc.a[q / Cfg::TN], fc.b[q % Cfg::TN], acc[q / Cfg::TN][q % Cfg::TN]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      fc = fn;
    }
    __syncthreads();
    Frags<Cfg> fn;
    read_group<Cfg>(nxt, 0, wm, wn, fn);
    __builtin_amdgcn_sched_barrier(0);
    mma_group<Cfg>(fc, acc);
    __builtin_amdgcn_sched_barrier(0);
    fc = fn;
    if constexpr (CHAIN > 0) {
      if ((s + 1) % CHAIN == 0 && s < last) {
        add_acc<Cfg>(sums, acc);
        zero_acc<Cfg>(acc);
      }
    }
  }
  if constexpr (CHAIN > 0) add_acc<Cfg>(acc, sums);
  __syncthreads();
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
