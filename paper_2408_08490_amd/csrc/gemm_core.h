// MFMA GEMM core shared by the layer GEMMs: tile movers (global -> registers -> LDS), MFMA fragment reads,
// the software-pipelined K loop over a tile's segments, and the LDS-staged epilogue.
#pragma once
#include <type_traits>

#include "common.h"
#include "device_types.h"

namespace hgnn {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// A block is 2x2 wavefronts; every wavefront owns MI x NI accumulators of 32x32, so the block tile is
// (64 MI) x (64 NI).  BM x BN is the default tile (MI = NI = 2); launches that would not fill the chip with
// those use 64x64 tiles (MI = NI = 1).
constexpr int BM = 128, BN = 128, kThreads = 256;

template <typename T> struct Mma;
template <> struct Mma<bf16> {
  static constexpr int BK = 64, KSTEP = 16, VEC = 8, PKC = BK + 8, KSPAD = 16;  // KS pitch = extent + KSPAD: four k-rows of a transposing read on disjoint banks
};
template <> struct Mma<float> {
  static constexpr int BK = 32, KSTEP = 2, VEC = 4, PKC = BK + 4, KSPAD = 4;
};
// LDS pitch (elements) of an operand tile kept with its OUTPUT index contiguous ("KS": rows = k).  A 128-wide bf16
// tile is kept unpadded (a row = 64 dwords = the LDS's 64 banks) with the four 64-byte column blocks of a row
// XOR-swizzled by the row's low two bits: the transposing fragment read touches four consecutive k-rows at one
// column block per 32 lanes, which then sit on four different quarters of the banks (with a 16-element pad they
// overlapped in pairs: a quarter of the weight-gradient kernel's LDS cycles were bank conflicts).  Other shapes
// keep the pad.
template <typename T> constexpr bool ks_swizzled(int extent) { return sizeof(T) == 2 && extent == 128; }
template <typename T> constexpr int ks_pitch(int extent) { return ks_swizzled<T>(extent) ? extent : extent + Mma<T>::KSPAD; }
__device__ __forceinline__ int ks_swizzle_col(int col, int row) { return (((col >> 5) ^ (row & 3)) << 5) | (col & 31); }
// elements of one LDS stage of an operand tile with `extent` output indices, in either orientation or with K contiguous
template <typename T> constexpr int lds_elems(int extent, bool kc) {
  return kc || extent * Mma<T>::PKC > Mma<T>::BK * ks_pitch<T>(extent) ? extent * Mma<T>::PKC : Mma<T>::BK * ks_pitch<T>(extent);
}

// One K-segment of a tile's reduction: sum over k in [kb, ke) of Aop[.][k] * Bop[.][k].
template <typename T> struct Seg {
  const T *A, *B;
  int lda, ldb, kb, ke;
};

// One operand tile on its way global -> registers -> LDS.  The tile is ROWS x COLS in the operand's own
// row-major orientation (COLS contiguous).
//  * FAST: per-thread byte offsets are computed once per segment (`setup`); a K-step is NV 16-byte buffer loads from a
//    wave-uniform base.  Pieces whose OUTPUT index is out of range read a clamped address: they only feed output rows / columns
//    that the epilogue never writes.  Pieces beyond the segment's end, and whole steps beyond the last (krem <= 0), ask for an
//    offset outside the buffer, which gives zeros and fetches nothing.  So a K loop issues its loads without a branch around
//    them: where there is one, the compiler waits for the newest loads before it stores the oldest, and two steps in flight are one.
//  * generic: element-wise, zero-filled loads.
template <typename T, int ROWS, int COLS, int PITCH, bool KC>
struct TileMover {
  static constexpr int VEC = 16 / sizeof(T), VPR = COLS / VEC, NV = ROWS * VPR / kThreads;
  static_assert(ROWS * VPR % kThreads == 0, "tile must split evenly over the block");
  typedef const unsigned short __attribute__((address_space(1))) *g16_t;
  typedef const unsigned int __attribute__((address_space(1))) *g32_t;
  u32x4 reg[NV];
  unsigned okmask;        // pieces inside the segment (FAST); the others are zero

  struct Offsets {   // byte offsets of this thread's pieces from a K-step's base (FAST), the same for all steps of a segment
    unsigned voff[NV];
    // `o0` = first output index of the tile, `extent` = number of valid output indices, ld in elements.
    __device__ __forceinline__ void setup(int ld, int extent, int o0) {
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const int v = threadIdx.x + i * kThreads;
        const int r = v / VPR, c = (v % VPR) * VEC;
        if constexpr (KC) {  // rows = output index, cols = k
          voff[i] = (unsigned)(min(r, extent - 1 - o0) * ld + c) * (unsigned)sizeof(T);
        } else {             // rows = k, cols = output index
          voff[i] = (unsigned)(r * ld + (c < extent - o0 ? c : 0)) * (unsigned)sizeof(T);
        }
      }
    }
  };
  // base = operand base advanced to the tile's first output index and to the K-step; krem = ke - k0
  __device__ __forceinline__ void load_fast(const Offsets &at, const T *base, int krem) {
    constexpr int kInside = 0x7ffffff0;
    constexpr unsigned kOutside = 0x80000000u;
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<T *>(base), 0, krem > 0 ? kInside : 0, 0x00027000);
    okmask = 0;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int v = threadIdx.x + i * kThreads;
      const int kk = KC ? (v % VPR) * VEC : v / VPR;   // first k index of the piece within the step
      const bool ok = kk < krem;                        // K extents are multiples of VEC here
      reg[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, ok ? at.voff[i] : kOutside, 0, 0);
      okmask |= ok ? (1u << i) : 0u;
    }
  }
  __device__ __forceinline__ void load_slow(const T *base, int64_t ld, int nrows, int ncols, int r0, int c0) {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int v = threadIdx.x + i * kThreads;
      const int gr = r0 + v / VPR, gc = c0 + (v % VPR) * VEC;
      unsigned int e[VEC];
#pragma unroll
      for (int j = 0; j < VEC; ++j) {
        const bool ok = gr < nrows && gc + j < ncols;
        const T *p = ok ? base + (int64_t)gr * ld + gc + j : base;
        unsigned int x;
        if constexpr (sizeof(T) == 2) x = *(g16_t)p; else x = *(g32_t)p;
        e[j] = ok ? x : 0u;
      }
      if constexpr (sizeof(T) == 2)
        reg[i] = u32x4{e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16)};
      else
        reg[i] = u32x4{e[0], e[1], e[2], e[3]};
    }
  }
  __device__ __forceinline__ void store(T *lds) {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int v = threadIdx.x + i * kThreads;
      int col = (v % VPR) * VEC;
      if constexpr (!KC && ks_swizzled<T>(COLS)) col = ks_swizzle_col(col, v / VPR);
      T *q = lds + (v / VPR) * PITCH + col;
      if constexpr ((PITCH * sizeof(T)) % 16 == 0) {
        *reinterpret_cast<u32x4 *>(q) = reg[i];
      } else {
        static_assert((PITCH * sizeof(T)) % 8 == 0, "LDS pitch must keep 8-byte alignment");
        reinterpret_cast<u32x2 *>(q)[0] = u32x2{reg[i].x, reg[i].y};
        reinterpret_cast<u32x2 *>(q)[1] = u32x2{reg[i].z, reg[i].w};
      }
    }
  }
};

// MFMA operand fragments out of LDS.  `o` = output index handled by this lane's fragment block.
template <bool KC, int PITCH> __device__ __forceinline__ bf16x8_t frag_bf16(const bf16 *s, int o, int ks, int lane) {
  if constexpr (KC) {
    return *reinterpret_cast<const bf16x8_t *>(s + (o + (lane & 31)) * PITCH + ks * 16 + 8 * (lane >> 5));
  } else {
    // The operand lies in LDS with the output index contiguous; the transposing LDS read hands every lane
    // four consecutive k of one output index.  Within a group of 16 lanes, lane p passes the address of four
    // contiguous 16-bit values ("row" p) and lane i receives rows (i / 4) + 4 j, j = 0..3, at position i % 4:
    // with row p = (k0 + p / 4, outputs o16 + 4 (p % 4) ...) lane i ends up with k0..k0+3 of output o16 + i.
    typedef short v4i16 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) v4i16 *lds_v4;
    const int p = lane & 15;
    const int row = ks * 16 + 8 * (lane >> 5) + (p >> 2);
    int col = o + 16 * ((lane >> 4) & 1) + 4 * (p & 3);
    if constexpr (PITCH == 128) col = ks_swizzle_col(col, row);  // the unpadded, swizzled 128-wide tile (row + 4 has the same low bits)
    const bf16 *q = s + row * PITCH + col;
    union { bf16x8_t v; v4i16 h[2]; } u;
    u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4)q);
    u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4)(q + 4 * PITCH));
    return u.v;
  }
}
template <bool KC, int PITCH> __device__ __forceinline__ float frag_f32(const float *s, int o, int ks, int lane) {
  if constexpr (KC) return s[(o + (lane & 31)) * PITCH + ks * 2 + (lane >> 5)];
  else return s[(ks * 2 + (lane >> 5)) * PITCH + o + (lane & 31)];
}

template <typename T, bool AKC, bool BKC, int MI, int NI>
__device__ __forceinline__ void mma_tile(f32x16 (&acc)[MI][NI], const T *As, const T *Bs, int wm, int wn, int lane) {
  using M = Mma<T>;
  constexpr int PA = AKC ? M::PKC : ks_pitch<T>(64 * MI), PB = BKC ? M::PKC : ks_pitch<T>(64 * NI);
  if constexpr (sizeof(T) == 4 && AKC && BKC) {
    // Eight K at a time: a lane reads four of its row, the lower half of the wavefront the first ones, and the halves swap two of
    // them, which leaves the operands of four MFMAs in order.  Read one by one, in front of every second MFMA, the reads' latency
    // was on the way of an accumulator's chain.
    constexpr int G = M::BK / 8;
    float a[G][MI][4], b[G][NI][4];
    auto read = [&](float (&f)[4], const float *s, int o, int pitch, int g) {
      const u32x4 q = *reinterpret_cast<const u32x4 *>(s + (o + (lane & 31)) * pitch + 8 * g + 4 * (lane >> 5));
      const auto lo = __builtin_amdgcn_permlane32_swap(q.x, q.y, false, false), hi = __builtin_amdgcn_permlane32_swap(q.z, q.w, false, false);
      f[0] = __uint_as_float(lo[0]);
      f[1] = __uint_as_float(hi[0]);
      f[2] = __uint_as_float(lo[1]);
      f[3] = __uint_as_float(hi[1]);
    };
    constexpr int GG = MI * NI > 1 ? 2 : G;   // read ahead
#pragma unroll
    for (int g0 = 0; g0 < G; g0 += GG) {
#pragma unroll
      for (int g = g0; g < g0 + GG; ++g) {
#pragma unroll
        for (int i = 0; i < MI; ++i) read(a[g][i], reinterpret_cast<const float *>(As), wm + i * 32, PA, g);
#pragma unroll
        for (int j = 0; j < NI; ++j) read(b[g][j], reinterpret_cast<const float *>(Bs), wn + j * 32, PB, g);
      }
#pragma unroll
      for (int g = g0; g < g0 + GG; ++g)
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
          for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[g][i][k], b[g][j][k], acc[i][j], 0, 0, 0);
    }
    return;
  }
#pragma unroll
  for (int ks = 0; ks < M::BK / M::KSTEP; ++ks) {
    if constexpr (sizeof(T) == 2) {
      bf16x8_t a[MI], b[NI];
#pragma unroll
      for (int i = 0; i < MI; ++i) a[i] = frag_bf16<AKC, PA>(reinterpret_cast<const bf16 *>(As), wm + i * 32, ks, lane);
#pragma unroll
      for (int j = 0; j < NI; ++j) b[j] = frag_bf16<BKC, PB>(reinterpret_cast<const bf16 *>(Bs), wn + j * 32, ks, lane);
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    } else {
      float a[MI], b[NI];
#pragma unroll
      for (int i = 0; i < MI; ++i) a[i] = frag_f32<AKC, PA>(reinterpret_cast<const float *>(As), wm + i * 32, ks, lane);
#pragma unroll
      for (int j = 0; j < NI; ++j) b[j] = frag_f32<BKC, PB>(reinterpret_cast<const float *>(Bs), wn + j * 32, ks, lane);
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j], acc[i][j], 0, 0, 0);
    }
  }
}

// fp32 products on the bf16 matrix cores.  An fp32 value is the exact sum of three bf16 values x0 + x1 + x2 (8 + 8 + 8
// significant bits; rounding to nearest makes |x1| <= 2^-9 |x|, |x2| <= 2^-18 |x|), and a product of two bf16 values is
// exact in fp32.  Of the nine products six are taken; x1 y2 + x2 y1 + x2 y2, at most 2^-26 |x y| and of either sign, lie
// below the rounding of the fp32 sum.  Six bf16 MFMAs take 6/16 of the time of the fp32 MFMA's.  The MFMA's own sum over 16
// terms is not rounded to nearest, and over a whole reduction that shows (bias gradients 2x further off); so a K-step's sum
// starts from zero and the vector unit adds it to the accumulator: against 64 bits, outputs and weight gradients are then
// 0.1 to 0.5 of the distance that the fp32 MFMA leaves (1024 targets, fan-out 25 and 20: outputs 9e-7 -> 4e-7, weight
// gradients 1e-6 -> 2e-7 of their norm).
// Measured with 1024 targets in fp32 (us, fp32 MFMA -> this): forward of 1400 tiles of 64, no ReLU, 50 -> 39, backward of the first
// layer 96 -> 66, of ragged widths 84 -> 69; the weight gradient of the semantic attention (560k rows, with dm) 739 -> 600.
// An operand's three planes lie one behind the other in the LDS of its two fp32 stages; with one stage a K-step costs two
// barriers, which the other block of the compute unit covers.
constexpr int kSplitPKC = Mma<float>::BK + 8;   // elements of a bf16 row with K contiguous (rows on disjoint banks)
template <bool KC> constexpr int split_pitch(int extent) { return KC ? kSplitPKC : ks_pitch<bf16>(extent); }
template <bool KC> constexpr int split_plane(int extent) { return KC ? extent * kSplitPKC : Mma<float>::BK * ks_pitch<bf16>(extent); }

// Four fp32 values, times kSplitScale, as the three planes' four bf16 values.  bf16 has fp32's exponents, so without the
// scale the low planes of values below 1e-33 would fall off its lower end (gradients of 1e-35 lost 2.7e-6 of their norm, of
// 1e-37 2.7e-4); scaled, every normal fp32 value has normal planes.  Values and sums beyond what the scale leaves room for
// (2e31 and 1e24) do not come out finite and take the fp32 MFMA (gemm_finite).
constexpr float kSplitScale = 0x1p24f;
__device__ __forceinline__ void split3(const f32x4 v, u32x2 (&w)[3]) {
  float d[4] = {v.x * kSplitScale, v.y * kSplitScale, v.z * kSplitScale, v.w * kSplitScale};
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    w[p] = u32x2{pack2(d[0], d[1]), pack2(d[2], d[3])};
    if (p < 2) {
      d[0] -= __uint_as_float(w[p].x << 16);
      d[1] -= __uint_as_float(w[p].x & 0xffff0000u);
      d[2] -= __uint_as_float(w[p].y << 16);
      d[3] -= __uint_as_float(w[p].y & 0xffff0000u);
    }
  }
}
// acc += part / scale, exact but for the sum's own rounding (scale: a power of two)
template <int NI> __device__ __forceinline__ void add_unscaled(f32x16 (&acc)[NI], const f32x16 (&part)[NI], float scale) {
#pragma unroll
  for (int j = 0; j < NI; ++j)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[j][v] = fmaf(part[j][v], 1.f / scale, acc[j][v]);
}

// Stores the operand tile of a mover of fp32 values as three planes.
template <bool KC, int EXTENT, typename Mover>
__device__ __forceinline__ void split_store(Mover &mv, bf16 *lds) {
  constexpr int COLS = KC ? Mma<float>::BK : EXTENT, VPR = COLS / 4, NV = sizeof(mv.reg) / sizeof(mv.reg[0]);
  constexpr int PITCH = split_pitch<KC>(EXTENT), PLANE = split_plane<KC>(EXTENT);
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int v = threadIdx.x + i * kThreads, row = v / VPR;
    int col = (v % VPR) * 4;
    if constexpr (!KC && ks_swizzled<bf16>(EXTENT)) col = ks_swizzle_col(col, row);
    u32x2 w[3];
    split3(__builtin_bit_cast(f32x4, mv.reg[i]), w);
#pragma unroll
    for (int p = 0; p < 3; ++p) *reinterpret_cast<u32x2 *>(lds + p * PLANE + row * PITCH + col) = w[p];
  }
}

template <bool AKC, bool BKC, int MI, int NI>
__device__ __forceinline__ void mma_tile_split(f32x16 (&acc)[MI][NI], const bf16 *As, const bf16 *Bs, int wm, int wn, int lane) {
  constexpr int PA = split_pitch<AKC>(64 * MI), PB = split_pitch<BKC>(64 * NI);
  constexpr int QA = split_plane<AKC>(64 * MI), QB = split_plane<BKC>(64 * NI);
  constexpr int NK = Mma<float>::BK / 16;
  bf16x8_t b[3][NK][NI];
#pragma unroll
  for (int q = 0; q < 3; ++q)
#pragma unroll
    for (int ks = 0; ks < NK; ++ks)
#pragma unroll
      for (int j = 0; j < NI; ++j) b[q][ks][j] = frag_bf16<BKC, PB>(Bs + q * QB, wn + j * 32, ks, lane);
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    f32x16 part[NI];
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) part[j][v] = 0.f;
#pragma unroll
    for (int p = 2; p >= 0; --p)   // smallest products first
#pragma unroll
      for (int ks = 0; ks < NK; ++ks) {
        const bf16x8_t a = frag_bf16<AKC, PA>(As + p * QA, wm + i * 32, ks, lane);
#pragma unroll
        for (int q = 2 - p; q >= 0; --q)
#pragma unroll
          for (int j = 0; j < NI; ++j) part[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b[q][ks][j], part[j], 0, 0, 0);
      }
    add_unscaled(acc[i], part, kSplitScale * kSplitScale);
  }
}

// LDS of one block: two stages of (A tile, B tile), reused as the output staging tile by the epilogues.
// KC: both operands with K contiguous.
template <typename T, int MI = 2, int NI = 2, bool KC = false> struct GemmLds {
  __attribute__((aligned(16))) T a[2][lds_elems<T>(64 * MI, KC)];
  __attribute__((aligned(16))) T b[2][lds_elems<T>(64 * NI, KC)];
  // a factor per row of the output tile, behind the staged tile (once the K loop is done)
  __device__ __forceinline__ float *rowscale() {
    static_assert(sizeof(b) >= sizeof(float) * 64 * MI && sizeof(a) + sizeof(b) - sizeof(float) * 64 * MI >= sizeof(float) * (64 * NI + 8) * 64 * MI);
    return reinterpret_cast<float *>(&b[2]) - 64 * MI;
  }
};
constexpr int kOutPitchPad = 8;  // floats: staged rows stay 16-byte aligned, rows r and r + 4 lie 32 banks apart

// A pointer that is the same in every lane, moved to scalar registers.
template <typename P> __device__ __forceinline__ const P *uniform_ptr(const P *p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<const P *>(((uint64_t)hi << 32) | lo);
}

struct NoXform {
  template <typename M> __device__ __forceinline__ void operator()(M &, int) const {}
};

// A reduction over one segment.  AHEAD: K-steps whose loads are under way in front of the one that is multiplied, where fp32 operands
// are split into planes.
template <typename T, int AHEAD = 2> struct OneSeg {
  static constexpr int kAhead = AHEAD;
  static constexpr bool kRedo = true;   // on the fp32 MFMA it is only what gemm_finite falls back on
  Seg<T> g;
  __device__ __forceinline__ int steps() const { return (g.ke - g.kb + Mma<T>::BK - 1) / Mma<T>::BK; }
  __device__ __forceinline__ void next(Seg<T> &o) { o = g; }
};

// Runs the K-steps of the segments that `segs` hands out one after the other (the same ones to every lane) into `acc`; steps():
// how many there are.  Segments come from scalar registers and scalar loads: a table of them in LDS, made by the first wavefront
// from the general tables, was 2.7 us in front of a tile's first load.
// KC operand: matrix [extent x K] row-major (ld); KS operand: matrix [K x extent] row-major (ld).
// xa(mover, step) / xb: what happens to a K-step's operand tile in the registers, on its way to LDS.
// FAST fp32 tiles run on the bf16 matrix cores (see mma_tile_split) unless SPLIT is false; call them through
// gemm_finite, which sees to infinities.
template <typename T, bool FAST, bool AKC, bool BKC, bool SPLIT = FAST && sizeof(T) == 4, int MI, int NI, bool LKC, typename Segs, typename XA = NoXform, typename XB = NoXform>
__device__ __forceinline__ void gemm_run(f32x16 (&acc)[MI][NI], GemmLds<T, MI, NI, LKC> &sm, Segs segs, int a_extent, int a0,
                                         int b_extent, int b0, XA xa = XA(), XB xb = XB()) {
  using M = Mma<T>;
  static_assert(!LKC || (AKC && BKC));
  constexpr int TM = 64 * MI, TN = 64 * NI;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = (wave >> 1) * 32 * MI, wn = (wave & 1) * 32 * NI;
  using MoverA = TileMover<T, AKC ? TM : M::BK, AKC ? M::BK : TM, AKC ? M::PKC : ks_pitch<T>(TM), AKC>;
  using MoverB = TileMover<T, BKC ? TN : M::BK, BKC ? M::BK : TN, BKC ? M::PKC : ks_pitch<T>(TN), BKC>;
  MoverA ta0, ta1;
  MoverB tb0, tb1;
  const int total = __builtin_amdgcn_readfirstlane(segs.steps());
  // cursor of the loader, two K-steps ahead of the multiplier, and its segment; behind the last step it loads nothing
  Seg<T> g{};
  int k_ld = 0, to_load = total;
  typename MoverA::Offsets oa;
  typename MoverB::Offsets ob;
  auto issue = [&](MoverA &ta, MoverB &tb) {
    if (to_load > 0 && k_ld >= g.ke) {
      Seg<T> v;
      segs.next(v);
      g.A = uniform_ptr(v.A);
      g.B = uniform_ptr(v.B);
      g.lda = __builtin_amdgcn_readfirstlane(v.lda);
      g.ldb = __builtin_amdgcn_readfirstlane(v.ldb);
      g.kb = __builtin_amdgcn_readfirstlane(v.kb);
      g.ke = __builtin_amdgcn_readfirstlane(v.ke);
      k_ld = g.kb;
      if constexpr (FAST) {
        oa.setup(g.lda, a_extent, a0);
        ob.setup(g.ldb, b_extent, b0);
      }
    }
    if constexpr (FAST) {
      const int krem = to_load > 0 ? g.ke - k_ld : 0;
      ta.load_fast(oa, AKC ? g.A + (int64_t)a0 * g.lda + k_ld : g.A + (int64_t)k_ld * g.lda + a0, krem);
      tb.load_fast(ob, BKC ? g.B + (int64_t)b0 * g.ldb + k_ld : g.B + (int64_t)k_ld * g.ldb + b0, krem);
    } else if (to_load > 0) {
      if constexpr (AKC) ta.load_slow(g.A, g.lda, a_extent, g.ke, a0, k_ld);
      else ta.load_slow(g.A, g.lda, g.ke, a_extent, k_ld, a0);
      if constexpr (BKC) tb.load_slow(g.B, g.ldb, b_extent, g.ke, b0, k_ld);
      else tb.load_slow(g.B, g.ldb, g.ke, b_extent, k_ld, b0);
    }
    --to_load;
    k_ld += M::BK;
  };
  if (total <= 0) return;
  if constexpr (FAST && sizeof(T) == 4 && !SPLIT && Segs::kRedo) {   // nothing in flight: it needs no registers beside the planes' form
#pragma unroll 1
    for (int step = 0; step < total; ++step) {
      issue(ta0, tb0);
      xa(ta0, step);
      xb(tb0, step);
      ta0.store(sm.a[0]);
      tb0.store(sm.b[0]);
      __syncthreads();
      mma_tile<T, AKC, BKC>(acc, sm.a[0], sm.b[0], wm, wn, lane);
      __syncthreads();
    }
    return;
  }
  issue(ta0, tb0);
  if constexpr (!SPLIT || Segs::kAhead == 2) issue(ta1, tb1);
  if constexpr (SPLIT) {
    static_assert(3 * split_plane<AKC>(TM) * sizeof(bf16) <= sizeof(sm.a) && 3 * split_plane<BKC>(TN) * sizeof(bf16) <= sizeof(sm.b), "planes must fit the stages");
    bf16 *pa = reinterpret_cast<bf16 *>(&sm.a[0][0]), *pb = reinterpret_cast<bf16 *>(&sm.b[0][0]);
    auto one = [&](MoverA &ta, MoverB &tb, int step) {
      xa(ta, step);
      xb(tb, step);
      split_store<AKC, TM>(ta, pa);
      split_store<BKC, TN>(tb, pb);
      __syncthreads();
      issue(ta, tb);
      mma_tile_split<AKC, BKC>(acc, pa, pb, wm, wn, lane);
      __syncthreads();
    };
    if constexpr (Segs::kAhead == 1) {
#pragma unroll 1
      for (int step = 0; step < total; ++step) one(ta0, tb0, step);
      return;
    }
    for (int step = 0;; step += 2) {
      one(ta0, tb0, step);
      if (step + 1 >= total) break;
      one(ta1, tb1, step + 1);
      if (step + 2 >= total) break;
    }
    return;
  }
  auto one = [&](MoverA &ta, MoverB &tb, int stage, int step, bool more = true) {
    xa(ta, step);
    xb(tb, step);
    ta.store(sm.a[stage]);
    tb.store(sm.b[stage]);
    __syncthreads();
    if (more) issue(ta, tb);
    mma_tile<T, AKC, BKC>(acc, sm.a[stage], sm.b[stage], wm, wn, lane);
  };
  int step = 0;
  for (; step + 1 < total; step += 2) {   // one way back to the loop's head: see TileMover
    one(ta0, tb0, 0, step);
    one(ta1, tb1, 1, step + 1);
  }
  if (step < total) one(ta0, tb0, 0, step, false);
  __syncthreads();  // the stages may be rewritten by the caller
}

template <int MI, int NI> __device__ __forceinline__ void zero_acc(f32x16 (&acc)[MI][NI]) {
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
}

// A tile's products through run(split): an infinity, or a value beyond the planes' range, leaves NaN where the fp32
// product would be infinite or large (inf - inf in the planes, 0 * inf between them), so a tile that did not come out
// finite is multiplied again on the fp32 MFMA (acc starts from zero both times).  fp32_mfma: sums that go through a ReLU
// stay there altogether (see gemm_fwd_kernel), and so do sums of at most kFewTerms terms, which it rounds less:
// products alone, against 64 bits, 2.6e-8 of their norm (the planes 3.4e-8, twice the largest error), sums of two 3.1e-8
// (3.3e-8), of three 3.4e-8 (3.2e-8), of 64 1.5e-7 (6e-8).
constexpr int kFewTerms = 2;
template <typename T, bool FAST, int MI, int NI, typename F>
__device__ __forceinline__ void gemm_finite(f32x16 (&acc)[MI][NI], F run, bool fp32_mfma = false) {
  zero_acc(acc);
  if constexpr (FAST && sizeof(T) == 4) {
    if (fp32_mfma) {
      run(std::false_type());
      return;
    }
  }
  run(std::integral_constant<bool, FAST && sizeof(T) == 4>());
  if constexpr (FAST && sizeof(T) == 4) {
    float s = 0.f;   // 0 * v is 0 for finite v only
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) s += acc[i][j][v] * 0.f;
    if (__syncthreads_or(!(s == 0.f))) {
      zero_acc(acc);
      run(std::false_type());
    }
  }
}

// Element (row, col) of the block tile held in acc[i][j][v] by this lane (32x32 MFMA output layout:
// lane%32 is the column, the 16 values are rows 8*(v/4) + 4*(lane/32) + v%4).
#define HGNN_FOR_EACH_ACC(body)                                                     \
  {                                                                                 \
    const int lane_ = threadIdx.x & 63, wave_ = threadIdx.x >> 6;                   \
    constexpr int MI_ = sizeof(acc) / sizeof(acc[0]), NI_ = sizeof(acc[0]) / sizeof(acc[0][0]); \
    _Pragma("unroll") for (int i_ = 0; i_ < MI_; ++i_) _Pragma("unroll") for (int j_ = 0; j_ < NI_; ++j_) \
    _Pragma("unroll") for (int v_ = 0; v_ < 16; ++v_) {                             \
      const int row = (wave_ >> 1) * 32 * MI_ + i_ * 32 + 8 * (v_ >> 2) + 4 * (lane_ >> 5) + (v_ & 3); \
      const int col = (wave_ & 1) * 32 * NI_ + j_ * 32 + (lane_ & 31);              \
      const float val = acc[i_][j_][v_];                                            \
      body                                                                          \
    }                                                                               \
  }

// Writes the block's tile `out[(row0 + r) * ld + col0 + c] = f(acc, r, c)` for r < rows, c < cols.
// When rows of `out` are 16-byte aligned the tile goes through LDS (the K loop's stages are free by then)
// and leaves as whole 16-byte pieces; otherwise element by element.  `f(val, row, col)` returns the value.
// The output type TO may differ from the operands' T (bf16 operands, fp32 result).  The staged tile is fp32 whatever T is: 32-bit LDS writes with a pitch that puts the two half-waves
// (rows r and r + 4 of one store) on disjoint banks; two lanes writing the halves of one dword would be
// serialised.  Conversion to T happens on the way out.
template <typename T, typename TO, typename F, int MI, int NI, bool LKC>
__device__ __forceinline__ void write_tile(f32x16 (&acc)[MI][NI], GemmLds<T, MI, NI, LKC> &sm, TO *out, int64_t ld, int rows, int cols, F f) {
  constexpr int TM = 64 * MI, TN = 64 * NI;
  constexpr int V = 16 / sizeof(TO), P = TN + kOutPitchPad;
  static_assert(sizeof(sm.a) + sizeof(sm.b) >= sizeof(float) * P * TM, "fp32 output tile must fit the stages");
  const bool vec = (ld % V) == 0 && (reinterpret_cast<uintptr_t>(out) & 15) == 0;
  if (vec) {
    float *stage = reinterpret_cast<float *>(&sm.a[0][0]);
    HGNN_FOR_EACH_ACC({ stage[row * P + col] = f(val, row, col); })
    __syncthreads();
    constexpr int VPR = TN / V;
#pragma unroll
    for (int i = 0; i < TM * VPR / kThreads; ++i) {
      const int v = threadIdx.x + i * kThreads;
      const int r = v / VPR, c = (v % VPR) * V;
      if (r < rows && c < cols) {
        const float *sp = stage + r * P + c;
        u32x4 piece;
        if constexpr (sizeof(TO) == 4) {
          piece = *reinterpret_cast<const u32x4 *>(sp);
        } else {
          const f32x4 lo = *reinterpret_cast<const f32x4 *>(sp), hi = *reinterpret_cast<const f32x4 *>(sp + 4);
          piece = u32x4{pack2(lo.x, lo.y), pack2(lo.z, lo.w), pack2(hi.x, hi.y), pack2(hi.z, hi.w)};
        }
        TO *dst = out + (int64_t)r * ld + c;
        if (c + V <= cols) {
          *reinterpret_cast<u32x4 *>(dst) = piece;
        } else {  // last, partial piece of a row: element by element out of the registers
#pragma unroll
          for (int j = 0; j < V; ++j) {
            if (c + j < cols) {
              if constexpr (sizeof(TO) == 4) {
                reinterpret_cast<unsigned *>(dst)[j] = piece[j];
              } else {
                const unsigned w = piece[j >> 1];
                reinterpret_cast<unsigned short *>(dst)[j] = (unsigned short)((j & 1) ? (w >> 16) : (w & 0xffffu));
              }
            }
          }
        }
      }
    }
  } else {
    HGNN_FOR_EACH_ACC({
      if (row < rows && col < cols) out[(int64_t)row * ld + col] = from_float<TO>(f(val, row, col));
    })
  }
}

// Blocks are spread round-robin over the 8 XCDs by the hardware; give each XCD a contiguous range of tiles
// so that tiles sharing operand rows meet in the same L2.
__device__ __forceinline__ int xcd_tile(int bid, int nblocks) {
  const int per = nblocks >> 3;
  return (bid & 7) * per + (bid >> 3);
}
static inline int round_up8(int n) { return (n + 7) & ~7; }

// The same idea for tiles of unequal cost: group g holds tiles [tile_off[g], tile_off[g+1]) of cost[g] each;
// every XCD gets a contiguous range of about one eighth of the total cost.  Block b works on tile
// first[b & 7] + (b >> 3) when that lies below first[(b & 7) + 1], else on nothing.
struct XcdMap {
  int32_t first[9];
};
// Returns the number of blocks to launch.
static inline int balance_xcd(const int32_t *tile_off, const int64_t *cost, int ngroups, XcdMap &m) {
  int64_t total = 0;
  for (int g = 0; g < ngroups; ++g) total += (int64_t)(tile_off[g + 1] - tile_off[g]) * cost[g];
  const int ntiles = tile_off[ngroups];
  m.first[0] = 0;
  int g = 0, longest = 0;
  int64_t before = 0;  // cost of the tiles before group g
  for (int x = 1; x <= 8; ++x) {
    int t = ntiles;
    if (x < 8) {
      const int64_t target = (total * x + 7) / 8;  // first tile whose preceding cost reaches the target
      while (g < ngroups && before + (int64_t)(tile_off[g + 1] - tile_off[g]) * cost[g] < target) {
        before += (int64_t)(tile_off[g + 1] - tile_off[g]) * cost[g];
        ++g;
      }
      t = g < ngroups ? tile_off[g] + (int)((target - before + cost[g] - 1) / cost[g]) : ntiles;
      if (t < m.first[x - 1]) t = m.first[x - 1];
      if (t > ntiles) t = ntiles;
    }
    m.first[x] = t;
    if (t - m.first[x - 1] > longest) longest = t - m.first[x - 1];
  }
  return longest * 8;
}

}  // namespace hgnn
