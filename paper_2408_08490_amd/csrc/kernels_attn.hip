// Attention variant of the layer (the paper evaluates R-GAT, Section 5.1, and names semantic fusion as the
// layer's last stage, Section 2.2), forward part:
//   projection   Z = X W_t per vertex type, all source rows                 (MFMA GEMM, weights read in place)
//   aggregation  one launch over the merged CSR: per row and head a softmax over the row's edges of
//                LeakyReLU(a_src . z_u + a_dst . z_v), evaluated in one pass with a running maximum
//   fusion       semantic attention: tanh MLP scores per relation segment (MFMA GEMM with the row reduction
//                in its epilogue), softmax over the relations of a destination type, weighted sum + bias + act
// Everything between the boundary's tensors (z, m, t, dm and the small statistics) is fp32 in both storage types; the
// kernels read parameters, the incoming gradient and the features in the storage type TS and widen them on load.
#include <cmath>
#include <cstring>

#include "attn_layer.h"
#include "gemm_core.h"
#include "long_rows.h"

namespace hgnn {

constexpr float kLeaky = 0.2f;
constexpr int kSemDim = 128;
constexpr int kAttnMaxH = 256;  // widest layer output (64 lanes x 16 bytes of fp32)

// four consecutive scalars of the storage type, as floats
template <typename T> struct Quad;
template <> struct Quad<float> {
  static __device__ __forceinline__ void load(float *f, const float *p) {
    const f32x4 v = *reinterpret_cast<const f32x4 *>(p);
    f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
  }
  static __device__ __forceinline__ void store(float *p, const float *f) {
    *reinterpret_cast<f32x4 *>(p) = f32x4{f[0], f[1], f[2], f[3]};
  }
};
template <> struct Quad<bf16> {
  static __device__ __forceinline__ void load(float *f, const bf16 *p) {
    const u32x2 v = *reinterpret_cast<const u32x2 *>(p);
    f[0] = __uint_as_float(v.x << 16);
    f[1] = __uint_as_float(v.x & 0xffff0000u);
    f[2] = __uint_as_float(v.y << 16);
    f[3] = __uint_as_float(v.y & 0xffff0000u);
  }
  static __device__ __forceinline__ void store(bf16 *p, const float *f) {
    *reinterpret_cast<u32x2 *>(p) = u32x2{pack2(f[0], f[1]), pack2(f[2], f[3])};
  }
};
typedef Quad<float> Q4;

__device__ __forceinline__ int find_le(const int32_t *off, int n, int x) {  // largest i in [0, n) with off[i] <= x
  int lo = 0, hi = n;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (off[mid] <= x) lo = mid; else hi = mid;
  }
  return lo;
}

// Sums over the lanes of a head (hl: a power of two, the same for the whole launch), for several values at once; every lane
// gets them.  Inside 16 lanes the adds take their operand from the other lane directly (DPP), which has no single move to the
// lane 4 away and inside 8 lanes adds neighbours first; a cross-lane read through LDS, with its latency, is left to wider heads.
// The scores stand in front of a softmax, a LeakyReLU and the next layers' ReLUs, so the order of their sums is fixed: pieces
// of four floats hl / 2 apart first, then hl / 4, down to neighbours.  The lanes therefore hold the pieces of 8 of them in
// bit-reversed places (head_piece), which costs nothing: they are one line of 128 bytes.  (Over 16 lanes, two lines, the
// aggregation with heads of 64 floats took 2 % longer.  With the pieces in the lanes' order a score moves by an fp32 rounding,
// and behind two hidden layers over 600k rows single units decided otherwise: input gradients off by up to their own size.)
__device__ __forceinline__ int head_piece(int lane, int hl) {   // the piece of its row that lane `lane` of a lane group holds
  if (hl >= 8) return (lane & ~5) | (lane & 1) << 2 | (lane & 4) >> 2;
  if (hl == 4) return (lane & ~3) | (lane & 1) << 1 | (lane & 2) >> 1;
  return lane;
}
template <int CTRL> __device__ __forceinline__ float other_lane(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int N> __device__ __forceinline__ void head_sums(float (&v)[N], int hl) {
#define HGNN_STEP(other)                       \
  {                                            \
    _Pragma("unroll") for (int i = 0; i < N; ++i) v[i] += other; \
  }
  if (hl >= 64) HGNN_STEP(__shfl_xor(v[i], 32))
  if (hl >= 32) HGNN_STEP(__shfl_xor(v[i], 16))
  if (hl >= 16) HGNN_STEP(other_lane<0x128>(v[i]))   // the sixteen turned by eight
  if (hl >= 2) HGNN_STEP(other_lane<0xb1>(v[i]))     // lanes 1 0 3 2: pieces min(hl, 8) / 2 apart
  if (hl >= 4) HGNN_STEP(other_lane<0x4e>(v[i]))     // lanes 2 3 0 1
  if (hl >= 8) HGNN_STEP(other_lane<0x141>(v[i]))    // the eight lanes mirrored: the other four hold one value
#undef HGNN_STEP
}
// A lane's four products of the destination's score, one after the other.
__device__ __forceinline__ float dot_in_order(const float (&a)[4], const float (&b)[4]) {
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < 4; ++j) s += a[j] * b[j];
  return s;
}

__device__ __forceinline__ float leaky(float s) { return s > 0.f ? s : kLeaky * s; }

// ------------------------------------------------------------------------------------------
// Products of an fp32 operand with a bf16 one on the bf16 matrix cores.  An fp32 value is the exact sum of three bf16
// values (8 + 8 + 8 significant bits), a product of two bf16 values is exact in fp32, so three MFMAs give what the fp32
// MFMA would, at 3/16 of its cost.  A tile of A (fp32, K contiguous) is split into its three planes on the way from the
// registers to LDS; B goes through the ordinary mover.  One LDS stage (74 KB, two blocks per CU: the other block's MFMAs
// cover a block's barriers), the next K-step's loads in flight during the MFMAs.  Where that does not come out finite
// (gemm_finite) the tile of A stays as it is, B is widened as it is read, and the fp32 MFMA multiplies them.
constexpr int kWideBK = 64, kWidePF = kWideBK + 4;   // pitch of a tile of A that is kept in fp32
template <int MI, int NI> struct WideLds {
  static constexpr int PA = kWideBK + 8, TM = 64 * MI, TN = 64 * NI;
  static constexpr int B_ELEMS = TN * PA > kWideBK * ks_pitch<bf16>(TN) ? TN * PA : kWideBK * ks_pitch<bf16>(TN);
  __attribute__((aligned(16))) bf16 a[3][TM * PA];
  __attribute__((aligned(16))) bf16 b[B_ELEMS];
};

template <int TM> struct WideMover {
  static constexpr int VPR = kWideBK / 4, NV = TM * VPR / kThreads, PA = kWideBK + 8;
  f32x4 reg[NV];
  // rows o0.. of A (clamped to the extent), K columns k0..k0+63
  __device__ __forceinline__ void load(const float *A, int lda, int extent, int o0, int k0, int k_end) {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int v = threadIdx.x + i * kThreads, r = v / VPR, c = (v % VPR) * 4;
      const int o = min(o0 + r, extent - 1);
      f32x4 x = *reinterpret_cast<const f32x4 *>(A + (int64_t)o * lda + min(k0 + c, k_end - 4));
      if (k0 + c >= k_end) x = f32x4{0.f, 0.f, 0.f, 0.f};
      reg[i] = x;
    }
  }
  template <typename F> __device__ __forceinline__ void store(bf16 (*a)[TM * PA], F f) {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int v = threadIdx.x + i * kThreads, r = v / VPR, c = (v % VPR) * 4;
      u32x2 w[3];
      split3(f(reg[i]), w);
#pragma unroll
      for (int p = 0; p < 3; ++p) *reinterpret_cast<u32x2 *>(a[p] + r * PA + c) = w[p];
    }
  }
};

// acc += f(A)[a0.., k] * B[k, b0..] over k in [0, K).  BKC: B is [b_extent x K] (K contiguous), else [K x b_extent].
// `f(piece, k)` maps four consecutive values of A starting at column k.
template <bool BKC, int MI, int NI, typename F>
__device__ __forceinline__ void wide_run(f32x16 (&acc)[MI][NI], WideLds<MI, NI> &sm, const float *A, int lda, int a_extent, int a0,
                                         const bf16 *B, int ldb, int b_extent, int b0, int K, F f) {
  constexpr int TM = 64 * MI, TN = 64 * NI, PA = kWideBK + 8, PB = BKC ? PA : ks_pitch<bf16>(TN);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = (wave >> 1) * 32 * MI, wn = (wave & 1) * 32 * NI;
  WideMover<TM> ma;
  TileMover<bf16, BKC ? TN : kWideBK, BKC ? kWideBK : TN, PB, BKC> mb;
  typename decltype(mb)::Offsets ob;
  ob.setup(ldb, b_extent, b0);
  ma.load(A, lda, a_extent, a0, 0, K);
  const bf16 *bt = BKC ? B + (int64_t)b0 * ldb : B + b0;
  mb.load_fast(ob, bt, K);
  for (int k0 = 0; k0 < K; k0 += kWideBK) {
    const int kc = k0 + (threadIdx.x % WideMover<TM>::VPR) * 4;
    ma.store(sm.a, [&](f32x4 v) { return f(v, kc); });
    mb.store(sm.b);
    __syncthreads();
    if (k0 + kWideBK < K) {
      ma.load(A, lda, a_extent, a0, k0 + kWideBK, K);
      mb.load_fast(ob, BKC ? bt + k0 + kWideBK : bt + (int64_t)(k0 + kWideBK) * ldb, K - k0 - kWideBK);
    }
    constexpr int NK = kWideBK / 16;
    bf16x8_t b[NK][NI];
#pragma unroll
    for (int ks = 0; ks < NK; ++ks)
#pragma unroll
      for (int j = 0; j < NI; ++j) b[ks][j] = frag_bf16<BKC, PB>(sm.b, wn + j * 32, ks, lane);
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      f32x16 part[NI];   // a K-step's sum, added by the vector unit: see mma_tile_split
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) part[j][v] = 0.f;
#pragma unroll
      for (int p = 2; p >= 0; --p)   // smallest plane first
#pragma unroll
        for (int ks = 0; ks < NK; ++ks) {
          const bf16x8_t a = frag_bf16<true, PA>(sm.a[p], wm + i * 32, ks, lane);
#pragma unroll
          for (int j = 0; j < NI; ++j) part[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b[ks][j], part[j], 0, 0, 0);
        }
      add_unscaled(acc[i], part, kSplitScale);
    }
    __syncthreads();
  }
}

// The same on the fp32 MFMA, for tiles that did not come out finite; nothing is prefetched, so that it needs no registers
// beside the other one's.
template <bool BKC, int MI, int NI, typename F>
__device__ __forceinline__ void wide_run_f32(f32x16 (&acc)[MI][NI], WideLds<MI, NI> &sm, const float *A, int lda, int a_extent, int a0,
                                             const bf16 *B, int ldb, int b_extent, int b0, int K, F f) {
  constexpr int TM = 64 * MI, TN = 64 * NI, PB = BKC ? kWideBK + 8 : ks_pitch<bf16>(TN);
  static_assert(TM * kWidePF * sizeof(float) <= sizeof(sm.a), "a tile of A in fp32 must fit the planes");
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));   // nothing of this is worth keeping in registers during wide_run
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = (wave >> 1) * 32 * MI, wn = (wave & 1) * 32 * NI;
  float *af = reinterpret_cast<float *>(&sm.a[0][0]);
#pragma unroll 1
  for (int k0 = 0; k0 < K; k0 += kWideBK) {
    {
#pragma unroll 1
      for (int v = tid; v < TM * (kWideBK / 4); v += kThreads) {
        const int r = v / (kWideBK / 4), c = (v % (kWideBK / 4)) * 4;
        f32x4 x = *reinterpret_cast<const f32x4 *>(A + (int64_t)min(a0 + r, a_extent - 1) * lda + min(k0 + c, K - 4));
        if (k0 + c >= K) x = f32x4{0.f, 0.f, 0.f, 0.f};
        *reinterpret_cast<f32x4 *>(af + r * kWidePF + c) = f(x, k0 + c);
      }
      TileMover<bf16, BKC ? TN : kWideBK, BKC ? kWideBK : TN, PB, BKC> mb;
      typename decltype(mb)::Offsets ob;
      ob.setup(ldb, b_extent, b0);
      mb.load_fast(ob, BKC ? B + (int64_t)b0 * ldb + k0 : B + (int64_t)k0 * ldb + b0, K - k0);
      mb.store(sm.b);
    }
    __syncthreads();
#pragma unroll 1
    for (int ks = 0; ks < kWideBK / 2; ++ks) {
      const int k = ks * 2 + (lane >> 5);
      float a[MI], b[NI];
#pragma unroll
      for (int i = 0; i < MI; ++i) a[i] = af[(wm + i * 32 + (lane & 31)) * kWidePF + k];
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        const int col = wn + j * 32 + (lane & 31);
        if constexpr (BKC) b[j] = to_float(sm.b[col * PB + k]);
        else b[j] = to_float(sm.b[k * PB + (ks_swizzled<bf16>(TN) ? ks_swizzle_col(col, k) : col)]);
      }
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    __syncthreads();
  }
}

// Hands the block's tile out of LDS in pieces of four columns: f(row, col, values) for rows below `rows`.  A thread's
// column is the same in all its pieces.
template <int MI, int NI, typename F>
__device__ __forceinline__ void tile_pieces(f32x16 (&acc)[MI][NI], float *stage, int rows, F f) {
  constexpr int TM = 64 * MI, TN = 64 * NI, P = TN + kOutPitchPad, VPR = TN / 4;
  HGNN_FOR_EACH_ACC({ stage[row * P + col] = val; })
  __syncthreads();
  const int c = (threadIdx.x % VPR) * 4;
#pragma unroll
  for (int i = 0; i < TM * VPR / kThreads; ++i) {
    const int r = threadIdx.x / VPR + i * (kThreads / VPR);
    if (r < rows) f(r, c, *reinterpret_cast<const f32x4 *>(stage + r * P + c));
  }
}

// LDS of a block that multiplies an fp32 matrix with one of the storage type.
template <typename TS, int MI> struct MixLds;
template <int MI> struct MixLds<bf16, MI> {
  WideLds<MI, 2> w;
  __device__ __forceinline__ float *stage() { return reinterpret_cast<float *>(&w); }
  static_assert(sizeof(WideLds<MI, 2>) >= sizeof(float) * 64 * MI * (128 + kOutPitchPad), "output tile must fit");
};
template <int MI> struct MixLds<float, MI> {
  GemmLds<float, MI, 2> g;
  __device__ __forceinline__ float *stage() { return reinterpret_cast<float *>(&g.a[0][0]); }
};

// AHEAD: K-steps of fp32 operands whose loads are under way.  One where a tile has up to four, on tiles of 128 rows: there the second set
// costs more than it brings, and in the backward it does not fit beside what `f` and the epilogue keep in registers (17 of a lane's were
// in scratch memory).  The launch, us, two steps / one: backward, 23k rows of 4 relations of 128 columns 85 / 73, 84k of 4 of 256 465 / 423;
// scores of 128 columns, 23k rows of 4 47.5 / 44, of 8 84.5 / 79.5.  Of 256 columns, eight steps, two are better (66.5 / 68.5), on tiles of 64
// rows too (a step on 200 targets 206.5 / 207.9).
template <bool BKC, int AHEAD, typename TS, int MI, typename F>
__device__ __forceinline__ void mix_run(f32x16 (&acc)[MI][2], MixLds<TS, MI> &sm, const float *A, int lda, int a_extent, int a0,
                                        const TS *B, int ldb, int b_extent, int b0, int K, F f) {
  if constexpr (sizeof(TS) == 2) {
    gemm_finite<float, true>(acc, [&](auto split) {
      if constexpr (split.value) wide_run<BKC>(acc, sm.w, A, lda, a_extent, a0, B, ldb, b_extent, b0, K, f);
      else wide_run_f32<BKC>(acc, sm.w, A, lda, a_extent, a0, B, ldb, b_extent, b0, K, f);
    });
  } else {
    const OneSeg<float, AHEAD> one{Seg<float>{A, B, lda, ldb, 0, K}};
    gemm_finite<float, true>(acc, [&](auto split) {
      gemm_run<float, true, true, BKC, split.value>(acc, sm.g, one, a_extent, a0, b_extent, b0, [&](auto &mv, int step) {
        const int kc = step * Mma<float>::BK + (threadIdx.x % (Mma<float>::BK / 4)) * 4;
        for (auto &r : mv.reg) r = __builtin_bit_cast(u32x4, f(__builtin_bit_cast(f32x4, r), kc));
      });
    });
  }
}

// ------------------------------------------------------------------------------------------
// Projection: Z[row_off[t] + i, :] = X_t[i, :] W_t for every source row of every type, fp32 result (the products of two
// bf16 numbers are exact in fp32).  Its first block also clears the score sums of the kernel after next.
template <typename TS, int MI>
__global__ void __launch_bounds__(kThreads, 2) attn_proj_kernel(TypeTab tt, PtrTab pt, SegTab tiles, int H, const TS *__restrict__ x,
                                                              float *__restrict__ z, double *__restrict__ wsum) {
  constexpr int BM = 64 * MI, BN = 64 * MI;
  __shared__ GemmLds<TS, MI, MI> sm;
  if (blockIdx.x == 0 && threadIdx.x < kMaxR) wsum[threadIdx.x] = 0.0;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int T_ = tt.num_types;
  if (tile >= tiles.tile_off[T_]) return;
  int t = 0;
  while (tile >= tiles.tile_off[t + 1]) ++t;
  const int tiles_n = (H + BN - 1) / BN;
  const int local = tile - tiles.tile_off[t];
  const int m0 = (local / tiles_n) * BM, n0 = (local % tiles_n) * BN;
  const int M = tt.row_off[t + 1] - tt.row_off[t], F = tt.in_dim[t];
  f32x16 acc[MI][MI];
  const OneSeg<TS> one{Seg<TS>{x + tt.elem_off[t], reinterpret_cast<const TS *>(pt.w_root[t]), F, H, 0, F}};
  gemm_finite<TS, true>(acc, [&](auto split) { gemm_run<TS, true, true, false, split.value>(acc, sm, one, M, m0, H, n0); });
  write_tile(acc, sm, z + ((int64_t)tt.row_off[t] + m0) * H + n0, H, M - m0, H - n0, [](float v, int, int) { return v; });
}

// ------------------------------------------------------------------------------------------
// Row pointers and column indices of the consecutive merged rows that a block walks, in LDS: row pointer -> index ->
// neighbour row are three dependent loads, and a row has three or four edges, so that without this a lane group spends
// most of its time on the first two.  Entries beyond kStageCols are read where they lie.
constexpr int kStageRows = 256, kStageCols = 1024;
struct RowStage {
  int32_t ptr[kStageRows + 1], col[kStageCols];
  // n <= kStageRows rows from merged row `row0` on; called by the whole block
  __device__ __forceinline__ void load(const LayerDev &L, int64_t row0, int n) {
    for (int i = threadIdx.x; i <= n; i += 256) ptr[i] = L.rowptr[row0 + i];
    __syncthreads();
    const int e0 = ptr[0], m = min(ptr[n] - e0, kStageCols);
    for (int i = threadIdx.x; i < m; i += 256) col[i] = L.colidx[e0 + i];
    __syncthreads();
  }
  __device__ __forceinline__ int column(const LayerDev &L, int e) const {
    const int i = e - ptr[0];
    return i < kStageCols ? col[i] : L.colidx[e];
  }
};

// Aggregation.  Blocks are cut per relation (the relation, its vectors and its rows are then the same for the whole
// block).  A group of `lpr` lanes owns one merged row at a time; a lane holds its q-th four floats (head_piece); `hl` lanes form
// a head.
// Softmax over the row's edges in one pass: running maximum m, running sum l and accumulator rescaled whenever the
// maximum grows; four neighbour rows in flight.  Bound: the gather of fp32 rows (1 KB at H = 256; 2.3 GB through the L2s at
// 6.5 TB/s, the caches in front of HBM included) and, close behind, the vector unit.  561k rows of 1.6M edges: 425 us with a
// chain of three loads and cross-lane reads through LDS on every row, 355 with both gone.
template <typename TS, bool PAST>
__global__ void __launch_bounds__(256) attn_agg_kernel(LayerDev L, RelRows rr, AttnPtrs ap, int H, int heads, int lpr_log2, int hl,
                                                       int rpg, const float *__restrict__ z, float *__restrict__ mout,
                                                       float *__restrict__ mx, float *__restrict__ ls) {
  __shared__ RowStage st;
  const int gpb = 256 >> lpr_log2;
  const int q = head_piece(threadIdx.x & ((1 << lpr_log2) - 1), hl), grp = threadIdx.x >> lpr_log2;
  const int r = wave_find(rr.tile_off, rr.n, (int)blockIdx.x);
  const int row0 = rr.row_off[r], M = rr.row_off[r + 1] - row0;
  const int v0 = ((int)blockIdx.x - rr.tile_off[r]) * gpb * rpg, rows = min(gpb * rpg, M - v0);
  const float *zd = z + (int64_t)(rr.zdst[r] + v0) * H + q * 4;
  const float *zq = z + q * 4;
  const int k = (q * 4) / (H / heads);
  float as[4], ad[4];
  Quad<TS>::load(as, reinterpret_cast<const TS *>(ap.a_src[r]) + q * 4);
  Quad<TS>::load(ad, reinterpret_cast<const TS *>(ap.a_dst[r]) + q * 4);
  st.load(L, row0 + v0, rows);
  for (int i = grp; i < rows; i += gpb) {
    const int64_t rho = row0 + v0 + i;
    const int e0 = st.ptr[i], e1 = st.ptr[i + 1];
    float zv[4], acc[4] = {0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, l = 0.f;
    if (e1 > e0) {
      float zu[4][4], s[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) Q4::load(zu[j], zq + (int64_t)st.column(L, min(e0 + j, e1 - 1)) * H);
      Q4::load(zv, zd + (int64_t)i * H);
      float sd[1] = {dot_in_order(ad, zv)};
      head_sums(sd, hl);
      for (int e = e0;;) {
#pragma unroll
        for (int j = 0; j < 4; ++j) s[j] = (as[0] * zu[j][0] + as[1] * zu[j][1]) + (as[2] * zu[j][2] + as[3] * zu[j][3]);
        head_sums(s, hl);
#pragma unroll
        for (int j = 0; j < 4; ++j) s[j] = e + j < e1 ? leaky(s[j] + sd[0]) : -INFINITY;
        const float mn = fmaxf(m, fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])));
        const float c = __expf(m - mn);
        float p[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) p[j] = __expf(s[j] - mn);
        l = l * c + ((p[0] + p[1]) + (p[2] + p[3]));
#pragma unroll
        for (int d = 0; d < 4; ++d)
          acc[d] = acc[d] * c + ((p[0] * zu[0][d] + p[1] * zu[1][d]) + (p[2] * zu[2][d] + p[3] * zu[3][d]));
        m = mn;
        e += 4;
        if (e >= e1) break;
#pragma unroll
        for (int j = 0; j < 4; ++j) Q4::load(zu[j], zq + (int64_t)st.column(L, min(e + j, e1 - 1)) * H);
      }
      const float inv = 1.f / l;
#pragma unroll
      for (int d = 0; d < 4; ++d) acc[d] *= inv;
    }
    // PAST: the caches keep what the L2 holds of popular neighbours (573 MB of aggregates: fetched 1.7 GB for the 2.2 GB asked for;
    // 366 -> 355 us).
    const f32x4 out = {acc[0], acc[1], acc[2], acc[3]};
    if constexpr (PAST) __builtin_nontemporal_store(out, reinterpret_cast<f32x4 *>(mout + rho * H + q * 4));
    else *reinterpret_cast<f32x4 *>(mout + rho * H + q * 4) = out;
    if ((q & (hl - 1)) == 0) {
      mx[rho * heads + k] = e1 > e0 ? m : 0.f;
      ls[rho * heads + k] = l;
    }
  }
}

// ------------------------------------------------------------------------------------------
// Semantic scores: t = tanh(m W_s + b_s) stored for the backward pass; wsum[r] += sum over the segment's rows of q . t
// The blocks' sums are added in 64 bits: in 32 their order, which is not fixed, moved a relation's weight by a rounding and
// with it every row of the output, and single units of the layers behind decided otherwise from one run to the next.
// The blocks take the rows from the end: what the kernel in front wrote last is still in the memory-side cache (256 MB)
// when it is read first, and the kernel behind, from the start again, finds what this one touched last.  The same order in
// the backward's launch between mask and aggregation (561k rows, m and dm of 573 MB each, us: scores 238 -> 230, fusion
// 168 -> 161, backward 630 -> 617 and the aggregation's rows behind it 569 -> 558).
template <typename TS, int MI, int AHEAD>
__global__ void __launch_bounds__(kThreads, 2) attn_sem_kernel(RelRows rr, int H, const float *__restrict__ mbuf, const TS *__restrict__ w_sem,
                                                             const TS *__restrict__ b_sem, const TS *__restrict__ q_sem,
                                                             float *__restrict__ tbuf, double *__restrict__ wsum) {
  constexpr int TM = 64 * MI;
  __shared__ MixLds<TS, MI> sm;
  __shared__ float red[4];
  const int b = (int)(gridDim.x - 1 - blockIdx.x);
  const int r = wave_find(rr.tile_off, rr.n, b);
  const int m0 = (b - rr.tile_off[r]) * TM;
  const int64_t row0 = rr.row_off[r];
  const int M = rr.row_off[r + 1] - (int)row0;
  f32x16 acc[MI][2];
  mix_run<false, AHEAD>(acc, sm, mbuf + row0 * H, H, M, m0, w_sem, kSemDim, kSemDim, 0, H, [](f32x4 v, int) { return v; });
  float bs[4], qs[4], part = 0.f;
  const int cc = (threadIdx.x % (kSemDim / 4)) * 4;
  Quad<TS>::load(bs, b_sem + cc);
  Quad<TS>::load(qs, q_sem + cc);
  tile_pieces(acc, sm.stage(), M - m0, [&](int row, int col, f32x4 v) {
    float t[4] = {tanhf(v.x + bs[0]), tanhf(v.y + bs[1]), tanhf(v.z + bs[2]), tanhf(v.w + bs[3])};
    part += (t[0] * qs[0] + t[1] * qs[1]) + (t[2] * qs[2] + t[3] * qs[3]);
    Q4::store(tbuf + (row0 + m0 + row) * kSemDim + col, t);
  });
  for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = part;
  __syncthreads();
  if (threadIdx.x == 0) unsafeAtomicAdd(wsum + r, (double)(red[0] + red[1] + red[2] + red[3]));   // device memory: the hardware's add
}

// beta[r] = softmax over the relations with the same destination type of wsum[r] / M_d, for all relations by the first
// threads of a block.  `wsum` is in LDS: each thread walks all of it twice (108 relations, a layer's forward: read and
// converted from global memory on the way 64.4 us, 52.9 so).
__device__ __forceinline__ void relation_softmax(const RelRows &rr, const float *wsum, float *out) {
  const int r = threadIdx.x;
  if (r >= rr.n) return;
  const int d = rr.dst[r], M = rr.row_off[r + 1] - rr.row_off[r];
  if (M == 0) {
    out[r] = 0.f;
    return;
  }
  float mxv = -INFINITY, s = 0.f;
  for (int o = 0; o < rr.n; ++o)
    if (rr.dst[o] == d) mxv = fmaxf(mxv, wsum[o] / (float)M);
  for (int o = 0; o < rr.n; ++o)
    if (rr.dst[o] == d) s += __expf(wsum[o] / (float)M - mxv);
  out[r] = __expf(wsum[r] / (float)M - mxv) / s;
}

// h[v] = act( sum_{r -> type(v)} beta_r m[rel_row_off[r] + v] + b ).  Every block takes the softmax over the relations
// itself (a few hundred flops; as a launch of one block it cost 5 us); the first one writes it out for the backward.
// A lane group takes U rows, their loads of one relation in flight together: bound by the read of m (169k rows of 1 KB, 561k
// of m: one row after the other 161 us, four at once 132, 5 TB/s).
template <typename TS, int U>
__global__ void __launch_bounds__(256) attn_fuse_kernel(RelRows rr, TypeTiles ty, RelsOfType ro, PtrTab pt, int H, int relu, int lpr_log2,
                                                        const float *__restrict__ mbuf, const double *__restrict__ wsum,
                                                        float *__restrict__ beta, TS *__restrict__ h) {
  __shared__ float sb[kMaxR], sw[kMaxR];
  if (threadIdx.x < rr.n) sw[threadIdx.x] = (float)wsum[threadIdx.x];
  __syncthreads();
  relation_softmax(rr, sw, sb);
  __syncthreads();
  if (blockIdx.x == 0 && threadIdx.x < rr.n) beta[threadIdx.x] = sb[threadIdx.x];
  const int gpb = 256 >> lpr_log2;
  const int q = threadIdx.x & ((1 << lpr_log2) - 1), grp = threadIdx.x >> lpr_log2;
  const int d = wave_find(ty.tile_off, ty.n, (int)blockIdx.x);
  const int M = ty.row_off[d + 1] - ty.row_off[d];
  const int v0 = ((int)blockIdx.x - ty.tile_off[d]) * gpb * U + grp;
  if (v0 >= M) return;
  float acc[U][4];
#pragma unroll
  for (int c = 0; c < 4; ++c) acc[0][c] = 0.f;
  if (pt.bias[d]) Quad<TS>::load(acc[0], reinterpret_cast<const TS *>(pt.bias[d]) + q * 4);
#pragma unroll
  for (int u = 1; u < U; ++u)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[u][c] = acc[0][c];
  for (int j = ro.first[d]; j < ro.first[d + 1]; ++j) {
    const int r = ro.rel[j];
    const float b = sb[r];
    const float *mr = mbuf + (int64_t)rr.row_off[r] * H + q * 4;
    float mv[U][4];
#pragma unroll
    for (int u = 0; u < U; ++u) Q4::load(mv[u], mr + (int64_t)min(v0 + u * gpb, M - 1) * H);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[u][c] += b * mv[u][c];
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    if (v0 + u * gpb >= M) break;
    if (relu) {
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[u][c] = fmaxf(acc[u][c], 0.f);
    }
    Quad<TS>::store(h + ((int64_t)ty.row_off[d] + v0 + u * gpb) * H + q * 4, acc[u]);
  }
}

// ------------------------------------------------------------------------------------------
// launchers (forward)
static int log2_exact(int n) {
  int l = 0;
  while ((1 << l) < n) ++l;
  return l;
}

// Tiles of `rows` rows, cut per relation; returns their number.
static int tile_relations(RelRows &rr, int rows) {
  rr.tile_off[0] = 0;
  for (int r = 0; r < rr.n; ++r) rr.tile_off[r + 1] = rr.tile_off[r] + (rr.row_off[r + 1] - rr.row_off[r] + rows - 1) / rows;
  return rr.tile_off[rr.n];
}
static int tile_types(TypeTiles &ty, int rows) {
  ty.tile_off[0] = 0;
  for (int t = 0; t < ty.n; ++t) ty.tile_off[t + 1] = ty.tile_off[t] + (ty.row_off[t + 1] - ty.row_off[t] + rows - 1) / rows;
  return ty.tile_off[ty.n];
}
// Rows a lane group walks: one while that leaves fewer than `blocks` blocks, at most `most`.
static int rows_per_group(int64_t rows, int gpb, int blocks, int most) {
  int n = 1;
  while (n < most && rows >= (int64_t)gpb * n * 2 * blocks) n *= 2;
  return n;
}

hgnn_status launch_attn_proj(hipStream_t s, int dtype, const TypeTab &tt, const PtrTab &w_type_as_root, int H, const void *x, float *z,
                             double *wsum) {
  SegTab tiles;
  std::memset(&tiles, 0, sizeof(tiles));
  tiles.num_segs = tt.num_types;
  int mi = 2;
  for (;; mi = 1) {   // 64x64 tiles where 128x128 ones would leave compute units without a block
    const int e = 64 * mi, tn = (H + e - 1) / e;
    for (int t = 0; t < tt.num_types; ++t)
      tiles.tile_off[t + 1] = tiles.tile_off[t] + ((tt.row_off[t + 1] - tt.row_off[t] + e - 1) / e) * tn;
    if (mi == 1 || tiles.tile_off[tt.num_types] >= 512) break;
  }
  const int n = tiles.tile_off[tt.num_types];
  if (n == 0) return HGNN_OK;
  dim3 grid(round_up8(n)), blk(kThreads);
#define HGNN_PROJ(TY, MI_) HGNN_LAUNCH((attn_proj_kernel<TY, MI_>), grid, blk, 0, s, tt, w_type_as_root, tiles, H, (const TY *)x, z, wsum)
  if (dtype == HGNN_BF16) {
    if (mi == 2) HGNN_PROJ(bf16, 2); else HGNN_PROJ(bf16, 1);
  } else {
    if (mi == 2) HGNN_PROJ(float, 2); else HGNN_PROJ(float, 1);
  }
#undef HGNN_PROJ
  HGNN_HIP(hipGetLastError());
  return HGNN_OK;
}

// Aggregates go past the caches where the memory-side one (256 MB) cannot hold them beside the projected rows until the scores'
// kernel reads them (forward of a layer, us, through the caches / past them: 160k rows from 35k of 256 floats, 200 MB, 191 / 207;
// 110k from 179k, 290 MB, 168.9 / 165.8; 561k from 607k, 1.2 GB, 871 / 858).
constexpr int64_t kMemorySideCache = (int64_t)256 << 20;

hgnn_status launch_attn_agg(hipStream_t s, int dtype, const LayerDev &L, RelRows rr, const AttnPtrs &ap, int H, int heads,
                            const float *z, float *mout, float *mx, float *ls) {
  if (L.rows == 0) return HGNN_OK;
  const int lpr = H / 4, l2 = log2_exact(lpr), hl = (H / heads) / 4, gpb = 256 >> l2;
  const int rpg = std::min(kStageRows / gpb, rows_per_group(L.rows, gpb, 4096, 4));
  const bool past = ((int64_t)L.rows + L.src_rows) * H * 4 > kMemorySideCache;
  dim3 grid(tile_relations(rr, gpb * rpg));
#define HGNN_AGG(TY, PAST) HGNN_LAUNCH((attn_agg_kernel<TY, PAST>), grid, dim3(256), 0, s, L, rr, ap, H, heads, l2, hl, rpg, z, mout, mx, ls)
  if (dtype == HGNN_BF16) {
    if (past) HGNN_AGG(bf16, true); else HGNN_AGG(bf16, false);
  } else {
    if (past) HGNN_AGG(float, true); else HGNN_AGG(float, false);
  }
#undef HGNN_AGG
  HGNN_HIP(hipGetLastError());
  return HGNN_OK;
}

// Rows per tile of the semantic-attention GEMMs: 64 where 128 would leave compute units without a block.
static int sem_tile_rows(RelRows &rr) { return tile_relations(rr, 128) >= 512 ? 128 : 64; }

hgnn_status launch_attn_sem(hipStream_t s, int dtype, RelRows rr, int H, const float *mbuf, const void *w_sem, const void *b_sem,
                            const void *q_sem, float *tbuf, double *wsum) {
  const int tm = sem_tile_rows(rr);
  const int n = tile_relations(rr, tm);
  if (n == 0) return HGNN_OK;
#define HGNN_SEM(TY, MI_, AHEAD_)                                                                                               \
  HGNN_LAUNCH((attn_sem_kernel<TY, MI_, AHEAD_>), dim3(n), dim3(kThreads), 0, s, rr, H, mbuf, (const TY *)w_sem, (const TY *)b_sem, \
              (const TY *)q_sem, tbuf, wsum)
  if (dtype == HGNN_BF16) {
    if (tm == 128) HGNN_SEM(bf16, 2, 2); else HGNN_SEM(bf16, 1, 2);
  } else if (tm == 128) {
    if (H <= 128) HGNN_SEM(float, 2, 1); else HGNN_SEM(float, 2, 2);
  } else {
    HGNN_SEM(float, 1, 2);
  }
#undef HGNN_SEM
  HGNN_HIP(hipGetLastError());
  return HGNN_OK;
}

static void rels_of_type(const RelRows &rr, int num_types, RelsOfType &ro) {
  std::memset(&ro, 0, sizeof(ro));
  int n = 0;
  for (int d = 0; d < num_types; ++d) {
    ro.first[d] = (uint16_t)n;
    for (int r = 0; r < rr.n; ++r)
      if (rr.dst[r] == d) ro.rel[n++] = (uint8_t)r;
  }
  ro.first[num_types] = (uint16_t)n;
}

static void dst_types(const TypeTab &tt, TypeTiles &ty) {
  std::memset(&ty, 0, sizeof(ty));
  ty.n = tt.num_types;
  for (int t = 0; t <= ty.n; ++t) ty.row_off[t] = tt.out_row_off[t];
}

hgnn_status launch_attn_fuse(hipStream_t s, int dtype, const TypeTab &tt, const RelRows &rr, const PtrTab &pt, int H, int relu,
                             const float *mbuf, const double *wsum, float *beta, void *h) {
  TypeTiles ty;
  dst_types(tt, ty);
  const int64_t rows = ty.row_off[ty.n];
  if (rows == 0) return HGNN_OK;
  RelsOfType ro;
  rels_of_type(rr, tt.num_types, ro);
  const int l2 = log2_exact(H / 4), gpb = 256 >> l2;
  const bool four = rows >= (int64_t)gpb * 4 * 1024;   // while that leaves four blocks per compute unit
  dim3 grid(tile_types(ty, gpb * (four ? 4 : 1)));
#define HGNN_FUSE(TY, U_) HGNN_LAUNCH((attn_fuse_kernel<TY, U_>), grid, dim3(256), 0, s, rr, ty, ro, pt, H, relu, l2, mbuf, wsum, beta, (TY *)h)
  if (dtype == HGNN_BF16) {
    if (four) HGNN_FUSE(bf16, 4); else HGNN_FUSE(bf16, 1);
  } else {
    if (four) HGNN_FUSE(float, 4); else HGNN_FUSE(float, 1);
  }
#undef HGNN_FUSE
  HGNN_HIP(hipGetLastError());
  return HGNN_OK;
}

// ==========================================================================================
// Backward part.
//   fusion      G' = G [h > 0] and db; dbeta_r = sum_v G'_v . m_v^r in the same pass;
//               du = coef_r q (1 - t^2) with coef from the softmax over relations (taken in each block that needs it),
//               never stored: dW_s += m^T du, dq, db_s (column sums) and dm = beta_r G'_v + du W_s^T build it as they load t
//   aggregation per merged row, one pass over its edges: alpha from the saved maximum and sum, dalpha = dm . z_u,
//               (alpha, dalpha) stored per edge and sum_u alpha_u dalpha_u per row, so that the score gradient
//               ds = alpha (dalpha - sum) LeakyReLU' can be formed where it is used; per source row (transpose):
//               dz = sum over its edges of alpha dm_v + ds a_src, plus, for a destination row, sum_r (sum_u ds) a_dst
//   projection  dW_t = X_t^T dZ_t and dX_t = dZ_t W_t^T run on the layer GEMMs of the mean variant.
// ==========================================================================================
struct ZeroList {
  float *p[2 * kMaxR + 2 * kMaxT + 8];
  int32_t n[2 * kMaxR + 2 * kMaxT + 8];
  int32_t count;
};
__global__ void attn_zero_kernel(ZeroList zl) {
  const int i = blockIdx.y;
  if (i >= zl.count) return;
  float *p = zl.p[i];
  for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < zl.n[i]; j += gridDim.x * blockDim.x) p[j] = 0.f;
}

// The rows of a block against N relations of their type (FIRST: also gp and the bias sums): a lane group takes four rows at a time,
// the loads of all N relations for them are under way together, and a lane keeps its share of the dots until its last row.
template <typename TS, int N, bool FIRST>
__device__ __forceinline__ void mask_dbeta_rows(const float *const *mr, float *dot, float *bsum, int64_t row0, int M, int vb, int gpb, int trips,
                                                int H, int q, int relu, const TS *__restrict__ g, const TS *__restrict__ h, TS *__restrict__ gp) {
  const TS *hp = relu ? h : g;
  for (int it = 0; it < trips && vb < M; ++it, vb += gpb * 4) {   // whole groups
    float gv[4][4], hv[4][4], mv[N ? N : 1][4][4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t at = (row0 + min(vb + u * gpb, M - 1)) * H + q * 4;
      Quad<TS>::load(gv[u], g + at);
      Quad<TS>::load(hv[u], hp + at);
    }
#pragma unroll
    for (int j = 0; j < N; ++j)
#pragma unroll
      for (int u = 0; u < 4; ++u) Q4::load(mv[j][u], mr[j] + (int64_t)min(vb + u * gpb, M - 1) * H);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool on = vb + u * gpb < M;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if (!on || (relu && !(hv[u][c] > 0.f))) gv[u][c] = 0.f;
        if (FIRST) bsum[c] += gv[u][c];
      }
      if (FIRST && relu && on) Quad<TS>::store(gp + (row0 + vb + u * gpb) * H + q * 4, gv[u]);
    }
#pragma unroll
    for (int j = 0; j < N; ++j)
#pragma unroll
      for (int u = 0; u < 4; ++u)
        dot[j] += (gv[u][0] * mv[j][u][0] + gv[u][1] * mv[j][u][1]) + (gv[u][2] * mv[j][u][2] + gv[u][3] * mv[j][u][3]);
  }
}

// One pass over the incoming gradient: mask by the activation (gp), bias gradient, and dbeta[r] += sum of G'[v] . m[row]
// for every relation that ends in the row's type, up to four of them at a time.  Bound: the read of m where that is large (169k rows
// of 256 columns with 561k aggregates, bf16: one relation after the other 177 us, so 156 or 5.3 TB/s), a chain of latencies where it is not
// (1.3k rows of 128 columns in fp32 10 -> 8.7 us).  One after the other, with seven wavefronts on a SIMD instead of three, also: 23k rows of
// 128 columns in fp32, 1 relation 26.3 / 27, 4 30.5 / 30, 8 36.8 / 37; 84k of 256 in bf16, 1 67 / 57, 5 125 / 121; but 150k, 8 relations
// without an activation, where the gradients are read twice, 230 / 250.
template <typename TS>
__global__ void __launch_bounds__(256) attn_mask_dbeta_kernel(RelRows rr, TypeTiles ty, RelsOfType ro, GradPtrTab gt, int H, int relu,
                                                              int lpr_log2, int trips, const TS *__restrict__ g, const TS *__restrict__ h,
                                                              TS *__restrict__ gp, const float *__restrict__ mbuf,
                                                              float *__restrict__ dbeta) {
  __shared__ float part[kMaxR];
  __shared__ float s_b[kAttnMaxH];
  const int lpr = 1 << lpr_log2, gpb = 256 >> lpr_log2;
  const int q = threadIdx.x & (lpr - 1), grp = threadIdx.x >> lpr_log2;
  const int d = wave_find(ty.tile_off, ty.n, (int)blockIdx.x);
  const int M = ty.row_off[d + 1] - ty.row_off[d];
  const int vb = ((int)blockIdx.x - ty.tile_off[d]) * gpb * 4 * trips + grp;
  const int j0 = ro.first[d], j1 = ro.first[d + 1];
  for (int i = threadIdx.x; i < kMaxR; i += 256) part[i] = 0.f;
  for (int i = threadIdx.x; i < kAttnMaxH; i += 256) s_b[i] = 0.f;
  __syncthreads();
  float bsum[4] = {0.f, 0.f, 0.f, 0.f};
  int j = j0;
  do {
    const int n = min(4, j1 - j);
    const float *mr[4];
    float dot[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < 4; ++k) mr[k] = k < n ? mbuf + (int64_t)rr.row_off[ro.rel[j + k]] * H + q * 4 : mbuf;
#define HGNN_ROWS(N_, F_) mask_dbeta_rows<TS, N_, F_>(mr, dot, bsum, ty.row_off[d], M, vb, gpb, trips, H, q, relu, g, h, gp)
    if (j == j0) {
      if (n == 4) HGNN_ROWS(4, true);
      else if (n == 3) HGNN_ROWS(3, true);
      else if (n == 2) HGNN_ROWS(2, true);
      else if (n == 1) HGNN_ROWS(1, true);
      else HGNN_ROWS(0, true);
    } else if (n > 2) {
      if (n == 4) HGNN_ROWS(4, false); else HGNN_ROWS(3, false);
    } else {
      if (n == 2) HGNN_ROWS(2, false); else HGNN_ROWS(1, false);
    }
#undef HGNN_ROWS
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (k >= n) break;
      for (int o = 32; o > 0; o >>= 1) dot[k] += __shfl_xor(dot[k], o);
      if ((threadIdx.x & 63) == 0) atomicAdd(&part[j + k - j0], dot[k]);
    }
    j += 4;
  } while (j < j1);
  float *db = gt.dbias[d];
  if (db) {
#pragma unroll
    for (int c = 0; c < 4; ++c) atomicAdd(&s_b[q * 4 + c], bsum[c]);
  }
  __syncthreads();
  if (db)
    for (int i = threadIdx.x; i < H; i += 256) atomicAdd(db + i, s_b[i]);
  for (int i = threadIdx.x; i < j1 - j0; i += 256) atomicAdd(dbeta + ro.rel[j0 + i], part[i]);
}

// coef_r = beta_r (dbeta_r - sum_r' beta_r' dbeta_r') / M_d, the factor of q (1 - t^2) in du.  A lane takes a relation each, so
// that the sum costs one memory round trip; r is the same for the wavefront.  (561k rows, 8 relations, one after the other 620 us, so 601.)
typedef const RelRows __attribute__((address_space(4))) *rel_rows_t;   // an argument, read where it lies
__device__ __forceinline__ float relation_coef(rel_rows_t rr, const float *__restrict__ beta, const float *__restrict__ dbeta, int r) {
  const int d = rr->dst[r], lane = threadIdx.x & 63;
  const float br = beta[r], dbr = dbeta[r];
  float dot = 0.f;
  for (int o = lane; o < rr->n; o += 64)
    if (rr->dst[o] == d) dot += beta[o] * dbeta[o];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) dot += __shfl_xor(dot, o);
  return br * (dbr - dot) / (float)(rr->row_off[r + 1] - rr->row_off[r]);
}

// dW_s += m^T du, dq += coef sum t, db_s += coef q sum (1 - t^2) over `rows` rows of one relation: the block multiplies
// m^T (1 - t^2) and scales the result.  Both operands are split into planes on the way (six bf16 MFMAs per product): the
// splitting and the LDS traffic of two fp32 tiles per K-step bound this part (on the fp32 MFMA, whose rate bound it, the
// launch with dm took 739 us on 560k rows, so 600).
__device__ __forceinline__ void attn_dws_part(GemmLds<float, 2, 2> &sm, const float *m, const float *t, int64_t row0, int k_begin, int k_end,
                                              int H, int f0, float coef, const float *qs, float *__restrict__ dws,
                                              float *__restrict__ dq, float *__restrict__ dbs) {
  f32x16 acc[2][2];
  const OneSeg<float> one{Seg<float>{m + row0 * H, t + row0 * kSemDim, H, kSemDim, k_begin, k_end}};
  float st[4], s1[4];
  gemm_finite<float, true>(acc, [&](auto split) {
#pragma unroll
    for (int c = 0; c < 4; ++c) st[c] = s1[c] = 0.f;
    gemm_run<float, true, false, false, split.value>(acc, sm, one, H, f0, kSemDim, 0, NoXform(), [&](auto &mv, int) {
      int i = 0;
      for (auto &rg : mv.reg) {
        const f32x4 v = __builtin_bit_cast(f32x4, rg);
        const f32x4 w = {1.f - v.x * v.x, 1.f - v.y * v.y, 1.f - v.z * v.z, 1.f - v.w * v.w};
        if ((mv.okmask >> i) & 1u) {
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            st[c] += v[c];
            s1[c] += w[c];
          }
        }
        rg = __builtin_bit_cast(u32x4, w);
        ++i;
      }
    });
  }, k_end - k_begin <= kFewTerms);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float qc[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) qc[j] = coef * qs[(wave & 1) * 64 + j * 32 + (lane & 31)];
  HGNN_FOR_EACH_ACC({
    if (f0 + row < H) atomicAdd(dws + (int64_t)(f0 + row) * kSemDim + col, val * qc[j_]);
  })
  if (f0 != 0) return;   // one block per row slice adds the column sums
  float *red = reinterpret_cast<float *>(&sm.a[0][0]);   // [8 row lanes][128], twice
  const int c0 = (threadIdx.x % 32) * 4, part = threadIdx.x / 32;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    red[part * kSemDim + c0 + c] = st[c];
    red[1024 + part * kSemDim + c0 + c] = s1[c];
  }
  __syncthreads();
  const int c = threadIdx.x & (kSemDim - 1), half = threadIdx.x >> 7;
  float s = 0.f;
#pragma unroll
  for (int p = 0; p < 8; ++p) s += red[half * 1024 + p * kSemDim + c];
  if (half == 0) atomicAdd(dq + c, coef * s);
  else atomicAdd(dbs + c, coef * qs[c] * s);
}

// dm[row] = du[row] W_s^T + beta_r G'[v], one tile of 64 MI rows x 128 columns.
template <typename TS, int MI>
__device__ __forceinline__ void attn_dm_part(MixLds<TS, MI> &sm, const float *t, const TS *__restrict__ w_sem, const TS *__restrict__ gp,
                                             float *__restrict__ dm, int64_t row0, int M, int m0, int n0, int H, float coef, float beta,
                                             const float *qs) {
  f32x16 acc[MI][2];
  mix_run<true, MI == 2 ? 1 : 2>(acc, sm, t + row0 * kSemDim, kSemDim, M, m0, w_sem, kSemDim, H, n0, kSemDim, [&](f32x4 v, int k) {
    const f32x4 q = *reinterpret_cast<const f32x4 *>(qs + k);
    return f32x4{coef * q.x * (1.f - v.x * v.x), coef * q.y * (1.f - v.y * v.y), coef * q.z * (1.f - v.z * v.z), coef * q.w * (1.f - v.w * v.w)};
  });
  tile_pieces(acc, sm.stage(), M - m0, [&](int row, int col, f32x4 v) {
    if (n0 + col >= H) return;
    float gv[4];
    Quad<TS>::load(gv, gp + (int64_t)(m0 + row) * H + n0 + col);
    float o[4] = {v.x + beta * gv[0], v.y + beta * gv[1], v.z + beta * gv[2], v.w + beta * gv[3]};
    Q4::store(dm + (row0 + m0 + row) * H + n0 + col, o);
  });
}

// Both products of the semantic attention's backward in ONE launch, their blocks interleaved: dW_s is bound by splitting its
// operands and by LDS, dm by memory, and neither depends on the other.
template <typename TS, int MI>
__global__ void __launch_bounds__(kThreads, 2) attn_sem_bwd_kernel(RelRows, RelRows, SemBwd p, int H, const float *__restrict__ mbuf,
                                                                 const float *__restrict__ tbuf, const TS *__restrict__ w_sem,
                                                                 const TS *__restrict__ q_sem, const TS *__restrict__ gp,
                                                                 const float *__restrict__ beta, const float *__restrict__ dbeta,
                                                                 float *__restrict__ dm, float *__restrict__ dws, float *__restrict__ dq,
                                                                 float *__restrict__ dbs) {
  union Lds {
    GemmLds<float, 2, 2> dw;
    MixLds<TS, MI> dm;
  };
  __shared__ Lds sm;
  __shared__ __attribute__((aligned(16))) float qs[kSemDim];
  const float qv = threadIdx.x < kSemDim ? to_float(q_sem[threadIdx.x]) : 0.f;
  const int64_t total = gridDim.x, b = total - 1 - blockIdx.x;   // from the end: see attn_sem_kernel
  const int before = (int)(b * p.n_dw / total), tiles_n = (H + 127) / 128;
  const bool dw = (int)((b + 1) * p.n_dw / total) > before;
  const int item = dw ? before : (int)b - before, col = item % tiles_n, tl = item / tiles_n;
  const rel_rows_t rr = (rel_rows_t)__builtin_amdgcn_kernarg_segment_ptr() + (dw ? 0 : 1);   // dwt or dmt
  const int r = __builtin_amdgcn_readfirstlane(wave_find(rr->tile_off, rr->n, tl)), k0 = tl - rr->tile_off[r];
  const int64_t row0 = rr->row_off[r];
  const int M = rr->row_off[r + 1] - (int)row0;
  const float coef = relation_coef(rr, beta, dbeta, r);
  if (threadIdx.x < kSemDim) qs[threadIdx.x] = qv;
  __syncthreads();
  if (dw)
    attn_dws_part(sm.dw, mbuf, tbuf, row0, k0 * p.dw_rows, min((k0 + 1) * p.dw_rows, M), H, col * 128, coef, qs, dws, dq, dbs);
  else
    attn_dm_part<TS, MI>(sm.dm, tbuf, w_sem, gp + (int64_t)rr->gdst[r] * H, dm, row0, M, k0 * 64 * MI, col * 128, H, coef, beta[r], qs);
}

// Aggregation backward, by merged row; blocks are cut per relation.  A lane group walks `rpg` rows and keeps the sums
// for da_src / da_dst in registers; the block's groups meet in LDS and leave with one atomic add per element.
// With ds_u = alpha_u f_u (x_u - X), f = LeakyReLU' (1 or 0.2), x_u = dalpha_u - c and X = sum_u alpha_u x_u, one pass over
// the edges is enough (two read every neighbour row twice): sum ds z = S1 - X S2 with S1 = sum alpha f x z and
// S2 = sum alpha f z, and likewise for sum ds.  ds does not depend on c (the alphas add up to 1), its rounding does: c has
// to lie where the weight is, so it is the weighted mean of the edges so far, moved (with the sums) before each four of
// them; X is then rounding only.  Relative to any one edge, S1 and X S2 cancel when that edge is far from the others and
// has next to no weight: sums of ten edges, fp32 against 64 bits: 1.2e-7 with the mean, 2.4e-7 with the first edge, 1.1e-4
// with a first edge 1000 times as long; two passes 1.3e-7.  The mean, c + X, per row and, per edge, (alpha with the sign of
// the score, dalpha) are stored for the pass over the transpose.
// Bound: the vector unit (70 % of the time at 561k rows of 1.6M edges); 675 -> 565 us with the rows' indices in LDS and the
// heads' sums on DPP adds.
template <typename TS>
__global__ void __launch_bounds__(256) attn_agg_bwd_rows_kernel(LayerDev L, RelRows rr, AttnPtrs ap, AttnPtrs dap, int H, int heads,
                                                                int lpr_log2, int hl, int rpg, const float *__restrict__ z,
                                                                const float *__restrict__ dm, const float *__restrict__ mx,
                                                                const float *__restrict__ ls, float2 *__restrict__ ead,
                                                                float *__restrict__ xsum, float *__restrict__ dsum) {
  __shared__ float s_das[kAttnMaxH], s_dad[kAttnMaxH];
  __shared__ RowStage st;
  const int gpb = 256 >> lpr_log2;
  const int q = head_piece(threadIdx.x & ((1 << lpr_log2) - 1), hl), grp = threadIdx.x >> lpr_log2;
  const int k = (q * 4) / (H / heads);
  const bool lead = (q & (hl - 1)) == 0;
  const int r = wave_find(rr.tile_off, rr.n, (int)blockIdx.x);
  const int row0 = rr.row_off[r], M = rr.row_off[r + 1] - row0;
  const int v0 = ((int)blockIdx.x - rr.tile_off[r]) * gpb * rpg, rows = min(gpb * rpg, M - v0);
  for (int i = threadIdx.x; i < H; i += 256) s_das[i] = s_dad[i] = 0.f;
  const float *zd = z + (int64_t)(rr.zdst[r] + v0) * H + q * 4, *zq = z + q * 4;
  float as[4], ad[4], das[4] = {0.f, 0.f, 0.f, 0.f}, dad[4] = {0.f, 0.f, 0.f, 0.f};
  Quad<TS>::load(as, reinterpret_cast<const TS *>(ap.a_src[r]) + q * 4);
  Quad<TS>::load(ad, reinterpret_cast<const TS *>(ap.a_dst[r]) + q * 4);
  st.load(L, row0 + v0, rows);
  for (int i = grp; i < rows; i += gpb) {
    const int64_t rho = row0 + v0 + i;
    const int e0 = st.ptr[i], e1 = st.ptr[i + 1];
    if (e1 == e0) {
      if (lead) {
        xsum[rho * heads + k] = 0.f;
        dsum[rho * heads + k] = 0.f;
      }
      continue;
    }
    float zv[4], g[4], zu[4][4];
#pragma unroll
    for (int j = 0; j < 4; ++j) Q4::load(zu[j], zq + (int64_t)st.column(L, min(e0 + j, e1 - 1)) * H);
    Q4::load(zv, zd + (int64_t)i * H);
    Q4::load(g, dm + rho * H + q * 4);
    const float mxk = mx[rho * heads + k], inv_l = 1.f / ls[rho * heads + k];
    float sdv[1] = {dot_in_order(ad, zv)};
    head_sums(sdv, hl);
    const float sd = sdv[0];
    float S1[4] = {0.f, 0.f, 0.f, 0.f}, S2[4] = {0.f, 0.f, 0.f, 0.f};
    float X = 0.f, w1 = 0.f, w2 = 0.f, c = 0.f, W = 0.f;
    for (int e = e0;;) {
      float ss[4], da[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        ss[j] = (as[0] * zu[j][0] + as[1] * zu[j][1]) + (as[2] * zu[j][2] + as[3] * zu[j][3]);
        da[j] = (g[0] * zu[j][0] + g[1] * zu[j][1]) + (g[2] * zu[j][2] + g[3] * zu[j][3]);
      }
      head_sums(ss, hl);
      head_sums(da, hl);
      float a[4], wg = 0.f, xg = X;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        a[j] = e + j < e1 ? __expf(leaky(ss[j] + sd) - mxk) * inv_l : 0.f;
        wg += a[j];
        xg += a[j] * (da[j] - c);
      }
      const float before = W, c_old = c;
      W += wg;
      if (W > 1e-30f) c += xg * __builtin_amdgcn_rcpf(W);   // below that no reciprocal, and nothing to be off by
      const float moved = c - c_old;
      X -= moved * before;
      w1 -= moved * w2;
#pragma unroll
      for (int i = 0; i < 4; ++i) S1[i] -= moved * S2[i];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const bool pos = ss[j] + sd > 0.f;
        const float af = pos ? a[j] : kLeaky * a[j], x = da[j] - c;
        X += a[j] * x;
        w1 += af * x;
        w2 += af;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          S1[i] += af * x * zu[j][i];
          S2[i] += af * zu[j][i];
        }
        if (lead && e + j < e1) ead[(int64_t)(e + j) * heads + k] = make_float2(pos ? a[j] : -a[j], da[j]);
      }
      e += 4;
      if (e >= e1) break;
#pragma unroll
      for (int j = 0; j < 4; ++j) Q4::load(zu[j], zq + (int64_t)st.column(L, min(e + j, e1 - 1)) * H);
    }
    const float ds = w1 - X * w2;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      das[i] += S1[i] - X * S2[i];
      dad[i] += ds * zv[i];
    }
    if (lead) {
      xsum[rho * heads + k] = c + X;
      dsum[rho * heads + k] = ds;
    }
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    atomicAdd(&s_das[q * 4 + c], das[c]);
    atomicAdd(&s_dad[q * 4 + c], dad[c]);
  }
  __syncthreads();
  float *ps = reinterpret_cast<float *>(const_cast<void *>(dap.a_src[r])), *pd = reinterpret_cast<float *>(const_cast<void *>(dap.a_dst[r]));
  for (int i = threadIdx.x; i < H; i += 256) {
    atomicAdd(ps + i, s_das[i]);
    atomicAdd(pd + i, s_dad[i]);
  }
}

// Aggregation backward, by source row (transpose): dz[c] = sum_j alpha_j dm[crow_j] + ds_j a_src[rel(crow_j)]
// (+ for a destination row: sum over the relations ending in its type of dsum[row] a_dst[r]).  The entries of a row
// ascend by merged row, so those of one relation are neighbours: their ds are summed and meet a_src once.
// The first blocks take the rows longer than kLongRow in pieces (long_rows.h); the others `rpb` consecutive
// source rows each.  Such a block first brings the row pointers and then all entries of its rows to LDS (two dependent
// loads per block, where a lane group per row spent them on every row of one or two entries), and its lane groups walk an
// equal number of rows each as one list of entries, four rows of dm in flight whatever rows they belong to.
// 569k source rows, 1.6M entries: 701 + 27 (the long rows' own launch) -> 497 us, 2.3 GB through the L2s.  Up to eight rows
// per lane group, fewer where the launch would have less than eight blocks per compute unit.
// The result leaves in the storage type (the projection's backward reads it there).
constexpr int kColRows = 64, kColEntries = kColRows * kLongRow;   // of a block, at most
static_assert(kColEntries >= 4 * kChunk, "the entries of four pieces");

// What a lane group does with its entries and its rows; lane q holds four floats of a row.
template <typename TS> struct ColSum {
  const RelRows &rr;
  const RelsOfType &ro;
  const AttnPtrs &ap;
  const float *dm, *xsum, *dsum;
  const float2 *ead;
  const int32_t *s_off;   // rr.row_off in LDS
  int H, heads, q, k;
  float acc[4] = {0.f, 0.f, 0.f, 0.f}, sds = 0.f;
  int r = -1;   // relation of the entries summed in sds

  __device__ __forceinline__ void flush() {
    if (r < 0) return;
    float as[4];
    Quad<TS>::load(as, reinterpret_cast<const TS *>(ap.a_src[r]) + q * 4);
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] += sds * as[i];
    sds = 0.f;
    r = -1;
  }
  // four entries; use(u): whether entry u counts, called in order before it is added
  template <typename Use> __device__ __forceinline__ void add4(const int (&rho)[4], const int (&e)[4], const int (&rel)[4], Use use) {
    float g[4][4], xs[4];
    float2 ad[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      Q4::load(g[u], dm + (int64_t)rho[u] * H + q * 4);
      ad[u] = ead[(int64_t)e[u] * heads + k];
      xs[u] = xsum[(int64_t)rho[u] * heads + k];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (!use(u)) break;
      if (rel[u] != r) {
        flush();
        r = rel[u];
      }
      const bool pos = !(__float_as_uint(ad[u].x) >> 31);
      const float a = fabsf(ad[u].x);
      sds += a * (ad[u].y - xs[u]) * (pos ? 1.f : kLeaky);
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i] += a * g[u][i];
    }
  }
  // the term of a destination row: vertex v of type t
  __device__ __forceinline__ void add_destination(int t, int v) {
    const int j1 = ro.first[t + 1];
    for (int j = ro.first[t]; j < j1; j += 4) {
      float sv[4], ad[4][4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int o = ro.rel[min(j + u, j1 - 1)];
        sv[u] = dsum[((int64_t)s_off[o] + v) * heads + k];
        Quad<TS>::load(ad[u], reinterpret_cast<const TS *>(ap.a_dst[o]) + q * 4);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (j + u >= j1) break;
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] += sv[u] * ad[u][i];
      }
    }
  }
};

template <typename TS, bool WAVE>
__global__ void __launch_bounds__(256) attn_agg_bwd_cols_kernel(LayerDev L, TypeTab tt, RelRows rr, RelsOfType ro, AttnPtrs ap, int H, int heads,
                                                                int lpr_log2, int rpb, const float *__restrict__ dm, const float2 *__restrict__ ead,
                                                                const float *__restrict__ xsum, const float *__restrict__ dsum,
                                                                TS *__restrict__ dz, float *__restrict__ partial) {
  __shared__ int32_t s_off[kMaxR + 1], s_ptr[kColRows + 1], s_first[kColRows + 1];   // s_first: entries of the block before its row i
  __shared__ int32_t s_rho[kColEntries], s_e[kColEntries];
  __shared__ uint8_t s_rel[kColEntries];
  for (int i = threadIdx.x; i <= rr.n; i += 256) s_off[i] = rr.row_off[i];
  const int q = threadIdx.x & ((1 << lpr_log2) - 1);
  ColSum<TS> cs{rr, ro, ap, dm, xsum, dsum, ead, s_off, H, heads, q, (q * 4) / (H / heads)};
  int t = 0;
  const int nb_long = long_blocks(L.n_chunks, WAVE);
  if ((int)blockIdx.x < nb_long) {
    __shared__ LongLds<4> sm;
    const LongSlot<WAVE> slot(L.n_chunks);
    const LongPiece p = long_piece(L, slot.item);
    while (p.c >= tt.row_off[t + 1]) ++t;
    __syncthreads();
    for (int i = slot.first; i < p.n; i += slot.step) {
      const int rho = L.crow[p.beg + i];
      s_rho[slot.lds + i] = rho;
      s_e[slot.lds + i] = L.cperm[p.beg + i];
      s_rel[slot.lds + i] = (uint8_t)find_le(s_off, rr.n, rho);
    }
    __syncthreads();
    if (!slot.on) return;   // whole wavefront
    auto sum = [&](int, int g, int groups, float (&acc)[4]) {
      for (int i = g; i < p.n; i += 4 * groups) {
        int rho[4], e[4], rel[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int at = slot.lds + min(i + u * groups, p.n - 1);
          rho[u] = s_rho[at];
          e[u] = s_e[at];
          rel[u] = s_rel[at];
        }
        cs.add4(rho, e, rel, [&](int u) { return i + u * groups < p.n; });
      }
      cs.flush();
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i] = cs.acc[i];
    };
    auto done = [&](int, float (&acc)[4]) {
#pragma unroll
      for (int i = 0; i < 4; ++i) cs.acc[i] = acc[i];
      const int v = p.c - tt.row_off[t];
      if (v < tt.n_dst[t]) cs.add_destination(t, v);
      Quad<TS>::store(dz + (int64_t)p.c * H + q * 4, cs.acc);
    };
    long_row<WAVE, 4>(p, slot.item, lpr_log2, H / 4, sm, partial, H, L.chunk_count, sum, done);
    return;
  }
  const int c0 = ((int)blockIdx.x - nb_long) * rpb, nr = min(rpb, L.src_rows - c0);
  if (threadIdx.x < kColRows) {   // one wavefront
    const int i = threadIdx.x, p0 = L.cptr[c0 + min(i, nr)], p1 = L.cptr[c0 + min(i + 1, nr)], len = p1 - p0;
    s_ptr[i] = p0;
    if (i == kColRows - 1) s_ptr[kColRows] = p1;
    int n = len > kLongRow ? 0 : len;
    const int own = n;
    for (int o = 1; o < 64; o <<= 1) {
      const int x = __shfl_up(n, o);
      if (i >= o) n += x;
    }
    s_first[i] = n - own;
    if (i == kColRows - 1) s_first[kColRows] = n;
  }
  __syncthreads();
  const int total = s_first[nr];
  for (int i = threadIdx.x; i < total; i += 256) {
    const int row = find_le(s_first, nr, i), j = s_ptr[row] + i - s_first[row];
    s_rho[i] = L.crow[j];
    s_e[i] = L.cperm[j];
    s_rel[i] = (uint8_t)find_le(s_off, rr.n, s_rho[i]);
  }
  __syncthreads();
  const int gpb = 256 >> lpr_log2, rpg = max(1, rpb / gpb);
  int row = (threadIdx.x >> lpr_log2) * rpg;
  const int row_end = min(row + rpg, nr);
  if (row >= row_end) return;
  while (c0 + row >= tt.row_off[t + 1]) ++t;
  auto finish = [&]() {   // row `row` has all its entries
    const int c = c0 + row;
    while (c >= tt.row_off[t + 1]) ++t;
    cs.flush();
    if (s_ptr[row + 1] - s_ptr[row] <= kLongRow) {
      const int v = c - tt.row_off[t];
      if (v < tt.n_dst[t]) cs.add_destination(t, v);
      Quad<TS>::store(dz + (int64_t)c * H + q * 4, cs.acc);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) cs.acc[i] = 0.f;
    ++row;
  };
  const int end = s_first[row_end];
  for (int j = s_first[row]; j < end; j += 4) {
    int rho[4], e[4], rel[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int at = min(j + u, end - 1);
      rho[u] = s_rho[at];
      e[u] = s_e[at];
      rel[u] = s_rel[at];
    }
    cs.add4(rho, e, rel, [&](int u) {
      if (j + u >= end) return false;
      while (j + u >= s_first[row + 1]) finish();
      return true;
    });
  }
  while (row < row_end) finish();
}

// ------------------------------------------------------------------------------------------
// launchers (backward)
hgnn_status launch_attn_zero(hipStream_t s, float *const *ptrs, const int64_t *counts, int n) {
  ZeroList zl;
  std::memset(&zl, 0, sizeof(zl));
  for (int i = 0; i < n; ++i) {
    if (!ptrs[i] || counts[i] <= 0) continue;
    zl.p[zl.count] = ptrs[i];
    zl.n[zl.count] = (int32_t)counts[i];
    ++zl.count;
  }
  if (zl.count == 0) return HGNN_OK;
  HGNN_LAUNCH(attn_zero_kernel, dim3(32, zl.count), dim3(256), 0, s, zl);
  HGNN_HIP(hipGetLastError());
  return HGNN_OK;
}

hgnn_status launch_attn_mask_dbeta(hipStream_t s, int dtype, const TypeTab &tt, const RelRows &rr, const GradPtrTab &gt, int H, int relu,
                                   const void *g, const void *h, void *gp, const float *mbuf, float *dbeta) {
  TypeTiles ty;
  dst_types(tt, ty);
  const int64_t rows = ty.row_off[ty.n];
  if (rows == 0) return HGNN_OK;
  RelsOfType ro;
  rels_of_type(rr, tt.num_types, ro);
  // A block ends with an atomic add to every dbeta and bias element of its type, some 30 ns of the launch, so that large batches take
  // more rows per block: about 1024 of them, and 2048, whose ends are evener, where the aggregates take longer than that to read.  us with
  // some 1300 / 2600: 84k rows, 1 relation of 256 columns, bf16, 57 / 80, 2 58 / 82, 5 121 / 122; 40k, 4 relations, 51 / 76; 84k, 4, fp32,
  // 93 / 94; 150k, 3, fp32, 193 / 186; 169k rows of four types with 561k aggregates, bf16, 163 / 156.
  const int blocks = (int64_t)rr.row_off[rr.n] * H * 4 > (int64_t)400 << 20 ? 2048 : 1024;
  const int l2 = log2_exact(H / 4), gpb = 256 >> l2, trips = rows_per_group(rows, gpb * 4, blocks, 16);
  dim3 grid(tile_types(ty, gpb * 4 * trips));
  if (dtype == HGNN_BF16)
    HGNN_LAUNCH(attn_mask_dbeta_kernel<bf16>, grid, dim3(256), 0, s, rr, ty, ro, gt, H, relu, l2, trips, (const bf16 *)g, (const bf16 *)h,
                (bf16 *)gp, mbuf, dbeta);
  else
    HGNN_LAUNCH(attn_mask_dbeta_kernel<float>, grid, dim3(256), 0, s, rr, ty, ro, gt, H, relu, l2, trips, (const float *)g, (const float *)h,
                (float *)gp, mbuf, dbeta);
  HGNN_HIP(hipGetLastError());
  return HGNN_OK;
}

hgnn_status launch_attn_sem_bwd(hipStream_t s, int dtype, const RelRows &rr, int H, const float *mbuf, const float *tbuf, const void *w_sem,
                                const void *q_sem, const void *gp, const float *beta, const float *dbeta, float *dm, float *dws, float *dq,
                                float *dbs) {
  if (rr.row_off[rr.n] == 0) return HGNN_OK;
  RelRows dwt = rr, dmt = rr;
  const int tiles = (H + 127) / 128, tm = sem_tile_rows(dmt);
  const int n_dm = tile_relations(dmt, tm) * tiles;
  // Rows per block of the dW_s part, in K-steps of 32: a block's chain grows with them, the atomic adds of whole 128x128 tiles
  // fall with them, so that the best number goes with the root of the work, and at least four steps.  Measured (steps: us with 1/1500
  // of them a block, and with this rule): 512: 28, 28; 2.9k: 118, 101; 4.1k: 106, 84; 4.5k: 172, 167; 36k: 592, 591; half as many
  // rows again or more is slower from 2.9k on (105, 88, 173, 606), two steps are below 512 (28 -> 36).
  SemBwd p;
  const int64_t steps = (int64_t)rr.row_off[rr.n] / 32 * tiles;
  p.dw_rows = 32 * std::max(4, (int)std::ceil(std::sqrt((double)steps) / 8));
  p.n_dw = tile_relations(dwt, p.dw_rows) * tiles;
#define HGNN_SEMB(TY, MI_)                                                                                                         \
  HGNN_LAUNCH((attn_sem_bwd_kernel<TY, MI_>), dim3(p.n_dw + n_dm), dim3(kThreads), 0, s, dwt, dmt, p, H, mbuf, tbuf,                 \
              (const TY *)w_sem, (const TY *)q_sem, (const TY *)gp, beta, dbeta, dm, dws, dq, dbs)
  if (dtype == HGNN_BF16) {
    if (tm == 128) HGNN_SEMB(bf16, 2); else HGNN_SEMB(bf16, 1);
  } else {
    if (tm == 128) HGNN_SEMB(float, 2); else HGNN_SEMB(float, 1);
  }
#undef HGNN_SEMB
  HGNN_HIP(hipGetLastError());
  return HGNN_OK;
}

hgnn_status launch_attn_agg_bwd(hipStream_t s, int dtype, const LayerDev &L, const TypeTab &tt, RelRows rr, const AttnPtrs &ap,
                                const AttnPtrs &dap, int H, int heads, const float *z, const float *dm, const float *mx, const float *ls,
                                void *edge_ad, float *xsum, float *dsum, void *dz, float *partial) {
  const int l2 = log2_exact(H / 4), hl = (H / heads) / 4, gpb = 256 >> l2;
  float2 *ead = (float2 *)edge_ad;
  if (L.rows > 0) {
    const int rpg = std::min(kStageRows / gpb, rows_per_group(L.rows, gpb, 1024, 16));
    dim3 grid(tile_relations(rr, gpb * rpg));
    if (dtype == HGNN_BF16)
      HGNN_LAUNCH(attn_agg_bwd_rows_kernel<bf16>, grid, dim3(256), 0, s, L, rr, ap, dap, H, heads, l2, hl, rpg, z, dm, mx, ls, ead, xsum, dsum);
    else
      HGNN_LAUNCH(attn_agg_bwd_rows_kernel<float>, grid, dim3(256), 0, s, L, rr, ap, dap, H, heads, l2, hl, rpg, z, dm, mx, ls, ead, xsum, dsum);
    HGNN_HIP(hipGetLastError());
  }
  if (L.src_rows > 0) {
    RelsOfType ro;
    rels_of_type(rr, tt.num_types, ro);
    const int cpb = std::min(kColRows, gpb * rows_per_group(L.src_rows, gpb, 2048, 8));
    const bool by_wave = long_rows_by_wave(L.n_chunks, l2);
    dim3 grid(long_blocks(L.n_chunks, by_wave) + (L.src_rows + cpb - 1) / cpb);
#define HGNN_COLS(TY, WAVE_)                                                                                                             \
  HGNN_LAUNCH((attn_agg_bwd_cols_kernel<TY, WAVE_>), grid, dim3(256), 0, s, L, tt, rr, ro, ap, H, heads, l2, cpb, dm, ead, xsum, dsum,   \
              (TY *)dz, partial)
    if (dtype == HGNN_BF16) {
      if (by_wave) HGNN_COLS(bf16, true); else HGNN_COLS(bf16, false);
    } else {
      if (by_wave) HGNN_COLS(float, true); else HGNN_COLS(float, false);
    }
#undef HGNN_COLS
    HGNN_HIP(hipGetLastError());
  }
  return HGNN_OK;
}

}  // namespace hgnn
