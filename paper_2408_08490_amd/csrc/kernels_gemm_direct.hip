// Forward GEMM of the layer for launches that a 64x64 tile per compute unit does not fill (small batches, last layers, many
// relations): h_d = act( [Z_r1 | Z_r2 | ... | X_d] . [W_r1; W_r2; ...; W_0^d] + b_d ), the contraction of
// gemm_fwd_kernel (kernels_gemm.hip), with the reduction split twice: over blocks and over the wavefronts of a block.
//
// What bounds those launches is a tile's own chain on a chip that is mostly idle: a compute unit takes in some 50 bytes
// per clock, and a destination type with thirty relations has megabytes of operands behind every tile; the LDS-staged
// kernel adds 0.5 us of load -> LDS -> barrier -> MFMA latency per K-step.  So a tile's K-steps are dealt to as many blocks
// as make about two for every compute unit, and inside a block every wavefront owns the whole tile for every fourth K-step
// and reads its MFMA fragments straight from global memory (both operands have K contiguous: a fragment is one 16-byte
// load per lane), so that there is no barrier before the end.  A K-step is 128 bytes of every row, a whole cache line,
// and a wavefront keeps the next one's loads in flight behind the one it multiplies.  16x16 MFMA tiles: four lanes read
// 64 contiguous bytes of a row (32x32 tiles read 32), the same MFMA rate.  The wavefronts' partial tiles meet in LDS; where
// a tile has several blocks each stores its partial tile, and a second kernel adds them up in a fixed order (the forward
// stays bit-identical from run to run, which atomic adds would not).
//
// fp32: the MFMA takes one K per lane; a lane's 16 bytes are four consecutive K, so K is handed out in another order than
// it lies in memory (the same one for both operands).
#include <algorithm>

#include "gemm_core.h"

namespace hgnn {

template <typename T> struct Direct;
template <> struct Direct<bf16> { static constexpr int KG = 32; };   // K of one group of fragments (16 bytes per lane)
template <> struct Direct<float> { static constexpr int KG = 16; };

// Everything a block has to look up, prepared by the host so that it is read with scalar loads at known places: building
// the list of K-segments in LDS from the general tables took several dependent round trips in front of the first load.
struct DirectSeg {
  uint32_t a4, b4;   // scalars/4 before the segment's rows of Z (of X for the root term) and its transposed weight
  int32_t F;         // K extent (both leading dimensions), negative for the root term
  int32_t first;     // K-steps of the type before the segment
};
struct DirectArgs {
  int32_t unit_off[kMaxT + 8];   // (tile, split) pairs before type t; INT_MAX beyond the last
  int32_t tile_off[kMaxT + 1];   // tiles before type t
  int32_t n_dst[kMaxT], out_row[kMaxT], steps[kMaxT];
  uint16_t seg0[kMaxT + 1], splits[kMaxT];
  const void *bias[kMaxT];
  DirectSeg seg[kMaxSeg + 1];
  int32_t num_types, H, relu;
};
typedef const DirectArgs __attribute__((address_space(4))) *direct_args_t;

// One K-step's fragments (two groups) in a wavefront's registers.
template <typename T, int MT, int NT> struct Stage {
  static constexpr int KG = Direct<T>::KG;
  u32x4 a[2][MT], b[2][NT];
  int kleft;   // K values of the segment from this step on

  // pieces beyond the segment's end read the row's start; multiply() counts them as zero
  __device__ __forceinline__ void load(const T *A, const T *B, int F, int k0, int fk, const int (&arow)[MT], const int (&brow)[NT]) {
    typedef const u32x4 __attribute__((address_space(1))) *gvec_t;
    typedef const char __attribute__((address_space(1))) *gbyte_t;
    kleft = F - k0;
    const gbyte_t pa = (gbyte_t)A, pb = (gbyte_t)B;
    const int kk0 = k0 + fk < F ? k0 + fk : 0, kk1 = k0 + KG + fk < F ? k0 + KG + fk : 0;
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      a[0][i] = *(gvec_t)(pa + (unsigned)(arow[i] * F + kk0) * (unsigned)sizeof(T));
      a[1][i] = *(gvec_t)(pa + (unsigned)(arow[i] * F + kk1) * (unsigned)sizeof(T));
    }
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      b[0][j] = *(gvec_t)(pb + (unsigned)(brow[j] * F + kk0) * (unsigned)sizeof(T));
      b[1][j] = *(gvec_t)(pb + (unsigned)(brow[j] * F + kk1) * (unsigned)sizeof(T));
    }
  }
  template <int C> __device__ __forceinline__ void multiply_group(f32x4 (&acc)[MT][NT], int fk) {
    if (kleft < (C + 1) * KG && C * KG + fk >= kleft) {
#pragma unroll
      for (int i = 0; i < MT; ++i) a[C][i] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
      for (int j = 0; j < NT; ++j) b[C][j] = u32x4{0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        if constexpr (sizeof(T) == 2) {
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a[C][i]), __builtin_bit_cast(bf16x8_t, b[C][j]), acc[i][j], 0, 0, 0);
        } else {
#pragma unroll
          for (int k = 0; k < 4; ++k)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[C][i][k]), __uint_as_float(b[C][j][k]), acc[i][j], 0, 0, 0);
        }
      }
  }
  __device__ __forceinline__ void multiply(f32x4 (&acc)[MT][NT], int fk) {
    multiply_group<0>(acc, fk);
    multiply_group<1>(acc, fk);
  }
};

// Writes four columns of a finished row.
template <typename T>
__device__ __forceinline__ void put_quad(T *q, int H, int ncols, f32x4 s, const float (&bv)[4], int relu) {
  float o[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    o[k] = s[k] + bv[k];
    if (relu) o[k] = fmaxf(o[k], 0.f);
  }
  if (ncols >= 4 && H % 4 == 0) {   // rows of a multiple of four scalars keep every piece aligned
    if constexpr (sizeof(T) == 2) *reinterpret_cast<u32x2 *>(q) = u32x2{pack2(o[0], o[1]), pack2(o[2], o[3])};
    else *reinterpret_cast<f32x4 *>(q) = f32x4{o[0], o[1], o[2], o[3]};
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (k < ncols) q[k] = from_float<T>(o[k]);
  }
}

// Wavefronts; 16x16 tiles per wavefront: 64 rows, and 64 columns where there are more than 32 (NT = 4).  A tile of 16 or 32
// columns is a quarter or half of the MFMAs, 1.7 us of a K-step of 64 columns in fp32 (one tile of 16 columns 8.5 -> 6.7 us; eight of
// 32, in pieces, with their sum 13.2 -> 10.8 in fp32).
constexpr int kDirW = 4, kDirMT = 4;

__device__ __forceinline__ int unit_type(direct_args_t pa, int unit) {
  int d = 0;
  for (int t0 = 1; t0 < pa->num_types; t0 += 8) {
#pragma unroll
    for (int i = 0; i < 8; ++i) d += unit >= pa->unit_off[t0 + i] ? 1 : 0;
  }
  return d;
}

template <typename T, int NT>
__global__ void __launch_bounds__(64 * kDirW, 2) gemm_fwd_direct_kernel(DirectArgs args, const T *__restrict__ x, const T *__restrict__ z,
                                                                        const T *__restrict__ zlo, const T *__restrict__ wtb, T *__restrict__ h,
                                                                        float *__restrict__ part) {
  constexpr int MT = kDirMT, W = kDirW, BM = 16 * MT, BN = 16 * NT, KS = 2 * Direct<T>::KG, VEC = 16 / sizeof(T), P = BN + 4;
  __shared__ __attribute__((aligned(16))) float red[W][BM * P];
  // The first argument, read where it lies (constant memory, scalar loads): indexed as an ordinary object it can end up
  // copied to every lane's scratch memory first.
  const direct_args_t pa = (direct_args_t)__builtin_amdgcn_kernarg_segment_ptr();
  (void)args;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int d = unit_type(pa, blockIdx.x);
  const int H = pa->H, M = pa->n_dst[d], splits = pa->splits[d], steps = pa->steps[d];
  const int tiles_d = pa->tile_off[d + 1] - pa->tile_off[d], tiles_n = (H + BN - 1) / BN;
  const int unit = (int)blockIdx.x - pa->unit_off[d], split = unit / tiles_d, tile = unit % tiles_d;
  const int m0 = (tile / tiles_n) * BM, n0 = (tile % tiles_n) * BN;
  const int begin = (int)((int64_t)steps * split / splits), end = (int)((int64_t)steps * (split + 1) / splits);
  constexpr int PPR = BN / 4;
  const int rows = min(BM, M - m0), cols = H - n0, c = (threadIdx.x % PPR) * 4;
  float bv[4];
  const T *bias = reinterpret_cast<const T *>(pa->bias[d]);
#pragma unroll
  for (int k = 0; k < 4; ++k) bv[k] = splits == 1 && bias && c + k < cols ? to_float(bias[n0 + c + k]) : 0.f;
  f32x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int fr = lane & 15, fk = (lane >> 4) * VEC;   // row of a fragment, first K of the lane's piece
  int arow[MT], brow[NT];
#pragma unroll
  for (int i = 0; i < MT; ++i) arow[i] = min(m0 + 16 * i + fr, M - 1);
#pragma unroll
  for (int j = 0; j < NT; ++j) brow[j] = min(n0 + 16 * j + fr, H - 1);
  const int si_last = pa->seg0[d + 1] - 1;
  int si = pa->seg0[d];
  {   // the segment of the wavefront's first K-step (wave_find on the steps in front of each)
    int c = 0;
    for (int b = si; b <= si_last; b += 64) c += __popcll(__ballot(b + lane <= si_last && pa->seg[min(b + lane, si_last)].first <= begin + wave));
    si += max(c - 1, 0);
  }
#define HGNN_LOAD(stage, step_)                                                                      \
  {                                                                                                  \
    const int step = min(step_, end - 1);                                                            \
    while (si < si_last && step >= pa->seg[si + 1].first) ++si;                                      \
    const int sF = pa->seg[si].F, F = sF < 0 ? -sF : sF, nk = (F + KS - 1) / KS;                     \
    const int ks = step - pa->seg[si].first;                                                         \
    const T *A = sF < 0 ? x : ks >= nk ? zlo : z; /* the low-order plane follows the values */       \
    stage.load(A + (int64_t)pa->seg[si].a4 * 4, wtb + (int64_t)pa->seg[si].b4 * 4, F, (ks >= nk ? ks - nk : ks) * KS, fk, arow, brow); \
  }
  if (begin + wave < end) {
    Stage<T, MT, NT> s0, s1;
    HGNN_LOAD(s0, begin + wave)
    for (int base = begin + wave; base < end; base += 2 * W) {
      HGNN_LOAD(s1, base + W)
      s0.multiply(acc, fk);
      HGNN_LOAD(s0, base + 2 * W)
      if (base + W < end) s1.multiply(acc, fk);
    }
  }
#undef HGNN_LOAD
  // 16x16 output layout: lane % 16 is the column, the four values are rows 4 (lane / 16) + v
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) red[wave][(16 * i + 4 * (lane >> 4) + v) * P + 16 * j + fr] = acc[i][j][v];
  __syncthreads();
  if (c >= cols) return;
  float *pt = part + (int64_t)(pa->unit_off[d] + tile * splits + split) * (64 * 64);
  T *out = h + ((int64_t)pa->out_row[d] + m0) * H + n0 + c;
  for (int r = threadIdx.x / PPR; r < rows; r += 64 * W / PPR) {
    f32x4 s = *reinterpret_cast<const f32x4 *>(&red[0][r * P + c]);
#pragma unroll
    for (int w = 1; w < W; ++w) s += *reinterpret_cast<const f32x4 *>(&red[w][r * P + c]);
    if (splits > 1) *reinterpret_cast<f32x4 *>(pt + r * 64 + c) = s;
    else put_quad(out + (int64_t)r * H, H, cols - c, s, bv, pa->relu);
  }
}

// Adds up the partial tiles of the types that have several: a block takes 16 rows of one tile.
template <typename T>
__global__ void __launch_bounds__(256) gemm_fwd_direct_sum_kernel(DirectArgs args, const float *__restrict__ part, T *__restrict__ h) {
  const direct_args_t pa = (direct_args_t)__builtin_amdgcn_kernarg_segment_ptr();
  (void)args;
  const int tile = blockIdx.x >> 2;
  int d = 0;
  while (tile >= pa->tile_off[d + 1]) ++d;
  const int H = pa->H, splits = pa->splits[d], tiles_n = (H + 63) / 64, local = tile - pa->tile_off[d];
  const int r = (local / tiles_n) * 64 + (blockIdx.x & 3) * 16 + (threadIdx.x >> 4), n0 = (local % tiles_n) * 64, c = (threadIdx.x & 15) * 4;
  if (splits == 1 || r >= pa->n_dst[d] || n0 + c >= H) return;
  const float *p = part + (int64_t)(pa->unit_off[d] + local * splits) * 4096 + (r & 63) * 64 + c;
  const T *bias = reinterpret_cast<const T *>(pa->bias[d]);
  float bv[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) bv[k] = bias && n0 + c + k < H ? to_float(bias[n0 + c + k]) : 0.f;
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
  for (int i = 0; i < splits; i += 4) {
    f32x4 v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = *reinterpret_cast<const f32x4 *>(p + (int64_t)min(i + j, splits - 1) * 4096);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (i + j < splits) s += v[j];
  }
  put_quad(h + ((int64_t)pa->out_row[d] + r) * H + n0 + c, H, H - n0 - c, s, bv, pa->relu);
}

// For launches of fewer than kDirectTiles tiles of 64x64 (a quarter of that in bf16); `part` holds kDirectPartBytes.
// Returns the kernels that it launches (with count_only: that it would launch), 0: not for this launch.  Beyond the line a tile
// per block keeps the compute units busy and the staged kernel, whose four wavefronts share a tile's operands, needs half the
// operand traffic; the fp32 products are 16 times as long, so that the line lies further out.  Both kernels of this file
// together against the staged one, in us (tiles: before -> now):
//   fp32  16: 43 -> 16, 27 -> 16 (104 relations)   96: 41 -> 23   312: 54 -> 48      700: 47 -> 52 (not taken)
//   bf16  72: 43 -> 22 (108 relations)   16: 24 -> 16   24: 15 -> 14   96: 24 -> 21   230: 15 -> 27 (not taken)
// In fp32 with a ReLU the line is at 64 tiles: a sum formed in another order gives units within a rounding of zero the other
// decision (three of ten million), which moves a whole term of the gradients away from what the staged kernel's forms of the
// layer give; up to 64 tiles there is next to never one.  How the K-steps are dealt out (`target` below) is part of that order:
// each number of splits rounds its sums its own way, below the line too.
static int launch_gemm_fwd_direct(hipStream_t s, int dtype, const TypeTab &tt, const RelTab &rt, const PtrTab &pt, const WtTab &wt,
                                   const uint32_t *live_mask, int H, int relu, const void *x, const void *z, const void *zlo,
                                   const void *wt_buf, void *h, float *part, bool count_only) {
  const int T = tt.num_types, R = rt.num_rels, ks = 2 * (dtype == HGNN_BF16 ? Direct<bf16>::KG : Direct<float>::KG);
  const int es = dtype == HGNN_BF16 ? 2 : 4;
  DirectArgs da;
  da.num_types = T;
  da.H = H;
  da.relu = relu;
  da.tile_off[0] = 0;
  for (int d = 0; d < T; ++d) da.tile_off[d + 1] = da.tile_off[d] + ((tt.n_dst[d] + 63) / 64) * ((H + 63) / 64);
  const int tiles = da.tile_off[T];
  if (tiles == 0 || tiles >= (dtype == HGNN_BF16 ? kDirectTiles / 4 : relu ? kDirectReluTiles : kDirectTiles)) return 0;
  int n = 0;
  int64_t work = 0;   // K-steps over all tiles
  for (int d = 0; d < T; ++d) {
    da.seg0[d] = (uint16_t)n;
    int steps = 0;
    auto put = [&](uint32_t a4, uint32_t b4, int F, bool root) {
      if ((int64_t)std::max(tt.n_dst[d], H) * F * es >= (int64_t)1 << 31) return false;   // 32-bit byte offsets inside an operand
      da.seg[n++] = DirectSeg{a4, b4, root ? -F : F, steps};
      steps += (!root && zlo ? 2 : 1) * ((F + ks - 1) / ks);
      return true;
    };
    if (tt.n_dst[d] > 0) {
      for (int r = 0; r < R; ++r)
        if (rt.dst[r] == d && ((live_mask[r >> 5] >> (r & 31)) & 1u) && !put(rt.z_off4[r], wt.rel4[r], tt.in_dim[rt.src[r]], false)) return 0;
      if (pt.w_root[d] && (tt.xroot_off[d] / 4 > UINT32_MAX || !put((uint32_t)(tt.xroot_off[d] / 4), wt.root4[d], tt.in_dim[d], true))) return 0;
    }
    da.n_dst[d] = tt.n_dst[d];
    da.out_row[d] = tt.out_row_off[d];
    da.steps[d] = steps;
    da.bias[d] = pt.bias[d];
    work += (int64_t)steps * (da.tile_off[d + 1] - da.tile_off[d]);
  }
  da.seg0[T] = (uint16_t)n;
  da.seg[n] = DirectSeg{0, 0, 0, INT32_MAX};
  // K-steps per block: those of two blocks per compute unit, but two for every wavefront, which cost about what the block's own
  // start and end do.  In fp32, whose MFMAs take 1.7 us a step, one for every wavefront where the tiles are split in any case
  // into few blocks and few pieces: twice the pieces are written and added up again.  Forward of a layer, us, with two / one: 2
  // splits, 60 blocks 18.6 / 17.4; 3 splits, 90 blocks 18.9 / 18.0, 96 19.5 / 19.3; 5 splits, 95 blocks 20.8 / 20.5, 150 21.6 / 24.1;
  // 4 splits, 240 blocks 23.3 / 29.4; 8 splits, 8 blocks 18.2 / 17.5, 64 19.3 / 20.0; 9 splits, 9 blocks 18.3 / 17.6, 72 20.7 / 21.1.
  // 16 and 18 splits, as many blocks, 19.1 and 19.3 / 19.3 and 19.5: the second kernel's chain.  Where two a wavefront are the
  // whole tile, splitting it would only add that kernel (28 tiles of 8 steps 13.4 / 15.5).
  int64_t most = 0, blocks = 0;
  for (int d = 0; d < T; ++d) {
    const int td = da.tile_off[d + 1] - da.tile_off[d];
    if (td > 0) most = std::max<int64_t>(most, da.steps[d]);
    blocks += (int64_t)td * ((da.steps[d] + 2 * kDirW - 1) / (2 * kDirW));
  }
  const bool single = dtype != HGNN_BF16 && most > 2 * kDirW && most <= 10 * 2 * kDirW && blocks < (most <= 5 * 2 * kDirW ? 112 : 64);
  const int64_t target = std::max<int64_t>(single ? kDirW : 2 * kDirW, (work + 511) / 512);
  int units = 0, max_splits = 1;
  for (int i = 0; i < kMaxT + 8; ++i) da.unit_off[i] = INT32_MAX;
  for (int d = 0; d < T; ++d) {
    const int td = da.tile_off[d + 1] - da.tile_off[d];
    da.splits[d] = (uint16_t)std::max<int64_t>(1, (da.steps[d] + target - 1) / target);
    da.unit_off[d] = units;
    units += td * da.splits[d];
    if (td > 0) max_splits = std::max(max_splits, (int)da.splits[d]);
  }
  da.unit_off[T] = units;
  if (units > kDirectUnits) return 0;
  const int launches = max_splits > 1 ? 2 : 1;
  if (count_only) return launches;
#define HGNN_DIRECT(TY, NT)                                                                                                           \
  HGNN_LAUNCH((gemm_fwd_direct_kernel<TY, NT>), dim3(units), dim3(64 * kDirW), 0, s, da, (const TY *)x, (const TY *)z, (const TY *)zlo, \
              (const TY *)wt_buf, (TY *)h, part)
#define HGNN_DIRECT_N(TY)                                                                                             \
  {                                                                                                                   \
    if (H <= 16) HGNN_DIRECT(TY, 1);                                                                                  \
    else if (H <= 32) HGNN_DIRECT(TY, 2);                                                                             \
    else HGNN_DIRECT(TY, 4);                                                                                          \
    if (launches > 1) HGNN_LAUNCH(gemm_fwd_direct_sum_kernel<TY>, dim3(tiles * 4), dim3(256), 0, s, da, part, (TY *)h); \
  }
  if (dtype == HGNN_BF16) HGNN_DIRECT_N(bf16) else HGNN_DIRECT_N(float)
#undef HGNN_DIRECT_N
#undef HGNN_DIRECT
  return launches;
}

static const bool registered = [] {
  optional_launchers().gemm_fwd_direct = launch_gemm_fwd_direct;
  return true;
}();

}  // namespace hgnn
