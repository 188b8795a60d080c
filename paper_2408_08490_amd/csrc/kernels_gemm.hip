// MFMA GEMMs of the layer path (gfx950, wave64):
//   forward : h_d = act( [Z_r1 | Z_r2 | ... | X_d] . [W_r1; W_r2; ...; W_0^d] + b_d )   per destination type d
//             -- projection and semantic fusion in one contraction (the K loop walks the relations that
//             end in d, then the root term), bias and activation in the epilogue;
//   dA      : dZ_s = (G' W_s^T) scaled per row by 1/|N_r(v)|                          per K-segment s
//   dW      : dW_s = A_s^T G'  (reduction over the destination rows, split and added atomically)
// One 256-thread block (2x2 wavefronts) computes a 128x128 tile, every wavefront 64x64 of it as 2x2 MFMA 32x32
// accumulators, or a 64x64 tile, 32x32 each.  The reduction runs as ONE flat sequence of K-steps over all segments of
// the tile, software-pipelined: operands go global -> registers -> LDS, and the global loads of the next
// two K-steps are in flight while the current one is multiplied.  LDS is double-buffered, so that a step costs one
// barrier, but for fp32 operands split into three bf16 planes, which take both stages: two barriers.  An operand is kept
// in LDS the way it lies in memory: "KC" = the reduction index is contiguous (rows = output index), "KS" = the output
// index is contiguous.
// Every kernel exists in a FAST form (all operands 16-byte aligned: per-thread offsets are computed once
// per segment, a K-step is one to four vector loads per operand and lane from wave-uniform bases) and a generic form
// (element-wise, zero-filled loads) for unaligned shapes.
#include "bias_reduce.h"
#include "gemm_core.h"

namespace hgnn {

// What a block has to look up lies in the first argument, prepared by the host, and is read with scalar loads at known places
// (constant memory): a tile's type with one batch of loads, the type's record with a second, a segment's with a third.  Found in the
// general tables, in part with vector loads and through a table in LDS, it was 3 us in front of a tile, and a launch of large tiles
// has two or three of them one after the other per place.  Forward of the headline's first layer (1444 tiles of 128x128) 69.6 -> 62.8 us,
// of the second (384 of 64x64) 27.4 -> 25.4, the backward's launches 65 -> 63 and 39.8 -> 39.3; fp32, 1024 targets: forward 48.5 -> 44.8,
// backward 56.5 -> 49 and 37.7 -> 34 (these also with four small tiles on a compute unit instead of three).
__device__ __forceinline__ int tile_type(const int32_t __attribute__((address_space(4))) *tile_off, int num_types, int tile) {
  int d = 0;   // entries beyond the last type's are INT32_MAX
  for (int t0 = 1; t0 < num_types; t0 += 8) {
#pragma unroll
    for (int i = 0; i < 8; ++i) d += tile >= tile_off[t0 + i] ? 1 : 0;
  }
  return d;
}
static void put_tile_off(int32_t (&off)[kMaxT + 8], const int32_t *from, int num_types) {
  for (int i = 0; i < kMaxT + 8; ++i) off[i] = i < num_types ? from[i] : INT32_MAX;
}

// ------------------------------------------------------------------------------------------
// Forward.  `live` has bit r set when relation r has at least one edge in this layer.
struct FwdType {
  int32_t n_dst, out_row, steps, seg0;   // steps: K-steps over the type's segments, from seg0 on
  const void *bias;
  int64_t xroot;   // scalars of x before the root term's rows
};
struct FwdSeg {
  uint32_t a4, b4;   // scalars/4 before the segment's rows of Z and before its transposed weight
  int32_t F, root;   // K extent (both leading dimensions); whether it is the root term
};
struct FwdArgs {
  int32_t tile_off[kMaxT + 8];   // tiles before type t
  XcdMap xmap;
  int32_t num_types, H, relu;
  FwdType type[kMaxT];
  FwdSeg seg[kMaxSeg + 1];
};
typedef const FwdArgs __attribute__((address_space(4))) *fwd_args_t;

// A destination type's K-segments: the aggregate of every relation ending in it (and, when the layer keeps it, the aggregate's
// low-order remainder against the same weights), then the root term.
template <typename T> struct FwdSegs {
  static constexpr bool kRedo = false;
  static constexpr int kAhead = 2;
  fwd_args_t args;
  const T *x, *z, *zlo, *wtb;
  int64_t xroot;
  int si, n_steps;
  bool low;   // the remainder of the segment handed out last comes next
  __device__ __forceinline__ int steps() const { return n_steps; }
  __device__ __forceinline__ void next(Seg<T> &g) {
    const uint32_t a4 = args->seg[si].a4, b4 = args->seg[si].b4;
    const int F = args->seg[si].F;
    const bool root = args->seg[si].root != 0;
    g.A = root ? x + xroot : (low ? zlo : z) + (int64_t)a4 * 4;
    g.B = wtb + (int64_t)b4 * 4;
    g.lda = g.ldb = g.ke = F;
    g.kb = 0;
    low = zlo && !root && !low;
    if (!low) ++si;
  }
};

// Four of the small tiles are resident on a compute unit (their LDS holds operands with K contiguous only): the 950 tiles of 12000
// rows and 264 columns in bf16 are one round then and not two, 28.2 -> 20.7 us.
template <typename T, bool FAST, int MI>
__global__ void __launch_bounds__(kThreads, MI == 1 ? 4 : 2) gemm_fwd_kernel(FwdArgs args_, const T *__restrict__ x, const T *__restrict__ z,
                                                            const T *__restrict__ zlo, const T *__restrict__ wtb,
                                                            T *__restrict__ h, float *__restrict__ acc32) {
  constexpr int BM = 64 * MI, BN = 64 * MI;
  __shared__ GemmLds<T, MI, MI, true> sm;
  const fwd_args_t args = (fwd_args_t)__builtin_amdgcn_kernarg_segment_ptr();
  (void)args_;
  const int xcd = blockIdx.x & 7, tile = args->xmap.first[xcd] + (int)(blockIdx.x >> 3);
  if (tile >= args->xmap.first[xcd + 1]) return;
  const int d = tile_type(args->tile_off, args->num_types, tile), H = args->H, relu = args->relu;
  const int tiles_n = (H + BN - 1) / BN;
  const int local = tile - args->tile_off[d];
  const int m0 = (local / tiles_n) * BM, n0 = (local % tiles_n) * BN;
  const int M = args->type[d].n_dst;
  const T *bias = reinterpret_cast<const T *>(args->type[d].bias);
  float bv[MI];
  const int wn0 = ((threadIdx.x >> 6) & 1) * 32 * MI;
#pragma unroll
  for (int j = 0; j < MI; ++j) {
    const int c = n0 + wn0 + j * 32 + (threadIdx.x & 31);
    bv[j] = (bias && c < H) ? to_float(bias[c]) : 0.f;
  }
  f32x16 acc[MI][MI];
  const FwdSegs<T> segs{args, x, z, zlo, wtb, args->type[d].xroot, args->type[d].seg0, args->type[d].steps, false};
  // fp32 with a ReLU: a unit within a rounding of zero takes the other decision when its sum is formed another way, and moves
  // a whole term of the gradients; three of ten million units do (1024 targets, 256 wide: gradients 2e-3 apart).  Neither
  // decision is the wrong one -- the planes' sums are the nearer ones to 64 bits -- but these sums stay on the fp32 MFMA, so
  // that every form of the layer decides alike: 39 -> 50 us there, of a step of 310.
  gemm_finite<T, FAST>(acc, [&](auto split) { gemm_run<T, FAST, true, true, split.value>(acc, sm, segs, M, m0, H, n0); }, relu != 0);
  const int64_t orow = args->type[d].out_row;
  if (acc32) {
    HGNN_FOR_EACH_ACC({
      if (m0 + row < M && n0 + col < H) acc32[(orow + m0 + row) * H + n0 + col] += val;
    })
    return;
  }
  write_tile(acc, sm, h + (orow + m0) * H + n0, H, M - m0, H - n0, [&](float v, int, int col) {
    const float o = v + bv[(col - wn0) >> 5];
    return relu ? fmaxf(o, 0.f) : o;
  });
}

hgnn_status launch_gemm_fwd(hipStream_t s, int dtype, const LayerDev &L, const TypeTab &tt, const RelTab &rt,
                            const PtrTab &pt, const WtTab &wt, const SegTab &tiles, const uint32_t *live_mask, int H,
                            int relu, const void *x, const void *z, const void *zlo, const void *wt_buf, void *h,
                            int only_seg, float *acc32, int tile_mn) {
  const int n = tiles.tile_off[tt.num_types];
  if (n == 0) return HGNN_OK;
  (void)L;
  const int T = tt.num_types, R = rt.num_rels, bk = dtype == HGNN_BF16 ? Mma<bf16>::BK : Mma<float>::BK;
  FwdArgs args;
  put_tile_off(args.tile_off, tiles.tile_off, T);
  args.num_types = T;
  args.H = H;
  args.relu = relu;
  // A tile's cost: its K-steps (destination types differ in the number of relations that end in them) plus
  // the fixed part (pipeline fill, epilogue), which is worth about four K-steps.
  int64_t cost[kMaxT];
  int ns = 0;
  for (int d = 0; d < T; ++d) {
    FwdType &ty = args.type[d];
    ty = FwdType{tt.n_dst[d], tt.out_row_off[d], 0, ns, pt.bias[d], tt.xroot_off[d]};
    for (int r = 0; r < R; ++r)
      if (rt.dst[r] == d && (only_seg < 0 || only_seg == r) && ((live_mask[r >> 5] >> (r & 31)) & 1u)) {   // no edge: all zero
        const int F = tt.in_dim[rt.src[r]];
        args.seg[ns++] = FwdSeg{rt.z_off4[r], wt.rel4[r], F, 0};
        ty.steps += (zlo ? 2 : 1) * ((F + bk - 1) / bk);
      }
    if (pt.w_root[d] && (only_seg < 0 || only_seg == R + d)) {
      args.seg[ns++] = FwdSeg{0, wt.root4[d], tt.in_dim[d], 1};
      ty.steps += (tt.in_dim[d] + bk - 1) / bk;
    }
    cost[d] = ty.steps + 4;
  }
  dim3 grid(balance_xcd(tiles.tile_off, cost, T, args.xmap));
  // operands of the forward are the library's own aligned buffers (aggregates, transposed weights) and
  // x_merged, whose row widths are multiples of 16 bytes: always the FAST form
#define HGNN_FWD(TY, MI_)                                                                                                        \
  HGNN_LAUNCH((gemm_fwd_kernel<TY, true, MI_>), grid, dim3(kThreads), 0, s, args, (const TY *)x, (const TY *)z, (const TY *)zlo, \
              (const TY *)wt_buf, (TY *)h, acc32)
  if (dtype == HGNN_BF16) {
    if (tile_mn == 64) HGNN_FWD(bf16, 1); else HGNN_FWD(bf16, 2);
  } else {
    if (tile_mn == 64) HGNN_FWD(float, 1); else HGNN_FWD(float, 2);
  }
#undef HGNN_FWD
  HGNN_HIP(hipGetLastError());
  return HGNN_OK;
}

// ------------------------------------------------------------------------------------------
// Backward.  One K-segment (relation r -> segment r, root of type t -> segment R + t):
struct BwdSeg {
  uint32_t z4, dz4;   // scalars/4 before its rows of Z and of dZ
  int32_t F, row0;    // input width; first merged row, -1 for a root term
  const void *W;
  float *dW;
};
struct BwdType {
  int32_t n_dst, g0;   // destination rows, and the first one's row of G'
  int64_t xroot;       // scalars of x before the root term's rows
};
struct BwdTiles {   // a DwTab
  int32_t tile_off[kMaxT + 8], first[kMaxT], entries[kMaxT], u_total[kMaxT];
  uint32_t ent[kMaxSeg + 8];   // u_off, and the segment << 16
};
struct BwdArgs {
  BwdTiles dw, da;
  XcdMap xmap;   // of the dW tiles
  int32_t num_types, n_dw, split_rows, H, ldg, rpb, n_bias;
  BwdType type[kMaxT];
  float *dbias[kMaxT];
  BwdSeg seg[kMaxSeg];
};
typedef const BwdArgs __attribute__((address_space(4))) *bwd_args_t;
typedef const BwdTiles __attribute__((address_space(4))) *bwd_tiles_t;
typedef const BwdSeg __attribute__((address_space(4))) *bwd_seg_t;

// The entry of type d that holds block u of its columns.
__device__ __forceinline__ uint32_t bwd_entry(bwd_tiles_t tiles, int d, int u) {
  const int e0 = tiles->first[d], n = tiles->entries[d];
  int c = 0;
  if (n <= 24) {
    for (int b = 0; b < n; b += 8) {   // the eight places behind the last entry exist
#pragma unroll
      for (int i = 0; i < 8; ++i) c += b + i < n && (int)(tiles->ent[e0 + b + i] & 0xffffu) <= u ? 1 : 0;
    }
  } else {
    const int lane = threadIdx.x & 63;
    for (int b = 0; b < n; b += 64) c += __popcll(__ballot(b + lane < n && (int)(tiles->ent[e0 + min(b + lane, n - 1)] & 0xffffu) <= u));
  }
  return tiles->ent[e0 + c - 1];
}

// dZ_s = (G' W_s^T) / deg.  G' has leading dimension ldg (>= H; the columns H..ldg-1 are zero), and so have
// the weights (the caller's own when H is a multiple of 16 bytes, zero-padded copies
// otherwise), so that the reduction simply runs over ldg.
// One tile of dZ_seg: destination rows m0.., columns n0.. of the segment's input width.
template <typename T, bool FAST, int MI>
__device__ __forceinline__ void da_tile_at(GemmLds<T, MI, MI> &sm, bwd_args_t args, bwd_seg_t seg, int d, int m0, int n0,
                                           const int32_t *__restrict__ rowptr, const T *__restrict__ gp, T *__restrict__ dz) {
  constexpr int BM = 64 * MI;
  const int F = seg->F, row0 = seg->row0, M = args->type[d].n_dst, ldg = args->ldg;
  int beg = 0, end = 1;   // 1/|N_r(v)| of the tile's rows (1 for the root term): the loads are under way while the tile is multiplied
  if (row0 >= 0 && (int)threadIdx.x < BM && m0 + (int)threadIdx.x < M) {
    const int32_t *rp = rowptr + row0 + m0 + threadIdx.x;
    beg = rp[0];
    end = rp[1];
  }
  const OneSeg<T> one{Seg<T>{gp + (int64_t)args->type[d].g0 * ldg, reinterpret_cast<const T *>(seg->W), ldg, ldg, 0, ldg}};
  f32x16 acc[MI][MI];
  gemm_finite<T, FAST>(acc, [&](auto split) { gemm_run<T, FAST, true, true, split.value>(acc, sm, one, M, m0, F, n0); });
  float *rowscale = sm.rowscale();
  if (threadIdx.x < BM) rowscale[threadIdx.x] = end > beg ? 1.f / (float)(end - beg) : 0.f;
  __syncthreads();
  write_tile(acc, sm, dz + (int64_t)seg->dz4 * 4 + (int64_t)m0 * F + n0, F, M - m0, F - n0,
             [&](float v, int row, int) { return v * rowscale[row]; });
}

// Tiles grouped by destination type and row block (the DwTab's `u` then runs over the column blocks of all the
// type's segments): the tiles that read the same 128 rows of G' are neighbours, in one XCD, and fetch them once.
template <typename T, bool FAST, int MI>
__device__ __forceinline__ void da_tile_grouped(GemmLds<T, MI, MI> &sm, bwd_args_t args, int bid, int nblocks,
                                                const int32_t *__restrict__ rowptr, const T *__restrict__ gp, T *__restrict__ dz) {
  constexpr int BM = 64 * MI, BN = 64 * MI;
  const bwd_tiles_t tiles = &args->da;
  const int tile = xcd_tile(bid, nblocks);
  const int d = tile_type(tiles->tile_off, args->num_types, tile);
  const int local = tile - tiles->tile_off[d], total = tiles->u_total[d];
  if (total == 0) return;
  const int u = local % total, mt = local / total;
  if (mt * BM >= args->type[d].n_dst) return;   // behind the last tile
  const uint32_t e = bwd_entry(tiles, d, u);
  da_tile_at<T, FAST, MI>(sm, args, &args->seg[e >> 16], d, mt * BM, (u - (int)(e & 0xffffu)) * BN, rowptr, gp, dz);
}

// One segment's tiles after the other's: `tile_off` has the tiles before each.
template <typename T, bool FAST>
__global__ void __launch_bounds__(kThreads, 2) gemm_da_kernel(BwdArgs args_, RelTab rt, SegTab tiles, const int32_t *__restrict__ rowptr,
                                                           const T *__restrict__ gp, T *__restrict__ dz) {
  __shared__ GemmLds<T, 2, 2> sm;
  const bwd_args_t args = (bwd_args_t)__builtin_amdgcn_kernarg_segment_ptr();
  (void)args_;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  if (tile >= tiles.tile_off[tiles.num_segs]) return;
  const int s = wave_find(tiles.tile_off, tiles.num_segs, tile), R = rt.num_rels;
  const int F = args->seg[s].F, tiles_n = (F + BN - 1) / BN, local = tile - tiles.tile_off[s];
  da_tile_at<T, FAST, 2>(sm, args, &args->seg[s], s < R ? rt.dst[s] : s - R, (local / tiles_n) * BM, (local % tiles_n) * BN, rowptr, gp, dz);
}

static void put_bwd_tiles(BwdTiles &to, const DwTab &tl, int num_types) {
  put_tile_off(to.tile_off, tl.tile_off, num_types);
  for (int d = 0; d < num_types; ++d) {
    to.first[d] = tl.first[d];
    to.entries[d] = tl.first[d + 1] - tl.first[d];
    to.u_total[d] = tl.u_total[d];
  }
  for (int i = 0; i < tl.first[num_types]; ++i) to.ent[i] = (uint32_t)tl.u_off[i] | (uint32_t)tl.seg[i] << 16;
}

// The parts of the argument that do not depend on the tiles.
static void put_bwd_args(BwdArgs &a, const TypeTab &tt, const RelTab &rt, const PtrTab *pt, const GradPtrTab *gt, int H, int ldg) {
  const int T = tt.num_types, R = rt.num_rels;
  a.num_types = T;
  a.n_dw = a.split_rows = a.rpb = a.n_bias = 0;
  a.H = H;
  a.ldg = ldg;
  for (int d = 0; d < T; ++d) {
    a.type[d] = BwdType{tt.n_dst[d], tt.out_row_off[d], tt.xroot_off[d]};
    a.dbias[d] = gt ? gt->dbias[d] : nullptr;
    a.seg[R + d] = BwdSeg{0, rt.zroot_off4[d], tt.in_dim[d], -1, pt ? pt->w_root[d] : nullptr, gt ? gt->dw_root[d] : nullptr};
  }
  int row0 = 0;
  for (int r = 0; r < R; ++r) {
    a.seg[r] = BwdSeg{rt.z_off4[r], rt.z_off4[r], tt.in_dim[rt.src[r]], row0, pt ? pt->w_rel[r] : nullptr, gt ? gt->dw_rel[r] : nullptr};
    row0 += tt.n_dst[rt.dst[r]];
  }
}

hgnn_status launch_gemm_da(hipStream_t s, int dtype, const LayerDev &L, const TypeTab &tt, const RelTab &rt,
                           const PtrTab &pt, const SegTab &tiles, int ldg, bool fast, const void *gp, void *dz) {
  const int n = tiles.tile_off[tiles.num_segs];
  if (n == 0) return HGNN_OK;
  dim3 grid(round_up8(n)), blk(kThreads);
  BwdArgs args;
  put_bwd_args(args, tt, rt, &pt, nullptr, 0, ldg);
#define HGNN_DA(TY, FA) \
  HGNN_LAUNCH((gemm_da_kernel<TY, FA>), grid, blk, 0, s, args, rt, tiles, L.rowptr, (const TY *)gp, (TY *)dz)
  if (dtype == HGNN_BF16) {
    if (fast) HGNN_DA(bf16, true); else HGNN_DA(bf16, false);
  } else {
    if (fast) HGNN_DA(float, true); else HGNN_DA(float, false);
  }
#undef HGNN_DA
  HGNN_HIP(hipGetLastError());
  return HGNN_OK;
}

// ------------------------------------------------------------------------------------------
// dW_s += A_s^T G' over the destination-row slice [k_begin, k_end) of this block.
template <typename T, bool FAST, int MI>
__device__ __forceinline__ void dw_tile(GemmLds<T, MI, MI> &sm, bwd_args_t args, int bid, const T *__restrict__ x, const T *__restrict__ z,
                                        const T *__restrict__ gp) {
  constexpr int BM = 64 * MI, BN = 64 * MI;
  const int xcd = bid & 7, tile = args->xmap.first[xcd] + (bid >> 3);
  if (tile >= args->xmap.first[xcd + 1]) return;
  const bwd_tiles_t tiles = &args->dw;
  const int d = tile_type(tiles->tile_off, args->num_types, tile), H = args->H, ldg = args->ldg, split_rows = args->split_rows;
  // inside the type: row slice, then block of dW rows over the type's segments, then column block
  const int tiles_h = (H + BN - 1) / BN, total = tiles->u_total[d];
  int local = tile - tiles->tile_off[d];
  const int th = local % tiles_h;
  local /= tiles_h;
  const int u = local % total, sp = local / total;
  const uint32_t e = bwd_entry(tiles, d, u);
  const bwd_seg_t seg = &args->seg[e >> 16];
  const int F = seg->F, M = args->type[d].n_dst;
  const T *A = seg->row0 >= 0 ? z + (int64_t)seg->z4 * 4 : x + args->type[d].xroot;
  const int f0 = (u - (int)(e & 0xffffu)) * BM, h0 = th * BN;
  const int k_begin = sp * split_rows, k_end = min(M, k_begin + split_rows);
  f32x16 acc[MI][MI];
  const OneSeg<T> one{Seg<T>{A, gp + (int64_t)args->type[d].g0 * ldg, F, ldg, k_begin, k_end}};
  gemm_finite<T, FAST>(acc, [&](auto split) { gemm_run<T, FAST, false, false, split.value>(acc, sm, one, F, f0, ldg, h0); },
                       k_end - k_begin <= kFewTerms);
  float *dW = seg->dW;
  HGNN_FOR_EACH_ACC({
    if (f0 + row < F && h0 + col < H) atomicAdd(dW + (int64_t)(f0 + row) * H + h0 + col, val);
  })
}

template <typename T, bool FAST, int MI>
__global__ void __launch_bounds__(kThreads, MI == 1 ? 4 : 2) gemm_dw_kernel(BwdArgs args_, const T *__restrict__ x, const T *__restrict__ z,
                                                           const T *__restrict__ gp) {
  __shared__ GemmLds<T, MI, MI> sm;
  const bwd_args_t args = (bwd_args_t)__builtin_amdgcn_kernarg_segment_ptr();
  (void)args_;
  dw_tile<T, FAST, MI>(sm, args, blockIdx.x, x, z, gp);
}

// Both backward GEMMs of a layer in ONE launch: the first n_dw blocks compute weight-gradient tiles (long
// reductions), the others input-gradient tiles (short ones).  Each kernel alone leaves compute units idle at its
// end -- the weight gradient has fewer tiles than the chip has block slots -- and the other one's tiles fill them.
// The last n_bias blocks (when bpart is given) add up the partial bias-gradient sums that the row pass over G'
// left: a few microseconds of work that would otherwise be a launch of its own.
template <typename T, bool FAST, int MI>
__global__ void __launch_bounds__(kThreads, MI == 1 ? 4 : 2) gemm_bwd_kernel(BwdArgs args_, const int32_t *__restrict__ rowptr,
                                                            const T *__restrict__ x, const T *__restrict__ z, const T *__restrict__ gp,
                                                            T *__restrict__ dz, const float *__restrict__ bpart) {
  __shared__ GemmLds<T, MI, MI> sm;
  const bwd_args_t args = (bwd_args_t)__builtin_amdgcn_kernarg_segment_ptr();
  (void)args_;
  const int n_gemm = (int)gridDim.x - args->n_bias, n_dw = args->n_dw;
  if ((int)blockIdx.x >= n_gemm) {
    struct TypeRows {   // destination rows per type
      bwd_args_t args;
      __device__ __forceinline__ int operator[](int t) const { return args->type[t].n_dst; }
    };
    bias_reduce_part(TypeRows{args}, args->dbias, args->H, args->rpb, bpart, (int)blockIdx.x - n_gemm, reinterpret_cast<float *>(&sm));
    return;
  }
  if ((int)blockIdx.x < n_dw) dw_tile<T, FAST, MI>(sm, args, blockIdx.x, x, z, gp);
  else da_tile_grouped<T, FAST, MI>(sm, args, blockIdx.x - n_dw, n_gemm - n_dw, rowptr, gp, dz);
}

static int dw_blocks(int dtype, const TypeTab &tt, const DwTab &tiles, int split_rows, XcdMap &xmap) {
  // a tile's cost: the K-steps of its row slice (the average over the type's slices) plus the fixed part
  int64_t cost[kMaxT];
  const int bk = dtype == HGNN_BF16 ? Mma<bf16>::BK : Mma<float>::BK;
  for (int d = 0; d < tt.num_types; ++d) {
    const int64_t slices = (tt.n_dst[d] + split_rows - 1) / split_rows;
    cost[d] = 4 + (slices > 0 ? (tt.n_dst[d] / slices + bk - 1) / bk : 0);
  }
  return balance_xcd(tiles.tile_off, cost, tt.num_types, xmap);
}

hgnn_status launch_gemm_bwd(hipStream_t s, int dtype, const LayerDev &L, const TypeTab &tt, const RelTab &rt,
                            const PtrTab &pt, const DwTab &da_tiles, const GradPtrTab &gt, const DwTab &dw_tiles,
                            int split_rows, int H, int ldg, bool fast, const void *x, const void *z, const void *gp, void *dz,
                            const float *bpart, int rpb) {
  BwdArgs args;
  put_bwd_args(args, tt, rt, &pt, &gt, H, ldg);
  put_bwd_tiles(args.dw, dw_tiles, tt.num_types);
  put_bwd_tiles(args.da, da_tiles, tt.num_types);
  const int n_dw = dw_blocks(dtype, tt, dw_tiles, split_rows, args.xmap);
  const int n_da = round_up8(da_tiles.tile_off[tt.num_types]);
  const int n_bias = bpart ? bias_reduce_blocks(tt.num_types, H) : 0;
  args.n_dw = n_dw;
  args.split_rows = split_rows;
  args.rpb = rpb;
  args.n_bias = n_bias;
  dim3 grid(n_dw + n_da + n_bias), blk(kThreads);
#define HGNN_BWD2(TY, FA, MI_)                                                                                       \
  HGNN_LAUNCH((gemm_bwd_kernel<TY, FA, MI_>), grid, blk, 0, s, args, L.rowptr, (const TY *)x, (const TY *)z, (const TY *)gp, (TY *)dz, bpart)
#define HGNN_BWD(TY, FA) { if (dw_tiles.edge == 64) HGNN_BWD2(TY, FA, 1); else HGNN_BWD2(TY, FA, 2); }
  if (dtype == HGNN_BF16) {
    if (fast) HGNN_BWD(bf16, true) else HGNN_BWD(bf16, false)
  } else {
    if (fast) HGNN_BWD(float, true) else HGNN_BWD(float, false)
  }
#undef HGNN_BWD
#undef HGNN_BWD2
  HGNN_HIP(hipGetLastError());
  return HGNN_OK;
}

hgnn_status launch_gemm_dw(hipStream_t s, int dtype, const LayerDev &L, const TypeTab &tt, const RelTab &rt,
                           const GradPtrTab &gt, const DwTab &tiles, int split_rows, int H, int ldg, bool fast,
                           const void *x, const void *z, const void *gp) {
  const int n = tiles.tile_off[tt.num_types];
  if (n == 0) return HGNN_OK;
  (void)L;
  BwdArgs args;
  put_bwd_args(args, tt, rt, nullptr, &gt, H, ldg);
  put_bwd_tiles(args.dw, tiles, tt.num_types);
  args.split_rows = split_rows;
  dim3 grid(dw_blocks(dtype, tt, tiles, split_rows, args.xmap)), blk(kThreads);
#define HGNN_DW(TY, FA, MI_) \
  HGNN_LAUNCH((gemm_dw_kernel<TY, FA, MI_>), grid, blk, 0, s, args, (const TY *)x, (const TY *)z, (const TY *)gp)
#define HGNN_DW2(TY, FA) { if (tiles.edge == 64) HGNN_DW(TY, FA, 1); else HGNN_DW(TY, FA, 2); }
  if (dtype == HGNN_BF16) {
    if (fast) HGNN_DW2(bf16, true) else HGNN_DW2(bf16, false)
  } else {
    if (fast) HGNN_DW2(float, true) else HGNN_DW2(float, false)
  }
#undef HGNN_DW2
#undef HGNN_DW
  HGNN_HIP(hipGetLastError());
  return HGNN_OK;
}

}  // namespace hgnn
