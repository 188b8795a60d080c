// Memory-bound kernels of the layer path (gfx950): type-first feature gather, the relation-
// segmented gather-mean over the merged CSR (paper Algorithm 1, evaluated without materialising
// the per-edge feature copies), its transpose for the backward pass, and small element-wise
// helpers.  Every feature row is moved in 16-byte pieces by a power-of-two group of lanes.
#include <cstring>
#include "common.h"
#include "bias_reduce.h"
#include "device_types.h"
#include "long_rows.h"
#include "transpose_jobs.h"

namespace hgnn {

// ------------------------------------------------------------------------------------------
// Stage 0: gather mini-batch rows from the per-type stores into the type-first buffer.
// ------------------------------------------------------------------------------------------
struct MergeTab {
  const void *store[kMaxT];
  const int64_t *ids[kMaxT];
  const int32_t *pos[kMaxT];   // index-first baseline: row of the interleaved buffer that holds row i of type t
  const char *inter;           // mode 2: the interleaved buffer rows are read from
  int64_t elem_off[kMaxT + 1];
  int32_t row_off[kMaxT + 4];
  int32_t dim[kMaxT];
  int32_t num_types;
  int32_t mode;                // 0: stores -> type-first buffer; 1: stores -> interleaved buffer; 2: interleaved -> type-first
};

__global__ void __launch_bounds__(256) merge_kernel(MergeTab mt, char *out, int esize, int lpr_log2) {
  const int lpr = 1 << lpr_log2;
  const int row = blockIdx.x * (256 >> lpr_log2) + (threadIdx.x >> lpr_log2);
  const int lane = threadIdx.x & (lpr - 1);
  if (row >= mt.row_off[mt.num_types]) return;
  int t = 0;   // scalar loads that do not depend on each other; the entries behind the last type's are never reached
  for (int t0 = 1; t0 < mt.num_types; t0 += 4) {
#pragma unroll
    for (int u = 0; u < 4; ++u) t += row >= mt.row_off[t0 + u] && t0 + u < mt.num_types ? 1 : 0;
  }
  const int i = row - mt.row_off[t];
  const int nvec = (mt.dim[t] * esize) >> 4;
  // interleaved position, clamped into the buffer (a caller's bad position cannot leave it)
  const int64_t at = mt.mode ? min(max(mt.pos[t][i], 0), mt.row_off[mt.num_types] - 1) : 0;
  const uint4 *src = mt.mode == 2 ? reinterpret_cast<const uint4 *>(mt.inter) + at * nvec
                                  : reinterpret_cast<const uint4 *>(mt.store[t]) + mt.ids[t][i] * nvec;
  uint4 *dst = mt.mode == 1 ? reinterpret_cast<uint4 *>(out) + at * nvec
                            : reinterpret_cast<uint4 *>(out + mt.elem_off[t] * esize) + (int64_t)i * nvec;
  for (int c = lane; c < nvec; c += 2 * lpr) {  // both loads before the stores
    const int c2 = c + lpr;
    const uint4 a = src[c];
    const uint4 b = c2 < nvec ? src[c2] : a;
    dst[c] = a;
    if (c2 < nvec) dst[c2] = b;
  }
}

hgnn_status launch_merge(hipStream_t s, int dtype, int T, const void *const *store, const int32_t *feat_dim,
                         const int64_t *const *ids, const int64_t *n_rows, const int64_t *elem_off, void *out, int mode,
                         const int32_t *const *pos, const void *interleaved) {
  MergeTab mt;
  std::memset(&mt, 0, sizeof(mt));
  const int es = dtype == HGNN_BF16 ? 2 : 4;
  int maxd = 0;
  mt.row_off[0] = 0;
  mt.mode = mode;
  mt.inter = (const char *)interleaved;
  for (int t = 0; t < T; ++t) {
    mt.store[t] = store ? store[t] : nullptr;
    mt.ids[t] = ids ? ids[t] : nullptr;
    mt.pos[t] = pos ? pos[t] : nullptr;
    mt.elem_off[t] = elem_off[t];
    mt.row_off[t + 1] = mt.row_off[t] + (int32_t)n_rows[t];
    mt.dim[t] = feat_dim[t];
    if (n_rows[t] > 0) maxd = std::max(maxd, feat_dim[t]);
  }
  mt.elem_off[T] = elem_off[T];
  mt.num_types = T;
  const int total = mt.row_off[T];
  if (total == 0) return HGNN_OK;
  // two 16-byte pieces per lane: both loads of a lane are in flight together (a lane per piece left the copy
  // waiting on one load at a time: 50 -> 43 us on the headline's 400k rows of 256 bytes; four per lane gain nothing)
  const int l2 = std::max(0, lanes_log2_for(maxd, es) - 1);
  const int rpb = 256 >> l2;
  HGNN_LAUNCH(merge_kernel, dim3((total + rpb - 1) / rpb), dim3(256), 0, s, mt, (char *)out, es, l2);
  HGNN_HIP(hipGetLastError());
  return HGNN_OK;
}

// ------------------------------------------------------------------------------------------
// Stage 3 for ragged widths: z[rho] = mean over the merged CSR row rho of the source rows of x.  Blocks are cut per
// relation, so that the relation, its source type and the lanes a row needs (16 bytes each) are the same for the whole
// block and live in scalar registers: a row costs the dependent loads row pointer -> index -> features and no search,
// and a narrow type does not leave most lanes of a group sized for the widest one idle.
// (10 types of 32 to 384 floats, 512 targets: 34 -> 21 us.)
// ------------------------------------------------------------------------------------------
struct RelTiles {
  int32_t tile_off[kMaxR + 1];   // blocks before relation r
  int32_t lo[kMaxR], hi[kMaxR];  // its merged rows (those asked for)
};
__host__ __device__ static inline int row_lanes_log2(int nvec) {  // lanes that share a row of nvec 16-byte pieces
  int l = 0;
  while ((1 << l) < nvec && l < 6) ++l;
  return l;
}

template <typename T>
__global__ void __launch_bounds__(256) spmm_fwd_kernel(LayerDev L, TypeTab tt, RelTab rt, RelTiles rtl, const T *__restrict__ x,
                                                        T *__restrict__ z, T *__restrict__ zlo, TransposeJobs tj) {
  using V = Vec16<T>;
  __shared__ T tile[32][33];
  if ((int)blockIdx.x < tj.blocks) {   // in front: see JobSplit
    transpose_jobs_block<T>(tj, blockIdx.x, tj.blocks, tile);
    return;
  }
  const int b = (int)blockIdx.x - tj.blocks;
  const int r = wave_find(rtl.tile_off, rt.num_rels, b);
  const int st = rt.src[r];
  const int F = tt.in_dim[st];
  const int nvec = F / V::N, l2 = row_lanes_log2(nvec), lpr = 1 << l2;
  const int row = rtl.lo[r] + (b - rtl.tile_off[r]) * (256 >> l2) + (threadIdx.x >> l2);
  const int lane = threadIdx.x & (lpr - 1);
  if (row >= rtl.hi[r]) return;
  const uint4 *xb = reinterpret_cast<const uint4 *>(x + tt.elem_off[st]) - (int64_t)tt.row_off[st] * nvec;
  const int64_t zoff = (int64_t)rt.z_off4[r] * 4 + (int64_t)(row - L.rel_row_off[r]) * F;
  uint4 *zr = reinterpret_cast<uint4 *>(z + zoff);
  const int beg = L.rowptr[row], end = L.rowptr[row + 1];
  const float inv = end > beg ? 1.0f / (float)(end - beg) : 0.0f;
  for (int c = lane; c < nvec; c += lpr) {
    float acc[V::N];
#pragma unroll
    for (int i = 0; i < V::N; ++i) acc[i] = 0.f;
    for (int e = beg; e < end; e += 4) {
      uint4 v[4];
      int col[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) col[j] = L.colidx[min(e + j, end - 1)];
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = xb[(int64_t)col[j] * nvec + c];
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (e + j < end) V::add(acc, v[j]);
    }
#pragma unroll
    for (int i = 0; i < V::N; ++i) acc[i] *= inv;
    const uint4 hi = V::pack(acc);
    zr[c] = hi;
    if (zlo) reinterpret_cast<uint4 *>(zlo + zoff)[c] = V::pack_remainder(acc, hi);
  }
}

hgnn_status launch_spmm_fwd(hipStream_t s, int dtype, const LayerDev &L, const TypeTab &tt, const RelTab &rt,
                            int max_dim, const void *x, void *z, void *zlo, int row_begin, int row_end,
                            const TransposeJobs *tj) {
  (void)max_dim;
  if (row_end <= row_begin) return tj ? launch_transpose_jobs(s, dtype, *tj) : HGNN_OK;
  const int es = dtype == HGNN_BF16 ? 2 : 4;
  bool uniform = true;
  for (int t = 0; t < tt.num_types; ++t) uniform &= tt.in_dim[t] == tt.in_dim[0];
  if (uniform && launch_spmm_fwd_uniform(s, dtype, L, tt.in_dim[0], x, z, zlo, row_begin, row_end, nullptr, tj)) {
    HGNN_HIP(hipGetLastError());
    return HGNN_OK;
  }
  TransposeJobs none;
  if (!tj) {
    std::memset(&none, 0, sizeof(none));
    tj = &none;
  }
  RelTiles rtl;
  std::memset(&rtl, 0, sizeof(rtl));
  for (int r = 0, at = 0; r < rt.num_rels; ++r) {
    const int rows = tt.n_dst[rt.dst[r]], rpb = 256 >> row_lanes_log2(tt.in_dim[rt.src[r]] * es / 16);
    rtl.lo[r] = std::max(at, row_begin);
    rtl.hi[r] = std::max(rtl.lo[r], std::min(at + rows, row_end));
    rtl.tile_off[r + 1] = rtl.tile_off[r] + (rtl.hi[r] - rtl.lo[r] + rpb - 1) / rpb;
    at += rows;
  }
  dim3 grid(tj->blocks + rtl.tile_off[rt.num_rels]);
  if (dtype == HGNN_BF16)
    HGNN_LAUNCH(spmm_fwd_kernel<bf16>, grid, dim3(256), 0, s, L, tt, rt, rtl, (const bf16 *)x, (bf16 *)z, (bf16 *)zlo, *tj);
  else
    HGNN_LAUNCH(spmm_fwd_kernel<float>, grid, dim3(256), 0, s, L, tt, rt, rtl, (const float *)x, (float *)z, (float *)nullptr, *tj);
  HGNN_HIP(hipGetLastError());
  return HGNN_OK;
}

// ------------------------------------------------------------------------------------------
// Backward of the aggregation for ragged widths: dx[c] = sum over the transpose row c of dz[crow] (dz rows arrive
// already scaled by 1/|N_r(v)|) plus, for destination rows, the root-term gradient.
// Rows longer than kLongRow are taken in pieces by the first blocks (long_rows.h).  The others are cut per vertex type
// (lanes per row then fit the type's width).  The dz row of an entry starts at base_r + rho F with one constant per
// relation; the relation of an entry is one of the few that read this type, which a scan with the constants in scalar
// registers finds without a memory access (a binary search per entry cost five dependent loads: 114 us -> 33 us on 10 types
// of 32 to 384 floats, 512 targets).
// ------------------------------------------------------------------------------------------
struct SrcRel {
  int64_t base;   // 16-byte pieces before the dz row of merged row 0, as if the relation's rows went back to there
  int32_t off;    // merged rows before the relation's
  int32_t pad;
};
struct SrcTiles {
  int32_t tile_off[kMaxT + 1];   // blocks before vertex type t
  int32_t first[kMaxT + 1];      // relations reading type t: rel[first[t] .. first[t + 1]), ascending
  SrcRel rel[kMaxR + 4];
};
typedef const SrcTiles __attribute__((address_space(4))) *src_tiles_t;   // the kernel's first argument, read where it lies

// Where the dz rows of U merged rows start, in 16-byte pieces, for one of the relations [j0, j1) that read a type of nvec
// pieces: ascending relations, the last one that starts at or before the row is its own.  Their constants come four at a time: one
// relation after the other, through a list and two tables, each was three dependent loads for every four entries (72k source rows of
// 32 to 384 floats, 268k entries, with the root term's row loaded behind its entries' instead of before: 48.3 -> 41.6 us).
template <int U> __device__ __forceinline__ void dz_rows(src_tiles_t sl, int j0, int j1, int nvec, const int (&rho)[U], int64_t (&at)[U]) {
#pragma unroll
  for (int u = 0; u < U; ++u) at[u] = 0;
  for (int j = j0; j < j1; j += 4) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {   // four places behind the last one exist
      const int off = j + k < j1 ? sl->rel[j + k].off : INT32_MAX;
      const int64_t base = sl->rel[j + k].base;
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (rho[u] >= off) at[u] = base;
    }
  }
#pragma unroll
  for (int u = 0; u < U; ++u) at[u] += (int64_t)rho[u] * nvec;
}

template <typename T, bool WAVE>
__global__ void __launch_bounds__(256) spmm_bwd_kernel(SrcTiles sl_, LayerDev L, TypeTab tt, RelTab rt, uint32_t root_mask, uint32_t want,
                                                        const T *__restrict__ dz, T *__restrict__ dx,
                                                        float *__restrict__ partial, int max_dim, int halves) {
  using V = Vec16<T>;
  const src_tiles_t sl = (src_tiles_t)__builtin_amdgcn_kernarg_segment_ptr();
  (void)sl_;
  const uint4 *zb = reinterpret_cast<const uint4 *>(dz);
  int t = 0;
  const int pieces = WAVE ? L.n_chunks : L.n_chunks << halves, nb_long = long_blocks(pieces, WAVE);
  if ((int)blockIdx.x < nb_long) {
    __shared__ LongLds<V::N> sm;
    __shared__ int64_t s_ats[(WAVE ? 4 : 1) * kChunk];
    const LongSlot<WAVE> slot(pieces);
    const LongPiece p = long_piece(L, slot.item, WAVE ? 0 : halves);
    while (p.c >= tt.row_off[t + 1]) ++t;
    const bool wanted = slot.on && ((want >> t) & 1u);   // else the caller does not want input gradients of this vertex type
    if (!WAVE && (!wanted || p.n <= 0)) return;
    const int F = tt.in_dim[t], nvec = F / V::N, cl = p.c - tt.row_off[t];
    int64_t *s_at = s_ats + slot.lds;
    for (int i = slot.first; i < p.n; i += slot.step) {
      const int rho[1] = {L.crow[p.beg + i]};
      int64_t at[1];
      dz_rows(sl, sl->first[t], sl->first[t + 1], nvec, rho, at);
      s_at[i] = at[0];
    }
    __syncthreads();
    if (!wanted) return;   // whole wavefront
    auto sum = [&](int q, int g, int groups, float (&acc)[V::N]) {
      for (int i = g; i < p.n; i += 4 * groups) {
        uint4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = zb[s_at[min(i + u * groups, p.n - 1)] + q];
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (i + u * groups < p.n) V::add(acc, v[u]);
      }
    };
    auto done = [&](int q, float (&acc)[V::N]) {
      if (cl < tt.n_dst[t] && ((root_mask >> t) & 1u)) V::add(acc, reinterpret_cast<const uint4 *>(dz + (int64_t)rt.zroot_off4[t] * 4 + (int64_t)cl * F)[q]);
      reinterpret_cast<uint4 *>(dx + tt.elem_off[t] + (int64_t)cl * F)[q] = V::pack(acc);
    };
    long_row<WAVE, V::N>(p, slot.item, row_lanes_log2(nvec), nvec, sm, partial, max_dim, L.chunk_count, sum, done);
    return;
  }
  const int b = (int)blockIdx.x - nb_long;
  while (b >= sl->tile_off[t + 1]) ++t;
  const int F = tt.in_dim[t], nvec = F / V::N, l2 = row_lanes_log2(nvec);
  const int c = tt.row_off[t] + (b - sl->tile_off[t]) * (256 >> l2) + (threadIdx.x >> l2);
  if (c >= tt.row_off[t + 1]) return;
  const int beg = L.cptr[c], end = L.cptr[c + 1];
  const int lpr = 1 << l2, lane = threadIdx.x & (lpr - 1);
  const int cl = c - tt.row_off[t];
  const int j0 = sl->first[t], j1 = sl->first[t + 1];
  const bool root = cl < tt.n_dst[t] && ((root_mask >> t) & 1u);
  const uint4 *zr = reinterpret_cast<const uint4 *>(dz + (int64_t)rt.zroot_off4[t] * 4 + (int64_t)cl * F);
  if (end - beg > kLongRow) return;
  for (int q = lane; q < nvec; q += lpr) {
    uint4 rv = make_uint4(0, 0, 0, 0);   // under way while the entries are looked up
    if (root) rv = zr[q];
    float acc[V::N];
#pragma unroll
    for (int i = 0; i < V::N; ++i) acc[i] = 0.f;
    for (int e = beg; e < end; e += 4) {
      int rho[4];
      int64_t at[4];
      uint4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) rho[u] = L.crow[min(e + u, end - 1)];
      dz_rows(sl, j0, j1, nvec, rho, at);
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = zb[at[u] + q];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (e + u < end) V::add(acc, v[u]);
    }
    if (root) V::add(acc, rv);
    reinterpret_cast<uint4 *>(dx + tt.elem_off[t] + (int64_t)cl * F)[q] = V::pack(acc);
  }
}

hgnn_status launch_spmm_bwd(hipStream_t s, int dtype, const LayerDev &L, const TypeTab &tt, const RelTab &rt,
                            const PtrTab &pt, int max_dim, uint32_t want, const void *dz, void *dx, float *partial) {
  if (L.src_rows == 0) return HGNN_OK;
  const int es = dtype == HGNN_BF16 ? 2 : 4;
  uint32_t root_mask = 0;
  bool uniform = true;  // every relation's aggregate rows have the same width: dz row rho starts at rho * F
  for (int t = 0; t < tt.num_types; ++t) {
    if (pt.w_root[t]) root_mask |= 1u << t;
    if (tt.in_dim[t] != tt.in_dim[0]) uniform = false;
  }
  // the uniform-width kernel when it applies, else the one for ragged widths (the rows of `partial` are max_dim floats
  // long, which is the common width in the uniform one)
  if (uniform && launch_spmm_bwd_uniform(s, dtype, L, tt, rt, pt, tt.in_dim[0], want, dz, dx, partial)) {
    HGNN_HIP(hipGetLastError());
  } else {
    SrcTiles sl;
    int n = 0, row_off[kMaxR];
    row_off[0] = 0;
    for (int r = 1; r < rt.num_rels; ++r) row_off[r] = row_off[r - 1] + tt.n_dst[rt.dst[r - 1]];
    sl.tile_off[0] = 0;
    for (int t = 0; t < tt.num_types; ++t) {
      const int nvec = tt.in_dim[t] * es / 16, rpb = 256 >> row_lanes_log2(nvec), rows = ((want >> t) & 1u) ? tt.row_off[t + 1] - tt.row_off[t] : 0;
      sl.tile_off[t + 1] = sl.tile_off[t] + (rows + rpb - 1) / rpb;
      sl.first[t] = n;
      for (int r = 0; r < rt.num_rels; ++r)
        if (rt.src[r] == t) sl.rel[n++] = SrcRel{(int64_t)rt.z_off4[r] * 4 * es / 16 - (int64_t)row_off[r] * nvec, row_off[r], 0};
    }
    sl.first[tt.num_types] = n;
    for (int i = n; i < n + 4; ++i) sl.rel[i] = SrcRel{0, INT32_MAX, 0};
    const int l2 = row_lanes_log2(max_dim * es / 16), halves = long_halves(L.n_chunks, l2);
    const bool by_wave = long_rows_by_wave(L.n_chunks, l2);
    const dim3 grid(long_blocks(L.n_chunks << halves, by_wave) + sl.tile_off[tt.num_types]);
    if (grid.x > 0) {
#define HGNN_BWD(TY, WAVE)                                                                                                        \
  HGNN_LAUNCH((spmm_bwd_kernel<TY, WAVE>), grid, dim3(256), 0, s, sl, L, tt, rt, root_mask, want, (const TY *)dz, (TY *)dx, partial, \
              max_dim, halves)
      if (dtype == HGNN_BF16) {
        if (by_wave) HGNN_BWD(bf16, true); else HGNN_BWD(bf16, false);
      } else {
        if (by_wave) HGNN_BWD(float, true); else HGNN_BWD(float, false);
      }
#undef HGNN_BWD
      HGNN_HIP(hipGetLastError());
    }
  }
  return HGNN_OK;
}

// ------------------------------------------------------------------------------------------
// Weight transposes: Wt[h][f] = W[f][h] for every relation and root weight, as a job list.
// ------------------------------------------------------------------------------------------
void make_transpose_jobs(const TypeTab &tt, const RelTab &rt, const PtrTab &pt, const WtTab &wt, int H, void *wt_buf,
                         TransposeJobs &tj) {
  std::memset(&tj, 0, sizeof(tj));
  tj.H = H;
  tj.out = wt_buf;
  const int R = rt.num_rels, tiles_h = (H + 31) / 32;
  for (int seg = 0; seg < R + tt.num_types; ++seg) {
    const void *w = seg < R ? pt.w_rel[seg] : pt.w_root[seg - R];
    if (!w || tt.n_dst[seg < R ? rt.dst[seg] : seg - R] == 0) continue;  // no destination rows: no tile reads this weight
    const int F = tt.in_dim[seg < R ? rt.src[seg] : seg - R];
    tj.w[tj.n] = w;
    tj.F[tj.n] = F;
    tj.off4[tj.n] = seg < R ? wt.rel4[seg] : wt.root4[seg - R];
    tj.tile_off[tj.n + 1] = tj.tile_off[tj.n] + ((F + 31) / 32) * tiles_h;
    ++tj.n;
  }
  // a tile per block (two dependent memory round trips) up to 2048 blocks: over long before the launch they ride in
  tj.blocks = std::min(2048, tj.tile_off[tj.n]);
}

template <typename T>
__global__ void __launch_bounds__(256) transpose_weights_kernel(TransposeJobs tj) {
  __shared__ T tile[32][33];
  transpose_jobs_block<T>(tj, blockIdx.x, gridDim.x, tile);
}

hgnn_status launch_transpose_jobs(hipStream_t s, int dtype, const TransposeJobs &tj) {
  if (tj.blocks == 0) return HGNN_OK;
  if (dtype == HGNN_BF16) HGNN_LAUNCH(transpose_weights_kernel<bf16>, dim3(tj.blocks), dim3(256), 0, s, tj);
  else HGNN_LAUNCH(transpose_weights_kernel<float>, dim3(tj.blocks), dim3(256), 0, s, tj);
  HGNN_HIP(hipGetLastError());
  return HGNN_OK;
}

hgnn_status launch_transpose_weights(hipStream_t s, int dtype, const TypeTab &tt, const RelTab &rt,
                                     const PtrTab &pt, const WtTab &wt, int H, void *wt_buf) {
  TransposeJobs tj;
  make_transpose_jobs(tt, rt, pt, wt, H, wt_buf, tj);
  return launch_transpose_jobs(s, dtype, tj);
}

// Zero-padded copies: out[off + f*Hp + c] = c < H ? W[f*H + c] : 0  (segment = blockIdx.y).
// Block bx of gx works on segment seg.
template <typename T>
__device__ __forceinline__ void pad_weights_part(const TypeTab &tt, const RelTab &rt, const PtrTab &pt, const WtTab &wo, int H,
                                                 int Hp, T *out, int seg, int bx, int gx) {
  const int R = rt.num_rels;
  const T *w = (const T *)(seg < R ? pt.w_rel[seg] : pt.w_root[seg - R]);
  if (!w || tt.n_dst[seg < R ? rt.dst[seg] : seg - R] == 0) return;  // no destination rows: no tile reads this copy
  const int F = tt.in_dim[seg < R ? rt.src[seg] : seg - R];
  T *o = out + (int64_t)(seg < R ? wo.rel4[seg] : wo.root4[seg - R]) * 4;
  // a block takes whole rows (no division per element)
  for (int f = bx; f < F; f += gx)
    for (int c = threadIdx.x; c < Hp; c += 256) o[(int64_t)f * Hp + c] = c < H ? w[(int64_t)f * H + c] : from_float<T>(0.f);
}

template <typename T>
__global__ void __launch_bounds__(256) pad_weights_kernel(TypeTab tt, RelTab rt, PtrTab pt, WtTab wo, int H, int Hp, T *out) {
  pad_weights_part<T>(tt, rt, pt, wo, H, Hp, out, blockIdx.y, blockIdx.x, gridDim.x);
}

hgnn_status launch_pad_weights(hipStream_t s, int dtype, const TypeTab &tt, const RelTab &rt, const PtrTab &pt,
                               const WtTab &wo, int H, int Hp, void *out) {
  dim3 grid(64, rt.num_rels + tt.num_types);
  if (dtype == HGNN_BF16)
    HGNN_LAUNCH(pad_weights_kernel<bf16>, grid, dim3(256), 0, s, tt, rt, pt, wo, H, Hp, (bf16 *)out);
  else
    HGNN_LAUNCH(pad_weights_kernel<float>, grid, dim3(256), 0, s, tt, rt, pt, wo, H, Hp, (float *)out);
  HGNN_HIP(hipGetLastError());
  return HGNN_OK;
}

// ------------------------------------------------------------------------------------------
// Backward epilogue: gp = grad_h * [h > 0] (when the layer has a ReLU) and dbias_t = column sums.
// One block = kRowsPerBlock rows of one type; a thread owns columns tid, tid+256, ...  The block's column sums are added
// to dbias_t, or, when `bpart` is given, stored as row `block` of bpart [blocks x H] for a later pass that adds
// the rows of a type up (no atomics, and dbias needs no zeroing first).
// ------------------------------------------------------------------------------------------
constexpr int kVecRows = 64;  // rows per block of the 16-bytes-per-lane row pass (32: the same; 128: +3 us; 16, 256: +10 us on the headline)
constexpr int kRowsPerBlock = 8;  // of the element-wise row pass (a multiple of the eight loads in flight per lane)
template <typename T>
__device__ __forceinline__ void relu_bias_rows(const TypeTab &tt, int block, int H, int ldo, int relu, int write,
                                               const T *__restrict__ g, const T *__restrict__ h, T *__restrict__ gp,
                                               const GradPtrTab &gt, float *__restrict__ bpart) {
  int b = block, t = 0;
  for (;; ++t) {
    const int nb = (tt.n_dst[t] + kRowsPerBlock - 1) / kRowsPerBlock;
    if (b < nb) break;
    b -= nb;
  }
  const int r0 = tt.out_row_off[t] + b * kRowsPerBlock;
  const int r1 = min(r0 + kRowsPerBlock, tt.out_row_off[t] + tt.n_dst[t]);
  float *db = gt.dbias[t];
  for (int c = threadIdx.x; c < ldo; c += 256) {
    float sum = 0.f;
    if (c < H) {
      // the block's rows, eight independent loads at a time
      for (int rb = r0; rb < r1; rb += 8) {
        float v[8], hv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int64_t i = (int64_t)min(rb + u, r1 - 1) * H + c;
          v[u] = to_float(g[i]);
          hv[u] = relu ? to_float(h[i]) : 1.f;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          if (rb + u >= r1) break;
          const float x = hv[u] > 0.f ? v[u] : 0.f;
          if (write) gp[(int64_t)(rb + u) * ldo + c] = from_float<T>(x);
          sum += x;
        }
      }
      if (bpart) bpart[(int64_t)block * H + c] = sum;
      else if (db) atomicAdd(db + c, sum);
    } else if (write) {
      for (int r = r0; r < r1; ++r) gp[(int64_t)r * ldo + c] = from_float<T>(0.f);
    }
  }
}

template <typename T>
__global__ void __launch_bounds__(256) relu_bias_bwd_kernel(TypeTab tt, int H, int ldo, int relu, int write, const T *__restrict__ g,
                                                             const T *__restrict__ h, T *__restrict__ gp, GradPtrTab gt) {
  relu_bias_rows<T>(tt, blockIdx.x, H, ldo, relu, write, g, h, gp, gt, nullptr);
}

// Same, 16 bytes per lane: a block owns kVecRows rows of one type, 256/(H/VEC) rows are in flight at a time.
template <typename T>
__device__ __forceinline__ void relu_bias_rows_vec(const TypeTab &tt, int block, int H, int relu, const T *__restrict__ g,
                                                   const T *__restrict__ h, T *__restrict__ gp, const GradPtrTab &gt,
                                                   float *__restrict__ bpart) {
  using V = Vec16<T>;
  __shared__ float red[256 * V::N];
  int b = block, t = 0;
  for (;; ++t) {
    const int nb = (tt.n_dst[t] + kVecRows - 1) / kVecRows;
    if (b < nb) break;
    b -= nb;
  }
  const int chunks = H / V::N;          // <= 256
  const int rif = 256 / chunks;         // rows in flight
  const int c = threadIdx.x % chunks, rg = threadIdx.x / chunks;
  const int r0 = tt.out_row_off[t] + b * kVecRows;
  const int r1 = min(r0 + kVecRows, tt.out_row_off[t] + tt.n_dst[t]);
  float sum[V::N];
#pragma unroll
  for (int i = 0; i < V::N; ++i) sum[i] = 0.f;
  if (rg < rif) {
    // four rows per trip: eight 16-byte loads in flight per lane (a block has few rows, so there are few
    // wavefronts per compute unit to hide the latency otherwise)
    constexpr int U = 4;
    for (int r = r0 + rg; r < r1; r += U * rif) {
      uint4 gv[U], hv4[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int ru = r + u * rif;
        const int64_t i = ((int64_t)(ru < r1 ? ru : r) * H) / V::N + c;
        gv[u] = reinterpret_cast<const uint4 *>(g)[i];
        if (relu) hv4[u] = reinterpret_cast<const uint4 *>(h)[i];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int ru = r + u * rif;
        if (ru >= r1) break;
        const int64_t i = ((int64_t)ru * H) / V::N + c;
        float v[V::N];
#pragma unroll
        for (int k = 0; k < V::N; ++k) v[k] = 0.f;
        V::add(v, gv[u]);
        if (relu) {
          float hv[V::N];
#pragma unroll
          for (int k = 0; k < V::N; ++k) hv[k] = 0.f;
          V::add(hv, hv4[u]);
#pragma unroll
          for (int k = 0; k < V::N; ++k)
            if (!(hv[k] > 0.f)) v[k] = 0.f;
          reinterpret_cast<uint4 *>(gp)[i] = V::pack(v);
        }
#pragma unroll
        for (int k = 0; k < V::N; ++k) sum[k] += v[k];
      }
    }
  }
  float *db = gt.dbias[t];
  if (!db) return;
#pragma unroll
  for (int k = 0; k < V::N; ++k) red[threadIdx.x * V::N + k] = sum[k];
  __syncthreads();
  for (int col = threadIdx.x; col < H; col += 256) {
    const int cc = col / V::N, k = col % V::N;
    float a = 0.f;
    for (int q = 0; q < rif; ++q) a += red[(q * chunks + cc) * V::N + k];
    if (bpart) bpart[(int64_t)block * H + col] = a;
    else atomicAdd(db + col, a);
  }
}

template <typename T>
__global__ void __launch_bounds__(256) relu_bias_bwd_vec_kernel(TypeTab tt, int H, int relu, const T *__restrict__ g,
                                                                 const T *__restrict__ h, T *__restrict__ gp, GradPtrTab gt) {
  relu_bias_rows_vec<T>(tt, blockIdx.x, H, relu, g, h, gp, gt, nullptr);
}

hgnn_status launch_relu_bias_bwd(hipStream_t s, int dtype, const TypeTab &tt, int H, int ldo, int relu,
                                 const void *grad_h, const void *h, void *gp, const GradPtrTab &gt) {
  const int vec = dtype == HGNN_BF16 ? 8 : 4;
  const bool fast = ldo == H && H % vec == 0 && H / vec <= 256 && (((uintptr_t)grad_h | (uintptr_t)h | (uintptr_t)gp) & 15) == 0;
  const int rpb = fast ? kVecRows : kRowsPerBlock;
  const int write = relu || ldo != H;
  int blocks = 0;
  for (int t = 0; t < tt.num_types; ++t) blocks += (tt.n_dst[t] + rpb - 1) / rpb;
  if (blocks == 0) return HGNN_OK;
  if (fast) {
    if (dtype == HGNN_BF16)
      HGNN_LAUNCH(relu_bias_bwd_vec_kernel<bf16>, dim3(blocks), dim3(256), 0, s, tt, H, relu, (const bf16 *)grad_h,
                         (const bf16 *)h, (bf16 *)gp, gt);
    else
      HGNN_LAUNCH(relu_bias_bwd_vec_kernel<float>, dim3(blocks), dim3(256), 0, s, tt, H, relu, (const float *)grad_h,
                         (const float *)h, (float *)gp, gt);
  } else if (dtype == HGNN_BF16) {
    HGNN_LAUNCH(relu_bias_bwd_kernel<bf16>, dim3(blocks), dim3(256), 0, s, tt, H, ldo, relu, write, (const bf16 *)grad_h,
                       (const bf16 *)h, (bf16 *)gp, gt);
  } else {
    HGNN_LAUNCH(relu_bias_bwd_kernel<float>, dim3(blocks), dim3(256), 0, s, tt, H, ldo, relu, write, (const float *)grad_h,
                       (const float *)h, (float *)gp, gt);
  }
  HGNN_HIP(hipGetLastError());
  return HGNN_OK;
}

// ------------------------------------------------------------------------------------------
__device__ __forceinline__ void zero_grads_part(const TypeTab &tt, const RelTab &rt, const GradPtrTab &gt, int H, int seg,
                                                int bx, int gx, bool bias_too) {
  const int R = rt.num_rels;
  float *w;
  int64_t n;
  if (seg < R) {
    w = gt.dw_rel[seg];
    n = (int64_t)tt.in_dim[rt.src[seg]] * H;
  } else {
    const int t = seg - R;
    w = gt.dw_root[t];
    n = (int64_t)tt.in_dim[t] * H;
    float *b = gt.dbias[t];
    if (b && bias_too)
      for (int i = bx * 256 + threadIdx.x; i < H; i += gx * 256) b[i] = 0.f;
  }
  if (!w) return;
  for (int64_t i = bx * 256 + threadIdx.x; i < n; i += (int64_t)gx * 256) w[i] = 0.f;
}

__global__ void __launch_bounds__(256) zero_grads_kernel(TypeTab tt, RelTab rt, GradPtrTab gt, int H) {
  zero_grads_part(tt, rt, gt, H, blockIdx.y, blockIdx.x, gridDim.x, true);
}

hgnn_status launch_zero_grads(hipStream_t s, const TypeTab &tt, const RelTab &rt, const GradPtrTab &gt, int H) {
  HGNN_LAUNCH(zero_grads_kernel, dim3(32, rt.num_rels + tt.num_types), dim3(256), 0, s, tt, rt, gt, H);
  HGNN_HIP(hipGetLastError());
  return HGNN_OK;
}

// The start of a layer's backward pass in ONE launch: the ReLU mask / bias column sums over G (the first
// nb_relu blocks; column sums go to bpart), zeroing of the weight gradients (nb_zero blocks) and of the counters of long
// transpose rows (nb_count), and the zero-padded weight copies (the rest).  They touch different memory and none is big enough to fill the chip alone.
template <typename T, bool VEC>
__global__ void __launch_bounds__(256) bwd_prep_kernel(TypeTab tt, RelTab rt, PtrTab pt, WtTab wo, GradPtrTab gt, int H, int ldo,
                                                        int relu, int write, const T *__restrict__ g, const T *__restrict__ h,
                                                        T *__restrict__ gp, float *__restrict__ bpart, int nb_relu, int nb_zero,
                                                        int nb_count, T *__restrict__ wpad) {
  int b = blockIdx.x;
  if (b < nb_relu) {
    if constexpr (VEC) relu_bias_rows_vec<T>(tt, b, H, relu, g, h, gp, gt, bpart);
    else relu_bias_rows<T>(tt, b, H, ldo, relu, write, g, h, gp, gt, bpart);
    return;
  }
  b -= nb_relu;
  if (b < nb_zero) {
    zero_grads_part(tt, rt, gt, H, b / 32, b % 32, 32, false);
    return;
  }
  b -= nb_zero;
  if (b < nb_count) {
    for (int i = b * 256 + threadIdx.x; i < gt.n_counters; i += nb_count * 256) gt.counters[i] = 0;
    return;
  }
  b -= nb_count;
  pad_weights_part<T>(tt, rt, pt, wo, H, ldo, wpad, b / 64, b % 64, 64);
}

hgnn_status launch_bwd_prep(hipStream_t s, int dtype, const TypeTab &tt, const RelTab &rt, const PtrTab &pt, const WtTab &wo,
                            const GradPtrTab &gt, int H, int ldo, int relu, bool do_rows, bool do_zero, const void *grad_h,
                            const void *h, void *gp, float *bpart, size_t bpart_rows, void *wpad, int *rows_per_block) {
  const int vec = dtype == HGNN_BF16 ? 8 : 4;
  const bool fast = ldo == H && H % vec == 0 && H / vec <= 256 && (((uintptr_t)grad_h | (uintptr_t)h | (uintptr_t)gp) & 15) == 0;
  const int rpb = fast ? kVecRows : kRowsPerBlock;
  *rows_per_block = rpb;
  const int write = relu || ldo != H;
  int nb_relu = 0;
  if (do_rows)
    for (int t = 0; t < tt.num_types; ++t) nb_relu += (tt.n_dst[t] + rpb - 1) / rpb;
  if (bpart && (size_t)nb_relu > bpart_rows) {  // the caller sized the area for another form of the row pass
    set_error("partial bias sums: %d rows for an area of %zu", nb_relu, bpart_rows);
    return HGNN_EINVAL;
  }
  const int segs = rt.num_rels + tt.num_types;
  const int nb_zero = do_zero ? 32 * segs : 0, nb_pad = wpad ? 64 * segs : 0;
  const int nb_count = std::min(32, (gt.n_counters + 255) / 256);
  const int blocks = nb_relu + nb_zero + nb_count + nb_pad;
  if (blocks == 0) return HGNN_OK;
#define HGNN_PREP(TY, VE)                                                                                              \
  HGNN_LAUNCH((bwd_prep_kernel<TY, VE>), dim3(blocks), dim3(256), 0, s, tt, rt, pt, wo, gt, H, ldo, relu, write,        \
              (const TY *)grad_h, (const TY *)h, (TY *)gp, bpart, nb_relu, nb_zero, nb_count, (TY *)wpad)
  if (dtype == HGNN_BF16) {
    if (fast) HGNN_PREP(bf16, true); else HGNN_PREP(bf16, false);
  } else {
    if (fast) HGNN_PREP(float, true); else HGNN_PREP(float, false);
  }
#undef HGNN_PREP
  HGNN_HIP(hipGetLastError());
  return HGNN_OK;
}

__global__ void __launch_bounds__(256) bias_reduce_kernel(TypeTab tt, GradPtrTab gt, int H, int rpb, const float *__restrict__ bpart) {
  __shared__ float red[256];
  bias_reduce_part(tt.n_dst, gt.dbias, H, rpb, bpart, blockIdx.x, red);
}

hgnn_status launch_bias_reduce(hipStream_t s, const TypeTab &tt, const GradPtrTab &gt, int H, int rpb, const float *bpart) {
  HGNN_LAUNCH(bias_reduce_kernel, dim3(bias_reduce_blocks(tt.num_types, H)), dim3(256), 0, s, tt, gt, H, rpb, bpart);
  HGNN_HIP(hipGetLastError());
  return HGNN_OK;
}

__global__ void __launch_bounds__(256) fill_zero_kernel(uint4 *p, size_t n16, char *tail, size_t ntail) {
  const uint4 z = make_uint4(0, 0, 0, 0);
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n16; i += (size_t)gridDim.x * 256) p[i] = z;
  if (blockIdx.x == 0 && threadIdx.x < ntail) tail[threadIdx.x] = 0;
}

hgnn_status launch_fill_zero(hipStream_t s, void *p, size_t bytes) {
  if (bytes == 0) return HGNN_OK;
  const size_t n16 = bytes / 16;
  const int blocks = (int)std::min<size_t>(2048, (n16 + 255) / 256 + 1);
  HGNN_LAUNCH(fill_zero_kernel, dim3(blocks), dim3(256), 0, s, (uint4 *)p, n16, (char *)p + n16 * 16, bytes - n16 * 16);
  HGNN_HIP(hipGetLastError());
  return HGNN_OK;
}

// ------------------------------------------------------------------------------------------
// Naive-structure helper: h = act(acc32 + bias) for one vertex type.
// ------------------------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(256) bias_act_kernel(int64_t row0, int64_t n_rows, int H, int relu, const float *bias,
                                                        const float *__restrict__ acc, T *__restrict__ h) {
  const int64_t n = n_rows * H;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    float v = acc[row0 * H + i];
    if (bias) v += bias[i % H];
    if (relu) v = fmaxf(v, 0.f);
    h[row0 * H + i] = from_float<T>(v);
  }
}

template <typename T>
__global__ void __launch_bounds__(256) bias_act_typed_kernel(int64_t row0, int64_t n_rows, int H, int relu, const T *bias,
                                                              const float *__restrict__ acc, T *__restrict__ h) {
  const int64_t n = n_rows * H;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    float v = acc[row0 * H + i];
    if (bias) v += to_float(bias[i % H]);
    if (relu) v = fmaxf(v, 0.f);
    h[row0 * H + i] = from_float<T>(v);
  }
}

hgnn_status launch_bias_act(hipStream_t s, int dtype, const TypeTab &tt, const PtrTab &pt, int H, int relu,
                            int type, const float *acc32, void *h) {
  const int64_t n_rows = tt.n_dst[type];
  if (n_rows == 0) return HGNN_OK;
  const int blocks = (int)std::min<int64_t>(4096, (n_rows * H + 255) / 256);
  if (dtype == HGNN_BF16)
    HGNN_LAUNCH(bias_act_typed_kernel<bf16>, dim3(blocks), dim3(256), 0, s, (int64_t)tt.out_row_off[type], n_rows, H,
                       relu, (const bf16 *)pt.bias[type], acc32, (bf16 *)h);
  else
    HGNN_LAUNCH(bias_act_typed_kernel<float>, dim3(blocks), dim3(256), 0, s, (int64_t)tt.out_row_off[type], n_rows, H,
                       relu, (const float *)pt.bias[type], acc32, (float *)h);
  HGNN_HIP(hipGetLastError());
  return HGNN_OK;
}

// ------------------------------------------------------------------------------------------
// Mean softmax cross-entropy and its gradient.
// ------------------------------------------------------------------------------------------
// V = values a lane keeps per row (C <= 64 V).  A wavefront takes kXentRows rows at a time: their values and labels are
// read with unconditional loads (clamped indices) that are all in flight together, so a trip costs one memory round
// trip, and the arithmetic runs out of registers.  The loss leaves a block as ONE atomic add, and the grid is kept to
// 256 blocks: adds to one address are serialised by the memory system at ~11 ns each (1024 blocks of one row per
// wavefront spent 11 of their 16 us there).  V = 0 is the form for any C, which re-reads a row for each of its passes.
constexpr int kXentRows = 4;
template <typename T, int V>
__global__ void __launch_bounds__(256) xent_kernel(const T *__restrict__ logits, const int64_t *__restrict__ labels,
                                                    int64_t rows, int C, float *loss, T *__restrict__ grad) {
  __shared__ float part[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const float inv_rows = 1.0f / (float)rows;
  float my_loss = 0.f;
  if constexpr (V > 0) {
    for (int64_t row0 = ((int64_t)blockIdx.x * 4 + wave) * kXentRows; row0 < rows; row0 += (int64_t)gridDim.x * 4 * kXentRows) {
      float x[kXentRows][V];
      int lab[kXentRows];
#pragma unroll
      for (int j = 0; j < kXentRows; ++j) {
        const int64_t row = min(row0 + j, rows - 1);
        lab[j] = (int)labels[row];
#pragma unroll
        for (int i = 0; i < V; ++i) {
          const int c = lane + 64 * i;
          const float v = to_float(logits[row * C + min(c, C - 1)]);
          x[j][i] = c < C ? v : -INFINITY;
        }
      }
#pragma unroll
      for (int j = 0; j < kXentRows; ++j) {
        if (row0 + j >= rows) break;
        float m = x[j][0];
#pragma unroll
        for (int i = 1; i < V; ++i) m = fmaxf(m, x[j][i]);
        for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
        float sum = 0.f, zl = 0.f;
#pragma unroll
        for (int i = 0; i < V; ++i) {
          if (lane + 64 * i == lab[j]) zl = x[j][i];
          x[j][i] = __expf(x[j][i] - m);   // exp(-inf) = 0 beyond the row
          sum += x[j][i];
        }
        for (int o = 32; o > 0; o >>= 1) {
          sum += __shfl_xor(sum, o);
          zl += __shfl_xor(zl, o);
        }
        const float inv_sum = 1.0f / sum;
#pragma unroll
        for (int i = 0; i < V; ++i) {
          const int c = lane + 64 * i;
          float p = x[j][i] * inv_sum;
          if (c == lab[j]) p -= 1.0f;
          if (c < C) grad[(row0 + j) * C + c] = from_float<T>(p * inv_rows);
        }
        my_loss += (logf(sum) + m - zl) * inv_rows;
      }
    }
  } else {
    for (int64_t row = (int64_t)blockIdx.x * 4 + wave; row < rows; row += (int64_t)gridDim.x * 4) {
      const T *z = logits + row * C;
      const int lab = (int)labels[row];
      float m = -INFINITY;
      for (int c = lane; c < C; c += 64) m = fmaxf(m, to_float(z[c]));
      for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
      float sum = 0.f;
      for (int c = lane; c < C; c += 64) sum += __expf(to_float(z[c]) - m);
      for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
      const float inv_sum = 1.0f / sum;
      for (int c = lane; c < C; c += 64) {
        float p = __expf(to_float(z[c]) - m) * inv_sum;
        if (c == lab) p -= 1.0f;
        grad[row * C + c] = from_float<T>(p * inv_rows);
      }
      my_loss += (logf(sum) + m - to_float(z[lab])) * inv_rows;
    }
  }
  if (lane == 0) part[wave] = my_loss;
  __syncthreads();
  if (threadIdx.x == 0) atomicAdd(loss, part[0] + part[1] + part[2] + part[3]);
}

template <typename T>
static void launch_xent_typed(hipStream_t s, const void *logits, const int64_t *labels, int64_t rows, int C, float *loss, void *grad) {
  dim3 grid((unsigned)std::min<int64_t>(256, (rows + 4 * kXentRows - 1) / (4 * kXentRows)));
#define HGNN_XENT(V_) HGNN_LAUNCH((xent_kernel<T, V_>), grid, dim3(256), 0, s, (const T *)logits, labels, rows, C, loss, (T *)grad)
  if (C <= 128) HGNN_XENT(2);
  else if (C <= 256) HGNN_XENT(4);
  else if (C <= 384) HGNN_XENT(6);
  else if (C <= 512) HGNN_XENT(8);
  else HGNN_XENT(0);
#undef HGNN_XENT
}

hgnn_status launch_xent(hipStream_t s, int dtype, const void *logits, const int64_t *labels, int64_t rows,
                        int classes, float *loss, void *grad) {
  hgnn_status st = launch_fill_zero(s, loss, sizeof(float));
  if (st != HGNN_OK) return st;
  if (rows == 0) return HGNN_OK;
  if (dtype == HGNN_BF16) launch_xent_typed<bf16>(s, logits, labels, rows, classes, loss, grad);
  else launch_xent_typed<float>(s, logits, labels, rows, classes, loss, grad);
  HGNN_HIP(hipGetLastError());
  return HGNN_OK;
}

}  // namespace hgnn
