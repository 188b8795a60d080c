// Host side of the attention variant (per-relation edge attention with semantic-attention fusion): argument checks,
// work-area layout and launch sequences of its forward and backward passes.
#include <algorithm>
#include <cstring>

#include "attn_layer.h"
#include "layer_host.h"

namespace hgnn {
namespace {

constexpr int kSemDimHost = 128;

// Plan (tables, work-area layout) shared by forward and backward.
struct AttnPlan {
  TypeTab tt;
  RelTab rt;
  RelRows rr;
  PtrTab pt;      // w_root := w_type (per-type projection), bias
  AttnPtrs ap;
  LayerDev dev;
  int H = 0, heads = 1;
  int64_t src_rows = 0, rows = 0, edges = 0, total_dst = 0;
  // saved (forward -> backward)
  size_t s_z = 0, s_m = 0, s_t = 0, s_mx = 0, s_ls = 0, s_beta = 0, s_wsum = 0, saved_bytes = 0;
  // scratch (backward)
  size_t c_gp = 0, c_dbeta = 0, c_dm = 0, c_edge = 0, c_xsum = 0, c_dsum = 0, c_dz = 0, c_partial = 0, c_count = 0, scratch_bytes = 0;
};

hgnn_status make_attn_plan(hgnn_ctx *ctx, hgnn_graph *g, int32_t layer, const hgnn_layer_params *p, AttnPlan &pl, bool need_built) {
  if (!ctx || !g || !p) HGNN_FAIL(HGNN_EINVAL, "NULL context, graph or parameters");
  if (layer < 0 || layer >= g->num_layers) HGNN_FAIL(HGNN_EINVAL, "layer %d outside [0,%d)", layer, g->num_layers);
  if (ctx->fuse != HGNN_FUSE_SEMATTN) HGNN_FAIL(HGNN_EUNSUPPORTED, "attention aggregation is implemented with semantic-attention fusion only");
  if (!p->in_dim || !p->w_type || !p->a_src || !p->a_dst || !p->w_sem || !p->b_sem || !p->q_sem || p->out_dim <= 0)
    HGNN_FAIL(HGNN_EINVAL, "incomplete attention layer parameters");
  const int T = ctx->T, R = ctx->R;
  const LayerHost &L = g->L[layer];
  // The attention variant computes and keeps its intermediates (projected features, aggregates, scores, every
  // gradient between the stages) in fp32 whatever the storage type: the gradients of the attention vectors are what
  // is left of a cancellation between the neighbours of a vertex (the softmax gradient sums to zero over them), and
  // the ReLU decisions sit on sums without head-room, so both need more than bf16 intermediates carry.  In bf16
  // storage the kernels widen inputs, parameters and the incoming gradient as they load them (exact); the layer output,
  // the input gradient and the projected features' gradient are rounded once on the way out.
  const int vec = 4, es = esize(ctx->dtype), vec_io = 16 / es;
  pl.H = p->out_dim;
  pl.heads = ctx->heads;
  if (pl.H % pl.heads) HGNN_FAIL(HGNN_EINVAL, "out_dim %d is not a multiple of heads %d", pl.H, pl.heads);
  const int D = pl.H / pl.heads;
  auto pow2 = [](int n) { return n > 0 && (n & (n - 1)) == 0; };
  if (D % vec || !pow2(D / vec) || !pow2(pl.H / vec) || pl.H / vec > 64)
    HGNN_FAIL(HGNN_EUNSUPPORTED, "attention needs out_dim/heads = %d scalars x a power of two and out_dim/%d a power of two <= 64", vec, vec);
  if (L.tmask != ~0u) HGNN_FAIL(HGNN_EINVAL, "the attention variant needs the transpose entries of every vertex type");
  if (es == 2 && pl.H % vec_io) HGNN_FAIL(HGNN_EUNSUPPORTED, "out_dim %d is not a multiple of %d", pl.H, vec_io);
  std::memset(&pl.tt, 0, sizeof(pl.tt));
  std::memset(&pl.rt, 0, sizeof(pl.rt));
  std::memset(&pl.rr, 0, sizeof(pl.rr));
  std::memset(&pl.pt, 0, sizeof(pl.pt));
  std::memset(&pl.ap, 0, sizeof(pl.ap));
  pl.tt.num_types = T;
  pl.rt.num_rels = R;
  pl.rr.n = R;
  int64_t eo = 0;
  for (int t = 0; t < T; ++t) {
    if (p->in_dim[t] <= 0 || p->in_dim[t] % vec_io != 0)
      HGNN_FAIL(HGNN_EUNSUPPORTED, "in_dim[%d]=%d is not a positive multiple of %d", t, p->in_dim[t], vec_io);
    if (!p->w_type[t] || ((uintptr_t)p->w_type[t] & 15)) HGNN_FAIL(HGNN_EINVAL, "w_type[%d] is NULL or not 16-byte aligned", t);
    pl.tt.in_dim[t] = p->in_dim[t];
    pl.tt.n_dst[t] = (int32_t)L.n_dst[t];
    pl.tt.elem_off[t] = eo;
    pl.tt.xroot_off[t] = eo;
    eo += L.n_src[t] * (int64_t)p->in_dim[t];
    pl.tt.row_off[t + 1] = pl.tt.row_off[t] + (int32_t)L.n_src[t];
    pl.tt.out_row_off[t + 1] = pl.tt.out_row_off[t] + (int32_t)L.n_dst[t];
    pl.pt.w_root[t] = p->w_type[t];
    pl.pt.bias[t] = p->bias ? p->bias[t] : nullptr;
  }
  pl.tt.elem_off[T] = eo;
  for (int r = 0; r < R; ++r) {
    if (!p->a_src[r] || !p->a_dst[r] || (((uintptr_t)p->a_src[r] | (uintptr_t)p->a_dst[r]) & 15))
      HGNN_FAIL(HGNN_EINVAL, "a_src[%d] / a_dst[%d] is NULL or not 16-byte aligned", r, r);
    const int d = ctx->rel_dst[r];
    pl.rt.src[r] = (uint8_t)ctx->rel_src[r];
    pl.rt.dst[r] = pl.rr.dst[r] = (uint8_t)d;
    pl.rr.row_off[r + 1] = pl.rr.row_off[r] + pl.tt.n_dst[d];
    pl.rr.zdst[r] = pl.tt.row_off[d];
    pl.rr.gdst[r] = pl.tt.out_row_off[d];
    pl.ap.a_src[r] = p->a_src[r];
    pl.ap.a_dst[r] = p->a_dst[r];
  }
  if (((uintptr_t)p->w_sem | (uintptr_t)p->b_sem | (uintptr_t)p->q_sem) & 15) HGNN_FAIL(HGNN_EINVAL, "semantic attention parameters must be 16-byte aligned");
  pl.src_rows = L.src_rows; pl.rows = L.rows; pl.edges = L.edges; pl.total_dst = pl.tt.out_row_off[T];
  const size_t H = (size_t)pl.H, hd = (size_t)pl.heads;
  auto take = [](size_t &o, size_t bytes) { const size_t at = o; o += align_up(std::max<size_t>(bytes, 1), 256); return at; };
  size_t o = 0;
  pl.s_z = take(o, (size_t)pl.src_rows * H * 4);
  pl.s_m = take(o, (size_t)pl.rows * H * 4);
  pl.s_t = take(o, (size_t)pl.rows * kSemDimHost * 4);
  pl.s_mx = take(o, (size_t)pl.rows * hd * 4);
  pl.s_ls = take(o, (size_t)pl.rows * hd * 4);
  pl.s_beta = take(o, (size_t)kMaxR * 4);
  pl.s_wsum = take(o, (size_t)kMaxR * 8);
  pl.saved_bytes = o;
  o = 0;
  pl.c_gp = take(o, (size_t)pl.total_dst * H * es);            // incoming gradient masked by the activation
  pl.c_dbeta = take(o, (size_t)kMaxR * 4);
  pl.c_dm = take(o, (size_t)pl.rows * H * 4);
  pl.c_edge = take(o, (size_t)pl.edges * hd * 8);              // per edge and head: (alpha, dalpha)
  pl.c_xsum = take(o, (size_t)pl.rows * hd * 4);
  pl.c_dsum = take(o, (size_t)pl.rows * hd * 4);
  pl.c_dz = take(o, (size_t)pl.src_rows * H * es);
  pl.c_partial = take(o, (size_t)L.max_chunks * H * 4);
  pl.c_count = take(o, (size_t)L.max_chunks * 4);
  pl.scratch_bytes = o;
  if (need_built) return layer_dev(ctx, g, layer, pl.dev);
  return HGNN_OK;
}

hgnn_status attn_workspace(hgnn_ctx *ctx, hgnn_graph *g, int32_t layer, const hgnn_layer_params *p, size_t *saved_bytes, size_t *scratch_bytes) {
  AttnPlan pl;
  const hgnn_status st = make_attn_plan(ctx, g, layer, p, pl, false);
  if (st != HGNN_OK) return st;
  if (saved_bytes) *saved_bytes = pl.saved_bytes;
  if (scratch_bytes) *scratch_bytes = pl.scratch_bytes;
  return HGNN_OK;
}

hgnn_status attn_fwd(hgnn_ctx *ctx, void *stream, hgnn_graph *g, int32_t layer, const hgnn_layer_params *p, const void *x, void *h,
                     void *saved, size_t saved_bytes, void *scratch, size_t scratch_bytes) {
  AttnPlan pl;
  hgnn_status st = make_attn_plan(ctx, g, layer, p, pl, true);
  if (st != HGNN_OK) return st;
  if (pl.src_rows > 0 && !x) HGNN_FAIL(HGNN_EINVAL, "x_merged is NULL");
  if (pl.total_dst > 0 && !h) HGNN_FAIL(HGNN_EINVAL, "h_out is NULL");
  if (!saved || !scratch) HGNN_FAIL(HGNN_EINVAL, "NULL work area");
  if (saved_bytes < pl.saved_bytes || scratch_bytes < pl.scratch_bytes)
    HGNN_FAIL(HGNN_EINVAL, "work areas too small: need %zu saved, %zu scratch bytes", pl.saved_bytes, pl.scratch_bytes);
  if (((uintptr_t)saved | (uintptr_t)scratch | (uintptr_t)x | (uintptr_t)h) & 15)
    HGNN_FAIL(HGNN_EINVAL, "device buffers must be 16-byte aligned");
  hipStream_t s = (hipStream_t)stream;
  HGNN_HIP(wait_upload(g, s));
  char *sv = (char *)saved;
  float *z = (float *)(sv + pl.s_z), *m = (float *)(sv + pl.s_m), *t = (float *)(sv + pl.s_t);
  double *wsum = (double *)(sv + pl.s_wsum);
  float *beta = (float *)(sv + pl.s_beta);
  {
    Probe pb(ctx, HGNN_K_GEMM_FWD, layer);
    if ((st = launch_attn_proj(s, ctx->dtype, pl.tt, pl.pt, pl.H, x, z, wsum)) != HGNN_OK) return st;
  }
  {
    Probe pb(ctx, HGNN_K_SPMM_FWD, layer);
    if ((st = launch_attn_agg(s, ctx->dtype, pl.dev, pl.rr, pl.ap, pl.H, pl.heads, z, m, (float *)(sv + pl.s_mx), (float *)(sv + pl.s_ls))) != HGNN_OK) return st;
  }
  if ((st = launch_attn_sem(s, ctx->dtype, pl.rr, pl.H, m, p->w_sem, p->b_sem, p->q_sem, t, wsum)) != HGNN_OK) return st;
  return launch_attn_fuse(s, ctx->dtype, pl.tt, pl.rr, pl.pt, pl.H, p->relu, m, wsum, beta, h);
}

hgnn_status attn_bwd(hgnn_ctx *ctx, void *stream, hgnn_graph *g, int32_t layer, const hgnn_layer_params *p, const void *x,
                     const void *h_out, const void *saved, const void *grad_h, void *grad_x, const hgnn_layer_grads *go, void *scratch,
                     size_t scratch_bytes) {
  AttnPlan pl;
  hgnn_status st = make_attn_plan(ctx, g, layer, p, pl, true);
  if (st != HGNN_OK) return st;
  if (!saved || !scratch || !go) HGNN_FAIL(HGNN_EINVAL, "NULL work area or gradient table");
  if (!go->dw_type || !go->da_src || !go->da_dst || !go->dw_sem || !go->db_sem || !go->dq_sem)
    HGNN_FAIL(HGNN_EINVAL, "the attention backward needs every gradient buffer of the attention parameters");
  if (pl.total_dst > 0 && (!x || !grad_h || (p->relu && !h_out))) HGNN_FAIL(HGNN_EINVAL, "NULL input");
  if (scratch_bytes < pl.scratch_bytes) HGNN_FAIL(HGNN_EINVAL, "scratch too small: need %zu bytes", pl.scratch_bytes);
  if (((uintptr_t)saved | (uintptr_t)scratch | (uintptr_t)x | (uintptr_t)grad_h | (uintptr_t)grad_x | (uintptr_t)(p->relu ? h_out : nullptr)) & 15)
    HGNN_FAIL(HGNN_EINVAL, "device buffers must be 16-byte aligned");
  const int R = ctx->R, T = ctx->T, H = pl.H, dtype = ctx->dtype;
  hipStream_t s = (hipStream_t)stream;
  HGNN_HIP(wait_upload(g, s));
  const char *sv = (const char *)saved;
  char *sc = (char *)scratch;
  const LayerHost &L = g->L[layer];
  const float *z = (const float *)(sv + pl.s_z), *m = (const float *)(sv + pl.s_m), *t = (const float *)(sv + pl.s_t);
  const float *beta = (const float *)(sv + pl.s_beta);
  float *dbeta = (float *)(sc + pl.c_dbeta), *dm = (float *)(sc + pl.c_dm);
  // zero everything that is accumulated into
  GradPtrTab gt;
  AttnPtrs dap;
  std::memset(&gt, 0, sizeof(gt));
  std::memset(&dap, 0, sizeof(dap));
  {
    float *zp[2 * kMaxR + 2 * kMaxT + 8];   // the launcher's table holds as many
    int64_t zn[2 * kMaxR + 2 * kMaxT + 8];
    int n = 0;
    auto zero = [&](float *q, int64_t len) { zp[n] = q; zn[n++] = len; };
    for (int i = 0; i < T; ++i) {
      if (!go->dw_type[i]) HGNN_FAIL(HGNN_EINVAL, "dw_type[%d] is NULL", i);
      gt.dw_root[i] = go->dw_type[i];
      gt.dbias[i] = (go->dbias && p->bias && p->bias[i]) ? go->dbias[i] : nullptr;
      zero(go->dw_type[i], (int64_t)p->in_dim[i] * H);
      if (gt.dbias[i]) zero(gt.dbias[i], H);
    }
    for (int r = 0; r < R; ++r) {
      if (!go->da_src[r] || !go->da_dst[r]) HGNN_FAIL(HGNN_EINVAL, "da_src[%d] / da_dst[%d] is NULL", r, r);
      dap.a_src[r] = go->da_src[r];
      dap.a_dst[r] = go->da_dst[r];
      zero(go->da_src[r], H);
      zero(go->da_dst[r], H);
    }
    zero(go->dw_sem, (int64_t)H * kSemDimHost);
    zero(go->db_sem, kSemDimHost);
    zero(go->dq_sem, kSemDimHost);
    zero(dbeta, kMaxR);
    pl.dev.chunk_count = (uint32_t *)(sc + pl.c_count);
    zero((float *)pl.dev.chunk_count, pl.dev.n_chunks);
    Probe pb(ctx, HGNN_K_ZERO_GRADS, layer);
    if ((st = launch_attn_zero(s, zp, zn, n)) != HGNN_OK) return st;
  }
  const void *gp = p->relu ? sc + pl.c_gp : grad_h;   // without an activation the incoming gradient is G' itself
  {
    Probe pb(ctx, HGNN_K_RELU_BIAS_BWD, layer);
    if ((st = launch_attn_mask_dbeta(s, dtype, pl.tt, pl.rr, gt, H, p->relu, grad_h, h_out, sc + pl.c_gp, m, dbeta)) != HGNN_OK) return st;
  }
  {
    Probe pb(ctx, HGNN_K_GEMM_DA, layer);
    if ((st = launch_attn_sem_bwd(s, dtype, pl.rr, H, m, t, p->w_sem, p->q_sem, gp, beta, dbeta, dm, go->dw_sem, go->dq_sem, go->db_sem)) != HGNN_OK) return st;
  }
  {
    Probe pb(ctx, HGNN_K_SPMM_BWD, layer);
    if ((st = launch_attn_agg_bwd(s, dtype, pl.dev, pl.tt, pl.rr, pl.ap, dap, H, pl.heads, z, dm, (const float *)(sv + pl.s_mx),
                                  (const float *)(sv + pl.s_ls), sc + pl.c_edge, (float *)(sc + pl.c_xsum), (float *)(sc + pl.c_dsum),
                                  sc + pl.c_dz, (float *)(sc + pl.c_partial))) != HGNN_OK) return st;
  }
  if (pl.src_rows == 0) return HGNN_OK;
  // Projection backward on the layer GEMMs: every type is a "root" segment over ALL its source rows.  In bf16 storage both
  // products run on the bf16 MFMA kernels, on the caller's own x and weights and on dZ rounded to bf16 (a relative 2^-9
  // per element of a gradient that is summed over the rows; no decision hangs on it).
  TypeTab tt2 = pl.tt;
  RelTab rt2 = pl.rt;
  DwTab dt, da;
  for (int i = 0; i < T; ++i) {
    tt2.n_dst[i] = (int32_t)L.n_src[i];
    tt2.out_row_off[i + 1] = pl.tt.row_off[i + 1];
    rt2.zroot_off4[i] = (uint32_t)(pl.tt.elem_off[i] / 4);
  }
  // tiles of 128 rows and columns, or of 64 (bwd_small_tiles)
  int split_rows = 0;
  BwdCols cols;
  for (int i = 0; i < T; ++i)
    if (L.n_src[i] > 0) {
      cols.segment(p->in_dim[i]);
      ++cols.types;
    }
  for (int edge = 128;; edge = 64) {
    std::memset(&dt, 0, sizeof(dt));
    std::memset(&da, 0, sizeof(da));
    dt.edge = da.edge = edge;
    const int bk = dtype == HGNN_BF16 ? 64 : 32, tiles_h = (H + edge - 1) / edge;
    int64_t dw_steps = 0;
    int ne = 0, na = 0;
    for (int i = 0; i < T; ++i) {
      dt.first[i] = (uint16_t)ne;
      da.first[i] = (uint16_t)na;
      const int u = L.n_src[i] > 0 ? (p->in_dim[i] + edge - 1) / edge : 0;
      const bool want = grad_x && u && (!p->input_grad || p->input_grad[i]);
      if (u) dt.seg[ne++] = (uint8_t)(R + i);
      if (want) da.seg[na++] = (uint8_t)(R + i);
      dt.u_total[i] = (uint16_t)u;
      da.u_total[i] = (uint16_t)(want ? u : 0);
      da.tile_off[i + 1] = da.tile_off[i] + (want ? u * (int)((L.n_src[i] + edge - 1) / edge) : 0);
      dw_steps += (int64_t)u * tiles_h * ((L.n_src[i] + bk - 1) / bk);
    }
    dt.first[T] = (uint16_t)ne;
    da.first[T] = (uint16_t)na;
    split_rows = dw_slice_rows(dtype, edge, dw_steps, (int64_t)da.tile_off[T] * ((H + bk - 1) / bk));
    for (int i = 0; i < T; ++i)
      dt.tile_off[i + 1] = dt.tile_off[i] + dt.u_total[i] * tiles_h * (int)((L.n_src[i] + split_rows - 1) / split_rows);
    if (edge == 64 || !bwd_small_tiles(dtype, dt.tile_off[T] + da.tile_off[T], H, cols, da.tile_off[T] > 0)) break;
  }
  Probe pb(ctx, HGNN_K_GEMM_DW, layer);
  const void *dzp = sc + pl.c_dz;
  if (da.tile_off[T] > 0)
    return launch_gemm_bwd(s, dtype, pl.dev, tt2, rt2, pl.pt, da, gt, dt, split_rows, H, H, true, x, nullptr, dzp, grad_x, nullptr, 0);
  return launch_gemm_dw(s, dtype, pl.dev, tt2, rt2, gt, dt, split_rows, H, H, true, x, nullptr, dzp);
}

hgnn_status attn_launch_count(hgnn_ctx *ctx, hgnn_graph *g, int32_t layer, const hgnn_layer_params *p, int32_t *fwd, int32_t *bwd) {
  AttnPlan pl;
  const hgnn_status st = make_attn_plan(ctx, g, layer, p, pl, true);
  if (st != HGNN_OK) return st;
  // projection, aggregation, semantic scores, fusion
  if (fwd) *fwd = (pl.src_rows > 0) + 2 * (pl.rows > 0) + (pl.total_dst > 0);
  // zero, mask + relation dots, semantic products, row pass, transpose pass, projection
  if (bwd) *bwd = 1 + (pl.total_dst > 0) + 2 * (pl.rows > 0) + (pl.src_rows > 0 ? 2 : 0);
  return HGNN_OK;
}

const bool registered = [] {
  attn_variant() = AttnVariant{attn_workspace, attn_fwd, attn_bwd, attn_launch_count};
  return true;
}();

}  // namespace
}  // namespace hgnn
