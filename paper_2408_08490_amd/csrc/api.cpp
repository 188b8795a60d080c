// C ABI entry points: argument checks, per-call planning (offset tables), launch sequences.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <unistd.h>

#include "layer_host.h"

namespace hgnn {
const char *get_error();

// Works off the context's queue with one of its builders (on a thread of the crew), as long as no other context's task
// waits for a thread: between two graphs the task then goes to the end of the crew's list.
static void build_queued(hgnn_ctx *ctx) {
  if (ctx->device >= 0) (void)hipSetDevice(ctx->device);
  Builder *bd = nullptr;
  for (;;) {
    hgnn_graph *g = nullptr;
    {
      std::lock_guard<std::mutex> lk(ctx->qm);
      if (!bd) {
        // there is one for each task (enqueue_graph); best one whose scratch this thread used before or nobody did
        // (it then lies in memory near the thread), else the one used last
        auto &idle = ctx->idle_builders;
        size_t at = idle.size() - 1;
        const int me = Crew::index();
        for (size_t i = 0; i < idle.size(); ++i)
          if (idle[i]->user == me) { at = i; break; }
          else if (idle[i]->user < 0) at = i;
        bd = idle[at];
        idle.erase(idle.begin() + at);
        bd->user = me;
      } else if (!ctx->queue.empty() && Crew::get().wanted()) {
        ctx->idle_builders.push_back(bd);
        Crew::get().submit([ctx] { build_queued(ctx); });
        return;
      }
      if (ctx->queue.empty()) {
        ctx->idle_builders.push_back(bd);
        --ctx->building;
        ctx->qcv.notify_all();   // under the lock: hgnn_destroy frees the context once it holds it
        return;
      }
      g = ctx->queue.front();
      ctx->queue.pop_front();
    }
    build_graph_job(ctx, *bd, g);
  }
}

static void free_slab(hgnn_ctx *ctx, Slab &s) {
  if (ctx->device >= 0) {
    if (s.host) (void)hipHostFree(s.host);
    if (s.dev) (void)hipFree(s.dev);
  } else {
    free(s.host);
  }
  s = Slab();
}

// Looks at the state for a while: a build that is under way often ends before a sleeping thread would be awake again.
static void look_built(hgnn_graph *g) {
  if (!Crew::get().look()) return;
  const auto t0 = std::chrono::steady_clock::now();
  for (int i = 1; g->state.load(std::memory_order_acquire) == 0; ++i) {
    cpu_relax();
    if (i % 64 == 0 && std::chrono::steady_clock::now() - t0 > std::chrono::microseconds(2 * Crew::kSpinUs)) break;
  }
}

static hgnn_status wait_built(hgnn_graph *g) {
  look_built(g);
  std::unique_lock<std::mutex> lk(g->m);   // also when the state is known: the builder's last touch of g is under it
  g->cv.wait(lk, [&] { return g->state != 0; });
  if (g->state == 2) HGNN_FAIL((hgnn_status)g->status, "graph build failed: %s", g->err.c_str());
  return HGNN_OK;
}

// Everything a layer call derives from (schema, graph, parameters) before launching.
struct Plan {
  TypeTab tt;
  RelTab rt;
  PtrTab pt;
  WtTab wt;
  LayerDev dev;
  int H = 0, max_dim = 0, es = 4;
  int64_t total_dst = 0;
  size_t z_elems = 0, zroot_elems = 0, wt_elems = 0;
  size_t saved_bytes = 0, scratch_bytes = 0;
  size_t off_wt = 0, off_gp = 0, off_dz = 0, off_partial = 0, off_count = 0, off_acc32 = 0, off_bpart = 0, bpart_rows = 0, off_zlo = 0, off_gaddr = 0, off_part = 0;
};

// The buffer the root term reads holds the destination rows only (n_dst[t] rows per type, back to back).
static void root_rows_only(Plan &pl) {
  int64_t o = 0;
  for (int t = 0; t < pl.tt.num_types; ++t) {
    pl.tt.xroot_off[t] = o;
    o += (int64_t)pl.tt.n_dst[t] * pl.tt.in_dim[t];
  }
  pl.tt.xroot_off[pl.tt.num_types] = o;
}

static hgnn_status make_plan(hgnn_ctx *ctx, hgnn_graph *g, int32_t layer, const hgnn_layer_params *p, Plan &pl,
                             bool need_built) {
  if (!ctx || !g || !p) HGNN_FAIL(HGNN_EINVAL, "NULL context, graph or parameters");
  if (layer < 0 || layer >= g->num_layers) HGNN_FAIL(HGNN_EINVAL, "layer %d outside [0,%d)", layer, g->num_layers);
  if (ctx->agg != HGNN_AGG_MEAN || ctx->fuse != HGNN_FUSE_SUM)
    HGNN_FAIL(HGNN_EUNSUPPORTED, "only mean aggregation with sum fusion is implemented");
  if (!p->in_dim || !p->w_rel || !p->w_root || p->out_dim <= 0) HGNN_FAIL(HGNN_EINVAL, "incomplete layer parameters");
  const int T = ctx->T, R = ctx->R;
  const LayerHost &L = g->L[layer];
  pl.es = esize(ctx->dtype);
  const int vec = 16 / pl.es;
  pl.H = p->out_dim;
  std::memset(&pl.tt, 0, sizeof(pl.tt));
  std::memset(&pl.rt, 0, sizeof(pl.rt));
  std::memset(&pl.pt, 0, sizeof(pl.pt));
  std::memset(&pl.wt, 0, sizeof(pl.wt));
  pl.tt.num_types = T;
  pl.rt.num_rels = R;
  int64_t eo = 0;
  for (int t = 0; t < T; ++t) {
    if (p->in_dim[t] <= 0 || p->in_dim[t] % vec != 0)
      HGNN_FAIL(HGNN_EUNSUPPORTED, "in_dim[%d]=%d is not a positive multiple of %d", t, p->in_dim[t], vec);
    pl.tt.in_dim[t] = p->in_dim[t];
    pl.tt.n_dst[t] = (int32_t)L.n_dst[t];
    pl.tt.elem_off[t] = eo;
    pl.tt.xroot_off[t] = eo;
    eo += L.n_src[t] * (int64_t)p->in_dim[t];
    pl.tt.row_off[t + 1] = pl.tt.row_off[t] + (int32_t)L.n_src[t];
    pl.tt.out_row_off[t + 1] = pl.tt.out_row_off[t] + (int32_t)L.n_dst[t];
    if (L.n_src[t] > 0) pl.max_dim = std::max(pl.max_dim, p->in_dim[t]);
    pl.pt.w_root[t] = p->w_root[t];
    pl.pt.bias[t] = p->bias ? p->bias[t] : nullptr;
  }
  pl.tt.elem_off[T] = eo;
  pl.tt.xroot_off[T] = eo;
  pl.total_dst = pl.tt.out_row_off[T];
  if ((int64_t)pl.total_dst * pl.H >= (int64_t)1 << 40) HGNN_FAIL(HGNN_EOVERFLOW, "output too large");
  size_t z = 0, w = 0;
  for (int r = 0; r < R; ++r) {
    const int s = ctx->rel_src[r], d = ctx->rel_dst[r];
    if (!p->w_rel[r]) HGNN_FAIL(HGNN_EINVAL, "w_rel[%d] is NULL", r);
    pl.rt.src[r] = (uint8_t)s;
    pl.rt.dst[r] = (uint8_t)d;
    pl.rt.z_off4[r] = (uint32_t)(z / 4);
    z += (size_t)L.n_dst[d] * p->in_dim[s];
    pl.pt.w_rel[r] = p->w_rel[r];
    pl.wt.rel4[r] = (uint32_t)(w / 4);
    w += (size_t)p->in_dim[s] * pl.H;
  }
  pl.rt.z_off4[R] = (uint32_t)(z / 4);
  pl.z_elems = z;
  size_t zr = z;
  for (int t = 0; t < T; ++t) {
    pl.rt.zroot_off4[t] = (uint32_t)(zr / 4);
    if (p->w_root[t]) zr += (size_t)L.n_dst[t] * p->in_dim[t];
    pl.wt.root4[t] = (uint32_t)(w / 4);
    if (p->w_root[t]) w += (size_t)p->in_dim[t] * pl.H;
  }
  pl.rt.zroot_off4[T] = (uint32_t)(zr / 4);
  pl.zroot_elems = zr - z;
  pl.wt_elems = w;
  if (zr / 4 >= ((size_t)1 << 32) || w / 4 >= ((size_t)1 << 32)) HGNN_FAIL(HGNN_EOVERFLOW, "work area too large");
  pl.saved_bytes = align_up(std::max<size_t>(z, 1) * pl.es, 256);
  size_t o = 0;
  const size_t Hpad = ((size_t)pl.H + vec - 1) / vec * vec;  // the backward pads H to whole 16-byte pieces when needed
  pl.off_wt = o;      o += align_up(std::max<size_t>(w / pl.H * Hpad, 1) * pl.es, 256);
  pl.off_gp = o;      o += align_up(std::max<size_t>((size_t)pl.total_dst * Hpad, 1) * pl.es, 256);
  pl.off_dz = o;      o += align_up(std::max<size_t>(zr, 1) * pl.es, 256);
  pl.off_partial = o; o += align_up(std::max<size_t>((size_t)long_partials(L.max_chunks) * std::max(pl.max_dim, 1), 1) * 4, 256);
  pl.off_count = o;   o += align_up((size_t)L.max_chunks * 4, 256);
  pl.off_acc32 = o;   o += align_up(std::max<size_t>((size_t)pl.total_dst * pl.H, 1) * 4, 256);
  // partial bias-gradient sums: one row of H floats per block of destination rows of a type (64 rows per block
  // when the row pass runs in its 16-bytes-per-lane form, which the width decides; 8 otherwise)
  const bool row_pass_vec = pl.H % vec == 0 && pl.H / vec <= 256;
  pl.bpart_rows = (size_t)pl.total_dst / (row_pass_vec ? 64 : 8) + T;
  pl.off_bpart = o;   o += align_up(pl.bpart_rows * pl.H * 4, 256);
  pl.off_zlo = o;     o += (pl.es == 2 && p->relu) ? align_up(std::max<size_t>(z, 1) * pl.es, 256) : 0;
  pl.off_gaddr = o;   o += align_up(std::max<size_t>((size_t)L.edges, 1) * 8, 256);  // per-edge row addresses (gather from the stores)
  int64_t tiles64 = 0;  // partial tiles of the forward's split reduction
  for (int t = 0; t < T; ++t) tiles64 += (L.n_dst[t] + 63) / 64 * ((pl.H + 63) / 64);
  pl.off_part = o;    o += tiles64 < (pl.es == 2 ? kDirectTiles / 4 : p->relu ? kDirectReluTiles : kDirectTiles) ? kDirectPartBytes : 0;
  pl.scratch_bytes = o;
  if (need_built) {
    hgnn_status st = layer_dev(ctx, g, layer, pl.dev);
    if (st != HGNN_OK) return st;
  }
  return HGNN_OK;
}

// Waits for the host build and fills the device-side view of one layer's index arrays.
hgnn_status layer_dev(hgnn_ctx *ctx, hgnn_graph *g, int32_t layer, LayerDev &D) {
  const LayerHost &L = g->L[layer];
  {
    hgnn_status st = wait_built(g);
    if (st != HGNN_OK) return st;
    if (ctx->device < 0) HGNN_FAIL(HGNN_EUNSUPPORTED, "host-only context cannot run device work");
    const int32_t *b = g->slab.dev;
    D.rel_row_off = b + L.o_rel_row_off; D.rel_edge_off = b + L.o_rel_edge_off;
    D.rowptr = b + L.o_rowptr; D.colidx = b + L.o_colidx; D.cptr = b + L.o_cptr; D.crow = b + L.o_crow;
    D.cperm = b + L.o_cperm;
    D.chunk_row = b + L.o_chunk_row; D.chunk_beg = b + L.o_chunk_beg;
    D.rows = (int32_t)L.rows; D.edges = (int32_t)L.edges; D.src_rows = (int32_t)L.src_rows;
    D.chunk_count = nullptr;
    D.n_chunks = L.n_chunks;
  }
  return HGNN_OK;
}

// While alive, the launches made on this thread are timed if the probe selects (kernel, layer).
static thread_local hgnn_ctx *tl_probe_ctx = nullptr;
static thread_local int tl_probe_slot = -1;
static thread_local bool tl_probe_first = false;

Probe::Probe(hgnn_ctx *c, int kernel, int layer, bool enabled) {
  int slot = -1;
  if (!enabled) return;
  for (int i = 0; i < c->probe_n; ++i)
    if (c->probe_sel[i][0] == kernel && (c->probe_sel[i][1] < 0 || c->probe_sel[i][1] == layer)) slot = i;
  if (slot < 0) return;
  tl_probe_ctx = c;
  tl_probe_slot = slot;
  tl_probe_first = true;
  active = true;
}
Probe::~Probe() {
  if (active) tl_probe_ctx = nullptr;
}

OptionalLaunchers &optional_launchers() {
  static OptionalLaunchers l;
  return l;
}
AttnVariant &attn_variant() {
  static AttnVariant v;
  return v;
}

bool probe_take_events(hipEvent_t *start, hipEvent_t *stop) {
  hgnn_ctx *c = tl_probe_ctx;
  if (!c) return false;
  if (c->probe_used == c->probe_events.size()) {
    hipEvent_t a, b;
    if (hipEventCreate(&a) != hipSuccess) return false;
    if (hipEventCreate(&b) != hipSuccess) { (void)hipEventDestroy(a); return false; }
    c->probe_events.emplace_back(a, b);
  }
  c->probe_slot.resize(c->probe_events.size());
  c->probe_first.resize(c->probe_events.size());
  c->probe_slot[c->probe_used] = tl_probe_slot;
  c->probe_first[c->probe_used] = tl_probe_first ? 1 : 0;
  tl_probe_first = false;
  auto &pr = c->probe_events[c->probe_used++];
  *start = pr.first;
  *stop = pr.second;
  return true;
}

// Tile table of the forward GEMM; returns the tile edge (128 or 64).
static int fwd_tiles(const Plan &pl, SegTab &tl, bool relu, bool allow_small) {
  const int T = pl.tt.num_types;
  for (int mn = 128;; mn = 64) {
    std::memset(&tl, 0, sizeof(tl));
    const int tn = (pl.H + mn - 1) / mn;
    for (int t = 0; t < T; ++t) tl.tile_off[t + 1] = tl.tile_off[t] + ((pl.tt.n_dst[t] + mn - 1) / mn) * tn;
    tl.num_segs = T;
    if (mn == 64 || !allow_small || !fwd_small_tiles(pl.es == 2 ? HGNN_BF16 : HGNN_F32, pl.H, relu, tl.tile_off[T])) return mn;
  }
}

}  // namespace hgnn

using namespace hgnn;

extern "C" {

const char *hgnn_last_error(void) { return hgnn::get_error(); }

hgnn_status hgnn_create(hgnn_ctx **out, const hgnn_schema *s, int device, int host_threads, int concurrent_builds) {
  if (!out || !s || !s->rel_src_type || !s->rel_dst_type) HGNN_FAIL(HGNN_EINVAL, "NULL argument");
  *out = nullptr;
  if (s->num_types < 1 || s->num_types > kMaxT) HGNN_FAIL(HGNN_EINVAL, "num_types %d outside [1,%d]", s->num_types, kMaxT);
  if (s->num_rels < 1 || s->num_rels > kMaxR) HGNN_FAIL(HGNN_EINVAL, "num_rels %d outside [1,%d]", s->num_rels, kMaxR);
  if (s->dtype != HGNN_F32 && s->dtype != HGNN_BF16) HGNN_FAIL(HGNN_EINVAL, "unknown dtype %d", s->dtype);
  for (int r = 0; r < s->num_rels; ++r)
    if (s->rel_src_type[r] < 0 || s->rel_src_type[r] >= s->num_types || s->rel_dst_type[r] < 0 ||
        s->rel_dst_type[r] >= s->num_types)
      HGNN_FAIL(HGNN_EINVAL, "relation %d has a vertex type outside [0,%d)", r, s->num_types);
  hgnn_ctx *c = new (std::nothrow) hgnn_ctx();
  if (!c) HGNN_FAIL(HGNN_ENOMEM, "out of host memory");
  c->device = device;
  c->T = s->num_types;
  c->R = s->num_rels;
  for (int r = 0; r < c->R; ++r) {
    c->rel_src[r] = s->rel_src_type[r];
    c->rel_dst[r] = s->rel_dst_type[r];
  }
  c->heads = s->heads < 1 ? 1 : s->heads;
  c->agg = s->agg;
  c->fuse = s->fuse;
  c->dtype = s->dtype;
  c->legacy_gemm = getenv("HGNN_DMA_GEMM") == nullptr;
  if (device >= 0) {
    hipError_t e = hipSetDevice(device);
    if (e == hipSuccess) e = hipStreamCreateWithFlags(&c->side, hipStreamNonBlocking);
    if (e != hipSuccess) {
      delete c;
      HGNN_FAIL(HGNN_EHIP, "device %d: %s", device, hipGetErrorString(e));
    }
    const hgnn_status sst = static_scratch_init(device);  // where this device keeps hgnn_layer_fwd_static's work area
    if (sst != HGNN_OK) {
      (void)hipStreamDestroy(c->side);
      delete c;
      return sst;
    }
  }
  int n = host_threads;
  if (n <= 0) {
    long on = sysconf(_SC_NPROCESSORS_ONLN);
    n = (int)std::min<long>(16, std::max<long>(1, on));
  }
  // Graphs are independent, so several are built at once.  Few at a time finish one build soonest (the other threads take
  // part in its phases); one per host thread gives the most builds per second (no barriers between the phases of a
  // build), which is what a caller that queues many mini-batches ahead wants.  One of the n threads is the caller's own.
  const int nb = concurrent_builds > 0 ? std::min(n, concurrent_builds) : std::max(1, std::min(4, n / 4));
  c->pool.reset(new ThreadPool(n - nb + 1));
  for (int i = 0; i < nb; ++i) {
    c->builders.emplace_back(new Builder());
    c->builders.back()->pool = c->pool.get();
    c->idle_builders.push_back(c->builders.back().get());
  }
  c->crew_threads = std::max(nb, n - 1);
  c->crew = &Crew::get();
  c->crew->join(c->crew_threads, c->pool->size() > 1);
  *out = c;
  return HGNN_OK;
}

void hgnn_destroy(hgnn_ctx *c) {
  if (!c) return;
  if (c->crew == &Crew::get()) {   // else: inherited through a fork, whose child has none of its threads
    {
      std::unique_lock<std::mutex> lk(c->qm);
      c->qcv.wait(lk, [&] { return c->building == 0; });   // queued builds are finished
    }
    c->crew->leave(c->crew_threads, c->pool->size() > 1);
  }
  if (c->device >= 0) {
    (void)hipSetDevice(c->device);
    (void)hipStreamSynchronize(c->side);
  }
  for (auto &s : c->free_slabs) free_slab(c, s);
  for (auto e : c->free_events) (void)hipEventDestroy(e);
  for (auto &pr : c->probe_events) {
    (void)hipEventDestroy(pr.first);
    (void)hipEventDestroy(pr.second);
  }
  if (c->side) (void)hipStreamDestroy(c->side);
  if (c->dev_tmp) (void)hipFree(c->dev_tmp);
  if (c->dev_types8) (void)hipFree(c->dev_types8);
  delete c;
}

hgnn_status hgnn_merge_features(hgnn_ctx *ctx, void *stream, const void *const *store, const int32_t *feat_dim,
                                const int64_t *const *ids, const int64_t *n_rows, void *x_merged, int32_t *row_off,
                                int64_t *elem_off) {
  if (!ctx || !store || !feat_dim || !ids || !n_rows || !row_off || !elem_off) HGNN_FAIL(HGNN_EINVAL, "NULL argument");
  const int T = ctx->T, vec = 16 / esize(ctx->dtype);
  int64_t ro = 0, eo = 0;
  int64_t tmp_eo[kMaxT + 1];
  int32_t tmp_ro[kMaxT + 1];
  for (int t = 0; t < T; ++t) {
    if (n_rows[t] < 0) HGNN_FAIL(HGNN_EINVAL, "n_rows[%d] is negative", t);
    if (feat_dim[t] <= 0 || feat_dim[t] % vec != 0)
      HGNN_FAIL(HGNN_EINVAL, "feat_dim[%d]=%d is not a positive multiple of %d", t, feat_dim[t], vec);
    if (n_rows[t] > 0 && (!store[t] || !ids[t])) HGNN_FAIL(HGNN_EINVAL, "type %d has rows but a NULL store or id list", t);
    tmp_ro[t] = (int32_t)ro;
    tmp_eo[t] = eo;
    ro += n_rows[t];
    eo += n_rows[t] * (int64_t)feat_dim[t];
    if (ro > INT32_MAX) HGNN_FAIL(HGNN_EOVERFLOW, "more than 2^31-1 merged rows");
  }
  tmp_ro[T] = (int32_t)ro;
  tmp_eo[T] = eo;
  if (ro > 0 && !x_merged) HGNN_FAIL(HGNN_EINVAL, "x_merged is NULL");
  if (ctx->device < 0) HGNN_FAIL(HGNN_EUNSUPPORTED, "host-only context cannot run device work");
  hgnn_status st;
  {
    Probe pb(ctx, HGNN_K_MERGE, -1);
    st = launch_merge((hipStream_t)stream, ctx->dtype, T, store, feat_dim, ids, n_rows, tmp_eo, x_merged);
  }
  if (st != HGNN_OK) return st;
  std::memcpy(row_off, tmp_ro, sizeof(int32_t) * (T + 1));
  std::memcpy(elem_off, tmp_eo, sizeof(int64_t) * (T + 1));
  return HGNN_OK;
}

// The two halves of the index-first baseline: offsets as hgnn_merge_features computes them, one width for all types.
static hgnn_status index_first_common(hgnn_ctx *ctx, const int32_t *feat_dim, const int64_t *n_rows, const int32_t *const *pos,
                                      int64_t *tmp_eo, int32_t *tmp_ro) {
  const int T = ctx->T, vec = 16 / esize(ctx->dtype);
  int64_t ro = 0, eo = 0;
  for (int t = 0; t < T; ++t) {
    if (n_rows[t] < 0) HGNN_FAIL(HGNN_EINVAL, "n_rows[%d] is negative", t);
    if (feat_dim[t] <= 0 || feat_dim[t] % vec != 0)
      HGNN_FAIL(HGNN_EINVAL, "feat_dim[%d]=%d is not a positive multiple of %d", t, feat_dim[t], vec);
    if (feat_dim[t] != feat_dim[0]) HGNN_FAIL(HGNN_EUNSUPPORTED, "an interleaved buffer needs one width for all types");
    if (n_rows[t] > 0 && !pos[t]) HGNN_FAIL(HGNN_EINVAL, "type %d has rows but a NULL position list", t);
    tmp_ro[t] = (int32_t)ro;
    tmp_eo[t] = eo;
    ro += n_rows[t];
    eo += n_rows[t] * (int64_t)feat_dim[t];
    if (ro > INT32_MAX) HGNN_FAIL(HGNN_EOVERFLOW, "more than 2^31-1 merged rows");
  }
  tmp_ro[T] = (int32_t)ro;
  tmp_eo[T] = eo;
  if (ctx->device < 0) HGNN_FAIL(HGNN_EUNSUPPORTED, "host-only context cannot run device work");
  return HGNN_OK;
}

hgnn_status hgnn_merge_features_index_first(hgnn_ctx *ctx, void *stream, const void *const *store, const int32_t *feat_dim,
                                            const int64_t *const *ids, const int64_t *n_rows, const int32_t *const *pos,
                                            void *x_interleaved) {
  if (!ctx || !store || !feat_dim || !ids || !n_rows || !pos) HGNN_FAIL(HGNN_EINVAL, "NULL argument");
  int64_t tmp_eo[kMaxT + 1];
  int32_t tmp_ro[kMaxT + 1];
  hgnn_status st = index_first_common(ctx, feat_dim, n_rows, pos, tmp_eo, tmp_ro);
  if (st != HGNN_OK) return st;
  for (int t = 0; t < ctx->T; ++t)
    if (n_rows[t] > 0 && (!store[t] || !ids[t])) HGNN_FAIL(HGNN_EINVAL, "type %d has rows but a NULL store or id list", t);
  if (tmp_ro[ctx->T] > 0 && !x_interleaved) HGNN_FAIL(HGNN_EINVAL, "x_interleaved is NULL");
  Probe pb(ctx, HGNN_K_MERGE, -1);
  return launch_merge((hipStream_t)stream, ctx->dtype, ctx->T, store, feat_dim, ids, n_rows, tmp_eo, x_interleaved, 1, pos, nullptr);
}

hgnn_status hgnn_select_type_first(hgnn_ctx *ctx, void *stream, const void *x_interleaved, const int32_t *feat_dim,
                                   const int32_t *const *pos, const int64_t *n_rows, void *x_merged, int32_t *row_off,
                                   int64_t *elem_off) {
  if (!ctx || !feat_dim || !pos || !n_rows || !row_off || !elem_off) HGNN_FAIL(HGNN_EINVAL, "NULL argument");
  int64_t tmp_eo[kMaxT + 1];
  int32_t tmp_ro[kMaxT + 1];
  hgnn_status st = index_first_common(ctx, feat_dim, n_rows, pos, tmp_eo, tmp_ro);
  if (st != HGNN_OK) return st;
  if (tmp_ro[ctx->T] > 0 && (!x_interleaved || !x_merged)) HGNN_FAIL(HGNN_EINVAL, "NULL buffer");
  {
    Probe pb(ctx, HGNN_K_MERGE, -1);
    st = launch_merge((hipStream_t)stream, ctx->dtype, ctx->T, nullptr, feat_dim, nullptr, n_rows, tmp_eo, x_merged, 2, pos, x_interleaved);
  }
  if (st != HGNN_OK) return st;
  std::memcpy(row_off, tmp_ro, sizeof(int32_t) * (ctx->T + 1));
  std::memcpy(elem_off, tmp_eo, sizeof(int64_t) * (ctx->T + 1));
  return HGNN_OK;
}

extern "C++" {
namespace hgnn {
constexpr size_t kMaxTypeRuns = 32;
void index_edge_type_runs(hgnn_ctx *ctx) {
  ctx->run_end.clear();
  ctx->run_rel.clear();
  const std::vector<uint8_t> &t = ctx->edge_types8;
  for (size_t i = 0; i < t.size(); ++i)
    if (i + 1 == t.size() || t[i + 1] != t[i]) {
      ctx->run_end.push_back((int64_t)i + 1);
      ctx->run_rel.push_back(t[i]);
      if (ctx->run_end.size() > kMaxTypeRuns) {  // not grouped by relation: the byte table it is
        ctx->run_end.clear();
        ctx->run_rel.clear();
        return;
      }
    }
  ctx->run_shift = 0;
  while ((t.size() >> ctx->run_shift) > 1024) ++ctx->run_shift;
  ctx->run_lut.assign((t.size() >> ctx->run_shift) + 1, 0);
  for (size_t b = 0, j = 0; b < ctx->run_lut.size(); ++b) {
    while (j + 1 < ctx->run_end.size() && (int64_t)(b << ctx->run_shift) >= ctx->run_end[j]) ++j;
    ctx->run_lut[b] = (uint8_t)j;
  }
}

// Validates the layers' inputs (g->L[l].in), lays the index arrays out in one block and takes a pinned/device
// block and an event from the context's pool (or allocates them).  Runs on the caller's thread for
// hgnn_build_semantic_csr and on a builder's thread for sampled mini-batches, hence the message by reference.
hgnn_status plan_graph(hgnn_ctx *ctx, hgnn_graph *g, std::string &msg) {
  const int T = ctx->T, R = ctx->R, num_layers = g->num_layers;
  g->with_perm = ctx->build_perm || ctx->agg == HGNN_AGG_ATTN;  // the attention backward walks cperm
  char buf[256];
  auto fail = [&](hgnn_status st, const char *fmt, auto... a) {
    std::snprintf(buf, sizeof(buf), fmt, a...);
    msg = buf;
    return st;
  };
  size_t o = 0;
  auto take = [&](size_t n) {
    size_t at = o;
    o += (n + 63) / 64 * 64;  // keep every array 256-byte aligned
    return at;
  };
  for (int l = 0; l < num_layers; ++l) {
    LayerHost &L = g->L[l];
    const hgnn_coo_layer &in = L.in;
    if (in.num_edges < 0 || !in.n_src || !in.n_dst) return fail(HGNN_EINVAL, "layer %d: bad edge count or NULL n_src/n_dst", l);
    if (in.num_edges > 0 && !in.edge_type && in.edge_id && !in.global_edge_type && ctx->edge_types8.empty())
      return fail(HGNN_EINVAL, "layer %d: edge_id without a global edge-type table (none given, none registered)", l);
    if (in.num_edges > 0 && (!in.edge_index || (!in.edge_type && !in.edge_id))) return fail(HGNN_EINVAL, "layer %d: NULL edge arrays", l);
    if (in.num_edges > INT32_MAX) return fail(HGNN_EOVERFLOW, "layer %d: more than 2^31-1 edges", l);
    L.edges = in.num_edges;
    int64_t src_rows = 0, rows = 0;
    for (int t = 0; t < T; ++t) {
      if (in.n_src[t] < 0 || in.n_dst[t] < 0 || in.n_dst[t] > in.n_src[t])
        return fail(HGNN_EINVAL, "layer %d: type %d has n_dst=%lld, n_src=%lld (need 0 <= n_dst <= n_src)", l, t,
                    (long long)in.n_dst[t], (long long)in.n_src[t]);
      L.n_src[t] = in.n_src[t];
      L.n_dst[t] = in.n_dst[t];
      if (in.transpose_types && !in.transpose_types[t]) L.tmask &= ~(1u << t);
      src_rows += in.n_src[t];
    }
    for (int r = 0; r < R; ++r) rows += in.n_dst[ctx->rel_dst[r]];
    if (src_rows > INT32_MAX - 1 || rows > INT32_MAX - 1) return fail(HGNN_EOVERFLOW, "layer %d: more than 2^31-2 rows", l);
    L.rows = rows;
    L.src_rows = src_rows;
    L.max_chunks = (int32_t)(L.edges / kChunk + L.edges / (kLongRow + 1) + 1);   // whole ones, and a last one per long row
    L.o_rel_row_off = take(R + 1);
    L.o_rel_edge_off = take(R + 1);
    L.o_rowptr = take(rows + 1);
    L.o_colidx = take(L.edges);
    L.o_cptr = take(src_rows + 1);
    L.o_crow = take(L.edges);
    L.o_chunk_row = take(L.max_chunks);
    L.o_chunk_beg = take(L.max_chunks);
  }
  const bool cperm_on_device = ctx->agg == HGNN_AGG_ATTN;   // the attention backward walks edges by CSR position
  if (cperm_on_device)
    for (int l = 0; l < num_layers; ++l) g->L[l].o_cperm = take(g->L[l].edges);
  if (g->job)  // a sampled mini-batch carries the global ids of its first layer's source rows (int64)
    for (int t = 0; t < T; ++t) g->o_ids[t] = take(2 * g->job->ids[t].size());
  const size_t dev_used = o;  // arrays below stay on the host (views only)
  for (int l = 0; l < num_layers; ++l) {
    g->L[l].o_perm = take(g->L[l].edges);
    if (!cperm_on_device) g->L[l].o_cperm = take(g->L[l].edges);
  }
  g->used = dev_used;
  const size_t need = std::max<size_t>(o, 64);
  // a pooled slab (with its two events) or a new one
  {
    std::lock_guard<std::mutex> lk(ctx->pm);
    for (size_t i = 0; i < ctx->free_slabs.size(); ++i)
      if (ctx->free_slabs[i].cap >= need) {
        g->slab = ctx->free_slabs[i];
        ctx->free_slabs.erase(ctx->free_slabs.begin() + i);
        break;
      }
    if (!g->slab.host && !ctx->free_slabs.empty()) {  // too small: drop one so the pool does not grow forever
      free_slab(ctx, ctx->free_slabs.back());
      ctx->free_slabs.pop_back();
    }
    if (!ctx->free_events.empty()) {
      g->ready = ctx->free_events.back();
      ctx->free_events.pop_back();
    }
  }
  if (!g->slab.host) {
    const size_t cap = need + need / 4;
    if (ctx->device >= 0) {
      (void)hipSetDevice(ctx->device);
      hipError_t e = hipHostMalloc((void **)&g->slab.host, cap * sizeof(int32_t), hipHostMallocDefault);
      if (e == hipSuccess) e = hipMalloc((void **)&g->slab.dev, cap * sizeof(int32_t));
      if (e != hipSuccess) {
        free_slab(ctx, g->slab);
        g->slab = Slab();
        return fail(HGNN_ENOMEM, "graph buffers (%zu bytes): %s", cap * sizeof(int32_t), hipGetErrorString(e));
      }
    } else {
      g->slab.host = (int32_t *)malloc(cap * sizeof(int32_t));
      if (!g->slab.host) return fail(HGNN_ENOMEM, "out of host memory (%zu bytes)", cap * sizeof(int32_t));
    }
    g->slab.cap = cap;
  }
  if (ctx->device >= 0 && !g->ready) {
    hipError_t e = hipEventCreateWithFlags(&g->ready, hipEventDisableTiming);
    if (e != hipSuccess) return fail(HGNN_EHIP, "hipEventCreate: %s", hipGetErrorString(e));
  }
  return HGNN_OK;
}
}  // namespace hgnn
}  // extern "C++"

// Hands a planned (or to-be-sampled) graph to the builders.
static void enqueue_graph(hgnn_ctx *ctx, hgnn_graph *g) {
  bool start = false;
  {
    std::lock_guard<std::mutex> lk(ctx->qm);
    ctx->queue.push_back(g);
    if (ctx->building < (int)ctx->builders.size()) {
      ++ctx->building;
      start = true;
    }
  }
  if (start) Crew::get().submit([ctx] { build_queued(ctx); });
}

// Gives back whatever plan_graph took and deletes the graph (error paths before the graph reaches a builder).
static void drop_graph(hgnn_ctx *ctx, hgnn_graph *g) {
  {
    std::lock_guard<std::mutex> lk(ctx->pm);
    if (g->slab.host) ctx->free_slabs.push_back(g->slab);
    if (g->ready) ctx->free_events.push_back(g->ready);
  }
  delete g;
}

hgnn_status hgnn_build_semantic_csr(hgnn_ctx *ctx, int32_t num_layers, const hgnn_coo_layer *layers, hgnn_graph **out) {
  if (!ctx || !layers || !out) HGNN_FAIL(HGNN_EINVAL, "NULL argument");
  *out = nullptr;
  if (num_layers < 1 || num_layers > kMaxLayers) HGNN_FAIL(HGNN_EINVAL, "num_layers %d outside [1,%d]", num_layers, kMaxLayers);
  hgnn_graph *g = new (std::nothrow) hgnn_graph();
  if (!g) HGNN_FAIL(HGNN_ENOMEM, "out of host memory");
  g->num_layers = num_layers;
  for (int l = 0; l < num_layers; ++l) g->L[l].in = layers[l];
  std::string msg;
  const hgnn_status st = plan_graph(ctx, g, msg);
  if (st != HGNN_OK) {
    drop_graph(ctx, g);
    HGNN_FAIL(st, "%s", msg.c_str());
  }
  enqueue_graph(ctx, g);
  *out = g;
  return HGNN_OK;
}

hgnn_status hgnn_sample_and_build(hgnn_ctx *ctx, const hgnn_sampler *sm, int32_t target_type, const int64_t *targets,
                                  int64_t num_targets, int32_t num_layers, const int32_t *fanouts, uint64_t seed,
                                  const int32_t *const *transpose_types, hgnn_graph **out) {
  if (!ctx || !sm || !fanouts || !out || num_targets < 0 || (num_targets > 0 && !targets)) HGNN_FAIL(HGNN_EINVAL, "NULL argument");
  *out = nullptr;
  if (num_layers < 1 || num_layers > kMaxLayers) HGNN_FAIL(HGNN_EINVAL, "num_layers %d outside [1,%d]", num_layers, kMaxLayers);
  if (target_type < 0 || target_type >= ctx->T) HGNN_FAIL(HGNN_EINVAL, "target_type %d outside [0,%d)", target_type, ctx->T);
  for (int h = 0; h < num_layers; ++h)
    if (fanouts[h] < 1 || fanouts[h] > 64) HGNN_FAIL(HGNN_EINVAL, "fanouts[%d]=%d outside [1,64]", h, fanouts[h]);
  for (int64_t i = 0; i < num_targets; ++i)
    if (targets[i] < 0 || targets[i] >= sm->num_nodes[target_type])
      HGNN_FAIL(HGNN_EINVAL, "targets[%lld]=%lld is not a vertex of type %d", (long long)i, (long long)targets[i], target_type);
  hgnn_graph *g = new (std::nothrow) hgnn_graph();
  if (!g) HGNN_FAIL(HGNN_ENOMEM, "out of host memory");
  g->num_layers = num_layers;
  {
    std::lock_guard<std::mutex> lk(ctx->pm);
    if (!ctx->free_jobs.empty()) {
      g->job = std::move(ctx->free_jobs.back());
      ctx->free_jobs.pop_back();
    }
  }
  if (!g->job) g->job.reset(new SampleJob());
  SampleJob &job = *g->job;
  for (int l = 0; l < kMaxLayers; ++l) job.transpose[l].clear();
  job.sampler = sm;
  job.target_type = target_type;
  job.seed = seed;
  job.targets.assign(targets, targets + num_targets);
  job.fanouts.assign(fanouts, fanouts + num_layers);
  if (transpose_types)
    for (int l = 0; l < num_layers; ++l)
      if (transpose_types[l]) job.transpose[l].assign(transpose_types[l], transpose_types[l] + ctx->T);
  enqueue_graph(ctx, g);
  *out = g;
  return HGNN_OK;
}

hgnn_status hgnn_graph_ids(hgnn_ctx *ctx, hgnn_graph *g, int64_t *n_rows, const int64_t **host_ids, const int64_t **device_ids) {
  if (!ctx || !g) HGNN_FAIL(HGNN_EINVAL, "NULL argument");
  if (!g->job) HGNN_FAIL(HGNN_EINVAL, "the graph was not made by hgnn_sample_and_build");
  if (device_ids) look_built(g);
  {
    std::unique_lock<std::mutex> lk(g->m);
    g->cv.wait(lk, [&] { return g->sampled || g->state != 0; });
    if (!g->sampled) HGNN_FAIL((hgnn_status)g->status, "%s", g->err.c_str());
  }
  if (device_ids) {  // their place in the block is fixed by the plan that follows the sampling
    std::unique_lock<std::mutex> lk(g->m);
    g->cv.wait(lk, [&] { return g->state != 0; });
    if (g->state != 1) HGNN_FAIL((hgnn_status)g->status, "%s", g->err.c_str());
  }
  for (int t = 0; t < ctx->T; ++t) {
    const size_t n = g->job->ids[t].size();
    if (n_rows) n_rows[t] = (int64_t)n;
    if (host_ids) host_ids[t] = n ? g->job->ids[t].data() : nullptr;
    if (device_ids) device_ids[t] = (n && g->slab.dev) ? reinterpret_cast<const int64_t *>(g->slab.dev + g->o_ids[t]) : nullptr;
  }
  return HGNN_OK;
}

hgnn_status hgnn_graph_minibatch_view(hgnn_ctx *ctx, hgnn_graph *g, int32_t layer, hgnn_minibatch_view *view) {
  if (!ctx || !g || !view) HGNN_FAIL(HGNN_EINVAL, "NULL argument");
  if (!g->job) HGNN_FAIL(HGNN_EINVAL, "the graph was not made by hgnn_sample_and_build");
  if (layer < 0 || layer >= g->num_layers) HGNN_FAIL(HGNN_EINVAL, "layer %d outside [0,%d)", layer, g->num_layers);
  const hgnn_status st = wait_built(g);   // host arrays: nothing to wait for on the device
  if (st != HGNN_OK) return st;
  std::memset(view, 0, sizeof(*view));
  for (int t = 0; t < ctx->T; ++t) {
    view->n_src[t] = g->job->n_src[layer][t];
    view->n_dst[t] = g->job->n_dst[layer][t];
  }
  view->num_edges = (int64_t)g->job->edge_id[layer].size();
  view->edge_index = g->job->edge_index[layer].data();
  view->edge_id = g->job->edge_id[layer].data();
  return HGNN_OK;
}

hgnn_status hgnn_graph_wait_stream(hgnn_ctx *ctx, hgnn_graph *g, void *stream) {
  if (!ctx || !g) HGNN_FAIL(HGNN_EINVAL, "NULL argument");
  if (ctx->device < 0) HGNN_FAIL(HGNN_EUNSUPPORTED, "host-only context cannot run device work");
  {
    std::unique_lock<std::mutex> lk(g->m);
    g->cv.wait(lk, [&] { return g->state != 0; });
    if (g->state != 1) HGNN_FAIL((hgnn_status)g->status, "%s", g->err.c_str());
  }
  HGNN_HIP(wait_upload(g, (hipStream_t)stream));
  return HGNN_OK;
}

hgnn_status hgnn_set_edge_types(hgnn_ctx *ctx, const int32_t *global_edge_type, int64_t num_global_edges) {
  if (!ctx || num_global_edges < 0 || (num_global_edges > 0 && !global_edge_type)) HGNN_FAIL(HGNN_EINVAL, "NULL argument");
  std::vector<uint8_t> t((size_t)num_global_edges);
  for (int64_t i = 0; i < num_global_edges; ++i) {
    const int32_t r = global_edge_type[i];
    if (r < 0 || r >= ctx->R) HGNN_FAIL(HGNN_EINVAL, "global_edge_type[%lld]=%d outside [0,%d)", (long long)i, r, ctx->R);
    t[(size_t)i] = (uint8_t)r;
  }
  ctx->edge_types8.swap(t);
  ++ctx->types_version;
  index_edge_type_runs(ctx);
  return HGNN_OK;
}

hgnn_status hgnn_set_build_permutation(hgnn_ctx *ctx, int32_t enabled) {
  if (!ctx) HGNN_FAIL(HGNN_EINVAL, "NULL context");
  ctx->build_perm = enabled != 0;
  return HGNN_OK;
}

hgnn_status hgnn_graph_wait(hgnn_ctx *ctx, hgnn_graph *g) {
  if (!ctx || !g) HGNN_FAIL(HGNN_EINVAL, "NULL argument");
  hgnn_status st = wait_built(g);
  if (st != HGNN_OK) return st;
  if (ctx->device >= 0 && !g->uploaded.load(std::memory_order_acquire)) {
    HGNN_HIP(hipEventSynchronize(g->ready));
    g->uploaded.store(true, std::memory_order_release);
  }
  return HGNN_OK;
}

hgnn_status hgnn_graph_host_view(hgnn_ctx *ctx, hgnn_graph *g, int32_t layer, hgnn_csr_view *v) {
  if (!ctx || !g || !v) HGNN_FAIL(HGNN_EINVAL, "NULL argument");
  if (layer < 0 || layer >= g->num_layers) HGNN_FAIL(HGNN_EINVAL, "layer %d outside [0,%d)", layer, g->num_layers);
  hgnn_status st = wait_built(g);
  if (st != HGNN_OK) return st;
  const LayerHost &L = g->L[layer];
  const int32_t *b = g->slab.host;
  v->rows = L.rows; v->edges = L.edges; v->src_rows = L.src_rows; v->transpose_edges = L.tedges;
  v->rel_row_off = b + L.o_rel_row_off; v->rel_edge_off = b + L.o_rel_edge_off;
  v->rowptr = b + L.o_rowptr; v->colidx = b + L.o_colidx; v->perm = g->with_perm ? b + L.o_perm : nullptr;
  v->cptr = b + L.o_cptr; v->crow = b + L.o_crow; v->cperm = g->with_perm ? b + L.o_cperm : nullptr;
  return HGNN_OK;
}

void hgnn_graph_release(hgnn_ctx *ctx, hgnn_graph *g) {
  if (!ctx || !g) return;
  {
    std::unique_lock<std::mutex> lk(g->m);
    g->cv.wait(lk, [&] { return g->state != 0; });
  }
  // the pinned block is rewritten by the next build: its upload must have left it
  if (ctx->device >= 0 && g->state == 1) (void)hipEventSynchronize(g->ready);
  {
    std::lock_guard<std::mutex> lk(ctx->pm);
    if (g->slab.host) ctx->free_slabs.push_back(g->slab);
    if (g->ready) ctx->free_events.push_back(g->ready);
    if (g->job && ctx->free_jobs.size() < 64) ctx->free_jobs.push_back(std::move(g->job));
  }
  delete g;
}

hgnn_status hgnn_layer_workspace_bytes(hgnn_ctx *ctx, hgnn_graph *g, int32_t layer, const hgnn_layer_params *p,
                                       size_t *saved_bytes, size_t *scratch_bytes) {
  if (ctx && ctx->agg == HGNN_AGG_ATTN) {
    return attn_variant().workspace(ctx, g, layer, p, saved_bytes, scratch_bytes);
  }
  Plan pl;
  hgnn_status st = make_plan(ctx, g, layer, p, pl, false);
  if (st != HGNN_OK) return st;
  if (saved_bytes) *saved_bytes = pl.saved_bytes;
  if (scratch_bytes) *scratch_bytes = pl.scratch_bytes;
  return HGNN_OK;
}

// Whether there is an aggregation launch (which carries the weight transposes as its first or last blocks).
static bool transposes_ride(const Plan &pl) { return pl.dev.rows > 0; }

// Bit r: relation r has an edge in the layer.
static void live_relations(const hgnn_ctx *ctx, const hgnn_graph *g, int32_t layer, uint32_t (&live)[kMaxR / 32]) {
  std::memset(live, 0, sizeof(live));
  const int32_t *reo = g->slab.host + g->L[layer].o_rel_edge_off;
  for (int r = 0; r < ctx->R; ++r)
    if (reo[r + 1] > reo[r]) live[r >> 5] |= 1u << (r & 31);
}

static hgnn_status fwd_common(hgnn_ctx *ctx, void *stream, hgnn_graph *g, int32_t layer, const hgnn_layer_params *p,
                              const void *x, void *h, void *saved, size_t saved_bytes, void *scratch, size_t scratch_bytes,
                              bool naive, int32_t *launches, void *feature_cat = nullptr, size_t feature_cat_bytes = 0,
                              bool static_area = false, const void *const *gather_store = nullptr,
                              const int64_t *const *gather_ids = nullptr) {
  Plan pl;
  hgnn_status st = make_plan(ctx, g, layer, p, pl, true);
  if (st != HGNN_OK) return st;
  if (pl.total_dst > 0 && (!x || !h)) HGNN_FAIL(HGNN_EINVAL, "x_merged or h_out is NULL");
  GatherSrc gs;
  if (gather_store) {
    // source rows are read where they live: x holds the destination rows only
    std::memset(&gs, 0, sizeof(gs));
    gs.num_types = ctx->T;
    for (int t = 0; t < ctx->T; ++t) {
      if (p->in_dim[t] != p->in_dim[0]) HGNN_FAIL(HGNN_EUNSUPPORTED, "gathering from the stores needs one input width for all types");
      gs.row_off[t + 1] = pl.tt.row_off[t + 1];
      if (g->L[layer].n_src[t] > 0 && (!gather_store[t] || !gather_ids || !gather_ids[t]))
        HGNN_FAIL(HGNN_EINVAL, "type %d has source rows but a NULL store or id list", t);
      if ((uintptr_t)gather_store[t] & 15) HGNN_FAIL(HGNN_EINVAL, "feature stores must be 16-byte aligned");
      gs.store[t] = gather_store[t];
      gs.ids[t] = gather_ids[t];
    }
    root_rows_only(pl);
  }
  if (!saved || !scratch) HGNN_FAIL(HGNN_EINVAL, "NULL work area");
  if (static_area) {
    // the forward's own part of the work area, laid out back to back: transposed weights, low-order plane
    const size_t wt_bytes = pl.off_gp - pl.off_wt, zlo_bytes = pl.off_gaddr - pl.off_zlo;
    if (wt_bytes + zlo_bytes > scratch_bytes)
      HGNN_FAIL(HGNN_EINVAL, "layer needs %zu bytes of work area, the static one holds %zu: use hgnn_layer_fwd with a caller-provided area",
                wt_bytes + zlo_bytes, scratch_bytes);
    pl.off_wt = 0;
    pl.off_zlo = wt_bytes;
    pl.scratch_bytes = wt_bytes + zlo_bytes;
    pl.off_part = scratch_bytes;   // behind the area (noalloc.hip)
  }
  if (saved_bytes < pl.saved_bytes || scratch_bytes < pl.scratch_bytes)
    HGNN_FAIL(HGNN_EINVAL, "work areas too small: need %zu saved, %zu scratch bytes", pl.saved_bytes, pl.scratch_bytes);
  if (((uintptr_t)saved | (uintptr_t)scratch | (uintptr_t)x | (uintptr_t)h) & 15)
    HGNN_FAIL(HGNN_EINVAL, "device buffers must be 16-byte aligned");
  hipStream_t s = (hipStream_t)stream;
  HGNN_HIP(wait_upload(g, s));
  char *sc = (char *)scratch;
  void *wtb = sc + pl.off_wt;
  // bf16 storage, layer with an activation: the aggregate is kept as a pair (rounded value, remainder), so that the
  // pre-activation -- and with it the decision of every unit, which the backward pass depends on discontinuously --
  // does not carry the rounding of the aggregate to 8 significant bits
  void *zlo = (ctx->dtype == HGNN_BF16 && p->relu) ? sc + pl.off_zlo : nullptr;
  int n = 0;
  SegTab tl;
  const int tile_mn = fwd_tiles(pl, tl, p->relu != 0, !naive);
  const int R = ctx->R, T = ctx->T;
  uint32_t live[kMaxR / 32];
  live_relations(ctx, g, layer, live);
  // The weight transposes ride in the aggregation launch (JobSplit) where there is one; otherwise they are a launch of
  // their own.
  // A relation without edges takes no part in the products: no tile reads its weight.
  TransposeJobs tj;
  PtrTab used = pl.pt;
  for (int r = 0; r < R; ++r)
    if (!((live[r >> 5] >> (r & 31)) & 1u)) used.w_rel[r] = nullptr;
  make_transpose_jobs(pl.tt, pl.rt, used, pl.wt, pl.H, wtb, tj);
  const bool rides = !naive && !feature_cat && transposes_ride(pl);
  if (!rides) {
    Probe pb(ctx, HGNN_K_TRANSPOSE_W, layer, !static_area);
    if ((st = launch_transpose_jobs(s, ctx->dtype, tj)) != HGNN_OK) return st;
    ++n;
  }
  if (!naive) {
    if (feature_cat) {
      // Algorithm 1 in two steps (gather into FeatureCat, then reduce by destination) instead of the fused kernel
      for (int t = 0; t < T; ++t)
        if (p->in_dim[t] != p->in_dim[0]) HGNN_FAIL(HGNN_EUNSUPPORTED, "the two-step aggregation needs one input width for all types");
      const size_t need = (size_t)pl.dev.edges * p->in_dim[0] * pl.es;
      if (feature_cat_bytes < need) HGNN_FAIL(HGNN_EINVAL, "feature_cat too small: need %zu bytes", need);
      if ((uintptr_t)feature_cat & 15) HGNN_FAIL(HGNN_EINVAL, "device buffers must be 16-byte aligned");
      Probe pb(ctx, HGNN_K_SPMM_FWD, layer, !static_area);
      if ((st = launch_aggregate_literal(s, ctx->dtype, pl.dev, p->in_dim[0], x, feature_cat, saved, zlo)) != HGNN_OK) return st;
      n += (pl.dev.edges > 0) + (pl.dev.rows > 0);
    } else {
      if (gather_store) {
        uint64_t *gaddr = (uint64_t *)(sc + pl.off_gaddr);
        if ((st = launch_gather_addresses(s, pl.dev, gs, p->in_dim[0] * pl.es, gaddr)) != HGNN_OK) return st;
        if (pl.dev.edges > 0) ++n;
        Probe pb(ctx, HGNN_K_SPMM_FWD, layer);
        if (pl.dev.rows > 0) {
          if (!launch_spmm_fwd_uniform(s, ctx->dtype, pl.dev, p->in_dim[0], nullptr, saved, zlo, 0, pl.dev.rows, gaddr, rides ? &tj : nullptr))
            HGNN_FAIL(HGNN_EUNSUPPORTED, "input width %d is outside what the gather kernels cover", p->in_dim[0]);
          HGNN_HIP(hipGetLastError());
          ++n;
        }
      } else {
        Probe pb(ctx, HGNN_K_SPMM_FWD, layer, !static_area);
        if ((st = launch_spmm_fwd(s, ctx->dtype, pl.dev, pl.tt, pl.rt, pl.max_dim, x, saved, zlo, 0, pl.dev.rows, rides ? &tj : nullptr)) != HGNN_OK) return st;
        if (pl.dev.rows > 0) ++n;
      }
    }
    {
      Probe pb(ctx, HGNN_K_GEMM_FWD, layer, !static_area);
      int kernels = 0;
      if (ctx->dtype == HGNN_BF16 && !ctx->legacy_gemm) {
        kernels = launch_gemm2_fwd(s, pl.tt, pl.rt, pl.pt, pl.wt, live, pl.H, p->relu, x, saved, zlo, wtb, h, &st);
        if (kernels && st != HGNN_OK) return st;
      }
      if (!kernels && optional_launchers().gemm_fwd_direct) {
        kernels = optional_launchers().gemm_fwd_direct(s, ctx->dtype, pl.tt, pl.rt, pl.pt, pl.wt, live, pl.H, p->relu, x, saved, zlo, wtb, h,
                                                       (float *)(sc + pl.off_part), false);
        if (kernels) HGNN_HIP(hipGetLastError());
      }
      if (!kernels) {
        if ((st = launch_gemm_fwd(s, ctx->dtype, pl.dev, pl.tt, pl.rt, pl.pt, pl.wt, tl, live, pl.H, p->relu, x, saved, zlo, wtb, h, -1, nullptr, tile_mn)) != HGNN_OK) return st;
        kernels = tl.tile_off[T] > 0;
      }
      n += kernels;
    }
  } else {
    // the un-merged launch structure: one aggregation and one projection launch per relation, one root
    // projection and one bias/activation launch per vertex type (the projections are told of the activation that follows:
    // see gemm_fwd_kernel on sums that go through a ReLU)
    float *acc32 = (float *)(sc + pl.off_acc32);
    if ((st = launch_fill_zero(s, acc32, (size_t)pl.total_dst * pl.H * 4)) != HGNN_OK) return st;
    ++n;
    const LayerHost &L = g->L[layer];
    const int32_t *rro = g->slab.host + L.o_rel_row_off;
    for (int r = 0; r < R; ++r) {
      if (rro[r + 1] == rro[r]) continue;
      if ((st = launch_spmm_fwd(s, ctx->dtype, pl.dev, pl.tt, pl.rt, pl.max_dim, x, saved, zlo, rro[r], rro[r + 1])) != HGNN_OK) return st;
      ++n;
      SegTab one;
      std::memset(&one, 0, sizeof(one));
      one.num_segs = T;
      const int d = ctx->rel_dst[r];
      for (int t = 0; t < T; ++t)
        one.tile_off[t + 1] = one.tile_off[t] + (t == d ? tl.tile_off[t + 1] - tl.tile_off[t] : 0);
      if ((st = launch_gemm_fwd(s, ctx->dtype, pl.dev, pl.tt, pl.rt, pl.pt, pl.wt, one, live, pl.H, p->relu, x, saved, zlo, wtb, h, r, acc32)) != HGNN_OK) return st;
      ++n;
    }
    for (int t = 0; t < T; ++t) {
      if (pl.tt.n_dst[t] == 0) continue;
      if (p->w_root[t]) {
        SegTab one;
        std::memset(&one, 0, sizeof(one));
        one.num_segs = T;
        for (int u = 0; u < T; ++u)
          one.tile_off[u + 1] = one.tile_off[u] + (u == t ? tl.tile_off[u + 1] - tl.tile_off[u] : 0);
        if ((st = launch_gemm_fwd(s, ctx->dtype, pl.dev, pl.tt, pl.rt, pl.pt, pl.wt, one, live, pl.H, p->relu, x, saved, zlo, wtb, h, R + t, acc32)) != HGNN_OK) return st;
        ++n;
      }
      if ((st = launch_bias_act(s, ctx->dtype, pl.tt, pl.pt, pl.H, p->relu, t, acc32, h)) != HGNN_OK) return st;
      ++n;
    }
  }
  if (launches) *launches = n;
  return HGNN_OK;
}

extern "C++" {
namespace hgnn {
hgnn_status layer_fwd_static_area(hgnn_ctx *ctx, void *stream, hgnn_graph *g, int32_t layer, const hgnn_layer_params *p,
                                  const void *x, void *h, void *saved, size_t saved_bytes, void *area, size_t area_bytes) {
  if (ctx->agg == HGNN_AGG_ATTN) HGNN_FAIL(HGNN_EUNSUPPORTED, "hgnn_layer_fwd_static covers the mean-aggregation layer only");
  return fwd_common(ctx, stream, g, layer, p, x, h, saved, saved_bytes, area, area_bytes, false, nullptr, nullptr, 0, true);
}
}  // namespace hgnn
}  // extern "C++"

hgnn_status hgnn_layer_fwd(hgnn_ctx *ctx, void *stream, hgnn_graph *g, int32_t layer, const hgnn_layer_params *p,
                           const void *x_merged, void *h_out, void *saved, size_t saved_bytes, void *scratch,
                           size_t scratch_bytes) {
  if (ctx && ctx->agg == HGNN_AGG_ATTN)
    return attn_variant().fwd(ctx, stream, g, layer, p, x_merged, h_out, saved, saved_bytes, scratch, scratch_bytes);
  return fwd_common(ctx, stream, g, layer, p, x_merged, h_out, saved, saved_bytes, scratch, scratch_bytes, false, nullptr);
}

hgnn_status hgnn_layer_fwd_gather(hgnn_ctx *ctx, void *stream, hgnn_graph *g, int32_t layer, const hgnn_layer_params *p,
                                  const void *const *store, const int64_t *const *ids, const void *x_dst, void *h_out,
                                  void *saved, size_t saved_bytes, void *scratch, size_t scratch_bytes) {
  if (!ctx || !store || !ids) HGNN_FAIL(HGNN_EINVAL, "NULL argument");
  if (ctx->agg == HGNN_AGG_ATTN) HGNN_FAIL(HGNN_EUNSUPPORTED, "hgnn_layer_fwd_gather covers the mean-aggregation layer only");
  return fwd_common(ctx, stream, g, layer, p, x_dst, h_out, saved, saved_bytes, scratch, scratch_bytes, false, nullptr, nullptr, 0,
                    false, store, ids);
}

hgnn_status hgnn_layer_fwd_naive(hgnn_ctx *ctx, void *stream, hgnn_graph *g, int32_t layer, const hgnn_layer_params *p,
                                 const void *x_merged, void *h_out, void *saved, size_t saved_bytes, void *scratch,
                                 size_t scratch_bytes, int32_t *launches) {
  return fwd_common(ctx, stream, g, layer, p, x_merged, h_out, saved, saved_bytes, scratch, scratch_bytes, true, launches);
}

hgnn_status hgnn_layer_fwd_two_step(hgnn_ctx *ctx, void *stream, hgnn_graph *g, int32_t layer, const hgnn_layer_params *p,
                                    const void *x_merged, void *h_out, void *saved, size_t saved_bytes, void *scratch,
                                    size_t scratch_bytes, void *feature_cat, size_t feature_cat_bytes, int32_t *launches) {
  if (!feature_cat) HGNN_FAIL(HGNN_EINVAL, "feature_cat is NULL");
  return fwd_common(ctx, stream, g, layer, p, x_merged, h_out, saved, saved_bytes, scratch, scratch_bytes, false, launches,
                    feature_cat, feature_cat_bytes);
}

static void seg_tiles_da(hgnn_ctx *ctx, const Plan &pl, const hgnn_layer_params *p, const int32_t *rel_edge_off, SegTab &tl) {
  const int R = ctx->R, T = ctx->T;
  std::memset(&tl, 0, sizeof(tl));
  tl.num_segs = R + T;
  for (int sgi = 0; sgi < R + T; ++sgi) {
    int cnt = 0;
    const bool is_rel = sgi < R;
    const int d = is_rel ? ctx->rel_dst[sgi] : sgi - R;
    const int F = pl.tt.in_dim[is_rel ? ctx->rel_src[sgi] : d];
    bool live = is_rel ? rel_edge_off[sgi + 1] > rel_edge_off[sgi] : p->w_root[d] != nullptr;
    if (p->input_grad && !p->input_grad[is_rel ? ctx->rel_src[sgi] : d]) live = false;  // nobody reads this dZ
    if (live && pl.tt.n_dst[d] > 0) cnt = ((pl.tt.n_dst[d] + 127) / 128) * ((F + 127) / 128);
    tl.tile_off[sgi + 1] = tl.tile_off[sgi] + cnt;
  }
}

// The same tiles (of any edge) grouped for the merged backward launch: per destination type, per row block, the column blocks
// of every live segment whose input gradient is wanted.
static void grouped_tiles_da(hgnn_ctx *ctx, const Plan &pl, const SegTab &by_seg, int edge, DwTab &tl) {
  const int R = ctx->R, T = ctx->T;
  std::memset(&tl, 0, sizeof(tl));
  tl.edge = edge;
  int ne = 0;
  for (int d = 0; d < T; ++d) {
    tl.first[d] = (uint16_t)ne;
    int u = 0;
    for (int sgi = 0; sgi < R + T; ++sgi) {
      const bool is_rel = sgi < R;
      if ((is_rel ? ctx->rel_dst[sgi] : sgi - R) != d || by_seg.tile_off[sgi + 1] == by_seg.tile_off[sgi]) continue;
      tl.seg[ne] = (uint8_t)sgi;
      tl.u_off[ne] = (uint16_t)u;
      u += (pl.tt.in_dim[is_rel ? ctx->rel_src[sgi] : d] + edge - 1) / edge;
      ++ne;
    }
    tl.u_total[d] = (uint16_t)u;
    tl.tile_off[d + 1] = tl.tile_off[d] + u * ((pl.tt.n_dst[d] + edge - 1) / edge);
  }
  tl.first[T] = (uint16_t)ne;
}

static hgnn_status bwd_common(hgnn_ctx *ctx, void *stream, hgnn_graph *g, int32_t layer, const hgnn_layer_params *p,
                              const void *x_merged, const void *h_out, const void *saved, const void *grad_h,
                              void *grad_x_merged, const hgnn_layer_grads *go, void *scratch, size_t scratch_bytes, bool naive,
                              int32_t *launches, bool x_dst_only = false) {
  if (launches) *launches = 0;
  if (ctx && ctx->agg == HGNN_AGG_ATTN) {
    if (naive) HGNN_FAIL(HGNN_EUNSUPPORTED, "the per-relation launch loop exists for the mean-aggregation layer only");
    return attn_variant().bwd(ctx, stream, g, layer, p, x_merged, h_out, saved, grad_h, grad_x_merged, go, scratch, scratch_bytes);
  }
  Plan pl;
  hgnn_status st = make_plan(ctx, g, layer, p, pl, true);
  if (st != HGNN_OK) return st;
  if (x_dst_only) root_rows_only(pl);
  if (!saved || !scratch || !go) HGNN_FAIL(HGNN_EINVAL, "NULL work area or gradient table");
  if (pl.total_dst > 0 && (!x_merged || !grad_h || (p->relu && !h_out))) HGNN_FAIL(HGNN_EINVAL, "NULL input");
  if (scratch_bytes < pl.scratch_bytes) HGNN_FAIL(HGNN_EINVAL, "scratch too small: need %zu bytes", pl.scratch_bytes);
  if (((uintptr_t)saved | (uintptr_t)scratch | (uintptr_t)x_merged | (uintptr_t)grad_h | (uintptr_t)grad_x_merged |
       (uintptr_t)h_out) & 15)
    HGNN_FAIL(HGNN_EINVAL, "device buffers must be 16-byte aligned");
  const int R = ctx->R, T = ctx->T;
  GradPtrTab gt;
  std::memset(&gt, 0, sizeof(gt));
  bool any_dw = false, any_db = false;
  for (int r = 0; r < R; ++r) {
    gt.dw_rel[r] = go->dw_rel ? go->dw_rel[r] : nullptr;
    any_dw |= gt.dw_rel[r] != nullptr;
  }
  for (int t = 0; t < T; ++t) {
    gt.dw_root[t] = (go->dw_root && p->w_root[t]) ? go->dw_root[t] : nullptr;
    gt.dbias[t] = (go->dbias && p->bias && p->bias[t]) ? go->dbias[t] : nullptr;
    any_dw |= gt.dw_root[t] != nullptr;
    any_db |= gt.dbias[t] != nullptr;
  }
  hipStream_t s = (hipStream_t)stream;
  HGNN_HIP(wait_upload(g, s));
  char *sc = (char *)scratch;
  const LayerHost &L = g->L[layer];
  const int32_t *reo = g->slab.host + L.o_rel_edge_off;
  pl.dev.chunk_count = gt.counters = (uint32_t *)(sc + pl.off_count);
  gt.n_counters = grad_x_merged ? pl.dev.n_chunks : 0;
  if ((any_dw || any_db) && pl.total_dst == 0) {  // nothing flows back: the gradients are zero
    Probe pb(ctx, HGNN_K_ZERO_GRADS, layer);
    return launch_zero_grads(s, pl.tt, pl.rt, gt, pl.H);
  }
  // The GEMMs want 16-byte aligned rows.  When H is not a multiple of 16 bytes (or a weight pointer is not
  // aligned) they run on zero-padded copies: G' gets leading dimension Hp in the scratch area (written by the
  // ReLU/bias pass, which then always runs) and so do the weights.
  const int vec = 16 / pl.es;
  const int Hp = (pl.H + vec - 1) / vec * vec;
  bool pad = Hp != pl.H;
  for (int r = 0; r < R; ++r) pad |= ((uintptr_t)p->w_rel[r] & 15) != 0;
  for (int t = 0; t < T; ++t) pad |= p->w_root[t] && ((uintptr_t)p->w_root[t] & 15) != 0;
  int ldg = pl.H;
  PtrTab wpt = pl.pt;
  WtTab wo;
  std::memset(&wo, 0, sizeof(wo));
  void *wpad = nullptr;
  if (pad && pl.total_dst > 0) {
    ldg = Hp;
    size_t w = 0;
    char *wp = sc + pl.off_wt;
    for (int r = 0; r < R; ++r) {
      wo.rel4[r] = (uint32_t)(w / 4);
      wpt.w_rel[r] = wp + w * pl.es;
      w += (size_t)p->in_dim[ctx->rel_src[r]] * Hp;
    }
    for (int t = 0; t < T; ++t) {
      wo.root4[t] = (uint32_t)(w / 4);
      if (p->w_root[t]) {
        wpt.w_root[t] = wp + w * pl.es;
        w += (size_t)p->in_dim[t] * Hp;
      }
    }
    if (grad_x_merged) wpad = wp;
  }
  if (naive) {
    // The un-merged launch structure: the same kernels, launched once per vertex type (ReLU mask / bias gradient,
    // transposed aggregation) and once per relation or root term (weight gradient, input gradient), after one
    // launch that zeroes the gradients (and one that pads the weights where the width asks for it).
    int n = 0;
    void *gpw = sc + pl.off_gp;
    const void *gpn = grad_h;
    if (wpad) {
      if ((st = launch_pad_weights(s, ctx->dtype, pl.tt, pl.rt, pl.pt, wo, pl.H, ldg, wpad)) != HGNN_OK) return st;
      ++n;
    }
    if (any_dw || any_db) {
      if ((st = launch_zero_grads(s, pl.tt, pl.rt, gt, pl.H)) != HGNN_OK) return st;
      ++n;
    }
    if (pl.total_dst > 0 && (p->relu || any_db || ldg != pl.H)) {
      for (int t = 0; t < T; ++t) {
        if (pl.tt.n_dst[t] == 0) continue;
        TypeTab one = pl.tt;
        for (int u = 0; u < T; ++u)
          if (u != t) one.n_dst[u] = 0;
        if ((st = launch_relu_bias_bwd(s, ctx->dtype, one, pl.H, ldg, p->relu, grad_h, h_out, gpw, gt)) != HGNN_OK) return st;
        ++n;
      }
      if (p->relu || ldg != pl.H) gpn = gpw;
    }
    const bool fastn = (ldg % (16 / pl.es)) == 0;
    const bool want_dxn = grad_x_merged && pl.dev.src_rows > 0;
    if (want_dxn)
      for (int t = 0; t < T; ++t)
        if ((!p->input_grad || p->input_grad[t]) && !((L.tmask >> t) & 1u) && L.n_src[t] > 0)
          HGNN_FAIL(HGNN_EINVAL, "input gradient of type %d asked for, but the graph was built without its transpose entries", t);
    if (want_dxn && gt.n_counters > 0) {
      if ((st = launch_fill_zero(s, gt.counters, (size_t)gt.n_counters * 4)) != HGNN_OK) return st;
      ++n;
    }
    void *dzn = sc + pl.off_dz;
    const int tiles_hn = (pl.H + 127) / 128;
    for (int sgi = 0; sgi < R + T && pl.total_dst > 0; ++sgi) {
      const bool is_rel = sgi < R;
      const int d = is_rel ? ctx->rel_dst[sgi] : sgi - R;
      const int F = pl.tt.in_dim[is_rel ? ctx->rel_src[sgi] : d];
      if (pl.tt.n_dst[d] == 0) continue;
      const bool live = is_rel ? reo[sgi + 1] > reo[sgi] : p->w_root[d] != nullptr;
      if (!live) continue;
      if (is_rel ? gt.dw_rel[sgi] != nullptr : gt.dw_root[d] != nullptr) {  // weight gradient of this segment
        DwTab one;
        std::memset(&one, 0, sizeof(one));
        for (int u = 0; u <= T; ++u) one.first[u] = (uint16_t)(u > d ? 1 : 0);
        one.seg[0] = (uint8_t)sgi;
        one.u_off[0] = 0;
        one.u_total[d] = (uint16_t)((F + 127) / 128);
        const int split_rows = 2048;
        const int cnt = one.u_total[d] * tiles_hn * ((pl.tt.n_dst[d] + split_rows - 1) / split_rows);
        for (int u = d; u < T; ++u) one.tile_off[u + 1] = cnt;
        if ((st = launch_gemm_dw(s, ctx->dtype, pl.dev, pl.tt, pl.rt, gt, one, split_rows, pl.H, ldg, fastn, x_merged, saved, gpn)) != HGNN_OK) return st;
        ++n;
      }
      if (want_dxn && (!p->input_grad || p->input_grad[is_rel ? ctx->rel_src[sgi] : d])) {  // input gradient of this segment
        SegTab one;
        std::memset(&one, 0, sizeof(one));
        one.num_segs = R + T;
        const int cnt = ((pl.tt.n_dst[d] + 127) / 128) * ((F + 127) / 128);
        for (int u = sgi; u < R + T; ++u) one.tile_off[u + 1] = cnt;
        if ((st = launch_gemm_da(s, ctx->dtype, pl.dev, pl.tt, pl.rt, wpt, one, ldg, fastn, gpn, dzn)) != HGNN_OK) return st;
        ++n;
      }
    }
    if (want_dxn) {
      for (int t = 0; t < T; ++t) {
        if ((p->input_grad && !p->input_grad[t]) || L.n_src[t] == 0) continue;
        if ((st = launch_spmm_bwd(s, ctx->dtype, pl.dev, pl.tt, pl.rt, pl.pt, pl.max_dim, 1u << t, dzn, grad_x_merged, (float *)(sc + pl.off_partial))) != HGNN_OK) return st;
        ++n;
      }
    }
    if (launches) *launches = n;
    return HGNN_OK;
  }
  // One launch: the row pass over G (ReLU mask, padded copy, column sums for the bias gradient as partial sums
  // per block), zeroing of the weight gradients, the padded weights.  The partial sums are added up by a few
  // blocks of the backward GEMM launch below, or by a launch of their own when that one does not run.
  const void *gp = grad_h;
  const bool row_pass = pl.total_dst > 0 && (p->relu || any_db || ldg != pl.H);
  float *bpart = any_db ? (float *)(sc + pl.off_bpart) : nullptr;
  int rpb = 0;  // rows of G per row of bpart: set by the launcher
  if (pl.total_dst > 0) {
    void *gpw = sc + pl.off_gp;
    PtrTab used = pl.pt;   // a relation without edges has no input gradient, so that nobody reads a padded copy of its weight
    for (int r = 0; r < R; ++r)
      if (reo[r + 1] == reo[r]) used.w_rel[r] = nullptr;
    Probe pb(ctx, HGNN_K_RELU_BIAS_BWD, layer);
    if ((st = launch_bwd_prep(s, ctx->dtype, pl.tt, pl.rt, used, wo, gt, pl.H, ldg, p->relu, row_pass, any_dw, grad_h, h_out, gpw,
                              bpart, pl.bpart_rows, wpad, &rpb)) != HGNN_OK) return st;
    if (p->relu || ldg != pl.H) gp = gpw;
  }
  const bool fast = (ldg % vec) == 0;
  const bool want_dx = grad_x_merged && pl.dev.src_rows > 0;
  if (want_dx)
    for (int t = 0; t < T; ++t)
      if ((!p->input_grad || p->input_grad[t]) && !((L.tmask >> t) & 1u) && L.n_src[t] > 0)
        HGNN_FAIL(HGNN_EINVAL, "input gradient of type %d asked for, but the graph was built without its transpose entries", t);
  SegTab da_tl;
  if (want_dx) seg_tiles_da(ctx, pl, p, reo, da_tl);
  void *dz = sc + pl.off_dz;
  bool da_done = false;
  if (any_dw && pl.total_dst > 0) {
    // Work list: per destination type its live segments (relations with edges, then the root) and the row blocks of
    // their weight gradients, with the input-gradient tiles of the same launch beside it.  Tiles have 128 rows and
    // columns, or 64 (bwd_small_tiles).
    DwTab tl, da_grouped;
    const bool both = want_dx && da_tl.tile_off[da_tl.num_segs] > 0;
    const int bk = pl.es == 2 ? 64 : 32;
    int split_rows = 0;
    BwdCols cols;
    for (int edge = 128;; edge = 64) {
      std::memset(&tl, 0, sizeof(tl));
      tl.edge = edge;
      int ne = 0;
      int64_t dw_steps = 0, da_steps = 0;
      const int tiles_h = (pl.H + edge - 1) / edge;
      for (int d = 0; d < T; ++d) {
        tl.first[d] = (uint16_t)ne;
        int u = 0;
        if (pl.tt.n_dst[d] > 0)
          for (int sgi = 0; sgi < R + T; ++sgi) {
            const bool is_rel = sgi < R;
            if (is_rel ? (ctx->rel_dst[sgi] != d || reo[sgi + 1] == reo[sgi] || !gt.dw_rel[sgi]) : (sgi - R != d || !gt.dw_root[d])) continue;
            tl.seg[ne] = (uint8_t)sgi;
            tl.u_off[ne] = (uint16_t)u;
            const int F = pl.tt.in_dim[is_rel ? ctx->rel_src[sgi] : d];
            u += (F + edge - 1) / edge;
            if (edge == 128) cols.segment(F);
            ++ne;
          }
        tl.u_total[d] = (uint16_t)u;
        if (edge == 128 && u > 0) ++cols.types;
        dw_steps += (int64_t)u * tiles_h * ((pl.tt.n_dst[d] + bk - 1) / bk);
      }
      tl.first[T] = (uint16_t)ne;
      if (both) {
        grouped_tiles_da(ctx, pl, da_tl, edge, da_grouped);
        da_steps = (int64_t)da_grouped.tile_off[T] * ((ldg + bk - 1) / bk);
      }
      split_rows = dw_slice_rows(ctx->dtype, edge, dw_steps, da_steps);
      for (int d = 0; d < T; ++d)
        tl.tile_off[d + 1] = tl.tile_off[d] + tl.u_total[d] * tiles_h * ((pl.tt.n_dst[d] + split_rows - 1) / split_rows);
      if (edge == 64 || !bwd_small_tiles(ctx->dtype, tl.tile_off[T] + (both ? da_grouped.tile_off[T] : 0), ldg, cols, both)) break;
    }
    Probe pb(ctx, HGNN_K_GEMM_DW, layer);
    if (both && tl.tile_off[T] > 0) {
      // both backward GEMMs read G' and are independent of each other: one launch
      if ((st = launch_gemm_bwd(s, ctx->dtype, pl.dev, pl.tt, pl.rt, wpt, da_grouped, gt, tl, split_rows, pl.H, ldg, fast, x_merged,
                                saved, gp, dz, bpart, rpb)) != HGNN_OK) return st;
      da_done = true;
      bpart = nullptr;
    } else if ((st = launch_gemm_dw(s, ctx->dtype, pl.dev, pl.tt, pl.rt, gt, tl, split_rows, pl.H, ldg, fast, x_merged, saved, gp)) != HGNN_OK) {
      return st;
    }
  }
  if (bpart && (st = launch_bias_reduce(s, pl.tt, gt, pl.H, rpb, bpart)) != HGNN_OK) return st;
  if (want_dx) {
    if (!da_done) {
      Probe pb(ctx, HGNN_K_GEMM_DA, layer);
      if ((st = launch_gemm_da(s, ctx->dtype, pl.dev, pl.tt, pl.rt, wpt, da_tl, ldg, fast, gp, dz)) != HGNN_OK) return st;
    }
    Probe pb(ctx, HGNN_K_SPMM_BWD, layer);
    uint32_t want = 0;
    for (int t = 0; t < T; ++t)
      if (!p->input_grad || p->input_grad[t]) want |= 1u << t;
    if ((st = launch_spmm_bwd(s, ctx->dtype, pl.dev, pl.tt, pl.rt, pl.pt, pl.max_dim, want, dz, grad_x_merged, (float *)(sc + pl.off_partial))) != HGNN_OK) return st;
  }
  return HGNN_OK;
}

hgnn_status hgnn_layer_bwd(hgnn_ctx *ctx, void *stream, hgnn_graph *g, int32_t layer, const hgnn_layer_params *p,
                           const void *x_merged, const void *h_out, const void *saved, const void *grad_h,
                           void *grad_x_merged, const hgnn_layer_grads *go, void *scratch, size_t scratch_bytes) {
  return bwd_common(ctx, stream, g, layer, p, x_merged, h_out, saved, grad_h, grad_x_merged, go, scratch, scratch_bytes, false, nullptr);
}

hgnn_status hgnn_layer_bwd_gather(hgnn_ctx *ctx, void *stream, hgnn_graph *g, int32_t layer, const hgnn_layer_params *p,
                                  const void *x_dst, const void *h_out, const void *saved, const void *grad_h,
                                  void *grad_x_merged, const hgnn_layer_grads *go, void *scratch, size_t scratch_bytes) {
  if (ctx && ctx->agg == HGNN_AGG_ATTN) HGNN_FAIL(HGNN_EUNSUPPORTED, "hgnn_layer_bwd_gather covers the mean-aggregation layer only");
  return bwd_common(ctx, stream, g, layer, p, x_dst, h_out, saved, grad_h, grad_x_merged, go, scratch, scratch_bytes, false, nullptr, true);
}

hgnn_status hgnn_layer_bwd_naive(hgnn_ctx *ctx, void *stream, hgnn_graph *g, int32_t layer, const hgnn_layer_params *p,
                                 const void *x_merged, const void *h_out, const void *saved, const void *grad_h,
                                 void *grad_x_merged, const hgnn_layer_grads *go, void *scratch, size_t scratch_bytes,
                                 int32_t *launches) {
  return bwd_common(ctx, stream, g, layer, p, x_merged, h_out, saved, grad_h, grad_x_merged, go, scratch, scratch_bytes, true, launches);
}

hgnn_status hgnn_layer_launch_count(hgnn_ctx *ctx, hgnn_graph *g, int32_t layer, const hgnn_layer_params *p,
                                    int32_t *fwd_launches, int32_t *bwd_launches) {
  if (ctx && ctx->agg == HGNN_AGG_ATTN) {
    return attn_variant().launch_count(ctx, g, layer, p, fwd_launches, bwd_launches);
  }
  Plan pl;
  hgnn_status st = make_plan(ctx, g, layer, p, pl, true);
  if (st != HGNN_OK) return st;
  if (fwd_launches) {
    int gemm = 0;
    if (optional_launchers().gemm_fwd_direct && (ctx->dtype != HGNN_BF16 || ctx->legacy_gemm)) {
      uint32_t live[kMaxR / 32];
      live_relations(ctx, g, layer, live);
      const void *zlo = ctx->dtype == HGNN_BF16 && p->relu ? &pl : nullptr;   // whether there is one is all that counts
      gemm = optional_launchers().gemm_fwd_direct(nullptr, ctx->dtype, pl.tt, pl.rt, pl.pt, pl.wt, live, pl.H, p->relu, nullptr, nullptr,
                                                  zlo, nullptr, nullptr, nullptr, true);
    }
    *fwd_launches = (transposes_ride(pl) ? 0 : 1) + (pl.dev.rows > 0) + (gemm ? gemm : pl.total_dst > 0);
  }
  if (bwd_launches) {
    // zero grads + ReLU mask + bias partial sums (one launch), dW and dA GEMMs + bias sums (one launch), transposed
    // aggregation; without destination rows only the zeroing
    *bwd_launches = pl.total_dst > 0 ? 2 + (pl.dev.src_rows > 0) : 1;
  }
  return HGNN_OK;
}

hgnn_status hgnn_softmax_xent(hgnn_ctx *ctx, void *stream, const void *logits, const int64_t *labels, int64_t rows,
                              int32_t classes, float *loss, void *grad_logits) {
  if (!ctx || !loss) HGNN_FAIL(HGNN_EINVAL, "NULL argument");
  if (rows < 0 || classes < 1) HGNN_FAIL(HGNN_EINVAL, "bad shape %lld x %d", (long long)rows, classes);
  if (rows > 0 && (!logits || !labels || !grad_logits)) HGNN_FAIL(HGNN_EINVAL, "NULL argument");
  if (ctx->device < 0) HGNN_FAIL(HGNN_EUNSUPPORTED, "host-only context cannot run device work");
  Probe pb(ctx, HGNN_K_XENT, -1);
  return launch_xent((hipStream_t)stream, ctx->dtype, logits, labels, rows, classes, loss, grad_logits);
}

static hgnn_status check_adam(const hgnn_adam_params *hp, double &c1, double &c2) {
  if (!hp) HGNN_FAIL(HGNN_EINVAL, "NULL argument");
  if (hp->step < 1 || !(hp->beta1 >= 0.f && hp->beta1 < 1.f) || !(hp->beta2 >= 0.f && hp->beta2 < 1.f) || !(hp->eps >= 0.f))
    HGNN_FAIL(HGNN_EINVAL, "Adam needs step >= 1, beta1 and beta2 in [0,1), eps >= 0");
  c1 = 1.0 / (1.0 - std::pow((double)hp->beta1, (double)hp->step));
  c2 = 1.0 / (1.0 - std::pow((double)hp->beta2, (double)hp->step));
  return HGNN_OK;
}

hgnn_status hgnn_adam_update(hgnn_ctx *ctx, void *stream, int32_t n, void *const *param, float *const *master,
                             const float *const *grad, float *const *m, float *const *v, const int64_t *numel,
                             const hgnn_adam_params *hp) {
  if (!ctx || n < 0 || (n > 0 && (!param || !grad || !m || !v || !numel))) HGNN_FAIL(HGNN_EINVAL, "NULL argument");
  double c1, c2;
  hgnn_status st = check_adam(hp, c1, c2);
  if (st != HGNN_OK) return st;
  for (int i = 0; i < n; ++i) {
    if (numel[i] < 0 || numel[i] > (int64_t)INT32_MAX * 1024) HGNN_FAIL(HGNN_EINVAL, "numel[%d]=%lld out of range", i, (long long)numel[i]);
    if (numel[i] > 0 && (!param[i] || !grad[i] || !m[i] || !v[i])) HGNN_FAIL(HGNN_EINVAL, "tensor %d: NULL pointer", i);
    if (numel[i] > 0 && ctx->dtype != HGNN_F32 && (!master || !master[i]))
      HGNN_FAIL(HGNN_EINVAL, "tensor %d: a bf16 parameter needs an fp32 master copy", i);
  }
  if (ctx->device < 0) HGNN_FAIL(HGNN_EUNSUPPORTED, "host-only context cannot run device work");
  return launch_adam_dense((hipStream_t)stream, ctx->dtype, n, param, master, grad, m, v, numel, hp->lr, hp->beta1, hp->beta2,
                           hp->eps, c1, c2);
}

hgnn_status hgnn_adam_update_rows(hgnn_ctx *ctx, void *stream, void *store, float *master, float *m, float *v,
                                  int32_t feat_dim, const int64_t *ids, int64_t n_rows, const void *grad_rows,
                                  const hgnn_adam_params *hp) {
  if (!ctx || n_rows < 0) HGNN_FAIL(HGNN_EINVAL, "NULL argument");
  double c1, c2;
  hgnn_status st = check_adam(hp, c1, c2);
  if (st != HGNN_OK) return st;
  const int vec = 16 / esize(ctx->dtype);
  if (feat_dim <= 0 || feat_dim % vec != 0) HGNN_FAIL(HGNN_EINVAL, "feat_dim=%d is not a positive multiple of %d", feat_dim, vec);
  if (n_rows > 0 && (!store || !m || !v || !ids || !grad_rows)) HGNN_FAIL(HGNN_EINVAL, "NULL argument");
  if (n_rows > 0 && ctx->dtype != HGNN_F32 && !master) HGNN_FAIL(HGNN_EINVAL, "a bf16 table needs an fp32 master copy");
  for (const void *p : {(const void *)store, (const void *)master, (const void *)m, (const void *)v, grad_rows})
    if (reinterpret_cast<uintptr_t>(p) & 15) HGNN_FAIL(HGNN_EINVAL, "tables and gradient rows must be 16-byte aligned");
  if (ctx->device < 0) HGNN_FAIL(HGNN_EUNSUPPORTED, "host-only context cannot run device work");
  return launch_adam_rows((hipStream_t)stream, ctx->dtype, store, master, m, v, feat_dim, ids, n_rows, grad_rows, hp->lr,
                          hp->beta1, hp->beta2, hp->eps, c1, c2);
}

hgnn_status hgnn_probe_select(hgnn_ctx *ctx, int32_t kernel, int32_t layer) {
  if (!ctx) HGNN_FAIL(HGNN_EINVAL, "NULL context");
  if (kernel > HGNN_K_XENT) HGNN_FAIL(HGNN_EINVAL, "unknown kernel id %d", kernel);
  if (kernel < 0) {
    ctx->probe_n = 0;
    ctx->probe_used = 0;
    return HGNN_OK;
  }
  if (ctx->probe_n >= 4) HGNN_FAIL(HGNN_EINVAL, "at most 4 kernels can be selected at a time");
  ctx->probe_sel[ctx->probe_n][0] = kernel;
  ctx->probe_sel[ctx->probe_n][1] = layer;
  ++ctx->probe_n;
  return HGNN_OK;
}

hgnn_status hgnn_probe_read(hgnn_ctx *ctx, int32_t kernel, int32_t layer, double *total_ms, int64_t *launches) {
  if (!ctx || !total_ms || !launches) HGNN_FAIL(HGNN_EINVAL, "NULL argument");
  double sum = 0;
  int64_t n = 0;
  for (size_t i = 0; i < ctx->probe_used; ++i) {
    const int sl = ctx->probe_slot[i];
    if (ctx->probe_sel[sl][0] != kernel || ctx->probe_sel[sl][1] != layer) continue;
    float ms = 0;
    HGNN_HIP(hipEventSynchronize(ctx->probe_events[i].second));
    HGNN_HIP(hipEventElapsedTime(&ms, ctx->probe_events[i].first, ctx->probe_events[i].second));
    sum += ms;
    n += ctx->probe_first[i];
  }
  *total_ms = sum;
  *launches = n;
  return HGNN_OK;
}

}  // extern "C"
