// Layer-wise neighbour sampling on the host (Section 2.3 step 1; Fig. 6's sampling thread), run as the first
// part of a builder's task so that sampling, edge index selection and upload of mini-batch i+k overlap the GPU
// work of mini-batch i.  The rule (order of visits, subset choice, generator) is the one stated with
// hgnn_sample_and_build in hgnn.h.
#include <algorithm>
#include <cstring>

#include "common.h"

namespace hgnn {

// SplitMix64 output function (Steele, Lea, Flood: "Fast splittable pseudorandom number generators", 2014)
static inline uint64_t mix64(uint64_t z) {
  z += 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// With several threads a hop is worked off in four passes over its merged rows (relations ascending, destinations ascending), each split over
// the host threads in tasks of kTaskRows destinations of one relation:
//   1  choose the neighbours; every source vertex that is no destination is claimed by the first row that reaches it
//      (a minimum over row numbers in the local-row table, so the outcome does not depend on which thread is first)
//   2  mark the edges that are the first to reach their vertex and count them per task
//   3  number those: a type's new rows follow in the order in which the rows reach them
//   4  write the lists
// What the passes cost is the local-row table's cache lines moving between the cores, so each looks at as few of its
// entries as it can: 2 at all edges', 3 writes those of new vertices, 4 reads those of the other edges.  (256 targets,
// 50k edges: 0.27 ms on 15 threads; a single thread takes 0.8 ms in one pass, and would take 1.6 ms in four.)
constexpr int kTaskRows = 64, kMaxFan = 64;
// Destination vertices are taken in blocks; inside a block every step (row pointers, neighbour positions, neighbour ids,
// local-row table) is done for all vertices before the next, each step prefetching what the next one reads: the reads are
// random accesses into arrays far larger than the caches, and this keeps dozens of them in flight instead of one.
constexpr int kBlock = 32;

// Neighbour positions of a block's vertices (their row pointers have been prefetched) and how many each keeps.
static inline void choose_block(const int64_t *ptr, const int32_t *nbr, const int64_t *vertex, int nb, int64_t fanout, uint64_t kr,
                                int64_t (*pos)[kMaxFan], int32_t *cnt) {
  for (int b = 0; b < nb; ++b) {
    const int64_t v = vertex[b];
    const int64_t first = ptr[v], deg = ptr[v + 1] - first;
    int64_t *pb = pos[b];
    if (deg <= fanout) {
      for (int64_t p = 0; p < deg; ++p) pb[p] = first + p;
      cnt[b] = (int32_t)deg;
      for (int64_t p = 0; p < deg; p += 16) __builtin_prefetch(nbr + first + p);
    } else {
      const uint64_t key = mix64(kr ^ (uint64_t)v);
      for (int64_t c = 0; c < fanout; ++c) {
        const int64_t j = deg - fanout + c;
        int64_t t = (int64_t)(((unsigned __int128)mix64(key + (uint64_t)c) * (uint64_t)(j + 1)) >> 64);
        bool again = false;
        for (int64_t q = 0; q < c; ++q) again |= pb[q] == first + t;  // no early exit: the loop vectorises
        if (again) t = j;
        pb[c] = first + t;
        __builtin_prefetch(nbr + first + t);
      }
      cnt[b] = (int32_t)fanout;
    }
  }
}

struct SampleTask {
  int32_t r;
  int32_t i0, i1;     // destinations of the relation
  int64_t row;        // merged row of destination i0
  int64_t at;         // its first edge inside the slice
  int64_t edges, fresh;              // edges kept; those that are the first to reach their vertex
  int64_t first_edge, first_fresh;   // where these start in the hop's lists and in the source type's
};

hgnn_status run_sample_job(hgnn_ctx *ctx, Builder &bd, hgnn_graph *g, std::string &msg) {
  PhaseTimer tm;
  SampleJob &job = *g->job;
  const hgnn_sampler &sm = *job.sampler;
  const int T = ctx->T, R = ctx->R, L = g->num_layers;
  ThreadPool &pool = *bd.pool;
  for (int t = 0; t < T; ++t)
    if ((int64_t)bd.local_of[t].size() != sm.num_nodes[t]) bd.local_of[t].assign((size_t)sm.num_nodes[t], -1);
  // global ids per type of the current hop; the buffers live in the builder and in the (pooled) job, so that a
  // steady stream of mini-batches allocates nothing and touches no fresh pages
  std::vector<int64_t> *dst = bd.hop_ids[0], *src = bd.hop_ids[1];
  for (int t = 0; t < T; ++t) dst[t].clear();
  dst[job.target_type] = job.targets;
  const uint64_t k0 = mix64(job.seed);
  hgnn_status st = HGNN_OK;
  std::vector<SampleTask> tasks;
  // runs fn(task, slice) for all tasks, each pass dealing the same slices of them, each slice's in order
  auto for_tasks = [&](auto fn) {
    const int n = (int)tasks.size(), slices = std::min({n, kSampleSlices, 2 * pool.size()});
    pool.parallel_for(slices, [&](int i) {
      for (int t = (int)((int64_t)n * i / slices); t < (int)((int64_t)n * (i + 1) / slices); ++t) fn(tasks[t], bd.slice[i]);
    });
  };
  // runs fn(first, last) over [0, n) in pieces of at least `least`
  auto split = [&](size_t n, size_t least, auto fn) {
    const int pieces = (int)std::min<size_t>((size_t)pool.size(), (n + least - 1) / least);
    pool.parallel_for(pieces, [&](int i) { fn(n * i / pieces, n * (i + 1) / pieces); });
  };
  for (int h = 1; h <= L && st == HGNN_OK; ++h) {
    const int l = L - h;
    const int64_t fanout = job.fanouts[h - 1];
    const uint64_t kh = mix64(k0 ^ (uint64_t)h);
    for (int t = 0; t < T; ++t) {
      src[t] = dst[t];
      int32_t *lut = bd.local_of[t].data();
      if (h > 1) {   // distinct by construction
        split(dst[t].size(), 4096, [&](size_t a, size_t b) {
          for (size_t i = a; i < b; ++i) lut[dst[t][i]] = (int32_t)i;
        });
      } else {
        for (size_t i = 0; i < dst[t].size(); ++i) {
          const int64_t v = dst[t][i];
          if (lut[v] >= 0) {
            msg = "target " + std::to_string(v) + " is listed twice";
            st = HGNN_EINVAL;
            src[t].resize(i);  // the entries to reset below
            break;
          }
          lut[v] = (int32_t)i;
        }
      }
      job.n_dst[l][t] = (int64_t)dst[t].size();
    }
    int64_t rows = 0;
    tasks.clear();
    for (int r = 0; r < R; ++r) {
      const int64_t nd = (int64_t)dst[ctx->rel_dst[r]].size();
      for (int64_t i = 0; i < nd; i += kTaskRows)
        tasks.push_back({r, (int32_t)i, (int32_t)std::min<int64_t>(nd, i + kTaskRows), rows + i, 0, 0, 0, 0, 0});
      rows += nd;
    }
    if (st == HGNN_OK && rows > (int64_t)INT32_MAX - 2) {
      msg = "more than 2^31-3 merged rows";
      st = HGNN_EOVERFLOW;
    }
    if (pool.size() == 1) {
      // a single thread: one pass that numbers the vertices as it reaches them
      I64Buf &es = job.edge_index[l], &ed = bd.dst_pos;  // local sources; the destinations are appended below
      I64Buf &eid = job.edge_id[l];
      std::vector<int32_t> &rp = job.row_ptr[l];
      {
        size_t bound = 0;  // every destination keeps at most `fanout` edges per relation
        for (int r = 0; r < R; ++r) bound += dst[ctx->rel_dst[r]].size() * (size_t)fanout;
        bound = std::min<size_t>(bound, (size_t)sm.edge_off[R]);
        if (!es.reserve(2 * bound + 1) || !ed.reserve(bound + 1) || !eid.reserve(bound + 1)) {
          msg = "out of host memory";
          st = HGNN_ENOMEM;
        }
      }
      int64_t *pes = es.p, *ped = ed.p, *peid = eid.p;
      size_t ne = 0;  // edges of this hop so far (the bound above holds, so the writes below need no check)
      int64_t row = 0;
      if (st == HGNN_OK) rp.resize((size_t)rows + 1);
      for (int r = 0; r < R && st == HGNN_OK; ++r) {
        const int s = ctx->rel_src[r], d = ctx->rel_dst[r];
        const int64_t nd = (int64_t)dst[d].size();
        if (nd == 0) continue;
        const int64_t *ptr = sm.in_indptr[r];
        const int32_t *nbr = sm.in_nbr[r];
        const int64_t e0 = sm.edge_off[r];
        int32_t *lut = bd.local_of[s].data();
        std::vector<int64_t> &sl = src[s];
        const uint64_t kr = mix64(kh ^ (uint64_t)r);
        int64_t pos[kBlock][kMaxFan];
        int32_t cnt[kBlock];
        for (int64_t i0 = 0; i0 < nd; i0 += kBlock) {
          const int nb = (int)std::min<int64_t>(kBlock, nd - i0);
          for (int b = 0; b < nb; ++b) __builtin_prefetch(ptr + dst[d][i0 + b]);
          if (i0 + kBlock < nd)
            for (int b = 0; b < kBlock && i0 + kBlock + b < nd; b += 8) __builtin_prefetch(&dst[d][i0 + kBlock + b]);
          choose_block(ptr, nbr, dst[d].data() + i0, nb, fanout, kr, pos, cnt);
          for (int b = 0; b < nb; ++b)
            for (int c = 0; c < cnt[b]; ++c) __builtin_prefetch(lut + nbr[pos[b][c]]);
          for (int b = 0; b < nb; ++b) {
            const int64_t i = i0 + b;
            rp[row++] = (int32_t)ne;
            for (int c = 0; c < cnt[b]; ++c) {
              const int64_t p = pos[b][c];
              const int64_t u = nbr[p];
              int32_t loc = lut[u];
              if (loc < 0) {
                loc = (int32_t)sl.size();
                lut[u] = loc;
                sl.push_back(u);
              }
              pes[ne] = loc;
              ped[ne] = i;
              peid[ne] = e0 + p;
              ++ne;
            }
          }
        }
        if (sl.size() > (size_t)INT32_MAX - 1) {
          msg = "more than 2^31-2 source rows of one type";
          st = HGNN_EOVERFLOW;
        }
      }
      if (st == HGNN_OK) rp[rows] = (int32_t)ne;
      if (st == HGNN_OK && ne) std::memcpy(pes + ne, ped, ne * sizeof(int64_t));
      es.n = 2 * ne;
      eid.n = ne;
    } else {
    if (st == HGNN_OK && !bd.edge_cnt.reserve((size_t)rows + 1)) {
      msg = "out of host memory";
      st = HGNN_ENOMEM;
    }
    int32_t *ecnt = bd.edge_cnt.p;
    if (st != HGNN_OK) tasks.clear();
    for (SampleSlice &sl : bd.slice) sl.src.n = 0;
    std::atomic<bool> no_memory{false};
    tm.lap("hop set-up");
    for_tasks([&](SampleTask &tk, SampleSlice &sl) {
      const int r = tk.r, s = ctx->rel_src[r], d = ctx->rel_dst[r];
      const int64_t *ptr = sm.in_indptr[r], *dv = dst[d].data();
      const int32_t *nbr = sm.in_nbr[r];
      const int64_t e0 = sm.edge_off[r];
      int32_t *lut = bd.local_of[s].data();
      const uint64_t kr = mix64(kh ^ (uint64_t)r);
      int64_t pos[kBlock][kMaxFan];
      tk.at = (int64_t)sl.src.n;
      for (int32_t i0 = tk.i0; i0 < tk.i1; i0 += kBlock) {
        const int nb = std::min(kBlock, tk.i1 - i0);
        const int64_t row0 = tk.row + (i0 - tk.i0);
        for (int b = 0; b < nb; ++b) __builtin_prefetch(ptr + dv[i0 + b]);
        choose_block(ptr, nbr, dv + i0, nb, fanout, kr, pos, ecnt + row0);
        size_t kept = 0, at = sl.src.n;
        for (int b = 0; b < nb; ++b) kept += (size_t)ecnt[row0 + b];
        // room for what is kept, not for `fanout` per row: most rows of a graph of many relations keep next to nothing
        if (no_memory.load(std::memory_order_relaxed) || !sl.src.reserve(at + kept) || !sl.pos.reserve(at + kept)) {
          no_memory.store(true, std::memory_order_relaxed);
          return;
        }
        sl.src.n = at + kept;
        tk.edges += (int64_t)kept;
        int32_t *u = sl.src.p + at;
        int64_t *p = sl.pos.p + at;
        for (int b = 0; b < nb; ++b)
          for (int c = 0; c < ecnt[row0 + b]; ++c) {
            const int32_t v = nbr[pos[b][c]];
            *u++ = v;
            *p++ = e0 + pos[b][c];
            __builtin_prefetch(lut + v, 1);   // to be written
          }
        u = sl.src.p + at;
        for (int b = 0; b < nb; ++b) {
          const int32_t mine = (int32_t)(-2 - (row0 + b));   // claims: -2 - row, so that an earlier row is the larger value
          for (int c = 0; c < ecnt[row0 + b]; ++c) {
            std::atomic_ref<int32_t> slot(lut[*u++]);
            int32_t cur = slot.load(std::memory_order_relaxed);
            while ((cur == -1 || cur < mine) && !slot.compare_exchange_weak(cur, mine, std::memory_order_relaxed)) {}
          }
        }
      }
    });
    tm.lap("choose and claim");
    if (no_memory.load()) {
      msg = "out of host memory";
      st = HGNN_ENOMEM;
    }
    // prefetches the table's entries of the edges some way ahead of edge `e` of a task that ends at `end`
    constexpr int64_t kAhead = 32;
    auto ahead = [&](const int32_t *lut, const int32_t *u, int64_t end, int64_t e, int cnt) {
      for (int64_t q = e + kAhead; q < std::min(end, e + kAhead + cnt); ++q) __builtin_prefetch(lut + (u[q] < 0 ? ~u[q] : u[q]));
    };
    if (st == HGNN_OK)
      for_tasks([&](SampleTask &tk, SampleSlice &sl) {
        const int32_t *lut = bd.local_of[ctx->rel_src[tk.r]].data();
        int32_t *u = sl.src.p + tk.at;
        int64_t e = 0;
        for (int64_t row = tk.row; row < tk.row + (tk.i1 - tk.i0); e += ecnt[row++]) {
          ahead(lut, u, tk.edges, e, ecnt[row]);
          int32_t *w = u + e;
          for (int c = 0; c < ecnt[row]; ++c)
            if (lut[w[c]] == (int32_t)(-2 - row)) {
              bool again = false;   // a vertex may be a row's neighbour twice
              for (int q = 0; q < c; ++q) again |= w[q] == ~w[c];
              if (again) continue;
              w[c] = ~w[c];         // marked (vertex ids are not negative)
              ++tk.fresh;
            }
        }
      });
    tm.lap("count");
    int64_t size[kMaxT], ne = 0;
    for (int t = 0; t < T; ++t) size[t] = (int64_t)src[t].size();
    for (SampleTask &tk : tasks) {
      tk.first_edge = ne;
      tk.first_fresh = size[ctx->rel_src[tk.r]];
      ne += tk.edges;
      size[ctx->rel_src[tk.r]] += tk.fresh;
    }
    for (int t = 0; t < T && st == HGNN_OK; ++t)
      if (size[t] > (int64_t)INT32_MAX - 1) {
        msg = "more than 2^31-2 source rows of one type";
        st = HGNN_EOVERFLOW;
      }
    I64Buf &es = job.edge_index[l];  // local sources, then local destinations
    I64Buf &eid = job.edge_id[l];
    if (st == HGNN_OK && (!es.reserve(2 * (size_t)ne + 1) || !eid.reserve((size_t)ne + 1))) {
      msg = "out of host memory";
      st = HGNN_ENOMEM;
    }
    if (st != HGNN_OK) {   // the claims go; the destinations' entries are reset below
      for (int t = 0; t < T; ++t)
        for (int32_t &v : bd.local_of[t]) v = std::max(v, -1);
    } else {
      for (int t = 0; t < T; ++t) src[t].resize((size_t)size[t]);
      std::vector<int32_t> &rp = job.row_ptr[l];
      rp.resize((size_t)rows + 1);
      rp[rows] = (int32_t)ne;
      for_tasks([&](SampleTask &tk, SampleSlice &sl) {
        const int s = ctx->rel_src[tk.r];
        int32_t *lut = bd.local_of[s].data();
        const int32_t *u = sl.src.p + tk.at;
        int64_t *ids = src[s].data(), next = tk.first_fresh;
        for (int64_t e = 0; e < tk.edges; ++e) {
          if (u[e] >= 0) continue;
          ids[next] = ~u[e];
          lut[~u[e]] = (int32_t)next++;   // this task's alone: no other reads or writes the entry in this pass
        }
      });
      tm.lap("number");
      int64_t *pes = es.p, *ped = es.p + ne, *peid = eid.p;
      for_tasks([&](SampleTask &tk, SampleSlice &sl) {
        const int32_t *lut = bd.local_of[ctx->rel_src[tk.r]].data(), *u = sl.src.p + tk.at;
        const int64_t *p = sl.pos.p + tk.at;
        int64_t e = 0, to = tk.first_edge, next = tk.first_fresh;
        for (int32_t i = tk.i0; i < tk.i1; ++i) {
          const int64_t row = tk.row + (i - tk.i0);
          ahead(lut, u, tk.edges, e, ecnt[row]);
          rp[row] = (int32_t)to;
          for (int c = 0; c < ecnt[row]; ++c, ++e, ++to) {
            pes[to] = u[e] < 0 ? next++ : lut[u[e]];
            ped[to] = i;
            peid[to] = p[e];
          }
        }
      });
      es.n = 2 * (size_t)ne;
      eid.n = (size_t)ne;
    }
    tm.lap("write");
    }
    // the lookup tables go back to "not in the hop"
    for (int t = 0; t < T; ++t) {
      job.n_src[l][t] = (int64_t)src[t].size();
      int32_t *lut = bd.local_of[t].data();
      split(src[t].size(), 4096, [&](size_t a, size_t b) {
        for (size_t i = a; i < b; ++i) lut[src[t][i]] = -1;
      });
    }
    std::swap(dst, src);
    tm.lap("reset");
  }
  if (st != HGNN_OK) return st;
  for (int t = 0; t < T; ++t) job.ids[t].assign(dst[t].begin(), dst[t].end());
  for (int l = 0; l < L; ++l) {
    hgnn_coo_layer &in = g->L[l].in;
    std::memset(&in, 0, sizeof(in));
    in.num_edges = (int64_t)job.edge_id[l].size();
    in.edge_index = job.edge_index[l].data();
    in.index_is_i64 = 1;
    in.edge_id = job.edge_id[l].data();
    in.n_src = job.n_src[l];
    in.n_dst = job.n_dst[l];
    in.transpose_types = job.transpose[l].empty() ? nullptr : job.transpose[l].data();
  }
  return HGNN_OK;
}

}  // namespace hgnn

using namespace hgnn;

hgnn_status hgnn_sampler_create(hgnn_ctx *ctx, const hgnn_host_graph *graph, hgnn_sampler **out) {
  if (!ctx || !graph || !out || !graph->num_nodes || !graph->in_indptr || !graph->in_nbr || !graph->edge_off)
    HGNN_FAIL(HGNN_EINVAL, "NULL argument");
  *out = nullptr;
  const int T = ctx->T, R = ctx->R;
  for (int t = 0; t < T; ++t)
    if (graph->num_nodes[t] < 0 || graph->num_nodes[t] > INT32_MAX)
      HGNN_FAIL(HGNN_EINVAL, "num_nodes[%d]=%lld outside [0, 2^31)", t, (long long)graph->num_nodes[t]);
  if (graph->edge_off[0] != 0) HGNN_FAIL(HGNN_EINVAL, "edge_off[0] must be 0");
  for (int r = 0; r < R; ++r) {
    const int64_t n = graph->num_nodes[ctx->rel_dst[r]], e = graph->edge_off[r + 1] - graph->edge_off[r];
    if (e < 0 || !graph->in_indptr[r] || (e > 0 && !graph->in_nbr[r])) HGNN_FAIL(HGNN_EINVAL, "relation %d: bad edge range or NULL arrays", r);
    const int64_t *p = graph->in_indptr[r];
    if (p[0] != 0 || p[n] != e) HGNN_FAIL(HGNN_EINVAL, "relation %d: in_indptr does not span its %lld edges", r, (long long)e);
    for (int64_t v = 0; v < n; ++v)
      if (p[v + 1] < p[v]) HGNN_FAIL(HGNN_EINVAL, "relation %d: in_indptr decreases at vertex %lld", r, (long long)v);
    const int64_t ns = graph->num_nodes[ctx->rel_src[r]];
    const int32_t *nb = graph->in_nbr[r];
    for (int64_t i = 0; i < e; ++i)
      if (nb[i] < 0 || nb[i] >= ns) HGNN_FAIL(HGNN_EINVAL, "relation %d: in_nbr[%lld]=%d outside its source type", r, (long long)i, nb[i]);
  }
  hgnn_sampler *s = new (std::nothrow) hgnn_sampler();
  if (!s) HGNN_FAIL(HGNN_ENOMEM, "out of host memory");
  s->num_nodes.assign(graph->num_nodes, graph->num_nodes + T);
  s->edge_off.assign(graph->edge_off, graph->edge_off + R + 1);
  s->in_indptr.assign(graph->in_indptr, graph->in_indptr + R);
  s->in_nbr.assign(graph->in_nbr, graph->in_nbr + R);
  // the edge-type table of Algorithm 2, in its compact form: edge ids of relation r are one contiguous range
  std::vector<uint8_t> types((size_t)s->edge_off[R]);
  for (int r = 0; r < R; ++r)
    std::memset(types.data() + s->edge_off[r], r, (size_t)(s->edge_off[r + 1] - s->edge_off[r]));
  ctx->edge_types8.swap(types);
  ++ctx->types_version;
  index_edge_type_runs(ctx);
  *out = s;
  return HGNN_OK;
}

void hgnn_sampler_destroy(hgnn_ctx *ctx, hgnn_sampler *s) {
  (void)ctx;
  delete s;
}
