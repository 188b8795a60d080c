// Host side of the semantic graph build (paper Section 4.3): edge-type matching and selection
// (Algorithm 2) fused with a stable parallel counting sort into one merged, relation-segmented
// CSR per layer, plus its transpose for the backward pass.  Integer work only.  The paper runs
// the selection with one OpenMP thread per relation; here the threads split the edge list
// instead (relations are very uneven in size), which yields the same arrays.
#include <pthread.h>

#include <algorithm>
#include <chrono>
#include <cstdlib>
#include <cstdarg>
#include <cstring>

#include "common.h"

namespace hgnn {

static thread_local char g_err[512] = "";
void set_error(const char *fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
}
const char *get_error() { return g_err; }

// ------------------------------------------------------------------------------------------
static std::atomic<Crew *> g_crew{nullptr};   // never destroyed: contexts may be released while the process's statics go

Crew &Crew::get() {
  Crew *c = g_crew.load(std::memory_order_acquire);
  if (!c) {
    static std::mutex making;
    // A forked child has none of its parent's threads, and the locks of the parent's crew as they stood: it starts afresh.
    // (Held across the fork, so that the child finds `making` free.)
    static const int hooked = pthread_atfork([] { making.lock(); }, [] { making.unlock(); }, [] {
      g_crew.store(nullptr, std::memory_order_relaxed);
      making.unlock();
    });
    (void)hooked;
    std::lock_guard<std::mutex> lk(making);
    c = g_crew.load(std::memory_order_relaxed);
    if (!c) g_crew.store(c = new Crew(), std::memory_order_release);
  }
  return *c;
}
void Crew::join(int threads, bool eager) {
  eager_.fetch_add(eager ? 1 : 0);
  std::lock_guard<std::mutex> lk(size_m_);
  sizes_.push_back(threads);
  const int most = *std::max_element(sizes_.begin(), sizes_.end());
  target_.store(most);
  while ((int)threads_.size() < most) threads_.emplace_back([this, i = (int)threads_.size()] { run(i); });
}
void Crew::leave(int threads, bool eager) {
  eager_.fetch_sub(eager ? 1 : 0);
  std::lock_guard<std::mutex> lk(size_m_);
  sizes_.erase(std::find(sizes_.begin(), sizes_.end(), threads));
  const int most = sizes_.empty() ? 0 : *std::max_element(sizes_.begin(), sizes_.end());
  target_.store(most);
  calls_.fetch_add(1);
  calls_.notify_all();
  while ((int)threads_.size() > most) {
    threads_.back().join();
    threads_.pop_back();
  }
}
static thread_local int tl_crew_index = 0;
int Crew::index() { return tl_crew_index; }
void Crew::drain(Job &j) {
  auto run_chunk = [&](int i) {
    try {
      (*j.fn)(i);
    } catch (...) {   // out of memory: the owner throws it on
      j.failed.store(true, std::memory_order_relaxed);
    }
    j.done.fetch_add(1, std::memory_order_release);
  };
  if (j.n > 64) {
    for (int i; (i = j.next.fetch_add(1, std::memory_order_relaxed)) < j.n;) run_chunk(i);
    return;
  }
  const int step = std::max(1, target_.load(std::memory_order_relaxed));
  auto take = [&](int i) {
    const uint64_t bit = (uint64_t)1 << i;
    if ((j.taken.load(std::memory_order_relaxed) & bit) || (j.taken.fetch_or(bit, std::memory_order_relaxed) & bit)) return;
    j.next.fetch_add(1, std::memory_order_relaxed);
    run_chunk(i);
  };
  for (int i = tl_crew_index; i < j.n; i += step) take(i);
  for (int k = 1; k <= j.n && j.next.load(std::memory_order_relaxed) < j.n; ++k) take((tl_crew_index + k) % j.n);
}
bool Crew::try_work() {
  if (active_.load(std::memory_order_relaxed) == 0) return false;
  bool did = false;
  for (Slot &s : slots_) {
    if (!s.job.load(std::memory_order_relaxed)) continue;
    s.users.fetch_add(1);            // before the job is read: its owner waits for users to drop once it is withdrawn
    if (Job *j = s.job.load()) {
      if (j->next.load(std::memory_order_relaxed) < j->n && j->joined.fetch_add(1) + 1 < j->width) {
        drain(*j);
        did = true;
      }
    }
    s.users.fetch_sub(1);
  }
  return did;
}
void Crew::run(int index) {
  tl_crew_index = index;
  auto idle = std::chrono::steady_clock::now();
  for (int spins = 0; index < target_.load(std::memory_order_relaxed);) {
    bool did = try_work();
    if (!did && waiting_tasks_.load(std::memory_order_relaxed) > 0) {
      std::function<void()> task;
      {
        std::lock_guard<std::mutex> lk(m_);
        if (!tasks_.empty()) {
          task = std::move(tasks_.front());
          tasks_.pop_front();
          waiting_tasks_.fetch_sub(1);
        }
      }
      if (task) {
        at_work_.fetch_add(1);
        task();
        idle_since_.store(std::chrono::steady_clock::now().time_since_epoch().count(), std::memory_order_relaxed);
        at_work_.fetch_sub(1);
        did = true;
      }
    }
    if (did) {
      idle = std::chrono::steady_clock::now();
      spins = 0;
      continue;
    }
    if (eager_.load(std::memory_order_relaxed) > 0) {
      cpu_relax();
      if (++spins % 64) continue;
      const auto idle_for = std::chrono::steady_clock::now() - idle;
      const int look_us = at_work_.load(std::memory_order_relaxed) > 0 ? kSpinUs : in_a_row_.load(std::memory_order_relaxed) ? kTailUs : 0;
      if (idle_for < std::chrono::microseconds(look_us)) continue;
    }
    // A sleeper looks once more after it has said so; work posted from there on changes the call it sleeps on.  No lock is
    // taken on the way out of the sleep: fifteen threads woken at once would pass it on one by one.
    const uint32_t call = calls_.load();
    sleepers_.fetch_add(1);
    if (index < target_.load() && active_.load() == 0 && waiting_tasks_.load() == 0) calls_.wait(call);
    sleepers_.fetch_sub(1);
    idle = std::chrono::steady_clock::now();
  }
}
void Crew::wake_all() {
  if (sleepers_.load() == 0) return;
  calls_.fetch_add(1);
  calls_.notify_all();
}
void Crew::submit(std::function<void()> task) {
  const int64_t idle_for = std::chrono::steady_clock::now().time_since_epoch().count() - idle_since_.load(std::memory_order_relaxed);
  in_a_row_.store(at_work_.load(std::memory_order_relaxed) > 0 || idle_for < (int64_t)kTailUs * 1000, std::memory_order_relaxed);
  {
    std::lock_guard<std::mutex> lk(m_);
    tasks_.push_back(std::move(task));
    waiting_tasks_.fetch_add(1);
  }
  if (eager_.load() > 0) {
    wake_all();   // the task's phases follow at once
  } else if (sleepers_.load() > 0) {
    calls_.fetch_add(1);
    calls_.notify_one();
  }
}
void Crew::parallel_for(int nchunks, int width, const std::function<void(int)> &fn) {
  Job j;
  j.fn = &fn;
  j.n = nchunks;
  j.width = width;
  Slot *mine = nullptr;
  for (Slot &s : slots_) {
    if (!s.taken.load(std::memory_order_relaxed) && !s.taken.exchange(true)) {
      mine = &s;
      mine->job.store(&j);
      break;
    }
  }
  if (mine) {
    active_.fetch_add(1);
    wake_all();
  }
  drain(j);
  auto wait = [](auto done) {   // the chunks still running are short, unless their thread lost its core
    for (int i = 0; !done(); ++i) {
      if (i < 20000) cpu_relax(); else std::this_thread::yield();
    }
  };
  wait([&] { return j.done.load(std::memory_order_acquire) >= nchunks; });
  if (mine) {
    active_.fetch_sub(1);
    mine->job.store(nullptr);
    wait([&] { return mine->users.load() == 0; });   // those still on their way out of this job: the slot takes no other before
    mine->taken.store(false);
  }
  if (j.failed.load(std::memory_order_relaxed)) throw std::bad_alloc();
}

// ------------------------------------------------------------------------------------------
namespace {

struct BuildError {
  std::mutex m;
  int status = HGNN_OK;
  std::string msg;
  std::atomic<bool> failed{false};
  void set(int st, const std::string &s) {
    std::lock_guard<std::mutex> lk(m);
    if (status == HGNN_OK) {
      status = st;
      msg = s;
      failed.store(true);
    }
  }
};

// At most 4096 consecutive keys form one bucket (its counters stay in L1); fewer where that makes too few buckets for
// the threads.
constexpr int kBucketShift = 12;
inline int bucket_shift(int64_t keys, int threads) {
  int s = kBucketShift;
  while (s > 7 && threads > 1 && (keys >> s) < 3 * threads) --s;
  return s;
}

}  // namespace

// Two-level stable counting sort, used twice per layer (edges by merged row; CSR positions by source
// row).  Level 1 splits the items into key-range buckets (threads own contiguous item slices, so the
// order inside a bucket is the input order); level 2 sorts every bucket on its own with a local
// histogram and writes the final arrays and the bucket's part of the row pointer.
// A level-1 record carries (key, item, payload).  Wide: three ints.  Packed: two ints -- only the key's offset
// inside its bucket is needed once the record lies in the bucket, and it fits above the payload when the
// payload stays below 2^(32 - kBucketShift): a third less to write, to fetch for ownership and to read back.
struct WideRec {
  static constexpr int W = 3;
  static void put(int32_t *r, int32_t key, int32_t item, int32_t payload) { r[0] = key; r[1] = item; r[2] = payload; }
  static int32_t key_low(const int32_t *r) { return r[0]; }
  static int32_t base(int32_t k0) { return k0; }   // key_low of the bucket's first key
  static int32_t item(const int32_t *r) { return r[1]; }
  static int32_t payload(const int32_t *r) { return r[2]; }
};
struct PackedRec {
  static constexpr int W = 2, kPayloadBits = 32 - kBucketShift;
  static void put(int32_t *r, int32_t key, int32_t item, int32_t payload) {
    r[0] = item;
    r[1] = (int32_t)(((uint32_t)key << kPayloadBits) | (uint32_t)payload);  // the shift drops the bucket's bits
  }
  static int32_t key_low(const int32_t *r) { return (int32_t)((uint32_t)r[1] >> kPayloadBits); }
  static int32_t base(int32_t k0) { return k0 & ((1 << kBucketShift) - 1); }
  static int32_t item(const int32_t *r) { return r[0]; }
  static int32_t payload(const int32_t *r) { return (int32_t)((uint32_t)r[1] & ((1u << kPayloadBits) - 1u)); }
};

// One int: for builds that leave the permutation out, the item is not carried at all.
struct SlimRec {
  static constexpr int W = 1, kPayloadBits = 32 - kBucketShift;
  static void put(int32_t *r, int32_t key, int32_t, int32_t payload) {
    r[0] = (int32_t)(((uint32_t)key << kPayloadBits) | (uint32_t)payload);
  }
  static int32_t key_low(const int32_t *r) { return (int32_t)((uint32_t)r[0] >> kPayloadBits); }
  static int32_t base(int32_t k0) { return k0 & ((1 << kBucketShift) - 1); }
  static int32_t item(const int32_t *) { return 0; }
  static int32_t payload(const int32_t *r) { return (int32_t)((uint32_t)r[0] & ((1u << kPayloadBits) - 1u)); }
};

static bool build_layer(hgnn_ctx *ctx, ThreadPool &pool, LayerScratch &bd, hgnn_graph *g, int l, BuildError &err) {
  PhaseTimer tm;
  LayerHost &L = g->L[l];
  const hgnn_coo_layer &in = L.in;
  const int T = ctx->T, R = ctx->R;
  int32_t *base = g->slab.host;
  int32_t *rel_row_off = base + L.o_rel_row_off, *rel_edge_off = base + L.o_rel_edge_off;
  int32_t *rowptr = base + L.o_rowptr, *colidx = base + L.o_colidx, *perm = base + L.o_perm;
  int32_t *cptr = base + L.o_cptr, *crow = base + L.o_crow, *cperm = base + L.o_cperm;
  int32_t row_off[kMaxT + 1];
  row_off[0] = 0;
  for (int t = 0; t < T; ++t) row_off[t + 1] = row_off[t] + (int32_t)L.n_src[t];
  rel_row_off[0] = 0;
  for (int r = 0; r < R; ++r) rel_row_off[r + 1] = rel_row_off[r] + (int32_t)L.n_dst[ctx->rel_dst[r]];
  const int64_t E = L.edges, rows = L.rows, src_rows = L.src_rows;
  const int P = (int)std::max<int64_t>(1, std::min<int64_t>(pool.size(), (E + 4095) / 4096));
  const int sh1 = bucket_shift(rows, P), sh2 = bucket_shift(src_rows, P);
  const int B1 = (int)((rows + (1 << sh1) - 1) >> sh1);
  const int B2 = (int)((src_rows + (1 << sh2) - 1) >> sh2);
  auto grow = [](std::vector<int32_t> &v, size_t n) {
    if (v.size() < n) v.resize(n + n / 4);
  };
  grow(bd.key, (size_t)E);
  grow(bd.col, (size_t)E);
  grow(bd.tkey, (size_t)E * 3);  // level-1 records: (key, item, payload)
  // counter rows are padded to whole 128-byte lines: neighbouring threads must not share a line
  const size_t S1 = ((size_t)B1 + 63) / 32 * 32, S2 = ((size_t)B2 + 63) / 32 * 32;
  grow(bd.hist, (size_t)P * S1 + (size_t)std::max(B1, 1) * S2 + B1 + B2 + 2 + 64);
  int32_t *key = bd.key.data(), *col = bd.col.data();
  int32_t *trec = bd.tkey.data();
  int32_t *cnt1 = reinterpret_cast<int32_t *>((reinterpret_cast<uintptr_t>(bd.hist.data()) + 127) & ~(uintptr_t)127);  // [P][S1]
  int32_t *cnt2 = cnt1 + (size_t)P * S1;                     // [B1][S2]
  int32_t *base1 = cnt2 + (size_t)std::max(B1, 1) * S2;      // [B1+1]
  int32_t *base2 = base1 + B1 + 1;                           // [B2+1]
  std::memset(cnt1, 0, sizeof(int32_t) * (size_t)P * S1);
  std::memset(cnt2, 0, sizeof(int32_t) * (size_t)std::max(B1, 1) * S2);
  tm.lap("setup");

  // A mini-batch drawn by the library's own sampler arrives relation by relation, destinations ascending, and
  // its edges were read off the graph: there is nothing to look up, check or sort -- the merged CSR is the input
  // order itself.
  // (a test can ask for the three-int records where the two-int ones would do)
  static const bool wide_records = getenv("HGNN_WIDE_RECORDS") != nullptr;
  const bool csc_packed = rows <= (int64_t)1 << PackedRec::kPayloadBits && !wide_records;
  const bool presorted = g->job != nullptr;
  const bool with_perm = g->with_perm;
  if (presorted) {
    const SampleJob &job = *g->job;
    const int64_t *es = job.edge_index[l].data();
    const int32_t *rp = job.row_ptr[l].data();
    // slices of merged rows (relations differ in size), cut at relation boundaries inside a slice
    pool.parallel_for(P, [&](int p) {
      const int64_t ra = rows * p / P, rb = rows * (p + 1) / P;
      std::memcpy(rowptr + ra, rp + ra, sizeof(int32_t) * (size_t)(rb - ra));
      for (int r = 0; r < R; ++r) {
        const int64_t a = std::max<int64_t>(ra, rel_row_off[r]), b = std::min<int64_t>(rb, rel_row_off[r + 1]);
        if (a >= b) continue;
        const int32_t col0 = row_off[ctx->rel_src[r]];
        for (int32_t e = rp[a]; e < rp[b]; ++e) {
          colidx[e] = col0 + (int32_t)es[e];
          if (with_perm) perm[e] = e;
        }
      }
    });
    for (int b = 0; b <= B1; ++b) base1[b] = b < B1 ? rp[(size_t)b << sh1] : (int32_t)E;
    tm.lap("csr from sampler order");
  } else {
  // Algorithm 2: the layer's edge types are looked up through the edge ids (or taken as given) and matched
  // against the relations -- for all relations in one pass: each edge gets its merged row and source row.
  const int64_t slice = (E + P - 1) / P;
  const int64_t *ei64 = in.index_is_i64 ? (const int64_t *)in.edge_index : nullptr;
  const int32_t *ei32 = in.index_is_i64 ? nullptr : (const int32_t *)in.edge_index;
  const uint8_t *types8 = ctx->edge_types8.data();
  const int64_t n_types8 = (int64_t)ctx->edge_types8.size();
  const int nruns = (int)ctx->run_end.size();
  const int64_t *run_end = ctx->run_end.data();
  const uint8_t *run_rel = ctx->run_rel.data(), *run_lut = ctx->run_lut.data();
  const int run_shift = ctx->run_shift;
  // Reports the first bad edge of [a, b).
  auto report = [&](int64_t a, int64_t b) {
    for (int64_t e = a; e < b; ++e) {
      int64_t r;
      if (in.edge_type) {
        r = in.edge_type[e];
      } else if (!in.global_edge_type && nruns > 0) {   // the registered table, as runs of equal type
        const int64_t id = in.edge_id[e];
        if (id < 0 || id >= n_types8) {
          err.set(HGNN_EINVAL, "layer " + std::to_string(l) + ": edge_id[" + std::to_string(e) + "]=" +
                                   std::to_string(id) + " outside the registered edge-type table");
          return;
        }
        int j = run_lut[id >> run_shift];
        while (id >= run_end[j]) ++j;  // ends: id < n_types8 = the last run's end
        r = run_rel[j];
      } else if (!in.global_edge_type) {   // the registered compact table
        const int64_t id = in.edge_id[e];
        if (id < 0 || id >= n_types8) {
          err.set(HGNN_EINVAL, "layer " + std::to_string(l) + ": edge_id[" + std::to_string(e) + "]=" +
                                   std::to_string(id) + " outside the registered edge-type table");
          return;
        }
        r = types8[id];
      } else {
        const int64_t id = in.edge_id[e];
        if (id < 0 || id >= in.num_global_edges) {
          err.set(HGNN_EINVAL, "layer " + std::to_string(l) + ": edge_id[" + std::to_string(e) + "]=" +
                                   std::to_string(id) + " outside the global edge-type table");
          return;
        }
        r = in.global_edge_type[id];
      }
      if (r < 0 || r >= R) {
        err.set(HGNN_EINVAL, "layer " + std::to_string(l) + ": edge " + std::to_string(e) + " has type " +
                                 std::to_string(r) + " outside [0," + std::to_string(R) + ")");
        return;
      }
      const int64_t s = ei64 ? ei64[e] : (int64_t)ei32[e];
      const int64_t d = ei64 ? ei64[E + e] : (int64_t)ei32[E + e];
      const int ts = ctx->rel_src[r], td = ctx->rel_dst[r];
      if (s < 0 || s >= L.n_src[ts] || d < 0 || d >= L.n_dst[td]) {
        err.set(HGNN_EINVAL, "layer " + std::to_string(l) + ": edge " + std::to_string(e) + " (" +
                                 std::to_string(s) + "->" + std::to_string(d) + ", relation " +
                                 std::to_string(r) + ") outside its source/destination row range");
        return;
      }
    }
  };
  // What an edge of relation r becomes; one record per relation, so that an edge costs one look-up.
  struct RelRec {
    int32_t row, col;
    uint32_t n_src, n_dst;
  } rec[kMaxR];
  for (int r = 0; r < R; ++r) {
    const int ts = ctx->rel_src[r];
    rec[r] = RelRec{rel_row_off[r], row_off[ts], (uint32_t)L.n_src[ts], (uint32_t)L.n_dst[ctx->rel_dst[r]]};
  }
  // The loop does not leave early: a bad edge is noted, takes row 0, and is looked for afterwards.
  auto select = [&](int p, auto type_of, auto index) {
    const int64_t a = std::min<int64_t>(E, p * slice), b = std::min<int64_t>(E, a + slice);
    int32_t *cnt = cnt1 + (size_t)p * S1;
    const auto *src = index, *dst = index + E;
    bool bad = false;
    for (int64_t e = a; e < b; ++e) {
      const uint64_t r = type_of(e, b);
      const bool known = r < (uint64_t)R;
      const RelRec q = rec[known ? r : 0];
      const uint64_t s = (uint64_t)src[e], d = (uint64_t)dst[e];
      const bool ok = known & (s < q.n_src) & (d < q.n_dst);
      bad |= !ok;
      const int32_t k = ok ? q.row + (int32_t)d : 0;
      key[e] = k;
      col[e] = q.col + (int32_t)s;
      ++cnt[k >> sh1];
    }
    if (bad) report(a, b);
  };
  auto select_by = [&](auto type_of) {
    pool.parallel_for(P, [&](int p) {
      if (ei64) select(p, type_of, ei64); else select(p, type_of, ei32);
    });
  };
  constexpr uint64_t kNone = ~(uint64_t)0;   // no relation: an id outside its table
  if (in.edge_type) {
    select_by([&](int64_t e, int64_t) { return (uint64_t)(int64_t)in.edge_type[e]; });
  } else if (!in.global_edge_type && nruns > 0) {   // the registered table, as runs of equal type
    select_by([&](int64_t e, int64_t) {
      const int64_t id = in.edge_id[e];
      if ((uint64_t)id >= (uint64_t)n_types8) return kNone;
      int j = run_lut[id >> run_shift];
      while (id >= run_end[j]) ++j;  // ends: id < n_types8 = the last run's end
      return (uint64_t)run_rel[j];
    });
  } else if (!in.global_edge_type) {   // the registered compact table
    select_by([&](int64_t e, int64_t b) {
      if (e + 48 < b) {
        const int64_t nid = in.edge_id[e + 48];
        if (nid >= 0 && nid < n_types8) __builtin_prefetch(types8 + nid);
      }
      const int64_t id = in.edge_id[e];
      return (uint64_t)id < (uint64_t)n_types8 ? (uint64_t)types8[id] : kNone;
    });
  } else {
    select_by([&](int64_t e, int64_t b) {
      if (e + 48 < b) {
        const int64_t nid = in.edge_id[e + 48];
        if (nid >= 0 && nid < in.num_global_edges) __builtin_prefetch(in.global_edge_type + nid);
      }
      const int64_t id = in.edge_id[e];
      return (uint64_t)id < (uint64_t)in.num_global_edges ? (uint64_t)(int64_t)in.global_edge_type[id] : kNone;
    });
  }
  if (err.failed.load()) return false;
  tm.lap("select (Alg.2) + count");

  // ---- merged CSR: stable by (relation, destination) ----
  {
    int32_t run = 0;
    for (int b = 0; b < B1; ++b) {
      base1[b] = run;
      for (int p = 0; p < P; ++p) {
        const int32_t t = cnt1[(size_t)p * S1 + b];
        cnt1[(size_t)p * S1 + b] = run;
        run += t;
      }
    }
    base1[B1] = run;
  }
  auto csr_sort = [&](auto rec_format, auto perm_flag) {
    using Rec = decltype(rec_format);
    constexpr bool kPerm = decltype(perm_flag)::value;
    pool.parallel_for(P, [&](int p) {
      const int64_t a = std::min<int64_t>(E, p * slice), b = std::min<int64_t>(E, a + slice);
      int32_t *off = cnt1 + (size_t)p * S1;
      for (int64_t e = a; e < b; ++e) {
        const int32_t q = off[key[e] >> sh1]++;
        Rec::put(trec + (size_t)q * Rec::W, key[e], (int32_t)e, col[e]);
      }
    });
    tm.lap("csr level-1 scatter");
    pool.parallel_for(B1, [&](int b) {
      int32_t h[(1 << kBucketShift) + 1];
      const int32_t k0 = b << sh1;
      const int32_t nk = (int32_t)std::min<int64_t>(1 << sh1, rows - k0);
      std::memset(h, 0, sizeof(int32_t) * (nk + 1));
      int32_t *const hk = h - Rec::base(k0);
      const int32_t ja = base1[b], jb = base1[b + 1];
      for (int32_t j = ja; j < jb; ++j) ++hk[Rec::key_low(trec + (size_t)j * Rec::W)];
      int32_t run = ja;
      for (int32_t i = 0; i < nk; ++i) {
        const int32_t t = h[i];
        h[i] = run;
        rowptr[k0 + i] = run;
        run += t;
      }
      for (int32_t j = ja; j < jb; ++j) {
        const int32_t *rec = trec + (size_t)j * Rec::W;
        const int32_t pos = hk[Rec::key_low(rec)]++;
        colidx[pos] = Rec::payload(rec);
        if constexpr (kPerm) perm[pos] = Rec::item(rec);
      }
    });
    tm.lap("csr level-2 buckets");
  };
  const bool fits = src_rows <= (int64_t)1 << PackedRec::kPayloadBits && !wide_records;
  if (with_perm) {
    if (fits) csr_sort(PackedRec(), std::true_type());
    else csr_sort(WideRec(), std::true_type());
  } else {
    if (fits) csr_sort(SlimRec(), std::false_type());
    else csr_sort(WideRec(), std::false_type());
  }
  }
  rowptr[rows] = (int32_t)E;
  for (int r = 0; r <= R; ++r) rel_edge_off[r] = rowptr[rel_row_off[r]];

  // All sources of a relation have one type, and the CSR is ordered by relation: the positions whose source row
  // is wanted are whole relation ranges, so the others are skipped without being read.
  int n_pr = 0;
  int32_t pr_lo[kMaxR], pr_hi[kMaxR];
  for (int r = 0; r < R; ++r) {
    if (!((L.tmask >> ctx->rel_src[r]) & 1u) || rel_edge_off[r + 1] == rel_edge_off[r]) continue;
    if (n_pr > 0 && pr_hi[n_pr - 1] == rel_edge_off[r]) pr_hi[n_pr - 1] = rel_edge_off[r + 1];
    else { pr_lo[n_pr] = rel_edge_off[r]; pr_hi[n_pr] = rel_edge_off[r + 1]; ++n_pr; }
  }
  // level-1 counts of the transpose: per CSR bucket, how many of its wanted positions fall into each bucket of
  // source rows (a sweep of its own over the wanted ranges: inside the scatter loop above the test "is this
  // source row wanted" is a coin flip for the branch predictor and cost more than the whole sweep)
  pool.parallel_for(B1, [&](int b1) {
    int32_t *c2 = cnt2 + (size_t)b1 * S2;
    for (int i = 0; i < n_pr; ++i) {
      const int32_t ka = std::max(base1[b1], pr_lo[i]), kb = std::min(base1[b1 + 1], pr_hi[i]);
      for (int32_t k = ka; k < kb; ++k) ++c2[colidx[k] >> sh2];
    }
  });
  // ---- transpose: CSR positions grouped by source row, ascending position inside a group ----
  // the level-1 slices are the CSR position ranges of the buckets above (already in CSR order)
  {
    int32_t run = 0;
    for (int b2 = 0; b2 < B2; ++b2) {
      base2[b2] = run;
      for (int b1 = 0; b1 < B1; ++b1) {
        const int32_t t = cnt2[(size_t)b1 * S2 + b2];
        cnt2[(size_t)b1 * S2 + b2] = run;
        run += t;
      }
    }
    base2[B2] = run;
  }
  pool.parallel_for(B1, [&](int b1) {
    int32_t *off = cnt2 + (size_t)b1 * S2;
    for (int i = 0; i < n_pr; ++i) {
      const int32_t ka = std::max(base1[b1], pr_lo[i]), kb = std::min(base1[b1 + 1], pr_hi[i]);
      if (ka >= kb) continue;
      // the merged row of CSR position k: positions are walked in order, so the row pointer is walked along
      int32_t row = b1 << sh1;
      {  // first row of the bucket that ends after ka
        int32_t hi = (int32_t)std::min<int64_t>(rows, (int64_t)(b1 + 1) << sh1);
        while (row + 1 < hi) {
          const int32_t mid = row + (hi - row) / 2;
          if (rowptr[mid] <= ka) row = mid; else hi = mid;
        }
      }
      for (int32_t k = ka; k < kb; ++k) {
        while (rowptr[row + 1] <= k) ++row;
        const int32_t c = colidx[k];
        const int32_t q = off[c >> sh2]++;
        if (!csc_packed) WideRec::put(trec + (size_t)q * WideRec::W, c, k, row);
        else if (with_perm) PackedRec::put(trec + (size_t)q * PackedRec::W, c, k, row);
        else SlimRec::put(trec + q, c, k, row);
      }
    }
  });
  tm.lap("csc level-1 scatter");
  std::vector<std::vector<int32_t>> &longs = bd.long_lists;
  if ((int)longs.size() < B2) longs.resize(B2);
  auto csc_level2 = [&](auto rec_format, auto perm_flag) {
    using Rec = decltype(rec_format);
    constexpr bool kPerm = decltype(perm_flag)::value;
    pool.parallel_for(B2, [&](int b) {
      int32_t h[(1 << kBucketShift) + 1];
      const int32_t k0 = b << sh2;
      const int32_t nk = (int32_t)std::min<int64_t>(1 << sh2, src_rows - k0);
      std::memset(h, 0, sizeof(int32_t) * (nk + 1));
      int32_t *const hk = h - Rec::base(k0);
      const int32_t ja = base2[b], jb = base2[b + 1];
      for (int32_t j = ja; j < jb; ++j) ++hk[Rec::key_low(trec + (size_t)j * Rec::W)];
      int32_t run = ja;
      longs[b].clear();
      for (int32_t i = 0; i < nk; ++i) {
        const int32_t t = h[i];
        if (t > kLongRow) longs[b].push_back(k0 + i);
        h[i] = run;
        cptr[k0 + i] = run;
        run += t;
      }
      for (int32_t j = ja; j < jb; ++j) {
        const int32_t *rec = trec + (size_t)j * Rec::W;
        const int32_t pos = hk[Rec::key_low(rec)]++;
        crow[pos] = Rec::payload(rec);
        if constexpr (kPerm) cperm[pos] = Rec::item(rec);
      }
    });
  };
  if (with_perm) {
    if (csc_packed) csc_level2(PackedRec(), std::true_type());
    else csc_level2(WideRec(), std::true_type());
  } else {
    if (csc_packed) csc_level2(SlimRec(), std::false_type());
    else csc_level2(WideRec(), std::false_type());
  }
  cptr[src_rows] = base2[B2];
  L.tedges = base2[B2];
  tm.lap("csc level-2 buckets");

  // long transpose rows are cut into chunks so that no single block walks thousands of edges
  int32_t *chunk_row = base + L.o_chunk_row, *chunk_beg = base + L.o_chunk_beg;
  int32_t nc = 0;
  for (int b = 0; b < B2; ++b)
    for (int32_t c : longs[b]) {
      for (int32_t q = cptr[c]; q < cptr[c + 1]; q += kChunk) {
        chunk_row[nc] = c;
        chunk_beg[nc] = q;
        ++nc;
      }
    }
  L.n_chunks = nc;
  tm.lap("long-row chunks");
  return true;
}

// Samples (where asked for), plans and builds; false: `err` or the first failed layer's error says why.
static bool sample_and_build(hgnn_ctx *ctx, Builder &bd, hgnn_graph *g, BuildError &err, BuildError *layer_err, PhaseTimer &tm) {
  if (g->job) {  // sample first; only then are the sizes known that the block is laid out for
    std::string m;
    hgnn_status st = run_sample_job(ctx, bd, g, m);
    if (st == HGNN_OK) {
      {
        std::lock_guard<std::mutex> lk(g->m);
        g->sampled = true;
      }
      g->cv.notify_all();
      st = plan_graph(ctx, g, m);
    }
    tm.lap("sample and plan");
    if (st != HGNN_OK) {
      err.set(st, m);
      return false;
    }
    for (int t = 0; t < ctx->T; ++t) {
      const std::vector<int64_t> &ids = g->job->ids[t];
      const int n = (int)std::min<size_t>((size_t)bd.pool->size(), (ids.size() + 8191) / 8192);
      bd.pool->parallel_for(n, [&](int i) {
        const size_t a = ids.size() * i / n, b = ids.size() * (i + 1) / n;
        std::memcpy(g->slab.host + g->o_ids[t] + 2 * a, ids.data() + a, (b - a) * sizeof(int64_t));
      });
    }
  }
  // the layers side by side: a small layer's phases are shorter than what it takes to start them
  bd.pool->parallel_for(g->num_layers, [&](int l) { (void)build_layer(ctx, *bd.pool, bd.layer[l], g, l, layer_err[l]); });
  bool ok = true;
  for (int l = 0; l < g->num_layers; ++l) ok = ok && !layer_err[l].failed.load();
  tm.lap("all layers");
  return ok;
}

void build_graph_job(hgnn_ctx *ctx, Builder &bd, hgnn_graph *g) {
  BuildError err, layer_err[kMaxLayers];
  bool ok = false;
  PhaseTimer tm;
  try {
    ok = sample_and_build(ctx, bd, g, err, layer_err, tm);
  } catch (const std::exception &) {   // a scratch array that could not grow
    err.set(HGNN_ENOMEM, "out of host memory");
    for (std::vector<int32_t> &t : bd.local_of) t.clear();   // the sampler may have left marks: it makes them anew
  }
  const BuildError *first = &err;   // of several bad layers the first is reported, whichever was done first
  for (int l = 0; l < g->num_layers && !first->failed.load(); ++l) first = &layer_err[l];
  int status = ok ? HGNN_OK : first->status;
  std::string msg = first->msg;
  if (ok && ctx->device >= 0) {
    hipError_t e = hipMemcpyAsync(g->slab.dev, g->slab.host, g->used * sizeof(int32_t), hipMemcpyHostToDevice, ctx->side);
    if (e == hipSuccess) e = hipEventRecord(g->ready, ctx->side);
    if (e != hipSuccess) {
      status = HGNN_EHIP;
      msg = std::string("graph upload: ") + hipGetErrorString(e);
    }
  }
  tm.lap("start of the upload");
  {
    // notified under the lock: a waiter may release (delete) the graph as soon as it sees the new state, so the
    // unlock must be this thread's last touch of it
    std::lock_guard<std::mutex> lk(g->m);
    g->status = status;
    g->err = msg;
    g->state = (status == HGNN_OK) ? 1 : 2;
    g->cv.notify_all();
  }
}

}  // namespace hgnn
