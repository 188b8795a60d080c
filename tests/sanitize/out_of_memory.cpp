// Allocations that fail on the host threads while a mini-batch is sampled and built: the graph's status says so, and the
// same context works when memory is there again.
#include <cstring>
#include <new>

#include "common.h"

static std::atomic<size_t> most{~(size_t)0};   // larger allocations fail, except the calling thread's
static thread_local bool calling = false;
void *operator new(size_t n) {
  if (calling || n <= most.load())
    if (void *p = malloc(n)) return p;
  throw std::bad_alloc();
}
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }

#define CHECK(c) if (!(c)) { printf("line %d: %s: %s\n", __LINE__, #c, hgnn_last_error()); return 1; }

int main() {
  calling = true;
  constexpr int N = 20000, E = 100000;
  std::vector<int64_t> indptr(N + 1), index(2 * E), targets(N);
  std::vector<int32_t> nbr(E), type(E, 0);
  for (int v = 0; v <= N; ++v) indptr[v] = (int64_t)v * E / N;
  for (int e = 0; e < E; ++e) index[e] = nbr[e] = (int)((int64_t)e * 7919 % N), index[E + e] = e % N;
  for (int v = 0; v < N; ++v) targets[v] = v;
  const int32_t zero = 0, fan = 4;
  const int64_t n = N, off[2] = {0, E}, *ip[1] = {indptr.data()};
  const int32_t *nb[1] = {nbr.data()};
  const hgnn_schema schema = {1, 1, &zero, &zero, 1, HGNN_AGG_MEAN, HGNN_FUSE_SUM, HGNN_F32};
  const hgnn_host_graph hg = {&n, ip, nb, off};
  hgnn_coo_layer layer;
  memset(&layer, 0, sizeof(layer));
  layer.num_edges = E;
  layer.edge_index = index.data();
  layer.index_is_i64 = 1;
  layer.edge_type = type.data();
  layer.n_src = layer.n_dst = &n;
  for (int threads : {1, 6})
    for (bool sampled : {false, true}) {
      hgnn_ctx *ctx;
      hgnn_sampler *s;
      CHECK(hgnn_create(&ctx, &schema, -1, threads, 1) == HGNN_OK)
      CHECK(hgnn_sampler_create(ctx, &hg, &s) == HGNN_OK)
      int refused = 0;
      // the scratch starts empty and grows as far as the limit lets it
      for (size_t limit : {(size_t)1 << 10, (size_t)1 << 15, (size_t)90000, (size_t)200000, (size_t)450000, ~(size_t)0}) {
        hgnn_graph *g;
        most = limit;
        CHECK((sampled ? hgnn_sample_and_build(ctx, s, 0, targets.data(), N, 1, &fan, 3, nullptr, &g)
                       : hgnn_build_semantic_csr(ctx, 1, &layer, &g)) == HGNN_OK)
        const hgnn_status st = hgnn_graph_wait(ctx, g);
        CHECK(st == HGNN_OK || st == HGNN_ENOMEM)
        refused += st == HGNN_ENOMEM;
        if (limit == ~(size_t)0) {
          hgnn_csr_view v;
          CHECK(st == HGNN_OK && hgnn_graph_host_view(ctx, g, 0, &v) == HGNN_OK && v.rows == N && v.rowptr[N] == v.edges)
        }
        hgnn_graph_release(ctx, g);
      }
      printf("%d threads, sampled %d: %d of 5 refused\n", threads, (int)sampled, refused);
      CHECK(refused >= 3)
      hgnn_sampler_destroy(ctx, s);
      hgnn_destroy(ctx);
    }
  printf("out of memory ok\n");
  return 0;
}
