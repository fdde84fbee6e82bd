// Scenarios over the library's host code (loads, whole-graph and per-seed
// calls, three events, top-k, batches) on the test doubles of host_stub.h,
// built with AddressSanitizer and UndefinedBehaviorSanitizer by
// tests/test_host_orchestration.py. argv[1] names the scenario; prints "ok" and
// exits 0 when it passes.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <random>
#include <string>
#include <vector>

#include "ef_internal.h"
#include "host_stub.h"

static int g_failed = 0;
#define CHECK(c)                                             \
  do {                                                       \
    if (!(c)) {                                              \
      std::printf("%s:%d: %s (last error: %s)\n", __FILE__, __LINE__, #c, ef_last_error()); \
      ++g_failed;                                            \
    }                                                        \
  } while (0)

struct Csr {
  std::vector<int32_t> rp{0}, ci;
  int32_t n() const { return (int32_t)rp.size() - 1; }
  int64_t nnz() const { return (int64_t)ci.size(); }
};

static Csr from_edges(int32_t n, const std::vector<std::pair<int32_t, int32_t>> &edges) {
  std::vector<std::vector<int32_t>> adj((size_t)n);
  for (auto &e : edges)
    if (e.first != e.second) {
      adj[(size_t)e.first].push_back(e.second);
      adj[(size_t)e.second].push_back(e.first);
    }
  Csr g;
  for (auto &a : adj) {
    std::sort(a.begin(), a.end());
    a.erase(std::unique(a.begin(), a.end()), a.end());
    g.ci.insert(g.ci.end(), a.begin(), a.end());
    g.rp.push_back((int32_t)g.ci.size());
  }
  return g;
}

// n nodes, each joined to m earlier ones, mostly to the first few: hubs,
// triangles and leaves
static Csr hubby(int32_t n, int32_t m, uint32_t seed) {
  std::mt19937 r(seed);
  std::vector<std::pair<int32_t, int32_t>> e;
  for (int32_t v = 1; v < n; ++v)
    for (int32_t j = 0; j < m; ++j) {
      const uint32_t cap = r() % 3 ? (uint32_t)v : std::min<uint32_t>((uint32_t)v, 4);
      e.push_back({v, (int32_t)(r() % cap)});
    }
  return from_edges(n, e);
}
static Csr ring(int32_t n, int32_t k) {  // each node joined to the k / 2 nearest on both sides
  std::vector<std::pair<int32_t, int32_t>> e;
  for (int32_t v = 0; v < n; ++v)
    for (int32_t j = 1; j <= k / 2; ++j) e.push_back({v, (v + j) % n});
  return from_edges(n, e);
}
static Csr complete(int32_t n) {
  Csr g;
  for (int32_t v = 0; v < n; ++v) {
    for (int32_t u = 0; u < n; ++u)
      if (u != v) g.ci.push_back(u);
    g.rp.push_back((int32_t)g.ci.size());
  }
  return g;
}

static ef_graph *load(const Csr &g, uint32_t flags = 0) {
  ef_graph *h = nullptr;
  const ef_status s = ef_graph_load_csr(g.n(), g.nnz(), g.rp.data(), g.ci.data(), flags, nullptr, &h);
  return s == EF_OK ? h : nullptr;
}

struct Out {
  std::vector<double> ef;
  std::vector<int64_t> D, N;
  size_t n;
  explicit Out(size_t count)
      : ef(std::max<size_t>(count, 1)), D(ef.size()), N(ef.size()), n(count) {}
};
// outputs on the device
struct DeviceOut {
  double *ef = nullptr;
  int64_t *D = nullptr, *N = nullptr;
  size_t n;
  explicit DeviceOut(size_t count) : n(count) {
    (void)hipMalloc(&ef, 8 * n);
    (void)hipMalloc(&D, 8 * n);
    (void)hipMalloc(&N, 8 * n);
  }
  ~DeviceOut() {
    (void)hipFree(ef);
    (void)hipFree(D);
    (void)hipFree(N);
  }
  ef_status call(ef_graph *h, ef_algo algo, ef_prec p, hipStream_t st) const {
    return ef_compute(h, algo, p, nullptr, 0, ef, D, N, EF_OUT_DEVICE, st);
  }
  void clear() { std::memset(ef, 0, 8 * n); }
  bool expected() const {
    for (size_t v = 0; v < n; ++v)
      if (ef[v] != (double)v + 0.5 || D[v] != 3 * (int64_t)v) return false;
    return true;
  }
};
static bool expected(const Out &o, const std::vector<int32_t> *seeds) {
  for (size_t i = 0; i < o.n; ++i) {
    const int32_t v = seeds ? (*seeds)[i] : (int32_t)i;
    if (o.ef[i] != v + 0.5 || o.D[i] != 3 * (int64_t)v || o.N[i] != 7 * (int64_t)v) return false;
  }
  return true;
}
// a whole-graph call with host outputs
static ef_status whole(ef_graph *h, ef_algo algo, ef_prec p) {
  Out o((size_t)h->g.n);
  const ef_status s = ef_compute(h, algo, p, nullptr, 0, o.ef.data(), o.D.data(), o.N.data(), 0,
                                 nullptr);
  if (s == EF_OK) CHECK(expected(o, nullptr));
  return s;
}
static ef_status some(ef_graph *h, ef_prec p, const std::vector<int32_t> &seeds, bool j3 = false) {
  Out o(seeds.size());
  const ef_status s =
      j3 ? ef_compute_j3(h, p, seeds.data(), (int32_t)seeds.size(), o.ef.data(), o.D.data(),
                         o.N.data(), 0, nullptr)
         : ef_compute(h, EF_ALGO_PER_SEED, p, seeds.data(), (int32_t)seeds.size(), o.ef.data(),
                      o.D.data(), o.N.data(), 0, nullptr);
  if (s == EF_OK) CHECK(expected(o, &seeds));
  return s;
}
static ef_status whole_j3(ef_graph *h, ef_prec p) {
  Out o((size_t)h->g.n);
  const ef_status s = ef_compute_j3(h, p, nullptr, 0, o.ef.data(), o.D.data(), o.N.data(), 0, nullptr);
  if (s == EF_OK) CHECK(expected(o, nullptr));
  return s;
}

// every kind of call on graphs of all sizes, outputs on the host
static void calls() {
  const Csr graphs[] = {from_edges(1, {}),  from_edges(7, {}),   from_edges(2, {{0, 1}}),
                        complete(5),        hubby(300, 3, 1),    hubby(3000, 6, 2),
                        hubby(20000, 4, 3), complete(90),        ring(1000, 6),
                        complete(1300)};
  for (const Csr &c : graphs) {
    ef_graph *h = load(c, EF_VALIDATE);
    CHECK(h != nullptr);
    if (!h) continue;
    std::vector<int32_t> seeds;
    for (int32_t i = 0; i < 40; ++i) seeds.push_back((int32_t)((i * 7919ll) % c.n()));
    for (int round = 0; round < 2; ++round) {
      for (ef_prec p : {EF_PREC_FP32C, EF_PREC_FP64}) {
        for (ef_algo a : {EF_ALGO_CLUSTER, EF_ALGO_PER_SEED, EF_ALGO_CLUSTER_AGG})
          CHECK(whole(h, a, p) == EF_OK);
        CHECK(some(h, p, seeds) == EF_OK);
        if (c.nnz() < 50000) {
          CHECK(whole_j3(h, p) == EF_OK);
          CHECK(some(h, p, seeds, true) == EF_OK);
        }
      }
      const int32_t k = std::min<int32_t>(c.n(), 50);
      std::vector<int32_t> nodes((size_t)k);
      std::vector<double> ef((size_t)k);
      CHECK(ef_topk(h, EF_ALGO_CLUSTER, EF_PREC_FP32C, k, nodes.data(), ef.data(), 0, nullptr) ==
            EF_OK);
      CHECK(nodes[0] == c.n() - 1 && ef[0] == c.n() - 0.5);
    }
    CHECK(ef_graph_free(h) == EF_OK);
    CHECK(stub::live_blocks() == 0);
  }
  // what the load refuses leaves nothing behind
  Csr bad = ring(50, 4);
  bad.ci[3] = 77;
  CHECK(load(bad) == nullptr && load(bad, EF_VALIDATE) == nullptr);
  bad = ring(50, 4);
  bad.ci.erase(bad.ci.begin());
  for (size_t i = 1; i < bad.rp.size(); ++i) bad.rp[i]--;
  CHECK(load(bad, EF_VALIDATE) == nullptr);
  CHECK(stub::live_blocks() == 0);
}

// batches of a few small graphs (empty ones among them), both designs, both
// precisions, tuned and not, replayed
static void batches() {
  std::mt19937 r(7);
  for (int t = 0; t < 24; ++t) {
    const int count = t % 8;
    std::vector<int32_t> off{0};
    Csr u;
    for (int q = 0; q < count; ++q) {
      const int32_t n = t < 16 ? (int32_t)(r() % 830) : (int32_t)(r() % 4000);
      const Csr c = n == 0 ? Csr() : r() % 2 ? ring(n, std::min(n - 1, 6)) : hubby(n, 1 + (int32_t)(r() % 5), r());
      for (int32_t v = 0; v < c.n(); ++v) {
        for (int32_t e = c.rp[(size_t)v]; e < c.rp[(size_t)v + 1]; ++e)
          u.ci.push_back(off.back() + c.ci[(size_t)e]);
        u.rp.push_back((int32_t)u.ci.size());
      }
      off.push_back(off.back() + c.n());
    }
    ef_batch *b = nullptr;
    CHECK(ef_batch_create(count, off.data(), u.nnz(), u.rp.data(), u.ci.data(), EF_VALIDATE, nullptr,
                          &b) == EF_OK);
    if (!b) continue;
    for (ef_prec p : {EF_PREC_FP32C, EF_PREC_FP64, EF_PREC_FP32C})
      for (uint32_t f : {EF_BATCH_PHASED, 0u, EF_BATCH_PERSISTENT, 0u, EF_BATCH_PHASED}) {
        Out o((size_t)off.back());
        CHECK(ef_batch_compute(b, p, o.ef.data(), o.D.data(), o.N.data(), f, nullptr) == EF_OK);
        CHECK(expected(o, nullptr));
        if (off.back() > 0 && r() % 4 == 0) CHECK(ef_batch_autotune(b, p) == EF_OK);
      }
    CHECK(ef_batch_free(b) == EF_OK);
    CHECK(stub::live_blocks() == 0);
  }
}

// a first use that runs out of memory half-way leaves nothing that a later call
// takes for the whole
static void first_use() {
  const Csr c = hubby(3000, 6, 4);
  ef_graph *h = load(c);
  stub::fail_mallocs(8 * ((size_t)c.n() + 1));  // the item offsets
  CHECK(whole_j3(h, EF_PREC_FP32C) == EF_ERR_NOMEM);
  CHECK(!h->g.j3_seeds && !h->g.j3_off);
  stub::fail_mallocs(0);
  CHECK(whole_j3(h, EF_PREC_FP32C) == EF_OK);
  std::vector<size_t> bins(efi::kSeedBins, 0);
  CHECK(whole(h, EF_ALGO_PER_SEED, EF_PREC_FP32C) == EF_OK);
  for (int b = 0; b < efi::kSeedBins; ++b) bins[(size_t)b] = 4 * (size_t)h->g.n_ps[b];
  CHECK(ef_graph_free(h) == EF_OK);
  h = load(c);
  CHECK(bins[1] > 0);
  stub::fail_mallocs(bins[1]);  // the second of the seed lists
  CHECK(whole(h, EF_ALGO_PER_SEED, EF_PREC_FP32C) == EF_ERR_NOMEM);
  CHECK(!h->g.ps_list[0] && !h->g.ps_ready);
  stub::fail_mallocs(0);
  CHECK(whole(h, EF_ALGO_PER_SEED, EF_PREC_FP32C) == EF_OK);
  CHECK(ef_graph_free(h) == EF_OK);
  CHECK(stub::live_blocks() == 0);
}

// a whole-graph call captured by the caller
static void capture(ef_graph *h, ef_algo algo, ef_prec p, const DeviceOut &o) {
  hipStream_t st;
  (void)hipStreamCreateWithFlags(&st, 0);
  CHECK(o.call(h, algo, p, st) == EF_OK);  // sizes the workspace
  CHECK(hipStreamSynchronize(st) == hipSuccess);
  stub::begin_capture(st);
  CHECK(o.call(h, algo, p, st) == EF_OK);
  stub::end_capture(st);
  (void)hipStreamDestroy(st);
}

// a captured graph's block outlives calls that need a larger one
static void captured() {
  const Csr c = ring(300000, 8);  // FP64 needs more than the load keeps
  DeviceOut o((size_t)c.n());
  for (int form = 0; form < 2; ++form) {
    ef_graph *h = load(c);
    if (form == 0) capture(h, EF_ALGO_CLUSTER, EF_PREC_FP32C, o);
    else capture(h, EF_ALGO_PER_SEED, EF_PREC_FP64, o);
    const size_t before = h->g.ws[0].bytes;
    CHECK(whole(h, EF_ALGO_CLUSTER, EF_PREC_FP64) == EF_OK);
    CHECK(h->g.ws[0].bytes > before);
    o.clear();
    stub::replay();
    CHECK(o.expected());
    CHECK(whole(h, EF_ALGO_CLUSTER, EF_PREC_FP64) == EF_OK);
    stub::replay();
    CHECK(ef_graph_free(h) == EF_OK);
  }
  // a batch's own graphs hold no block once they are replaced
  const int32_t off[2] = {0, c.n()};
  size_t held[2];
  for (int first = 0; first < 2; ++first) {
    ef_batch *b = nullptr;
    CHECK(ef_batch_create(1, off, c.nnz(), c.rp.data(), c.ci.data(), 0, nullptr, &b) == EF_OK);
    Out r((size_t)c.n());
    for (int q = first; q < 2; ++q)
      CHECK(ef_batch_compute(b, q == 0 ? EF_PREC_FP32C : EF_PREC_FP64, r.ef.data(), r.D.data(),
                             r.N.data(), EF_BATCH_PHASED, nullptr) == EF_OK);
    held[first] = stub::live_bytes();
    CHECK(ef_batch_free(b) == EF_OK);
  }
  CHECK(held[0] == held[1]);
}

// calls of one handle on different streams, without a wait between them, that
// share nothing the first one fills
static void streams() {
  const Csr c = hubby(3000, 6, 5);
  hipStream_t a, b;
  (void)hipStreamCreateWithFlags(&a, 0);
  (void)hipStreamCreateWithFlags(&b, 0);
  DeviceOut o((size_t)c.n()), o3((size_t)c.n());
  for (ef_prec p : {EF_PREC_FP64, EF_PREC_FP32C}) {  // FP32C recomputes some seeds in FP64
    ef_graph *h = load(c);
    for (int round = 0; round < 2; ++round) {
      CHECK(o.call(h, EF_ALGO_CLUSTER, EF_PREC_FP64, a) == EF_OK);
      CHECK(ef_compute_j3(h, p, nullptr, 0, o3.ef, o3.D, o3.N, EF_OUT_DEVICE, b) == EF_OK);
      CHECK(o.expected() && o3.expected());
    }
    CHECK(whole(h, EF_ALGO_CLUSTER, EF_PREC_FP64) == EF_OK);
    CHECK(!h->g.score_pending);
    CHECK(ef_graph_free(h) == EF_OK);
  }
  // a call that waits by itself fills the table, or fails before it waits
  for (bool fails : {false, true}) {
    ef_graph *h = load(c);
    if (fails) stub::fail_copies(8 * (size_t)c.n());  // of its results
    Out r((size_t)c.n());
    CHECK((ef_compute_j3(h, EF_PREC_FP64, nullptr, 0, r.ef.data(), r.D.data(), r.N.data(), 0, a) ==
           EF_OK) == !fails);
    stub::fail_copies(0);
    CHECK(h->g.score64 && h->g.score_pending == fails);
    CHECK(o.call(h, EF_ALGO_CLUSTER, EF_PREC_FP64, b) == EF_OK);
    CHECK(o.call(h, EF_ALGO_CLUSTER, EF_PREC_FP64, a) == EF_OK);
    CHECK(o.expected() && ef_graph_free(h) == EF_OK);
  }
  (void)hipStreamDestroy(a);
  (void)hipStreamDestroy(b);
}

// device bytes of a handle's node lists, without the padding between them
static int64_t list_bytes(const efi::Graph &g) {
  return 16 * (g.n_tri_lane + g.n_tri[0] + g.n_tri[1] + g.n_tri[2]) +
         4 * (g.n_tri[1] + g.n_tri[3] + g.n_fin + g.n_fin_group);
}
// what a loaded handle holds for calls that may not come
static void idle() {
  const Csr graphs[] = {from_edges(40000, {}), ring(1400000, 8), from_edges(3000, {{0, 1}}),
                        hubby(3000, 6, 6), ring(100000, 8)};
  for (const Csr &c : graphs) {
    ef_graph *h = load(c);
    const size_t bytes = h->g.ws[0].bytes;
    CHECK(bytes <= (256u << 20) && bytes <= 40 * (size_t)c.nnz());
    CHECK((bytes > 0) == (&c >= graphs + 3));
    CHECK(whole(h, EF_ALGO_CLUSTER, EF_PREC_FP32C) == EF_OK);
    CHECK(bytes == 0 || h->g.ws[0].bytes == bytes);
    CHECK(ef_graph_free(h) == EF_OK);
  }
}
// a batch of the persistent design finds room that the block kept by its load
// would take
static void batch_room() {
  const Csr c = ring(20000, 8);
  const int32_t off[2] = {0, c.n()};
  ef_graph *h = load(c);
  const size_t block = h->g.ws[0].bytes;
  CHECK(ef_graph_free(h) == EF_OK && block > 0);
  size_t held = 0;
  for (int round = 0; round < 2; ++round) {
    stub::set_capacity(round == 0 ? 0 : held - block / 2);
    ef_batch *b = nullptr;
    CHECK(ef_batch_create(1, off, c.nnz(), c.rp.data(), c.ci.data(), 0, nullptr, &b) == EF_OK);
    Out r((size_t)c.n());
    CHECK(ef_batch_compute(b, EF_PREC_FP32C, r.ef.data(), r.D.data(), r.N.data(),
                           EF_BATCH_PERSISTENT, nullptr) == EF_OK);
    CHECK(expected(r, nullptr));
    held = stub::live_bytes();
    stub::set_capacity(0);
    CHECK(ef_batch_compute(b, EF_PREC_FP32C, r.ef.data(), r.D.data(), r.N.data(), EF_BATCH_PHASED,
                           nullptr) == EF_OK);
    CHECK(ef_batch_free(b) == EF_OK);
  }
}
// a load accepted under one limit is accepted under any larger one: here what is
// left after a block for ef_compute has room for half of the triangle slots that
// are cleared before each pass
static void limits() {
  const Csr c = complete(2200);
  ef_graph *h = load(c);
  const efi::Graph &g = h->g;
  CHECK(g.n_tri_zero > 0);
  CHECK(whole(h, EF_ALGO_CLUSTER, EF_PREC_FP32C) == EF_OK);
  const int64_t main = (int64_t)h->g.ws[0].bytes, slots = 4 * g.n_tri_zero;
  int64_t other = 0;  // the other workspace
  for (int i = 1; i < 16; ++i) other += (int64_t)h->g.ws[i].bytes;
  const int64_t arrays = g.owned_bytes - main - slots - list_bytes(g) - other;
  CHECK(ef_graph_free(h) == EF_OK);
  for (int64_t limit : {arrays + main - 4, arrays + main + slots / 2, arrays + main + 2 * slots}) {
    setenv("EF_MAX_DEVICE_BYTES", std::to_string(limit).c_str(), 1);
    h = load(c);
    CHECK(h != nullptr);
    if (h) CHECK(ef_graph_free(h) == EF_OK);
  }
  unsetenv("EF_MAX_DEVICE_BYTES");
  CHECK(stub::live_blocks() == 0);
}

int main(int argc, char **argv) {
  const std::map<std::string, std::function<void()>> all = {
      {"calls", calls},
      {"batches", batches},
      {"first_use", first_use},
      {"captured", captured},
      {"streams", streams},
      {"idle", idle},
      {"batch_room", batch_room},
      {"limits", limits},
  };
  const auto it = argc == 2 ? all.find(argv[1]) : all.end();
  if (it == all.end()) return 2;
  it->second();
  if (g_failed || stub::errors()) return 1;
  std::printf("ok\n");
  return 0;
}
