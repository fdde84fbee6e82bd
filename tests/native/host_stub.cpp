// See host_stub.h. Device memory is filled with a pattern when it is
// allocated, so that a value the library never wrote is not a plausible one.
#include "host_stub.h"

#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <memory>
#include <set>
#include <vector>

#include "ef_internal.h"

using namespace efi;

namespace {

int g_errors = 0;
void fail(const char *fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  std::vprintf(fmt, ap);
  va_end(ap);
  std::printf("\n");
  std::fflush(stdout);
  ++g_errors;
}

std::map<void *, size_t> g_mem;
size_t g_fail_bytes = 0, g_fail_copy = 0, g_capacity = 0;

// What has happened before what: per stream, the operations of every stream
// that its next one follows; the host follows what it has waited for.
using Clock = std::map<const void *, uint64_t>;
Clock g_host;
std::map<const void *, Clock> g_streams;
std::map<const void *, Clock> g_events;
std::map<const void *, std::pair<const void *, uint64_t>> g_writer;

void join(Clock &a, const Clock &b) {
  for (const auto &x : b) a[x.first] = std::max(a[x.first], x.second);
}
uint64_t op(hipStream_t st) {
  Clock &c = g_streams[st];
  join(c, g_host);
  return ++c[st];
}
void wrote(const void *p, hipStream_t st) { g_writer[p] = {st, g_streams[st][st]}; }
void reads(const void *p, hipStream_t st, const char *what) {
  const auto it = g_writer.find(p);
  if (it == g_writer.end()) return fail("%s: read but never filled", what);
  if (g_streams[st][it->second.first] < it->second.second)
    fail("%s: read by a stream that does not follow its fill", what);
}

using Work = std::vector<std::function<void()>>;
std::map<const void *, Work> g_capture;  // streams being captured
Work g_last;                             // the last caller's capture
struct GraphObj {
  Work work;
};

template <typename F> hipError_t queue(hipStream_t st, F f) {
  op(st);
  const auto it = g_capture.find(st);
  if (it != g_capture.end()) it->second.push_back(f);
  else f();
  return hipSuccess;
}

template <typename V> void fill(V *p, int64_t n, V v) {
  for (int64_t i = 0; i < n; ++i) p[i] = v;
}
// reads n values
template <typename V> void look(const V *p, int64_t n) {
  const volatile unsigned char *c = (const volatile unsigned char *)p;
  for (int64_t i = 0; i < (int64_t)sizeof(V) * n; ++i) (void)c[i];
}
template <typename V> void in_range(const V *p, int64_t n, int64_t end, const char *what) {
  for (int64_t i = 0; i < n; ++i)
    if ((int64_t)p[i] < 0 || (int64_t)p[i] >= end)
      return fail("%s: entry %lld is %lld, outside [0, %lld)", what, (long long)i, (long long)p[i],
                  (long long)end);
}

// outputs, by node: what the host tests expect
double ef_of(int32_t v) { return v + 0.5; }

}  // namespace

namespace stub {
size_t live_blocks() { return g_mem.size(); }
bool live(const void *p) { return g_mem.count(const_cast<void *>(p)) > 0; }
size_t live_bytes() {
  size_t s = 0;
  for (const auto &m : g_mem) s += m.second;
  return s;
}
void fail_mallocs(size_t bytes) { g_fail_bytes = bytes; }
void fail_copies(size_t bytes) { g_fail_copy = bytes; }
void set_capacity(size_t bytes) { g_capacity = bytes; }
void begin_capture(hipStream_t st) { g_capture[st]; }
void end_capture(hipStream_t st) {
  g_last = g_capture[st];
  g_capture.erase(st);
}
void replay() {
  for (auto &f : g_last) f();
}
int errors() { return g_errors; }
}  // namespace stub

// ---------------------------------------------------------------------------
// HIP runtime
// ---------------------------------------------------------------------------
extern "C" {
hipError_t hipGetDeviceCount(int *n) {
  *n = 1;
  return hipSuccess;
}
hipError_t hipGetDevice(int *d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int) {
  std::memset(p, 0, sizeof(*p));
  std::strcpy(p->gcnArchName, "gfx950");
  return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetLastError() { return hipSuccess; }

hipError_t hipMalloc(void **p, size_t bytes) {
  if (!g_capture.empty()) fail("hipMalloc while a stream is captured");
  if (g_fail_bytes && bytes == g_fail_bytes) return hipErrorOutOfMemory;
  if (g_capacity && stub::live_bytes() + bytes > g_capacity) return hipErrorOutOfMemory;
  *p = std::malloc(bytes);  // exactly `bytes`: what follows is not readable
  if (!*p) return hipErrorOutOfMemory;
  std::memset(*p, 0xCD, bytes);
  g_mem[*p] = bytes;
  return hipSuccess;
}
hipError_t hipFree(void *p) {
  if (!p) return hipSuccess;
  if (!g_mem.count(p)) {
    fail("hipFree of a block that is not held");
    return hipErrorInvalidValue;
  }
  for (const auto &s : g_streams) join(g_host, s.second);  // waits for the device
  g_mem.erase(p);
  g_writer.erase(p);
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st) {
  if (g_fail_copy && n == g_fail_copy) return hipErrorUnknown;
  return queue(st, [=] { if (n) std::memcpy(d, s, n); });
}
hipError_t hipStreamSynchronize(hipStream_t st) {
  if (g_capture.count(st)) fail("a captured stream is waited for");
  join(g_host, g_streams[st]);
  return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind k) {
  (void)hipMemcpyAsync(d, s, n, k, nullptr);
  return hipStreamSynchronize(nullptr);
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t st) {
  return queue(st, [=] { std::memset(d, v, n); });
}
hipError_t hipStreamCreateWithFlags(hipStream_t *st, unsigned) {
  *st = (hipStream_t)std::malloc(1);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t st) {
  std::free((void *)st);
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t st, hipStreamCaptureStatus *s) {
  *s = g_capture.count(st) ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t st, hipStreamCaptureMode) {
  stub::begin_capture(st);
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t st, hipGraph_t *g) {
  *g = (hipGraph_t) new GraphObj{g_capture[st]};
  g_capture.erase(st);
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t g, hipGraphNode_t *, char *, size_t) {
  *x = (hipGraphExec_t) new GraphObj(*(GraphObj *)g);
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t st) {
  for (auto &f : ((GraphObj *)x)->work) (void)queue(st, f);
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) {
  delete (GraphObj *)g;
  return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t x) {
  delete (GraphObj *)x;
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
  *e = (hipEvent_t)std::malloc(1);
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) {
  g_events.erase(e);
  std::free((void *)e);
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t st) {
  op(st);
  g_events[e] = g_streams[st];
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t st, hipEvent_t e, unsigned) {
  op(st);
  join(g_streams[st], g_events[e]);
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
  join(g_host, g_events[e]);
  return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
  for (const auto &x : g_events[e])
    if (g_host[x.first] < x.second) return hipErrorNotReady;
  return hipSuccess;
}
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
  static uint32_t x = 1;  // any positive time
  x = x * 1664525u + 1013904223u;
  *ms = 1.0f + (float)(x >> 24);
  return hipSuccess;
}
}  // extern "C"

// ---------------------------------------------------------------------------
// kernel launchers
// ---------------------------------------------------------------------------
namespace efi {

int64_t scan_tmp_len(int64_t count) { return (count + 2047) / 2048 + 1; }
int64_t graph_prep_tmp_len(int64_t nnz) { return 4 * nnz + nnz / 2 + scan_tmp_len(nnz); }

hipError_t launch_graph_prep(Graph &g, int32_t *tmp, int64_t *work, bool, hipStream_t st) {
  const int64_t nnz = g.nnz, nup = nnz / 2;
  const int32_t n = g.n;
  (void)queue(st, [=, &g] {
    const int32_t *rp = g.row_ptr, *col = g.col_idx;
    int32_t *ctl = g.d_counters;
    fill(ctl, 64, 0);
    fill(tmp, graph_prep_tmp_len(std::max<int64_t>(nnz, 1)), 0x55555555);
    for (int32_t v = 0; v < n; ++v) g.deg[v] = rp[v + 1] - rp[v];
    auto less = [&](int32_t a, int32_t b) {
      return g.deg[a] < g.deg[b] || (g.deg[a] == g.deg[b] && a < b);
    };
    for (int64_t e = 0; e < nnz; ++e)
      if (col[e] < 0 || col[e] >= n) ctl[kCtlCol] = 1;
    if (ctl[kCtlCol]) {
      ctl[kCtlStop] = 1;
      return;
    }
    std::vector<int32_t> slot((size_t)nnz);
    std::vector<char> flag((size_t)nnz);
    int64_t up = 0;
    for (int32_t v = 0; v < n; ++v) {
      g.up_ptr[v] = (int32_t)std::min(up, nup);
      std::vector<std::pair<int32_t, int64_t>> row;
      for (int64_t e = rp[v]; e < rp[v + 1]; ++e) {
        const int32_t a = col[e];
        const int32_t *f = std::lower_bound(col + rp[a], col + rp[a + 1], v);
        const bool found = f < col + rp[a + 1] && *f == v;
        if (!found || a == v || (e > rp[v] && col[e - 1] >= a)) ctl[kCtlArc] = 1;
        g.src[e] = v;
        g.rev[e] = g.rrev[e] = found ? (int32_t)(f - col) : (int32_t)e;
        g.adj2[e] = make_int2(a, g.deg[a]);
        if (less(v, a)) row.push_back({a, e});
      }
      std::sort(row.begin(), row.end(), [&](auto &x, auto &y) { return less(x.first, y.first); });
      for (auto &x : row) {
        if (up < nup) {
          g.up_col[up] = x.first;
          g.up_deg[up] = g.deg[x.first];
        }
        slot[(size_t)x.second] = (int32_t)up++;
      }
    }
    g.up_ptr[n] = (int32_t)nup;
    if (2 * up != nnz) ctl[kCtlStop] = 1;
    if (ctl[kCtlStop]) return;
    // segments of the triangle pass, and the work at each node
    int64_t nd = 0;
    for (int32_t w = 0; w < n; ++w) {
      g.dn_ptr[w] = (int32_t)nd;
      work[w] = 0;
      int64_t as = 0;
      for (int64_t e = rp[w]; e < rp[w + 1]; ++e) {
        const int32_t u = col[e];
        as += g.deg[u];
        if (less(w, u)) continue;
        const int32_t s = slot[(size_t)g.rev[e]], tail = g.up_ptr[u + 1] - s - 1;
        if (tail <= 0 || g.up_ptr[w + 1] <= g.up_ptr[w]) continue;
        g.dn[nd++] = make_int4(s, tail, g.deg[u] + g.deg[w], u);
        flag[(size_t)e] = 1;
        work[w] += tail;
      }
      g.asum[w] = as;
    }
    g.dn_ptr[n] = (int32_t)nd;
    int32_t *zf = tmp + 2 * nnz, *zidx = tmp + nnz, zeros = 0;
    for (int32_t a = 0; a < n; ++a) {
      const int32_t m = g.up_ptr[a + 1] - g.up_ptr[a];
      for (int32_t s = g.up_ptr[a]; s < g.up_ptr[a + 1]; ++s) {
        zf[s] = g.dn_ptr[a + 1] > g.dn_ptr[a] && m > kTriBin2;
        zidx[s] = zeros;
        zeros += zf[s];
      }
    }
    ctl[kCtlZero] = zeros;
    for (int64_t e = 0; e < nnz; ++e) {
      const int32_t v = g.src[e], a = col[e];
      g.trec[e] = less(v, a) ? (flag[(size_t)g.rev[e]] ? (int32_t)(nup + slot[(size_t)e]) : -1)
                  : g.dn_ptr[a + 1] > g.dn_ptr[a] ? slot[(size_t)g.rev[e]]
                                                  : -1;
    }
    for (int32_t v = 0; v < n; ++v) {
      int64_t q = 0, a2 = 0;
      for (int64_t e = rp[v]; e < rp[v + 1]; ++e) {
        q += (int64_t)g.adj2[e].y * g.adj2[e].y;
        a2 += g.asum[col[e]];
      }
      g.qa[v] = make_longlong2(q, a2);
      g.nbm[v] = NbrMoments{g.asum[v], q, 0.0, 0.0};
    }
  });
  return hipSuccess;
}

hipError_t launch_big_sort(Graph &g, const int32_t *big, int32_t nbig, int32_t *scratch,
                           int32_t *seg, void *temp, size_t &temp_bytes, hipStream_t st) {
  if (!temp) {
    temp_bytes = 1000 + 8 * (size_t)nbig;
    return hipSuccess;
  }
  const size_t tb = temp_bytes;
  return queue(st, [=, &g] {
    std::memset(temp, 0, tb);
    fill(scratch, 4 * g.nnz, 0);
    fill(seg, 2 * (int64_t)nbig, 0);
    for (int32_t i = 0; i < nbig; ++i) {
      const int32_t v = big[i], b = g.row_ptr[v], k = g.row_ptr[v + 1] - b;
      std::vector<int32_t> o((size_t)k);
      for (int32_t j = 0; j < k; ++j) o[(size_t)j] = j;
      std::stable_sort(o.begin(), o.end(),
                       [&](int32_t x, int32_t y) { return g.adj2[b + x].y < g.adj2[b + y].y; });
      for (int32_t j = 0; j < k; ++j) {
        g.adjs[b + j] = make_int2(o[(size_t)j], g.adj2[b + o[(size_t)j]].y);
        g.rrev[g.rev[b + o[(size_t)j]]] = b + j;
      }
    }
  });
}

hipError_t launch_zero_list(Graph &g, const int32_t *tmp, hipStream_t st) {
  return queue(st, [=, &g] {
    const int32_t *zf = tmp + 2 * g.nnz, *zidx = tmp + g.nnz;
    for (int64_t i = 0; i < g.nnz / 2; ++i)
      if (zf[i]) g.tri_zero[zidx[i]] = (int32_t)i;
  });
}

hipError_t launch_lane_counts(Graph &, hipStream_t st) { return queue(st, [] {}); }

hipError_t launch_lane_recs(Graph &g, hipStream_t st) {
  return queue(st, [&g] {
    int64_t c = 0;
    for (int32_t v = 0; v < g.n; ++v) {
      const int32_t up = g.up_ptr[v + 1] - g.up_ptr[v], nd = g.dn_ptr[v + 1] - g.dn_ptr[v];
      int64_t walk = 0;
      for (int32_t i = g.dn_ptr[v]; i < g.dn_ptr[v + 1]; ++i) walk += g.dn[i].y;
      if (tri_lane_bin(up, nd, walk)) g.tri_recL[c++] = make_int4(v, 0, 0, 0);
    }
    if (c != g.n_tri_lane) fail("lane bin: %lld nodes, the host counted %lld", (long long)c,
                                (long long)g.n_tri_lane);
  });
}

hipError_t launch_zero_i32(int32_t *p, int32_t count, hipStream_t st) {
  return queue(st, [=] { fill(p, count, 0); });
}

hipError_t launch_bin_centres(const Graph &g, const int32_t *centres, int32_t n_centres, Bins &b,
                              hipStream_t st) {
  const Bins c = b;
  return queue(st, [=, &g] {
    fill(c.counters, 16, 0);
    int64_t n[4] = {}, mid = 0, midc[3] = {}, big = 0, tiles = 0, sb = 0;
    for (int32_t i = 0; i < n_centres; ++i) {
      const int32_t v = centres ? centres[i] : i, k = g.deg[v];
      if (k < 2) continue;
      if (k <= kSmallMax) {
        const int q = small_bin(k, c.thr);
        c.small[q][n[q]++] = v;
      } else if (k <= kSuper) {
        c.mid[mid++] = v;
        c.midc[mid_class(k)][midc[mid_class(k)]++] = v;
      } else {
        const int32_t ns = (k + kSuper - 1) / kSuper;
        c.big[big] = BigCentre{v, ns, tiles};
        for (int32_t P = 0; P < ns; ++P) {
          for (int32_t Q = P; Q < ns; ++Q) c.tiles[tiles++] = TileItem{(int32_t)big, P, Q};
          c.sblocks[sb++] = make_int2((int32_t)big, P);
        }
        ++big;
      }
    }
    for (int q = 0; q < 4; ++q)
      if (n[q] != c.n_smallb[q]) fail("small bin %d: %lld centres, the host counted %lld", q,
                                      (long long)n[q], (long long)c.n_smallb[q]);
    if (mid != c.n_mid || big != c.n_big || tiles != c.n_tiles || sb != c.n_sblocks)
      fail("mid and big bins differ from the host's counts");
  });
}

hipError_t launch_score_table(double *t, int32_t n, hipStream_t st) {
  const hipError_t e = queue(st, [=] { fill(t, n, 1.0); });
  wrote(t, st);
  return e;
}

hipError_t launch_pairs(const Graph &g, ef_prec prec, const Bins &b, void *R, void *records,
                        hipStream_t st, bool tab, hipEvent_t, hipEvent_t, hipEvent_t,
                        int32_t *agg_done) {
  const bool d = prec == EF_PREC_FP64;
  const double *t = d && tab ? g.score64 : nullptr;
  const int32_t nt = g.n_score64;
  op(st);
  if (t) reads(t, st, "score table");
  const Bins c = b;
  return queue(st, [=, &g] {
    if (t) look(t, nt);
    for (int q = 0; q < 4; ++q) in_range(c.small[q], c.n_smallb[q], g.n, "small centres");
    for (int q = 0; q < 3; ++q) in_range(c.midc[q], c.n_midc[q], g.n, "mid centres");
    if (agg_done) fill(agg_done, c.n_big, 0);
    if (d) {
      fill((double *)R, g.nnz, 1.0);
      fill((double *)records, c.n_tiles * kRecEntries, 1.0);
    } else {
      fill((float *)R, g.nnz, 1.0f);
      fill((float *)records, c.n_tiles * kRecEntries, 1.0f);
    }
  });
}

hipError_t launch_triangles(const Graph &g, ef_prec, TriSlot *Y, void *Z, int64_t *ZT,
                            hipStream_t st) {
  return queue(st, [=, &g] {
    in_range(g.tri_zero, g.n_tri_zero, std::max<int64_t>(g.nnz / 2, 1), "cleared slots");
    auto ids = [&](const int4 *r, int64_t n, const char *what) {
      for (int64_t i = 0; i < n; ++i)
        if (r[i].x < 0 || r[i].x >= g.n) return fail("%s: node %d", what, r[i].x);
    };
    ids(g.tri_recL, g.n_tri_lane, "lane bin");
    ids(g.tri_rec0, g.n_tri[0], "wavefront bin");
    ids(g.tri_recB[1], g.n_tri[1], "workgroup bin");
    ids(g.tri_recB[2], g.n_tri[2], "workgroup bin");
    in_range(g.tri_list[3], g.n_tri[3], g.n, "long lists");
    fill(Y, 2 * (g.nnz / 2), TriSlot{0, 0, 0});
    fill((double *)Z, g.n, 0.0);
    fill(ZT, g.n, (int64_t)0);
  });
}

static void outputs(int32_t pos, int32_t v, double *ef, int64_t *D, int64_t *N) {
  ef[pos] = ef_of(v);
  D[pos] = 3 * (int64_t)v;
  N[pos] = 7 * (int64_t)v;
}

hipError_t launch_finalize_cluster(const Graph &g, ef_prec prec, const void *R, const TriSlot *Y,
                                   const void *Z, const int64_t *ZT, double *ef, int64_t *D,
                                   int64_t *N, uint8_t *fl, int32_t *counts, hipStream_t st) {
  return queue(st, [=, &g] {
    in_range(g.fin_list, g.n_fin + g.n_fin_group, g.n, "finalize list");
    look((const char *)R, (prec == EF_PREC_FP64 ? 8 : 4) * g.nnz);
    look(Y, 2 * (g.nnz / 2));
    look((const double *)Z, g.n);
    look(ZT, g.n);
    if (counts) fill(counts, 2, 0);
    for (int32_t v = 0; v < g.n; ++v) {
      outputs(v, v, ef, D, N);
      fl[v] = v % 3 == 0;
    }
  });
}

hipError_t launch_per_seed(const Graph &g, ef_prec prec, const int32_t *seeds, const SeedLists &ls,
                           const void *R, uint32_t *bitmaps, double *ef, int64_t *D, int64_t *N,
                           uint8_t *fl, hipStream_t st, hipEvent_t) {
  const SeedLists l = ls;
  return queue(st, [=, &g] {
    look((const char *)R, (prec == EF_PREC_FP64 ? 8 : 4) * g.nnz);
    const int64_t words = ((int64_t)g.n + 31) / 32;
    for (int64_t i = 0; i < words * l.count[kSeedBins - 1]; ++i)
      if (bitmaps[i]) return fail("membership bitmaps: not clear");
    int64_t total = 0;
    for (int b = 0; b < kSeedBins; ++b) total += l.count[b];
    for (int b = 0; b < kSeedBins; ++b) {
      in_range(l.list[b], l.count[b], total, "seed list");
      for (int64_t i = 0; i < l.count[b]; ++i) {
        const int32_t pos = l.list[b][i], v = seeds ? seeds[pos] : pos;
        outputs(pos, v, ef, D, N);
        fl[pos] = v % 3 == 0;
      }
      for (int64_t i = l.first[b]; i < l.first[b + 1]; ++i) {
        const int4 it = l.items[i];
        if (it.y < 0 || it.y >= l.split[b] || l.list[b][it.y] != it.x || it.z >= it.w)
          return fail("seed pieces: item %lld", (long long)i);
      }
    }
    if (l.parts) std::memset(l.parts, 0, kSeedPart * (size_t)l.first[kSeedBins]);
  });
}

hipError_t launch_pass2(const Graph &g, const int32_t *seeds, const uint8_t *fl, int64_t n,
                        int32_t *listed, int32_t *counts, double *ef, const int64_t *D,
                        hipStream_t st) {
  (void)g;
  return queue(st, [=] {
    for (int64_t i = 0; i < n; ++i) {
      if (n > kPass2Scan) listed[i] = (int32_t)i;
      counts[0] += fl[i] & 1;
      const int32_t v = seeds ? seeds[i] : (int32_t)i;
      if (D[i] != 3 * (int64_t)v) return fail("pass 2: D of position %lld", (long long)i);
      ef[i] = ef_of(v);
    }
  });
}

hipError_t launch_gather_outputs(const int32_t *inv, int32_t count, const double *ef_u,
                                 const int64_t *D_u, const int64_t *N_u, double *ef, int64_t *D,
                                 int64_t *N, hipStream_t st) {
  return queue(st, [=] {
    for (int32_t i = 0; i < count; ++i) {
      ef[i] = ef_u[inv[i]];
      if (D) D[i] = D_u[inv[i]];
      if (N) N[i] = N_u[inv[i]];
    }
  });
}

hipError_t launch_j3_items(const Graph &g, bool fp64, bool tab, bool, const int32_t *seeds,
                           const int64_t *off, int32_t nseeds, int64_t n_items, int32_t *lists,
                           int32_t *counts, long long *PN, long long *PD, double *PS,
                           hipStream_t st) {
  const double *t = fp64 && tab ? g.score64 : nullptr;
  const int32_t nt = g.n_score64;
  op(st);
  if (t) reads(t, st, "score table");
  return queue(st, [=, &g] {
    if (t) look(t, nt);
    fill(lists, 5 * n_items, 0);
    fill(counts, 5, 0);
    if (!seeds || !off) return fail("three events: no seed list");
    in_range(seeds, nseeds, g.n, "three events: seeds");
    if (off[0] != 0 || off[nseeds] != n_items) return fail("three events: item offsets");
    for (int32_t i = 0; i < nseeds; ++i)
      for (int32_t e = g.row_ptr[seeds[i]]; e < g.row_ptr[seeds[i] + 1]; ++e) {
        PN[e] = PD[e] = 0;
        PS[e] = 0.0;
      }
  });
}

hipError_t launch_j3_finish(const Graph &, bool, const long long *, const long long *,
                            const double *, const int32_t *nodes, const int32_t *pos,
                            int32_t count, double *ef, int64_t *D, int64_t *N, uint8_t *fl,
                            hipStream_t st) {
  return queue(st, [=] {
    for (int32_t i = 0; i < count; ++i) {
      const int32_t p = pos ? pos[i] : i, v = nodes ? nodes[p] : p;
      outputs(p, v, ef, D, N);
      if (fl) fl[p] = v % 3 == 0;
    }
  });
}

size_t topk_scratch_bytes(int32_t, int32_t k) { return 4096 + 12 * (size_t)k; }
bool topk_direct(const double *, int32_t n, int32_t, const int32_t *, const double *) {
  return n <= 64;
}
hipError_t launch_topk(const double *vals, int32_t n, int32_t k, void *scratch,
                       size_t scratch_bytes, int32_t *nodes, double *ef_out, hipStream_t st) {
  return queue(st, [=] {
    look(vals, n);
    if (n > 64) std::memset(scratch, 0, scratch_bytes);
    for (int32_t i = 0; i < k; ++i) {
      nodes[i] = n - 1 - i;
      if (ef_out) ef_out[i] = vals[n - 1 - i];
    }
  });
}

hipError_t launch_batch_persist(const Graph &g, ef_prec, const PersistPlan &plan, void *R,
                                void *rec, TriSlot *Y, void *Z, int64_t *ZT, double *ef,
                                int64_t *D, int64_t *N, uint8_t *fl, hipStream_t st) {
  const PersistPlan p = plan;
  return queue(st, [=, &g] {
    look(p.pend, 3 * p.n_graphs);
    look(p.pend0, 3 * p.n_graphs);
    fill(p.ctl, 16, 0);
    fill((double *)R, g.nnz, 1.0);
    (void)rec;
    fill(Y, 2 * (g.nnz / 2), TriSlot{0, 0, 0});
    fill((double *)Z, g.n, 0.0);
    fill(ZT, g.n, (int64_t)0);
    std::vector<char> done((size_t)g.n);
    for (int32_t i = 0; i < p.n_items; ++i) {
      const int4 it = p.items[i];
      const int64_t cnt = it.w - it.z;
      if (it.x < 0 || it.x >= PI_TYPES || it.y < 0 || it.y >= p.n_graphs || cnt <= 0)
        return fail("persistent items: item %d", i);
      const int32_t *ids = nullptr;
      switch (it.x) {
        case PI_PAIR_LANE: case PI_PAIR_S16: case PI_PAIR_S32: case PI_PAIR_S64:
          ids = p.pair[it.x - PI_PAIR_LANE];
          break;
        case PI_PAIR_M4: case PI_PAIR_M2: case PI_PAIR_M1: ids = p.pair[4 + it.x - PI_PAIR_M4]; break;
        case PI_TRI_BLOCK: ids = p.tri_block; break;
        case PI_TRI_LONG: ids = p.tri_long; break;
        case PI_TRI_LANE: look(g.tri_recL + it.z, cnt); break;
        case PI_TRI_WAVE: look(p.tri_wave + it.z, cnt); break;
        case PI_PAIR_BIG: look(p.tiles + it.z, cnt); break;
        case PI_REDUCE: look(p.reduce + it.z, cnt); break;
        case PI_FIN_G8: ids = p.fin_list[0]; break;
        case PI_FIN_G32: ids = p.fin_list[1]; break;
        case PI_FIN_G64: ids = p.fin_list[2]; break;
        case PI_FIN_HUB: ids = p.fin_list[3]; break;
      }
      if (ids) in_range(ids + it.z, cnt, g.n, "persistent items");
      for (int64_t q = it.z; q < it.w; ++q) {
        const bool range = it.x == PI_FIN_LANE;
        const bool list = it.x >= PI_FIN_G8 && it.x <= PI_FIN_HUB;
        if (!range && !list) break;
        const int32_t v = range ? (int32_t)q : ids[q];
        if (range && g.deg[v] > kFinLaneMax) continue;
        if (done[(size_t)v]++) return fail("persistent items: node %d finalised twice", v);
        outputs(v, v, ef, D, N);
        fl[v] = 0;
      }
    }
    for (int32_t v = 0; v < g.n; ++v)
      if (!done[(size_t)v]) return fail("persistent items: node %d never finalised", v);
  });
}

}  // namespace efi
