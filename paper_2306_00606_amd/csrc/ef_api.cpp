// C-ABI of the Expected Force library: argument checks, CSR validation, graph
// loading, workspace management and the launch sequence of each entry point.
// All arithmetic of the method runs in the kernels of the .hip files.
#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <numeric>
#include <string>
#include <memory>
#include <vector>

#include "csr_check.h"
#include "ef_internal.h"


namespace efi {

static thread_local std::string t_err;

void set_error(const char *fmt, ...) {
  char buf[1024];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  t_err = buf;
}

ef_status hip_status(hipError_t e, const char *what) {
  if (e == hipSuccess) return EF_OK;
  set_error("%s: HIP error %d (%s)", what, (int)e, hipGetErrorString(e));
  if (e == hipErrorOutOfMemory || e == hipErrorMemoryAllocation) return EF_ERR_NOMEM;
  return EF_ERR_DEVICE;
}

static int64_t max_device_bytes() {
  const char *s = std::getenv("EF_MAX_DEVICE_BYTES");
  if (!s || !*s) return INT64_MAX;
  char *end = nullptr;
  long long v = std::strtoll(s, &end, 10);
  return v > 0 ? (int64_t)v : INT64_MAX;
}

// allocation accounted against EF_MAX_DEVICE_BYTES (`counted` bytes where given:
// a block of several arrays counts them without the padding between)
static ef_status dev_alloc(Graph &g, void **p, size_t bytes, const char *what,
                           size_t counted = 0) {
  *p = nullptr;
  if (bytes == 0) bytes = 8;
  if (counted == 0) counted = bytes;
  if (g.owned_bytes + (int64_t)counted > max_device_bytes()) {
    set_error("%s: %zu bytes would exceed EF_MAX_DEVICE_BYTES", what, bytes);
    return EF_ERR_NOMEM;
  }
  hipError_t e = hipMalloc(p, bytes);
  if (e != hipSuccess) {
    *p = nullptr;
    (void)hipGetLastError();
    set_error("%s: device allocation of %zu bytes failed", what, bytes);
    return EF_ERR_NOMEM;
  }
  g.owned_bytes += (int64_t)counted;
  return EF_OK;
}

static void dev_free(Graph &g, void *p, size_t bytes) {
  if (!p) return;
  (void)hipFree(p);
  g.owned_bytes -= (int64_t)(bytes ? bytes : 8);
}

// workspace slots
enum {
  WS_MAIN = 0,  // ef_compute's sums and records (ComputeWs), and the load's scratch
  WS_FLAG, WS_BINS, WS_OUT, WS_BITMAP, WS_SEEDS, WS_UOUT, WS_TOPK, WS_SURR, WS_J3, WS_J3P, WS_J3L,
  WS_SPLIT  // pieces of the seeds of per-seed calls and their sums
};

// Host outputs of up to kOneCopy nodes come back in one copy, with the counters,
// and are spread by the host: a copy to pageable memory costs some 15 us beside
// its bytes, four of them as much as the host takes for these nodes.
constexpr int32_t kOneCopy = 16384;

// Byte offsets in WS_MAIN of one ef_compute call: per-arc sums, super-tile
// records, flag list and bytes, output staging and pass 2's counters, triangle records
// and node sums (cluster-centric only). One block: an allocation and a free of tens of
// megabytes cost some 0.3 ms each.
struct ComputeWs {
  size_t R = 0, rec = 0, flag = 0, out = 0, Y = 0, Z = 0, ZT = 0, bytes = 0;
};
static ComputeWs compute_ws(const Graph &g, bool fp64, int64_t n_tiles, int64_t n_work,
                            bool triangles) {
  const size_t nnz = (size_t)std::max<int64_t>(g.nnz, 1), n = (size_t)std::max(g.n, 1),
               nup = (size_t)std::max<int64_t>(g.nnz / 2, 1),
               w = (size_t)std::max<int64_t>(n_work, 1);
  const size_t sz = fp64 ? sizeof(double) : sizeof(float);  // a sum, and a record entry
  ComputeWs L;
  size_t p = 0;
  auto take = [&](size_t b) {
    const size_t r = p;
    p += (b + 15) & ~(size_t)15;
    return r;
  };
  L.R = take(sz * nnz);
  L.rec = take(sz * kRecEntries * (size_t)std::max<int64_t>(n_tiles, 1));
  L.flag = take((w > (size_t)kPass2Scan ? sizeof(int32_t) : 0) * w + w);
  L.out = take((sizeof(double) + 2 * sizeof(int64_t)) * w + 2 * sizeof(int32_t));
  if (triangles) {
    L.Y = take(sizeof(TriSlot) * 2 * nup);
    L.Z = take(sizeof(double) * n);  // FP32C: a float pair
    L.ZT = take(sizeof(int64_t) * n);
  }
  L.bytes = p;
  return L;
}

// Largest block that a load keeps for the first ef_compute (FP64's size up to
// kMainKept64, FP32C's above). Allocating and freeing it costs 0.3 ms for tens of
// megabytes, 1 ms for a hundred, a tenth of the load that is over by then; larger
// graphs load for longer, and idle handles would hold gigabytes.
constexpr size_t kMainKept = (size_t)256 << 20, kMainKept64 = (size_t)64 << 20;

// Gives up ef_compute's block when no call is using it (the free waits for work
// in flight) and no captured graph refers to it.
static bool drop_main(Graph &g) {
  if (g.main_busy || g.main_captured || !g.ws[WS_MAIN].p) return false;
  dev_free(g, g.ws[WS_MAIN].p, g.ws[WS_MAIN].bytes);
  g.ws[WS_MAIN] = DevBuf{};
  return true;
}

// Device arrays that a call builds on first use and its handle keeps: filled as
// they are added, and freed again unless the call comes to keep() them, so that
// after a failure the handle holds none of them.
class KeptArrays {
 public:
  explicit KeptArrays(Graph &g) : g_(g) {}
  ~KeptArrays() {
    for (const DevBuf &b : held_) dev_free(g_, b.p, b.bytes);
  }
  ef_status add(void **out, const void *src, size_t bytes, const char *what) {
    DevBuf b;
    b.bytes = std::max<size_t>(bytes, 4);
    ef_status s = dev_alloc(g_, &b.p, b.bytes, what);
    if (s != EF_OK && drop_main(g_)) s = dev_alloc(g_, &b.p, b.bytes, what);
    if (s != EF_OK) return s;
    held_.push_back(b);
    *out = b.p;
    return bytes ? hip_status(hipMemcpy(b.p, src, bytes, hipMemcpyHostToDevice), what) : EF_OK;
  }
  void keep() { held_.clear(); }

 private:
  Graph &g_;
  std::vector<DevBuf> held_;
};

static ef_status ws_ensure(Graph &g, int slot, size_t bytes, const char *what) {
  DevBuf &b = g.ws[slot];
  if (b.bytes >= bytes && b.p) return EF_OK;
  // a replay writes to the block it was captured with, whatever the calls since
  // have needed
  const DevBuf captured = slot == WS_MAIN && g.main_captured ? b : DevBuf{};
  if (b.p && !captured.p) dev_free(g, b.p, b.bytes);
  b = DevBuf{};
  size_t want = std::max<size_t>(bytes, slot == WS_MAIN ? 16 : 256);
  ef_status s = dev_alloc(g, &b.p, want, what);
  if (s != EF_OK && g.score64) {
    // the FP64 score table only saves time: workspace comes first
    dev_free(g, g.score64, sizeof(double) * (size_t)g.n_score64);
    g.score64 = nullptr;
    g.n_score64 = 0;
    s = dev_alloc(g, &b.p, want, what);
  }
  if (s != EF_OK && slot != WS_SPLIT && g.ws[WS_SPLIT].p) {
    // so do the pieces that the largest seeds are cut into
    dev_free(g, g.ws[WS_SPLIT].p, g.ws[WS_SPLIT].bytes);
    g.ws[WS_SPLIT] = DevBuf{};
    g.split_kept = false;
    s = dev_alloc(g, &b.p, want, what);
  }
  if (s != EF_OK && slot != WS_MAIN && drop_main(g)) s = dev_alloc(g, &b.p, want, what);
  if (s != EF_OK) {
    b = captured;
    return s;
  }
  b.bytes = want;
  if (captured.p) {
    g.main_old.push_back(captured);
    g.main_captured = false;
  }
  return EF_OK;
}

static ef_status check_device(int *dev) {
  int count = 0;
  hipError_t e = hipGetDeviceCount(&count);
  if (e != hipSuccess || count <= 0) {
    (void)hipGetLastError();
    set_error("no HIP device visible");
    return EF_ERR_DEVICE;
  }
  e = hipGetDevice(dev);
  if (e != hipSuccess) return hip_status(e, "hipGetDevice");
  hipDeviceProp_t prop;
  e = hipGetDeviceProperties(&prop, *dev);
  if (e != hipSuccess) return hip_status(e, "hipGetDeviceProperties");
  if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0) {
    set_error("device %d is %s; this library is built for gfx950", *dev, prop.gcnArchName);
    return EF_ERR_DEVICE;
  }
  return EF_OK;
}

static inline bool rank_less_h(int32_t a, int32_t ka, int32_t b, int32_t kb) {
  return ka < kb || (ka == kb && a < b);
}

// Largest degree for which every cluster degree (< 3 k_max) is exact in
// FP32 and every D(s) (< 6 k_max^3) fits in int64.

}  // namespace efi

using namespace efi;

extern "C" {

const char *ef_last_error(void) { return t_err.c_str(); }

int32_t ef_version(void) { return 10000; }

ef_status ef_device_count(int32_t *count) {
  if (!count) {
    set_error("ef_device_count: null output");
    return EF_ERR_ARG;
  }
  *count = 0;
  int c = 0;
  if (hipGetDeviceCount(&c) != hipSuccess) {
    (void)hipGetLastError();
    return EF_OK;
  }
  int32_t ok = 0;
  for (int i = 0; i < c; ++i) {
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, i) == hipSuccess &&
        std::strncmp(prop.gcnArchName, "gfx950", 6) == 0)
      ++ok;
  }
  *count = ok;
  return EF_OK;
}

ef_status ef_validate_csr(int32_t n, int64_t nnz, const int32_t *row_ptr, const int32_t *col_idx) {
  char msg[256] = "";
  const ef_status s = csr_validate(n, nnz, row_ptr, col_idx, msg, sizeof(msg));
  if (s != EF_OK) set_error("ef_validate_csr: %s", msg);
  return s;
}

ef_status ef_graph_free(ef_graph *h) {
  if (!h) {
    set_error("ef_graph_free: null handle");
    return EF_ERR_ARG;
  }
  Graph &g = h->g;
  void *blocks[] = {g.arena, g.lists, g.tri_zero, g.j3_seeds, g.j3_off, g.ps_list[0], g.ps_list[1],
                    g.ps_list[2], g.ps_list[3], g.ps_list[4], g.score64};
  for (void *p : blocks)
    if (p) (void)hipFree(p);
  for (auto &b : g.ws)
    if (b.p) (void)hipFree(b.p);
  for (auto &b : g.main_old) (void)hipFree(b.p);
  if (g.ev_ready)
    for (auto &e : g.ev) (void)hipEventDestroy(e);
  if (g.score_ev) (void)hipEventDestroy(g.score_ev);
  delete h;
  return EF_OK;
}

ef_status ef_graph_load_csr(int32_t n, int64_t nnz, const int32_t *row_ptr,
                            const int32_t *col_idx, uint32_t flags, void *hip_stream,
                            ef_graph **out) {
  return efi::graph_load(n, nnz, row_ptr, col_idx, flags, hip_stream, nullptr, 0, out);
}

}  // extern "C"

namespace efi {

ef_status graph_load(int32_t n, int64_t nnz, const int32_t *row_ptr, const int32_t *col_idx,
                     uint32_t flags, void *hip_stream, const int64_t *part_off, int32_t n_parts,
                     ef_graph **out) {
  if (!out) {
    set_error("ef_graph_load_csr: null output handle");
    return EF_ERR_ARG;
  }
  *out = nullptr;
  if (n < 0 || nnz < 0 || !row_ptr || (nnz > 0 && !col_idx)) {
    set_error("ef_graph_load_csr: bad arguments (n=%d, nnz=%lld)", n, (long long)nnz);
    return EF_ERR_ARG;
  }
  if (flags & ~(EF_VALIDATE | EF_DEVICE_PTRS)) {
    set_error("ef_graph_load_csr: unknown flags 0x%x", flags);
    return EF_ERR_ARG;
  }
  if (nnz >= (int64_t)INT32_MAX) {
    set_error("ef_graph_load_csr: nnz=%lld does not fit int32 offsets", (long long)nnz);
    return EF_ERR_OVERFLOW;
  }
  hipStream_t stream = (hipStream_t)hip_stream;
  const bool devptr = (flags & EF_DEVICE_PTRS) != 0, validate = (flags & EF_VALIDATE) != 0;
  int dev = 0;
  ef_status st = EF_OK;

  // host view of the row offsets (bounds, and sizing of work lists)
  std::vector<int32_t> h_rp;
  const int32_t *hrp = row_ptr;
  if (devptr) {
    if ((st = check_device(&dev)) != EF_OK) return st;
    h_rp.resize((size_t)n + 1);
    hipError_t e = hipMemcpy(h_rp.data(), row_ptr, sizeof(int32_t) * ((size_t)n + 1),
                             hipMemcpyDeviceToHost);
    if (e != hipSuccess) return hip_status(e, "copy row_ptr to host");
    hrp = h_rp.data();
  }
  // The neighbour ids are checked by the preparation kernels (range always;
  // with EF_VALIDATE order, self-loops and reverse arcs). host_check is the
  // same check on the host, which names the first violation: run when the
  // device finds one, and before any other error is returned, so that a bad
  // CSR is reported as such whatever else fails.
  auto host_check = [&]() -> ef_status {
    std::vector<int32_t> h_ci;
    const int32_t *hci = col_idx;
    if (devptr) {
      if (!validate) return EF_OK;
      h_ci.resize((size_t)std::max<int64_t>(nnz, 1));
      if (nnz > 0) {
        hipError_t e = hipMemcpy(h_ci.data(), col_idx, sizeof(int32_t) * (size_t)nnz,
                                 hipMemcpyDeviceToHost);
        if (e != hipSuccess) return hip_status(e, "copy col_idx to host");
      }
      hci = h_ci.data();
    }
    if (validate) return ef_validate_csr(n, nnz, hrp, hci);
    char msg[256] = "";
    const ef_status s = csr_check_bounds(n, nnz, hrp, hci, msg, sizeof(msg));
    if (s != EF_OK) set_error("ef_graph_load_csr: %s", msg);
    return s;
  };
  // an error other than the CSR's own: the CSR's comes first
  auto after_check = [&](auto report) -> ef_status {
    const ef_status s = host_check();
    return s != EF_OK ? s : report();
  };
  {
    char msg[256] = "";
    st = csr_check_bounds(n, nnz, hrp, nullptr, msg, sizeof(msg));
    if (st != EF_OK) {
      set_error("%s: %s", validate ? "ef_validate_csr" : "ef_graph_load_csr", msg);
      return st;
    }
  }
  ef_graph *h = new (std::nothrow) ef_graph();
  if (!h) {
    set_error("host allocation failed");
    return EF_ERR_NOMEM;
  }
  Graph &g = h->g;
  g.h_deg.resize((size_t)n);
  int32_t kmax = 0;
  int64_t n_over = 0;  // centres of degree > kSmallMax
  for (int32_t v = 0; v < n; ++v) {
    const int32_t k = hrp[v + 1] - hrp[v];
    g.h_deg[(size_t)v] = k;
    kmax = std::max(kmax, k);
    n_over += k > kSmallMax;
  }
  if (kmax > kMaxDegree) {
    delete h;
    return after_check([&] {
      set_error("max degree %d exceeds %d (exact cluster degrees / int64 sums)", kmax, kMaxDegree);
      return EF_ERR_OVERFLOW;
    });
  }
  // the arrays every graph holds, against EF_MAX_DEVICE_BYTES, before the
  // device is touched (graph-dependent arrays are accounted as allocated)
  {
    const int64_t n1 = (int64_t)n + 1, m = std::max<int64_t>(nnz, 1),
                  mu = std::max<int64_t>(nnz / 2, 1), nn = std::max<int64_t>(n, 1);
    const int64_t need = (devptr ? 0 : 4 * n1 + 4 * m) + 4 * nn + (4 + 4 + 8 + 4) * m +
                         (8 + 16) * nn + 2 * 4 * n1 + (4 + 4 + 16) * mu + 256;
    if (need > max_device_bytes()) {
      delete h;
      return after_check([&] {
        set_error("ef_graph_load_csr: the graph's %lld device bytes would exceed "
                  "EF_MAX_DEVICE_BYTES", (long long)need);
        return EF_ERR_NOMEM;
      });
    }
  }
  if (!devptr && check_device(&dev) != EF_OK) {
    delete h;
    return after_check([&] { return check_device(&dev); });
  }
  g.dev = dev;
  g.n = n;
  g.nnz = nnz;
  ef_graph_info &inf = g.info;
  inf.n = n;
  inf.nnz = nnz;
  inf.max_degree = kmax;
  inf.up_arcs = nnz / 2;
  const size_t N1 = (size_t)n + 1, NN = (size_t)std::max(n, 1),
               NNZ = (size_t)std::max<int64_t>(nnz, 1),
               NUP = (size_t)std::max<int64_t>(nnz / 2, 1);
  // every array of known size in one block; first what the host reads back
  {
    struct Piece {
      void **p;
      size_t bytes;
    };
    std::vector<Piece> pieces = {
        {(void **)&g.d_counters, sizeof(int32_t) * 64},
        {(void **)&g.up_ptr, sizeof(int32_t) * N1},
        {(void **)&g.dn_ptr, sizeof(int32_t) * N1},
        {(void **)&g.deg, sizeof(int32_t) * NN},
        {(void **)&g.src, sizeof(int32_t) * NNZ},
        {(void **)&g.rev, sizeof(int32_t) * NNZ},
        {(void **)&g.rrev, sizeof(int32_t) * NNZ},
        {(void **)&g.adj2, sizeof(int2) * NNZ},
        {(void **)&g.asum, sizeof(int64_t) * NN},
        {(void **)&g.qa, sizeof(longlong2) * NN},
        {(void **)&g.nbm, sizeof(NbrMoments) * NN},
        {(void **)&g.up_col, sizeof(int32_t) * NUP},
        {(void **)&g.up_deg, sizeof(int32_t) * NUP},
        {(void **)&g.trec, sizeof(int32_t) * NNZ},
        {(void **)&g.dn, sizeof(int4) * NUP},
    };
    if (!devptr) {
      pieces.push_back({(void **)&g.row_ptr, sizeof(int32_t) * N1});
      pieces.push_back({(void **)&g.col_idx, sizeof(int32_t) * NNZ});
    }
    // degree-ordered rows of the mid and big centres (the tile pair loops,
    // which store their per-arc sums by sorted position)
    if (n_over > 0) pieces.push_back({(void **)&g.adjs, sizeof(int2) * NNZ});
    size_t total = 0, sum = 0;
    for (const Piece &q : pieces) {
      total += (q.bytes + 255) & ~(size_t)255;
      sum += q.bytes;
    }
    st = dev_alloc(g, &g.arena, total, "graph arrays", sum);
    if (st == EF_OK) {
      char *p = (char *)g.arena;
      for (const Piece &q : pieces) {
        *q.p = p;
        p += (q.bytes + 255) & ~(size_t)255;
      }
    }
  }
  if (devptr) {
    g.row_ptr = const_cast<int32_t *>(row_ptr);
    g.col_idx = const_cast<int32_t *>(col_idx);
  }
  // Scratch of the preparation: WS_MAIN. Where a cluster-centric call (FP64's,
  // or FP32C's) will want at most kMainKept and not much more than the scratch
  // itself, it has that size and is kept for the call; otherwise it is freed at
  // the end, since a handle need not ever score.
  const int64_t nn_tiles = [&] {
    int64_t t = 0;
    for (int32_t v = 0; v < n && kmax > kSuper; ++v)
      if (g.h_deg[(size_t)v] > kSuper) {
        const int64_t ns = ((int64_t)g.h_deg[(size_t)v] + kSuper - 1) / kSuper;
        t += ns * (ns + 1) / 2;
      }
    return t;
  }();
  const size_t work_bytes = sizeof(int64_t) * NN;
  const size_t prep_bytes = sizeof(int32_t) * (size_t)graph_prep_tmp_len((int64_t)NNZ);
  size_t sort_temp = 0;
  if (st == EF_OK && n_over > 0) {
    const hipError_t e = launch_big_sort(g, nullptr, (int32_t)n_over, nullptr, nullptr, nullptr,
                                         sort_temp, stream);
    if (e != hipSuccess) st = hip_status(e, "degree-ordered rows");
  }
  sort_temp = (sort_temp + 15) & ~(size_t)15;
  const size_t sort_bytes =
      n_over > 0 ? sort_temp + sizeof(int32_t) * (4 * NNZ + 3 * (size_t)n_over) : 0;
  const size_t scratch_bytes = std::max(work_bytes + prep_bytes, sort_bytes);
  size_t kept_bytes = 0;
  for (const bool fp64 : {false, true}) {
    const size_t w = compute_ws(g, fp64, nn_tiles, n, true).bytes;
    if (nnz > 0 && w <= (fp64 ? kMainKept64 : kMainKept) && w <= 2 * scratch_bytes) kept_bytes = w;
  }
  if (st == EF_OK) {
    const size_t want = std::max(scratch_bytes, kept_bytes);
    st = ws_ensure(g, WS_MAIN, want, "preprocessing scratch");
    if (st != EF_OK && want > scratch_bytes)
      st = ws_ensure(g, WS_MAIN, scratch_bytes, "preprocessing scratch");
  }
  if (st != EF_OK) {
    const std::string text = t_err;
    ef_graph_free(h);
    return after_check([&] {
      set_error("%s", text.c_str());
      return st;
    });
  }
  int64_t *work = nullptr;
  int32_t *tmp = nullptr;
  auto prepare = [&]() -> hipError_t {
    work = (int64_t *)g.ws[WS_MAIN].p;
    tmp = (int32_t *)((char *)g.ws[WS_MAIN].p + work_bytes);
    return launch_graph_prep(g, tmp, work, validate, stream);
  };
  hipError_t e = hipSuccess;
  if (!devptr) {
    e = hipMemcpyAsync(g.row_ptr, row_ptr, sizeof(int32_t) * N1, hipMemcpyHostToDevice, stream);
    if (e == hipSuccess && nnz > 0)
      e = hipMemcpyAsync(g.col_idx, col_idx, sizeof(int32_t) * (size_t)nnz,
                         hipMemcpyHostToDevice, stream);
  }
  if (e == hipSuccess) e = prepare();
  // one read-back of the control record and the list offsets, one of the tail
  // entries walked at each node by the triangle pass (binning)
  const size_t ptr_stride = (sizeof(int32_t) * N1 + 255) & ~(size_t)255;
  // (not cleared first: the copies fill them)
  const std::unique_ptr<char[]> h_back(new char[256 + 2 * ptr_stride]);
  const std::unique_ptr<int64_t[]> h_work(new int64_t[NN]);
  if (e == hipSuccess)
    e = hipMemcpyAsync(h_back.get(), g.d_counters, 256 + ptr_stride + sizeof(int32_t) * N1,
                       hipMemcpyDeviceToHost, stream);
  if (e == hipSuccess && n > 0)
    e = hipMemcpyAsync(h_work.get(), work, sizeof(int64_t) * (size_t)n, hipMemcpyDeviceToHost,
                       stream);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  if (e != hipSuccess) {
    ef_graph_free(h);
    return after_check([&] { return hip_status(e, "graph preprocessing"); });
  }
  const int32_t *h_ctl = (const int32_t *)h_back.get();
  const int32_t *h_up_ptr = (const int32_t *)(h_back.get() + 256);
  const int32_t *h_dn_ptr = (const int32_t *)(h_back.get() + 256 + ptr_stride);
  if (nnz > 0 && (h_ctl[kCtlStop] || h_ctl[kCtlCol])) {
    const bool col_bad = h_ctl[kCtlCol] != 0;
    ef_graph_free(h);
    return after_check([&] {
      if (col_bad) {
        set_error("ef_graph_load_csr: a neighbour id is outside [0, %d)", n);
        return EF_ERR_RANGE;
      }
      set_error("the CSR is not simple and symmetric (load with EF_VALIDATE for details)");
      return EF_ERR_NOT_SYMMETRIC;
    });
  }
  g.n_tri_zero = nnz > 0 ? h_ctl[kCtlZero] : 0;
  if (g.n_tri_zero > 0) {
    const size_t zero_bytes = sizeof(int32_t) * (size_t)g.n_tri_zero;
    st = dev_alloc(g, (void **)&g.tri_zero, zero_bytes, "zero slots");
    if (st != EF_OK && g.ws[WS_MAIN].bytes > scratch_bytes) {
      // room after all when the block is no more than the preparation's scratch,
      // whose contents go with it
      drop_main(g);
      st = ws_ensure(g, WS_MAIN, scratch_bytes, "preprocessing scratch");
      if (st == EF_OK) e = prepare();
      if (st == EF_OK && e == hipSuccess)
        st = dev_alloc(g, (void **)&g.tri_zero, zero_bytes, "zero slots");
    }
    if (st != EF_OK || e != hipSuccess) {
      ef_graph_free(h);
      return st != EF_OK ? st : hip_status(e, "graph preprocessing");
    }
    e = launch_zero_list(g, tmp, stream);
  }
  if (e == hipSuccess) e = launch_lane_counts(g, stream);
  // degree-ordered rows, sorted while the host builds the node lists
  std::vector<int32_t> hb;
  if (e == hipSuccess && n_over > 0) {
    hb.reserve((size_t)n_over);
    for (int32_t v = 0; v < n; ++v)
      if (g.h_deg[(size_t)v] > kSmallMax) hb.push_back(v);
    void *temp = g.ws[WS_MAIN].p;
    int32_t *scratch = (int32_t *)((char *)temp + sort_temp);
    int32_t *d_big = scratch + 4 * NNZ;
    int32_t *seg = d_big + n_over;
    e = hipMemcpyAsync(d_big, hb.data(), sizeof(int32_t) * (size_t)n_over, hipMemcpyHostToDevice,
                       stream);
    if (e == hipSuccess)
      e = launch_big_sort(g, d_big, (int32_t)n_over, scratch, seg, temp, sort_temp, stream);
  }
  if (e != hipSuccess) {
    ef_graph_free(h);
    return hip_status(e, "degree-ordered rows");
  }
  // (what most nodes are is counted without branches, which their degrees, in
  // no order, would mispredict: 1.0 ms for 200k nodes with them)
  std::vector<int32_t> tri[4], fin_tier[3];
  const std::unique_ptr<int32_t[]> fin_group(new int32_t[NN]);
  const bool parts = part_off && n_parts > 0;
  static_assert(kFinLaneMax < kFinGroupMax && kFinGroupMax <= kSmallMax, "tiers by degree");
  int64_t by_deg[kSmallMax + 2] = {};
  for (int32_t v = 0; v < n; ++v) {
    const int64_t k = g.h_deg[v];
    const int32_t up = h_up_ptr[v + 1] - h_up_ptr[v], nd = h_dn_ptr[v + 1] - h_dn_ptr[v];
    inf.clusters += k * (k - 1) / 2;
    inf.sum_sq_degree += k * k;
    inf.wedge_checks += h_work[v];
    by_deg[std::min<int64_t>(k, kSmallMax + 1)]++;
    const bool lane = (nd > 0) & (up <= kTriLaneM) & (h_work[v] <= kTriLaneWork) &
                      (nd <= kTriLaneSegs);  // tri_lane_bin
    g.n_tri_lane += lane;
    if ((nd > 0) & !lane) {
      const int bin = (up <= kTriBin0 && h_work[v] <= kTriWaveWork && nd <= kTriWaveSegs) ? 0
                      : up <= kTriBin1                                                  ? 1
                      : up <= kTriBin2                                                  ? 2
                                                                                        : 3;
      tri[bin].push_back(v);
    }
    if (parts && lane) g.h_tri_lane.push_back(v);
    fin_group[(size_t)g.n_fin_group] = v;
    g.n_fin_group += (k > kFinLaneMax) & (k <= kFinGroupMax);
    if (k > kFinGroupMax) fin_tier[k > kFinBlockMin ? 0 : k > kFinHalfMax ? 1 : 2].push_back(v);
  }
  for (int64_t k = 2; k <= kSmallMax; ++k) {
    g.all_small += by_deg[k];
    g.all_small_deg[k] = by_deg[k];
    g.all_pairs_small += by_deg[k] * (k * (k - 1) / 2);
  }
  for (int32_t v : hb) {  // the nodes of degree > kSmallMax
    const int64_t k = g.h_deg[v];
    if (k <= kSuper) {
      g.all_mid++;
      g.all_midc[mid_class((int32_t)k)]++;
      g.all_pairs_mid += k * (k - 1) / 2;
    } else {
      const int64_t ns = (k + kSuper - 1) / kSuper;
      g.all_big++;
      g.all_tiles += ns * (ns + 1) / 2;
      g.all_pairs_big += k * (k - 1) / 2;
      g.all_sblocks += ns;
    }
  }
  // graph by graph when the nodes are a union of parts (a batch), then
  // longest walks first
  std::vector<int32_t> part;
  if (parts) {
    part.resize((size_t)n);
    for (int32_t q = 0; q < n_parts; ++q)
      for (int64_t v = part_off[q]; v < part_off[q + 1]; ++v) part[(size_t)v] = q;
  }
  auto part_of = [&](int32_t v) { return part.empty() ? 0 : part[(size_t)v]; };
  // (a list in id order, so part by part: each part by its value, descending,
  // then by id, as 64-bit keys)
  std::vector<uint64_t> keys;
  auto sort_parts = [&](std::vector<int32_t> &l, size_t from, auto value) {
    for (size_t i = from; i < l.size();) {
      const int32_t q = part_of(l[i]);
      keys.clear();
      const size_t i0 = i;
      for (; i < l.size() && part_of(l[i]) == q; ++i) {
        const uint64_t x = (uint64_t)std::min<int64_t>(value(l[i]), UINT32_MAX);
        keys.push_back((UINT32_MAX - x) << 32 | (uint32_t)l[i]);
      }
      std::sort(keys.begin(), keys.end());
      for (size_t j = 0; j < keys.size(); ++j) l[i0 + j] = (int32_t)(uint32_t)keys[j];
    }
  };
  for (int bin = 0; bin < 4; ++bin) {
    sort_parts(tri[bin], 0, [&](int32_t v) { return h_work[v]; });
    g.n_tri[bin] = (int64_t)tri[bin].size();
  }
  std::vector<int4> rec0(tri[0].size());
  for (size_t i = 0; i < tri[0].size(); ++i) {
    const int32_t v = tri[0][i];
    const int32_t m = h_up_ptr[v + 1] - h_up_ptr[v], nd = h_dn_ptr[v + 1] - h_dn_ptr[v];
    rec0[i] = make_int4(v, h_up_ptr[v], h_dn_ptr[v], m | (nd << 16));
  }
  // workgroup bins: |up(w)| <= kTriBin2 < 2^12, segments <= degree < 2^20
  static_assert(kTriBin2 < (1 << 12) && kMaxDegree < (1 << 20), "workgroup-bin record packing");
  std::vector<int4> recB[3];
  for (int bin = 1; bin <= 2; ++bin) {
    recB[bin].resize(tri[bin].size());
    for (size_t i = 0; i < tri[bin].size(); ++i) {
      const int32_t v = tri[bin][i];
      const int32_t m = h_up_ptr[v + 1] - h_up_ptr[v], nd = h_dn_ptr[v + 1] - h_dn_ptr[v];
      recB[bin][i] = make_int4(v, h_up_ptr[v], h_dn_ptr[v], m | (nd << 12));
    }
  }
  // tiers by degree (descending), each graph by graph
  auto by_degree = [&](int32_t v) { return (int64_t)g.h_deg[v]; };
  std::vector<int32_t> &fin = fin_tier[0];
  g.n_fin_hub = (int64_t)fin.size();
  g.n_fin_half = (int64_t)fin_tier[2].size();
  sort_parts(fin, 0, by_degree);
  for (int t = 1; t < 3; ++t) {
    const size_t from = fin.size();
    fin.insert(fin.end(), fin_tier[t].begin(), fin_tier[t].end());
    sort_parts(fin, from, by_degree);
  }
  g.n_fin = (int64_t)fin.size();
  fin.insert(fin.end(), fin_group.get(), fin_group.get() + g.n_fin_group);
  if (!part.empty()) {
    // node ids of the lists, for schedules that split them by graph
    g.h_fin = fin;
    for (int bin = 0; bin < 4; ++bin) g.h_tri[bin] = tri[bin];
  }
  // every list in one block, uploaded by one copy but for the last one, which
  // the device fills
  {
    struct Piece {
      void **p;
      const void *src;
      size_t bytes;
    };
    const Piece pieces[] = {
        {(void **)&g.tri_rec0, rec0.data(), sizeof(int4) * rec0.size()},
        {(void **)&g.tri_recB[1], recB[1].data(), sizeof(int4) * recB[1].size()},
        {(void **)&g.tri_recB[2], recB[2].data(), sizeof(int4) * recB[2].size()},
        {(void **)&g.tri_list[1], tri[1].data(), sizeof(int32_t) * tri[1].size()},
        {(void **)&g.tri_list[3], tri[3].data(), sizeof(int32_t) * tri[3].size()},
        {(void **)&g.fin_list, fin.data(), sizeof(int32_t) * fin.size()},
    };
    const size_t lane_bytes = sizeof(int4) * (size_t)g.n_tri_lane;
    size_t up_bytes = 0, sum = lane_bytes;
    for (const Piece &q : pieces) {
      up_bytes += (q.bytes + 255) & ~(size_t)255;
      sum += q.bytes;
    }
    const size_t total = up_bytes + lane_bytes;
    std::vector<char> all(up_bytes);
    st = dev_alloc(g, &g.lists, total, "node lists", sum);
    if (st != EF_OK) {
      // room after all when the scratch goes (its work has to end first)
      e = hipStreamSynchronize(stream);
      dev_free(g, g.ws[WS_MAIN].p, g.ws[WS_MAIN].bytes);
      g.ws[WS_MAIN] = DevBuf{};
      st = e == hipSuccess ? dev_alloc(g, &g.lists, total, "node lists", sum)
                           : hip_status(e, "degree-ordered rows");
    }
    size_t at = 0;
    for (const Piece &q : pieces) {
      if (st == EF_OK) *q.p = (char *)g.lists + at;
      if (q.bytes) std::memcpy(all.data() + at, q.src, q.bytes);
      at += (q.bytes + 255) & ~(size_t)255;
    }
    if (st == EF_OK) {
      g.tri_recL = (int4 *)((char *)g.lists + up_bytes);
      e = launch_lane_recs(g, stream);
      if (e == hipSuccess && up_bytes > 0)
        e = hipMemcpyAsync(g.lists, all.data(), up_bytes, hipMemcpyHostToDevice, stream);
      // (the load is complete when it returns; the host vectors go)
      if (e == hipSuccess) e = hipStreamSynchronize(stream);
      if (e != hipSuccess) st = hip_status(e, "upload node lists");
      if (kept_bytes == 0) drop_main(g);
    }
    if (st != EF_OK) {
      (void)hipStreamSynchronize(stream);
      ef_graph_free(h);
      return st;
    }
  }
  *out = h;
  return EF_OK;
}

}  // namespace efi

extern "C" {

ef_status ef_graph_from_edges(int32_t n, int64_t m, const int32_t *src, const int32_t *dst,
                              void *hip_stream, ef_graph **out) {
  if (!out || n < 0 || m < 0 || (m > 0 && (!src || !dst))) {
    set_error("ef_graph_from_edges: bad arguments");
    return EF_ERR_ARG;
  }
  std::vector<int64_t> cnt((size_t)n + 1, 0);
  for (int64_t i = 0; i < m; ++i) {
    const int32_t u = src[i], v = dst[i];
    if (u < 0 || u >= n || v < 0 || v >= n) {
      set_error("edge %lld: endpoint out of range [0, %d)", (long long)i, n);
      return EF_ERR_RANGE;
    }
    if (u == v) continue;
    cnt[u + 1]++;
    cnt[v + 1]++;
  }
  for (int32_t v = 0; v < n; ++v) cnt[v + 1] += cnt[v];
  if (cnt[n] >= (int64_t)INT32_MAX) {
    set_error("ef_graph_from_edges: too many arcs");
    return EF_ERR_OVERFLOW;
  }
  std::vector<int32_t> col((size_t)cnt[n]);
  std::vector<int64_t> pos(cnt.begin(), cnt.end() - 1);
  for (int64_t i = 0; i < m; ++i) {
    const int32_t u = src[i], v = dst[i];
    if (u == v) continue;
    col[pos[u]++] = v;
    col[pos[v]++] = u;
  }
  std::vector<int32_t> rp((size_t)n + 1, 0);
  int64_t w = 0;
  for (int32_t v = 0; v < n; ++v) {
    auto b = col.begin() + cnt[v], e = col.begin() + cnt[v + 1];
    std::sort(b, e);
    auto last = std::unique(b, e);
    for (auto it = b; it != last; ++it) col[w++] = *it;
    rp[v + 1] = (int32_t)w;
  }
  return ef_graph_load_csr(n, w, rp.data(), col.data(), 0, hip_stream, out);
}

ef_status ef_graph_info_get(const ef_graph *h, ef_graph_info *out) {
  if (!h || !out) {
    set_error("ef_graph_info_get: null argument");
    return EF_ERR_ARG;
  }
  *out = h->g.info;
  return EF_OK;
}

ef_status ef_stats(const ef_graph *h, ef_run_stats *out) {
  if (!h || !out) {
    set_error("ef_stats: null argument");
    return EF_ERR_ARG;
  }
  *out = h->g.stats;
  return EF_OK;
}

}  // extern "C"

namespace efi {

// scratch for other translation units (kept in the handle, grow-only)
ef_status graph_scratch(Graph &g, size_t bytes, void **out) {
  ef_status s = ws_ensure(g, WS_SURR, bytes, "scratch");
  *out = s == EF_OK ? g.ws[WS_SURR].p : nullptr;
  return s;
}

bool graph_drop_block(Graph &g) { return drop_main(g); }

static bool capturing(hipStream_t st) {
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &cap) != hipSuccess) {
    (void)hipGetLastError();
    cap = hipStreamCaptureStatusActive;
  }
  return cap != hipStreamCaptureStatusNone;
}

// The score table is behind stream st from here on, whichever stream its fill
// was queued on. (A pending fill without an event is one whose call failed
// before it had waited for it: the table goes, and the free waits.)
static ef_status score_follow(Graph &g, hipStream_t st) {
  if (!g.score64 || !g.score_pending) return EF_OK;
  if (g.score_recorded) return hip_status(hipStreamWaitEvent(st, g.score_ev, 0), "score table");
  dev_free(g, g.score64, sizeof(double) * (size_t)g.n_score64);
  g.score64 = nullptr;
  g.n_score64 = 0;
  return EF_OK;
}

// The FP64 score table of the graph: built on the stream of the first FP64
// call and kept until memory runs short. Without memory for it, and in a call
// that a caller captures (whose replays it might not outlive), the kernels
// compute every score. waits: the call waits for its stream before it returns,
// and no event has to follow the fill for later ones (in a new graph's one call
// the event took 45 us of 350).
static ef_status score_table(Graph &g, hipStream_t st, bool waits) {
  const ef_status s = score_follow(g, st);
  if (s != EF_OK || g.score64) return s;
  // cluster degrees are below 3 k_max, with three events below 4 k_max
  const int32_t n = 4 * g.info.max_degree + 1;
  const size_t bytes = sizeof(double) * (size_t)n;
  void *t = nullptr;
  if (dev_alloc(g, &t, bytes, "score table") != EF_OK) return EF_OK;
  hipError_t e = hipSuccess;
  if (!waits && !g.score_ev) e = hipEventCreateWithFlags(&g.score_ev, hipEventDisableTiming);
  if (e == hipSuccess) e = launch_score_table((double *)t, n, st);
  if (e == hipSuccess && !waits) e = hipEventRecord(g.score_ev, st);
  if (e != hipSuccess) {
    dev_free(g, t, bytes);
    return hip_status(e, "score table");
  }
  g.score64 = (double *)t;
  g.n_score64 = n;
  g.score_pending = true;
  g.score_recorded = !waits;
  return EF_OK;
}

// Cuts the seeds of bins 1-4 whose 2-hop work is above a piece's (the leading
// ones: lst is by work, descending) into pieces: their number depends on the
// seeds alone, and is at most 2 * kSeedPieces and a chunk's rounding per seed.
static void seed_pieces(const Graph &g, const int32_t *useeds,
                        const std::vector<int32_t> (&lst)[kSeedBins], std::vector<int4> &items,
                        int64_t (&split)[kSeedBins], int64_t (&first)[kSeedBins + 1]) {
  items.clear();
  int64_t total = 0;
  auto node = [&](int32_t pos) { return useeds ? useeds[pos] : pos; };
  for (int b = 1; b < kSeedBins; ++b)
    for (int32_t pos : lst[b]) total += g.h_asum[node(pos)];
  split[0] = first[0] = first[1] = 0;
  for (int b = 1; b < kSeedBins; ++b) {
    const int64_t piece = std::max<int64_t>(kSeedPiece * seed_waves(b), total / kSeedPieces);
    split[b] = 0;
    for (int32_t pos : lst[b]) {
      const int64_t work = g.h_asum[node(pos)];
      if (work <= piece) break;
      const int64_t chunks = (g.h_deg[node(pos)] + seed_chunk(b) - 1) / seed_chunk(b);
      const int64_t want = (work + piece - 1) / piece;
      const int32_t pieces = (int32_t)((want + chunks - 1) / chunks * chunks);
      for (int32_t p = 0; p < pieces; ++p)
        items.push_back(make_int4(pos, (int32_t)split[b], p, pieces));
      split[b]++;
    }
    first[b + 1] = (int64_t)items.size();
  }
}

// WS_SPLIT with the pieces and room for their sums; without memory the slot
// stays empty. The pieces of whole-graph calls are kept there until others are
// needed.
static ef_status split_buffer(Graph &g, const std::vector<int4> &items, bool all, hipStream_t st) {
  if (items.empty()) return EF_OK;
  DevBuf &b = g.ws[WS_SPLIT];
  const size_t bytes = (sizeof(int4) + kSeedPart) * items.size();
  if (b.bytes < bytes) {
    dev_free(g, b.p, b.bytes);
    b = DevBuf{};
    g.split_kept = false;
    if (dev_alloc(g, &b.p, bytes, "seed pieces") != EF_OK) {
      b.p = nullptr;
      return EF_OK;
    }
    b.bytes = bytes;
  }
  if (all && g.split_kept) return EF_OK;
  hipError_t e = hipMemcpyAsync(b.p, items.data(), sizeof(int4) * items.size(),
                                hipMemcpyHostToDevice, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);  // a call's items go out of scope
  g.split_kept = all && e == hipSuccess;
  return hip_status(e, "upload seed pieces");
}

static void host_bins(const Graph &g, const int32_t *centres, int64_t count, Bins &b) {
  b.n_small = b.n_mid = b.n_big = b.n_tiles = 0;
  b.pairs_small = b.pairs_mid = b.pairs_big = 0;
  b.n_sblocks = 0;
  for (auto &c : b.n_smallb) c = 0;
  for (auto &c : b.n_midc) c = 0;
  for (int64_t i = 0; i < count; ++i) {
    const int64_t k = g.h_deg[centres ? centres[i] : i];
    if (k < 2) continue;
    if (k <= kSmallMax) {
      b.n_small++;
      b.n_smallb[small_bin((int32_t)k, b.thr)]++;
      b.pairs_small += k * (k - 1) / 2;
    } else if (k <= kSuper) {
      b.n_mid++;
      b.n_midc[mid_class((int32_t)k)]++;
      b.pairs_mid += k * (k - 1) / 2;
    } else {
      const int64_t ns = (k + kSuper - 1) / kSuper;
      b.n_big++;
      b.n_tiles += ns * (ns + 1) / 2;
      b.pairs_big += k * (k - 1) / 2;
      b.n_sblocks += ns;
    }
  }
}

static ef_status alloc_bins(Graph &g, Bins &b) {
  const size_t bytes = sizeof(int32_t) * (size_t)(b.n_small + 2 * b.n_mid + 16) + 8 * 256 +
                       sizeof(BigCentre) * (size_t)(b.n_big + 1) +
                       sizeof(int32_t) * (size_t)(b.n_big + 1) +
                       sizeof(TileItem) * (size_t)(b.n_tiles + 1) +
                       sizeof(int2) * (size_t)(b.n_sblocks + 1) + 4096;
  ef_status s = ws_ensure(g, WS_BINS, bytes, "work lists");
  if (s != EF_OK) return s;
  char *p = (char *)g.ws[WS_BINS].p;
  auto take = [&](size_t n) {
    char *r = p;
    p += (n + 255) & ~(size_t)255;
    return r;
  };
  b.counters = (int32_t *)take(sizeof(int32_t) * 16);
  for (int i = 0; i < 4; ++i)
    b.small[i] = (int32_t *)take(sizeof(int32_t) * (size_t)(b.n_smallb[i] + 1));
  b.mid = (int32_t *)take(sizeof(int32_t) * (size_t)(b.n_mid + 1));
  for (int c = 0; c < 3; ++c)
    b.midc[c] = (int32_t *)take(sizeof(int32_t) * (size_t)(b.n_midc[c] + 1));
  b.big = (BigCentre *)take(sizeof(BigCentre) * (size_t)(b.n_big + 1));
  b.agg_done = (int32_t *)take(sizeof(int32_t) * (size_t)(b.n_big + 1));
  b.tiles = (TileItem *)take(sizeof(TileItem) * (size_t)(b.n_tiles + 1));
  b.sblocks = (int2 *)take(sizeof(int2) * (size_t)(b.n_sblocks + 1));
  return EF_OK;
}

struct Prof {
  Graph &g;
  bool on;
  hipStream_t st;
  int used = 0;
  int idx[16];
  Prof(Graph &gg, bool o, hipStream_t s) : g(gg), on(o), st(s) {}
  ef_status init() {
    if (!on || g.ev_ready) return EF_OK;
    for (auto &e : g.ev) {
      hipError_t r = hipEventCreate(&e);
      if (r != hipSuccess) return hip_status(r, "hipEventCreate");
    }
    g.ev_ready = true;
    return EF_OK;
  }
  hipEvent_t ev(int i) { return on ? g.ev[i] : nullptr; }
  void mark(int i) {
    if (on) (void)hipEventRecord(g.ev[i], st);
  }
  double ms(int a, int b) {
    float t = 0.f;
    if (!on) return 0.0;
    if (hipEventElapsedTime(&t, g.ev[a], g.ev[b]) != hipSuccess) {
      (void)hipGetLastError();
      return 0.0;
    }
    return (double)t;
  }
};

}  // namespace efi

extern "C" ef_status ef_compute(ef_graph *h, ef_algo algo, ef_prec prec, const int32_t *seeds,
                                int32_t n_seeds, double *ef, int64_t *D, int64_t *N,
                                uint32_t flags, void *hip_stream) {
  if (!h || !ef) {
    set_error("ef_compute: null handle or output");
    return EF_ERR_ARG;
  }
  if ((algo != EF_ALGO_CLUSTER && algo != EF_ALGO_PER_SEED && algo != EF_ALGO_CLUSTER_AGG) ||
      (prec != EF_PREC_FP64 && prec != EF_PREC_FP32C)) {
    set_error("ef_compute: bad algorithm or precision");
    return EF_ERR_ARG;
  }
  if (flags & ~(EF_OUT_DEVICE | EF_PROFILE | kInternalNoReadback)) {
    set_error("ef_compute: unknown flags 0x%x", flags);
    return EF_ERR_ARG;
  }
  Graph &g = h->g;
  if (seeds && n_seeds < 0) {
    set_error("ef_compute: negative n_seeds");
    return EF_ERR_ARG;
  }
  if (seeds && n_seeds == 0) return EF_OK;
  if (seeds) {
    for (int32_t i = 0; i < n_seeds; ++i)
      if (seeds[i] < 0 || seeds[i] >= g.n) {
        set_error("ef_compute: seed %d at position %d out of range [0, %d)", seeds[i], i, g.n);
        return EF_ERR_RANGE;
      }
  }
  if (!seeds && g.n == 0) return EF_OK;
  hipStream_t st = (hipStream_t)hip_stream;
  const bool out_dev = (flags & EF_OUT_DEVICE) != 0;
  Prof prof(g, (flags & EF_PROFILE) != 0, st);
  ef_status s = prof.init();
  if (s != EF_OK) return s;
  g.stats = ef_run_stats{};

  // seeds: unique sorted list + inverse map
  const bool all = seeds == nullptr;
  std::vector<int32_t> useeds, inv;
  int32_t n_out = all ? g.n : n_seeds;
  if (!all) {
    useeds.assign(seeds, seeds + n_seeds);
    std::sort(useeds.begin(), useeds.end());
    useeds.erase(std::unique(useeds.begin(), useeds.end()), useeds.end());
    inv.resize((size_t)n_seeds);
    for (int32_t i = 0; i < n_seeds; ++i)
      inv[i] = (int32_t)(std::lower_bound(useeds.begin(), useeds.end(), seeds[i]) - useeds.begin());
  }
  const bool per_seed = !all || algo == EF_ALGO_PER_SEED;
  const int32_t n_work = all ? g.n : (int32_t)useeds.size();

  // work lists of the pair loop
  Bins b;
  if (all) {
    b.thr = g.thr;
    b.n_small = g.all_small;
    for (int k = 2; k <= kSmallMax; ++k) b.n_smallb[small_bin(k, b.thr)] += g.all_small_deg[k];
    b.n_mid = g.all_mid;
    for (int c = 0; c < 3; ++c) b.n_midc[c] = g.all_midc[c];
    b.n_big = g.all_big;
    b.n_tiles = g.all_tiles;
    b.pairs_small = g.all_pairs_small;
    b.pairs_mid = g.all_pairs_mid;
    b.pairs_big = g.all_pairs_big;
    b.n_sblocks = g.all_sblocks;
  } else {
    b.thr = g.thr;
    host_bins(g, useeds.data(), (int64_t)useeds.size(), b);
  }
  if ((s = alloc_bins(g, b)) != EF_OK) return s;
  const ComputeWs L = compute_ws(g, prec == EF_PREC_FP64, b.n_tiles, n_work, !per_seed);
  hipError_t e = hipSuccess;
  // device seed arrays: the unique work list (all nodes: none, position =
  // node id), the inverse map, and output positions by seed degree bin
  int32_t *d_useeds = nullptr, *d_inv = nullptr;
  SeedLists ls;
  std::vector<int4> items;  // pieces of a call with seeds
  int64_t split[kSeedBins], first[kSeedBins + 1];
  if (per_seed && g.h_asum.empty() && g.n > 0) {
    g.h_asum.resize((size_t)g.n);
    e = hipMemcpy(g.h_asum.data(), g.asum, sizeof(int64_t) * (size_t)g.n, hipMemcpyDeviceToHost);
    if (e != hipSuccess) {
      g.h_asum.clear();
      return hip_status(e, "copy neighbour-degree sums");
    }
  }
  auto seed_bin = [&](int32_t v) {
    const int32_t k = g.h_deg[v];
    if (k <= kSeedBin0 && g.h_asum[v] <= kSeedWaveWork) return 0;
    return k <= kSeedBin1 ? 1 : k <= kSeedBin2 ? 2 : k <= kSeedBin3 ? 3 : 4;
  };
  // largest 2-hop work first
  auto by_work = [&](int32_t a, int32_t c) {
    const int64_t wa = g.h_asum[a], wc = g.h_asum[c];
    return wa != wc ? wa > wc : a < c;
  };
  if (per_seed && all) {
    if (!g.ps_ready) {
      std::vector<int32_t> lst[kSeedBins];
      for (int32_t v = 0; v < g.n; ++v) lst[seed_bin(v)].push_back(v);
      // (the handle gets the lists when all are there)
      KeptArrays kept(g);
      int32_t *list[kSeedBins];
      for (int bin = 0; bin < kSeedBins; ++bin) {
        std::sort(lst[bin].begin(), lst[bin].end(), by_work);
        if ((s = kept.add((void **)&list[bin], lst[bin].data(),
                          sizeof(int32_t) * lst[bin].size(), "seed lists")) != EF_OK)
          return s;
      }
      kept.keep();
      for (int bin = 0; bin < kSeedBins; ++bin) {
        g.ps_list[bin] = list[bin];
        g.n_ps[bin] = (int64_t)lst[bin].size();
      }
      seed_pieces(g, nullptr, lst, g.h_ps_items, g.ps_split, g.ps_first);
      g.ps_ready = true;
    }
    for (int bin = 0; bin < kSeedBins; ++bin) {
      ls.list[bin] = g.ps_list[bin];
      ls.count[bin] = g.n_ps[bin];
    }
  } else if (per_seed) {
    std::vector<int32_t> lst[kSeedBins];
    std::vector<int32_t> order(useeds.size());
    std::iota(order.begin(), order.end(), 0);
    std::sort(order.begin(), order.end(),
              [&](int32_t a, int32_t c) { return by_work(useeds[a], useeds[c]); });
    for (int32_t i : order) lst[seed_bin(useeds[i])].push_back(i);
    // one upload: the seeds, the bins' lists, the inverse map
    std::vector<int32_t> up = useeds;
    up.reserve(useeds.size() * 2 + inv.size());
    for (int bin = 0; bin < kSeedBins; ++bin) up.insert(up.end(), lst[bin].begin(), lst[bin].end());
    up.insert(up.end(), inv.begin(), inv.end());
    if ((s = ws_ensure(g, WS_SEEDS, sizeof(int32_t) * (up.size() + 4), "seed lists")) != EF_OK)
      return s;
    d_useeds = (int32_t *)g.ws[WS_SEEDS].p;
    int32_t *p = d_useeds + useeds.size();
    for (int bin = 0; bin < kSeedBins; ++bin) {
      ls.list[bin] = p;
      ls.count[bin] = (int64_t)lst[bin].size();
      p += lst[bin].size();
    }
    d_inv = p;
    e = hipMemcpyAsync(d_useeds, up.data(), sizeof(int32_t) * up.size(), hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);  // host vectors go out of scope
    if (e != hipSuccess) return hip_status(e, "upload seeds");
    seed_pieces(g, useeds.data(), lst, items, split, first);
  }
  if (per_seed && ls.count[kSeedBins - 1] > 0) {
    const size_t words = ((size_t)g.n + 31) / 32;
    const size_t need = sizeof(uint32_t) * words * (size_t)ls.count[kSeedBins - 1];
    const bool fresh = g.ws[WS_BITMAP].bytes < need;
    if ((s = ws_ensure(g, WS_BITMAP, need, "membership bitmaps")) != EF_OK) return s;
    if (fresh) {
      e = hipMemsetAsync(g.ws[WS_BITMAP].p, 0, g.ws[WS_BITMAP].bytes, st);
      if (e != hipSuccess) return hip_status(e, "clear bitmaps");
    }
  }

  // the block last: the buffers above may take the place of a larger one
  if ((s = ws_ensure(g, WS_MAIN, L.bytes, "workspace")) != EF_OK) return s;
  struct MainUse {
    Graph &g;
    explicit MainUse(Graph &gg) : g(gg) { g.main_busy = true; }
    ~MainUse() { g.main_busy = false; }
  } main_use(g);
  char *const ws = (char *)g.ws[WS_MAIN].p;
  void *const ws_R = ws + L.R, *const ws_Z = ws + L.Z;
  TriSlot *const ws_Y = (TriSlot *)(ws + L.Y);
  int64_t *const ws_ZT = (int64_t *)(ws + L.ZT);
  // outputs of the unique work list: straight into the caller's device arrays
  // when possible, else into staging
  double *ef_w = (double *)(ws + L.out);
  int64_t *D_w = (int64_t *)(ef_w + std::max(n_work, 1)), *N_w = D_w + std::max(n_work, 1);
  if (all && out_dev) {
    ef_w = ef;
    if (D) D_w = D;
    if (N) N_w = N;
  }
  // FP32C: [0] positions recomputed by pass 2, [1] finalised in FP64
  int32_t *cnt = (int32_t *)(ws + L.out + 24 * (size_t)n_work);
  int32_t *listed = (int32_t *)(ws + L.flag);
  uint8_t *flag_bytes = (uint8_t *)(listed + (n_work > kPass2Scan ? n_work : 0));

  // whole-graph calls bin every node with the graph's thresholds: their
  // lists are kept and reused (not while the stream is being captured, so
  // that a captured graph bins by itself)
  const int32_t *centres = per_seed ? d_useeds : nullptr;
  // (the pieces only save time: without memory for them, or in a captured
  // call, whose replays must not depend on them, no seed is cut)
  const bool eager = !capturing(st);
  g.main_captured |= !eager;
  if (per_seed && eager) {
    const std::vector<int4> &pc = all ? g.h_ps_items : items;
    if ((s = split_buffer(g, pc, all, st)) != EF_OK) return s;
    if (!pc.empty() && g.ws[WS_SPLIT].p) {
      std::copy_n(all ? g.ps_split : split, kSeedBins, ls.split);
      std::copy_n(all ? g.ps_first : first, kSeedBins + 1, ls.first);
      ls.items = (const int4 *)g.ws[WS_SPLIT].p;
      ls.parts = (char *)g.ws[WS_SPLIT].p + sizeof(int4) * pc.size();
    }
  }
  // (a batch captures right after a call that kept its lists, and no other call
  // of its handle comes between: its replays read those)
  const bool replay_own = (flags & kInternalNoReadback) != 0;
  const bool whole = centres == nullptr && (eager || replay_own);
  const bool reuse = whole && g.bins_kept && g.bins_buf == g.ws[WS_BINS].p &&
                     g.bins_thr.t8 == b.thr.t8 && g.bins_thr.t16 == b.thr.t16 &&
                     g.bins_thr.t32 == b.thr.t32;
  if (prec == EF_PREC_FP64 && eager && (s = score_table(g, st, !out_dev)) != EF_OK)
    return s;
  const bool tab = eager || replay_own;
  prof.mark(0);
  if (!reuse) {
    e = launch_bin_centres(g, centres, n_work, b, st);
    if (e != hipSuccess) return hip_status(e, "binning");
  }
  g.bins_kept = reuse || (whole && eager);
  g.bins_thr = b.thr;
  g.bins_buf = g.ws[WS_BINS].p;
  prof.mark(1);
  e = launch_pairs(g, prec, b, ws_R, ws + L.rec, st, tab, prof.ev(2), prof.ev(3), prof.ev(4),
                   algo == EF_ALGO_CLUSTER_AGG ? b.agg_done : nullptr);
  if (e != hipSuccess) return hip_status(e, "pair loop");
  prof.mark(5);
  if (!per_seed) {
    e = launch_triangles(g, prec, ws_Y, ws_Z, ws_ZT, st);
    if (e != hipSuccess) return hip_status(e, "triangle pass");
    prof.mark(6);
    e = launch_finalize_cluster(g, prec, ws_R, ws_Y, ws_Z, ws_ZT, ef_w, D_w, N_w, flag_bytes,
                                prec == EF_PREC_FP32C ? cnt : nullptr, st);
    if (e != hipSuccess) return hip_status(e, "finalize");
    prof.mark(7);
  } else {
    if (prec == EF_PREC_FP32C) e = launch_zero_i32(cnt, 2, st);
    if (e == hipSuccess)
      e = launch_per_seed(g, prec, d_useeds, ls, ws_R, (uint32_t *)g.ws[WS_BITMAP].p, ef_w, D_w,
                          N_w, flag_bytes, st, prof.ev(6));
    if (e != hipSuccess) return hip_status(e, "per-seed stream");
    prof.mark(7);
  }
  if (prec == EF_PREC_FP32C) {
    e = launch_pass2(g, per_seed ? d_useeds : nullptr, flag_bytes, n_work, listed, cnt, ef_w,
                     D_w, st);
    if (e != hipSuccess) return hip_status(e, "pass 2");
  }
  prof.mark(8);

  // deliver outputs
  int32_t hc[2] = {0, 0};
  bool counted = false;
  if (!all) {
    if (out_dev) {
      e = launch_gather_outputs(d_inv, n_seeds, ef_w, D_w, N_w, ef, D, N, st);
      if (e != hipSuccess) return hip_status(e, "scatter outputs");
    } else {
      // the staged EF, D and N and the counters lie one after the other: one copy
      std::vector<int64_t> h(3 * (size_t)n_work + 1);
      e = hipMemcpyAsync(h.data(), ef_w, sizeof(int64_t) * h.size(), hipMemcpyDeviceToHost, st);
      if (e == hipSuccess) e = hipStreamSynchronize(st);
      if (e != hipSuccess) return hip_status(e, "copy outputs");
      const double *hef = (const double *)h.data();
      const int64_t *hD = h.data() + n_work, *hN = hD + n_work;
      std::memcpy(hc, hN + n_work, sizeof(hc));
      counted = true;
      for (int32_t i = 0; i < n_seeds; ++i) {
        ef[i] = hef[inv[i]];
        if (D) D[i] = hD[inv[i]];
        if (N) N[i] = hN[inv[i]];
      }
    }
  } else if (!out_dev && n_out <= kOneCopy) {
    std::vector<int64_t> h(3 * (size_t)n_out + 1);
    e = hipMemcpyAsync(h.data(), ef_w, sizeof(int64_t) * h.size(), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return hip_status(e, "copy outputs");
    const size_t bytes = sizeof(int64_t) * (size_t)n_out;
    std::memcpy(ef, h.data(), bytes);
    if (D) std::memcpy(D, h.data() + n_out, bytes);
    if (N) std::memcpy(N, h.data() + 2 * (size_t)n_out, bytes);
    std::memcpy(hc, h.data() + 3 * (size_t)n_out, sizeof(hc));
    counted = true;
  } else if (!out_dev) {
    e = hipMemcpyAsync(ef, ef_w, sizeof(double) * (size_t)n_out, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess && D)
      e = hipMemcpyAsync(D, D_w, sizeof(int64_t) * (size_t)n_out, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess && N)
      e = hipMemcpyAsync(N, N_w, sizeof(int64_t) * (size_t)n_out, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return hip_status(e, "copy outputs");
  }
  g.stats.pair_tiles = b.n_tiles;
  g.stats.pairs_small = b.pairs_small;
  g.stats.pairs_mid = b.pairs_mid;
  g.stats.pairs_big = b.pairs_big;
  g.stats.seeds = n_work;
  if (prec == EF_PREC_FP64 && !out_dev) g.score_pending = false;  // st has been waited for
  if ((prof.on || !out_dev) && !(flags & kInternalNoReadback)) {
    if (prec == EF_PREC_FP32C && !counted)
      e = hipMemcpyAsync(hc, cnt, sizeof(hc), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess && (prof.on || !counted)) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return hip_status(e, "read counters");
    if (prec != EF_PREC_FP32C) hc[0] = hc[1] = 0;  // not written
    g.stats.promoted = hc[0];
    g.stats.fp64_finalized = hc[1];
  }
  if (prof.on) {
    g.stats.t_bin_ms = prof.ms(0, 1);
    g.stats.t_pairs_small_ms = prof.ms(1, 2);
    g.stats.t_pairs_mid_ms = prof.ms(2, 3);
    g.stats.t_pairs_big_ms = prof.ms(3, 4);
    g.stats.t_pairs_ms = prof.ms(1, 4);
    g.stats.t_reduce_ms = prof.ms(4, 5);
    if (!per_seed) {
      g.stats.t_triangles_ms = prof.ms(5, 6);
      g.stats.t_finalize_ms = prof.ms(6, 7);
    } else {
      g.stats.t_stream_ms = prof.ms(5, 7);
    }
    g.stats.t_pass2_ms = prof.ms(7, 8);
    g.stats.t_total_ms = prof.ms(0, 8);
  }
  return EF_OK;
}

extern "C" ef_status ef_compute_j3(ef_graph *h, ef_prec prec, const int32_t *seeds,
                                   int32_t n_seeds, double *ef, int64_t *D, int64_t *N,
                                   uint32_t flags, void *hip_stream) {
  if (!h || !ef) {
    set_error("ef_compute_j3: null handle or output");
    return EF_ERR_ARG;
  }
  if (prec != EF_PREC_FP64 && prec != EF_PREC_FP32C) {
    set_error("ef_compute_j3: bad precision");
    return EF_ERR_ARG;
  }
  if (flags & ~(EF_OUT_DEVICE | EF_PROFILE)) {
    set_error("ef_compute_j3: unknown flags 0x%x", flags);
    return EF_ERR_ARG;
  }
  Graph &g = h->g;
  if (seeds && n_seeds < 0) {
    set_error("ef_compute_j3: negative n_seeds");
    return EF_ERR_ARG;
  }
  if (seeds && n_seeds == 0) return EF_OK;
  if (seeds)
    for (int32_t i = 0; i < n_seeds; ++i)
      if (seeds[i] < 0 || seeds[i] >= g.n) {
        set_error("ef_compute_j3: seed %d at position %d out of range [0, %d)", seeds[i], i,
                  g.n);
        return EF_ERR_RANGE;
      }
  if (!seeds && g.n == 0) return EF_OK;
  hipStream_t st = (hipStream_t)hip_stream;
  const bool out_dev = (flags & EF_OUT_DEVICE) != 0;
  Prof prof(g, (flags & EF_PROFILE) != 0, st);
  ef_status s = prof.init();
  if (s != EF_OK) return s;
  g.stats = ef_run_stats{};
  hipError_t e = hipSuccess;

  // host copies of the per-node sums (work estimates and the int64 bound)
  if (g.h_asum.empty() && g.n > 0) {
    g.h_asum.resize((size_t)g.n);
    e = hipMemcpy(g.h_asum.data(), g.asum, sizeof(int64_t) * (size_t)g.n, hipMemcpyDeviceToHost);
    if (e != hipSuccess) {
      g.h_asum.clear();
      return hip_status(e, "copy neighbour-degree sums");
    }
  }
  if (g.h_qa.empty() && g.n > 0) {
    g.h_qa.resize((size_t)g.n);
    e = hipMemcpy(g.h_qa.data(), g.qa, sizeof(longlong2) * (size_t)g.n, hipMemcpyDeviceToHost);
    if (e != hipSuccess) {
      g.h_qa.clear();
      return hip_status(e, "copy neighbour-degree moments");
    }
  }
  // N_3(s) is the two-event degree sum D_2(s), at most its triangle-free
  // closed form; every cluster degree is below k_s + 3 k_max
  auto n3_bound = [&](int32_t v) {
    const double k = g.h_deg[v], A = (double)g.h_asum[v];
    const double Q = (double)g.h_qa[v].x, A2 = (double)g.h_qa[v].y;
    return std::max(0.0, k * (k - 4) * (k - 2) + (3 * k - 7) * A + Q + A2 - k * k);
  };
  const bool all = seeds == nullptr;
  std::vector<int32_t> useeds, inv;
  if (!all) {
    useeds.assign(seeds, seeds + n_seeds);
    std::sort(useeds.begin(), useeds.end());
    useeds.erase(std::unique(useeds.begin(), useeds.end()), useeds.end());
    inv.resize((size_t)n_seeds);
    for (int32_t i = 0; i < n_seeds; ++i)
      inv[i] = (int32_t)(std::lower_bound(useeds.begin(), useeds.end(), seeds[i]) - useeds.begin());
  }
  const int32_t n_work = all ? g.n : (int32_t)useeds.size();
  const double dmax = (double)g.info.max_degree;
  for (int32_t i = 0; i < n_work; ++i) {
    const int32_t v = all ? i : useeds[i];
    if (n3_bound(v) * ((double)g.h_deg[v] + 3 * dmax) > 4.0e18) {
      set_error("ef_compute_j3: the sums of seed %d (degree %d) could exceed int64", v,
                g.h_deg[v]);
      return EF_ERR_OVERFLOW;
    }
  }
  // items: the arcs of the seeds, largest seeds first
  auto order_of = [&](std::vector<int32_t> &ord, std::vector<int64_t> &off) {
    std::sort(ord.begin(), ord.end(), [&](int32_t a, int32_t c) {
      const double wa = n3_bound(a), wc = n3_bound(c);
      return wa != wc ? wa > wc : a < c;
    });
    off.assign(ord.size() + 1, 0);
    for (size_t i = 0; i < ord.size(); ++i) off[i + 1] = off[i] + g.h_deg[ord[i]];
  };
  const int64_t nnz = std::max<int64_t>(g.nnz, 1);
  if ((s = ws_ensure(g, WS_J3P, (2 * sizeof(long long) + sizeof(double)) * (size_t)nnz,
                     "per-arc partial sums")) != EF_OK)
    return s;
  long long *PN = (long long *)g.ws[WS_J3P].p, *PD = PN + nnz;
  double *PS = (double *)(PD + nnz);
  const int32_t *d_ord = nullptr;
  const int64_t *d_off = nullptr;
  int64_t n_items = 0;
  int32_t *d_useeds = nullptr;
  if (all) {
    if (!g.j3_seeds) {
      std::vector<int32_t> ord((size_t)g.n);
      std::iota(ord.begin(), ord.end(), 0);
      std::vector<int64_t> off;
      order_of(ord, off);
      KeptArrays kept(g);
      int32_t *seeds_d;
      int64_t *off_d;
      if ((s = kept.add((void **)&seeds_d, ord.data(), sizeof(int32_t) * ord.size(),
                        "j3 order")) != EF_OK ||
          (s = kept.add((void **)&off_d, off.data(), sizeof(int64_t) * off.size(),
                        "j3 offsets")) != EF_OK)
        return s;
      kept.keep();
      g.j3_seeds = seeds_d;
      g.j3_off = off_d;
    }
    d_ord = g.j3_seeds;
    d_off = g.j3_off;
    n_items = g.nnz;
  } else {
    std::vector<int32_t> ord(useeds);
    std::vector<int64_t> off;
    order_of(ord, off);
    n_items = off.back();
    const size_t bytes = sizeof(int64_t) * off.size() + sizeof(int32_t) * (2 * useeds.size()) + 64;
    if ((s = ws_ensure(g, WS_J3, bytes, "j3 seed lists")) != EF_OK) return s;
    int64_t *po = (int64_t *)g.ws[WS_J3].p;
    int32_t *pord = (int32_t *)(po + off.size());
    d_useeds = pord + ord.size();
    e = hipMemcpyAsync(po, off.data(), sizeof(int64_t) * off.size(), hipMemcpyHostToDevice, st);
    if (e == hipSuccess)
      e = hipMemcpyAsync(pord, ord.data(), sizeof(int32_t) * ord.size(), hipMemcpyHostToDevice,
                         st);
    if (e == hipSuccess)
      e = hipMemcpyAsync(d_useeds, useeds.data(), sizeof(int32_t) * useeds.size(),
                         hipMemcpyHostToDevice, st);
    if (e != hipSuccess) return hip_status(e, "upload seeds");
    d_ord = pord;
    d_off = po;
  }
  // outputs of the unique work list (staging unless they can go straight to
  // the caller's device arrays) and flag bytes
  const size_t out_bytes = (sizeof(double) + 2 * sizeof(int64_t)) * (size_t)std::max(n_work, 1);
  if ((s = ws_ensure(g, WS_UOUT, out_bytes, "output staging")) != EF_OK) return s;
  if ((s = ws_ensure(g, WS_FLAG, (sizeof(int32_t) + 1) * (size_t)std::max(n_work, 1),
                     "flag list")) != EF_OK)
    return s;
  double *ef_w = (double *)g.ws[WS_UOUT].p;
  int64_t *D_w = (int64_t *)(ef_w + std::max(n_work, 1)), *N_w = D_w + std::max(n_work, 1);
  if (all && out_dev) {
    ef_w = ef;
    if (D) D_w = D;
    if (N) N_w = N;
  }
  int32_t *fpos = (int32_t *)g.ws[WS_FLAG].p;
  uint8_t *fl = (uint8_t *)(fpos + std::max(n_work, 1));
  // per-bin item lists and their counts
  if ((s = ws_ensure(g, WS_J3L, sizeof(int32_t) * (5 * (size_t)std::max<int64_t>(n_items, 1) + 8),
                     "item lists")) != EF_OK)
    return s;
  int32_t *j3_lists = (int32_t *)g.ws[WS_J3L].p;
  int32_t *j3_counts = j3_lists + 5 * std::max<int64_t>(n_items, 1);
  const bool fp64 = prec == EF_PREC_FP64;
  const bool tab = !capturing(st);
  if (fp64 && tab && (s = score_table(g, st, !out_dev)) != EF_OK) return s;
  prof.mark(0);
  e = launch_j3_items(g, fp64, tab, all, d_ord, d_off, n_work, n_items, j3_lists, j3_counts, PN, PD,
                      PS, st);
  if (e != hipSuccess) return hip_status(e, "three-event items");
  prof.mark(1);
  e = launch_j3_finish(g, fp64, PN, PD, PS, d_useeds, nullptr, n_work, ef_w, D_w, N_w,
                       fp64 ? nullptr : fl, st);
  if (e != hipSuccess) return hip_status(e, "three-event finalize");
  prof.mark(2);
  int32_t n_flag = 0;
  if (!fp64) {
    // seeds whose FP32 EF cancels: their items again in FP64
    std::vector<uint8_t> hf((size_t)n_work);
    e = hipMemcpyAsync(hf.data(), fl, (size_t)n_work, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return hip_status(e, "read flags");
    std::vector<int32_t> fpos_h, ford;
    for (int32_t i = 0; i < n_work; ++i)
      if (hf[i]) {
        fpos_h.push_back(i);
        ford.push_back(all ? i : useeds[i]);
      }
    n_flag = (int32_t)fpos_h.size();
    if (n_flag > 0) {
      std::vector<int64_t> foff;
      order_of(ford, foff);
      const size_t bytes = sizeof(int64_t) * foff.size() + sizeof(int32_t) * ford.size() + 64;
      if ((s = ws_ensure(g, WS_SEEDS, bytes, "promoted seeds")) != EF_OK) return s;
      int64_t *po = (int64_t *)g.ws[WS_SEEDS].p;
      int32_t *pord = (int32_t *)(po + foff.size());
      e = hipMemcpyAsync(po, foff.data(), sizeof(int64_t) * foff.size(), hipMemcpyHostToDevice,
                         st);
      if (e == hipSuccess)
        e = hipMemcpyAsync(pord, ford.data(), sizeof(int32_t) * ford.size(),
                           hipMemcpyHostToDevice, st);
      if (e == hipSuccess)
        e = hipMemcpyAsync(fpos, fpos_h.data(), sizeof(int32_t) * fpos_h.size(),
                           hipMemcpyHostToDevice, st);
      if (e == hipSuccess && tab && (s = score_follow(g, st)) != EF_OK) return s;
      if (e == hipSuccess)
        e = launch_j3_items(g, true, tab, false, pord, po, n_flag, foff.back(), j3_lists, j3_counts,
                            PN, PD, PS, st);
      if (e == hipSuccess)
        e = launch_j3_finish(g, true, PN, PD, PS, d_useeds, fpos, n_flag, ef_w, D_w, N_w,
                             nullptr, st);
      if (e == hipSuccess) e = hipStreamSynchronize(st);
      if (e != hipSuccess) return hip_status(e, "three-event FP64 recompute");
    }
  }
  prof.mark(3);
  // deliver outputs
  if (!all) {
    if (out_dev) {
      if ((s = ws_ensure(g, WS_SEEDS, sizeof(int32_t) * inv.size() + 64, "inverse map")) != EF_OK)
        return s;
      int32_t *d_inv = (int32_t *)g.ws[WS_SEEDS].p;
      e = hipMemcpyAsync(d_inv, inv.data(), sizeof(int32_t) * inv.size(), hipMemcpyHostToDevice,
                         st);
      if (e == hipSuccess) e = launch_gather_outputs(d_inv, n_seeds, ef_w, D_w, N_w, ef, D, N, st);
      if (e != hipSuccess) return hip_status(e, "scatter outputs");
    } else {
      std::vector<double> hef((size_t)n_work);
      std::vector<int64_t> hD((size_t)n_work), hN((size_t)n_work);
      e = hipMemcpyAsync(hef.data(), ef_w, sizeof(double) * n_work, hipMemcpyDeviceToHost, st);
      if (e == hipSuccess)
        e = hipMemcpyAsync(hD.data(), D_w, sizeof(int64_t) * n_work, hipMemcpyDeviceToHost, st);
      if (e == hipSuccess)
        e = hipMemcpyAsync(hN.data(), N_w, sizeof(int64_t) * n_work, hipMemcpyDeviceToHost, st);
      if (e == hipSuccess) e = hipStreamSynchronize(st);
      if (e != hipSuccess) return hip_status(e, "copy outputs");
      for (int32_t i = 0; i < n_seeds; ++i) {
        ef[i] = hef[inv[i]];
        if (D) D[i] = hD[inv[i]];
        if (N) N[i] = hN[inv[i]];
      }
    }
  } else if (!out_dev) {
    e = hipMemcpyAsync(ef, ef_w, sizeof(double) * (size_t)g.n, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess && D)
      e = hipMemcpyAsync(D, D_w, sizeof(int64_t) * (size_t)g.n, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess && N)
      e = hipMemcpyAsync(N, N_w, sizeof(int64_t) * (size_t)g.n, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return hip_status(e, "copy outputs");
  }
  if (fp64 && !out_dev) g.score_pending = false;  // st has been waited for
  g.stats.seeds = n_work;
  g.stats.promoted = n_flag;
  if (prof.on) {
    e = hipStreamSynchronize(st);
    if (e != hipSuccess) return hip_status(e, "profile");
    g.stats.t_stream_ms = prof.ms(0, 1);
    g.stats.t_finalize_ms = prof.ms(1, 2);
    g.stats.t_pass2_ms = prof.ms(2, 3);
    g.stats.t_total_ms = prof.ms(0, 3);
  }
  return EF_OK;
}

// Top-k over device EF values of the graph's nodes, in the handle's workspace;
// host outputs go through a device staging area after the top-k scratch.
static ef_status topk_device_values(Graph &g, const double *ef_all, int32_t k, int32_t *nodes,
                                    double *ef, bool out_dev, hipStream_t st) {
  // (staged outputs lie apart from the values)
  const bool direct = topk_direct(ef_all, g.n, k, out_dev ? nodes : nullptr, out_dev ? ef : nullptr);
  const size_t sort_bytes = direct ? 0 : (topk_scratch_bytes(g.n, k) + 255) & ~(size_t)255;
  const size_t node_bytes = (sizeof(int32_t) * (size_t)k + 255) & ~(size_t)255;
  const size_t stage = out_dev ? 0 : node_bytes + sizeof(double) * (size_t)k;
  ef_status s = ws_ensure(g, WS_TOPK, sort_bytes + stage, "top-k scratch");
  if (s != EF_OK) return s;
  char *base = (char *)g.ws[WS_TOPK].p;
  int32_t *nodes_d = nodes;
  double *ef_d = ef;
  if (!out_dev) {
    nodes_d = (int32_t *)(base + sort_bytes);
    ef_d = (double *)(base + sort_bytes + node_bytes);
  }
  hipError_t e = launch_topk(ef_all, g.n, k, base, sort_bytes, nodes_d, ef ? ef_d : nullptr, st);
  if (e != hipSuccess) return hip_status(e, "top-k");
  if (!out_dev) {
    e = hipMemcpyAsync(nodes, nodes_d, sizeof(int32_t) * (size_t)k, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess && ef)
      e = hipMemcpyAsync(ef, ef_d, sizeof(double) * (size_t)k, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return hip_status(e, "copy top-k");
  }
  return EF_OK;
}

extern "C" ef_status ef_topk(ef_graph *h, ef_algo algo, ef_prec prec, int32_t k, int32_t *nodes,
                             double *ef, uint32_t flags, void *hip_stream) {
  if (!h || !nodes) {
    set_error("ef_topk: null handle or output");
    return EF_ERR_ARG;
  }
  Graph &g = h->g;
  if (k < 0 || k > g.n) {
    set_error("ef_topk: k=%d outside [0, n=%d]", k, g.n);
    return EF_ERR_ARG;
  }
  if (flags & ~(EF_OUT_DEVICE | EF_PROFILE)) {
    set_error("ef_topk: unknown flags 0x%x", flags);
    return EF_ERR_ARG;
  }
  if (k == 0) return EF_OK;
  const size_t n = (size_t)g.n;
  ef_status s = ws_ensure(g, WS_OUT, sizeof(double) * n + 2 * sizeof(int64_t) * n + 2048,
                          "all-node outputs");
  if (s != EF_OK) return s;
  double *ef_all = (double *)g.ws[WS_OUT].p;
  int64_t *D_all = (int64_t *)(ef_all + n);
  int64_t *N_all = D_all + n;
  s = ef_compute(h, algo, prec, nullptr, 0, ef_all, D_all, N_all,
                 EF_OUT_DEVICE | (flags & EF_PROFILE), hip_stream);
  if (s != EF_OK) return s;
  return topk_device_values(g, ef_all, k, nodes, ef, (flags & EF_OUT_DEVICE) != 0,
                            (hipStream_t)hip_stream);
}

extern "C" ef_status ef_topk_values(ef_graph *h, const double *ef_in, int32_t k, int32_t *nodes,
                                    double *ef, uint32_t flags, void *hip_stream) {
  if (!h || !nodes || (!ef_in && k > 0)) {
    set_error("ef_topk_values: null handle, values or output");
    return EF_ERR_ARG;
  }
  Graph &g = h->g;
  if (k < 0 || k > g.n) {
    set_error("ef_topk_values: k=%d outside [0, n=%d]", k, g.n);
    return EF_ERR_ARG;
  }
  if (flags & ~EF_OUT_DEVICE) {
    set_error("ef_topk_values: unknown flags 0x%x", flags);
    return EF_ERR_ARG;
  }
  if (k == 0) return EF_OK;
  return topk_device_values(g, ef_in, k, nodes, ef, (flags & EF_OUT_DEVICE) != 0,
                            (hipStream_t)hip_stream);
}
