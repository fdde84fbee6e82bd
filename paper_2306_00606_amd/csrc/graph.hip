// Graph preprocessing on the device: degrees, arc sources, reverse arcs, the
// packed (id, degree) adjacency, neighbour-degree sums and the
// degree-oriented half adjacency used by the triangle pass.
//
// The orientation ranks nodes by (degree, id): rank(a) < rank(b) when
// k_a < k_b, or k_a == k_b and a < b. up(u) = {w in N(u) : rank(w) > rank(u)}
// keeps every undirected edge exactly once and bounds |up(u)| by
// sqrt(2 * edges), which keeps the triangle pass short on skewed graphs.
// Each up(u) is stored in rank order, so the part of up(u) ranked above one
// of its members w is the contiguous tail after w. The triangle pass lists a
// triangle u < w < x at its middle node w, walking for every lower neighbour
// u of w that tail of up(u) against up(w); the per-node lists of those tails
// ("segments": slot of {u, w} in up(u), tail length, k_u + k_w) are built
// here, and every arc gets the index of the triangle record that holds the
// credits to its source node (-1 when no walk writes one).
#include <hipcub/hipcub.hpp>

#include "ef_internal.h"

namespace efi {

__device__ __forceinline__ bool rank_less(int32_t a, int32_t ka, int32_t b, int32_t kb) {
  return ka < kb || (ka == kb && a < b);
}

// Checks on the device while the graph is prepared (ctl, 64 ints, cleared
// first): [kCtlCol] a neighbour id lies outside [0, n), [kCtlArc] a row with a
// self-loop, not ascending, or an arc without its reverse, [kCtlStop] set by
// k_gate when the arrays cannot be filled, [kCtlUp] up-arcs found, [kCtlZero]
// triangle slots to clear. Kernels that index by neighbour ids leave when
// kCtlCol is set, those after the gate when kCtlStop is, so the host reads the
// outcome once, at the end.
// a simple symmetric graph has exactly nnz / 2 up-arcs: the up-arc arrays are
// sized for that many
__global__ void k_gate(int32_t *__restrict__ ctl, const int32_t *__restrict__ up_total,
                       int64_t nnz, bool validate) {
  const int32_t up = *up_total;
  ctl[kCtlUp] = up;
  ctl[kCtlStop] = (ctl[kCtlCol] || (validate && ctl[kCtlArc]) || 2 * (int64_t)up != nnz) ? 1 : 0;
}

__global__ void k_ctl_zero_total(int32_t *__restrict__ ctl, const int32_t *__restrict__ total) {
  ctl[kCtlZero] = *total;
}

// degrees; clears the control record
__global__ void k_degree(const int32_t *__restrict__ row_ptr, int32_t n,
                         int32_t *__restrict__ deg, int32_t *__restrict__ ctl) {
  if (blockIdx.x == 0 && threadIdx.x < 64) ctl[threadIdx.x] = 0;
  for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n;
       v += (int64_t)gridDim.x * blockDim.x)
    deg[v] = row_ptr[v + 1] - row_ptr[v];
}

// src[e] = the row that holds arc e (binary search over row_ptr); checks the
// neighbour ids.
__global__ void k_arc_src(const int32_t *__restrict__ row_ptr, const int32_t *__restrict__ col,
                          int32_t n, int64_t nnz, int32_t *__restrict__ src,
                          int32_t *__restrict__ ctl) {
  bool bad = false;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < nnz;
       e += (int64_t)gridDim.x * blockDim.x) {
    int32_t lo = 0, hi = n;  // find largest v with row_ptr[v] <= e
    while (hi - lo > 1) {
      int32_t mid = (lo + hi) >> 1;
      if (row_ptr[mid] <= e) lo = mid; else hi = mid;
    }
    src[e] = lo;
    bad |= (uint32_t)col[e] >= (uint32_t)n;
  }
  // one atomic per wavefront that saw a bad id
  if (__ballot(bad) && (threadIdx.x & 63) == 0) atomicOr(&ctl[kCtlCol], 1);
}

__global__ void k_arc_rev(const int32_t *__restrict__ row_ptr, const int32_t *__restrict__ col,
                          const int32_t *__restrict__ src, const int32_t *__restrict__ deg,
                          int64_t nnz, int32_t *__restrict__ rev, int32_t *__restrict__ rrev,
                          int2 *__restrict__ adj2, int32_t *__restrict__ upflag,
                          int32_t *__restrict__ ctl, bool validate) {
  if (ctl[kCtlCol]) return;
  bool bad = false;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < nnz;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int32_t s = src[e], a = col[e];
    int32_t lo = row_ptr[a], hi = row_ptr[a + 1];  // first position with col >= s
    while (lo < hi) {
      int32_t mid = (lo + hi) >> 1;
      if (col[mid] < s) lo = mid + 1; else hi = mid;
    }
    // on a valid (symmetric) graph the reverse arc is always found; keep the
    // index inside the row otherwise
    const bool found = lo < row_ptr[a + 1] && col[lo] == s;
    const int32_t r = found ? lo : (int32_t)e;
    rev[e] = r;
    rrev[e] = r;  // until the rows of mid and big centres remap it
    // (in ascending rows the search finds every reverse arc there is; a row
    // out of order is bad by itself)
    bad |= !found || a == s || (e > row_ptr[s] && col[e - 1] >= a);
    const int32_t ka = deg[a];
    adj2[e] = make_int2(a, ka);
    upflag[e] = rank_less(s, deg[s], a, ka) ? 1 : 0;
  }
  if (validate && __ballot(bad) && (threadIdx.x & 63) == 0) atomicOr(&ctl[kCtlArc], 1);
}

__global__ void k_up_fill(const int32_t *__restrict__ row_ptr, const int32_t *__restrict__ col,
                          const int32_t *__restrict__ rev, const int32_t *__restrict__ upflag,
                          const int32_t *__restrict__ upidx, int32_t n, int64_t nnz,
                          int32_t *__restrict__ up_ptr, int32_t *__restrict__ up_col,
                          int32_t *__restrict__ tslot,
    const int32_t *__restrict__ ctl) {
  if (ctl[kCtlStop]) return;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < nnz; e += stride) {
    if (upflag[e]) {
      up_col[upidx[e]] = col[e];
      tslot[e] = upidx[e];
    } else {
      tslot[e] = upidx[rev[e]];
    }
  }
  for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v <= n; v += stride) {
    if (v < n) up_ptr[v] = (row_ptr[v] < nnz) ? upidx[row_ptr[v]] : (int32_t)(nnz / 2);
    else up_ptr[v] = (int32_t)(nnz / 2);
  }
}

// ---------------------------------------------------------------------------
// Rank order inside every up(u) (rows are in id order after k_up_fill).
// ---------------------------------------------------------------------------
__global__ void k_up_keys(const int32_t *__restrict__ up_col, const int32_t *__restrict__ deg,
                          int64_t nup, int32_t *__restrict__ upk,
    const int32_t *__restrict__ ctl) {
  if (ctl[kCtlStop]) return;
  for (int64_t s = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; s < nup;
       s += (int64_t)gridDim.x * blockDim.x)
    upk[s] = deg[up_col[s]];
}

// For every up-arc u -> x: its rank position r inside up(u) (number of
// members ranked below x); newcol[up_ptr[u] + r] = x, newdeg[...] = k_x,
// perm[old slot] = new slot. Quadratic in |up(u)|, which is at most sqrt(2 * edges).
__global__ void k_up_sort(const int32_t *__restrict__ src, const int2 *__restrict__ adj2,
                          const int32_t *__restrict__ upflag, const int32_t *__restrict__ upidx,
                          int64_t nnz, const int32_t *__restrict__ up_ptr,
                          const int32_t *__restrict__ up_col, const int32_t *__restrict__ upk,
                          int32_t *__restrict__ newcol, int32_t *__restrict__ newdeg,
                          int32_t *__restrict__ perm,
    const int32_t *__restrict__ ctl) {
  if (ctl[kCtlStop]) return;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < nnz;
       e += (int64_t)gridDim.x * blockDim.x) {
    if (!upflag[e]) continue;
    const int32_t u = src[e];
    const int2 xk = adj2[e];
    const int32_t b0 = up_ptr[u], b1 = up_ptr[u + 1];
    int32_t r = 0;
    for (int32_t j = b0; j < b1; ++j) r += rank_less(up_col[j], upk[j], xk.x, xk.y) ? 1 : 0;
    newcol[b0 + r] = xk.x;
    newdeg[b0 + r] = xk.y;
    perm[upidx[e]] = b0 + r;
  }
}

// slots and up_col in the new order
__global__ void k_tslot_remap(int32_t *__restrict__ tslot, const int32_t *__restrict__ perm,
                              int64_t nnz, const int32_t *__restrict__ newcol,
                              int32_t *__restrict__ up_col, const int32_t *__restrict__ ctl) {
  if (ctl[kCtlStop]) return;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < nnz;
       e += (int64_t)gridDim.x * blockDim.x) {
    tslot[e] = perm[tslot[e]];
    if (e < nnz / 2) up_col[e] = newcol[e];
  }
}

// Segments: a down-arc w -> u (rank(u) < rank(w)) with a non-empty tail of
// up(u) above w, at a node w with up(w) non-empty (otherwise no triangle
// has w in the middle).
__global__ void k_dn_flag(const int32_t *__restrict__ src, const int32_t *__restrict__ col,
                          const int32_t *__restrict__ upflag, const int32_t *__restrict__ tslot,
                          const int32_t *__restrict__ up_ptr, int64_t nnz,
                          int32_t *__restrict__ dnflag,
    const int32_t *__restrict__ ctl) {
  if (ctl[kCtlStop]) return;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < nnz;
       e += (int64_t)gridDim.x * blockDim.x) {
    int32_t f = 0;
    if (!upflag[e]) {
      const int32_t w = src[e], u = col[e];
      const int32_t tail = up_ptr[u + 1] - tslot[e] - 1;
      f = (tail > 0 && up_ptr[w + 1] > up_ptr[w]) ? 1 : 0;
    }
    dnflag[e] = f;
  }
}

__global__ void k_dn_fill(const int32_t *__restrict__ row_ptr, const int32_t *__restrict__ src,
                          const int32_t *__restrict__ col,
                          const int32_t *__restrict__ deg, const int32_t *__restrict__ tslot,
                          const int32_t *__restrict__ up_ptr, const int32_t *__restrict__ dnflag,
                          const int32_t *__restrict__ dnidx, int32_t n, int64_t nnz,
                          int4 *__restrict__ dn, int32_t *__restrict__ dn_ptr,
    const int32_t *__restrict__ ctl) {
  if (ctl[kCtlStop]) return;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int32_t ndn = nnz > 0 ? dnidx[nnz - 1] + dnflag[nnz - 1] : 0;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < nnz; e += stride) {
    if (dnflag[e]) {
      const int32_t u = col[e], s = tslot[e];
      dn[dnidx[e]] = make_int4(s, up_ptr[u + 1] - s - 1, deg[u] + deg[src[e]], u);
    }
  }
  for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v <= n; v += stride)
    dn_ptr[v] = (v < n && row_ptr[v] < nnz) ? dnidx[row_ptr[v]] : ndn;
}

// Upper-end slots of long-list nodes with segments: their walk adds with
// atomics, so they are cleared before each pass.
__global__ void k_zero_flag(const int32_t *__restrict__ src, const int32_t *__restrict__ upflag,
                            const int32_t *__restrict__ tslot, const int32_t *__restrict__ up_ptr,
                            const int32_t *__restrict__ dn_ptr, int64_t nnz,
                            int32_t *__restrict__ zf,
    const int32_t *__restrict__ ctl) {
  if (ctl[kCtlStop]) return;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < nnz;
       e += (int64_t)gridDim.x * blockDim.x) {
    if (!upflag[e]) continue;
    const int32_t a = src[e];
    const int32_t nd = dn_ptr[a + 1] - dn_ptr[a], m = up_ptr[a + 1] - up_ptr[a];
    zf[tslot[e]] = (nd > 0 && m > kTriBin2) ? 1 : 0;
  }
}

// Per arc v -> a: the triangle record that holds the credits to v, in place
// of tslot. An edge to a lower-ranked a: a's upper-end slot of {a, v},
// written by a's walk when a has segments. An edge to a higher-ranked a: the
// lower-end slot nup + slot of {v, a}, written by a's walk when {v, a} is a
// segment of a. Otherwise -1: no walk writes the record and readers skip it.
__global__ void k_trec(const int32_t *__restrict__ col, const int32_t *__restrict__ rev,
                       const int32_t *__restrict__ upflag, const int32_t *__restrict__ dn_ptr,
                       const int32_t *__restrict__ dnflag, int64_t nnz, int64_t nup,
                       int32_t *__restrict__ tslot,
    const int32_t *__restrict__ ctl) {
  if (ctl[kCtlStop]) return;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < nnz;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int32_t s = tslot[e];
    int32_t r;
    if (upflag[e]) {
      r = dnflag[rev[e]] ? (int32_t)(nup + s) : -1;
    } else {
      const int32_t a = col[e];
      r = dn_ptr[a + 1] > dn_ptr[a] ? s : -1;
    }
    tslot[e] = r;
  }
}

__global__ void k_zero_fill(const int32_t *__restrict__ zf, const int32_t *__restrict__ zidx,
                            int64_t count, int32_t *__restrict__ list) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count;
       i += (int64_t)gridDim.x * blockDim.x)
    if (zf[i]) list[zidx[i]] = (int32_t)i;
}

// Per-node sums over a row of entries [ptr[v], ptr[v+1]): 8 lanes per node for
// rows of up to kRowShort, then a wavefront per longer row, which the
// wavefronts of the same launch find by a ballot over up to 64 nodes at a time
// (a wavefront per node left most lanes without an entry on sparse graphs:
// sums of BA n = 200k, m = 5 in 36 and 105 us). The nodes of a ballot are as far
// apart as there are wavefronts: hubs are often neighbours by id, and 64 of them
// on one wavefront took that graph's degree sums to 170 us and k_qa to 272 (now
// 20 each).
// sum(v, on, first, lanes) adds its lanes' entries, reduces and stores.
constexpr int32_t kRowShort = 128;

template <typename Sum>
__device__ __forceinline__ void for_rows(const int32_t *__restrict__ ptr, int32_t n, Sum sum) {
  const int64_t tid = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t nth = (int64_t)gridDim.x * blockDim.x;
  const int sub = threadIdx.x & 7;
  const int64_t rounds = (n + nth / 8 - 1) / (nth / 8);
  for (int64_t r = 0; r < rounds; ++r) {
    const int64_t v = r * (nth / 8) + tid / 8;
    const int32_t len = v < n ? ptr[v + 1] - ptr[v] : kRowShort + 1;
    sum((int32_t)(v < n ? v : 0), len <= kRowShort, sub, 8);
  }
  const int lane = threadIdx.x & 63;
  const int64_t nw = nth >> 6;
  for (int64_t v0 = tid >> 6; v0 < n; v0 += 64 * nw) {
    const int64_t v = v0 + lane * nw;
    unsigned long long m = __ballot(v < n && ptr[v + 1] - ptr[v] > kRowShort);
    while (m != 0ull) {
      const int j = __builtin_ctzll(m);
      m &= m - 1ull;
      sum((int32_t)(v0 + j * nw), true, lane, 64);
    }
  }
}
template <typename V> __device__ __forceinline__ V lanes_sum(V x, int lanes) {
  for (int off = lanes / 2; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
  return x;
}

// tail entries walked at w (sum of its segment lengths), and the sum of its
// neighbours' degrees
__global__ void k_dn_work(const int32_t *__restrict__ dn_ptr, const int4 *__restrict__ dn,
                          const int32_t *__restrict__ row_ptr, const int2 *__restrict__ adj2,
                          int32_t n, int64_t *__restrict__ work, int64_t *__restrict__ asum,
                          const int32_t *__restrict__ ctl) {
  if (ctl[kCtlStop]) return;
  for_rows(dn_ptr, n, [&](int32_t v, bool on, int first, int lanes) {
    int64_t acc = 0;
    if (on)
#pragma unroll 4
      for (int32_t i = dn_ptr[v] + first; i < dn_ptr[v + 1]; i += lanes) acc += dn[i].y;
    acc = lanes_sum(acc, lanes);
    if (on && first == 0) work[v] = acc;
  });
  for_rows(row_ptr, n, [&](int32_t v, bool on, int first, int lanes) {
    int64_t acc = 0;
    if (on)
#pragma unroll 4
      for (int32_t e = row_ptr[v] + first; e < row_ptr[v + 1]; e += lanes) acc += adj2[e].y;
    acc = lanes_sum(acc, lanes);
    if (on && first == 0) asum[v] = acc;
  });
}

// sum of squared neighbour degrees and sum of the neighbours'
// neighbour-degree sums (with k and asum, they give N and D of the node in
// closed form)
__global__ void k_qa(const int32_t *__restrict__ row_ptr, const int2 *__restrict__ adj2,
                     const int64_t *__restrict__ asum, int32_t n, longlong2 *__restrict__ qa,
                     NbrMoments *__restrict__ nbm, const int32_t *__restrict__ ctl) {
  if (ctl[kCtlStop]) return;
  for_rows(row_ptr, n, [&](int32_t v, bool on, int first, int lanes) {
    int64_t q = 0, a2 = 0;
    double c3 = 0.0, c4 = 0.0;
    if (on)
#pragma unroll 4
      for (int32_t e = row_ptr[v] + first; e < row_ptr[v + 1]; e += lanes) {
        const int2 ad = adj2[e];
        q += (int64_t)ad.y * ad.y;
        a2 += asum[ad.x];
        const double kb = (double)ad.y, kb2 = kb * kb;
        c3 += kb2 * kb;
        c4 += kb2 * kb2;
      }
    q = lanes_sum(q, lanes);
    a2 = lanes_sum(a2, lanes);
    c3 = lanes_sum(c3, lanes);
    c4 = lanes_sum(c4, lanes);
    if (on && first == 0) {
      qa[v] = make_longlong2(q, a2);
      nbm[v] = NbrMoments{asum[v], q, c3, c4};
    }
  });
}

// ---------------------------------------------------------------------------
// Exclusive scan of int32 (three passes: block totals, scan of the totals in
// one workgroup, block-local scans with offsets).
// ---------------------------------------------------------------------------
constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;
constexpr int kScanTile = kScanThreads * kScanItems;

int64_t scan_tmp_len(int64_t count) { return (count + kScanTile - 1) / kScanTile + 1; }
// the scan leaves the total after its block offsets
static int64_t scan_blocks(int64_t count) { return (count + kScanTile - 1) / kScanTile; }

__device__ int32_t block_exclusive_scan(int32_t x, int32_t *sh, int32_t &total) {
  // sh: kScanThreads / 64 ints
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int32_t incl = x;
  for (int off = 1; off < 64; off <<= 1) {
    int32_t y = __shfl_up(incl, off, 64);
    if (lane >= off) incl += y;
  }
  if (lane == 63) sh[w] = incl;
  __syncthreads();
  int32_t woff = 0, tot = 0;
  for (int i = 0; i < kScanThreads / 64; ++i) {
    if (i < w) woff += sh[i];
    tot += sh[i];
  }
  __syncthreads();
  total = tot;
  return woff + incl - x;
}

__global__ void k_scan_totals(const int32_t *__restrict__ in, int64_t count,
                              int32_t *__restrict__ totals) {
  __shared__ int32_t sh[kScanThreads / 64];
  const int64_t base = (int64_t)blockIdx.x * kScanTile;
  int32_t s = 0;
  for (int i = 0; i < kScanItems; ++i) {
    int64_t idx = base + (int64_t)threadIdx.x * kScanItems + i;
    if (idx < count) s += in[idx];
  }
  int32_t tot;
  block_exclusive_scan(s, sh, tot);
  if (threadIdx.x == 0) totals[blockIdx.x] = tot;
}

__global__ void k_scan_totals_single(int32_t *__restrict__ totals, int64_t nblocks) {
  __shared__ int32_t sh[kScanThreads / 64];
  int32_t carry = 0;
  for (int64_t base = 0; base < nblocks; base += kScanThreads) {
    int64_t idx = base + threadIdx.x;
    int32_t x = idx < nblocks ? totals[idx] : 0;
    int32_t tot;
    int32_t ex = block_exclusive_scan(x, sh, tot);
    if (idx < nblocks) totals[idx] = carry + ex;
    carry += tot;
  }
  if (threadIdx.x == 0) totals[nblocks] = carry;
}

__global__ void k_scan_apply(const int32_t *__restrict__ in, int64_t count,
                             const int32_t *__restrict__ totals, int32_t *__restrict__ out) {
  __shared__ int32_t sh[kScanThreads / 64];
  const int64_t base = (int64_t)blockIdx.x * kScanTile;
  int32_t v[kScanItems];
  int32_t s = 0;
  for (int i = 0; i < kScanItems; ++i) {
    int64_t idx = base + (int64_t)threadIdx.x * kScanItems + i;
    v[i] = idx < count ? in[idx] : 0;
    s += v[i];
  }
  int32_t tot;
  int32_t run = block_exclusive_scan(s, sh, tot) + totals[blockIdx.x];
  for (int i = 0; i < kScanItems; ++i) {
    int64_t idx = base + (int64_t)threadIdx.x * kScanItems + i;
    if (idx < count) out[idx] = run;
    run += v[i];
  }
}

// The scan of up to kScanOne values by one workgroup: a launch in place of three
// (a new graph of 8000 arcs runs three scans).
constexpr int64_t kScanOne = 16 * kScanTile;
__global__ __launch_bounds__(1024) void k_scan_one(const int32_t *__restrict__ in, int64_t count,
                                                   int32_t *__restrict__ out,
                                                   int32_t *__restrict__ total) {
  __shared__ int32_t sh[16];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int32_t carry = 0;
  for (int64_t base = 0; base < count; base += 1024 * kScanItems) {
    const int64_t i0 = base + (int64_t)threadIdx.x * kScanItems;
    int32_t v[kScanItems], s = 0;
    for (int i = 0; i < kScanItems; ++i) {
      v[i] = i0 + i < count ? in[i0 + i] : 0;
      s += v[i];
    }
    int32_t incl = s;
    for (int off = 1; off < 64; off <<= 1) {
      const int32_t y = __shfl_up(incl, off, 64);
      if (lane >= off) incl += y;
    }
    if (lane == 63) sh[w] = incl;
    __syncthreads();
    int32_t run = carry + incl - s;
    for (int i = 0; i < 16; ++i) {
      if (i < w) run += sh[i];
      carry += sh[i];
    }
    __syncthreads();
    for (int i = 0; i < kScanItems; ++i) {
      if (i0 + i < count) out[i0 + i] = run;
      run += v[i];
    }
  }
  if (threadIdx.x == 0) *total = carry;
}

hipError_t launch_exclusive_scan_i32(const int32_t *in, int32_t *out, int64_t count,
                                     int32_t *block_tmp, int64_t block_tmp_len,
                                     hipStream_t st) {
  if (count <= 0) return hipSuccess;
  const int64_t nb = (count + kScanTile - 1) / kScanTile;
  if (block_tmp_len < nb + 1) return hipErrorInvalidValue;
  if (count <= kScanOne) {
    hipLaunchKernelGGL(k_scan_one, dim3(1), dim3(1024), 0, st, in, count, out, block_tmp + nb);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_scan_totals, dim3((unsigned)nb), dim3(kScanThreads), 0, st, in, count,
                     block_tmp);
  hipLaunchKernelGGL(k_scan_totals_single, dim3(1), dim3(kScanThreads), 0, st, block_tmp, nb);
  hipLaunchKernelGGL(k_scan_apply, dim3((unsigned)nb), dim3(kScanThreads), 0, st, in, count,
                     block_tmp, out);
  return hipGetLastError();
}

static unsigned grid_for(int64_t work, int threads) {
  int64_t b = (work + threads - 1) / threads;
  if (b < 1) b = 1;
  if (b > 65535LL * 32) b = 65535LL * 32;
  return (unsigned)b;
}

// Scratch of launch_graph_prep, in ints:
//   [0, nnz)          up flags          [nnz, 2 nnz)   up indices, then cleared-slot indices
//   [2 nnz, 3 nnz)    rank keys | rank-sorted up_col, then segment indices, then cleared-slot flags
//   [3 nnz, 4 nnz)    segment flags     [4 nnz, 4 nnz + nup)   slot permutation
//   then the scan's block totals
int64_t graph_prep_tmp_len(int64_t nnz) {
  return 4 * nnz + nnz / 2 + scan_tmp_len(nnz);
}

// Everything but the zero-slot list, whose length (ctl[kCtlZero]) the caller
// reads back to size it; work[v] = tail entries walked at v. Asynchronous: the
// caller reads ctl when it has all run.
hipError_t launch_graph_prep(Graph &g, int32_t *tmp, int64_t *work, bool validate,
                             hipStream_t st) {
  const int T = 256;
  int32_t *ctl = g.d_counters;
  hipLaunchKernelGGL(k_degree, dim3(grid_for(g.n, T)), dim3(T), 0, st, g.row_ptr, g.n, g.deg, ctl);
  if (g.nnz > 0) {
    const int64_t nnz = g.nnz, nup = nnz / 2;
    int32_t *upflag = tmp, *upidx = tmp + nnz, *G = tmp + 2 * nnz, *dnflag = tmp + 3 * nnz,
            *perm = tmp + 4 * nnz, *scan_tmp = tmp + 4 * nnz + nup;
    const int64_t sl = scan_tmp_len(nnz);
    hipLaunchKernelGGL(k_arc_src, dim3(grid_for(nnz, T)), dim3(T), 0, st, g.row_ptr, g.col_idx,
                       g.n, nnz, g.src, ctl);
    hipLaunchKernelGGL(k_arc_rev, dim3(grid_for(nnz, T)), dim3(T), 0, st, g.row_ptr,
                       g.col_idx, g.src, g.deg, nnz, g.rev, g.rrev, g.adj2, upflag, ctl, validate);
    hipError_t e = launch_exclusive_scan_i32(upflag, upidx, nnz, scan_tmp, sl, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_gate, dim3(1), dim3(1), 0, st, ctl, scan_tmp + scan_blocks(nnz), nnz,
                       validate);
    hipLaunchKernelGGL(k_up_fill, dim3(grid_for(nnz, T)), dim3(T), 0, st, g.row_ptr,
                       g.col_idx, g.rev, upflag, upidx, g.n, nnz, g.up_ptr, g.up_col,
                       g.trec, ctl);
    // rank order inside each up(u)
    int32_t *upk = G, *newcol = G + nup;
    hipLaunchKernelGGL(k_up_keys, dim3(grid_for(nup, T)), dim3(T), 0, st, g.up_col, g.deg, nup,
                       upk, ctl);
    hipLaunchKernelGGL(k_up_sort, dim3(grid_for(nnz, T)), dim3(T), 0, st, g.src, g.adj2,
                       upflag, upidx, nnz, g.up_ptr, g.up_col, upk, newcol, g.up_deg, perm, ctl);
    hipLaunchKernelGGL(k_tslot_remap, dim3(grid_for(nnz, T)), dim3(T), 0, st, g.trec, perm,
                       nnz, newcol, g.up_col, ctl);
    // segments of the triangle pass
    int32_t *dnidx = G;
    hipLaunchKernelGGL(k_dn_flag, dim3(grid_for(nnz, T)), dim3(T), 0, st, g.src, g.col_idx,
                       upflag, g.trec, g.up_ptr, nnz, dnflag, ctl);
    e = launch_exclusive_scan_i32(dnflag, dnidx, nnz, scan_tmp, sl, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_dn_fill, dim3(grid_for(nnz, T)), dim3(T), 0, st, g.row_ptr, g.src,
                       g.col_idx, g.deg, g.trec, g.up_ptr, dnflag, dnidx, g.n, nnz, g.dn,
                       g.dn_ptr, ctl);
    hipLaunchKernelGGL(k_dn_work, dim3(grid_for((int64_t)g.n * 8, T)), dim3(T), 0, st,
                       g.dn_ptr, g.dn, g.row_ptr, g.adj2, g.n, work, g.asum, ctl);
    // slots cleared before each pass (long lists), then their scan
    int32_t *zf = G, *zidx = upidx;
    hipLaunchKernelGGL(k_zero_flag, dim3(grid_for(nnz, T)), dim3(T), 0, st, g.src, upflag,
                       g.trec, g.up_ptr, g.dn_ptr, nnz, zf, ctl);
    e = launch_exclusive_scan_i32(zf, zidx, nup, scan_tmp, sl, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_ctl_zero_total, dim3(1), dim3(1), 0, st, ctl,
                       scan_tmp + scan_blocks(nup));
    // tslot becomes the per-arc triangle record index
    hipLaunchKernelGGL(k_trec, dim3(grid_for(nnz, T)), dim3(T), 0, st, g.col_idx, g.rev, upflag,
                       g.dn_ptr, dnflag, nnz, nup, g.trec, ctl);
    hipLaunchKernelGGL(k_qa, dim3(grid_for((int64_t)g.n * 8, T)), dim3(T), 0, st, g.row_ptr,
                       g.adj2, g.asum, g.n, g.qa, g.nbm, ctl);
  } else {
    hipLaunchKernelGGL(k_up_fill, dim3(grid_for(g.n + 1, T)), dim3(T), 0, st, g.row_ptr,
                       g.col_idx, g.rev, tmp, tmp, g.n, (int64_t)0, g.up_ptr, g.up_col,
                       g.trec, ctl);
    hipLaunchKernelGGL(k_dn_fill, dim3(grid_for(g.n + 1, T)), dim3(T), 0, st, g.row_ptr, g.src,
                       g.col_idx, g.deg, g.trec, g.up_ptr, tmp, tmp, g.n, (int64_t)0, g.dn,
                       g.dn_ptr, ctl);
    (void)hipMemsetAsync(g.asum, 0, sizeof(int64_t) * (size_t)g.n, st);
    (void)hipMemsetAsync(g.qa, 0, sizeof(longlong2) * (size_t)g.n, st);
    (void)hipMemsetAsync(g.nbm, 0, sizeof(NbrMoments) * (size_t)g.n, st);
    (void)hipMemsetAsync(work, 0, sizeof(int64_t) * (size_t)g.n, st);
  }
  return hipGetLastError();
}

// Records of the triangle pass's lane bin, in id order (tri_lane_bin has the
// rule). Each workgroup owns a contiguous range of nodes; pass 0 counts the
// bin's nodes in it (more than one workgroup), pass 1 starts from the counts of
// those before and writes. Bound by the walk's loads on 48 workgroups (BA n = 200k,
// m = 5: 73 us each; the counts run while the host builds the other lists).
// Built by the host and uploaded, the 190k records took 0.1 ms more.
constexpr int kLaneBlocks = 48;  // counts fit the control record
constexpr int kLaneOneBlock = 4096;
template <int PASS>
__global__ __launch_bounds__(1024) void k_lane_recs(const int32_t *__restrict__ up_ptr,
                                                    const int32_t *__restrict__ dn_ptr,
                                                    const int4 *__restrict__ dn, int32_t n,
                                                    int32_t *__restrict__ counts,
                                                    int4 *__restrict__ recs) {
  __shared__ int32_t wsum[16];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int32_t per = (int32_t)(((int64_t)n + gridDim.x - 1) / gridDim.x);
  const int64_t lo = blockIdx.x * (int64_t)per, hi = lo + per < n ? lo + per : n;
  int32_t run = 0;
  if constexpr (PASS == 1)
    for (unsigned i = 0; i < blockIdx.x; ++i) run += counts[i];
  for (int64_t v0 = lo; v0 < hi; v0 += 1024) {
    const int64_t v = v0 + tid;
    int32_t u0 = 0, d0 = 0, up = 0, nd = 0, walk = 0;
    if (v < hi) {
      u0 = up_ptr[v];
      d0 = dn_ptr[v];
      up = up_ptr[v + 1] - u0;
      nd = dn_ptr[v + 1] - d0;
      if (nd <= kTriLaneSegs && up <= kTriLaneM)
#pragma unroll 4
        for (int32_t i = 0; i < nd; ++i) walk += dn[d0 + i].y;
    }
    const bool in = v < hi && tri_lane_bin(up, nd, walk);
    const unsigned long long m = __ballot(in);
    if (lane == 0) wsum[wv] = __popcll(m);
    __syncthreads();
    int32_t pre = 0, tot = 0;
    for (int i = 0; i < 16; ++i) {
      if (i < wv) pre += wsum[i];
      tot += wsum[i];
    }
    if (PASS == 1 && in)
      recs[run + pre + __popcll(m & ((1ull << lane) - 1))] =
          make_int4((int32_t)v, u0, d0, up | (nd << 8) | (walk << 16));
    run += tot;
    __syncthreads();
  }
  if (PASS == 0 && tid == 0) counts[blockIdx.x] = run;
}

static_assert(kCtlWords + kLaneBlocks <= 64, "the record and the counts share d_counters");
static int lane_blocks(const Graph &g) { return g.n <= kLaneOneBlock ? 1 : kLaneBlocks; }

hipError_t launch_lane_counts(Graph &g, hipStream_t st) {
  if (g.nnz <= 0 || lane_blocks(g) == 1) return hipSuccess;
  hipLaunchKernelGGL(k_lane_recs<0>, dim3(lane_blocks(g)), dim3(1024), 0, st, g.up_ptr, g.dn_ptr,
                     g.dn, g.n, g.d_counters + kCtlWords, nullptr);
  return hipGetLastError();
}

hipError_t launch_lane_recs(Graph &g, hipStream_t st) {
  if (g.n_tri_lane <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_lane_recs<1>, dim3(lane_blocks(g)), dim3(1024), 0, st, g.up_ptr, g.dn_ptr,
                     g.dn, g.n, g.d_counters + kCtlWords, g.tri_recL);
  return hipGetLastError();
}

hipError_t launch_zero_list(Graph &g, const int32_t *tmp, hipStream_t st) {
  const int64_t nnz = g.nnz, nup = nnz / 2;
  if (nup <= 0 || g.n_tri_zero <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_zero_fill, dim3(grid_for(nup, 256)), dim3(256), 0, st, tmp + 2 * nnz,
                     tmp + nnz, nup, g.tri_zero);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// degree-ordered rows of the big centres, for the super-tile pair loop: with
// the neighbours in ascending degree, the degrees inside a 64 x 64 tile are
// close, so most tiles can read their scores from a small table
// ---------------------------------------------------------------------------
__global__ void k_big_keys(const int32_t *__restrict__ row_ptr, const int2 *__restrict__ adj2,
                           const int32_t *__restrict__ big, int32_t nbig,
                           int32_t *__restrict__ kin, int32_t *__restrict__ vin,
                           int32_t *__restrict__ seg_beg, int32_t *__restrict__ seg_end) {
  for (int32_t i = blockIdx.x; i < nbig; i += gridDim.x) {
    const int32_t v = big[i], b = row_ptr[v], e = row_ptr[v + 1];
    if (threadIdx.x == 0) {
      seg_beg[i] = b;
      seg_end[i] = e;
    }
    for (int32_t x = b + threadIdx.x; x < e; x += blockDim.x) {
      kin[x] = adj2[x].y;
      vin[x] = x - b;
    }
  }
}

__global__ void k_big_pack(const int32_t *__restrict__ row_ptr, const int32_t *__restrict__ big,
                           int32_t nbig, const int32_t *__restrict__ kout,
                           const int32_t *__restrict__ vout, int2 *__restrict__ adjs) {
  for (int32_t i = blockIdx.x; i < nbig; i += gridDim.x) {
    const int32_t v = big[i], b = row_ptr[v], e = row_ptr[v + 1];
    for (int32_t x = b + threadIdx.x; x < e; x += blockDim.x) adjs[x] = make_int2(vout[x], kout[x]);
  }
}

// a big centre stores the per-arc sums of its row by sorted position: the
// reverse of the arc at sorted position x of its row finds its sum at x
__global__ void k_rrev_big(const int32_t *__restrict__ row_ptr, const int32_t *__restrict__ big,
                           int32_t nbig, const int32_t *__restrict__ rev,
                           const int2 *__restrict__ adjs, int32_t *__restrict__ rrev) {
  for (int32_t i = blockIdx.x; i < nbig; i += gridDim.x) {
    const int32_t v = big[i], b = row_ptr[v], e = row_ptr[v + 1];
    for (int32_t x = b + threadIdx.x; x < e; x += blockDim.x) rrev[rev[b + adjs[x].x]] = x;
  }
}

hipError_t launch_big_sort(Graph &g, const int32_t *big, int32_t nbig, int32_t *scratch,
                           int32_t *seg, void *temp, size_t &temp_bytes, hipStream_t st) {
  const int64_t nnz = g.nnz;
  int32_t *kin = scratch, *kout = scratch + nnz, *vin = scratch + 2 * nnz,
          *vout = scratch + 3 * nnz;
  int end_bit = 1;
  while (end_bit < 31 && (int64_t(1) << end_bit) <= (int64_t)g.info.max_degree) ++end_bit;
  if (temp == nullptr) {
    return hipcub::DeviceSegmentedRadixSort::SortPairs(
        nullptr, temp_bytes, kin, kout, vin, vout, (int)nnz, (int)nbig, seg, seg + nbig, 0,
        end_bit, st);
  }
  const unsigned grid = (unsigned)std::min<int64_t>(std::max<int32_t>(nbig, 1), 65536);
  hipLaunchKernelGGL(k_big_keys, dim3(grid), dim3(256), 0, st, g.row_ptr, g.adj2, big, nbig, kin,
                     vin, seg, seg + nbig);
  hipError_t e = hipcub::DeviceSegmentedRadixSort::SortPairs(
      temp, temp_bytes, kin, kout, vin, vout, (int)nnz, (int)nbig, seg, seg + nbig, 0, end_bit,
      st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_big_pack, dim3(grid), dim3(256), 0, st, g.row_ptr, big, nbig, kout, vout,
                     g.adjs);
  hipLaunchKernelGGL(k_rrev_big, dim3(grid), dim3(256), 0, st, g.row_ptr, big, nbig, g.rev,
                     g.adjs, g.rrev);
  return hipGetLastError();
}

}  // namespace efi
