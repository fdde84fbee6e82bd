// Top-k spreaders: the k nodes of largest Expected Force ("identification of
// key nodes", the paper's title and Sec. 1). Order: EF descending, ties by
// node id ascending.
//
// EF values are non-negative, so their IEEE bit patterns order like the values
// as unsigned integers; a value that is not positive (or NaN) takes key 0.
// Up to kTkDirect values are ranked against each other in one launch. Above
// that, three phases, none with a device-wide sort:
//
//   1. Radix select of the k-th largest key, six digits of 11, 11, 11, 10, 10
//      and 10 bits below the sign bit (the first is the exponent). Each pass
//      histograms one digit of the keys whose known high bits match, in LDS,
//      and adds the bins it met to the pass's histogram in device memory. The
//      next launch's workgroups each pick the digit of the k-th key from that
//      histogram before they start (8 KB, one prefix sum), so a pass is one
//      launch, and the passes need no host round trip.
//   2. Order-preserving compaction of the winners: every key above the k-th
//      key's bucket, and the first `need` keys inside it in id order (ties at
//      the k-th value go to the smallest ids). Counts per wavefront, then a
//      launch that sums the counts before each wavefront and writes with
//      ballot ranks, which keeps each class in id order.
//   3. Sort of the k winners by key descending, ties by id: tiles of kTkSort
//      winners are sorted by counting, for every winner, those before it (one
//      tile: straight to the outputs); up to kTkMerge winners, a winner's
//      place is its rank in its tile plus binary searches of the other tiles;
//      above that a stable LSD radix sort (8-bit digits, ballot-ranked stable
//      scatter), which keeps the id order of equal keys that the compaction
//      produced.
//
// Bound by the passes over the n values (8 bytes each; the ones after the
// first come from the last-level cache) and by launch latency below about a
// million values: the 1000 best of 4 million take 120 us a call with the
// copy to the host, against 1410 us when one thread per bin summed 1024
// histograms of 8-bit digits in each of eight passes.
#include <mutex>

#include "ef_internal.h"

namespace efi {

namespace {

constexpr int kTkThreads = 256;    // workgroup of the radix sort passes (4 wavefronts)
constexpr int kTkTile = 4096;      // records per workgroup in a radix sort pass
constexpr int kTkSelBlocks = 256;  // most workgroups of a selection pass, 16 wavefronts each
constexpr int kTkSelThreads = 1024;
constexpr int kTkSelWaves = kTkSelThreads / 64;
constexpr int kTkPasses = 6;
constexpr int kTkBins = 2048;
// up to this many values, ranking all of them costs less than the selection's
// ten launches (a call on 8192 values: 22 us against 31; on 16384: 43 against 32)
constexpr int32_t kTkDirect = 8192;
constexpr int32_t kTkSort = 4096;  // winners per counting-sorted tile (32 KB of keys in LDS)
// up to this many winners, merging sorted tiles by binary searches (work: k
// times the tiles) costs less than the radix sort's 24 launches (a call for
// 16384 winners: 52 us against 230; 131072: 161 against 310; 262144: 299
// against 427, and four times the searches at twice the winners)
constexpr int32_t kTkMerge = 262144;

__host__ __device__ constexpr int tk_shift(int pass) {
  constexpr int s[kTkPasses] = {52, 41, 30, 20, 10, 0};
  return s[pass];
}
__host__ __device__ constexpr int tk_bits(int pass) { return pass < 3 ? 11 : 10; }

// selection state after a pass; record 0 is the state before the first
struct TkState {
  unsigned long long prefix;  // digits of the k-th key fixed so far
  unsigned long long mask;    // their bit positions
  long long need;             // keys still to take among those matching prefix
  int32_t done;               // exactly `need` keys match: later passes skip
  int32_t skip;               // sort pass: every key has the same digit
  int32_t pad[8];
};
static_assert(sizeof(TkState) == 64, "state record is one 64-byte line");

__device__ __forceinline__ unsigned long long tk_key(double v) {
  return v > 0.0 ? (unsigned long long)__double_as_longlong(v) : 0ull;
}
__device__ __forceinline__ double tk_value(unsigned long long key) {
  return __longlong_as_double((long long)key);
}

// number of set bits of m in the lanes below this one
__device__ __forceinline__ uint32_t lanes_below(unsigned long long m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// clears the passes' histograms and sets the state before the first pass
__global__ __launch_bounds__(1024) void k_tk_init(TkState *st, uint32_t *__restrict__ hist,
                                                  int32_t k) {
  const int i = blockIdx.x * 1024 + threadIdx.x;
  if (i < kTkPasses * kTkBins) hist[i] = 0u;
  if (i == 0) {
    TkState s{};
    s.need = k;
    st[0] = s;
  }
}

// State after pass `pass` from the state before it and its histogram: the
// digit of the k-th key, counting bins from the top. Every thread of a
// workgroup of kTkSelThreads calls it and gets the state.
__device__ TkState tk_pick(const TkState *st, const uint32_t *__restrict__ hist, int pass) {
  __shared__ TkState sh;
  __shared__ uint32_t wsum[kTkSelWaves];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  TkState s = st[pass];
  if (s.done) return s;  // uniform: read from memory
  // thread t: bins top = kTkBins - 1 - 2t and top - 1, prefix sums from the top
  const int top = kTkBins - 1 - 2 * t;
  const uint32_t c0 = hist[pass * kTkBins + top], c1 = hist[pass * kTkBins + top - 1];
  uint32_t incl = c0 + c1;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(incl, o, 64);
    if (lane >= o) incl += y;
  }
  if (lane == 63) wsum[w] = incl;
  __syncthreads();
  uint32_t before = 0;
  for (int j = 0; j < w; ++j) before += wsum[j];
  const long long a0 = (long long)before + incl - c0 - c1;  // keys above bin `top`
  const long long a1 = a0 + c0, a2 = a1 + c1;
  // exactly one bin holds the need-th key from the top
  const bool in0 = a0 < s.need && s.need <= a1, in1 = a1 < s.need && s.need <= a2;
  if (in0 || in1) {
    const int j = in0 ? top : top - 1;
    s.prefix |= (unsigned long long)j << tk_shift(pass);
    s.mask |= ((1ull << tk_bits(pass)) - 1ull) << tk_shift(pass);
    s.need -= in0 ? a0 : a1;
    s.done = (long long)(in0 ? c0 : c1) == s.need ? 1 : 0;
    sh = s;
  }
  __syncthreads();
  return sh;
}

// Phase 1, one digit: state of this pass, then the digit's histogram over the
// keys that match its prefix. `chunk` values per workgroup.
__global__ __launch_bounds__(kTkSelThreads) void k_tk_sel(const double *__restrict__ vals,
                                                          int32_t n, int64_t chunk, int pass,
                                                          TkState *st, uint32_t *hist) {
  __shared__ uint32_t h[kTkBins];
  TkState s = st[0];
  if (pass > 0) {
    s = tk_pick(st, hist, pass - 1);
    if (blockIdx.x == 0 && threadIdx.x == 0) st[pass] = s;
  }
  if (s.done) return;
  const int t = threadIdx.x;
  h[t] = 0u;
  h[t + 1024] = 0u;
  __syncthreads();
  const int shift = tk_shift(pass);
  const uint32_t bins = (1u << tk_bits(pass)) - 1u;
  const int64_t lo = (int64_t)blockIdx.x * chunk;
  const int64_t hi = min((int64_t)n, lo + chunk);
  // four loads in flight per thread
  for (int64_t i0 = lo + t; i0 < hi; i0 += 4 * kTkSelThreads) {
    double v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t i = i0 + q * kTkSelThreads;
      v[q] = vals[i < hi ? i : i0];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const unsigned long long key = tk_key(v[q]);
      if (i0 + q * kTkSelThreads < hi && (key & s.mask) == s.prefix)
        atomicAdd(&h[(uint32_t)(key >> shift) & bins], 1u);
    }
  }
  __syncthreads();
  uint32_t *out = hist + pass * kTkBins;
  for (int j = t; j < kTkBins; j += kTkSelThreads)
    if (h[j]) atomicAdd(&out[j], h[j]);
}

// The wavefront's share of the values in phase 2: contiguous, in id order.
__device__ __forceinline__ void tk_share(int32_t n, int64_t wchunk, int64_t &lo, int64_t &hi) {
  lo = ((int64_t)blockIdx.x * kTkSelWaves + (threadIdx.x >> 6)) * wchunk;
  hi = min((int64_t)n, lo + wchunk);
}

// Phase 2: per wavefront, keys above the bucket (gt) and inside it (eq).
__global__ __launch_bounds__(kTkSelThreads) void k_tk_count(const double *__restrict__ vals,
                                                            int32_t n, int64_t wchunk,
                                                            TkState *st, const uint32_t *hist,
                                                            int32_t *__restrict__ cnt_gt,
                                                            int32_t *__restrict__ cnt_eq) {
  const TkState s = tk_pick(st, hist, kTkPasses - 1);
  if (blockIdx.x == 0 && threadIdx.x == 0) st[kTkPasses] = s;
  const int lane = threadIdx.x & 63;
  int32_t ng = 0, ne = 0;
  int64_t lo, hi;
  tk_share(n, wchunk, lo, hi);
  for (int64_t i0 = lo + lane; i0 < hi; i0 += 256) {
    double v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = vals[i0 + 64 * q < hi ? i0 + 64 * q : i0];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const unsigned long long m = tk_key(v[q]) & s.mask;
      const bool in = i0 + 64 * q < hi;
      ng += in && m > s.prefix;
      ne += in && m == s.prefix;
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
    ng += __shfl_xor(ng, off, 64);
    ne += __shfl_xor(ne, off, 64);
  }
  if (lane == 0) {
    const int w = blockIdx.x * kTkSelWaves + (threadIdx.x >> 6);
    cnt_gt[w] = ng;
    cnt_eq[w] = ne;
  }
}

// Phase 2: write the winners, each class in id order: gt keys at their rank,
// eq keys after all gt keys while their rank among eq keys is below `need`.
// Each workgroup sums the counts of all wavefronts before its own (at most
// 4096) first; a wavefront without a winner skips its values.
__global__ __launch_bounds__(kTkSelThreads) void k_tk_write(
    const double *__restrict__ vals, int32_t n, int64_t wchunk, const TkState *__restrict__ st,
    const int32_t *__restrict__ cnt_gt, const int32_t *__restrict__ cnt_eq,
    unsigned long long *__restrict__ okey, int32_t *__restrict__ oid) {
  __shared__ int32_t sg[kTkSelWaves], se[kTkSelWaves], sa[kTkSelWaves];
  __shared__ int32_t wg[kTkSelWaves], we[kTkSelWaves];
  const TkState s = st[kTkPasses];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int first = blockIdx.x * kTkSelWaves, nw = (int)gridDim.x * kTkSelWaves;
  int32_t bg = 0, be = 0, all = 0;
  for (int i = t; i < nw; i += kTkSelThreads) {
    const int32_t g = cnt_gt[i];
    all += g;
    if (i < first) {
      bg += g;
      be += cnt_eq[i];
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
    bg += __shfl_xor(bg, off, 64);
    be += __shfl_xor(be, off, 64);
    all += __shfl_xor(all, off, 64);
  }
  if (lane == 0) {
    sg[w] = bg;
    se[w] = be;
    sa[w] = all;
    wg[w] = cnt_gt[first + w];
    we[w] = cnt_eq[first + w];
  }
  __syncthreads();
  int32_t run_g = 0, run_e = 0, gt_total = 0;
  for (int j = 0; j < kTkSelWaves; ++j) {
    run_g += sg[j] + (j < w ? wg[j] : 0);
    run_e += se[j] + (j < w ? we[j] : 0);
    gt_total += sa[j];
  }
  if (wg[w] == 0 && (we[w] == 0 || run_e >= s.need)) return;
  int64_t lo, hi;
  tk_share(n, wchunk, lo, hi);
  for (int64_t base = lo; base < hi; base += 256) {
    double v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t i = base + 64 * q + lane;
      v[q] = vals[i < hi ? i : base];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t i = base + 64 * q + lane;
      const unsigned long long key = tk_key(v[q]), m = key & s.mask;
      const bool gt = i < hi && m > s.prefix, eq = i < hi && m == s.prefix;
      const unsigned long long mg = __ballot(gt), me = __ballot(eq);
      if (gt) {
        const int32_t r = run_g + (int32_t)lanes_below(mg);
        okey[r] = key;
        oid[r] = (int32_t)i;
      }
      if (eq) {
        const int32_t r = run_e + (int32_t)lanes_below(me);
        if (r < s.need) {
          okey[gt_total + r] = key;
          oid[gt_total + r] = (int32_t)i;
        }
      }
      run_g += __popcll(mg);
      run_e += __popcll(me);
    }
  }
}

// Phase 3: ranks by counting inside tiles of at most `tile` records (a record
// is before another when its key is larger, or equal at a smaller position:
// the compaction keeps equal keys in id order). A workgroup ranks 64 records
// of one tile, one per lane, its 16 wavefronts counting a sixteenth of the
// tile's keys each from LDS (one broadcast read of two keys per two
// comparisons). DIRECT: the records are the values themselves, position = id,
// and only ranks below k are written; else (okey, oid). `final`: nodes and
// ef_out get the tile's records, otherwise skey and sid do, tile by tile.
template <bool DIRECT, int MAXT>
__global__ __launch_bounds__(kTkSelThreads) void k_tk_rank(
    const double *__restrict__ vals, const unsigned long long *__restrict__ okey,
    const int32_t *__restrict__ oid, int32_t m, int32_t k, bool final, int32_t *__restrict__ nodes,
    double *__restrict__ ef_out, unsigned long long *__restrict__ skey,
    int32_t *__restrict__ sid) {
  __shared__ __align__(16) unsigned long long keys[MAXT];
  __shared__ int32_t part[kTkSelWaves][64];
  constexpr int32_t kGroups = MAXT / 64;  // workgroups per tile
  const int32_t tile = (int32_t)blockIdx.x / kGroups;
  const int32_t t0 = tile * MAXT, cnt = min(MAXT, m - t0);
  const int32_t i0 = ((int32_t)blockIdx.x - tile * kGroups) * 64;
  if (i0 >= cnt) return;  // uniform
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int32_t padded = (cnt + 31) & ~31;  // 16 wavefronts, two keys a step
  for (int32_t j = t; j < padded; j += kTkSelThreads) {
    unsigned long long key = 0ull;  // past the end: before no record
    if (j < cnt) {
      if constexpr (DIRECT) key = tk_key(vals[t0 + j]);
      else key = okey[t0 + j];
    }
    keys[j] = key;
  }
  __syncthreads();
  const int32_t i = i0 + lane;
  const unsigned long long ki = keys[i < cnt ? i : 0];
  const int32_t per = padded / kTkSelWaves, j0 = w * per, j1 = j0 + per;
  int32_t c = 0;
  // keys before this record's position count when equal, later ones do not:
  // positions below i0 are before every record here, positions from i0 + 64
  // on after; between them compare positions too
  int32_t j = j0;
  const int32_t ja = min(max(i0, j0), j1), jb = min(max(i0 + 64, j0), j1);
  for (; j < ja; j += 2) {
    const ulonglong2 kk = *reinterpret_cast<const ulonglong2 *>(&keys[j]);
    c += (kk.x >= ki) + (kk.y >= ki);
  }
  for (; j < jb; j += 2) {
    const ulonglong2 kk = *reinterpret_cast<const ulonglong2 *>(&keys[j]);
    c += (kk.x > ki || (kk.x == ki && j < i)) + (kk.y > ki || (kk.y == ki && j + 1 < i));
  }
  for (; j < j1; j += 2) {
    const ulonglong2 kk = *reinterpret_cast<const ulonglong2 *>(&keys[j]);
    c += (kk.x > ki) + (kk.y > ki);
  }
  part[w][lane] = c;
  __syncthreads();
  if (w == 0 && i < cnt) {
    int32_t r = 0;
    for (int q = 0; q < kTkSelWaves; ++q) r += part[q][lane];
    int32_t id;
    if constexpr (DIRECT) id = i;
    else id = oid[t0 + i];
    if (final) {
      if (!DIRECT || r < k) {
        nodes[r] = id;
        if (ef_out) ef_out[r] = tk_value(ki);
      }
    } else {
      skey[t0 + r] = ki;
      sid[t0 + r] = id;
    }
  }
}

// Phase 3, kTkSort < k <= kTkMerge: the place of a record of a sorted tile is
// its rank there plus, for every other tile, the number of records before it
// (equal keys of earlier tiles are before it, of later tiles after it).
__global__ __launch_bounds__(256) void k_tk_merge(const unsigned long long *__restrict__ skey,
                                                  const int32_t *__restrict__ sid, int32_t k,
                                                  int32_t *__restrict__ nodes,
                                                  double *__restrict__ ef_out) {
  const int32_t i = (int32_t)(blockIdx.x * 256 + threadIdx.x);
  if (i >= k) return;
  const unsigned long long ki = skey[i];
  const int32_t mine = i / kTkSort, tiles = (k + kTkSort - 1) / kTkSort;
  int32_t r = i - mine * kTkSort;
  for (int32_t q = 0; q < tiles; ++q) {
    if (q == mine) continue;
    const int32_t b = q * kTkSort;
    int32_t lo = 0, hi = min(kTkSort, k - b);  // first record of the tile not before i
    while (lo < hi) {
      const int32_t mid = (lo + hi) >> 1;
      const unsigned long long x = skey[b + mid];
      if (x > ki || (x == ki && q < mine)) lo = mid + 1; else hi = mid;
    }
    r += lo;
  }
  nodes[r] = sid[i];
  if (ef_out) ef_out[r] = tk_value(ki);
}

// Phase 3, k > kTkMerge: one stable LSD pass on the digit 255 - byte (keys
// descending). Histogram per tile, stored digit-major for the scan.
__global__ __launch_bounds__(kTkThreads) void k_tk_rhist(const unsigned long long *__restrict__ key,
                                                         int32_t k, int shift, int32_t nblk,
                                                         uint32_t *__restrict__ hist) {
  __shared__ uint32_t h[256];
  h[threadIdx.x] = 0;
  __syncthreads();
  const int64_t lo = (int64_t)blockIdx.x * kTkTile;
  const int64_t hi = min((int64_t)k, lo + kTkTile);
  for (int64_t i = lo + threadIdx.x; i < hi; i += kTkThreads)
    atomicAdd(&h[255u - ((uint32_t)(key[i] >> shift) & 255u)], 1u);
  __syncthreads();
  hist[(size_t)threadIdx.x * nblk + blockIdx.x] = h[threadIdx.x];
}

// Exclusive scan of the digit-major histogram (256 rows of nblk tiles), in
// place: four threads per digit row. A digit holding all k keys sets skip.
__global__ __launch_bounds__(1024) void k_tk_rscan(uint32_t *hist, int32_t nblk, int32_t k,
                                                   TkState *st) {
  __shared__ uint32_t part[1024];
  __shared__ uint32_t rowsum[256];
  const int t = threadIdx.x, d = t >> 2, q = t & 3;
  const int32_t per = (nblk + 3) / 4;
  const int32_t b0 = min(nblk, q * per), b1 = min(nblk, b0 + per);
  uint32_t *row = hist + (size_t)d * nblk;
  uint32_t s = 0;
  for (int32_t b = b0; b < b1; ++b) s += row[b];
  part[t] = s;
  __syncthreads();
  if (t < 256) rowsum[t] = part[4 * t] + part[4 * t + 1] + part[4 * t + 2] + part[4 * t + 3];
  __syncthreads();
  if (t == 0) {
    uint32_t acc = 0;
    int32_t same = 0;
    for (int j = 0; j < 256; ++j) {
      same |= rowsum[j] == (uint32_t)k;
      const uint32_t v = rowsum[j];
      rowsum[j] = acc;
      acc += v;
    }
    st->skip = same;
  }
  __syncthreads();
  uint32_t acc = rowsum[d];
  for (int j = 0; j < q; ++j) acc += part[4 * d + j];
  for (int32_t b = b0; b < b1; ++b) {
    const uint32_t v = row[b];
    row[b] = acc;
    acc += v;
  }
}

// Stable scatter of one tile: ranks among equal digits from wavefront
// ballots, in tile order (lanes, then wavefronts, then rounds).
__global__ __launch_bounds__(kTkThreads) void k_tk_scatter(
    const unsigned long long *__restrict__ kin, const int32_t *__restrict__ iin,
    unsigned long long *__restrict__ kout, int32_t *__restrict__ iout, int32_t k, int shift,
    const uint32_t *__restrict__ off, int32_t nblk, const TkState *__restrict__ st) {
  const int64_t lo = (int64_t)blockIdx.x * kTkTile;
  const int64_t hi = min((int64_t)k, lo + kTkTile);
  if (st->skip) {
    for (int64_t i = lo + threadIdx.x; i < hi; i += kTkThreads) {
      kout[i] = kin[i];
      iout[i] = iin[i];
    }
    return;
  }
  __shared__ uint32_t base[256];
  __shared__ uint32_t wc[4][256];
  const int t = threadIdx.x, w = t >> 6;
  base[t] = off[(size_t)t * nblk + blockIdx.x];
  wc[0][t] = wc[1][t] = wc[2][t] = wc[3][t] = 0;
  __syncthreads();
  for (int64_t b0 = lo; b0 < hi; b0 += kTkThreads) {
    const int64_t i = b0 + t;
    const bool valid = i < hi;
    unsigned long long key = 0;
    int32_t id = 0;
    uint32_t d = 0;
    if (valid) {
      key = kin[i];
      id = iin[i];
      d = 255u - ((uint32_t)(key >> shift) & 255u);
    }
    unsigned long long peers = __ballot(valid);
    for (int bit = 0; bit < 8; ++bit) {
      const bool on = (d >> bit) & 1u;
      const unsigned long long bb = __ballot(on);
      peers &= on ? bb : ~bb;
    }
    const uint32_t r = lanes_below(peers);
    if (valid && r == 0) wc[w][d] = (uint32_t)__popcll(peers);
    __syncthreads();
    if (valid) {
      uint32_t pos = base[d] + r;
      for (int j = 0; j < w; ++j) pos += wc[j][d];
      kout[pos] = key;
      iout[pos] = id;
    }
    __syncthreads();
    base[t] += wc[0][t] + wc[1][t] + wc[2][t] + wc[3][t];
    wc[0][t] = wc[1][t] = wc[2][t] = wc[3][t] = 0;
    __syncthreads();
  }
}

__global__ void k_tk_emit(const unsigned long long *__restrict__ key,
                          const int32_t *__restrict__ id, int32_t k, int32_t *__restrict__ nodes,
                          double *__restrict__ ef_out) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < k;
       i += (int64_t)gridDim.x * blockDim.x) {
    nodes[i] = id[i];
    if (ef_out) ef_out[i] = tk_value(key[i]);
  }
}

struct TkLayout {
  int32_t nblk = 1, ntile = 0, nsort = 0;
  int64_t chunk = 1;  // values per selection workgroup, a multiple of 16 * 64
  size_t state = 0, hist = 0, cgt = 0, ceq = 0, k0 = 0, k1 = 0, i0 = 0, i1 = 0, rhist = 0;
  size_t bytes = 0;
};

TkLayout tk_layout(int32_t n, int32_t k) {
  TkLayout L;
  const int64_t nn = std::max<int32_t>(n, 1);
  const int64_t nb = std::min<int64_t>(kTkSelBlocks, (nn + 4095) / 4096);
  L.chunk = ((nn + nb - 1) / nb + kTkSelThreads - 1) / kTkSelThreads * kTkSelThreads;
  L.nblk = (int32_t)((nn + L.chunk - 1) / L.chunk);
  L.ntile = (int32_t)(((int64_t)k + kTkSort - 1) / kTkSort);
  L.nsort = k > kTkMerge ? (int32_t)(((int64_t)k + kTkTile - 1) / kTkTile) : 0;
  size_t p = 0;
  auto take = [&](size_t b) {
    const size_t r = p;
    p += (b + 255) & ~(size_t)255;
    return r;
  };
  const size_t kk = (size_t)std::max<int32_t>(k, 1);
  L.state = take(sizeof(TkState) * (kTkPasses + 1));
  L.hist = take(sizeof(uint32_t) * kTkPasses * kTkBins);
  L.cgt = take(sizeof(int32_t) * (size_t)L.nblk * kTkSelWaves);
  L.ceq = take(sizeof(int32_t) * (size_t)L.nblk * kTkSelWaves);
  L.k0 = take(sizeof(unsigned long long) * kk);
  L.i0 = take(sizeof(int32_t) * kk);
  if (k > kTkSort) {
    L.k1 = take(sizeof(unsigned long long) * kk);
    L.i1 = take(sizeof(int32_t) * kk);
  }
  if (L.nsort > 0) L.rhist = take(sizeof(uint32_t) * 256 * (size_t)L.nsort);
  L.bytes = p;
  return L;
}

// whether [a, a + na) and [b, b + nb) share a byte
bool tk_overlap(const void *a, size_t na, const void *b, size_t nb) {
  const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
  return x < y + nb && y < x + na;
}

}  // namespace

size_t topk_scratch_bytes(int32_t n, int32_t k) { return tk_layout(n, k).bytes; }

// the one-launch form writes outputs while other workgroups still read the
// values: not for outputs placed over them
bool topk_direct(const double *vals, int32_t n, int32_t k, const int32_t *nodes,
                 const double *ef_out) {
  return n <= kTkDirect && !tk_overlap(vals, sizeof(double) * n, nodes, sizeof(int32_t) * k) &&
         !(ef_out && tk_overlap(vals, sizeof(double) * n, ef_out, sizeof(double) * k));
}

hipError_t launch_topk(const double *vals, int32_t n, int32_t k, void *scratch,
                       size_t scratch_bytes, int32_t *nodes, double *ef_out, hipStream_t st) {
  if (n <= 0 || k <= 0) return hipSuccess;
  if (k > n) return hipErrorInvalidValue;
  if (topk_direct(vals, n, k, nodes, ef_out)) {
    hipLaunchKernelGGL((k_tk_rank<true, kTkDirect>), dim3((n + 63) / 64), dim3(kTkSelThreads), 0,
                       st, vals, nullptr, nullptr, n, k, true, nodes, ef_out, nullptr, nullptr);
    return hipGetLastError();
  }
  const TkLayout L = tk_layout(n, k);
  if (L.bytes > scratch_bytes) return hipErrorInvalidValue;
  char *p = (char *)scratch;
  auto *state = (TkState *)(p + L.state);
  auto *hist = (uint32_t *)(p + L.hist);
  auto *cgt = (int32_t *)(p + L.cgt);
  auto *ceq = (int32_t *)(p + L.ceq);
  auto *k0 = (unsigned long long *)(p + L.k0);
  auto *i0 = (int32_t *)(p + L.i0);
  hipLaunchKernelGGL(k_tk_init, dim3(kTkPasses * kTkBins / 1024), dim3(1024), 0, st, state, hist,
                     k);
  for (int pass = 0; pass < kTkPasses; ++pass)
    hipLaunchKernelGGL(k_tk_sel, dim3(L.nblk), dim3(kTkSelThreads), 0, st, vals, n, L.chunk, pass,
                       state, hist);
  const int64_t wchunk = L.chunk / kTkSelWaves;
  hipLaunchKernelGGL(k_tk_count, dim3(L.nblk), dim3(kTkSelThreads), 0, st, vals, n, wchunk, state,
                     hist, cgt, ceq);
  hipLaunchKernelGGL(k_tk_write, dim3(L.nblk), dim3(kTkSelThreads), 0, st, vals, n, wchunk, state,
                     cgt, ceq, k0, i0);
  constexpr int kGroups = kTkSort / 64;
  if (k <= kTkSort) {
    hipLaunchKernelGGL((k_tk_rank<false, kTkSort>), dim3((k + 63) / 64), dim3(kTkSelThreads), 0,
                       st, nullptr, k0, i0, k, k, true, nodes, ef_out, nullptr, nullptr);
    return hipGetLastError();
  }
  auto *k1 = (unsigned long long *)(p + L.k1);
  auto *i1 = (int32_t *)(p + L.i1);
  if (k <= kTkMerge) {
    hipLaunchKernelGGL((k_tk_rank<false, kTkSort>), dim3(L.ntile * kGroups), dim3(kTkSelThreads),
                       0, st, nullptr, k0, i0, k, k, false, nullptr, nullptr, k1, i1);
    hipLaunchKernelGGL(k_tk_merge, dim3((k + 255) / 256), dim3(256), 0, st, k1, i1, k, nodes,
                       ef_out);
    return hipGetLastError();
  }
  auto *rh = (uint32_t *)(p + L.rhist);
  unsigned long long *ka = k0, *kb = k1;
  int32_t *ia = i0, *ib = i1;
  for (int shift = 0; shift < 64; shift += 8) {
    hipLaunchKernelGGL(k_tk_rhist, dim3(L.nsort), dim3(kTkThreads), 0, st, ka, k, shift, L.nsort,
                       rh);
    hipLaunchKernelGGL(k_tk_rscan, dim3(1), dim3(1024), 0, st, rh, L.nsort, k, state);
    hipLaunchKernelGGL(k_tk_scatter, dim3(L.nsort), dim3(kTkThreads), 0, st, ka, ia, kb, ib, k,
                       shift, rh, L.nsort, state);
    std::swap(ka, kb);
    std::swap(ia, ib);
  }
  hipLaunchKernelGGL(k_tk_emit, dim3((unsigned)std::min<int64_t>((k + 255) / 256, 4096)),
                     dim3(256), 0, st, ka, ia, k, nodes, ef_out);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Top-k for callers that cannot allocate (code under HIP graph capture,
// serving loops): the same kernels on a fixed scratch array instead of
// workspace from a graph handle. Each device holds its own copy of the array
// from module load to process end; host code reaches it only through the
// address hipGetSymbolAddress returns on that device.
// ---------------------------------------------------------------------------
constexpr size_t kNoAllocScratchBytes = (size_t)3 << 20;
constexpr int32_t kNoAllocMaxK = 65536;
constexpr int kNoAllocMaxDevices = 64;
static_assert(kNoAllocMaxK <= kTkMerge, "the largest k needs no radix sort scratch");

static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

namespace {
std::mutex g_scratch_mu;
void *g_scratch_ptr[kNoAllocMaxDevices] = {};

// device address of `scratch` on the current device, resolved once per device
hipError_t noalloc_scratch(void **out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kNoAllocMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!ptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}
}  // namespace

}  // namespace efi

extern "C" ef_status ef_topk_values_noalloc(const double *ef_in, int32_t n, int32_t k,
                                            int32_t *nodes, double *ef, uint32_t flags,
                                            void *hip_stream) {
  using namespace efi;
  if (n < 0 || k < 0 || k > n) {
    set_error("ef_topk_values_noalloc: need 0 <= k <= n (k=%d, n=%d)", k, n);
    return EF_ERR_ARG;
  }
  if (k > kNoAllocMaxK) {
    set_error("ef_topk_values_noalloc: k=%d above the fixed-scratch limit %d", k, kNoAllocMaxK);
    return EF_ERR_ARG;
  }
  if (flags != EF_OUT_DEVICE) {
    set_error("ef_topk_values_noalloc: flags must be EF_OUT_DEVICE (device outputs), got 0x%x",
              flags);
    return EF_ERR_ARG;
  }
  if (k == 0) return EF_OK;
  if (!ef_in || !nodes) {
    set_error("ef_topk_values_noalloc: null values or output");
    return EF_ERR_ARG;
  }
  const size_t need = topk_scratch_bytes(n, k);
  if (need > kNoAllocScratchBytes) {
    set_error("ef_topk_values_noalloc: n=%d, k=%d need %zu scratch bytes, above %zu", n, k, need,
              kNoAllocScratchBytes);
    return EF_ERR_ARG;
  }
  void *ptr = nullptr;
  hipError_t e = noalloc_scratch(&ptr);
  if (e != hipSuccess) return hip_status(e, "fixed scratch address");
  e = launch_topk(ef_in, n, k, ptr, kNoAllocScratchBytes, nodes, ef, (hipStream_t)hip_stream);
  if (e != hipSuccess) return hip_status(e, "top-k");
  return EF_OK;
}
