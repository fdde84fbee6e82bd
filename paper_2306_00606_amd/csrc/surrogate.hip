// Learned surrogate for Expected Force: per-node features, and a small MLP
// (16 -> 64 -> GELU -> 64 -> GELU -> 1, GELU in its tanh form) with BF16 operands and FP32
// accumulation on the gfx950 matrix cores (v_mfma_f32_32x32x16_bf16), trained
// on the GPU by its own forward and backward kernels and an Adam step.
//
// The network predicts the residual y = ln N(s) - EF(s) >= 0 (EF is at most
// ln N, with equality when all clusters of s have the same degree); the
// predicted EF is max(0, ln N - y).
//
// MFMA operand layouts (wave64, 32x32x16): lane l holds
//   A[i][k]  for i = l % 32, k = 8 (l / 32) + j          (8 bf16, j = 0..7)
//   B[k][n]  for n = l % 32, k = 8 (l / 32) + j          (8 bf16)
//   C[i][n]  for n = l % 32, i = 8 (r / 4) + 4 (l / 32) + r % 4  (16 fp32, r = 0..15)
// Weights are kept as FP32 masters and re-packed into the B layout (bf16)
// after every optimiser step.
#include "device_common.h"

namespace efi {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kF = 16, kH = 64;
// flat parameter vector
constexpr int kOffW1 = 0, kOffB1 = 1024, kOffW2 = 1088, kOffB2 = 5184, kOffW3 = 5248,
              kOffB3 = 5312, kParams = 5313;
// packed bf16 B-operand blocks (64 lanes x 8 values each)
constexpr int kPackW1 = 0;                  // kb 1 x nb 2
constexpr int kPackW2 = 2;                  // kb 4 x nb 2
constexpr int kPackW3 = 10;                 // kb 4 x nb 1 (column 0 = w3)
constexpr int kPackW2T = 14;                // kb 4 x nb 2 (W2 transposed)
constexpr int kPackBlocks = 22;

__device__ __forceinline__ int c_row(int r, int lane) {
  return ((r >> 2) << 3) + ((lane >> 5) << 2) + (r & 3);
}
__device__ __forceinline__ f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
// GELU in its tanh form (Hendrycks and Gimpel, 2016), the tanh from one
// exponential and one hardware reciprocal (v_rcp_f32, 1 ulp; the GELUs feed
// BF16 operands): tanh(u) = 1 - 2 / (1 + e^{2u}) (e^{2u} overflowing to inf
// gives 1, underflowing to 0 gives -1)
__device__ __forceinline__ float gelu_tanh_arg(float z) {
  return 0.7978845608028654f * (z + 0.044715f * z * z * z);
}
__device__ __forceinline__ float fast_tanh(float u) {
  return 1.0f - 2.0f * __builtin_amdgcn_rcpf(1.0f + __expf(2.0f * u));
}
__device__ __forceinline__ float gelu(float z) {
  return 0.5f * z * (1.0f + fast_tanh(gelu_tanh_arg(z)));
}
__device__ __forceinline__ float gelu_grad(float z) {
  const float t = fast_tanh(gelu_tanh_arg(z));
  return 0.5f * (1.0f + t) +
         0.5f * z * (1.0f - t * t) * 0.7978845608028654f * (1.0f + 0.134145f * z * z);
}
__device__ __forceinline__ float bf(float x) { return (float)(__bf16)x; }

// ---------------------------------------------------------------------------
// features: G lanes per node (8 for degree <= kFinGroupMax, 32 for degree <=
// kFinHalfMax, 64 up to kFinBlockMin), one workgroup per hub
// ---------------------------------------------------------------------------
// Moments of the cluster degrees. Per arc (s, a), with c = k_s + k_a - 4,
// the clusters through a have degree c + k_b for the n = k_s + k_a - 2
// nodes b in N(s) \ {a} (stars) and N(a) \ {s} (paths), so with P_j the
// sum of k_b^j over those b (from the sums of both nodes' neighbour degrees
// to the power j, less k_a^j and k_s^j),
//   sum d^2 = n c^2 + 2 c P_1 + P_2
//   sum d^3 = n c^3 + 3 c^2 P_1 + 3 c P_2 + P_3
//   sum d^4 = n c^4 + 4 c^3 P_1 + 6 c^2 P_2 + 4 c P_3 + P_4
// (triangle clusters taken without their -2). With x = d / mean - 1 over the
// node's event sequences, ln N - EF = E[(1 + x) ln(1 + x)]
// = m2 / 2 - m3 / 6 + m4 / 12 - ..., m_j = E[x^j]; the features carry m2,
// m3 and m4. No triangle pass is needed.
struct FeatAcc {  // POD (lives in LDS); start from feat_zero()
  int64_t B, Q;
  int32_t c1;
  float mx, mn;
  double s1, s2, e2, e3, e4;
  __device__ void add(int2 ad, const NbrMoments &t, int64_t k, const NbrMoments &own) {
    const int64_t ka = ad.y;
    B += ka * ka;
    Q += t.s1;
    c1 += ka == 1;
    const float lk = logf((float)ka);
    mx = fmaxf(mx, lk);
    mn = fminf(mn, lk);
    s1 += lk;
    s2 += (double)lk * lk;
    const double n = (double)(k + ka - 2), c = (double)(k + ka - 4);
    const double dk = (double)k, da = (double)ka, dk2 = dk * dk, da2 = da * da;
    const double p1 = (double)(own.s1 - ka + t.s1 - k);
    const double p2 = (double)(own.s2 - ka * ka + t.s2 - k * k);
    const double p3 = own.s3 - da2 * da + t.s3 - dk2 * dk;
    const double p4 = own.s4 - da2 * da2 + t.s4 - dk2 * dk2;
    const double c2 = c * c;
    e2 += n * c2 + 2.0 * c * p1 + p2;
    e3 += n * c2 * c + 3.0 * c2 * p1 + 3.0 * c * p2 + p3;
    e4 += n * c2 * c2 + 4.0 * c2 * c * p1 + 6.0 * c2 * p2 + 4.0 * c * p3 + p4;
  }
  __device__ void merge(const FeatAcc &o) {
    B += o.B;
    Q += o.Q;
    c1 += o.c1;
    mx = fmaxf(mx, o.mx);
    mn = fminf(mn, o.mn);
    s1 += o.s1;
    s2 += o.s2;
    e2 += o.e2;
    e3 += o.e3;
    e4 += o.e4;
  }
};

__device__ __forceinline__ FeatAcc feat_zero() {
  FeatAcc a;
  a.B = a.Q = a.c1 = 0;
  a.mx = -1e30f;
  a.mn = 1e30f;
  a.s1 = a.s2 = a.e2 = a.e3 = a.e4 = 0.0;
  return a;
}

// x of lane i ^ OFF, where the lanes of each group of OFF hold the same x
template <int OFF> __device__ __forceinline__ int32_t lane_xor(int32_t x) {
  // quad_perm [1,0,3,2] and [2,3,0,1], row_half_mirror, row_ror:8
  constexpr int kCtl = OFF == 1 ? 0xB1 : OFF == 2 ? 0x4E : OFF == 4 ? 0x141 : 0x128;
  if constexpr (OFF <= 8) return __builtin_amdgcn_update_dpp(0, x, kCtl, 0xF, 0xF, true);
  return __shfl_xor(x, OFF, 64);
}
template <int OFF> __device__ __forceinline__ long long lane_xor(long long x) {
  const int32_t lo = lane_xor<OFF>((int32_t)x), hi = lane_xor<OFF>((int32_t)(x >> 32));
  return (long long)(((unsigned long long)(uint32_t)hi << 32) | (uint32_t)lo);
}
template <int OFF> __device__ __forceinline__ float lane_xor(float x) {
  return __int_as_float(lane_xor<OFF>(__float_as_int(x)));
}
template <int OFF> __device__ __forceinline__ double lane_xor(double x) {
  return __longlong_as_double(lane_xor<OFF>((long long)__double_as_longlong(x)));
}

// the sums over the G lanes of a group, on each of them
template <int G, int OFF = 1> __device__ __forceinline__ void feat_reduce(FeatAcc &a) {
  if constexpr (OFF < G) {
    FeatAcc o;
    o.B = lane_xor<OFF>((long long)a.B);
    o.Q = lane_xor<OFF>((long long)a.Q);
    o.c1 = lane_xor<OFF>(a.c1);
    o.mx = lane_xor<OFF>(a.mx);
    o.mn = lane_xor<OFF>(a.mn);
    o.s1 = lane_xor<OFF>(a.s1);
    o.s2 = lane_xor<OFF>(a.s2);
    o.e2 = lane_xor<OFF>(a.e2);
    o.e3 = lane_xor<OFF>(a.e3);
    o.e4 = lane_xor<OFF>(a.e4);
    a.merge(o);
    feat_reduce<G, OFF * 2>(a);
  }
}

// two arcs of a row at a time, i and i + stride; the second repeats the first
// past the row's end, so that their loads are in flight together
struct FeatPair {
  int2 a0, a1;
};
__device__ __forceinline__ FeatPair feat_pair(const int2 *__restrict__ adj2, int32_t k,
                                              int32_t base, int32_t i, int32_t stride) {
  FeatPair p{{0, 0}, {0, 0}};
  if (i < k) {
    p.a0 = adj2[base + i];
    p.a1 = adj2[base + (i + stride < k ? i + stride : i)];
  }
  return p;
}
// arcs first, first + stride, ... of a node (degree k, own sums own); p: the
// first two
__device__ __forceinline__ void feat_arcs(const int2 *__restrict__ adj2,
                                          const NbrMoments *__restrict__ nbm, int32_t k,
                                          int32_t base, const NbrMoments &own, int32_t first,
                                          int32_t stride, FeatPair p, FeatAcc &f) {
  for (int32_t i = first; i < k; i += 2 * stride) {
    const NbrMoments m0 = nbm[p.a0.x], m1 = nbm[p.a1.x];
    const FeatPair q = feat_pair(adj2, k, base, i + 2 * stride, stride);
    f.add(p.a0, m0, k, own);
    if (i + stride < k) f.add(p.a1, m1, k, own);
    p = q;
  }
}

// the features of a node, standardised where mean is given; returns ln N(s)
__device__ __forceinline__ float feat_values(int32_t k, int64_t A, const FeatAcc &a,
                                             const float *__restrict__ mean,
                                             const float *__restrict__ inv_std, float (&f)[kF]) {
  const int64_t kk = k, B = a.B, Q = a.Q;
  const int64_t Ns = kk * kk - 2 * kk + A;
  // D without the triangle term
  const int64_t Ds = kk * (kk - 1) * (kk - 4) + 2 * (kk - 1) * A + (kk - 4) * (A - kk) +
                     (B - A) + (Q - kk * kk);
  // raw moments of d / mean, then the central moments of x = d / mean - 1
  double m2 = 0.0, m3 = 0.0, m4 = 0.0;
  if (Ns > 0 && Ds > 0) {
    const double q = (double)Ns / (double)Ds;  // 1 / mean
    const double r2 = a.e2 * q * q / (double)Ns, r3 = a.e3 * q * q * q / (double)Ns,
                 r4 = a.e4 * q * q * q * q / (double)Ns;
    m2 = r2 - 1.0;
    m3 = r3 - 3.0 * r2 + 2.0;
    m4 = r4 - 4.0 * r3 + 6.0 * r2 - 3.0;
  }
  f[0] = logf(1.0f + (float)kk);
  f[1] = logf(1.0f + (float)A);
  f[2] = logf(1.0f + (float)B);
  f[3] = (float)asinh(m3);
  f[4] = (float)asinh(m4);
  f[5] = logf(1.0f + (float)(A - kk));
  f[6] = logf(1.0f + (float)Ns);
  f[7] = logf(1.0f + (float)Ds);
  f[8] = (Ns > 0 && Ds > 0) ? (float)log((double)Ds / (double)Ns) : 0.0f;
  const double mean_lk = k > 0 ? a.s1 / k : 0.0;
  f[9] = k > 0 ? a.mx : 0.0f;
  f[10] = k > 0 ? a.mn : 0.0f;
  f[11] = (float)mean_lk;
  f[12] = k > 0 ? (float)sqrt(fmax(a.s2 / k - mean_lk * mean_lk, 0.0)) : 0.0f;
  f[13] = logf(1.0f + (float)Q);
  f[14] = k > 0 ? (float)a.c1 / (float)k : 0.0f;
  f[15] = (float)log1p(fmax(m2, 0.0));
  if (mean) {
#pragma unroll
    for (int i = 0; i < kF; ++i) f[i] = (f[i] - mean[i]) * inv_std[i];
  }
  return Ns > 0 ? logf((float)Ns) : 0.0f;
}

// ---------------------------------------------------------------------------
// MLP on one 32-row tile per wavefront
// ---------------------------------------------------------------------------
struct TileLds {  // training: one tile, shared by two wavefronts
  __bf16 x[32][kF];
  __bf16 h1[32][kH];
  __bf16 h2[32][kH];
  __bf16 dz[32][kH];
  float dy[32];
};
// inference: a wavefront's rows and one hidden layer at a time. Rows are 16
// bytes longer than their values, so that the A fragments of neighbouring rows
// lie in different banks.
constexpr int kXPad = kF + 8, kHPad = kH + 8;
struct __align__(16) FwdLds {
  __bf16 x[64][kXPad];
  __bf16 h[32][kHPad];
};

__device__ __forceinline__ bf16x8 lds_a(const __bf16 *rowmajor, int ld, int kb) {
  // A fragment: row lane % 32, columns 16 kb + 8 (lane / 32) .. + 7
  const int lane = threadIdx.x & 63;
  return *reinterpret_cast<const bf16x8 *>(rowmajor + (lane & 31) * ld + kb * 16 +
                                           ((lane >> 5) << 3));
}
// B fragment from a row-major [K][ld] LDS matrix: column nb*32 + lane%32,
// rows 16 kb + 8 (lane / 32) .. + 7
__device__ __forceinline__ bf16x8 lds_b(const __bf16 *rowmajor, int ld, int kb, int nb) {
  const int lane = threadIdx.x & 63;
  bf16x8 v;
  const int r0 = kb * 16 + ((lane >> 5) << 3), c = nb * 32 + (lane & 31);
#pragma unroll
  for (int j = 0; j < 8; ++j) v[j] = rowmajor[(r0 + j) * ld + c];
  return v;
}
// A fragment of the transpose of a row-major [K][ld] LDS matrix: A[m][kk] =
// M[kk][m], m = mb*32 + lane%32 (zero when m >= mlim), kk = 16 kb + 8 (lane/32) + j
__device__ __forceinline__ bf16x8 lds_at(const __bf16 *rowmajor, int ld, int kb, int mb,
                                         int mlim) {
  const int lane = threadIdx.x & 63;
  bf16x8 v;
  const int r0 = kb * 16 + ((lane >> 5) << 3), m = mb * 32 + (lane & 31);
#pragma unroll
  for (int j = 0; j < 8; ++j) v[j] = m < mlim ? rowmajor[(r0 + j) * ld + m] : (__bf16)0.0f;
  return v;
}
__device__ __forceinline__ bf16x8 wpack(const __bf16 *pack, int block) {
  return reinterpret_cast<const bf16x8 *>(pack)[block * 64 + (threadIdx.x & 63)];
}

// Forward of the 32 rows x on one wavefront; h: LDS for the hidden layers (the
// first is in registers, as A fragments, before the second takes its place).
// Returns y for the rows held by lanes 0 and 32 (C layout of column 0).
__device__ __forceinline__ f32x16 tile_forward(const __bf16 (*x)[kXPad], __bf16 (*h)[kHPad],
                                               const float *__restrict__ P,
                                               const __bf16 *__restrict__ pack) {
  const int lane = threadIdx.x & 63;
  wave_sync();
  const bf16x8 ax = lds_a(&x[0][0], kXPad, 0);
#pragma unroll
  for (int nb = 0; nb < 2; ++nb) {
    f32x16 c = {};
    c = mfma(ax, wpack(pack, kPackW1 + nb), c);
    const float b1 = P[kOffB1 + nb * 32 + (lane & 31)];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      c[r] += b1;
      h[c_row(r, lane)][nb * 32 + (lane & 31)] = (__bf16)gelu(c[r]);
    }
  }
  wave_sync();
  bf16x8 ah[4];
#pragma unroll
  for (int kb = 0; kb < 4; ++kb) ah[kb] = lds_a(&h[0][0], kHPad, kb);
  wave_sync();
#pragma unroll
  for (int nb = 0; nb < 2; ++nb) {
    f32x16 c = {};
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) c = mfma(ah[kb], wpack(pack, kPackW2 + kb * 2 + nb), c);
    const float b2 = P[kOffB2 + nb * 32 + (lane & 31)];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      c[r] += b2;
      h[c_row(r, lane)][nb * 32 + (lane & 31)] = (__bf16)gelu(c[r]);
    }
  }
  wave_sync();
  f32x16 c = {};
#pragma unroll
  for (int kb = 0; kb < 4; ++kb)
    c = mfma(lds_a(&h[0][0], kHPad, kb), wpack(pack, kPackW3 + kb), c);
  const float b3 = P[kOffB3];
#pragma unroll
  for (int r = 0; r < 16; ++r) c[r] += b3;
  return c;
}

// y of rows [0, rows) of X (rows past the end are zero)
__global__ __launch_bounds__(256) void k_mlp_forward(const float *__restrict__ X, int64_t rows,
                                                     const float *__restrict__ P,
                                                     const __bf16 *__restrict__ pack,
                                                     float *__restrict__ y_out) {
  __shared__ FwdLds lds[4];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  FwdLds &L = lds[wv];
  const int64_t tiles = (rows + 31) / 32;
  for (int64_t tile = (int64_t)blockIdx.x * 4 + wv; tile < tiles; tile += (int64_t)gridDim.x * 4) {
    const int i = lane & 31, c0 = (lane >> 5) * 8;
    const int64_t row = tile * 32 + i;
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
    if (row < rows) {
      a = *reinterpret_cast<const float4 *>(X + row * kF + c0);
      b = *reinterpret_cast<const float4 *>(X + row * kF + c0 + 4);
    }
    const float xv[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    for (int j = 0; j < 8; ++j) L.x[i][c0 + j] = (__bf16)xv[j];
    const f32x16 y = tile_forward(L.x, L.h, P, pack);
    if ((lane & 31) == 0) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t out = tile * 32 + c_row(r, lane);
        if (out < rows) y_out[out] = y[r];
      }
    }
  }
}

struct FeatArgs {
  const int32_t *row_ptr, *deg;
  const int2 *adj2;
  const NbrMoments *nbm;
  const float *mean, *inv_std;
  float *X, *lnN;         // features and ln N by node, or
  const float *P;         // the network and its predictions
  const __bf16 *pack;
  double *ef;
};
struct FeatNode {  // a lane's node (v < 0: none) and its sums
  FeatAcc f;
  int32_t v, k;
  int64_t s1;
};

// Item i0 of a wavefront: R rounds of 64 / G nodes of `nodes` (NULL: node ids
// 0..count-1 of degree <= kmax), G lanes per node. Lane r of a group keeps the
// node of round r, so that one pass over the features' formulas (some 900
// instructions, most in FP64) and the network serves 64 R / G nodes.
template <int G, int R>
__device__ __forceinline__ FeatNode feat_groups(const FeatArgs &A, const int32_t *nodes,
                                                int64_t count, int32_t kmax, int64_t i0) {
  static_assert(R <= G, "a lane keeps one node");
  constexpr int W = 64 / G;  // nodes per round
  const int lane = threadIdx.x & 63, sub = lane & (G - 1), grp = lane / G;
  FeatNode o{feat_zero(), -1, 0, 0};
  const int64_t it = i0 + sub * W + grp;
  int32_t bk = 0;
  if (sub < R && it < count) {
    o.v = nodes ? nodes[it] : (int32_t)it;
    o.k = A.deg[o.v];
    bk = A.row_ptr[o.v];
    if (!nodes && o.k > kmax) o.v = -1;
    if (o.v < 0) o.k = 0;
  }
  int32_t k = __shfl(o.k, 0, G), base = __shfl(bk, 0, G);
  FeatPair p = feat_pair(A.adj2, k, base, sub, G);
  for (int r = 0; r < R; ++r) {
    const int32_t v = __shfl(o.v, r, G);
    const int32_t kn = r + 1 < R ? __shfl(o.k, r + 1, G) : 0,
                  bn = r + 1 < R ? __shfl(bk, r + 1, G) : 0;
    const FeatPair q = feat_pair(A.adj2, kn, bn, sub, G);  // the next round's
    FeatAcc f = feat_zero();
    NbrMoments own{0, 0, 0.0, 0.0};
    if (v >= 0) {
      own = A.nbm[v];
      feat_arcs(A.adj2, A.nbm, k, base, own, sub, G, p, f);
    }
    feat_reduce<G>(f);
    if (sub == r) {
      o.f = f;
      o.s1 = own.s1;
    }
    k = kn;
    base = bn;
    p = q;
  }
  return o;
}

// hub v on the whole workgroup of NT threads; thread 0 holds it
template <int NT>
__device__ __forceinline__ FeatNode feat_hub(const FeatArgs &A, int32_t v) {
  __shared__ FeatAcc sh[NT / 64];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int32_t k = A.deg[v], base = A.row_ptr[v];
  FeatNode o{feat_zero(), tid == 0 ? v : -1, k, 0};
  const NbrMoments own = A.nbm[v];
  o.s1 = own.s1;
  feat_arcs(A.adj2, A.nbm, k, base, own, tid, NT, feat_pair(A.adj2, k, base, tid, NT), o.f);
  feat_reduce<64>(o.f);
  __syncthreads();  // the previous hub's sums have been read
  if (lane == 0) sh[wv] = o.f;
  __syncthreads();
  if (tid == 0)
    for (int w = 1; w < NT / 64; ++w) o.f.merge(sh[w]);
  return o;
}

// One launch for every node, the longest rows first: hubs, a workgroup each
// (blocks [0, b0)), degree kFinHalfMax+1 .. kFinBlockMin, a wavefront each
// ([b0, b1)), kFinGroupMax+1 .. kFinHalfMax, 32 lanes each ([b1, b2)), and the
// rest, 8 lanes each (node ids). PREDICT: the wavefront that has the features
// of its nodes runs the network on them and writes the predicted EF.
// Bound by the gathers of the neighbours' moments: a 128-byte sector of the
// memory-side cache for 32 bytes of each arc (BA n = 1M, m = 8: 15M of them,
// 7 TB/s), with the formulas and the GELUs beside them. That graph: 303 us; with
// the network in a launch of its own 355 us, and with a launch per tier and the
// formulas on one lane of eight 563 us.
template <int R, bool PREDICT, int NT>
__global__ __launch_bounds__(NT) void k_features(FeatArgs A, const int32_t *l_hub, int64_t n_hub,
                                                  const int32_t *l_wave, int64_t n_wave,
                                                  const int32_t *l_half, int64_t n_half, int64_t n,
                                                  int64_t b0, int64_t b1, int64_t b2) {
  constexpr int W = NT / 64;
  __shared__ FwdLds lds[PREDICT ? W : 1];
  const int64_t b = blockIdx.x;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  // this wavefront's items: first, step and end; and a lane's row in the tile
  // (feat_groups: round sub, group grp)
  int64_t i0, step, end;
  int row, rows;
  if (b < b0) {
    i0 = b, step = b0, end = n_hub, row = 0, rows = wv == 0 ? 1 : 0;
  } else if (b < b1) {
    i0 = (b - b0) * W + wv, step = (b1 - b0) * W, end = n_wave, row = lane, rows = 1;
  } else if (b < b2) {
    i0 = ((b - b1) * W + wv) * 2 * R, step = (b2 - b1) * W * 2 * R, end = n_half;
    row = (lane & 31) * 2 + (lane >> 5), rows = 2 * R;
  } else {
    i0 = ((b - b2) * W + wv) * 8 * R, step = ((int64_t)gridDim.x - b2) * W * 8 * R, end = n;
    row = (lane & 7) * 8 + (lane >> 3), rows = 8 * R;
  }
  for (; i0 < end; i0 += step) {
    const FeatNode o = b < b0   ? feat_hub<NT>(A, l_hub[i0])
                       : b < b1 ? feat_groups<64, 1>(A, l_wave, n_wave, 0, i0)
                       : b < b2 ? feat_groups<32, R>(A, l_half, n_half, 0, i0)
                                : feat_groups<8, R>(A, nullptr, n, kFinGroupMax, i0);
    float f[kF], ln = 0.0f;
    if (o.v >= 0) ln = feat_values(o.k, o.s1, o.f, A.mean, A.inv_std, f);
    if constexpr (!PREDICT) {
      if (o.v >= 0) {
        float *dst = A.X + (int64_t)o.v * kF;
#pragma unroll
        for (int i = 0; i < kF; ++i) dst[i] = f[i];
        A.lnN[o.v] = ln;
      }
    } else {
      FwdLds &L = lds[wv];
      wave_sync();  // the previous item's rows have been read
      if (o.v >= 0) {
#pragma unroll
        for (int i = 0; i < kF; ++i) L.x[row][i] = (__bf16)f[i];
      }
      // (rows without a node hold what was there: a row's values reach no other)
      for (int t = 0; t < rows; t += 32) {
        const f32x16 y = tile_forward(&L.x[t], L.h, A.P, A.pack);
        wave_sync();
        float *ys = reinterpret_cast<float *>(&L.h[0][0]);
        if ((lane & 31) == 0) {
#pragma unroll
          for (int r = 0; r < 16; ++r) ys[c_row(r, lane)] = y[r];
        }
        wave_sync();
        if (o.v >= 0 && row >= t && row < t + 32) {
          const float e = ln - ys[row - t];
          A.ef[o.v] = e > 0.0f ? (double)e : 0.0;
        }
        wave_sync();
      }
    }
  }
}

template <int R, bool PREDICT, int NT>
static hipError_t features_impl(const Graph &g, const FeatArgs &A, hipStream_t st) {
  constexpr int W = NT / 64;
  auto blocks = [](int64_t count, int64_t per) {
    return count > 0 ? std::min<int64_t>((count + per - 1) / per, 1 << 20) : 0;
  };
  const int64_t n_wave = g.n_fin - g.n_fin_hub - g.n_fin_half;
  const int32_t *l_wave = g.fin_list + g.n_fin_hub, *l_half = l_wave + n_wave;
  const int64_t b0 = blocks(g.n_fin_hub, 1), b1 = b0 + blocks(n_wave, W),
                b2 = b1 + blocks(g.n_fin_half, W * 2 * R), grid = b2 + blocks(g.n, W * 8 * R);
  hipLaunchKernelGGL((k_features<R, PREDICT, NT>), dim3((unsigned)grid), dim3(NT), 0, st, A,
                     g.fin_list, g.n_fin_hub, l_wave, n_wave, l_half, g.n_fin_half, (int64_t)g.n,
                     b0, b1, b2);
  return hipGetLastError();
}

// Eight rounds per wavefront from kFeatRounds nodes on: below, as many
// wavefronts as one round gives are wanted (predictions on BA, m = 8, one and
// eight rounds: 4000 nodes 12 and 27 us, 32000 30 and 41, 64000 52 and 46; a
// million 816 and 303).
constexpr int32_t kFeatRounds = 1 << 16;

// Workgroups of 512 threads, of which a hub takes one, where the largest hub
// alone takes longer than the rest of the graph: it sums its arcs at some 0.77 a
// nanosecond on 256 threads (bound by the formulas of one CU) and 1.2 on 512,
// the rest at some 50. Elsewhere 256: more workgroups per CU (predictions on
// stars of 50k, 200k and 1M arcs: 62, 191 and 830 us; 71, 282 and 1294 with 256
// threads, 75, 182 and 747 with 1024; R-MAT scale 22 2034 us against 1814, BA
// n = 1M, m = 8 361 against 340).
constexpr int32_t kFeatWide = 32768;
template <bool PREDICT>
static hipError_t features_by_size(const Graph &g, const FeatArgs &A, hipStream_t st) {
  const int32_t k = g.info.max_degree;
  const bool wide = k > kFeatWide && k > g.nnz / 64;
  if (g.n >= kFeatRounds)
    return wide ? features_impl<8, PREDICT, 512>(g, A, st)
                : features_impl<8, PREDICT, 256>(g, A, st);
  return wide ? features_impl<1, PREDICT, 512>(g, A, st)
              : features_impl<1, PREDICT, 256>(g, A, st);
}

hipError_t launch_features(const Graph &g, const float *mean, const float *inv_std, float *X,
                           float *lnN, hipStream_t st) {
  const FeatArgs A{g.row_ptr, g.deg, g.adj2, g.nbm, mean, inv_std, X, lnN, nullptr, nullptr,
                   nullptr};
  return features_by_size<false>(g, A, st);
}

// predicted EF of every node: max(0, ln N - y)
hipError_t launch_predict(const Graph &g, const float *mean, const float *inv_std, const float *P,
                          const __bf16 *pack, double *ef, hipStream_t st) {
  const FeatArgs A{g.row_ptr, g.deg, g.adj2, g.nbm, mean, inv_std, nullptr, nullptr, P, pack, ef};
  return features_by_size<true>(g, A, st);
}

// Training: gradients of the mean squared error over the rows perm[b0 .. b0+nb)
// (scale = 2 / nb), one workgroup per tile slot (tiles slot, slot + grid, ...),
// accumulated into part[slot][kParams]; the squared-error sum into
// part_loss[slot]. A tile is shared by two wavefronts, each with one half of
// the 64 hidden columns: a training step has one tile per slot and as many
// slots as fill half the CUs, so its time is the tile's serial chain, and the
// halves run the same products and sums (the same bits) with half the GELUs
// each (4096 rows: 12.8 us, 22.9 with one wavefront per tile).
__global__ __launch_bounds__(128) void k_mlp_grad(const float *__restrict__ X,
                                                  const float *__restrict__ Yt,
                                                  const int32_t *__restrict__ perm, int64_t b0,
                                                  int64_t nrows, const float *__restrict__ P,
                                                  const __bf16 *__restrict__ pack,
                                                  float *__restrict__ part,
                                                  float *__restrict__ part_loss) {
  __shared__ TileLds t;
  const int lane = threadIdx.x & 63, nb = threadIdx.x >> 6;  // nb: this wavefront's column half
  const int64_t tiles = (nrows + 31) / 32;
  const float scale = 2.0f / (float)nrows;
  const int col = lane & 31, hc = nb * 32 + col;
  f32x16 gW2[2] = {}, gW1 = {};
  float gb1 = 0.f, gb2 = 0.f, gw3 = 0.f, gb3 = 0.f, lsum = 0.f;
  const float w3b = bf(P[kOffW3 + hc]), b1 = P[kOffB1 + hc], b2 = P[kOffB2 + hc], b3 = P[kOffB3];
  // this half's weights stay in registers over the tiles
  const bf16x8 w1 = wpack(pack, kPackW1 + nb);
  bf16x8 w2[4], w2t[4], w3[4];
#pragma unroll
  for (int kb = 0; kb < 4; ++kb) {
    w2[kb] = wpack(pack, kPackW2 + kb * 2 + nb);
    w2t[kb] = wpack(pack, kPackW2T + kb * 2 + nb);
    w3[kb] = wpack(pack, kPackW3 + kb);
  }
  const int32_t *pr = perm + b0;
  for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    {
      const int i = threadIdx.x & 31, c0 = (threadIdx.x >> 5) * 4;
      const int64_t row = tile * 32 + i;
      float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
      if (row < nrows) a = *reinterpret_cast<const float4 *>(X + (int64_t)pr[row] * kF + c0);
      t.x[i][c0] = (__bf16)a.x;
      t.x[i][c0 + 1] = (__bf16)a.y;
      t.x[i][c0 + 2] = (__bf16)a.z;
      t.x[i][c0 + 3] = (__bf16)a.w;
    }
    __syncthreads();
    f32x16 z1 = {}, z2 = {}, yv = {};
    z1 = mfma(lds_a(&t.x[0][0], kF, 0), w1, z1);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      z1[r] += b1;
      t.h1[c_row(r, lane)][hc] = (__bf16)gelu(z1[r]);
    }
    __syncthreads();
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) z2 = mfma(lds_a(&t.h1[0][0], kH, kb), w2[kb], z2);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      z2[r] += b2;
      t.h2[c_row(r, lane)][hc] = (__bf16)gelu(z2[r]);
    }
    __syncthreads();
    if (nb == 0) {
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) yv = mfma(lds_a(&t.h2[0][0], kH, kb), w3[kb], yv);
      if (col == 0) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int i = c_row(r, lane);
          const int64_t row = tile * 32 + i;
          float d = 0.f;
          if (row < nrows) {
            const float res = yv[r] + b3 - Yt[pr[row]];
            lsum += res * res;
            d = scale * res;
          }
          t.dy[i] = d;
          gb3 += d;
        }
      }
    }
    __syncthreads();
    // layer 3 and dz2 = dy w3 * gelu'(z2)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = c_row(r, lane);
      const float d = t.dy[i];
      gw3 += (float)t.h2[i][hc] * d;
      const float dz = d * w3b * gelu_grad(z2[r]);
      gb2 += dz;
      t.dz[i][hc] = (__bf16)dz;
    }
    __syncthreads();
    // dW2 += h1^T dz2 ; dh1 = dz2 W2^T
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      const bf16x8 dzb = lds_b(&t.dz[0][0], kH, kb, nb);
#pragma unroll
      for (int mb = 0; mb < 2; ++mb)
        gW2[mb] = mfma(lds_at(&t.h1[0][0], kH, kb, mb, kH), dzb, gW2[mb]);
    }
    f32x16 dh1 = {};
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) dh1 = mfma(lds_a(&t.dz[0][0], kH, kb), w2t[kb], dh1);
    __syncthreads();
    // dz1 = dh1 * gelu'(z1)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float dz = dh1[r] * gelu_grad(z1[r]);
      gb1 += dz;
      t.dz[c_row(r, lane)][hc] = (__bf16)dz;
    }
    __syncthreads();
    // dW1 += x^T dz1 (rows 16..31 of the A operand are zero)
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
      gW1 = mfma(lds_at(&t.x[0][0], kF, kb, 0, kF), lds_b(&t.dz[0][0], kH, kb, nb), gW1);
    __syncthreads();
  }
  // write this slot's partial gradient
  float *g = part + (int64_t)blockIdx.x * kParams;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int m = c_row(r, lane);
    if (m < kF) g[kOffW1 + m * kH + hc] = gW1[r];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) g[kOffW2 + (mb * 32 + m) * kH + hc] = gW2[mb][r];
  }
  const float s1 = gb1 + __shfl_xor(gb1, 32, 64);
  const float s2 = gb2 + __shfl_xor(gb2, 32, 64);
  const float s3 = gw3 + __shfl_xor(gw3, 32, 64);
  if (lane < 32) {
    g[kOffB1 + hc] = s1;
    g[kOffB2 + hc] = s2;
    g[kOffW3 + hc] = s3;
  }
  const float sb = gb3 + __shfl_xor(gb3, 32, 64);
  const float ls = lsum + __shfl_xor(lsum, 32, 64);
  if (threadIdx.x == 0) {
    g[kOffB3] = sb;
    part_loss[blockIdx.x] = ls;
  }
}

// Sum of parameter p's partials over the slots (a workgroup of 256: 64
// parameters, a quarter of the slots per wavefront, eight loads in flight, in
// double), valid on wavefront 0; p = kParams: the squared-error sums. One
// thread per parameter walked every slot in turn (128 slots: 35 us).
__device__ __forceinline__ double grad_sum(const float *__restrict__ part,
                                           const float *__restrict__ part_loss, int32_t slots,
                                           int p) {
  __shared__ double sh[4][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int32_t per = (slots + 3) / 4, lo = w * per, hi = min(slots, lo + per);
  const float *src = p < kParams ? part + p : part_loss;
  const int64_t stride = p < kParams ? kParams : 1;
  double s = 0.0;
  if (p <= kParams) {
    int32_t i = lo;
    for (; i + 8 <= hi; i += 8) {
      float v[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = src[(i + q) * stride];
#pragma unroll
      for (int q = 0; q < 8; ++q) s += v[q];
    }
    for (; i < hi; ++i) s += src[i * stride];
  }
  sh[w][lane] = s;
  __syncthreads();
  return sh[0][lane] + sh[1][lane] + sh[2][lane] + sh[3][lane];
}

// grad[p] = sum over the slots (fixed order); loss = sum of part_loss
__global__ __launch_bounds__(256) void k_grad_reduce(const float *__restrict__ part,
                                                     const float *__restrict__ part_loss,
                                                     int32_t slots, float *__restrict__ grad,
                                                     float *__restrict__ loss) {
  const int p = blockIdx.x * 64 + (threadIdx.x & 63);
  const double s = grad_sum(part, part_loss, slots, p);
  if (threadIdx.x >= 64) return;
  if (p < kParams) grad[p] = (float)s;
  else if (p == kParams) *loss = (float)s;
}

// place of element (row k of the K dimension, column n) in packed block `block`
__device__ __forceinline__ int pack_at(int block, int k, int n) {
  return (block * 64 + (((k & 15) >> 3) << 5) + n) * 8 + (k & 7);
}

// One training step's update: the gradient's sum over the slots, Adam (Kingma
// and Ba, 2015) on the FP32 masters, step t (1-based), and the new weights'
// places in the BF16 operand blocks (the zero columns of the last layer's
// block stay as k_pack wrote them).
__global__ __launch_bounds__(256) void k_grad_step(const float *__restrict__ part, int32_t slots,
                                                   float *__restrict__ P, float *__restrict__ M,
                                                   float *__restrict__ V,
                                                   __bf16 *__restrict__ pack, float lr, float b1,
                                                   float b2, float eps, float wd, int32_t t) {
  const int p = blockIdx.x * 64 + (threadIdx.x & 63);
  const double s = grad_sum(part, nullptr, slots, p < kParams ? p : kParams + 1);
  if (threadIdx.x >= 64 || p >= kParams) return;
  const float c1 = 1.0f - powf(b1, (float)t), c2 = 1.0f - powf(b2, (float)t);
  const float g = (float)s;
  // (fused multiply-adds written out: which product is rounded decides bits)
  const float m = fmaf(1.0f - b1, g, b1 * M[p]);
  const float v = fmaf(g, (1.0f - b2) * g, b2 * V[p]);
  M[p] = m;
  V[p] = v;
  const float x = fmaf(-lr, fmaf(wd, P[p], (m / c1) / (sqrtf(v / c2) + eps)), P[p]);
  P[p] = x;
  const __bf16 w = (__bf16)x;
  if (p < kOffB1) {
    const int k = p / kH, n = p % kH;
    pack[pack_at(kPackW1 + n / 32, k, n % 32)] = w;
  } else if (p >= kOffW2 && p < kOffB2) {
    const int k = (p - kOffW2) / kH, n = (p - kOffW2) % kH;
    pack[pack_at(kPackW2 + (k / 16) * 2 + n / 32, k, n % 32)] = w;
    pack[pack_at(kPackW2T + (n / 16) * 2 + k / 32, n, k % 32)] = w;
  } else if (p >= kOffW3 && p < kOffB3) {
    const int k = p - kOffW3;
    pack[pack_at(kPackW3 + k / 16, k, 0)] = w;
  }
}

// ---------------------------------------------------------------------------
// standardisation of training rows: column means and spreads in double (two
// passes, per-workgroup sums added in a fixed order), then (x - mean) inv_std
// ---------------------------------------------------------------------------
constexpr int kStatBlocks = 256;

// part[block][c] = sum over the block's rows of x, or of (x - mean)^2
__global__ __launch_bounds__(256) void k_col_sums(const float *__restrict__ X, int64_t rows,
                                                  const double *__restrict__ mean,
                                                  double *__restrict__ part) {
  __shared__ double sh[16][kF];
  const int c = threadIdx.x & (kF - 1), r0 = threadIdx.x / kF;
  const double m = mean ? mean[c] : 0.0;
  double s = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * 16 + r0; i < rows; i += (int64_t)gridDim.x * 16) {
    const double d = (double)X[i * kF + c] - m;
    s += mean ? d * d : d;
  }
  sh[r0][c] = s;
  __syncthreads();
  if (threadIdx.x < kF) {
    double a = 0.0;
    for (int j = 0; j < 16; ++j) a += sh[j][c];
    part[blockIdx.x * kF + c] = a;
  }
}

// mean[c], or (spread) the float mean and 1 / standard deviation: 16 threads
// per column add the workgroups' sums
__global__ __launch_bounds__(256) void k_col_stats(const double *__restrict__ part,
                                                   int32_t blocks, int64_t rows,
                                                   double *__restrict__ mean, bool spread,
                                                   float *__restrict__ mean_f,
                                                   float *__restrict__ inv_f) {
  __shared__ double sh[16][kF];
  const int c = threadIdx.x & (kF - 1), j = threadIdx.x / kF;
  double s = 0.0;
  for (int32_t b = j; b < blocks; b += 16) s += part[b * kF + c];
  sh[j][c] = s;
  __syncthreads();
  if (j > 0) return;
  for (int q = 1; q < 16; ++q) s += sh[q][c];
  s /= (double)rows;
  if (!spread) {
    mean[c] = s;
    return;
  }
  const double sd = sqrt(s);
  mean_f[c] = (float)mean[c];
  inv_f[c] = (float)(sd > 1e-6 ? 1.0 / sd : 1.0);
}

__global__ __launch_bounds__(256) void k_standardise(float *__restrict__ X, int64_t count,
                                                     const float *__restrict__ mean,
                                                     const float *__restrict__ inv) {
  for (int64_t i = blockIdx.x * 256ll + threadIdx.x; i < count; i += (int64_t)gridDim.x * 256) {
    const int c = (int)(i & (kF - 1));
    X[i] = (X[i] - mean[c]) * inv[c];
  }
}

// Re-pack the BF16 B-operand blocks from the FP32 masters.
__global__ void k_pack(const float *__restrict__ P, __bf16 *__restrict__ pack) {
  for (int idx = blockIdx.x * blockDim.x + threadIdx.x; idx < kPackBlocks * 64 * 8;
       idx += gridDim.x * blockDim.x) {
    const int block = idx / 512, lane = (idx / 8) % 64, j = idx % 8;
    const int kin = (lane >> 5) * 8 + j, n = lane & 31;
    float v = 0.f;
    if (block < kPackW2) {  // W1: kb 0, nb = block
      v = P[kOffW1 + kin * kH + block * 32 + n];
    } else if (block < kPackW3) {  // W2: (kb, nb)
      const int b = block - kPackW2, kb = b / 2, nb = b % 2;
      v = P[kOffW2 + (kb * 16 + kin) * kH + nb * 32 + n];
    } else if (block < kPackW2T) {  // w3 as column 0
      const int kb = block - kPackW3;
      v = n == 0 ? P[kOffW3 + kb * 16 + kin] : 0.f;
    } else {  // W2^T: B[k][n] = W2[n][k]
      const int b = block - kPackW2T, kb = b / 2, nb = b % 2;
      v = P[kOffW2 + (nb * 32 + n) * kH + kb * 16 + kin];
    }
    pack[idx] = (__bf16)v;
  }
}

hipError_t launch_mlp_pack(const float *P, __bf16 *pack, hipStream_t st) {
  hipLaunchKernelGGL(k_pack, dim3(22), dim3(512), 0, st, P, pack);
  return hipGetLastError();
}

hipError_t launch_mlp_forward(const float *X, int64_t rows, const float *P, const __bf16 *pack,
                              float *y, hipStream_t st) {
  if (rows <= 0) return hipSuccess;
  const int64_t tiles = (rows + 31) / 32;
  const unsigned blocks = (unsigned)std::min<int64_t>((tiles + 3) / 4, 1 << 16);
  hipLaunchKernelGGL(k_mlp_forward, dim3(blocks), dim3(256), 0, st, X, rows, P, pack, y);
  return hipGetLastError();
}

// partial gradients of the mean squared error over perm[b0 .. b0+nrows) in
// `slots` tile slots; part has room for as many
hipError_t launch_mlp_partials(const float *X, const float *Yt, const int32_t *perm, int64_t b0,
                               int64_t nrows, const float *P, const __bf16 *pack, float *part,
                               float *part_loss, int32_t slots, hipStream_t st) {
  hipLaunchKernelGGL(k_mlp_grad, dim3(slots), dim3(128), 0, st, X, Yt, perm, b0, nrows, P, pack,
                     part, part_loss);
  return hipGetLastError();
}

// the gradient and the sum of squared errors from the partials
hipError_t launch_grad_reduce(const float *part, const float *part_loss, int32_t slots,
                              float *grad, float *loss, hipStream_t st) {
  hipLaunchKernelGGL(k_grad_reduce, dim3(kParams / 64 + 1), dim3(256), 0, st, part, part_loss,
                     slots, grad, loss);
  return hipGetLastError();
}

// one optimiser step from the partials: P, M, V and the packed weights
hipError_t launch_grad_step(const float *part, int32_t slots, float *P, float *M, float *V,
                            __bf16 *pack, float lr, float b1, float b2, float eps, float wd,
                            int32_t t, hipStream_t st) {
  hipLaunchKernelGGL(k_grad_step, dim3((kParams + 63) / 64), dim3(256), 0, st, part, slots, P, M,
                     V, pack, lr, b1, b2, eps, wd, t);
  return hipGetLastError();
}

// X (rows x 16, device) standardised in place; mean / inv: 16 floats each.
// scratch: standardise_scratch() doubles.
int64_t standardise_scratch() { return (int64_t)kStatBlocks * kF + kF; }
hipError_t launch_standardise(float *X, int64_t rows, double *scratch, float *mean, float *inv,
                              hipStream_t st) {
  const int32_t blocks = (int32_t)std::min<int64_t>(kStatBlocks, (rows + 15) / 16);
  double *m = scratch + (int64_t)kStatBlocks * kF;
  hipLaunchKernelGGL(k_col_sums, dim3(blocks), dim3(256), 0, st, X, rows, nullptr, scratch);
  hipLaunchKernelGGL(k_col_stats, dim3(1), dim3(256), 0, st, scratch, blocks, rows, m, false,
                     nullptr, nullptr);
  hipLaunchKernelGGL(k_col_sums, dim3(blocks), dim3(256), 0, st, X, rows, m, scratch);
  hipLaunchKernelGGL(k_col_stats, dim3(1), dim3(256), 0, st, scratch, blocks, rows, m, true, mean,
                     inv);
  hipLaunchKernelGGL(k_standardise,
                     dim3((unsigned)std::min<int64_t>((rows * kF + 255) / 256, 8192)), dim3(256),
                     0, st, X, rows * kF, mean, inv);
  return hipGetLastError();
}

int32_t mlp_param_count() { return kParams; }
int32_t mlp_pack_count() { return kPackBlocks * 64 * 8; }

}  // namespace efi
