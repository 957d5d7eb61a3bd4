// Stage-2 sampler, double elision (max_order 5), step by step over all samples.
//
// The method is gbs_sampler.hip's (App. C.1: Eqs. probade, probpartialade,
// probelidedade, probdoubleelidedade); this file evaluates it with the sums
// taken apart so that everything that depends on a sample only through the
// marginals of one top is done once, when that top is complete, for all later
// bits, as matrix products over the samples.  Write bits 1..M, chi_i =
// (-1)^x_i, q_i = chi_i p+(x_{n-1}..x_{i+1}) at step n, and
//     U(a; b, c) = chi_b chi_c p2(a - 1; b, c),  c < b < a,
// the two-elided marginal below bit a with the signs of its elided bits.  Then
//   p(x_n..x_1) = p(n-1)/2 + chi_n D_n,
//   D_n = kappa_n p(n-1)/2 + sum_i kappa_in chi_i p1(n-1, i)/4 + D3(n)/8
//       + sum_i q_i (Z4(n, i)/16 + ZR(n, i)/32),
//   D3(n)    = sum_{k>l} kappa_{kln}  U(n; k, l)
//   Z4(n, a) = sum_{k>l} kappa_{akln} U(a; k, l)
//   ZR(n, i) = sum_{j<i} [chi_j p+(x_{i-1}..x_{j+1})] Y(n, i, j)
//   Y(n, i, a) = sum_{k>l} kappa_{iakln} U(a; k, l)
// and the updates of the tables of top n (p1s(n, e) = chi_e p1(n, e)):
//   p+(x_n..x_l) = h p+(x_{n-1}..x_l) + chi_n sum_{j>=l} w_j p+(x_{j-1}..x_l),
//       w_j = kappa_jn q_j/4 + chi_j sum_{i>j} kappa_ijn q_i p+(x_{i-1}..x_{j+1})/8
//   p1s(n, e) = h p1s(n-1, e) + chi_n (B(n, n; e)/4
//             + (q_e Q(n, e) + sum_{a>e} q_a R(n, a; e))/8)
//   U(n+1; e, d) = h U(n; e, d) + chi_n (q_e B(n, e; d)
//                + sum_{e<i<n} kappa_in q_i U(i; e, d))/4
//   Q(n, a)    = sum_{k>l} kappa_{kln} U(a; k, l)
//   B(n, a; e) = sum_j kappa_jn  U(a; {j, e})
//   R(n, a; e) = sum_j kappa_ajn U(a; {j, e})
// with h = 1/2 + chi_n kappa_n/2.  Y, Z4, Q and D3 of a top a are one product
// (rows: every (n, i), inner index: the pairs (k, l), whose cumulants lie
// consecutively in the colex layout; columns: samples), B and R another; both
// run on the FP64 matrix units when bit a is reached.  What is left per bit is
// one pass over U (the last sum of the U update).
//
// Per sample the order-5 sum is C(M, 5) multiply-adds and reads C(M, 3) table
// entries once in all; the U update reads C(n - 1, 3) entries at step n, C(M, 4)
// in all, halved by taking two steps in a pass (update_kernel), and is bound by
// memory bandwidth (4.8 TB/s; a large copy reaches 4.6).
// M = 100, 4,096 samples: 44.6 ms (21 of them U updates, 17 products over pairs,
// 7 products over j) against 1,090 ms of one workgroup per 64 samples, which
// reads every U entry several times per bit.
//
// Storage: per block of 64 samples one contiguous block, entry-major, the 64
// samples of an entry consecutive, so every access of a wavefront is 512
// contiguous bytes and the 16 x 64 operand chunks of the products are 8 KB
// pieces.  B(n, e; d) waits in the slot of U(n+1; e, d) until step n replaces
// it, R(n, a; e) takes the slot of Y(n, a, e), which step a has used up.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "gbs_internal.h"
#include "gbs_sampler.h"
#include "gbs_sampler_product.h"

namespace gbs {

namespace {

// Entries of one sample's storage (each kSB doubles in a block).
struct Store {
  uint32_t U, Y;                  // tri(a, b, c)
  uint32_t Z4, ZR, Q, PP;         // pair (n, a); PP(b, a) at b(b-1)/2 + a - 1
  uint32_t P1[2], q[2];           // by parity of the top / of the step
  uint32_t w, chi, Bn, D3, P0, h; // P0: p of the last two tops
  uint32_t total;
  __host__ __device__ static Store make(int M) {
    Store s;
    const uint32_t m = (uint32_t)M, t3 = samp_c3(m) + 1, t2 = samp_c2(m + 1) + 1;
    uint32_t o = 0;
    s.U = o; o += t3;
    s.Y = o; o += t3;
    s.Z4 = o; o += t2;
    s.ZR = o; o += t2;
    s.Q = o; o += t2;
    s.PP = o; o += t2;
    for (int b = 0; b < 2; ++b) { s.P1[b] = o; o += m + 2; }
    for (int b = 0; b < 2; ++b) { s.q[b] = o; o += m + 2; }
    s.w = o; o += m + 2;
    s.chi = o; o += m + 2;
    s.Bn = o; o += m + 2;
    s.D3 = o; o += 1;
    s.P0 = o; o += 2;
    s.h = o; o += 1;
    s.total = o;
    return s;
  }
};

// U and Y index of (a; b, c), 1 <= c < b < a
__device__ __forceinline__ uint32_t tri(int a, int b, int c) {
  return samp_r3(a) + samp_r2(b) + (uint32_t)c - 1;
}
// index of the pair (n, a), 1 <= a < n
__device__ __forceinline__ uint32_t pair(int n, int a) { return samp_r2(n) + (uint32_t)a - 1; }

// v with C(v, 2) <= t < C(v + 1, 2)
__device__ __forceinline__ uint32_t tri_root(uint32_t t) {
  uint32_t v = (uint32_t)((1.0f + sqrtf(1.0f + 8.0f * (float)t)) * 0.5f);
  while (samp_c2(v) > t) --v;
  while (samp_c2(v + 1) <= t) ++v;
  return v;
}

struct StepArgs {
  const double* kap;
  KapOffsets ko;
  double* tab;
  Store st;
  int M, n;
};

__device__ __forceinline__ double* block_of(const StepArgs& A, uint32_t sb) {
  return A.tab + (uint64_t)sb * A.st.total * kSB;
}

// One row of a product: where its cumulants start and where its result goes.
struct Row {
  uint32_t kap, dest;
};

// Rows of the product with U(n; k, l): D3(n); Q(n', n); Z4(n', n); Y(n', i, n),
// n < i < n' <= M.
__device__ __forceinline__ Row pair_row(const StepArgs& A, int r) {
  const int n = A.n, m = A.M - n;
  const uint32_t o3 = A.ko.off[3], o4 = A.ko.off[4], o5 = A.ko.off[5];
  if (r == 0) return {o3 + samp_r3(n), A.st.D3};
  if (r <= m) return {o3 + samp_r3(n + r), A.st.Q + pair(n + r, n)};
  r -= m;
  if (r <= m) return {o4 + samp_r4(n + r) + samp_r3(n), A.st.Z4 + pair(n + r, n)};
  const uint32_t t = (uint32_t)(r - m - 1), v = tri_root(t);
  const int np = n + 1 + (int)v, i = n + 1 + (int)(t - samp_c2(v));
  return {o5 + samp_r5(np) + samp_r4(i) + samp_r3(n), A.st.Y + tri(np, i, n)};
}

// Rows of the product with U(n; {j, e}) over j: B(n', n; e) for n' = n..M-1
// (n' = n into its own row, the others into the slots of U(n'+1; n, e)) and
// R(n', n; e) for n' = n+1..M-1.
__device__ __forceinline__ Row single_row(const StepArgs& A, int r, int e) {
  const int n = A.n, m = A.M - n;
  if (r < m) {
    const int np = n + r;
    return {A.ko.off[2] + samp_r2(np), r == 0 ? A.st.Bn + (uint32_t)e : A.st.U + tri(np + 1, n, e)};
  }
  const int np = n + 1 + r - m;
  return {A.ko.off[3] + samp_r3(np) + samp_r2(n), A.st.Y + tri(np, n, e)};
}

// ---- the sums of step n that are not products, one wave per item ----

// w_j (j < n) and ZR(n', n) (n' > n): they need only p+ of top n - 1.
__device__ __forceinline__ void reduce_item(const StepArgs& A, uint32_t item, uint32_t nsb, int lane) {
  const int n = A.n;
  const uint32_t per = (uint32_t)(A.M - 1);  // n - 1 of w, M - n of ZR
  if (item >= per * nsb) return;
  const int it = (int)(item % per);
  double* blk = block_of(A, item / per) + lane;
  const double* q = blk + (uint64_t)A.st.q[n & 1] * kSB;
  if (it < n - 1) {
    const int j = it + 1;
    const double* k3 = A.kap + A.ko.off[3] + samp_r3(n) + (uint32_t)j - 1;
    const double* pp = blk + (uint64_t)(A.st.PP + (uint32_t)j) * kSB;  // p+(i-1, j+1) at C(i-1, 2) + j
    double s = 0.0;
    if (j + 1 < n) s = k3[samp_r2(j + 1)] * q[(uint64_t)(j + 1) * kSB];
#pragma unroll 4
    for (int i = j + 2; i < n; ++i)
      s = fma(k3[samp_r2(i)] * q[(uint64_t)i * kSB], pp[(uint64_t)samp_r2(i) * kSB], s);
    const double k2 = A.kap[A.ko.off[2] + samp_r2(n) + (uint32_t)j - 1];
    const double chij = blk[(uint64_t)(A.st.chi + (uint32_t)j) * kSB];
    blk[(uint64_t)(A.st.w + (uint32_t)j) * kSB] = fma(0.25 * k2, q[(uint64_t)j * kSB], 0.125 * chij * s);
  } else {
    const int np = it + 2;  // n + 1 .. M
    const double* Y = blk + (uint64_t)(A.st.Y + samp_r3(np) + samp_r2(n)) * kSB;
    double s = 0.0;
#pragma unroll 8
    for (int j = 3; j < n; ++j) s = fma(q[(uint64_t)j * kSB], Y[(uint64_t)(j - 1) * kSB], s);
    blk[(uint64_t)(A.st.ZR + pair(np, n)) * kSB] = s;
  }
}

// p+(x_n..x_l), l = 1..n, and from it q of step n + 1 (once bit n is known).
__device__ __forceinline__ void partial_item(const StepArgs& A, uint32_t item, uint32_t nsb, int lane) {
  const int n = A.n;
  if (item >= (uint32_t)n * nsb) return;
  const int l = 1 + (int)(item % (uint32_t)n);
  double* blk = block_of(A, item / (uint32_t)n) + lane;
  double v = blk[(uint64_t)A.st.h * kSB];
  if (l < n) {
    const double* wj = blk + (uint64_t)A.st.w * kSB;
    const double* pp = blk + (uint64_t)(A.st.PP + (uint32_t)l - 1) * kSB;  // p+(j-1, l) at C(j-1, 2) + l - 1
    double s = wj[(uint64_t)l * kSB];
#pragma unroll 8
    for (int j = l + 1; j < n; ++j) s = fma(wj[(uint64_t)j * kSB], pp[(uint64_t)samp_r2(j) * kSB], s);
    v = fma(blk[(uint64_t)(A.st.chi + (uint32_t)n) * kSB], s, v * pp[(uint64_t)samp_r2(n) * kSB]);
  }
  blk[(uint64_t)(A.st.PP + samp_r2(n + 1) + (uint32_t)l - 1) * kSB] = v;
  if (l >= 2)
    blk[(uint64_t)(A.st.q[(n + 1) & 1] + (uint32_t)l - 1) * kSB] =
        blk[(uint64_t)(A.st.chi + (uint32_t)l - 1) * kSB] * v;
}

// A product of step n, 64 rows x 64 samples per workgroup (gbs_sampler_product.h).
// SINGLE: the product over j at fixed e, else the product over pairs.
// Workgroups past the product's carry the sums that are independent of it: w
// and ZR beside the product over pairs, p+ beside the product over j.
template <bool SINGLE, int KS>
__global__ __launch_bounds__(256 * KS) void product_kernel(StepArgs A, int rows, int row_blocks,
                                                           uint32_t nprod, uint32_t nsb) {
  __shared__ double Bs[2][KS][kKC][kLdB];
  if (blockIdx.x >= nprod) {
    const uint32_t item = (blockIdx.x - nprod) * (4 * KS) + (threadIdx.x >> 6);
    if constexpr (SINGLE) partial_item(A, item, nsb, threadIdx.x & 63);
    else reduce_item(A, item, nsb, threadIdx.x & 63);
    return;
  }
  const int n = A.n, rb = (int)(blockIdx.x % (uint32_t)row_blocks);
  uint32_t sb = blockIdx.x / (uint32_t)row_blocks;
  if constexpr (SINGLE) {
    const int e = 1 + (int)(sb % (uint32_t)(n - 1));
    double* blk = block_of(A, sb / (uint32_t)(n - 1));
    const double* V = blk + (uint64_t)(A.st.U + samp_r3(n)) * kSB;
    product_block<KS>(
        rb, rows, n - 1, [&](int r) { return A.kap + single_row(A, r, e).kap; },
        [&](int k) -> const double* {
          const int j = k + 1;
          return j == e ? nullptr : V + (uint64_t)(samp_r2(max(j, e)) + (uint32_t)min(j, e) - 1) * kSB;
        },
        [&](int r) { return blk + (uint64_t)single_row(A, r, e).dest * kSB; }, Bs);
  } else {
    double* blk = block_of(A, sb);
    const double* V = blk + (uint64_t)(A.st.U + samp_r3(n)) * kSB;
    product_block<KS>(
        rb, rows, (int)samp_r2(n), [&](int r) { return A.kap + pair_row(A, r).kap; },
        [&](int k) { return V + (uint64_t)k * kSB; },
        [&](int r) { return blk + (uint64_t)pair_row(A, r).dest * kSB; }, Bs);
  }
}

// The product over pairs for few rows (late bits: few (n', i) left, long inner
// index): 16 rows x 64 samples per workgroup, the chunks of the inner index
// dealt to the waves, whose partial tiles are added in wave order.
constexpr int kSlimWaves = 8;
constexpr uint32_t kSlimRows = 128;
__global__ __launch_bounds__(64 * kSlimWaves) void product_slim_kernel(StepArgs A, int rows, int row_blocks,
                                                                       uint32_t nprod, uint32_t nsb) {
  __shared__ double part[kSlimWaves][16][kSB];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (blockIdx.x >= nprod) {
    reduce_item(A, (blockIdx.x - nprod) * kSlimWaves + (uint32_t)w, nsb, lane);
    return;
  }
  const int g = lane >> 4, c16 = lane & 15;
  const int rb = (int)(blockIdx.x % (uint32_t)row_blocks);
  const uint32_t sb = blockIdx.x / (uint32_t)row_blocks;
  const int L = (int)samp_r2(A.n);
  double* blk = block_of(A, sb);
  const double* V = blk + (uint64_t)(A.st.U + samp_r3(A.n)) * kSB;
  const int r0 = rb * 16;
  const double* ka = A.kap + pair_row(A, min(r0 + c16, rows - 1)).kap;
  double4 acc[4] = {};
  const int nch = (L + kKC - 1) / kKC;
  for (int c = w; c < nch; c += kSlimWaves) {
    const int k = c * kKC + 4 * g;
    double a[4], b[4][4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const bool in = k + t < L;
      a[t] = in ? ka[k + t] : 0.0;
      const double* p = V + (uint64_t)(in ? k + t : 0) * kSB + c16;
#pragma unroll
      for (int ct = 0; ct < 4; ++ct) b[t][ct] = in ? p[ct * 16] : 0.0;
    }
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int ct = 0; ct < 4; ++ct)
        acc[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t], b[t][ct], acc[ct], 0, 0, 0);
  }
#pragma unroll
  for (int v = 0; v < 4; ++v)
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) part[w][g + 4 * v][ct * 16 + c16] = acc[ct][v];
  __syncthreads();
  for (int rr = w; rr < 16; rr += kSlimWaves) {
    if (r0 + rr >= rows) continue;
    double s = 0.0;
#pragma unroll
    for (int v = 0; v < kSlimWaves; ++v) s += part[v][rr][lane];
    blk[(uint64_t)pair_row(A, r0 + rr).dest * kSB + lane] = s;
  }
}

// D_n, the bit and p(n): one workgroup per sample block.
__global__ __launch_bounds__(256) void bit_kernel(StepArgs A, const double* __restrict__ u, uint64_t ldu,
                                                  int64_t nsamp, uint8_t* __restrict__ bits_out,
                                                  double* __restrict__ prob, double* __restrict__ cond) {
  __shared__ double red[4][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int n = A.n;
  double* blk = block_of(A, blockIdx.x) + lane;
  const double* q = blk + (uint64_t)A.st.q[n & 1] * kSB;
  const double* p1 = blk + (uint64_t)A.st.P1[(n - 1) & 1] * kSB;
  const double* k2 = A.kap + A.ko.off[2] + samp_r2(n) - 1;
  const double* z4 = blk + (uint64_t)(A.st.Z4 + samp_r2(n) - 1) * kSB;
  const double* zr = blk + (uint64_t)(A.st.ZR + samp_r2(n) - 1) * kSB;
  const double pprev = n == 1 ? 1.0 : blk[(uint64_t)(A.st.P0 + ((uint32_t)(n - 1) & 1)) * kSB];
  double D2 = 0.0, D45 = 0.0;
#pragma unroll 4
  for (int i = 1 + w; i < n; i += 4) {
    D2 = fma(k2[i], p1[(uint64_t)i * kSB], D2);
    if (i >= 3) {
      const double z = fma(0.5, i >= 4 ? zr[(uint64_t)i * kSB] : 0.0, z4[(uint64_t)i * kSB]);
      D45 = fma(q[(uint64_t)i * kSB], z, D45);
    }
  }
  red[w][lane] = fma(0.25, D2, 0.0625 * D45);
  __syncthreads();
  if (w != 0) return;
  const double k1 = A.kap[A.ko.off[1] + (uint32_t)n - 1];
  double D = 0.5 * k1 * pprev;
  if (n >= 3) D = fma(0.125, blk[(uint64_t)A.st.D3 * kSB], D);
#pragma unroll
  for (int v = 0; v < 4; ++v) D += red[v][lane];
  const int64_t s = (int64_t)blockIdx.x * kSB + lane;
  const bool live = s < nsamp;
  const double cnd = pprev > 0.0 ? (0.5 * pprev - D) / pprev : 0.5;
  const double un = live ? u[(uint64_t)(n - 1) * ldu + (uint64_t)s] : 1.0;
  const uint32_t xn = un < cnd ? 1u : 0u;
  const double chi = xn ? -1.0 : 1.0;
  const double pn = fma(chi, D, 0.5 * pprev);
  blk[(uint64_t)(A.st.P0 + ((uint32_t)n & 1)) * kSB] = pn;
  blk[(uint64_t)(A.st.chi + (uint32_t)n) * kSB] = chi;
  blk[(uint64_t)A.st.h * kSB] = fma(0.5 * chi, k1, 0.5);
  blk[(uint64_t)(A.st.q[(n + 1) & 1] + (uint32_t)n) * kSB] = chi;               // p+ of no bits is 1
  blk[(uint64_t)(A.st.P1[n & 1] + (uint32_t)n) * kSB] = chi * pprev;            // p1(n, n) = p(n - 1)
  if (live) {
    bits_out[s * A.M + (n - 1)] = (uint8_t)xn;
    if (cond) cond[(uint64_t)(n - 1) * ldu + (uint64_t)s] = cnd;
    if (prob && n == A.M) prob[s] = pn;
  }
}

// Tables of top n (n < M) after p+ of top n: one wave per item, kRun
// consecutive pairs (e, d) of the U update or one entry of p1.
// The sum over i < n that the U update of step n + 1 needs has q of step n + 1
// for its weights, and those depend on bit n but not on U(n + 1).  So every
// other step (FULL) takes the sums of both steps in one pass over U(i; e, d),
// i < n, leaving step n + 1's (with its q_e B) in the slot of U(n+2; e, d), and
// the step after it only adds its one new term: half the passes over U.
constexpr int kRun = 8;
template <bool FULL>
__global__ __launch_bounds__(256) void update_kernel(StepArgs A, uint32_t nsb, uint32_t nruns) {
  const int lane = threadIdx.x & 63;
  const int n = A.n;
  const uint32_t per = nruns + (uint32_t)(n - 1);
  const uint32_t item = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (item >= per * nsb) return;
  const uint32_t it = item / nsb;  // the longest sums first
  double* blk = block_of(A, item % nsb) + lane;
  const double* q = blk + (uint64_t)A.st.q[n & 1] * kSB;
  const double chi = blk[(uint64_t)(A.st.chi + (uint32_t)n) * kSB];
  const double h = blk[(uint64_t)A.st.h * kSB];
  double* U = blk + (uint64_t)A.st.U * kSB;
  if (it < nruns) {
    const double* k2 = A.kap + A.ko.off[2] + samp_r2(n) - 1;
    const uint32_t p0 = it * kRun, np = samp_r2(n);
    int e[kRun];
    {
      uint32_t v = tri_root(p0);  // p = C(e-1, 2) + d - 1, so e = v + 1
      uint32_t end = samp_c2(v + 1);
#pragma unroll
      for (int r = 0; r < kRun; ++r) {
        if (p0 + r >= end) {
          ++v;
          end = samp_c2(v + 1);
        }
        e[r] = (int)v + 1;
      }
    }
    const double* un = U + (uint64_t)(samp_r3(n) + p0) * kSB;
    double* uo = U + (uint64_t)(samp_r3(n + 1) + p0) * kSB;
    if constexpr (FULL) {
      const double* qn = blk + (uint64_t)A.st.q[(n + 1) & 1] * kSB;
      const double* k2n = A.kap + A.ko.off[2] + samp_r2(n + 1) - 1;
      double acc[kRun] = {}, nxt[kRun] = {};
      int i = e[0] + 1;
      // bits i not above every e of the run: entries past C(i-1, 2) are not of top i
      for (; i <= e[kRun - 1] && i < n; ++i) {
        const double c = k2[i] * q[(uint64_t)i * kSB], cn = k2n[i] * qn[(uint64_t)i * kSB];
        const double* p = U + (uint64_t)(samp_r3(i) + p0) * kSB;
#pragma unroll
        for (int r = 0; r < kRun; ++r)
          if (e[r] < i) {
            const double x = p[r * kSB];
            acc[r] = fma(c, x, acc[r]);
            nxt[r] = fma(cn, x, nxt[r]);
          }
      }
#pragma unroll 2
      for (; i < n; ++i) {
        const double c = k2[i] * q[(uint64_t)i * kSB], cn = k2n[i] * qn[(uint64_t)i * kSB];
        const double* p = U + (uint64_t)(samp_r3(i) + p0) * kSB;
#pragma unroll
        for (int r = 0; r < kRun; ++r) {
          const double x = p[r * kSB];
          acc[r] = fma(c, x, acc[r]);
          nxt[r] = fma(cn, x, nxt[r]);
        }
      }
      double* us = U + (uint64_t)(samp_r3(n + 2) + p0) * kSB;
#pragma unroll
      for (int r = 0; r < kRun; ++r) {
        if (p0 + r >= np) break;
        const double s = fma(q[(uint64_t)e[r] * kSB], uo[r * kSB], acc[r]);
        uo[r * kSB] = fma(0.25 * chi, s, h * un[r * kSB]);
        us[r * kSB] = fma(qn[(uint64_t)e[r] * kSB], us[r * kSB], nxt[r]);
      }
    } else {
      const double* ul = U + (uint64_t)(samp_r3(n - 1) + p0) * kSB;
      const double ql = q[(uint64_t)(n - 1) * kSB], c = k2[n - 1] * ql;
#pragma unroll
      for (int r = 0; r < kRun; ++r) {
        if (p0 + r >= np) break;
        const double s = e[r] < n - 1 ? fma(c, ul[r * kSB], uo[r * kSB]) : ql * uo[r * kSB];
        uo[r * kSB] = fma(0.25 * chi, s, h * un[r * kSB]);
      }
    }
  } else {
    const int e = 1 + (int)(it - nruns);
    double s = e >= 3 ? q[(uint64_t)e * kSB] * blk[(uint64_t)(A.st.Q + pair(n, e)) * kSB] : 0.0;
    const double* R = blk + (uint64_t)(A.st.Y + samp_r3(n) + (uint32_t)e - 1) * kSB;
#pragma unroll 8
    for (int a = e + 1; a < n; ++a) s = fma(q[(uint64_t)a * kSB], R[(uint64_t)samp_r2(a) * kSB], s);
    const double b = blk[(uint64_t)(A.st.Bn + (uint32_t)e) * kSB];
    const double old = blk[(uint64_t)(A.st.P1[(n - 1) & 1] + (uint32_t)e) * kSB];
    blk[(uint64_t)(A.st.P1[n & 1] + (uint32_t)e) * kSB] = fma(chi, fma(0.25, b, 0.125 * s), h * old);
    U[(uint64_t)tri(n + 1, n, e) * kSB] = chi * old;  // p2(n, n, e) = p1(n - 1, e)
  }
}

// The product over pairs with KS workgroup parts, and the step's other sums.
template <int KS>
void launch_pairs(const StepArgs& A, uint32_t rows, uint32_t nsb, hipStream_t s) {
  const uint32_t rb = (rows + 63) / 64, per = 4 * KS;
  const uint32_t extra = ((uint32_t)(A.M - 1) * nsb + per - 1) / per;
  hipLaunchKernelGGL((product_kernel<false, KS>), dim3(rb * nsb + extra), dim3(256 * KS), 0, s, A, (int)rows,
                     (int)rb, rb * nsb, nsb);
}

}  // namespace

size_t double_sampler_bytes(int M) { return (size_t)Store::make(M).total * sizeof(double); }

hipError_t launch_double_sampler(int M, const double* kap, KapOffsets ko, int64_t nsamp, const double* u,
                                 uint64_t ldu, double* tab, uint8_t* bits, double* prob, double* cond,
                                 hipStream_t s) {
  const uint32_t nsb = (uint32_t)((nsamp + kSB - 1) / kSB);
  StepArgs A{kap, ko, tab, Store::make(M), M, 0};
  hipError_t e = hipSuccess;
  for (int n = 1; n <= M && e == hipSuccess; ++n) {
    A.n = n;
    const uint32_t m = (uint32_t)(M - n);
    {
      // Which kernel and how the inner index is split follow from the rows alone,
      // so that a sample's sums do not depend on the batch it is in.  Two parts
      // per tile: 47.2 ms at M = 100, 4,096 samples and 8.3 ms at M = 90, 200,
      // against 48.4 and 9.6 ms in one part, 50.1 and 8.0 ms in four.  Up to
      // kSlimRows rows the slim kernel: two 64-row tiles a block of samples leave
      // units idle, each with a long serial inner index.  Slim up to 16 / 64 / 128 /
      // 256 rows: 7.8 / 7.4 / 7.0 / 6.6 ms at M = 90, 200 samples; 100.1 / 99.3 /
      // 98.4 / 98.2 at M = 144, 2,048; 44.8 / 44.4 / 44.5 / 44.9 at M = 100, 4,096: more
      // than 128 gain with few samples and lose with many, and the rule must not go
      // by the samples.
      const uint32_t rows = n >= 3 ? 1 + 2 * m + samp_c2(m) : 0;
      if (rows <= kSlimRows) {
        const uint32_t rb = (rows + 15) / 16;
        const uint32_t extra = ((uint32_t)(M - 1) * nsb + kSlimWaves - 1) / kSlimWaves;
        hipLaunchKernelGGL(product_slim_kernel, dim3(rb * nsb + extra), dim3(64 * kSlimWaves), 0, s, A, (int)rows,
                           (int)rb, rb * nsb, nsb);
      } else {
        launch_pairs<2>(A, rows, nsb, s);
      }
    }
    hipLaunchKernelGGL(bit_kernel, dim3(nsb), dim3(256), 0, s, A, u, ldu, nsamp, bits, prob, cond);
    if (n < M) {
      const uint32_t rows = n >= 2 ? 2 * m - 1 : 0, rb = (rows + 63) / 64;
      const uint32_t nprod = rb * (uint32_t)(n - 1) * nsb, extra = ((uint32_t)n * nsb + 3) / 4;
      hipLaunchKernelGGL((product_kernel<true, 1>), dim3(nprod + extra), dim3(256), 0, s, A, (int)rows, (int)rb,
                         nprod, nsb);
      const uint32_t nruns = (samp_c2((uint32_t)n - 1) + kRun - 1) / kRun;
      const uint64_t items = (uint64_t)(nruns + (uint32_t)n - 1) * nsb;
      if (items) {
        if (((M - n) & 1) == 0)
          hipLaunchKernelGGL(update_kernel<true>, dim3((unsigned)((items + 3) / 4)), dim3(256), 0, s, A, nsb, nruns);
        else
          hipLaunchKernelGGL(update_kernel<false>, dim3((unsigned)((items + 3) / 4)), dim3(256), 0, s, A, nsb, nruns);
      }
    }
    e = hipGetLastError();
  }
  return e;
}

}  // namespace gbs
