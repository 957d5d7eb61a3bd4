// Stage-2 sampler, single elision (max_order 3), step by step over all samples.
//
// The method is gbs_sampler.hip's (Methods: Eqs. methprob, b, a), with the sums
// taken apart as in gbs_sampler_double.hip.  Bits 1..M, chi_i = (-1)^x_i,
// q_i = chi_i p+(x_{n-1}..x_{i+1}) at step n, h = 1/2 + chi_n kappa_n/2 and
//     V(a; b) = chi_b p1(a - 1; b),  b < a:
//   p(x_n..x_1) = p(n-1)/2 + chi_n D_n,
//   D_n = kappa_n p(n-1)/2 + sum_i kappa_in V(n; i)/4 + sum_i q_i Z3(n, i)/8
//   p+(x_n..x_l) = h p+(x_{n-1}..x_l) + chi_n sum_{j>=l} kappa_jn q_j p+(x_{j-1}..x_l)/4
//   V(n+1; e) = h V(n; e) + chi_n (q_e B(n, e) + sum_{e<i<n} kappa_in q_i V(i; e))/4
//   Z3(n, a) = sum_j kappa_ajn V(a; j),   B(n, a) = sum_j kappa_jn V(a; j)
// Z3 and B of a top a, for all later bits n, are one matrix product (rows: n,
// inner index: j, columns: samples) on the FP64 matrix units when bit a is
// reached.  What is left per bit reads the tables p+ and V once each: C(n, 2)
// entries each at step n, bound by memory bandwidth.  The sum of the V update of
// step n + 1 over i < n needs only q of step n + 1, which is known after bit n and
// p+ of top n, so every other step takes the V sums of two steps in one pass.
// M = 144, 65,536 samples: 96.3 ms, 7.5 MB of memory traffic per sample by the counters
// (7.1 read) at 5.1 TB/s, against 325 ms of one workgroup per 64 samples that read
// 20 MB per sample.
//
// Storage as in gbs_sampler_double.hip: blocks of 64 samples, entry-major.
// B(n, e) waits in the slot of V(n+1; e); Z3(n, a) in that of p+(x_n..x_a).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "gbs_internal.h"
#include "gbs_sampler.h"
#include "gbs_sampler_product.h"

namespace gbs {

namespace {

// Entries of one sample's storage (each kSB doubles in a block).
struct Store {
  uint32_t V;            // V(a; b) at C(a-1, 2) + b - 1
  uint32_t PP;           // p+(b, a) at b(b-1)/2 + a - 1
  uint32_t q[2];         // by parity of the step
  uint32_t chi, P0, h;   // P0: p of the last two tops
  uint32_t total;
  __host__ __device__ static Store make(int M) {
    Store s;
    const uint32_t m = (uint32_t)M, t2 = samp_c2(m + 1) + 1;
    uint32_t o = 0;
    s.V = o; o += t2;
    s.PP = o; o += t2;
    for (int b = 0; b < 2; ++b) { s.q[b] = o; o += m + 2; }
    s.chi = o; o += m + 2;
    s.P0 = o; o += 2;
    s.h = o; o += 1;
    s.total = o;
    return s;
  }
};

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

// D_n, the bit and p(n): one workgroup per sample block.
__global__ __launch_bounds__(256) void bit_kernel(StepArgs A, const double* __restrict__ u, uint64_t ldu,
                                                  int64_t nsamp, uint8_t* __restrict__ bits_out,
                                                  double* __restrict__ prob, double* __restrict__ cond) {
  __shared__ double red[4][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int n = A.n;
  double* blk = block_of(A, blockIdx.x) + lane;
  const double* q = blk + (uint64_t)A.st.q[n & 1] * kSB;
  const double* k2 = A.kap + A.ko.off[2] + samp_r2(n) - 1;
  const double* v = blk + (uint64_t)(A.st.V + samp_r2(n)) * kSB;        // V(n; i) at i - 1
  const double* z3 = blk + (uint64_t)(A.st.PP + samp_r2(n + 1)) * kSB;  // Z3(n, i) at i - 1
  const double pprev = n == 1 ? 1.0 : blk[(uint64_t)(A.st.P0 + ((uint32_t)(n - 1) & 1)) * kSB];
  double D2 = 0.0, D3 = 0.0;
#pragma unroll 4
  for (int i = 1 + w; i < n; i += 4) {
    D2 = fma(k2[i], v[(uint64_t)(i - 1) * kSB], D2);
    if (i >= 2) D3 = fma(q[(uint64_t)i * kSB], z3[(uint64_t)(i - 1) * kSB], D3);
  }
  red[w][lane] = fma(0.25, D2, 0.125 * D3);
  __syncthreads();
  if (w != 0) return;
  const double k1 = A.kap[A.ko.off[1] + (uint32_t)n - 1];
  double D = 0.5 * k1 * pprev;
#pragma unroll
  for (int p = 0; p < 4; ++p) D += red[p][lane];
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
  blk[(uint64_t)(A.st.q[(n + 1) & 1] + (uint32_t)n) * kSB] = chi;  // p+ of no bits is 1
  if (n < A.M)
    blk[(uint64_t)(A.st.V + samp_r2(n + 1) + (uint32_t)n - 1) * kSB] = chi * pprev;  // p1(n, n) = p(n - 1)
  if (live) {
    bits_out[s * A.M + (n - 1)] = (uint8_t)xn;
    if (cond) cond[(uint64_t)(n - 1) * ldu + (uint64_t)s] = cnd;
    if (prob && n == A.M) prob[s] = pn;
  }
}

// Table passes: kRun consecutive entries (4 KB in one piece) of a top per workgroup;
// its four waves take every fourth term of the sums, which are added in wave order.
// With a wave per run the longest sum, n terms one after the other, is the time of a
// launch with few blocks of samples.  M = 144, a wave per run / split: 500 samples
// 9.6 / 3.5 ms, 10,000 21.8 / 16.3, 20,000 34.6 / 30.4; M = 60, 5,000 2.4 / 1.35.  One
// form for every call: a sample's sums, and so its bits, depend on its own column of
// uniforms alone, not on how many samples are drawn with it.
constexpr int kRun = 8, kParts = 4, kOwn = kRun / kParts;
constexpr int kSumWords = kParts * kRun * kSB;

// acc[t] = the sum over the workgroup's waves of entry w kOwn + t of the run.
__device__ __forceinline__ void sum_waves(double (&acc)[kRun], double* red, int w, int lane) {
#pragma unroll
  for (int r = 0; r < kRun; ++r) red[(w * kRun + r) * kSB + lane] = acc[r];
  __syncthreads();
#pragma unroll
  for (int t = 0; t < kOwn; ++t) {
    acc[t] = red[(w * kOwn + t) * kSB + lane];
#pragma unroll
    for (int v = 1; v < kParts; ++v) acc[t] += red[(v * kRun + w * kOwn + t) * kSB + lane];
  }
}

// Run and block of samples of a pass's item: one group of the sample blocks after the
// other, the longest sums first within a group.  The runs of a block are neighbours in
// memory; with every block of a large call between them, the split reads them far
// apart.  M = 144, one group / groups of about 64 / 128 / 256 / 512 / 1,024 blocks, ms:
// 262,144 samples 423 / 386 / 383 / 384 / 389 / 408, 65,536 102.1 / 97.9 / 96.5 / 96.3 /
// 97.4 / 102.1 (a wave per run: 417, 97.9); 20,000 samples (313 blocks) 30.4 in one
// group, 31.3 as 256 and 57: hence groups of equal size, the nearest to kGroup.
constexpr uint32_t kGroup = 256;
struct Item {
  uint32_t run, sb;
};
__device__ __forceinline__ Item item_of(uint32_t item, uint32_t runs, uint32_t nsb, uint32_t group) {
  const uint32_t first = item / (runs * group) * group, m = min(group, nsb - first);
  const uint32_t r = item - first * runs;
  return {r / m, first + r % m};
}

// The terms j = first, first + kParts, .. < n of p+(x_n..x_l), l = l0..l0 + kRun - 1.
__device__ __forceinline__ void partial_terms(const double* q, const double* k2, const double* PP, int l0, int first,
                                              int n, double (&acc)[kRun]) {
  int j = first;
  // p+(j-1, l) is 1 for l = j and has no term for l > j
  for (; j < l0 + kRun && j < n; j += kParts) {
    const double c = k2[j] * q[(uint64_t)j * kSB];
    const double* p = PP + (uint64_t)samp_r2(j) * kSB;
#pragma unroll
    for (int r = 0; r < kRun; ++r) {
      if (l0 + r < j) acc[r] = fma(c, p[r * kSB], acc[r]);
      else if (l0 + r == j) acc[r] += c;
    }
  }
#pragma unroll 2
  for (; j < n; j += kParts) {
    const double c = k2[j] * q[(uint64_t)j * kSB];
    const double* p = PP + (uint64_t)samp_r2(j) * kSB;
#pragma unroll
    for (int r = 0; r < kRun; ++r) acc[r] = fma(c, p[r * kSB], acc[r]);
  }
}

// p+(x_n..x_l), and from it q of step n + 1.
__global__ __launch_bounds__(256) void partial_kernel(StepArgs A, uint32_t nsb, uint32_t runs,
                                                     uint32_t group) {
  __shared__ double red[kSumWords];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int n = A.n;
  const Item it = item_of(blockIdx.x, runs, nsb, group);
  const int l0 = 1 + (int)it.run * kRun;
  double* blk = block_of(A, it.sb) + lane;
  const double* q = blk + (uint64_t)A.st.q[n & 1] * kSB;
  const double* k2 = A.kap + A.ko.off[2] + samp_r2(n) - 1;
  double* PP = blk + (uint64_t)(A.st.PP + (uint32_t)l0 - 1) * kSB;  // p+(j-1, l0 + r) at C(j-1, 2) + l0 - 1 + r
  const double chi = blk[(uint64_t)(A.st.chi + (uint32_t)n) * kSB];
  const double h = blk[(uint64_t)A.st.h * kSB];
  double acc[kRun] = {};
  partial_terms(q, k2, PP, l0, l0 + w, n, acc);
  sum_waves(acc, red, w, lane);
#pragma unroll
  for (int t = 0; t < kOwn; ++t) {
    const int r = w * kOwn + t, l = l0 + r;
    if (l > n) break;
    const double old = l < n ? PP[(uint64_t)(samp_r2(n) + (uint32_t)r) * kSB] : 1.0;
    const double v = fma(0.25 * chi, acc[t], h * old);
    PP[(uint64_t)(samp_r2(n + 1) + (uint32_t)r) * kSB] = v;
    if (l >= 2)
      blk[(uint64_t)(A.st.q[(n + 1) & 1] + (uint32_t)l - 1) * kSB] =
          blk[(uint64_t)(A.st.chi + (uint32_t)l - 1) * kSB] * v;
  }
}

// The terms i = first, first + kParts, .. < n of V(n+1; e) (acc) and V(n+2; e)
// (nxt), e = e0..e0 + kRun - 1.
__device__ __forceinline__ void update_terms(const double* q, const double* k2, const double* qn, const double* k2n,
                                             const double* V, int e0, int first, int n, double (&acc)[kRun],
                                             double (&nxt)[kRun]) {
  int i = first;
  for (; i < e0 + kRun && i < n; i += kParts) {
    const double c = k2[i] * q[(uint64_t)i * kSB], cn = k2n[i] * qn[(uint64_t)i * kSB];
    const double* p = V + (uint64_t)samp_r2(i) * kSB;
#pragma unroll
    for (int r = 0; r < kRun; ++r)
      if (e0 + r < i) {
        const double x = p[r * kSB];
        acc[r] = fma(c, x, acc[r]);
        nxt[r] = fma(cn, x, nxt[r]);
      }
  }
#pragma unroll 2
  for (; i < n; i += kParts) {
    const double c = k2[i] * q[(uint64_t)i * kSB], cn = k2n[i] * qn[(uint64_t)i * kSB];
    const double* p = V + (uint64_t)samp_r2(i) * kSB;
#pragma unroll
    for (int r = 0; r < kRun; ++r) {
      const double x = p[r * kSB];
      acc[r] = fma(c, x, acc[r]);
      nxt[r] = fma(cn, x, nxt[r]);
    }
  }
}

// V(n+1; e), e < n.  FULL takes the sums of steps n and n + 1 (see
// gbs_sampler_double.hip), a workgroup per run; the step after it adds one term,
// a wave per run.
template <bool FULL>
__device__ __forceinline__ void update_item(const StepArgs& A, uint32_t b, uint32_t nsb, uint32_t runs, uint32_t group, int lane,
                                            int w, double* red) {
  const int n = A.n;
  const uint32_t item = FULL ? b : b * 4 + (uint32_t)w;
  if (item >= runs * nsb) return;
  const Item it = item_of(item, runs, nsb, group);
  const int e0 = 1 + (int)it.run * kRun;
  double* blk = block_of(A, it.sb) + lane;
  const double* q = blk + (uint64_t)A.st.q[n & 1] * kSB;
  const double* k2 = A.kap + A.ko.off[2] + samp_r2(n) - 1;
  double* V = blk + (uint64_t)(A.st.V + (uint32_t)e0 - 1) * kSB;  // V(i; e0 + r) at C(i-1, 2) + e0 - 1 + r
  const double chi = blk[(uint64_t)(A.st.chi + (uint32_t)n) * kSB];
  const double h = blk[(uint64_t)A.st.h * kSB];
  const double* vn = V + (uint64_t)samp_r2(n) * kSB;
  double* vo = V + (uint64_t)samp_r2(n + 1) * kSB;
  if constexpr (FULL) {
    const double* qn = blk + (uint64_t)A.st.q[(n + 1) & 1] * kSB;
    const double* k2n = A.kap + A.ko.off[2] + samp_r2(n + 1) - 1;
    double acc[kRun] = {}, nxt[kRun] = {};
    update_terms(q, k2, qn, k2n, V, e0, e0 + 1 + w, n, acc, nxt);
    sum_waves(acc, red, w, lane);
    __syncthreads();  // the sums of acc have been read
    sum_waves(nxt, red, w, lane);
    double* vs = V + (uint64_t)samp_r2(n + 2) * kSB;
#pragma unroll
    for (int t = 0; t < kOwn; ++t) {
      const int r = w * kOwn + t, e = e0 + r;
      if (e >= n) break;
      const double s = fma(q[(uint64_t)e * kSB], vo[r * kSB], acc[t]);
      vo[r * kSB] = fma(0.25 * chi, s, h * vn[r * kSB]);
      vs[r * kSB] = fma(qn[(uint64_t)e * kSB], vs[r * kSB], nxt[t]);
    }
  } else {
    const double* vl = V + (uint64_t)samp_r2(n - 1) * kSB;
    const double ql = q[(uint64_t)(n - 1) * kSB], c = k2[n - 1] * ql;
#pragma unroll
    for (int r = 0; r < kRun; ++r) {
      const int e = e0 + r;
      if (e >= n) break;
      const double s = e < n - 1 ? fma(c, vl[r * kSB], vo[r * kSB]) : ql * vo[r * kSB];
      vo[r * kSB] = fma(0.25 * chi, s, h * vn[r * kSB]);
    }
  }
}

// Rows of the product with V(n; j): Z3(n', n), n < n' <= M (into the slots of
// p+(x_n'..x_n)); B(n', n), n < n' < M (into those of V(n'+1; n)).
__device__ __forceinline__ void row_of(const StepArgs& A, int r, uint32_t* kap, uint32_t* dest) {
  const int n = A.n, m = A.M - n;
  if (r < m) {
    const int np = n + 1 + r;
    *kap = A.ko.off[3] + samp_r3(np) + samp_r2(n);
    *dest = A.st.PP + samp_r2(np + 1) + (uint32_t)n - 1;
  } else {
    const int np = n + 1 + r - m;
    *kap = A.ko.off[2] + samp_r2(np);
    *dest = A.st.V + samp_r2(np + 1) + (uint32_t)n - 1;
  }
}

// The V update of step n and the product with V(n; .), which are independent.
template <bool FULL>
__global__ __launch_bounds__(256) void step_kernel(StepArgs A, int rows, int row_blocks, uint32_t nprod,
                                                   uint32_t nsb, uint32_t runs, uint32_t group) {
  __shared__ double Bs[2][1][kKC][kLdB];
  static_assert(sizeof(Bs) >= kSumWords * sizeof(double), "the sums of a workgroup's waves fit the operand buffers");
  if (blockIdx.x >= nprod) {
    update_item<FULL>(A, blockIdx.x - nprod, nsb, runs, group, threadIdx.x & 63,
                             __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), &Bs[0][0][0][0]);
    return;
  }
  const int n = A.n;
  double* blk = block_of(A, blockIdx.x / (uint32_t)row_blocks);
  const double* V = blk + (uint64_t)(A.st.V + samp_r2(n)) * kSB;
  product_block<1>(
      (int)(blockIdx.x % (uint32_t)row_blocks), rows, n - 1,
      [&](int r) {
        uint32_t k, d;
        row_of(A, r, &k, &d);
        return A.kap + k;
      },
      [&](int k) { return V + (uint64_t)k * kSB; },
      [&](int r) {
        uint32_t k, d;
        row_of(A, r, &k, &d);
        return blk + (uint64_t)d * kSB;
      },
      Bs);
}

}  // namespace

size_t single_sampler_bytes(int M) { return (size_t)Store::make(M).total * sizeof(double); }

hipError_t launch_single_sampler(int M, const double* kap, KapOffsets ko, int64_t nsamp, const double* u,
                                 uint64_t ldu, double* tab, uint8_t* bits, double* prob, double* cond,
                                 hipStream_t s) {
  const uint32_t nsb = (uint32_t)((nsamp + kSB - 1) / kSB);
  const uint32_t groups = std::max(1u, (nsb + kGroup / 2) / kGroup), group = (nsb + groups - 1) / groups;
  StepArgs A{kap, ko, tab, Store::make(M), M, 0};
  hipError_t e = hipSuccess;
  for (int n = 1; n <= M && e == hipSuccess; ++n) {
    A.n = n;
    const uint32_t m = (uint32_t)(M - n);
    hipLaunchKernelGGL(bit_kernel, dim3(nsb), dim3(256), 0, s, A, u, ldu, nsamp, bits, prob, cond);
    if (n < M) {
      const uint32_t pr = ((uint32_t)n + kRun - 1) / kRun;
      hipLaunchKernelGGL(partial_kernel, dim3(pr * nsb), dim3(256), 0, s, A, nsb, pr, group);
      // at n = 1 the products have no terms: their slots are set to 0
      const bool full = (m & 1) == 0;
      const uint32_t rows = 2 * m - 1, rb = (rows + 63) / 64, runs = ((uint32_t)n - 1 + kRun - 1) / kRun;
      const uint32_t nprod = rb * nsb;
      const dim3 grid(nprod + (full ? runs * nsb : (runs * nsb + 3) / 4));
      const auto k = full ? step_kernel<true> : step_kernel<false>;
      hipLaunchKernelGGL(k, grid, dim3(256), 0, s, A, (int)rows, (int)rb, nprod, nsb, runs, group);
    }
    e = hipGetLastError();
  }
  return e;
}

}  // namespace gbs
