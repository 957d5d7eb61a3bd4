// Adjoint (vector-Jacobian product) of the correlator/cumulant path.
//
// Forward chain, for all subsets up to order K (m = mu for click, c for parity):
//   p(T) = det(Q_T)^(-1/2)                                   (App. D.1)
//   m(B) = sum_{T subset B} a(B,T) p(T),  a = (-1)^|T| (click) or (-1)^|B| (-2)^|T| (parity)
//   k(S) = sum_{pi partition of S} w(pi) prod_{B in pi} m(B) (Eq. cumulant_corr_main)
// Reverse, given the upstream gradients gm(S) (correlators) and gk(S) (cumulants):
//   mbar(B) = gm(B) + gk(B) + sum_{X disjoint from B, 1 <= |X| <= K-|B|} gk(B + X) D1(X),
//      where d k(S)/d m(B) = D1(S \ B) and, for X non-empty,
//      D1(X) = sum_{pi partition of X} (-1)^|pi| |pi|! prod_{B' in pi} m(B')
//      (the partitions of S having B as a block are pi' + {B}, pi' a partition of
//      S \ B, with weight w(|pi'| + 1) = (-1)^|pi'| |pi'|!);
//   pbar(T) = sum_{B superset of T, |B| <= K} a(B,T) mbar(B);
//   d p(T) / d Q_T = -p(T) Q_T^{-1} / 2   (d log det A = tr(A^{-1} dA)),
//   so the 2x2 block (i, j) of dL/dsigma is
//      G_ij = sum_{T containing i and j} -pbar(T) p(T) [Q_T^{-1}]_{ij} / 2.
// pbar is a sum over all supersets: with S_n(T) the sum of mbar over the supersets
// of T of size n, S_n(T) = sum_{x not in T} S_n(T + x) / (n - |T|), so each order
// reads M - |T| values of the order above.  G_ij needs [Q_T^{-1}]_ij for every T
// that holds i and j; the same factorisation gives the diagonal blocks ii and jj,
// which T's |T| - 1 pairs with i share, so one pass over the pairs serves all
// blocks.  Every sum is a gather owned by one workgroup or wavefront and reduced
// in a fixed order: no atomics, results are bitwise reproducible.
#include <hip/hip_runtime.h>

#include "gbs_internal.h"

namespace gbs {

namespace {

constexpr int kWave = 64;

// Set partitions of {0..n-1}, n <= 4, as block masks (restricted growth strings).
struct PartTable {
  int count[5];
  int nblocks[5][15];
  unsigned char blocks[5][15][4];
};

constexpr PartTable make_partitions() {
  PartTable t{};
  for (int n = 1; n <= 4; ++n) {
    int lab[4] = {0, 0, 0, 0};
    int total = 1;
    for (int i = 0; i < n; ++i) total *= n;
    int cnt = 0;
    for (int code = 0; code < total; ++code) {
      int c = code;
      for (int i = 0; i < n; ++i) {
        lab[i] = c % n;
        c /= n;
      }
      // restricted growth: lab[0] = 0, lab[i] <= 1 + max(lab[0..i-1])
      bool ok = lab[0] == 0;
      int mx = 0;
      for (int i = 1; i < n && ok; ++i) {
        if (lab[i] > mx + 1) ok = false;
        if (lab[i] > mx) mx = lab[i];
      }
      if (!ok) continue;
      t.nblocks[n][cnt] = mx + 1;
      for (int b = 0; b < 4; ++b) t.blocks[n][cnt][b] = 0;
      for (int i = 0; i < n; ++i) t.blocks[n][cnt][lab[i]] |= (unsigned char)(1u << i);
      ++cnt;
    }
    t.count[n] = cnt;
  }
  return t;
}

__constant__ PartTable kParts = make_partitions();

__device__ __forceinline__ uint64_t binom_at(const uint64_t* __restrict__ bin, int n, int k) {
  return bin[k * kBinLd + n];
}

__device__ __forceinline__ uint64_t rank_sorted(const uint64_t* __restrict__ bin, const int* s,
                                                int n) {
  uint64_t r = 0;
  for (int j = 0; j < n; ++j) r += binom_at(bin, s[j], j + 1);
  return r;
}

// j-subset of [0, universe) with colex rank r, ascending.
__device__ __forceinline__ void unrank_dyn(const uint64_t* __restrict__ bin, uint64_t r, int j,
                                           int universe, int* x) {
  int hi = universe;
  for (int t = j - 1; t >= 0; --t) {
    int lo = t, h = hi - 1;
    while (lo < h) {
      const int mid = (lo + h + 1) >> 1;
      if (binom_at(bin, mid, t + 1) <= r) lo = mid; else h = mid - 1;
    }
    x[t] = lo;
    r -= binom_at(bin, lo, t + 1);
    hi = lo;
  }
}

// C(x, k) for the colex rank (k = 1..5): closed forms where they are cheap
__device__ __forceinline__ uint64_t choose_k(const uint64_t* __restrict__ bin, int x, int k) {
  if (k == 1) return (uint64_t)x;
  if (k == 2) return (uint64_t)((uint32_t)x * (uint32_t)(x - 1) / 2);
  return binom_at(bin, x, k);
}

// j-subset of [0, universe) with colex rank r, ascending.
template <int J>
__device__ __forceinline__ void unrank_small(const uint64_t* __restrict__ bin, uint64_t r, int universe,
                                             int (&x)[J]) {
  if constexpr (J == 1) {
    x[0] = (int)r;
  } else if constexpr (J == 2) {
    const uint32_t q = (uint32_t)r;  // C(2048, 2) < 2^22
    int b = (int)(0.5f * (1.0f + sqrtf(fmaf(8.0f, (float)q, 1.0f))));
    while ((uint32_t)b * (uint32_t)(b - 1) / 2 > q) --b;
    while ((uint32_t)b * (uint32_t)(b + 1) / 2 <= q) ++b;
    x[1] = b;
    x[0] = (int)(q - (uint32_t)b * (uint32_t)(b - 1) / 2);
  } else {
    unrank_dyn(bin, r, J, universe, x);
  }
}

// Modes of a J-subset of the complement of B (sorted): complement index ->
// mode, skipping B's elements in increasing order.
template <int J, int KB>
__device__ __forceinline__ void complement_modes(const int (&B)[KB], int (&x)[J]) {
#pragma unroll
  for (int t = 0; t < J; ++t) {
    int m = x[t];
#pragma unroll
    for (int i = 0; i < KB; ++i) m += B[i] <= m ? 1 : 0;
    x[t] = m;
  }
}

// Colex rank of the union of two disjoint sorted sets.
template <int KB, int J>
__device__ __forceinline__ uint64_t union_rank(const uint64_t* __restrict__ bin, const int (&B)[KB],
                                               const int (&X)[J]) {
  uint64_t r = 0;
#pragma unroll
  for (int i = 0; i < KB; ++i) {
    int pos = i + 1;
#pragma unroll
    for (int j = 0; j < J; ++j) pos += X[j] < B[i] ? 1 : 0;
    r += choose_k(bin, B[i], pos);
  }
#pragma unroll
  for (int j = 0; j < J; ++j) {
    int pos = j + 1;
#pragma unroll
    for (int i = 0; i < KB; ++i) pos += B[i] < X[j] ? 1 : 0;
    r += choose_k(bin, X[j], pos);
  }
  return r;
}

template <int J>
__device__ __forceinline__ uint64_t set_rank(const uint64_t* __restrict__ bin, const int (&X)[J]) {
  uint64_t r = 0;
#pragma unroll
  for (int j = 0; j < J; ++j) r += choose_k(bin, X[j], j + 1);
  return r;
}

__device__ __forceinline__ uint64_t count_sized(const uint64_t* __restrict__ bin, int jmin, int jmax,
                                                int u) {
  uint64_t c = 0;
  for (int t = jmin; t <= jmax; ++t) c += binom_at(bin, u, t);
  return c;
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
  return v;
}

// Workgroups of up to this many threads share one superset sum (the sigma-bar
// kernel, whose per-superset inverse needs about 200 registers, up to
// kSigmaThreads).
constexpr int kSumThreads = 1024;
constexpr int kSigmaThreads = 256;

// Sum over the workgroup in a fixed order (lanes by the butterfly, then the
// waves in index order): deterministic for a given launch shape.  Valid in
// thread 0.
__device__ __forceinline__ double block_sum(double v) {
  __shared__ double part[kSumThreads / kWave];
  __syncthreads();  // thread 0 has read the previous call's partial sums
  v = wave_sum(v);
  const int w = threadIdx.x / kWave;
  if ((threadIdx.x & (kWave - 1)) == 0) part[w] = v;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0)
    for (int i = 0; i < (int)(blockDim.x / kWave); ++i) t += part[i];
  return t;
}

struct Offsets {
  int64_t off[kMaxOrder + 2];  // start of order-d block, off[1] = 0
};

// A superset sum of n terms split over nsplit workgroups (blockIdx.y): chunk y
// takes the terms [n y / nsplit, n (y + 1) / nsplit).  With nsplit > 1 each
// workgroup writes its partial sum to part[(item * nsplit + y) * width + e] and
// a finishing kernel adds the partials in chunk order, so the result stays
// deterministic for a given launch shape.
__device__ __forceinline__ void chunk_range(uint64_t n, uint64_t* lo, uint64_t* hi) {
  *lo = n * blockIdx.y / gridDim.y;
  *hi = n * (blockIdx.y + 1) / gridDim.y;
}

// ---------------------------------------------------------------------------
// D1(X) for every non-empty X with |X| <= K - 1 (one thread per X).
__global__ void d1_kernel(const double* __restrict__ m, int M, int K, Offsets o,
                          const uint64_t* __restrict__ bin, double* __restrict__ d1) {
  const int64_t total = o.off[K];  // orders 1..K-1
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (int64_t)gridDim.x * blockDim.x) {
    int j = 1;
    while (idx >= o.off[j + 1]) ++j;
    const uint64_t r = (uint64_t)(idx - o.off[j]);
    int x[kMaxOrder];
    unrank_dyn(bin, r, j, M, x);
    double mv[16];
    mv[0] = 1.0;
    for (unsigned mask = 1; mask < (1u << j); ++mask) {
      int sub[kMaxOrder], n = 0;
      for (int t = 0; t < j; ++t)
        if (mask & (1u << t)) sub[n++] = x[t];
      mv[mask] = m[o.off[n] + rank_sorted(bin, sub, n)];
    }
    double acc = 0.0;
    for (int q = 0; q < kParts.count[j]; ++q) {
      const int nb = kParts.nblocks[j][q];
      double w = (nb & 1) ? -1.0 : 1.0;
      for (int f = 2; f <= nb; ++f) w *= f;  // (-1)^nb nb!
      for (int b = 0; b < nb; ++b) w *= mv[kParts.blocks[j][q][b]];
      acc += w;
    }
    d1[idx] = acc;
  }
}

// The terms of mbar(B) with |X| = J, whose flat indices start at `first`.
template <int KB, int J>
__device__ __forceinline__ double mbar_terms(int M, const int (&B)[KB], uint64_t first, uint64_t lo, uint64_t hi,
                                             const Offsets& o, const uint64_t* __restrict__ bin,
                                             const double* __restrict__ gk, const double* __restrict__ d1) {
  const uint64_t n = binom_at(bin, M - KB, J);
  const uint64_t b = lo > first ? lo - first : 0, e = hi > first ? min(hi - first, n) : 0;
  const double* g = gk + o.off[KB + J];
  const double* d = d1 + o.off[J];
  double acc = 0.0;
  for (uint64_t q = b + threadIdx.x; q < e; q += blockDim.x) {
    int X[J];
    unrank_small<J>(bin, q, M - KB, X);
    complement_modes<J, KB>(B, X);
    acc = fma(g[union_rank<KB, J>(bin, B, X)], d[set_rank<J>(bin, X)], acc);
  }
  return acc;
}

// mbar(B) for every B of order KB (one workgroup per B and chunk of its supersets).
template <int KB>
__global__ __launch_bounds__(kSumThreads) void mbar_kernel(int M, int K, Offsets o, const uint64_t* __restrict__ bin,
                                                           const double* __restrict__ gm,
                                                           const double* __restrict__ gk,
                                                           const double* __restrict__ d1, double* __restrict__ mbar,
                                                           double* __restrict__ part) {
  const uint64_t rb = blockIdx.x;
  int B[KB];
  unrank_small<KB>(bin, rb, M, B);
  double acc = 0.0;
  if (gk) {
    uint64_t lo, hi, first = 0;
    chunk_range(count_sized(bin, 1, K - KB, M - KB), &lo, &hi);
    acc = mbar_terms<KB, 1>(M, B, first, lo, hi, o, bin, gk, d1);
    first += binom_at(bin, M - KB, 1);
    if constexpr (KB <= 3) {
      if (K - KB >= 2) acc += mbar_terms<KB, 2>(M, B, first, lo, hi, o, bin, gk, d1);
      first += binom_at(bin, M - KB, 2);
    }
    if constexpr (KB <= 2) {
      if (K - KB >= 3) acc += mbar_terms<KB, 3>(M, B, first, lo, hi, o, bin, gk, d1);
      first += binom_at(bin, M - KB, 3);
    }
    if constexpr (KB == 1) {
      if (K - KB >= 4) acc += mbar_terms<KB, 4>(M, B, first, lo, hi, o, bin, gk, d1);
    }
  }
  acc = block_sum(acc);
  if (threadIdx.x == 0) {
    if (gridDim.y > 1) {
      part[rb * gridDim.y + blockIdx.y] = acc;
      return;
    }
    const int64_t at = o.off[KB] + (int64_t)rb;
    double v = acc;
    if (gk) v += gk[at];
    if (gm) v += gm[at];
    mbar[at] = v;
  }
}

// The split mbar sums of order k: partials in chunk order, then as mbar_kernel.
__global__ void mbar_finish_kernel(int k, int nsplit, uint64_t count, Offsets o,
                                   const double* __restrict__ gm, const double* __restrict__ gk,
                                   const double* __restrict__ part, double* __restrict__ mbar) {
  const uint64_t rb = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (rb >= count) return;
  double v = 0.0;
  for (int y = 0; y < nsplit; ++y) v += part[rb * nsplit + y];
  const int64_t at = o.off[k] + (int64_t)rb;
  if (gk) v += gk[at];
  if (gm) v += gm[at];
  mbar[at] = v;
}

// The top order K has no proper supersets: mbar = gk + gm and
// pbar = (-1)^K mbar (click) or (-2)^K (-1)^K mbar (parity), one thread per subset.
__global__ void top_order_kernel(int64_t off, uint64_t count, int K, int parity,
                                 const double* __restrict__ gm, const double* __restrict__ gk,
                                 double* __restrict__ mbar, double* __restrict__ pbar) {
  const uint64_t r = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= count) return;
  const int64_t at = off + (int64_t)r;
  double v = 0.0;
  if (gk) v += gk[at];
  if (gm) v += gm[at];
  mbar[at] = v;
  double coef = (K & 1) ? -1.0 : 1.0;
  if (parity) coef *= (K & 1) ? -(double)(1 << K) : (double)(1 << K);
  pbar[at] = coef * v;
}

// Superset sums of order t, one wavefront per T: S_n(T) for n = t + 1..K, from
// mbar and the sums of order t + 1 (sup: for each order its K - t sums one array
// after the other, see sup_at), and with them pbar(T).
__host__ __device__ inline int64_t sup_at(const Offsets& o, int K, int t, int n) {
  // orders K - 1, K - 2, .. first; order t holds n = t + 1..K
  int64_t at = 0;
  for (int u = K - 1; u > t; --u) at += (int64_t)(K - u) * (o.off[u + 1] - o.off[u]);
  return at + (int64_t)(n - t - 1) * (o.off[t + 1] - o.off[t]);
}

template <int T>
__global__ __launch_bounds__(256) void pbar_kernel(int M, int K, int parity, Offsets o,
                                                   const uint64_t* __restrict__ bin, const double* __restrict__ mbar,
                                                   double* __restrict__ sup, double* __restrict__ pbar) {
  const int64_t rt = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (rt >= o.off[T + 1] - o.off[T]) return;
  const int lane = threadIdx.x & 63;
  int S[T];
  unrank_small<T>(bin, (uint64_t)rt, M, S);
  double acc[kMaxOrder - T] = {};
  for (int q = lane; q < M - T; q += 64) {
    int X[1] = {q};
    complement_modes<1, T>(S, X);
    const int64_t r = (int64_t)union_rank<T, 1>(bin, S, X);
    acc[0] += mbar[o.off[T + 1] + r];
#pragma unroll
    for (int d = 1; d < kMaxOrder - T; ++d)
      if (T + 1 + d <= K) acc[d] += sup[sup_at(o, K, T + 1, T + 1 + d) + r];
  }
  const double own = mbar[o.off[T] + rt];
  double total = (parity && (T & 1)) ? -own : own;
#pragma unroll
  for (int d = 0; d < kMaxOrder - T; ++d) {
    const int n = T + 1 + d;
    if (n > K) break;
    const double v = wave_sum(acc[d]) / (double)(d + 1);
    if (lane == 0) sup[sup_at(o, K, T, n) + rt] = v;
    total += (parity && (n & 1)) ? -v : v;
  }
  if (lane == 0) {
    // click: (-1)^t;  parity: (-2)^t (the (-1)^|B| factor is inside the sum)
    double coef = (T & 1) ? -1.0 : 1.0;
    if (parity) coef *= (double)(1 << T);
    pbar[o.off[T] + rt] = coef * total;
  }
}

// The blocks of Q_T^{-1} at the last two of T's modes [X (NX of them), i, j]: X is
// eliminated block by block, then the 4x4 Schur complement of (i, j) is inverted.
// G: block (i, j); Di, Dj: blocks (i, i), (j, j) (x-x, p-x, p-p).
template <int NX>
__device__ __forceinline__ void pair_inverse(const double* __restrict__ Qi, const double* __restrict__ Qd, int M,
                                             const int (&modes)[NX + 2], double (&G)[4], double (&Di)[3],
                                             double (&Dj)[3], bool& bad) {
  Tri<2 * NX + 4> A;
  gather_q_coalesced<NX + 2, 0>(Qi, Qd, M, modes, A);
  double S[tri_size(4)];
  auto pivot = [&](double a, double b, double c) {
    const double det = fma(a, c, -b * b);
    bad |= !(det > 0.0);
    return 1.0 / det;
  };
  if constexpr (NX == 0) {
#pragma unroll
    for (int q = 0; q < tri_size(4); ++q) S[q] = A.a[q];
  } else {
    Tri<2 * NX + 2> A1;
    schur_leading_block<2 * NX + 4>(A, pivot(A.a[0], A.a[1], A.a[2]), A1);
    if constexpr (NX == 1) {
#pragma unroll
      for (int q = 0; q < tri_size(4); ++q) S[q] = A1.a[q];
    } else {
      Tri<2 * NX> A2;
      schur_leading_block<2 * NX + 2>(A1, pivot(A1.a[0], A1.a[1], A1.a[2]), A2);
      if constexpr (NX == 2) {
#pragma unroll
        for (int q = 0; q < tri_size(4); ++q) S[q] = A2.a[q];
      } else {
        static_assert(NX == 3, "at most three eliminated blocks");
        Tri<2 * NX - 2> A3;
        schur_leading_block<2 * NX>(A2, pivot(A2.a[0], A2.a[1], A2.a[2]), A3);
#pragma unroll
        for (int q = 0; q < tri_size(4); ++q) S[q] = A3.a[q];
      }
    }
  }
  // [[A, Bm], [Bm^T, C]]^{-1}: with Y = A^{-1} Bm and Sc = C - Bm^T Y, the blocks
  // are Sc^{-1} at C, -Y Sc^{-1} off the diagonal, A^{-1} + Y Sc^{-1} Y^T at A.
  const double a00 = S[tri(0, 0)], a10 = S[tri(1, 0)], a11 = S[tri(1, 1)];
  const double b00 = S[tri(2, 0)], b01 = S[tri(3, 0)], b10 = S[tri(2, 1)], b11 = S[tri(3, 1)];
  const double ia = pivot(a00, a10, a11);
  const double ai00 = a11 * ia, ai01 = -a10 * ia, ai11 = a00 * ia;
  const double y00 = ai00 * b00 + ai01 * b10, y01 = ai00 * b01 + ai01 * b11;
  const double y10 = ai01 * b00 + ai11 * b10, y11 = ai01 * b01 + ai11 * b11;
  const double c00 = S[tri(2, 2)] - (b00 * y00 + b10 * y10);
  const double c01 = S[tri(3, 2)] - (b00 * y01 + b10 * y11);
  const double c11 = S[tri(3, 3)] - (b01 * y01 + b11 * y11);
  const double ic = pivot(c00, c01, c11);
  const double si00 = c11 * ic, si01 = -c01 * ic, si11 = c00 * ic;
  G[0] = -(y00 * si00 + y01 * si01);
  G[1] = -(y00 * si01 + y01 * si11);
  G[2] = -(y10 * si00 + y11 * si01);
  G[3] = -(y10 * si01 + y11 * si11);
  Dj[0] = si00;
  Dj[1] = si01;
  Dj[2] = si11;
  Di[0] = ai00 - (G[0] * y00 + G[1] * y01);
  Di[1] = ai01 - (G[2] * y00 + G[3] * y01);
  Di[2] = ai11 - (G[2] * y10 + G[3] * y11);
}

// The terms of a pair (i < j) with NX further modes.
template <int NX>
__device__ __forceinline__ void pair_terms(const double* __restrict__ Qi, const double* __restrict__ Qd, int M,
                                           const int (&base)[2], const Offsets& o, const uint64_t* __restrict__ bin,
                                           const double* __restrict__ ptab, const double* __restrict__ pbar,
                                           double (&acc)[4], double (&di)[3], double (&dj)[3], bool& bad) {
  const uint64_t n = NX == 0 ? 1 : binom_at(bin, M - 2, NX);
  for (uint64_t q = threadIdx.x; q < n; q += blockDim.x) {
    int modes[NX + 2];
    uint64_t rank;
    if constexpr (NX == 0) {
      rank = set_rank<2>(bin, base);
    } else {
      int X[NX];
      unrank_small<NX>(bin, q, M - 2, X);
      complement_modes<NX, 2>(base, X);
      rank = union_rank<2, NX>(bin, base, X);
#pragma unroll
      for (int t = 0; t < NX; ++t) modes[t] = X[t];
    }
    modes[NX] = base[0];
    modes[NX + 1] = base[1];
    const int64_t at = o.off[NX + 2] + (int64_t)rank;
    const double w = -0.5 * pbar[at] * ptab[at];
    double G[4], Di[3], Dj[3];
    pair_inverse<NX>(Qi, Qd, M, modes, G, Di, Dj, bad);
    const double wd = w / (double)(NX + 1);  // i's diagonal block is shared by T's NX + 1 pairs with i
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] = fma(w, G[e], acc[e]);
#pragma unroll
    for (int e = 0; e < 3; ++e) {
      di[e] = fma(wd, Di[e], di[e]);
      dj[e] = fma(wd, Dj[e], dj[e]);
    }
  }
}

// The 2x2 block (i, j) of dL/dsigma (interleaved (2i + a, 2j + b) -> xxpp
// (i + a M, j + b M)) and, for i != j, its mirror.
__device__ __forceinline__ void store_sigma_block(double* __restrict__ gsig, int M, int i, int j,
                                                  const double (&acc)[4]) {
  const size_t n2 = 2 * (size_t)M;
  const size_t xi = i, pi = i + M, xj = j, pj = j + M;
  gsig[xi * n2 + xj] = acc[0];
  gsig[xi * n2 + pj] = acc[1];
  gsig[pi * n2 + xj] = acc[2];
  gsig[pi * n2 + pj] = acc[3];
  if (i != j) {
    gsig[xj * n2 + xi] = acc[0];
    gsig[pj * n2 + xi] = acc[1];
    gsig[xj * n2 + pi] = acc[2];
    gsig[pj * n2 + pi] = acc[3];
  }
}

// One workgroup per pair i < j (colex): the block (i, j) of dL/dsigma, and the
// pair's share of the blocks (i, i) and (j, j) in diag[(i M + j) 3], diag[(j M + i) 3].
template <int KX>
__global__ __launch_bounds__(kSigmaThreads) void sigma_pairs_kernel(const double* __restrict__ Qi,
                                                                    const double* __restrict__ Qd, int M, Offsets o,
                                                                    const uint64_t* __restrict__ bin,
                                                                    const double* __restrict__ ptab,
                                                                    const double* __restrict__ pbar,
                                                                    double* __restrict__ gsig,
                                                                    double* __restrict__ diag,
                                                                    DeviceStatus* __restrict__ st) {
  int base[2];
  unrank_small<2>(bin, blockIdx.x, M, base);
  double acc[4] = {}, di[3] = {}, dj[3] = {};
  bool bad = false;
  pair_terms<0>(Qi, Qd, M, base, o, bin, ptab, pbar, acc, di, dj, bad);
  if constexpr (KX >= 1) pair_terms<1>(Qi, Qd, M, base, o, bin, ptab, pbar, acc, di, dj, bad);
  if constexpr (KX >= 2) pair_terms<2>(Qi, Qd, M, base, o, bin, ptab, pbar, acc, di, dj, bad);
  if constexpr (KX >= 3) pair_terms<3>(Qi, Qd, M, base, o, bin, ptab, pbar, acc, di, dj, bad);
  const int i = base[0], j = base[1];
  if (bad) latch_failure(st, 0, (int64_t)j * (j + 1) / 2 + i);  // pair index, i <= j
#pragma unroll
  for (int e = 0; e < 4; ++e) acc[e] = block_sum(acc[e]);
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    di[e] = block_sum(di[e]);
    dj[e] = block_sum(dj[e]);
  }
  if (threadIdx.x != 0) return;
  store_sigma_block(gsig, M, i, j, acc);
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    diag[((size_t)i * M + j) * 3 + e] = di[e];
    diag[((size_t)j * M + i) * 3 + e] = dj[e];
  }
}

// Order 1 alone reaches the diagonal blocks only: the others are 0.
__global__ void zero_kernel(double* __restrict__ gsig, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) gsig[i] = 0.0;
}
hipError_t launch_zero_offdiag(double* gsig, int M, hipStream_t s) {
  const size_t n = 4 * (size_t)M * M;
  hipLaunchKernelGGL(zero_kernel, dim3((unsigned)std::min<size_t>((n + 255) / 256, 4096)), dim3(256), 0, s, gsig, n);
  return hipGetLastError();
}

// The blocks (i, i): the subset {i} alone and the pairs' shares, one wavefront per i.
__global__ __launch_bounds__(256) void sigma_diag_kernel(const double* __restrict__ Qd, int M, int K,
                                                         const double* __restrict__ ptab,
                                                         const double* __restrict__ pbar,
                                                         const double* __restrict__ diag, double* __restrict__ gsig,
                                                         DeviceStatus* __restrict__ st) {
  const int i = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (i >= M) return;
  double d[3] = {};
  if (K >= 2)
    for (int j = lane; j < M; j += 64)
      if (j != i)
#pragma unroll
        for (int e = 0; e < 3; ++e) d[e] += diag[((size_t)i * M + j) * 3 + e];
#pragma unroll
  for (int e = 0; e < 3; ++e) d[e] = wave_sum(d[e]);
  if (lane != 0) return;
  const double a00 = Qd[4 * (size_t)i], a10 = Qd[4 * (size_t)i + 1], a11 = Qd[4 * (size_t)i + 2];
  const double det = fma(a00, a11, -a10 * a10);
  if (!(det > 0.0)) latch_failure(st, 0, (int64_t)i * (i + 1) / 2 + i);
  const double w = -0.5 * pbar[i] * ptab[i] / det;
  d[0] = fma(w, a11, d[0]);
  d[1] = fma(w, -a10, d[1]);
  d[2] = fma(w, a00, d[2]);
  const double acc[4] = {d[0], d[1], d[1], d[2]};
  store_sigma_block(gsig, M, i, i, acc);
}

}  // namespace

size_t adjoint_sup_doubles(int M, int K) {
  size_t n = 1;
  for (int t = 1; t < K; ++t) n += (size_t)(K - t) * host_binom(M, t);
  return n;
}

hipError_t launch_adjoint(int M, int K, int flags, const double* Qi, const double* Qd, const uint64_t* binom,
                          const double* m, const double* ptab, const double* gm, const double* gk,
                          double* d1, double* mbar, double* pbar, double* gsig, DeviceStatus* st,
                          double* part, double* sup, double* diag, hipStream_t s) {
  Offsets o{};
  o.off[1] = 0;
  for (int d = 1; d <= kMaxOrder; ++d) o.off[d + 1] = o.off[d] + (d <= K ? (int64_t)host_binom(M, d) : 0);
  hipError_t e = hipSuccess;
  const int parity = (flags & GBS_PARITY) ? 1 : 0;
  if (K >= 2 && gk) {
    e = timing_begin(s, GBS_STAGE_ADJOINT, 0);
    const int64_t n1 = o.off[K];
    const int grid = (int)std::min<int64_t>((n1 + 255) / 256, 65535);
    if (e == hipSuccess) hipLaunchKernelGGL(d1_kernel, dim3(grid), dim3(256), 0, s, m, M, K, o, binom, d1);
    if (e == hipSuccess) e = hipGetLastError();
    if (e == hipSuccess) e = timing_end(s);
  }
  // threads per workgroup for a sum over n terms: whole wavefronts, at most cap
  auto threads_for = [](uint64_t n, int cap) {
    const uint64_t w = std::max<uint64_t>(1, std::min<uint64_t>((n + kWave - 1) / kWave,
                                                                (uint64_t)(cap / kWave)));
    return (unsigned)(w * kWave);
  };
  // Workgroups per mbar sum: a launch of fewer than kAdjointSplitItems long sums
  // (the order-1 subsets) would leave compute units idle, so each sum is split into
  // chunks of at least 16,384 terms (16 rounds of a workgroup).  Gradient calls with
  // chunks of 512 / 2,048 / 4,096 / 16,384, us: M = 144, K = 3 (10,296 terms a sum) 194 /
  // 182 / 183 / 183, M = 30, K = 4 (4,089) 123 / 121 / 129 / 119, M = 40, K = 4 (9,919)
  // 157 / 147 / 168 / 167, M = 60, K = 4 (34,279) 293 / 265 / 274 / 309.
  auto split_for = [](uint64_t items, uint64_t n) -> unsigned {
    if (items >= (uint64_t)kAdjointSplitItems) return 1u;
    const uint64_t want = ((uint64_t)kAdjointSplitItems + items - 1) / items;
    return (unsigned)std::max<uint64_t>(1, std::min<uint64_t>({want, (uint64_t)kAdjointMaxSplit, n / 16384}));
  };
  for (int k = 1; k < K && e == hipSuccess; ++k) {
    e = timing_begin(s, GBS_STAGE_ADJOINT, k);
    const uint64_t items = host_binom(M, k);
    uint64_t n = 0;
    for (int j = 1; j <= K - k; ++j) n += host_binom(M - k, j);
    const unsigned ns = gk ? split_for(items, n) : 1u;
    const dim3 grid((unsigned)items, ns), wg(gk ? threads_for((n + ns - 1) / ns, kSumThreads) : kWave);
    if (e == hipSuccess) {
      switch (k) {
        case 1: hipLaunchKernelGGL(mbar_kernel<1>, grid, wg, 0, s, M, K, o, binom, gm, gk, d1, mbar, part); break;
        case 2: hipLaunchKernelGGL(mbar_kernel<2>, grid, wg, 0, s, M, K, o, binom, gm, gk, d1, mbar, part); break;
        case 3: hipLaunchKernelGGL(mbar_kernel<3>, grid, wg, 0, s, M, K, o, binom, gm, gk, d1, mbar, part); break;
        default: hipLaunchKernelGGL(mbar_kernel<4>, grid, wg, 0, s, M, K, o, binom, gm, gk, d1, mbar, part); break;
      }
      e = hipGetLastError();
    }
    if (e == hipSuccess && ns > 1)
      hipLaunchKernelGGL(mbar_finish_kernel, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, s, k, (int)ns,
                         items, o, gm, gk, part, mbar);
    if (e == hipSuccess) e = hipGetLastError();
    if (e == hipSuccess) e = timing_end(s);
  }
  if (e == hipSuccess) {  // order K: mbar and pbar together
    e = timing_begin(s, GBS_STAGE_ADJOINT, K);
    const uint64_t cnt = host_binom(M, K);
    if (e == hipSuccess)
      hipLaunchKernelGGL(top_order_kernel, dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0, s,
                         o.off[K], cnt, K, parity, gm, gk, mbar, pbar);
    if (e == hipSuccess) e = hipGetLastError();
    if (e == hipSuccess) e = timing_end(s);
  }
  for (int t = K - 1; t >= 1 && e == hipSuccess; --t) {  // each from the order above
    e = timing_begin(s, GBS_STAGE_ADJOINT, t);
    const dim3 grid((unsigned)((host_binom(M, t) + 3) / 4)), wg(256);
    if (e == hipSuccess) {
      switch (t) {
        case 1: hipLaunchKernelGGL(pbar_kernel<1>, grid, wg, 0, s, M, K, parity, o, binom, mbar, sup, pbar); break;
        case 2: hipLaunchKernelGGL(pbar_kernel<2>, grid, wg, 0, s, M, K, parity, o, binom, mbar, sup, pbar); break;
        case 3: hipLaunchKernelGGL(pbar_kernel<3>, grid, wg, 0, s, M, K, parity, o, binom, mbar, sup, pbar); break;
        default: hipLaunchKernelGGL(pbar_kernel<4>, grid, wg, 0, s, M, K, parity, o, binom, mbar, sup, pbar); break;
      }
      e = hipGetLastError();
    }
    if (e == hipSuccess) e = timing_end(s);
  }
  if (e == hipSuccess) {
    e = timing_begin(s, GBS_STAGE_ADJOINT, 0);
    const uint64_t pairs = (uint64_t)M * (M - 1) / 2;
    if (e == hipSuccess && K >= 2 && pairs) {
      const dim3 grid((unsigned)pairs), wg(threads_for(host_binom(M - 2, K - 2), kSigmaThreads));
      switch (K) {
        case 2: hipLaunchKernelGGL(sigma_pairs_kernel<0>, grid, wg, 0, s, Qi, Qd, M, o, binom, ptab, pbar, gsig, diag, st); break;
        case 3: hipLaunchKernelGGL(sigma_pairs_kernel<1>, grid, wg, 0, s, Qi, Qd, M, o, binom, ptab, pbar, gsig, diag, st); break;
        case 4: hipLaunchKernelGGL(sigma_pairs_kernel<2>, grid, wg, 0, s, Qi, Qd, M, o, binom, ptab, pbar, gsig, diag, st); break;
        default: hipLaunchKernelGGL(sigma_pairs_kernel<3>, grid, wg, 0, s, Qi, Qd, M, o, binom, ptab, pbar, gsig, diag, st); break;
      }
      e = hipGetLastError();
    }
    if (e == hipSuccess && K == 1 && pairs) e = launch_zero_offdiag(gsig, M, s);
    if (e == hipSuccess) {
      hipLaunchKernelGGL(sigma_diag_kernel, dim3((unsigned)((M + 3) / 4)), dim3(256), 0, s, Qd, M, K, ptab, pbar, diag,
                         gsig, st);
      e = hipGetLastError();
    }
    if (e == hipSuccess) e = timing_end(s);
  }
  return e;
}

}  // namespace gbs
