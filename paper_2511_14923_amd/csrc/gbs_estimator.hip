// Sample-side validation: click cumulants estimated from samples, and the
// Pearson coefficient against the ground truth (App. F, "Click cumulants,
// Pearson and Spearman coefficients"; Eqs. cumulants_test_def and
// pearson_correlation).
//
// The estimator is the unbiased one: every product of |pi| click moments in
// the partition sum of kappa~(S) becomes its average over ordered tuples of
// distinct samples.  Written through the power sums s_B (the number of samples
// in which every mode of B clicked), by Moebius inversion on the partitions of
// the |pi| blocks, it is
//     k(S) = sum_{tau in P(S)} c_N(tau) prod_{B in tau} s_B / N,
// with coefficients c_N(tau) that depend only on the block structure of tau
// and on N (computed on the host).  The work is therefore the power sums of
// every subset of orders <= K:
//   * the samples are packed into bit columns, 64 samples a word, in chunks of
//     512 samples that hold every mode's 64 bytes next to each other;
//   * s_S = sum over the samples of AND_{k in S} is a product of 0/1 matrices:
//     S = L + H with L its lowest one or two modes and H the rest, rows H,
//     columns L, inner index the samples, on the matrix units in FP4, whose 1.0
//     is one bit of a nibble: masking a word of the ANDed columns with every
//     fourth bit gives eight operands at once (count_kernel below);
//   * k(S) gathers the power sums of the 2^|S| - 1 subsets of S from the count
//     tables of the lower orders (colex ranks) and evaluates the sum over the
//     partitions of S.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <functional>
#include <vector>

#include "gbs_internal.h"

namespace gbs {

namespace {

constexpr int kEstThreads = 256;
constexpr int kChunkWords = 8;                    // 64-bit words per mode and chunk
constexpr int kChunkBytes = 8 * kChunkWords;      // 512 samples
constexpr int kPackSamples = 256;                 // samples per workgroup of the packing

// Bit columns: word w of mode k at (w / 8 * M + k) * 8 + w % 8; samples past N are 0.
__global__ __launch_bounds__(kPackSamples) void pack_columns_kernel(const uint8_t* __restrict__ bits, int64_t N,
                                                                    int M, int64_t words, int wide,
                                                                    uint64_t* __restrict__ cols) {
  extern __shared__ uint8_t rows[];  // kPackSamples x M
  const int64_t pack = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
  const int64_t s0 = pack * kPackSamples;
  const int64_t have = min((int64_t)kPackSamples, N - s0);
  const int64_t bytes = have > 0 ? have * M : 0;
  const uint8_t* src = bits + s0 * M;
  if (wide) {  // the caller's buffer starts on a 4-byte boundary, and s0 * M is a multiple of 4
    const int64_t q = bytes >> 2;
    for (int64_t i = threadIdx.x; i < q; i += kPackSamples)
      reinterpret_cast<uint32_t*>(rows)[i] = reinterpret_cast<const uint32_t*>(src)[i];
    for (int64_t i = q * 4 + threadIdx.x; i < bytes; i += kPackSamples) rows[i] = src[i];
  } else {
    for (int64_t i = threadIdx.x; i < bytes; i += kPackSamples) rows[i] = src[i];
  }
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int64_t w = pack * (kPackSamples / 64) + (threadIdx.x >> 6);
  if (w >= words) return;
  const bool live = w * 64 + lane < N;
  const uint8_t* row = rows + (int)threadIdx.x * M;
  uint64_t* out = cols + (w / kChunkWords * M) * kChunkWords + w % kChunkWords;
  for (int k0 = 0; k0 < M; k0 += 64) {
    uint64_t mine = 0;
    const int kn = min(64, M - k0);
    for (int q = 0; q < kn; ++q) {
      const uint64_t m = __ballot(live && row[k0 + q] != 0);
      if (lane == q) mine = m;
    }
    if (lane < kn) out[(int64_t)(k0 + lane) * kChunkWords] = mine;
  }
}

// ---- order 1: s_k = popcount of column k ----
__global__ void count1_kernel(const uint64_t* __restrict__ cols, int M, int64_t words,
                              uint32_t* __restrict__ out) {
  __shared__ uint32_t part[kEstThreads];
  const int k = blockIdx.x;
  uint32_t c = 0;
  for (int64_t w = threadIdx.x; w < words; w += blockDim.x)
    c += __popcll(cols[(w / kChunkWords * M + k) * kChunkWords + w % kChunkWords]);
  part[threadIdx.x] = c;
  __syncthreads();
  for (int h = blockDim.x / 2; h >= 1; h >>= 1) {
    if ((int)threadIdx.x < h) part[threadIdx.x] += part[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[k] = part[0];
}

__global__ void zero_counts_kernel(uint32_t* __restrict__ out, uint64_t n) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
    out[i] = 0;
}

// C(n, k) for small k without a table
__host__ __device__ inline uint64_t choose(uint32_t n, int k) {
  switch (k) {
    case 0: return 1;
    case 1: return n;
    case 2: return n < 2 ? 0 : (uint64_t)n * (n - 1) / 2;
    default: return n < 3 ? 0 : (uint64_t)n * (n - 1) * (n - 2) / 6;
  }
}

// colex unranking of a K-subset (K <= 3) of [0, hi), ascending
template <int K>
__host__ __device__ inline void unrank_small(uint32_t r, int hi, int (&s)[K]) {
  for (int j = K; j >= 1; --j) {
    int lo = j - 1, h = hi - 1;  // largest x < hi with C(x, j) <= r
    while (lo < h) {
      const int mid = (lo + h + 1) >> 1;
      if (choose((uint32_t)mid, j) <= r) lo = mid; else h = mid - 1;
    }
    s[j - 1] = lo;
    r -= (uint32_t)choose((uint32_t)lo, j);
    hi = lo;
  }
}

// Rows of the product: the sets H in colex order of their mirror images {M - 1 -
// m}, so that c = min H falls along the list and the columns L (subsets of
// [0, c), in colex order) that a run of rows needs are a prefix.
template <int DH>
__host__ __device__ inline void row_modes(uint32_t h, int M, int (&m)[DH]) {
  int x[DH];
  unrank_small<DH>(h, M, x);
  for (int j = 0; j < DH; ++j) m[j] = M - 1 - x[DH - 1 - j];
}

// Counts of a tile of kTH rows by kTL columns over a range of sample chunks.
//
// On v_mfma_scale_f32_32x32x64 with FP4 operands (10 PFLOP/s dense, against 8.6e12
// word AND-popcounts/s = 1.1 PFLOP/s of the 32-bit vector units): four waves,
// each 128 x 64 of the tile (4 x 2 accumulators of 32 x 32).  A chunk's ANDed
// words are staged in LDS as bits (64 bytes per row; rows 80 bytes apart, which
// spreads a quarter-wave's 16-byte reads over all banks); a lane reads 128
// samples of its row at once and masks them with 0x1, 0x2, 0x4 and (shifted)
// 0x4 per nibble: FP4 0.5, 1.0, 2.0 and 2.0, which the instruction's block
// scales 2, 1, 1/2, 1/2 of both operands bring to products of 1.  Every operand
// register is thus one or two vector instructions, and both operands meet the
// same samples in the same order by construction.
// Sums are exact: FP32 accumulators hold at most kSplitSamples ones.  Ranges of
// chunks of one tile (few tiles, or more samples than that) add up by integer
// atomics, whose order does not matter.
// Order 5 at M = 144, 262,144 samples: 44.0 ms, 5.7e15 operations/s on the
// 4.8e8 x 262,144 products wanted, against 286 ms of AND and popcount in 32-bit
// vector instructions (0.81 of their peak); 48.6 ms with the loads of the next
// chunk waited for where they are issued. What is left: tiles that reach past a
// row's columns (about 1.1 times the work), and per chunk the masking (20 vector
// instructions for 4 x 6 operands) beside the products.
constexpr int kTH = 256, kTL = 128;
constexpr int kRowBytes = kChunkBytes + 16;
constexpr int64_t kSplitSamples = 1 << 22;

typedef int int8v __attribute__((ext_vector_type(8)));
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));
typedef float float16v __attribute__((ext_vector_type(16)));

template <int T>
__device__ __forceinline__ int8v fp4_operand(const uint4v& w) {
  constexpr uint32_t kMask = T == 0 ? 0x11111111u : T == 1 ? 0x22222222u : 0x44444444u;
  const uint4v v = (T == 3 ? w >> 1 : w) & kMask;
  return int8v{(int)v.x, (int)v.y, (int)v.z, (int)v.w, 0, 0, 0, 0};
}

template <int T>
__device__ __forceinline__ void count_step(const uint4v (&h)[4], const uint4v (&l)[2], float16v (&acc)[4][2]) {
  constexpr int kScale = T == 0 ? 0x80808080 : T == 1 ? 0x7f7f7f7f : 0x7e7e7e7e;
  int8v b[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) b[j] = fp4_operand<T>(l[j]);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int8v a = fp4_operand<T>(h[i]);
#pragma unroll
    for (int j = 0; j < 2; ++j)
      acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b[j], acc[i][j], 4, 4, 0, kScale, 0, kScale);
  }
}

template <int DL, int DH>
__global__ __launch_bounds__(kEstThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void count_kernel(
    const uint8_t* __restrict__ cols, int M, int64_t chunks, int splits, int atomic,
    const uint64_t* __restrict__ binom, uint32_t* __restrict__ out) {
  __shared__ __attribute__((aligned(16))) uint8_t buf[2][(kTH + kTL) * kRowBytes];
  __shared__ uint64_t base[kTH];  // rank of the row's set with no column; ~0 for padding rows
  __shared__ uint32_t lim[kTH];   // its columns: C(c, DL)
  const uint32_t nrow = (uint32_t)choose((uint32_t)M, DH);
  const uint32_t h0 = blockIdx.y * kTH, l0 = blockIdx.x * kTL;
  {
    int m[DH];
    row_modes<DH>(h0, M, m);
    if (l0 >= choose((uint32_t)m[0], DL)) return;  // no column of this tile is below c
  }
  // this thread's six 16-byte pieces of a chunk: rows tid / 4 + 64 i (256 of H, 128
  // of L), bytes 16 (tid % 4); offsets of their modes' columns
  const int piece = (threadIdx.x & 3) * 16, rt = threadIdx.x >> 2;
  uint32_t ho[4][DH], lo[2][DL];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t h = h0 + rt + 64 * i;
    int m[DH];
    row_modes<DH>(min(h, nrow - 1), M, m);
    uint64_t rank = 0;
#pragma unroll
    for (int j = 0; j < DH; ++j) {
      ho[i][j] = (uint32_t)m[j] * kChunkBytes + piece;
      rank += binom[(DL + j + 1) * kBinLd + m[j]];
    }
    if (piece == 0) {
      base[rt + 64 * i] = rank;
      lim[rt + 64 * i] = h < nrow ? (uint32_t)choose((uint32_t)m[0], DL) : 0u;
    }
  }
  const uint32_t ncol = (uint32_t)choose((uint32_t)(M - DH), DL);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    int m[DL];
    unrank_small<DL>(min(l0 + rt + 64 * i, ncol - 1), M - DH, m);
#pragma unroll
    for (int j = 0; j < DL; ++j) lo[i][j] = (uint32_t)m[j] * kChunkBytes + piece;
  }
  const int64_t c0 = chunks * blockIdx.z / splits, c1 = chunks * (blockIdx.z + 1) / splits;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int wh = (w & 1) * 128, wl = (w >> 1) * 64;  // the wave's part of the tile
  const uint64_t stride = (uint64_t)M * kChunkBytes;
  // One of the thread's six pieces at a time: loaded ahead of the products that
  // run meanwhile, ANDed and written after them.
  uint4v rh[DH], rl[DL];
  auto fetch_h = [&](int64_t c, int i) {
    const uint8_t* src = cols + (uint64_t)c * stride;
#pragma unroll
    for (int j = 0; j < DH; ++j) rh[j] = *reinterpret_cast<const uint4v*>(src + ho[i][j]);
  };
  auto fetch_l = [&](int64_t c, int i) {
    const uint8_t* src = cols + (uint64_t)c * stride;
#pragma unroll
    for (int j = 0; j < DL; ++j) rl[j] = *reinterpret_cast<const uint4v*>(src + lo[i][j]);
  };
  auto commit_h = [&](uint8_t* dst, int i) {
    uint4v v = rh[0];
#pragma unroll
    for (int j = 1; j < DH; ++j) v &= rh[j];
    *reinterpret_cast<uint4v*>(dst + (rt + 64 * i) * kRowBytes + piece) = v;
  };
  auto commit_l = [&](uint8_t* dst, int i) {
    uint4v v = rl[0];
#pragma unroll
    for (int j = 1; j < DL; ++j) v &= rl[j];
    *reinterpret_cast<uint4v*>(dst + (kTH + rt + 64 * i) * kRowBytes + piece) = v;
  };
  float16v acc[4][2] = {};
  if (c0 < c1) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      fetch_h(c0, i);
      commit_h(buf[0], i);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      fetch_l(c0, i);
      commit_l(buf[0], i);
    }
  }
  __syncthreads();
  for (int64_t c = c0; c < c1; ++c) {
    const uint8_t* cur = buf[(c - c0) & 1];
    uint8_t* nxt = buf[(c - c0 + 1) & 1];
    const int64_t cn = min(c + 1, c1 - 1);  // the last chunk stages itself again, unread
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      fetch_h(cn, 2 * kk);
      fetch_l(cn, kk);
      const int off = (lane & 31) * kRowBytes + kk * 32 + (lane >> 5) * 16;
      uint4v h[4], l[2];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        h[i] = *reinterpret_cast<const uint4v*>(cur + (wh + 32 * i) * kRowBytes + off);
#pragma unroll
      for (int j = 0; j < 2; ++j)
        l[j] = *reinterpret_cast<const uint4v*>(cur + (kTH + wl + 32 * j) * kRowBytes + off);
      count_step<0>(h, l, acc);
      count_step<1>(h, l, acc);
      commit_h(nxt, 2 * kk);
      commit_l(nxt, kk);
      fetch_h(cn, 2 * kk + 1);
      count_step<2>(h, l, acc);
      count_step<3>(h, l, acc);
      commit_h(nxt, 2 * kk + 1);
    }
    __syncthreads();
  }
  // accumulator v of a lane: row 8 (v / 4) + 4 (lane / 32) + v % 4, column lane % 32
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int h = wh + 32 * i + 8 * (v / 4) + 4 * (lane >> 5) + v % 4;
      const uint32_t n = lim[h];
      const uint64_t b = base[h];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const uint32_t r = l0 + wl + 32 * j + (lane & 31);
        if (r >= n) continue;
        const uint32_t k = (uint32_t)acc[i][j][v];
        if (atomic) atomicAdd(out + b + r, k); else out[b + r] = k;
      }
    }
}

// ---- k-statistics from the power sums ----
struct KstatCoef {
  double coef[52];             // c_N(tau) for the moment form (prod of s_B / N), partitions
                               // in make_parts order
};

struct CountTables {
  uint32_t* cnt[kMaxOrder + 1];  // power sums of order d, colex order
};

// The partitions of [D] in the order kstat_coefficients lists them (restricted
// growth strings in lexicographic order), each as its block masks in ascending
// order (0 = no block), built at compile time so that the kernel's loop over
// them unrolls with constant indices into the register array of moments.
template <int D>
struct PartTable {
  int n = 0;
  uint32_t blk[52][5] = {};
};

template <int D>
constexpr PartTable<D> make_parts() {
  PartTable<D> T;
  int lab[D] = {};
  for (;;) {
    uint32_t mk[D] = {};
    int nb = 0;
    for (int i = 0; i < D; ++i) {
      mk[lab[i]] |= 1u << i;
      nb = lab[i] + 1 > nb ? lab[i] + 1 : nb;
    }
    for (int i = 1; i < nb; ++i)  // ascending masks (insertion sort)
      for (int j = i; j > 0 && mk[j - 1] > mk[j]; --j) {
        const uint32_t t = mk[j];
        mk[j] = mk[j - 1];
        mk[j - 1] = t;
      }
    for (int b = 0; b < nb; ++b) T.blk[T.n][b] = mk[b];
    ++T.n;
    // next restricted growth string: the last position that can grow
    int i = D - 1;
    for (; i >= 1; --i) {
      int mx = 0;
      for (int j = 0; j < i; ++j) mx = lab[j] > mx ? lab[j] : mx;
      if (lab[i] <= mx) break;
    }
    if (i < 1) break;
    ++lab[i];
    for (int j = i + 1; j < D; ++j) lab[j] = 0;
  }
  return T;
}

template <int D>
__global__ void kstat_kernel(CountTables tab, int M, uint64_t count, const uint64_t* __restrict__ binom,
                             double invN, KstatCoef cf, double* __restrict__ out) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t r = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; r < count; r += stride) {
    int s[D];
    colex_unrank<D>(r, M, binom, kBinLd, s);
    double m[1 << D];
    m[0] = 1.0;
#pragma unroll
    for (int B = 1; B < (1 << D); ++B) {
      uint64_t rk = 0;
      int j = 0;
#pragma unroll
      for (int i = 0; i < D; ++i)
        if (B & (1 << i)) rk += binom[(++j) * kBinLd + s[i]];
      m[B] = (double)tab.cnt[popcount_c((unsigned)B)][rk] * invN;
    }
    constexpr PartTable<D> kParts = make_parts<D>();
    double k = 0.0, comp = 0.0;
#pragma unroll
    for (int t = 0; t < kParts.n; ++t) {
      double v = cf.coef[t];
#pragma unroll
      for (int b = 0; b < D; ++b) {
        const uint32_t blk = kParts.blk[t][b];
        if (blk) v *= m[blk];
      }
      const double y = k + v;  // compensated sum
      comp += (fabs(k) >= fabs(v)) ? ((k - y) + v) : ((v - y) + k);
      k = y;
    }
    out[r] = k + comp;
  }
}

// The same with the subsets {a} + B of one B (a < min B, consecutive ranks)
// sharing what does not depend on a.  Every partition of {a} + B is a block
// {a} + V, V a subset of B, and a partition of B \ V, so
//   k({a} + B) = sum_V m({a} + V) G_V(B),
//   G_V(B) = sum over the partitions tau whose block of a is {a} + V of
//            c_N(tau) prod of the other blocks' moments:
// 2^(D-1) loads and products per subset instead of 2^D - 1 and one product per
// partition (52 at D = 5).  A workgroup takes kStatB consecutive B's: their G_V
// and the ranks of V go to LDS, then half waves walk a for one
// B each.  All sums are compensated, as in kstat_kernel.
// D = 5, M = 144 (4.8e8 subsets): 6.2 ms against 22.8 of kstat_kernel.
constexpr int kStatB = 64;
template <int D>
__global__ __launch_bounds__(256) void kstat_shared_kernel(CountTables tab, int M, uint64_t nb,
                                                           const uint64_t* __restrict__ binom, double invN,
                                                           KstatCoef cf, double* __restrict__ out) {
  constexpr int NV = 1 << (D - 1);
  constexpr PartTable<D> kParts = make_parts<D>();
  __shared__ double g[NV][kStatB];
  __shared__ double mb[NV][kStatB];      // moments of B's subsets
  __shared__ uint64_t rank[NV][kStatB];  // of {a} + V is a + this, V non-empty; [0]: of {a} + B
  __shared__ int amax[kStatB];
  extern __shared__ uint64_t bin[];      // C(x, k), k <= D, x <= M
  const int ld = M + 1;
  for (int i = threadIdx.x; i < (D + 1) * ld; i += 256) bin[i] = binom[i / ld * kBinLd + i % ld];
  __syncthreads();
  const int qb = threadIdx.x & (kStatB - 1), part = threadIdx.x / kStatB;  // four waves share the V's of a B
  int s[D - 1];
  s[0] = 0;
  {
    const uint64_t rb = (uint64_t)blockIdx.x * kStatB + qb;
    if (rb < nb) colex_unrank_est<D - 1>(rb, M, bin, ld, s);
    if (part == 0) amax[qb] = s[0];
    if (s[0] > 0) {
#pragma unroll
      for (int B = 1; B < NV; ++B) {
        if (B % 4 != part) continue;
        uint64_t lo = 0, up = 0;  // ranks of B's subset alone and with a below it
        int j = 0;
#pragma unroll
        for (int i = 0; i < D - 1; ++i)
          if (B & (1 << i)) {
            ++j;
            lo += bin[j * ld + s[i]];
            up += bin[(j + 1) * ld + s[i]];
          }
        mb[B][qb] = (double)tab.cnt[popcount_c((unsigned)B)][lo] * invN;
        rank[B < NV - 1 ? B : 0][qb] = up;
      }
    }
  }
  __syncthreads();
  {
    if (s[0] > 0) {
      double m[NV];
      m[0] = 1.0;
#pragma unroll
      for (int B = 1; B < NV; ++B) m[B] = mb[B][qb];
#pragma unroll
      for (int V = 0; V < NV; ++V) {
        if (V / (NV / 4) != part) continue;
        double k = 0.0, comp = 0.0;
#pragma unroll
        for (int t = 0; t < kParts.n; ++t) {
          bool has = false;
          double v = cf.coef[t];
#pragma unroll
          for (int b = 0; b < D; ++b) {
            const uint32_t blk = kParts.blk[t][b];  // element 0 is a, element i + 1 is s[i]
            if (blk == (uint32_t)(2 * V + 1)) has = true;
            else if (blk) v *= m[blk >> 1];
          }
          if (!has) continue;
          const double y = k + v;
          comp += (fabs(k) >= fabs(v)) ? ((k - y) + v) : ((v - y) + k);
          k = y;
        }
        g[V][qb] = (k + comp) * invN;  // a's factor is a count
      }
    }
  }
  __syncthreads();
  const int lane = threadIdx.x & 31;
  for (int q = threadIdx.x >> 5; q < kStatB; q += 8) {
    const int na = amax[q];
    if (na == 0) continue;
    const uint64_t full = rank[0][q];
    for (int a = lane; a < na; a += 32) {
      double k = 0.0, comp = 0.0;
#pragma unroll
      for (int V = 0; V < NV; ++V) {
        const uint64_t rk = V == 0 ? 0 : V == NV - 1 ? full : rank[V][q];
        const double v = g[V][q] * (double)tab.cnt[popcount_c((unsigned)V) + 1][rk + a];
        const double y = k + v, z = y - k;
        comp += (k - (y - z)) + (v - z);  // the rounding of k + v
        k = y;
      }
      out[full + a] = k + comp;
    }
  }
}

// ---- Pearson coefficient: two passes of FP64 block reductions, fixed order ----

// Sum of v over the workgroup: lanes by the butterfly, then the waves in order;
// valid in every thread.
template <int WAVES>
__device__ __forceinline__ double block_total(double v, double (&sh)[WAVES]) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  __syncthreads();  // the previous call's sums have been read
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  double t = 0.0;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) t += sh[w];
  return t;
}

// Sums over this workgroup's elements: x and y, or with means the centred
// products.  part[q * gridDim.x + block].
__device__ __forceinline__ void pearson_sums(const double* __restrict__ x, const double* __restrict__ y, uint64_t n,
                                             uint64_t first, uint64_t step, double mx, double my, bool centered,
                                             double& a, double& b, double& c) {
  for (uint64_t i = first; i < n; i += step) {
    if (centered) {
      const double dx = x[i] - mx, dy = y[i] - my;
      a = fma(dx, dy, a);
      b = fma(dx, dx, b);
      c = fma(dy, dy, c);
    } else {
      a += x[i];
      b += y[i];
    }
  }
}

// Few elements: everything in one workgroup.  Up to kPearsonOne elements a
// second launch costs more than the one compute unit's bandwidth.
constexpr int kPearsonThreads = 1024;
constexpr uint64_t kPearsonOne = 16384;
constexpr uint64_t kPearsonBlocks = 1024;  // partial sums of the two-pass kernels
__global__ __launch_bounds__(kPearsonThreads) void pearson_one_kernel(const double* __restrict__ x,
                                                                      const double* __restrict__ y, uint64_t n,
                                                                      double* __restrict__ r) {
  __shared__ double sh[kPearsonThreads / 64];
  double a = 0.0, b = 0.0, c = 0.0;
  pearson_sums(x, y, n, threadIdx.x, kPearsonThreads, 0.0, 0.0, false, a, b, c);
  const double mx = block_total(a, sh) / (double)n, my = block_total(b, sh) / (double)n;
  a = b = c = 0.0;
  pearson_sums(x, y, n, threadIdx.x, kPearsonThreads, mx, my, true, a, b, c);
  a = block_total(a, sh);
  b = block_total(b, sh);
  c = block_total(c, sh);
  if (threadIdx.x == 0) r[0] = a / sqrt(b * c);
}

__global__ __launch_bounds__(kEstThreads) void pearson_means_kernel(const double* __restrict__ x,
                                                                    const double* __restrict__ y, uint64_t n,
                                                                    double* __restrict__ part) {
  __shared__ double sh[kEstThreads / 64];
  double a = 0.0, b = 0.0, c = 0.0;
  pearson_sums(x, y, n, (uint64_t)blockIdx.x * kEstThreads + threadIdx.x, (uint64_t)gridDim.x * kEstThreads, 0.0, 0.0,
               false, a, b, c);
  a = block_total(a, sh);
  b = block_total(b, sh);
  if (threadIdx.x == 0) {
    part[blockIdx.x] = a;
    part[gridDim.x + blockIdx.x] = b;
  }
}

// The total of m partial sums, in the same order in every workgroup.
__device__ __forceinline__ double total_of(const double* __restrict__ part, int m, double (&sh)[kEstThreads / 64]) {
  double t = 0.0;
  for (int i = threadIdx.x; i < m; i += kEstThreads) t += part[i];
  return block_total(t, sh);
}

// part: 2 x gridDim.x sums of the first pass, then 3 x gridDim.x of this one.
__global__ __launch_bounds__(kEstThreads) void pearson_centred_kernel(const double* __restrict__ x,
                                                                      const double* __restrict__ y, uint64_t n,
                                                                      double* __restrict__ part) {
  __shared__ double sh[kEstThreads / 64];
  const int m = (int)gridDim.x;
  const double mx = total_of(part, m, sh) / (double)n, my = total_of(part + m, m, sh) / (double)n;
  double a = 0.0, b = 0.0, c = 0.0;
  pearson_sums(x, y, n, (uint64_t)blockIdx.x * kEstThreads + threadIdx.x, (uint64_t)m * kEstThreads, mx, my, true, a,
               b, c);
  a = block_total(a, sh);
  b = block_total(b, sh);
  c = block_total(c, sh);
  if (threadIdx.x == 0) {
    part[2 * m + blockIdx.x] = a;
    part[3 * m + blockIdx.x] = b;
    part[4 * m + blockIdx.x] = c;
  }
}

__global__ __launch_bounds__(kEstThreads) void pearson_finish_kernel(const double* __restrict__ part, int m,
                                                                     double* __restrict__ r) {
  __shared__ double sh[kEstThreads / 64];
  const double a = total_of(part + 2 * m, m, sh), b = total_of(part + 3 * m, m, sh), c = total_of(part + 4 * m, m, sh);
  if (threadIdx.x == 0) r[0] = a / sqrt(b * c);
}

// Coefficients c_N(tau) N^|tau| of k(S) = sum_tau coef(tau) prod_{B in tau} (s_B / N).
void kstat_coefficients(int d, double N, KstatCoef* out) {
  // all partitions of [d] as label vectors (restricted growth strings)
  std::vector<std::vector<int>> parts;
  std::vector<int> lab(d, 0);
  std::function<void(int, int)> rec = [&](int i, int nb) {
    if (i == d) {
      parts.push_back(lab);
      return;
    }
    for (int b = 0; b <= nb; ++b) {
      lab[i] = b;
      rec(i + 1, std::max(nb, b + 1));
    }
  };
  rec(0, 0);
  auto nblocks = [](const std::vector<int>& l) {
    int m = 0;
    for (int v : l) m = std::max(m, v + 1);
    return m;
  };
  auto masks = [&](const std::vector<int>& l) {
    std::vector<uint32_t> mk(nblocks(l), 0u);
    for (int i = 0; i < (int)l.size(); ++i) mk[l[i]] |= 1u << i;
    std::sort(mk.begin(), mk.end());
    return mk;
  };
  std::vector<double> coef(parts.size(), 0.0);
  std::vector<std::vector<uint32_t>> pm(parts.size());
  for (size_t t = 0; t < parts.size(); ++t) pm[t] = masks(parts[t]);
  for (size_t pi = 0; pi < parts.size(); ++pi) {
    const int p = nblocks(parts[pi]);
    // w(pi) / (N)_p
    double fall = 1.0;
    for (int i = 0; i < p; ++i) fall *= (N - i);
    double fact = 1.0;
    for (int i = 2; i < p; ++i) fact *= i;
    const double w = ((p - 1) % 2 ? -fact : fact) / fall;
    // coarsenings sigma of the p blocks: partitions of [p]
    std::vector<int> sl(p, 0);
    std::function<void(int, int)> rs = [&](int i, int nb) {
      if (i == p) {
        // tau = union of pi's blocks by sigma's labels; Moebius factor
        std::vector<int> tl(d);
        for (int e = 0; e < d; ++e) tl[e] = sl[parts[pi][e]];
        std::vector<int> cnt(nb, 0);
        for (int j = 0; j < p; ++j) cnt[sl[j]]++;
        double mob = 1.0;
        for (int C = 0; C < nb; ++C) {
          double f = 1.0;
          for (int i2 = 2; i2 < cnt[C]; ++i2) f *= i2;
          mob *= ((cnt[C] - 1) % 2 ? -f : f);
        }
        const std::vector<uint32_t> tm = masks(tl);
        for (size_t t = 0; t < parts.size(); ++t)
          if (pm[t] == tm) {
            coef[t] += w * mob;
            break;
          }
        return;
      }
      for (int b = 0; b <= nb; ++b) {
        sl[i] = b;
        rs(i + 1, std::max(nb, b + 1));
      }
    };
    rs(0, 0);
  }
  for (size_t t = 0; t < parts.size(); ++t) {
    double Np = 1.0;
    for (size_t b = 0; b < pm[t].size(); ++b) Np *= N;
    out->coef[t] = coef[t] * Np;
  }
}

// Power sums of order DL + DH.  Tiles past the last needed column leave at once.
// The samples are split over more workgroups while the tiles alone are fewer
// than two rounds of what runs at once (two workgroups per compute unit).
template <int DL, int DH>
hipError_t launch_counts(const uint64_t* cols, int M, int64_t chunks, const uint64_t* binom, uint32_t* out,
                         hipStream_t s) {
  if (M < DL + DH) return hipSuccess;
  const uint64_t nrow = host_binom(M, DH), ncol = host_binom(M - DH, DL);
  uint64_t tiles = 0;
  for (uint64_t h = 0; h < nrow; h += kTH) {
    int m[DH];
    row_modes<DH>((uint32_t)h, M, m);
    tiles += (host_binom(m[0], DL) + kTL - 1) / kTL;
  }
  const int64_t want = (1024 + (int64_t)tiles - 1) / (int64_t)tiles;
  const int64_t exact = (chunks * 64 * kChunkWords + kSplitSamples - 1) / kSplitSamples;
  const int splits = (int)std::max<int64_t>(exact, std::min<int64_t>(want, (chunks + 3) / 4));
  if (splits > 1) {
    const uint64_t n = host_binom(M, DL + DH);
    hipLaunchKernelGGL(zero_counts_kernel, dim3((unsigned)std::min<uint64_t>((n + 255) / 256, 4096)), dim3(256), 0, s,
                       out, n);
  }
  hipLaunchKernelGGL((count_kernel<DL, DH>),
                     dim3((unsigned)((ncol + kTL - 1) / kTL), (unsigned)((nrow + kTH - 1) / kTH), (unsigned)splits),
                     dim3(kEstThreads), 0, s, reinterpret_cast<const uint8_t*>(cols), M, chunks, splits, splits > 1,
                     binom, out);
  return hipGetLastError();
}

template <int D>
hipError_t launch_kstat(const CountTables& tab, int M, int64_t N, const uint64_t* binom, double* out, hipStream_t s) {
  KstatCoef cf{};
  kstat_coefficients(D, (double)N, &cf);
  if constexpr (D >= 4) {
    const uint64_t nb = host_binom(M, D - 1);
    hipLaunchKernelGGL(kstat_shared_kernel<D>, dim3((unsigned)((nb + kStatB - 1) / kStatB)), dim3(256),
                       (size_t)(D + 1) * (M + 1) * sizeof(uint64_t), s, tab, M,
                       nb, binom, 1.0 / (double)N, cf, out + gbs_order_offset(M, D));
  } else {
    const uint64_t count = host_binom(M, D);
    hipLaunchKernelGGL(kstat_kernel<D>, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, tab, M, count, binom,
                       1.0 / (double)N, cf, out + gbs_order_offset(M, D));
  }
  return hipGetLastError();
}

// Scratch of one call: the bit columns, then the counts of each order.
struct EstScratch {
  int64_t chunks;
  size_t cnt[kMaxOrder + 1];
  size_t bytes;
  static EstScratch make(int M, int64_t N, int K) {
    auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
    EstScratch S{};
    S.chunks = (N + 64 * kChunkWords - 1) / (64 * kChunkWords);
    S.bytes = al((size_t)M * (size_t)S.chunks * kChunkBytes);
    for (int d = 1; d <= K; ++d) {
      S.cnt[d] = S.bytes;
      S.bytes += al(host_binom(M, d) * sizeof(uint32_t));
    }
    return S;
  }
};

}  // namespace

size_t estimator_scratch(int M, int64_t N, int K) { return EstScratch::make(M, N, K).bytes; }

// Power sums and k-statistics of orders 1..K from nsamples samples.
hipError_t run_sample_cumulants(int M, int64_t N, const uint8_t* bits, int K,
                                const uint64_t* binom, double* out, void* lent, hipStream_t s) {
  const EstScratch S = EstScratch::make(M, N, K);
  void* scratch = lent;
  hipError_t e = hipSuccess;
  if (!lent) e = hipMallocAsync(&scratch, S.bytes, s);
  if (e != hipSuccess) return e;
  char* b = static_cast<char*>(scratch);
  uint64_t* cols = reinterpret_cast<uint64_t*>(b);
  CountTables tab{};
  for (int d = 1; d <= K; ++d) tab.cnt[d] = reinterpret_cast<uint32_t*>(b + S.cnt[d]);
  const int64_t words = S.chunks * kChunkWords;
  // 2^32 threads in one dimension of a launch (N near 2^32) would be refused
  const int64_t packs = (words * 64 + kPackSamples - 1) / kPackSamples, wide = std::min<int64_t>(packs, 1 << 20);
  hipLaunchKernelGGL(pack_columns_kernel, dim3((unsigned)wide, (unsigned)((packs + wide - 1) / wide)),
                     dim3(kPackSamples), (size_t)kPackSamples * M, s, bits, N, M, words, ((uintptr_t)bits & 3) == 0,
                     cols);
  e = hipGetLastError();
  if (e == hipSuccess) {
    hipLaunchKernelGGL(count1_kernel, dim3(M), dim3(kEstThreads), 0, s, cols, M, words, tab.cnt[1]);
    e = hipGetLastError();
  }
  if (e == hipSuccess && K >= 2) e = launch_counts<1, 1>(cols, M, S.chunks, binom, tab.cnt[2], s);
  if (e == hipSuccess && K >= 3) e = launch_counts<1, 2>(cols, M, S.chunks, binom, tab.cnt[3], s);
  if (e == hipSuccess && K >= 4) e = launch_counts<2, 2>(cols, M, S.chunks, binom, tab.cnt[4], s);
  if (e == hipSuccess && K >= 5) e = launch_counts<2, 3>(cols, M, S.chunks, binom, tab.cnt[5], s);
  if (e == hipSuccess) e = launch_kstat<1>(tab, M, N, binom, out, s);
  if (e == hipSuccess && K >= 2) e = launch_kstat<2>(tab, M, N, binom, out, s);
  if (e == hipSuccess && K >= 3) e = launch_kstat<3>(tab, M, N, binom, out, s);
  if (e == hipSuccess && K >= 4) e = launch_kstat<4>(tab, M, N, binom, out, s);
  if (e == hipSuccess && K >= 5) e = launch_kstat<5>(tab, M, N, binom, out, s);
  hipError_t f = lent ? hipSuccess : hipFreeAsync(scratch, s);
  return e != hipSuccess ? e : f;
}

size_t pearson_scratch() { return 5 * (size_t)kPearsonBlocks * sizeof(double); }

hipError_t run_pearson(uint64_t n, const double* x, const double* y, double* r, void* lent, hipStream_t s) {
  if (n <= kPearsonOne) {
    hipLaunchKernelGGL(pearson_one_kernel, dim3(1), dim3(kPearsonThreads), 0, s, x, y, n, r);
    return hipGetLastError();
  }
  const int nblk = (int)std::min<uint64_t>((n + kEstThreads - 1) / kEstThreads, kPearsonBlocks);
  void* scratch = lent;
  hipError_t e = hipSuccess;
  if (!lent) e = hipMallocAsync(&scratch, pearson_scratch(), s);
  if (e != hipSuccess) return e;
  double* part = static_cast<double*>(scratch);
  hipLaunchKernelGGL(pearson_means_kernel, dim3(nblk), dim3(kEstThreads), 0, s, x, y, n, part);
  hipLaunchKernelGGL(pearson_centred_kernel, dim3(nblk), dim3(kEstThreads), 0, s, x, y, n, part);
  hipLaunchKernelGGL(pearson_finish_kernel, dim3(1), dim3(kEstThreads), 0, s, part, nblk, r);
  e = hipGetLastError();
  hipError_t f = lent ? hipSuccess : hipFreeAsync(scratch, s);
  return e != hipSuccess ? e : f;
}

}  // namespace gbs
