// The FP64 matrix product of the step-by-step samplers: rows are cumulant rows
// (inner index consecutive in memory), columns the 64 samples of a block.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gbs {

typedef double double4 __attribute__((ext_vector_type(4)));
typedef double double2v __attribute__((ext_vector_type(2)));

constexpr int kSB = 64;        // samples per block of the tables
constexpr int kKC = 16;        // inner indices per operand chunk
constexpr int kLdB = kSB + 4;  // LDS row of an operand chunk (rows 4 apart fall on other banks)

// 64 rows x 64 samples of a product per workgroup of 4 KS waves: wave w owns
// rows 16 (w % 4).. + 15, all 64 samples (four 16 x 16 FP64 tiles) and every
// KS-th chunk of the inner index; the KS partial tiles are added in a fixed
// order through LDS.  The rows' cumulants go from memory straight to registers
// (a lane's four inner indices are consecutive); the samples' operand is shared
// by the waves through LDS, double-buffered.
//   row_kap(r)   first cumulant of row r
//   operand(k)   the 64 samples of inner index k, or null for zeros
//   dest(r)      where row r's 64 sums go
template <int KS, class RowKap, class Op, class Dest>
__device__ __forceinline__ void product_block(int r_block, int rows, int L, RowKap row_kap, Op operand,
                                              Dest dest, double (&Bs)[2][KS][kKC][kLdB]) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int g = lane >> 4, c16 = lane & 15, wr = w & 3, wk = w >> 2;
  const int r0 = r_block * 64 + wr * 16;
  const bool busy = r0 < rows;  // a wave of padding rows only shares the loads
  const double* ka = row_kap(min(r0 + c16, rows - 1));
  // this thread's share of an operand chunk: row kr, columns kc..kc + 3 of chunk wk
  const int kr = (threadIdx.x & 255) >> 4, kc = (threadIdx.x & 15) * 4;
  auto load_b = [&](int k0, double2v& b0, double2v& b1) {
    const int k = k0 + kr;
    b0 = double2v{0.0, 0.0};
    b1 = b0;
    const double* p = k < L ? operand(k) : nullptr;
    if (!p) return;
    p += kc;
    b0 = *reinterpret_cast<const double2v*>(p);
    b1 = *reinterpret_cast<const double2v*>(p + 2);
  };
  auto load_a = [&](int k0, double (&a)[4]) {
    const int k = k0 + 4 * g;
    if (k0 + kKC <= L) {
#pragma unroll
      for (int t = 0; t < 4; ++t) a[t] = ka[k + t];
    } else {
#pragma unroll
      for (int t = 0; t < 4; ++t) a[t] = k + t < L ? ka[k + t] : 0.0;
    }
  };
  double4 acc[4] = {};
  double a[4], an[4] = {};
  double2v b0, b1;
  load_b(wk * kKC, b0, b1);
  load_a(wk * kKC, a);
  const int nch = (L + kKC * KS - 1) / (kKC * KS);
  for (int c = 0; c < nch; ++c) {
    double (&S)[kKC][kLdB] = Bs[c & 1][wk];
    *reinterpret_cast<double2v*>(&S[kr][kc]) = b0;
    *reinterpret_cast<double2v*>(&S[kr][kc + 2]) = b1;
    __syncthreads();
    if (c + 1 < nch) {
      load_b(((c + 1) * KS + wk) * kKC, b0, b1);
      load_a(((c + 1) * KS + wk) * kKC, an);
    }
    if (busy) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
#pragma unroll
        for (int ct = 0; ct < 4; ++ct)
          acc[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t], S[4 * g + t][ct * 16 + c16], acc[ct], 0, 0, 0);
      }
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) a[t] = an[t];
  }
  if constexpr (KS > 1) {
    double* red = &Bs[0][0][0][0];  // KS / 2 x 64 x 64 fits the operand buffers
    for (int half = KS / 2; half >= 1; half /= 2) {
      __syncthreads();
      if (wk >= half && wk < 2 * half) {
#pragma unroll
        for (int ct = 0; ct < 4; ++ct)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            red[(((wk - half) * 4 + wr) * 16 + ct * 4 + v) * 64 + lane] = acc[ct][v];
      }
      __syncthreads();
      if (wk < half) {
#pragma unroll
        for (int ct = 0; ct < 4; ++ct)
#pragma unroll
          for (int v = 0; v < 4; ++v) acc[ct][v] += red[((wk * 4 + wr) * 16 + ct * 4 + v) * 64 + lane];
      }
    }
    if (wk != 0) return;
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int r = r0 + g + 4 * v;
    if (r >= rows) continue;
    double* o = dest(r) + c16;
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) o[ct * 16] = acc[ct][v];
  }
}

}  // namespace gbs
