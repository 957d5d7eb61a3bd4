// Shared by the sampler kernels: colex ranks of 1-based bits and the interface
// of the step-by-step double-elision path.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gbs {

__host__ __device__ constexpr uint32_t samp_c2(uint32_t x) { return x * (x - 1) / 2; }
__host__ __device__ constexpr uint32_t samp_c3(uint32_t x) {
  return x < 3 ? 0u : x * (x - 1) * (x - 2) / 6;
}

// C(x - 1, k): the part of bit x (1-based) at position k of a colex rank
__host__ __device__ constexpr uint32_t samp_r1(int x) { return (uint32_t)x - 1; }
__host__ __device__ constexpr uint32_t samp_r2(int x) { return samp_c2((uint32_t)x - 1); }
__host__ __device__ constexpr uint32_t samp_r3(int x) { return samp_c3((uint32_t)x - 1); }
__host__ __device__ constexpr uint32_t samp_r4(int x) {
  const uint32_t y = (uint32_t)x - 1;
  return y < 4 ? 0u : y * (y - 1) * (y - 2) * (y - 3) / 24;
}
__host__ __device__ constexpr uint32_t samp_r5(int x) {
  const uint64_t y = (uint64_t)x - 1;
  return y < 5 ? 0u : (uint32_t)(y * (y - 1) * (y - 2) * (y - 3) * (y - 4) / 120);
}

struct KapOffsets {
  uint32_t off[6];  // start of the order-d block of the cumulant array
};

// Double elision step by step (gbs_sampler_double.hip): bytes of tables per
// sample (a multiple of 64 samples is stored), and the launches of one batch of
// nsamp samples on tables tab.  u, cond: row stride ldu, the samples of the whole call.
size_t double_sampler_bytes(int M);
hipError_t launch_double_sampler(int M, const double* kap, KapOffsets ko, int64_t nsamp, const double* u,
                                 uint64_t ldu, double* tab, uint8_t* bits, double* prob, double* cond,
                                 hipStream_t s);
// The same for single elision (gbs_sampler_single.hip).
size_t single_sampler_bytes(int M);
hipError_t launch_single_sampler(int M, const double* kap, KapOffsets ko, int64_t nsamp, const double* u,
                                 uint64_t ldu, double* tab, uint8_t* bits, double* prob, double* cond,
                                 hipStream_t s);

}  // namespace gbs
