// Exclusive scans of int32 arrays for the set-up's tables: per block of kScanItems
// items, then the blocks' totals in one work-group, then written out by a kernel
// of the caller's (scan_apply). With FLAG the items are (value, 1 if value > 0)
// pairs, sums in the low word and counts in the high one (values adding up to
// less than 2^32); without, 64-bit sums.
#pragma once

#include <hip/hip_runtime.h>

#include "aim_internal.h"

namespace aim {
namespace {

__global__ void k_clear(int32_t *p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

constexpr int kScanThreads = 256, kScanPer = 8, kScanItems = kScanThreads * kScanPer;
inline int64_t scan_blocks(int64_t count) { return (count + kScanItems - 1) / kScanItems; }

template <bool FLAG>
__device__ inline uint64_t scan_item(int32_t v) {
  return (uint64_t)(uint32_t)v | (FLAG && v > 0 ? 1ull << 32 : 0);
}
__device__ inline uint64_t block_exclusive(uint64_t mine, uint64_t *total) {
  __shared__ uint64_t ws[kScanThreads / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint64_t scan = mine;
  for (int off = 1; off < 64; off <<= 1) {
    const uint64_t o = __shfl_up((unsigned long long)scan, off, 64);
    if (lane >= off) scan += o;
  }
  __syncthreads();
  if (lane == 63) ws[wave] = scan;
  __syncthreads();
  uint64_t before = 0, all = 0;
  for (int w = 0; w < kScanThreads / 64; ++w) {
    if (w < wave) before += ws[w];
    all += ws[w];
  }
  *total = all;
  return before + scan - mine;
}
template <bool FLAG>
__global__ void __launch_bounds__(kScanThreads)
    k_scan_blocks(const int32_t *v, int64_t n, uint64_t *sums) {
  const int64_t i0 = (int64_t)blockIdx.x * kScanItems + (int64_t)threadIdx.x * kScanPer;
  uint64_t mine = 0, total;
  for (int k = 0; k < kScanPer; ++k)
    if (i0 + k < n) mine += scan_item<FLAG>(v[i0 + k]);
  (void)block_exclusive(mine, &total);
  if (threadIdx.x == 0) sums[blockIdx.x] = total;
}
// sums[0 .. nb) to exclusive prefixes, sums[nb] the total
__global__ void __launch_bounds__(kScanThreads) k_scan_sums(uint64_t *sums, int64_t nb) {
  uint64_t carry = 0;
  for (int64_t b0 = 0; b0 < nb; b0 += kScanThreads) {
    const int64_t b = b0 + threadIdx.x;
    uint64_t total;
    const uint64_t ex = block_exclusive(b < nb ? sums[b] : 0, &total);
    if (b < nb) sums[b] = carry + ex;
    carry += total;
  }
  if (threadIdx.x == 0) sums[nb] = carry;
}
// In a launch of scan_blocks(n) x kScanThreads: f(i, value, exclusive prefix)
template <bool FLAG, class F>
__device__ inline void scan_apply(const int32_t *v, int64_t n, const uint64_t *sums, F f) {
  const int64_t i0 = (int64_t)blockIdx.x * kScanItems + (int64_t)threadIdx.x * kScanPer;
  int32_t x[kScanPer];
  uint64_t mine = 0, total;
  for (int k = 0; k < kScanPer; ++k) {
    x[k] = i0 + k < n ? v[i0 + k] : 0;
    mine += scan_item<FLAG>(x[k]);
  }
  uint64_t ex = sums[blockIdx.x] + block_exclusive(mine, &total);
  for (int k = 0; k < kScanPer; ++k) {
    if (i0 + k < n) f(i0 + k, x[k], ex);
    ex += scan_item<FLAG>(x[k]);
  }
}
// the block prefixes of v[0 .. count) into sums (scan_blocks(count) + 1 words);
// returns the total (synchronises s)
template <bool FLAG>
uint64_t scan_sums(const int32_t *v, int64_t count, uint64_t *sums, hipStream_t s) {
  const int64_t nb = scan_blocks(count);
  hipLaunchKernelGGL(k_scan_blocks<FLAG>, dim3((unsigned)nb), dim3(kScanThreads), 0, s, v, count,
                     sums);
  LAUNCHCHECK();
  hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(kScanThreads), 0, s, sums, nb);
  LAUNCHCHECK();
  uint64_t total = 0;
  HIPCHECK(hipMemcpyAsync(&total, sums + nb, sizeof(total), hipMemcpyDeviceToHost, s));
  HIPCHECK(hipStreamSynchronize(s));
  return total;
}

}  // namespace
}  // namespace aim
