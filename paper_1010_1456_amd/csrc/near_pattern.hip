// Near-zone CSR pattern of a plan on the GPU: the pairs |c_m - c_n| <= r_near, as
// the host planner lists them (the same cells, and the same distances in the same
// order of operations without fused multiply-adds, so the same pairs). A wave takes
// a row: the bases of the 3 x 3 runs of cells around it, counted, then written, then
// put in increasing order by rank. 16 host threads and the upload of the columns
// took 13 ms on the 4-lambda sphere (4.4 M pairs) and 0.66 s on the 128-lambda
// plate (285 M); this takes 0.4 and 25 ms.
#include <algorithm>
#include <cmath>

#include "aim_internal.h"
#include "scan.h"

namespace aim {

namespace {

struct Cells {
  double b[3], size;  // lowest centre, cell size
  int nc[3], reach;
  double r2;
  __device__ int index(const double *c, int d) const {
    const int v = (int)floor((c[d] - b[d]) / size);
    return min(max(v, 0), nc[d] - 1);
  }
};

__global__ void k_cell_count(const double *centre, int64_t n, Cells ce, int32_t *cell_of,
                             int32_t *count) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double *c = centre + 3 * i;
  const int32_t k = (ce.index(c, 0) * ce.nc[1] + ce.index(c, 1)) * ce.nc[2] + ce.index(c, 2);
  cell_of[i] = k;
  atomicAdd(&count[k], 1);
}
// starts[i] = exclusive prefix; count (if given) becomes the fill cursor
__global__ void __launch_bounds__(kScanThreads)
    k_starts(int32_t *count, int64_t n, const uint64_t *sums, int64_t nb, int32_t *starts,
             bool cursor) {
  scan_apply<false>(count, n, sums, [&](int64_t i, int32_t, uint64_t ex) {
    starts[i] = (int32_t)ex;
    if (cursor) count[i] = (int32_t)ex;
  });
  if (blockIdx.x == 0 && threadIdx.x == 0) starts[n] = (int32_t)sums[nb];
}
__global__ void k_cell_fill(const int32_t *cell_of, int64_t n, int32_t *cursor, int32_t *members) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) members[atomicAdd(&cursor[cell_of[i]], 1)] = (int32_t)i;
}

// Row m = wave: the bases near it, counted (WRITE false) or written from
// rowptr[m] in the order found
template <bool WRITE>
__global__ void __launch_bounds__(256)
    k_near_rows(const double *__restrict__ centre, int64_t n, int64_t group0, Cells ce,
                const int32_t *__restrict__ cstart, const int32_t *__restrict__ members,
                int32_t *count, const int32_t *rowptr, int32_t *cols) {
#pragma clang fp contract(off)
  const int lane = threadIdx.x & 63;
  const int64_t m = (group0 + blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (m >= n) return;
  const double cm[3] = {centre[3 * m], centre[3 * m + 1], centre[3 * m + 2]};
  const int c0 = ce.index(cm, 0), c1 = ce.index(cm, 1), c2 = ce.index(cm, 2);
  const int z0 = max(0, c2 - ce.reach), z1 = min(ce.nc[2] - 1, c2 + ce.reach);
  int found = WRITE ? rowptr[m] : 0;
  for (int a = max(0, c0 - ce.reach); a <= min(ce.nc[0] - 1, c0 + ce.reach); ++a)
    for (int b = max(0, c1 - ce.reach); b <= min(ce.nc[1] - 1, c1 + ce.reach); ++b) {
      const int row = (a * ce.nc[1] + b) * ce.nc[2];
      const int s0 = cstart[row + z0], s1 = cstart[row + z1 + 1];  // cells along z adjoin
      for (int s = s0; s < s1; s += 64) {
        bool near = false;
        int j = 0;
        if (s + lane < s1) {
          j = members[s + lane];
          const double d0 = cm[0] - centre[3 * (int64_t)j], d1 = cm[1] - centre[3 * (int64_t)j + 1],
                       d2 = cm[2] - centre[3 * (int64_t)j + 2];
          const double dd = d0 * d0 + d1 * d1 + d2 * d2;
          near = dd <= ce.r2 || j == m;
        }
        const unsigned long long hit = __ballot(near);
        if (WRITE && near) cols[found + __popcll(hit & ((1ull << lane) - 1))] = j;
        found += __popcll(hit);
      }
    }
  if (!WRITE && lane == 0) count[m] = found;
}

// Row m = wave: its columns (distinct) in increasing order, each placed by the
// number of smaller ones, read 64 at a time
__global__ void __launch_bounds__(256)
    k_sort_rows(const int32_t *__restrict__ in, const int32_t *__restrict__ rowptr, int64_t n,
                int64_t group0, int32_t *__restrict__ out) {
  const int lane = threadIdx.x & 63;
  const int64_t m = (group0 + blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (m >= n) return;
  const int e0 = rowptr[m], e1 = rowptr[m + 1];
  for (int e = e0; e < e1; e += 64) {
    const int mine = e + lane < e1 ? in[e + lane] : INT32_MAX;
    int rank = 0;
    for (int f = e0; f < e1; f += 64) {
      const int other = f + lane < e1 ? in[f + lane] : INT32_MAX;
      const int cnt = min(64, e1 - f);
      for (int k = 0; k < cnt; ++k) rank += __builtin_amdgcn_readlane(other, k) < mine;
    }
    if (e + lane < e1) out[e0 + rank] = mine;
  }
}

}  // namespace

void near_pattern_mesh(Plan *pl, MeshDev &md, hipStream_t s) {
  HostPlan &h = md.hp;
  const int64_t n = h.n;
  const NearCells hc = near_cells(h);
  Cells ce{};
  int64_t ncell = 1;
  for (int c = 0; c < 3; ++c) {
    ce.b[c] = hc.lo[c];
    ce.nc[c] = hc.nc[c];
    ncell *= hc.nc[c];
  }
  ce.size = hc.size;
  ce.reach = hc.reach;
  ce.r2 = h.r_near * h.r_near;
  std::vector<void *> tmp;
  auto ints = [&](int64_t count) {
    void *p = dev_alloc(pl, sizeof(int32_t) * (size_t)std::max<int64_t>(count, 1));
    tmp.push_back(p);
    return (int32_t *)p;
  };
  double *centre = (double *)dev_alloc(pl, sizeof(double) * 3 * n);
  tmp.push_back(centre);
  uint64_t *sums =
      (uint64_t *)dev_alloc(pl, sizeof(uint64_t) * (scan_blocks(std::max(ncell, n)) + 1));
  tmp.push_back(sums);
  HIPCHECK(hipMemcpyAsync(centre, h.centre.data(), sizeof(double) * 3 * n, hipMemcpyHostToDevice, s));
  int32_t *count = ints(std::max(ncell, n)), *cell_of = ints(n), *cstart = ints(ncell + 1),
          *members = ints(n);
  hipLaunchKernelGGL(k_clear, dim3(launch_blocks(ncell, 256)), dim3(256), 0, s, count, ncell);
  LAUNCHCHECK();
  hipLaunchKernelGGL(k_cell_count, dim3(launch_blocks(n, 256)), dim3(256), 0, s, centre, n, ce,
                     cell_of, count);
  LAUNCHCHECK();
  (void)scan_sums<false>(count, ncell, sums, s);
  hipLaunchKernelGGL(k_starts, dim3((unsigned)scan_blocks(ncell)), dim3(kScanThreads), 0, s, count,
                     ncell, sums, scan_blocks(ncell), cstart, true);
  LAUNCHCHECK();
  hipLaunchKernelGGL(k_cell_fill, dim3(launch_blocks(n, 256)), dim3(256), 0, s, cell_of, n, count,
                     members);
  LAUNCHCHECK();
  const int64_t row_groups = (n + 3) / 4;
  for_launches(row_groups, [&](int64_t g0, unsigned groups) {
    hipLaunchKernelGGL(k_near_rows<false>, dim3(groups), dim3(256), 0, s, centre, n, g0, ce, cstart,
                       members, count, nullptr, nullptr);
    LAUNCHCHECK();
  });
  const uint64_t nnz = scan_sums<false>(count, n, sums, s);
  if (nnz > (uint64_t)INT32_MAX)
    throw Error(AIM_ERR_ARG, "near zone too large for 32-bit indexing");
  h.nnz = (int64_t)nnz;
  md.rowptr = (int32_t *)dev_alloc(pl, sizeof(int32_t) * (n + 1));
  hipLaunchKernelGGL(k_starts, dim3((unsigned)scan_blocks(n)), dim3(kScanThreads), 0, s, count, n,
                     sums, scan_blocks(n), md.rowptr, false);
  LAUNCHCHECK();
  int32_t *found = ints(h.nnz);
  md.cols = (int32_t *)dev_alloc(pl, sizeof(int32_t) * std::max<int64_t>(h.nnz, 1));
  for_launches(row_groups, [&](int64_t g0, unsigned groups) {
    hipLaunchKernelGGL(k_near_rows<true>, dim3(groups), dim3(256), 0, s, centre, n, g0, ce, cstart,
                       members, nullptr, md.rowptr, found);
    LAUNCHCHECK();
  });
  for_launches(row_groups, [&](int64_t g0, unsigned groups) {
    hipLaunchKernelGGL(k_sort_rows, dim3(groups), dim3(256), 0, s, found, md.rowptr, n, g0, md.cols);
    LAUNCHCHECK();
  });
  HIPCHECK(hipStreamSynchronize(s));
  for (void *p : tmp) dev_free(pl, p);
}

}  // namespace aim
