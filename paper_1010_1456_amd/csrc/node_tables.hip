// Set-up tables by grid node: the transposed (node-ordered) projection that the
// gather form of anterpolation walks, and the occupied nodes and z lines that the
// product's passes are pruned to. All built on the GPU: a histogram of the
// non-zero stencil weights by node, scans, and a counting sort whose lists are
// then ordered, so that the tables do not depend on the order of the atomics. On
// the host (one thread, after copying the weights' mask back) they took 53 ms on
// the 8-lambda sphere and 345 ms on the 128-lambda plate.
#include <algorithm>

#include "aim_internal.h"
#include "scan.h"

namespace aim {

namespace {

// whether basis b has any non-zero weight at its stencil node u: projection or,
// for the combined field, curl weight (the node is then read by the
// interpolation even where its projection weights vanish, as off a flat face
// lying in a grid plane)
__device__ inline bool weighs(const double *lam, const double *curl, int64_t b, int u, int K) {
  bool nz = false;
  for (int q = 0; q < 4; ++q) nz |= lam[(b * 4 + q) * K + u] != 0.0;
  if (curl)
    for (int e = 0; e < 3; ++e) nz |= curl[(b * 3 + e) * K + u] != 0.0;
  return nz;
}

// count[v]: non-zero (basis, stencil node) weights at grid node v
__global__ void k_count(const double *lam, const double *curl, const int32_t *anchor_lin,
                        const int32_t *soff, int64_t n, int K, int32_t *count) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n * K) return;
  const int64_t b = t / K;
  const int u = (int)(t - b * K);
  if (weighs(lam, curl, b, u, K)) atomicAdd(&count[anchor_lin[b] + soff[u]], 1);
}

// the entries into their nodes' ranges, cursor[v] the next free place of node v
__global__ void k_fill(const double *lam, const double *curl, const int32_t *anchor_lin,
                       const int32_t *soff, int64_t n, int K, int32_t *cursor, int32_t *src) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n * K) return;
  const int64_t b = t / K;
  const int u = (int)(t - b * K);
  if (weighs(lam, curl, b, u, K)) src[atomicAdd(&cursor[anchor_lin[b] + soff[u]], 1)] = (int32_t)t;
}

// Each occupied node's entries in increasing order (basis, then stencil node). A
// node has one entry per basis whose stencil holds it: some 20 on a lambda/9 mesh
// with a lambda/10 grid, hundreds to thousands on finer meshes, all n on a body of
// a few grid cells. Lists of up to kShortList go to a thread each, by insertion;
// longer ones are left to k_order_long through long_list.
constexpr int kShortList = 64;
__global__ void k_order(const int32_t *occ_ptr, int64_t n_occ, int32_t *src, int32_t *long_list,
                        int32_t *n_long) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_occ) return;
  const int e0 = occ_ptr[i], e1 = occ_ptr[i + 1];
  if (e1 - e0 > kShortList) {
    long_list[atomicAdd(n_long, 1)] = (int32_t)i;
    return;
  }
  for (int e = e0 + 1; e < e1; ++e) {
    const int32_t v = src[e];
    int p = e;
    while (p > e0 && src[p - 1] > v) {
      src[p] = src[p - 1];
      --p;
    }
    src[p] = v;
  }
}
// The long lists, a work-group each: a stable counting sort by four bits at a time
// (each thread counts, then places, a run of the list; counters [digit][thread] in
// LDS), so the time is linear in the list's length: all of the set-up's projection
// phase takes 1.2 ms for 14 520 unknowns on a body of a few nodes and 6.3 ms for
// 100 920 there, where insertion would take n^2 / 4 dependent steps. On lists of some
// 20 the launch costs nothing that shows (4-lambda sphere 1.29 ms with and without).
// `bits` of the values, in pairs of digits, so that the result is back in src.
constexpr int kBins = 16;
constexpr int kSortGroups = 2048;  // work-groups (8 per CU) that share the long lists
__global__ void __launch_bounds__(kScanThreads)
    k_order_long(const int32_t *occ_ptr, const int32_t *long_list, const int32_t *n_long, int bits,
                 int32_t *src, int32_t *tmp) {
  __shared__ int32_t cnt[kBins * kScanThreads];
  const int tid = threadIdx.x;
  const int lists = *n_long;
  for (int l = blockIdx.x; l < lists; l += gridDim.x) {
    const int e0 = occ_ptr[long_list[l]], len = occ_ptr[long_list[l] + 1] - e0;
    const int per = (len + kScanThreads - 1) / kScanThreads;
    const int k0 = min(tid * per, len), k1 = min(k0 + per, len);
    int32_t *a = src + e0, *b = tmp + e0;
    for (int shift = 0; shift < bits || (shift / 4) % 2; shift += 4) {
      for (int d = 0; d < kBins; ++d) cnt[d * kScanThreads + tid] = 0;
      for (int k = k0; k < k1; ++k) ++cnt[((a[k] >> shift) & (kBins - 1)) * kScanThreads + tid];
      __syncthreads();
      uint64_t sum = 0, total;
      for (int q = 0; q < kBins; ++q) sum += cnt[tid * kBins + q];
      int32_t before = (int32_t)block_exclusive(sum, &total);
      for (int q = 0; q < kBins; ++q) {
        const int32_t c = cnt[tid * kBins + q];
        cnt[tid * kBins + q] = before;
        before += c;
      }
      __syncthreads();
      for (int k = k0; k < k1; ++k) {
        const int32_t v = a[k];
        b[cnt[((v >> shift) & (kBins - 1)) * kScanThreads + tid]++] = v;
      }
      __syncthreads();
      int32_t *const t = a;
      a = b;
      b = t;
    }
  }
}

// entry e with src[e] = b K + u: its basis b and lamT[e][q] = Lambda[b][q][u]
__global__ void k_lam_transpose(const double *lam, const int32_t *src, int64_t ne, int K,
                                int32_t *col, double *lamT64, float *lamT32) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= ne) return;
  const int b = src[e] / K, u = src[e] - b * K;
  col[e] = b;
  for (int q = 0; q < 4; ++q) {
    const double v = lam[((int64_t)b * 4 + q) * K + u];
    lamT64[e * 4 + q] = v;
    if (lamT32) lamT32[e * 4 + q] = (float)v;
  }
}

// node pointers, and the occupied nodes with their entry ranges; count becomes
// the fill cursor
__global__ void __launch_bounds__(kScanThreads)
    k_nodes(int32_t *count, int64_t V0, const uint64_t *sums, int64_t nb, int32_t *node_ptr,
            int32_t *occ, int32_t *occ_ptr) {
  scan_apply<true>(count, V0, sums, [&](int64_t v, int32_t c, uint64_t ex) {
    const int32_t e = (int32_t)(uint32_t)ex, i = (int32_t)(ex >> 32);
    node_ptr[v] = e;
    count[v] = e;
    if (c > 0) {
      occ[i] = (int32_t)v;
      occ_ptr[i] = e;
    }
  });
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    node_ptr[V0] = (int32_t)(uint32_t)sums[nb];
    occ_ptr[sums[nb] >> 32] = (int32_t)(uint32_t)sums[nb];
  }
}

// Per z line: whether it holds an occupied node, and {lo, g0, g1, hi}: its
// occupied nodes lie in [lo, hi) outside the longest unoccupied run [g0, g1)
// between them (a line through a closed surface crosses it twice)
__global__ void k_line_ranges(const int32_t *node_ptr, int64_t lines, int Nz, int32_t *any,
                              int32_t *range) {
  const int64_t l = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (l >= lines) return;
  int r0 = 0, r1 = 0, r2 = 0, r3 = 0;
  bool some = false;
  int e = node_ptr[l * Nz];
  for (int z = 0; z < Nz; ++z) {
    const int next = node_ptr[l * Nz + z + 1];
    if (next > e) {
      if (!some) {
        r0 = z;
        r1 = r2 = z + 1;
        some = true;
      } else if (z - r3 > r2 - r1) {  // a longer unoccupied run r3 .. z - 1
        r1 = r3;
        r2 = z;
      }
      r3 = z + 1;
    }
    e = next;
  }
  any[l] = some ? 1 : 0;
  range[4 * l] = r0, range[4 * l + 1] = r1, range[4 * l + 2] = r2, range[4 * l + 3] = r3;
}
__global__ void __launch_bounds__(kScanThreads)
    k_lines(const int32_t *any, int64_t lines, const uint64_t *sums, const int32_t *range,
            int32_t *occ_lines, int32_t *zrange) {
  scan_apply<true>(any, lines, sums, [&](int64_t l, int32_t c, uint64_t ex) {
    const int32_t i = (int32_t)(ex >> 32);
    if (c > 0) {
      occ_lines[i] = (int32_t)l;
      for (int q = 0; q < 4; ++q) zrange[4 * i + q] = range[4 * l + q];
    }
  });
}
// per x: the y range [lo, hi) of its occupied lines ([0, 0) if none); one wave
__global__ void __launch_bounds__(64) k_yrange(const int32_t *any, int Ny, int32_t *yr) {
  const int64_t x = blockIdx.x;
  int lo = Ny, hi = 0;
  for (int y = threadIdx.x; y < Ny; y += 64)
    if (any[x * Ny + y]) {
      lo = min(lo, y);
      hi = max(hi, y + 1);
    }
  for (int off = 32; off > 0; off >>= 1) {
    lo = min(lo, __shfl_xor(lo, off, 64));
    hi = max(hi, __shfl_xor(hi, off, 64));
  }
  if (threadIdx.x == 0) {
    yr[2 * x] = lo < hi ? lo : 0;
    yr[2 * x + 1] = lo < hi ? hi : 0;
  }
}

// the plane's occupied nodes x Ny + y from the grid's (all on one plane)
__global__ void k_plane(const int32_t *occ, int64_t n_occ, int Nz, int32_t *plane_occ) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n_occ) plane_occ[i] = occ[i] / Nz;
}

}  // namespace

void node_tables_mesh(Plan *pl, MeshDev &md, hipStream_t s) {
  const HostPlan &h = md.hp;
  const int64_t n = h.n, NK = n * h.K;
  const int Nx = h.grid[0], Ny = h.grid[1], Nz = h.grid[2];
  const int64_t A = (int64_t)Nx * Ny, V0 = A * Nz;
  if (NK > INT32_MAX) throw Error(AIM_ERR_ARG, "projection too large for 32-bit indexing");
  std::vector<void *> tmp;
  auto scratch = [&](size_t bytes) {
    void *p = dev_alloc(pl, bytes);
    tmp.push_back(p);
    return p;
  };
  uint64_t *sums = (uint64_t *)scratch(sizeof(uint64_t) * (scan_blocks(std::max(V0, A)) + 1));
  // scans v[0 .. count); returns (sum, occupied items)
  auto scan = [&](const int32_t *v, int64_t count) {
    const uint64_t total = scan_sums<true>(v, count, sums, s);
    return std::make_pair((int64_t)(uint32_t)total, (int64_t)(total >> 32));
  };
  auto ints = [&](int64_t count) {
    return (int32_t *)dev_alloc(pl, sizeof(int32_t) * (size_t)std::max<int64_t>(count, 1));
  };

  int32_t *count = (int32_t *)scratch(sizeof(int32_t) * V0);
  hipLaunchKernelGGL(k_clear, dim3(launch_blocks(V0, 256)), dim3(256), 0, s, count, V0);
  LAUNCHCHECK();
  hipLaunchKernelGGL(k_count, dim3(launch_blocks(NK, 256)), dim3(256), 0, s, md.lam64, md.curl64,
                     md.anchor_lin, md.stencil_off, n, h.K, count);
  LAUNCHCHECK();
  const auto nodes = scan(count, V0);
  const int64_t ne = nodes.first;
  md.n_entries = ne;
  md.n_occ = nodes.second;
  md.node_ptr = ints(V0 + 1);
  md.occ = ints(md.n_occ);
  md.occ_ptr = ints(md.n_occ + 1);
  const int64_t vb = scan_blocks(V0);
  hipLaunchKernelGGL(k_nodes, dim3((unsigned)vb), dim3(kScanThreads), 0, s, count, V0, sums, vb,
                     md.node_ptr, md.occ, md.occ_ptr);
  LAUNCHCHECK();
  int32_t *src = (int32_t *)scratch(sizeof(int32_t) * std::max<int64_t>(ne, 1));
  hipLaunchKernelGGL(k_fill, dim3(launch_blocks(NK, 256)), dim3(256), 0, s, md.lam64, md.curl64,
                     md.anchor_lin, md.stencil_off, n, h.K, count, src);
  LAUNCHCHECK();
  md.ent_col = ints(ne);
  md.lamT64 = (double *)dev_alloc(pl, sizeof(double) * 4 * std::max<int64_t>(ne, 1));
  if (pl->mixed) md.lamT32 = (float *)dev_alloc(pl, sizeof(float) * 4 * std::max<int64_t>(ne, 1));
  if (ne > 0) {
    // (the tables that k_lam_transpose writes are free until then: lamT64 holds the
    // long lists' nodes and ent_col the sort's other buffer; count[0] counts the lists)
    int32_t *long_list = (int32_t *)md.lamT64;
    hipLaunchKernelGGL(k_clear, dim3(1), dim3(64), 0, s, count, (int64_t)1);
    LAUNCHCHECK();
    hipLaunchKernelGGL(k_order, dim3(launch_blocks(md.n_occ, 64)), dim3(64), 0, s, md.occ_ptr,
                       md.n_occ, src, long_list, count);
    LAUNCHCHECK();
    int bits = 0;
    while (bits < 31 && ((NK - 1) >> bits) > 0) ++bits;
    hipLaunchKernelGGL(k_order_long, dim3((unsigned)std::min<int64_t>(md.n_occ, kSortGroups)),
                       dim3(kScanThreads), 0, s, md.occ_ptr, long_list, count, bits, src,
                       md.ent_col);
    LAUNCHCHECK();
    hipLaunchKernelGGL(k_lam_transpose, dim3(launch_blocks(ne, 256)), dim3(256), 0, s, md.lam64,
                       src, ne, h.K, md.ent_col, md.lamT64, md.lamT32);
    LAUNCHCHECK();
  }

  int32_t *any = (int32_t *)scratch(sizeof(int32_t) * A);
  int32_t *range = (int32_t *)scratch(sizeof(int32_t) * 4 * A);
  hipLaunchKernelGGL(k_line_ranges, dim3(launch_blocks(A, 64)), dim3(64), 0, s, md.node_ptr, A, Nz,
                     any, range);
  LAUNCHCHECK();
  md.n_occ_lines = scan(any, A).second;
  md.occ_lines = ints(md.n_occ_lines);
  md.occ_zrange = ints(4 * md.n_occ_lines);
  hipLaunchKernelGGL(k_lines, dim3((unsigned)scan_blocks(A)), dim3(kScanThreads), 0, s, any, A,
                     sums, range, md.occ_lines, md.occ_zrange);
  LAUNCHCHECK();
  md.occ_yrange = ints(2 * (int64_t)Nx);
  hipLaunchKernelGGL(k_yrange, dim3((unsigned)Nx), dim3(64), 0, s, any, Ny, md.occ_yrange);
  LAUNCHCHECK();

  if (md.planar_z >= 0) {
    md.n_plane_occ = md.n_occ;
    md.plane_occ = ints(md.n_occ);
    md.plane_occ_ptr = md.occ_ptr;  // the same entry ranges
    if (md.n_occ > 0) {
      hipLaunchKernelGGL(k_plane, dim3(launch_blocks(md.n_occ, 256)), dim3(256), 0, s, md.occ,
                         md.n_occ, Nz, md.plane_occ);
      LAUNCHCHECK();
    }
  }
  HIPCHECK(hipStreamSynchronize(s));
  for (void *p : tmp) dev_free(pl, p);
}

}  // namespace aim
