// The AIM product y = Z^near x + Z^grid x (hot path).
//
// Steps, in the paper's order (Section 4.1): projection of the basis
// currents onto the grid (anterpolation), propagation (forward FFTs, Green's
// spectrum multiply, inverse FFTs on the zero-padded grid), interpolation
// back to the testing functions, plus the sparse near-zone correction, fused
// with the interpolation so y is written once. The input vector may be of a
// wider type than the arithmetic (c128 Krylov vectors feeding the c64
// operator): the narrowing happens in registers as x is read.
#include <algorithm>
#include <type_traits>

#include "aim_internal.h"
#include "fft_map.h"
#include "multi_rhs.h"

namespace aim {

namespace {

// Gather form of anterpolation: grid node v sums Lambda_T[e] x_{col[e]} over
// its entries, so every node (also empty ones) is written exactly once, with
// no atomics and no clearing pass, in a fixed order (bitwise reproducible).
// Each 64-lane wave owns npw <= 64 consecutive nodes (fewer where nodes hold
// many entries, so that a wave's entries stay few), whose entries are contiguous:
// the wave loads them epl * 64 at a time (coalesced; every lane has epl
// independent gathers in flight), each lane forming its entries' four products
// in LDS; then the 64 / npw lanes of each node sum every (64 / npw)-th of its
// slots and combine their sums by exchanges within the group (one right-hand
// side per blockIdx.y). Entries per lane
// per chunk: 2 (measured on the sphere over the occupied nodes: 1 or 4 is
// slower for float, 1 for double by 30%)
template <typename T>
constexpr int anterp_epl() {
  return 2;
}
// occupied nodes per wave of the 3-D projection
// occupied nodes per wave of the gather: candidates timed at set-up (on the
// sphere: 64 0.079 ms, 32 0.067, 16 0.058, 8 0.056 for c64; 16 best for c128)
constexpr int kGatherNpwCand[3] = {8, 16, 32};
// With occ (the occupied nodes, increasing) the wave walks npw consecutive
// occupied nodes instead: node_ptr is then their compacted entry ranges, V0
// their count, and node i is written at grid index occ[i] of fields of Vg
// nodes; the other nodes are left untouched (zero in the caller's buffer).
template <typename T, typename TX>
__global__ void __launch_bounds__(256)
    k_anterp_gather(const cx<TX> *__restrict__ x, int64_t ldx, int nrhs,
                    const int32_t *__restrict__ node_ptr, const int32_t *__restrict__ occ,
                    const int32_t *__restrict__ ent_col, const T *__restrict__ lamT,
                    cx<T> *__restrict__ grid, int64_t V0, int64_t Vg, int npw) {
  constexpr int kEpl = anterp_epl<T>();
  constexpr int C = 64 * kEpl;      // entries per chunk
  __shared__ cx<T> slot[4][C][4];  // [wave][entry][q]
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t v0 = ((int64_t)blockIdx.x * (blockDim.x >> 6) + w) * npw;
  if (v0 >= V0) return;  // whole wave exits; no block-wide barrier is used
  // G = 64 / npw lanes per node (npw divides 64, checked by the launcher):
  // lane = node * G + sub
  const int G = 64 / npw, sub = lane & (G - 1);
  const int64_t v = v0 + lane / G;
  const bool ok = v < V0;
  const int64_t vend = (v0 + npw < V0) ? v0 + npw : V0;
  const int e0 = ok ? node_ptr[v] : 0, e1 = ok ? node_ptr[v + 1] : 0;
  const int w0 = node_ptr[v0], w1 = node_ptr[vend];
  {
    const int r = blockIdx.y;  // right-hand side
    const cx<TX> *xr = x + (int64_t)r * ldx;
    T a[4][2] = {{0, 0}, {0, 0}, {0, 0}, {0, 0}};
    for (int c0 = w0; c0 < w1; c0 += C) {
      int col[kEpl];
#pragma unroll
      for (int u = 0; u < kEpl; ++u) {
        const int e = c0 + u * 64 + lane;
        col[u] = e < w1 ? ent_col[e] : -1;
      }
#pragma unroll
      for (int u = 0; u < kEpl; ++u) {
        const int e = c0 + u * 64 + lane;
        if (col[u] >= 0) {
          const cx<TX> xv = xr[col[u]];
          const T xa = (T)xv.x, xb = (T)xv.y;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const T wq = lamT[(int64_t)e * 4 + q];
            cx<T> p;
            p.x = wq * xa;
            p.y = wq * xb;
            slot[w][u * 64 + lane][q] = p;
          }
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      const int lo = (e0 > c0 ? e0 : c0) - c0, hi = (e1 < c0 + C ? e1 : c0 + C) - c0;
      for (int k = lo + sub; k < hi; k += G) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const cx<T> p = slot[w][k][q];
          a[q][0] += p.x;
          a[q][1] += p.y;
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    for (int off = 1; off < G; off <<= 1)  // the group's partial sums, fixed order
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        a[q][0] += __shfl_xor(a[q][0], off, 64);
        a[q][1] += __shfl_xor(a[q][1], off, 64);
      }
    if (ok && sub == 0) {
      const int64_t node = occ ? (int64_t)occ[v] : v;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        cx<T> o;
        o.x = a[q][0];
        o.y = a[q][1];
        grid[((int64_t)(r * 4 + q)) * Vg + node] = o;
      }
    }
  }
}

// (grids of many right-hand sides have more elements than a launch has threads)
template <typename T>
__global__ void k_zero(cx<T> *__restrict__ p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i].x = p[i].y = 0;
}
template <typename T>
void clear(cx<T> *p, int64_t n, hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL((k_zero<T>), dim3(loop_blocks(n, 256)), dim3(256), 0, s, p, n);
  LAUNCHCHECK();
}

// thin [F][Pz][A] grid -> plain [F][A][Pz] (inspection)
template <typename T>
__global__ void k_kz_inner(const cx<T> *__restrict__ in, cx<T> *__restrict__ out, int64_t F,
                           int64_t A, int Pz) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= F * A * Pz) return;
  const int kz = (int)(t % Pz);
  const int64_t a = (t / Pz) % A, f = t / (Pz * A);
  out[t] = in[(f * Pz + kz) * A + a];
}

// kz-blocked [F][Pz/blk][Nx][Py][blk] grid -> plain [F][Nx][Py][Pz] (inspection)
template <typename T>
__global__ void k_unblock(const cx<T> *__restrict__ in, cx<T> *__restrict__ out, int64_t F, int Nx,
                          int Py, int Pz, int blk, int64_t fstride) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t tot = F * Nx * Py * Pz;
  if (t >= tot) return;
  const int kz = (int)(t % Pz);
  const int ky = (int)((t / Pz) % Py);
  const int x = (int)((t / ((int64_t)Py * Pz)) % Nx);
  const int64_t f = t / ((int64_t)Nx * Py * Pz);
  out[t] = in[f * fstride + ((int64_t)(kz / blk) * Nx + x) * Py * blk + (int64_t)ky * blk + kz % blk];
}

// Sum over the 16 or 32 lanes of a row (every lane gets it), by lane permutations
// (DPP: quad swaps, then mirrors of 8 and 16 lanes).
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true),
                          __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true));
}
template <int LANES, typename V>
__device__ __forceinline__ V row_sum(V v) {
  v.x += dpp<0xB1>(v.x), v.y += dpp<0xB1>(v.y);    // lane ^ 1
  v.x += dpp<0x4E>(v.x), v.y += dpp<0x4E>(v.y);    // lane ^ 2
  v.x += dpp<0x141>(v.x), v.y += dpp<0x141>(v.y);  // 7 - lane of 8
  v.x += dpp<0x140>(v.x), v.y += dpp<0x140>(v.y);  // 15 - lane of 16
  if (LANES == 32) v.x += __shfl_xor(v.x, 16, 64), v.y += __shfl_xor(v.y, 16, 64);
  return v;
}

// y_m = j k eta [sum_{q<3} Lambda_mq . phi_q - k^-2 Lambda_md . phi_d]
//       + sum_n Z^near_mn x_n.
//
// 16 lanes per row m, four rows per wave. Bound by the latency of its chain of
// loads, so the chain is kept short: row pointer, anchor and stencil offsets;
// then the near entries' columns and values, the stencil weights and the fields,
// all in flight together; then x at the columns. kNearUnroll entries per lane
// cover rows of up to 96 entries (the benchmark meshes have 72 to 81) in one
// pass, kStencilUnroll nodes per lane the 9 or 27 nodes of second order. With 32
// lanes per row (a last pass mostly idle, two rows per wave) and the stencil's
// chain before the near zone's, the 128-lambda plate took 1.21 ms (4.20 GB, 3.5
// TB/s) and now takes 0.83 (5.1 TB/s, the rate of a copy); the 8-lambda CFIE
// sphere 95 -> 87 us, third order with 3 right-hand sides in FP64 (2.7-lambda
// sphere, formerly one at a time) 99 -> 55 us.
constexpr int kRowLanes = 16;
constexpr int kNearUnroll = 6;
constexpr int kStencilUnroll = 2;
// 32 lanes per row, a half and the same number of these, where the fields of a volume
// (a plane's 9 nodes need none) meet fewer rows than 16 lanes each fill the chip with: the
// time is then one wave's chain (third order, 1-lambda sphere, 3 630 rows, c64:
// 7.9 -> 6.8 us; 25 230 rows: 16 lanes are faster; product of second order, 1 080 rows,
// c64 19.4 -> 18.6, FP64 20.3 -> 19.4, 3 630 rows 20.7 -> 19.9 and 23.4 -> 23.0)
constexpr int64_t kFewRows = 8192, kFewRowsLow = 4096;  // of 64 nodes and more, of fewer

// RB right-hand sides from r_first + RB blockIdx.y: the stencil weights, the
// near-zone entries and their columns are loaded once for the RB products.
// CF (combined field): y^far = keta j [sum_q Lambda_q^T phi_q - inv_k2
// Lambda_d^T phi_d] - eta_h sum_e W_e^T phi_e, with keta = alpha k eta and
// eta_h = (1 - alpha) eta; the curl weights W test the vector potential's curl.
template <typename T, typename TX, typename TY, int RB, bool CF, int LANES = kRowLanes>
__global__ void __launch_bounds__(256)
    k_interp_near(const cx<T> *__restrict__ phi, int64_t nf, int r_first,
                  const T *__restrict__ lam, const T *__restrict__ curl,
                  const int32_t *__restrict__ anchor_lin, const int32_t *__restrict__ soff, int K,
                  const int32_t *__restrict__ rowptr, const int32_t *__restrict__ cols,
                  const cx<T> *__restrict__ nearv, const cx<TX> *__restrict__ x, int64_t ldx,
                  cx<TY> *__restrict__ y, int64_t ldy, int64_t n, T keta, T inv_k2, T eta_h) {
  using V = cx<T>;
  constexpr int NU = kNearUnroll * kRowLanes / LANES, SU = kStencilUnroll;
  // near sums per lane: two with 16 lanes, so that they are as short as with 32
  // (8-lambda sphere in c64, error against FP64: one 1.043e-7, two 0.994e-7, 32 lanes
  // 1.025e-7; this kernel alone in FP64 on the 1-lambda sphere: 1.60e-16, 1.50e-16 and
  // 1.52e-16; the same registers and time)
  constexpr int NS = 32 / LANES;
  const int lane = threadIdx.x & (LANES - 1);
  const int64_t m = (int64_t)blockIdx.x * (256 / LANES) + threadIdx.x / LANES;
  if (m >= n) return;  // whole rows exit
  int so[SU];
#pragma unroll
  for (int k = 0; k < SU; ++k) so[k] = lane + LANES * k < K ? soff[lane + LANES * k] : 0;
  const int64_t a = anchor_lin[m];
  const int e0 = rowptr[m], e1 = rowptr[m + 1];
  const int r0 = r_first + blockIdx.y * RB;  // first right-hand side of this row
  V far[RB], nr[RB][NS], fk[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    far[rb].x = far[rb].y = fk[rb].x = fk[rb].y = 0;
#pragma unroll
    for (int j = 0; j < NS; ++j) nr[rb][j].x = nr[rb][j].y = 0;
  }
  V z[NU];
  int c[NU];
  auto load_near = [&](int eb) {  // entries eb, eb + 16, ... of this lane
#pragma unroll
    for (int k = 0; k < NU; ++k) c[k] = eb + LANES * k < e1 ? cols[eb + LANES * k] : -1;
#pragma unroll
    for (int k = 0; k < NU; ++k) {
      if (eb + LANES * k < e1) {
        z[k] = nearv[eb + LANES * k];
      } else {
        z[k].x = 0;
        z[k].y = 0;
      }
    }
  };
  auto add_near = [&]() {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const cx<TX> *xr = x + (int64_t)(r0 + rb) * ldx;
      cx<TX> xv[NU];
#pragma unroll
      for (int k = 0; k < NU; ++k) {
        if (c[k] >= 0)
          xv[k] = xr[c[k]];
        else
          xv[k].x = xv[k].y = 0;
      }
#pragma unroll
      for (int k = 0; k < NU; ++k) {
        const T xa = (T)xv[k].x, xb = (T)xv[k].y;
        nr[rb][k % NS].x += z[k].x * xa - z[k].y * xb;
        nr[rb][k % NS].y += z[k].x * xb + z[k].y * xa;
      }
    }
  };
  auto far_node = [&](int64_t o, T l0, T l1, T l2, T l3, T w0, T w1, T w2) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const V *ph = phi + o * nf + (r0 + rb) * 4;  // fields interleaved per node
      const V p0 = ph[0], p1 = ph[1], p2 = ph[2], p3 = ph[3];
      far[rb].x += l0 * p0.x + l1 * p1.x + l2 * p2.x - inv_k2 * l3 * p3.x;
      far[rb].y += l0 * p0.y + l1 * p1.y + l2 * p2.y - inv_k2 * l3 * p3.y;
      if (CF) {
        fk[rb].x += w0 * p0.x + w1 * p1.x + w2 * p2.x;
        fk[rb].y += w0 * p0.y + w1 * p1.y + w2 * p2.y;
      }
    }
  };
  const T *lm = lam + m * 4 * K, *wm = CF ? curl + m * 3 * K : nullptr;
  load_near(e0 + lane);
  for (int u0 = lane; u0 < K; u0 += LANES * SU) {
    T l[SU][4], w[SU][3];
#pragma unroll
    for (int k = 0; k < SU; ++k) {
      const int u = u0 + LANES * k;
#pragma unroll
      for (int q = 0; q < 4; ++q) l[k][q] = u < K ? lm[q * K + u] : (T)0;
#pragma unroll
      for (int q = 0; q < 3; ++q) w[k][q] = (CF && u < K) ? wm[q * K + u] : (T)0;
    }
#pragma unroll
    for (int k = 0; k < SU; ++k)
      if (u0 + LANES * k < K)
        far_node(a + so[k], l[k][0], l[k][1], l[k][2], l[k][3], w[k][0], w[k][1], w[k][2]);
    if (u0 + LANES * SU < K)  // the next nodes (orders above 2)
#pragma unroll
      for (int k = 0; k < SU; ++k) {
        const int u = u0 + LANES * (SU + k);
        so[k] = u < K ? soff[u] : 0;
      }
  }
  add_near();
  for (int eb = e0 + lane + LANES * NU; eb < e1; eb += LANES * NU) {
    load_near(eb);
    add_near();
  }
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    V acc;
    acc.x = -keta * far[rb].y;  // j k eta * far
    acc.y = keta * far[rb].x;
    if (CF) {
      acc.x -= eta_h * fk[rb].x;
      acc.y -= eta_h * fk[rb].y;
    }
#pragma unroll
    for (int j = 0; j < NS; ++j) {
      acc.x += nr[rb][j].x;
      acc.y += nr[rb][j].y;
    }
    acc = row_sum<LANES>(acc);
    if (lane == 0) {
      cx<TY> out;
      out.x = (decltype(out.x))acc.x;
      out.y = (decltype(out.y))acc.y;
      y[(int64_t)(r0 + rb) * ldy + m] = out;
    }
  }
}

template <typename T>
const T *lam_of(const MeshDev &md);
template <>
const double *lam_of<double>(const MeshDev &md) {
  return md.lam64;
}
template <>
const float *lam_of<float>(const MeshDev &md) {
  return md.lam32;
}
template <typename T>
const T *curl_of(const MeshDev &md);
template <>
const double *curl_of<double>(const MeshDev &md) {
  return md.curl64;
}
template <>
const float *curl_of<float>(const MeshDev &md) {
  return md.curl32;
}
template <typename T>
const T *plane_lam_of(const MeshDev &md);
template <>
const double *plane_lam_of<double>(const MeshDev &md) {
  return md.plane_lam64;
}
template <>
const float *plane_lam_of<float>(const MeshDev &md) {
  return md.plane_lam32;
}
template <typename T>
const T *lamT_of(const MeshDev &md);
template <>
const double *lamT_of<double>(const MeshDev &md) {
  return md.lamT64;
}
template <>
const float *lamT_of<float>(const MeshDev &md) {
  return md.lamT32;
}
template <typename T>
const cx<T> *near_of(const MeshDev &md);
template <>
const double2 *near_of<double>(const MeshDev &md) {
  return md.near64;
}
template <>
const float2 *near_of<float>(const MeshDev &md) {
  return md.near32;
}
template <typename T>
const cx<T> *ghat_of(const MeshDev &md);
template <>
const double2 *ghat_of<double>(const MeshDev &md) {
  return md.ghat64;
}
template <>
const float2 *ghat_of<float>(const MeshDev &md) {
  return md.ghat32;
}
template <typename T>
const cx<T> *ghat2d_of(const MeshDev &md);
template <>
const double2 *ghat2d_of<double>(const MeshDev &md) {
  return md.ghat2d64;
}
template <>
const float2 *ghat2d_of<float>(const MeshDev &md) {
  return md.ghat2d32;
}
template <typename T>
const cx<T> *ghatp_of(const MeshDev &md);
template <>
const double2 *ghatp_of<double>(const MeshDev &md) {
  return md.ghatp64;
}
template <>
const float2 *ghatp_of<float>(const MeshDev &md) {
  return md.ghatp32;
}
template <typename T>
const cx<T> *tw_of(const MeshDev &md, int d);
template <>
const double2 *tw_of<double>(const MeshDev &md, int d) {
  return md.tw64[d];
}
template <>
const float2 *tw_of<float>(const MeshDev &md, int d) {
  return md.tw32[d];
}

}  // namespace

// a per-mesh grid buffer of `bytes` (grown on demand) that is zero wherever
// the kernels writing it never write
template <typename T>
static cx<T> *zeroed_buffer(Plan *pl, void *(&buf)[2], size_t (&have)[2], size_t bytes,
                            hipStream_t s) {
  const int prec = sizeof(T) == 8 ? 0 : 1;
  if (have[prec] < bytes) {
    if (buf[prec]) dev_free(pl, buf[prec]);
    buf[prec] = nullptr;
    have[prec] = 0;
    buf[prec] = dev_alloc(pl, bytes);
    have[prec] = bytes;
    ++pl->work_gen;
    clear<T>((cx<T> *)buf[prec], (int64_t)(bytes / sizeof(cx<T>)), s);
  }
  return (cx<T> *)buf[prec];
}
// the mesh's projected source grid in `layout` (1: 3-D grid [F][V0], 2: the
// scatterer's plane [F][Nx Ny]), zero where no projection entry lands. The
// projection writes the occupied nodes only, so a buffer last written in the
// other layout (the full 3-D inspection of a planar scatterer, or the plane
// after it) is cleared first, and a captured graph of the other layout dropped.
template <typename T>
static cx<T> *src_buffer(Plan *pl, MeshDev &md, size_t bytes, int layout, hipStream_t s) {
  const int prec = sizeof(T) == 8 ? 0 : 1;
  const size_t had = md.src_bytes[prec];
  cx<T> *p = zeroed_buffer<T>(pl, md.src, md.src_bytes, bytes, s);
  if (md.src_layout[prec] != layout) {
    ++pl->work_gen;
    if (md.src_bytes[prec] == had)  // not just zeroed
      clear<T>(p, (int64_t)(had / sizeof(cx<T>)), s);
  }
  md.src_layout[prec] = layout;
  return p;
}

void *work_buffer(Plan *pl, int lane, int prec, int which, size_t bytes, hipStream_t s) {
  void *(&work)[4] = pl->work[lane][prec];
  size_t(&have)[4] = pl->work_bytes[lane][prec];
  if (have[which] < bytes) {
    if (work[which]) dev_free(pl, work[which]);
    work[which] = nullptr;
    have[which] = 0;
    work[which] = dev_alloc(pl, bytes);
    have[which] = bytes;
    ++pl->work_gen;
    if (which == 0) {
      // the propagated fields: the inverse z pass writes the occupied lines
      // only and the interpolation multiplies the others by zero weights, so
      // they must hold finite values
      if (prec == 0)
        clear<double>((double2 *)work[which], (int64_t)(bytes / sizeof(double2)), s);
      else
        clear<float>((float2 *)work[which], (int64_t)(bytes / sizeof(float2)), s);
    }
  }
  return work[which];
}

// Few rows: the time is one wave's chain, so each of several right-hand sides, or each two
// of an even number with 32 lanes (936 rows, third order, c64, 8: 38 us alone, 33 in
// twos), takes rows (waves) of its own, all in one launch, projected by the gather
// (product, us, groups of 4 and a launch for those left over or a lane each -> rows each;
// 225 rows, planar, second order, c64: 5 right-hand sides 15.7 -> 12.0, 9 18.5 -> 12.1;
// fifth order in FP64: 3 35 -> 30, 5 58 -> 43, 17 122 -> 55; CFIE spheres: 1 080 rows,
// third order in FP64, 17 76 -> 51; 2 430 rows, second order in FP64, 5 37 -> 32). Of more
// rows the gathers' traffic is what counts (3 630 rows, fourth order, c64: 5 53 -> 59), from 2 048 with stencils of 64
// nodes and more (2 133 rows, planar, fifth order in FP64: 8 87 -> 114), and so it is of
// many right-hand sides (936 rows, planar, fifth order in FP64: 24 105 -> 132, 64 168 ->
// 292; second order 64 31 -> 34), later where nodes with long lists are few, which half a
// wave each sums slowly (1 080 rows, sphere, c64: fifth order, 175 entries per node, 33
// 205 -> 128; fourth, 102 per node, 33 89 -> 76, 64 101 -> 122). 3 and 4 right-hand sides
// share what they load, which wins earlier (2 133 rows, second order in FP64, 4 equal;
// fourth 26 -> 28).
constexpr int64_t kLoneRows = 2560;       // n
constexpr int64_t kLoneRowsHigh = 2048;   // n, with kLoneHigh nodes per stencil and more
constexpr int kLoneHigh = 28;
constexpr int64_t kLoneFew = 6144, kLoneWork = 28672;       // n nrhs, up to 4; more
constexpr int64_t kLoneHighWork = 20480, kLoneLong = 36864;  // with those stencils
constexpr int64_t kLongList = 96;         // entries per node
static bool lone_rows(const MeshDev &md, int nrhs) {
  const int64_t n = md.hp.n, work = n * nrhs;
  if (nrhs < 3 || n > kLoneRows) return false;
  if (nrhs <= 4) return work <= kLoneFew;
  const bool plane = md.planar_z >= 0;
  const int K = plane ? md.plane_K : md.hp.K;
  if (K < kLoneHigh || nrhs == 5) return work <= kLoneWork;
  const bool longer = n * K >= kLongList * (plane ? md.n_plane_occ : md.n_occ);
  return n <= kLoneRowsHigh && work <= (longer ? kLoneLong : kLoneHighWork);
}

// Lanes per node (row) of the several-right-hand-sides kernels (multi_rhs.h), 0:
// the others. From 6 on they are faster on nearly every mesh of more rows (projection and
// interpolation together, 4-lambda CFIE sphere, the others -> these: 4 right-hand sides
// 82 -> 109 us in c64 and 154 -> 178 in FP64, 5 106 -> 111 and 191 -> 182; 16-lambda
// plate: 4 45 -> 56 and 74 -> 74, 5 58 -> 56 and 94 -> 75; 8 and 16 on that sphere take
// 118 and 185, and 200 and 290, where four per launch row took 149 and 276, and 354 and
// 671), but not in c64 at low order, where full groups of 4 are on up to 48 K rows together
// (products of second order, a lane each -> groups: 2 133 rows, planar, 16 right-hand sides
// 29.6 -> 25.8; 3 816 rows, planar, 8 26.6 -> 22.6; 3 630 rows, sphere, 8 51 -> 48, 16 57 ->
// 59; 5 070 rows, 12 within 5%)
constexpr int kMultiFrom = 6;
constexpr int64_t kGroupWork = 49152;
template <typename T>
static int multi_lanes(const MeshDev &md, int nrhs) {
  const int K = md.planar_z >= 0 ? md.plane_K : md.hp.K;
  const bool groups =
      sizeof(T) == 4 && nrhs % 4 == 0 && K < kLoneHigh && md.hp.n * nrhs <= kGroupWork;
  return nrhs < kMultiFrom || groups || lone_rows(md, nrhs) ? 0 : (nrhs <= 8 ? 8 : 16);
}

// x of one mesh transposed to [n][nrhs] in T
template <typename T, typename TX>
static cx<T> *transposed_x(Plan *pl, const MeshDev &md, int nrhs, const cx<TX> *x, int64_t ldx,
                           bool fill, hipStream_t s) {
  const int prec = sizeof(T) == 8 ? 0 : 1;
  const int64_t n = md.hp.n;
  cx<T> *xt = (cx<T> *)work_buffer(pl, md.lane, prec, 3, sizeof(cx<T>) * n * nrhs, s);
  if (fill) {
    hipLaunchKernelGGL((k_transpose_x<T, TX>), dim3(launch_blocks(n, 64), (nrhs + 15) / 16),
                       dim3(kMultiThreads), 0, s, x, ldx, nrhs, n, xt);
    LAUNCHCHECK();
  }
  return xt;
}

// projection of x onto the occupied nodes occ of grids of Vg nodes
template <typename T, typename TX>
static void project(Plan *pl, const MeshDev &md, int nrhs, const cx<TX> *x, int64_t ldx,
                    const int32_t *occ_ptr, const int32_t *occ, int64_t n_occ, cx<T> *grid,
                    int64_t Vg, hipStream_t s) {
  const int npw = md.gather_npw[sizeof(T) == 8 ? 0 : 1];
  const int LR = multi_lanes<T>(md, nrhs);
  if (LR > 0) {
    const cx<T> *xt = transposed_x<T, TX>(pl, md, nrhs, x, ldx, true, s);
    auto go = [&](auto kern) {
      hipLaunchKernelGGL(kern, dim3(launch_blocks(n_occ, kMultiRows), (nrhs + LR - 1) / LR),
                         dim3(kMultiThreads), 0, s, xt, nrhs, occ_ptr, occ, md.ent_col,
                         lamT_of<T>(md), grid, n_occ, Vg);
    };
    if (n_occ > 0) {
      if (LR == 8)
        go(k_anterp_multi<T, 8>);
      else
        go(k_anterp_multi<T, 16>);
    }
  } else if (n_occ > 0) {
    hipLaunchKernelGGL((k_anterp_gather<T, TX>),
                       dim3((unsigned)((n_occ + 4 * npw - 1) / (4 * npw)), nrhs), dim3(256), 0, s,
                       x, ldx, nrhs, occ_ptr, occ, md.ent_col, lamT_of<T>(md), grid, n_occ, Vg, npw);
  }
  LAUNCHCHECK();
}

// plane by plane where both lengths have the kernel; a flat scatterer's four planes
// per right-hand side only up to 90 points in c64 and 81 in c128, above which one
// work-group's chain takes longer than three launches (full plates, product, separate ->
// plane by plane with 1 and 16 right-hand sides, us: c64 81 points 19.1 -> 15.0 and 33.2
// -> 27.5, 90 18.8 -> 16.1 and 34.1 -> 30.1, 96 18.5 -> 19.4 and 34.2 -> 32.7, 126 20.0 ->
// 23.2 and 46.2 -> 44.6; c128 81 19.5 -> 19.2 and 43.3 -> 37.0, 90 20.2 -> 21.4 and 45.2
// -> 41.8, 126 22.6 -> 36.1 and 54.1 -> 60.6); a caller that asks for tile rows or field
// groups gets the passes these belong to
void choose_plane_fft(const Plan *pl, MeshDev &md) {
  auto range = [&](auto *v, int flat) {
    if ((pl->params.tuning & 0xffff) != 0 || md.plan[0].P != md.plan[1].P) return PlaneRange{};
    if (md.planar_z >= 0 ? md.plan[0].P > flat : !fft_zplane_available(v, md.plan[2]))
      return PlaneRange{};
    return fft_plane_range(v, md.plan[0]);
  };
  md.plane_fft[0] = range((const double2 *)nullptr, 81);
  md.plane_fft[1] = pl->mixed ? range((const float2 *)nullptr, 90) : PlaneRange{};
}
bool plane_by_plane(const MeshDev &md, int prec, int64_t nrhs) {
  return md.plane_fft[prec].has(4 * nrhs * (md.planar_z >= 0 ? 1 : md.hp.pad[2]));
}

template <typename T, typename TX>
void far_stages(Plan *pl, MeshDev &md, int nrhs, const cx<TX> *x, int64_t ldx, int stop,
                hipStream_t s, hipEvent_t *ev, bool full3d, StageView *views, int first) {
  auto mark = [&](int i) {
    if (ev) HIPCHECK(hipEventRecord(ev[i], s));
  };
  // records where stage st left its output: plain view [F][A][Z] with strides
  auto view = [&](int st, const void *p, int64_t A, int64_t Z, int64_t fs, int64_t as,
                  int64_t zs) {
    if (!views) return;
    StageView &v = views[st];
    v = StageView{};
    v.p = p;
    v.kind = 1;
    v.F = 4 * (int64_t)nrhs;
    v.A = A;
    v.Z = Z;
    v.fs = fs;
    v.as = as;
    v.zs = zs;
  };
  if (views)
    for (int i = 0; i < AIM_NSTAGE; ++i) views[i] = StageView{};
  const HostPlan &h = md.hp;
  const int prec = sizeof(T) == 8 ? 0 : 1;
  const int Nx = h.grid[0], Ny = h.grid[1], Nz = h.grid[2];
  const int Px = h.pad[0], Py = h.pad[1], Pz = h.pad[2];
  (void)Px;
  const int64_t F = 4 * (int64_t)nrhs;
  const int64_t V0 = (int64_t)Nx * Ny * Nz;
  const int blk = kGridBlock<T>;
  const int npw = md.gather_npw[prec];
  if (npw < 1 || npw > 64 || 64 % npw != 0)
    throw Error(AIM_ERR_ARG, "projection gather: nodes per wave must divide 64");
  // set-up: the buffers of such a product, without any stage
  const bool reserve = first > 6;
  // the passes along y and x plane by plane, when the product runs through (the
  // stage boundaries between them then fall together: the forward y step carries
  // the time of all three)
  const bool planes =
      plane_by_plane(md, prec, nrhs) && stop >= 6 && (first <= 1 || reserve) && !full3d;
  // work buffer `which` of `count` elements per field, where a stage that is asked for
  // touches it
  auto buf = [&](int which, int64_t count, bool touched) {
    return touched ? (cx<T> *)work_buffer(pl, md.lane, prec, which, sizeof(cx<T>) * F * count, s)
                   : nullptr;
  };
  if (reserve && (multi_lanes<T>(md, nrhs) > 0 || multi_lanes<T>(md, nrhs - 1) > 0))
    (void)transposed_x<T, TX>(pl, md, nrhs, x, ldx, false, s);  // (for nrhs or fewer)
  if (md.planar_z >= 0 && !full3d) {
    // every source on the plane z = planar_z, and only that plane weighted by
    // the interpolation: the plane alone, g0 = [F][Nx][Ny], 2-D propagation
    // (y passes, x pass with the 2-D spectrum)
    const int64_t A1 = (int64_t)Nx * Ny, V2 = (int64_t)Nx * Py;
    cx<T> *g0 = buf(0, A1, stop > 4);
    cx<T> *g2 = buf(2, V2, stop > 1 && !planes);
    cx<T> *gs = src_buffer<T>(pl, md, sizeof(cx<T>) * F * A1, 2, s);
    if (reserve) return;
    mark(0);
    if (first <= 1)
      project<T, TX>(pl, md, nrhs, x, ldx, md.plane_occ_ptr, md.plane_occ, md.n_plane_occ, gs, A1, s);
    mark(1);
    view(1, gs, Nx, Ny, A1, Ny, 1);
    if (stop <= 1) return;
    mark(2);
    if (planes) {
      fft_plane_pass(gs, g0, fftk::PlaneOut{1, 0, (int)(Ny * F), (int)F}, md.plan[0], Nx, Ny,
                     (int)F, 1, md.H[1], ghat2d_of<T>(md), tw_of<T>(md, 0), nullptr, s);
      for (int i = 3; i <= 6; ++i) mark(i);
      view(6, g0, Nx, Ny, 1, (int64_t)Ny * F, F);
      return;
    }
    if (first <= 3)
      fft_pass_contig(gs, g2, md.plan[1], Ny, Py, F * Nx, fftk::contig_map(Ny),
                      fftk::contig_map(Py), false, tw_of<T>(md, 1), s);
    mark(3);
    view(3, g2, Nx, Py, V2, Py, 1);
    if (stop <= 3) return;
    fft_mid_pass(g2, md.plan[0], Nx, (int)F, Py, 1, md.H[0], md.H[1], 1, ghat2d_of<T>(md),
                 tw_of<T>(md, 0), 0, V2, md.x_row[prec], s);
    mark(4);
    view(4, g2, Nx, Py, V2, Py, 1);
    if (stop <= 4) return;
    // into the field-interleaved plane [Nx][Ny][F] the interpolation reads
    fft_pass_contig(g2, g0, md.plan[1], Py, Ny, F * Nx, fftk::fields_inner(F, (int64_t)Nx * Py, Py, 1),
                    fftk::fields_inner(F, 1, (int64_t)Ny * F, F), true, tw_of<T>(md, 1), s);
    mark(5);
    mark(6);
    view(6, g0, Nx, Ny, 1, (int64_t)Ny * F, F);
    return;
  }
  if (planes) {
    // kz-outer grids gz and g1 [F][Pz][Nx][Ny] between the z passes
    const int64_t A1 = (int64_t)Nx * Ny, nl = md.n_occ_lines;
    cx<T> *g0 = buf(0, V0, true);
    cx<T> *g1 = buf(1, Pz * A1, true);
    cx<T> *gs = src_buffer<T>(pl, md, sizeof(cx<T>) * F * V0, 1, s);
    cx<T> *gz = zeroed_buffer<T>(pl, md.fzp, md.fzp_bytes, sizeof(cx<T>) * F * Pz * A1, s);
    if (reserve) return;
    mark(0);
    project<T, TX>(pl, md, nrhs, x, ldx, md.occ_ptr, md.occ, md.n_occ, gs, V0, s);
    mark(1);
    view(1, gs, A1, Nz, V0, Nz, 1);
    fft_zplane_pass(gs, gz, md.plan[2], Nz, Pz, (int)F, nl, md.occ_lines, md.occ_zrange, A1, false,
                    tw_of<T>(md, 2), s);
    mark(2);
    view(2, gz, A1, Pz, Pz * A1, 1, A1);
    fft_plane_pass(gz, g1, fftk::PlaneOut{Pz * A1, A1, Ny, 1}, md.plan[0], Nx, Ny, (int)F, Pz,
                   md.H[1], ghatp_of<T>(md), tw_of<T>(md, 0), md.occ_yrange, s);
    for (int i = 3; i <= 5; ++i) mark(i);
    view(5, g1, A1, Pz, Pz * A1, 1, A1);
    fft_zplane_pass(g1, g0, md.plan[2], Pz, Nz, (int)F, nl, md.occ_lines, md.occ_zrange, A1, true,
                    tw_of<T>(md, 2), s);
    view(6, g0, A1, Nz, 1, (int64_t)Nz * F, F);
    mark(6);
    return;
  }
  if (thin_layout<T>(Pz)) {
    // few kz (a flat scatterer): kz-outer layouts g1 [F][Pz][Nx][Ny] and
    // g2 [F][Pz][Nx][Py], no row padding; the y lines are contiguous, the x
    // pass tiles consecutive ky
    const int64_t A1 = (int64_t)Nx * Ny, V1 = Pz * A1, V2 = (int64_t)Pz * Nx * Py;
    cx<T> *g0 = buf(0, V0, stop > 5), *g1 = buf(1, V1, stop > 1), *g2 = buf(2, V2, stop > 2);
    cx<T> *gs = src_buffer<T>(pl, md, sizeof(cx<T>) * F * V0, 1, s);
    if (reserve) return;
    mark(0);
    if (first <= 1)
      project<T, TX>(pl, md, nrhs, x, ldx, md.occ_ptr, md.occ, md.n_occ, gs, V0, s);
    mark(1);
    view(1, gs, A1, Nz, V0, Nz, 1);
    if (stop <= 1) return;
    if (first <= 2)
      fft_pass_contig(gs, g1, md.plan[2], Nz, Pz, F * A1, fftk::contig_map(Nz),
                      fftk::contig_map(A1, V1, 1, A1), false, tw_of<T>(md, 2), s);
    mark(2);
    view(2, g1, A1, Pz, V1, 1, A1);
    if (stop <= 2) return;
    if (first <= 3)
      fft_pass_contig(g1, g2, md.plan[1], Ny, Py, F * Pz * Nx, fftk::contig_map(Ny),
                      fftk::contig_map(Py), false, tw_of<T>(md, 1), s);
    mark(3);
    view(3, g2, (int64_t)Nx * Py, Pz, V2, 1, (int64_t)Nx * Py);
    if (stop <= 3) return;
    fft_mid_pass(g2, md.plan[0], Nx, (int)F, Py, Pz, md.H[0], md.H[1], md.H[2], ghat_of<T>(md),
                 tw_of<T>(md, 0), 0, V2, md.x_row[prec], s);
    mark(4);
    view(4, g2, (int64_t)Nx * Py, Pz, V2, 1, (int64_t)Nx * Py);
    if (stop <= 4) return;
    fft_pass_contig(g2, g1, md.plan[1], Py, Ny, F * Pz * Nx, fftk::contig_map(Py),
                    fftk::contig_map(Ny), true, tw_of<T>(md, 1), s);
    mark(5);
    view(5, g1, A1, Pz, V1, 1, A1);
    if (stop <= 5) return;
    if (full3d) {  // inspection: every line
      fft_pass_contig(g1, g0, md.plan[2], Pz, Nz, F * A1, fftk::contig_map(A1, V1, 1, A1),
                      fftk::contig_map(Nz), true, tw_of<T>(md, 2), s);
    } else {  // the lines the interpolation reads
      // into the field-interleaved grid [Nx][Ny][Nz][F]
      const int64_t nl = md.n_occ_lines;
      fft_pass_contig(g1, g0, md.plan[2], Pz, Nz, F * nl,
                      fftk::fields_inner(F, V1, 1, A1, md.occ_lines, nl),
                      fftk::fields_inner(F, 1, (int64_t)Nz * F, F, md.occ_lines, nl), true,
                      tw_of<T>(md, 2), s);
      view(6, g0, A1, Nz, 1, (int64_t)Nz * F, F);
    }
    mark(6);
    return;
  }
  const int Pzs = (Pz + blk - 1) / blk * blk;  // z rows padded to 128-byte multiples
  const int64_t V1 = (int64_t)Nx * Ny * Pzs;
  const int64_t V2 = (int64_t)Nx * Py * ((Pz + blk - 1) / blk * blk);  // kz-blocked
  const int64_t A1 = (int64_t)Nx * Ny;
  cx<T> *g0 = buf(0, V0, stop > 5), *g1 = buf(1, V1, stop > 1), *g2 = buf(2, V2, stop > 2);
  const fftk::LineMap m1 = fftk::plain_map((int64_t)Ny * Pzs, Pzs);
  const fftk::LineMap m2 = fftk::blocked_map(V2, Nx, Py, blk);
  // projection fused with the forward z pass: the projected grid is never
  // stored (except for inspection, or for FFT lengths without a fused kernel).
  // The variant walks the right-hand sides in turn, so several take the two-launch
  // form (right-hand sides in parallel).
  const bool later = first > 2 && !reserve;  // (set-up) the passes after the forward z pass alone
  const bool fused = stop > 1 && md.fuse_proj[prec] && nrhs == 1 && fft_anterp_fused(md.plan[2]);
  cx<T> *gs = fused || later ? nullptr : src_buffer<T>(pl, md, sizeof(cx<T>) * F * V0, 1, s);
  // forward z output, forward y input: every line (fused, inspection), or the mesh's
  // zeroed buffer, of which the occupied lines are written
  const bool all_lines = (fused && !later) || full3d || stop <= 1;
  cx<T> *gz = all_lines ? g1 : zeroed_buffer<T>(pl, md.fz, md.fz_bytes, sizeof(cx<T>) * F * V1, s);
  if (reserve) return;
  mark(0);
  if (later) {
  } else if (fused) {
    if (!anterp_fftz(x, ldx, nrhs, md.node_ptr, md.ent_col, lamT_of<T>(md), Nz, A1, g1, Pzs, V1,
                     tw_of<T>(md, 2), md.plan[2], s))
      throw Error(AIM_ERR_ARG, "no fused projection for this FFT length");
    mark(1);
  } else {
    project<T, TX>(pl, md, nrhs, x, ldx, md.occ_ptr, md.occ, md.n_occ, gs, V0, s);
    mark(1);
    view(1, gs, A1, Nz, V0, Nz, 1);
    if (stop <= 1) return;
    if (full3d) {
      fft_pass_contig(gs, gz, md.plan[2], Nz, Pz, F * A1, fftk::contig_map(Nz),
                      fftk::contig_map(Pzs), false, tw_of<T>(md, 2), s);
    } else {
      const int64_t nl = md.n_occ_lines;
      fft_pass_contig(gs, gz, md.plan[2], Nz, Pz, F * nl,
                      fftk::select_lines(fftk::contig_map(Nz), md.occ_lines, nl, A1, md.occ_zrange),
                      fftk::select_lines(fftk::contig_map(Pzs), md.occ_lines, nl, A1), false,
                      tw_of<T>(md, 2), s);
    }
  }
  mark(2);
  view(2, gz, (int64_t)Nx * Ny, Pz, (int64_t)Nx * Ny * Pzs, Pzs, 1);
  if (stop <= 2) return;
  // y passes: rows outside a plane's occupied y range are zero on input
  // (forward) and never read on output (inverse); inspection keeps every row
  const fftk::LineMap m1y = full3d ? m1 : fftk::with_range(m1, md.occ_yrange, Nx);
  auto blocked_view = [&](int st) {
    if (!views) return;
    StageView &v = views[st];
    v = StageView{};
    v.p = g2;
    v.kind = 2;
    v.F = F;
    v.A = (int64_t)Nx * Py;
    v.Z = Pz;
    v.Nx = Nx;
    v.Py = Py;
    v.blk = blk;
    v.fstride = V2;
  };
  // the y, x and y passes pipelined over field groups (tuned at set-up) when
  // the product runs through; the stage boundaries then fall together (the
  // forward y step carries the time of all three)
  const int G = md.xy_groups[prec];
  if (stop >= 6 && !full3d && G > 1 && F % G == 0 &&
      xy_pipeline_available(md.plan[0], md.plan[1])) {
    fft_xy_pipeline(gz, g2, g1, md.plan[0], Nx, Ny, (int)F, G, Py, Pz, md.H[1], md.H[2],
                    ghat_of<T>(md), tw_of<T>(md, 0), tw_of<T>(md, 1), blk, V2, m1y, m2, s);
    mark(3);
    mark(4);
    blocked_view(4);
    mark(5);
  } else {
    if (first <= 3)
      fft_pass_strided(gz, g2, md.plan[1], Ny, Py, F * Nx, Pz, m1y, m2, false, tw_of<T>(md, 1),
                       md.y_row[prec], s);
    mark(3);
    blocked_view(3);
    if (stop <= 3) return;
    if (first <= 4)
      fft_mid_pass(g2, md.plan[0], Nx, (int)F, Py, Pz, md.H[0], md.H[1], md.H[2], ghat_of<T>(md),
                   tw_of<T>(md, 0), blk, V2, md.x_row[prec], s);
    mark(4);
    blocked_view(4);
    if (stop <= 4) return;
    fft_pass_strided(g2, g1, md.plan[1], Py, Ny, F * Nx, Pz, m2, m1y, true, tw_of<T>(md, 1),
                     md.y_row[prec], s);
    mark(5);
  }
  view(5, g1, (int64_t)Nx * Ny, Pz, (int64_t)Nx * Ny * Pzs, Pzs, 1);
  if (stop <= 5) return;
  if (full3d) {  // inspection: every line
    fft_pass_contig(g1, g0, md.plan[2], Pz, Nz, F * Nx * Ny, fftk::contig_map(Pzs),
                    fftk::contig_map(Nz), true, tw_of<T>(md, 2), s);
  } else {  // the lines the interpolation reads
    // into the field-interleaved grid [Nx][Ny][Nz][F]: the four fields of a
    // right-hand side at a stencil node are one 32-byte (c64) read
    const int64_t nl = md.n_occ_lines;
    fft_pass_contig(g1, g0, md.plan[2], Pz, Nz, F * nl,
                    fftk::fields_inner(F, V1, Pzs, 1, md.occ_lines, nl),
                    fftk::fields_inner(F, 1, (int64_t)Nz * F, F, md.occ_lines, nl, md.occ_zrange),
                    true, tw_of<T>(md, 2), s);
    view(6, g0, (int64_t)Nx * Ny, Nz, 1, (int64_t)Nz * F, F);
  }
  mark(6);
}

template <typename T, typename TX, typename TY>
void matvec_mesh(Plan *pl, MeshDev &md, int nrhs, const cx<TX> *x, int64_t ldx, cx<TY> *y,
                 int64_t ldy, hipStream_t s, hipEvent_t *ev) {
  const HostPlan &h = md.hp;
  const int prec = sizeof(T) == 8 ? 0 : 1;
  far_stages<T, TX>(pl, md, nrhs, x, ldx, 6, s, ev);
  const cx<T> *phi = (const cx<T> *)pl->work[md.lane][prec][0];
  const bool plane = md.planar_z >= 0;  // fields on the scatterer's grid plane only
  const int64_t nf = 4 * (int64_t)nrhs;  // fields per node of the interleaved grid
  const bool cf = h.cfie;
  if (cf && (plane || !curl_of<T>(md))) throw Error(AIM_ERR_STATE, "combined field without curl weights");
  auto launch = [&](auto kern, int r_first, int groups, int lanes = kRowLanes) {
    hipLaunchKernelGGL(kern, dim3(launch_blocks(h.n, 256 / lanes), groups), dim3(256), 0, s, phi, nf, r_first,
                       plane ? plane_lam_of<T>(md) : lam_of<T>(md), cf ? curl_of<T>(md) : nullptr,
                       plane ? md.plane_anchor : md.anchor_lin,
                       plane ? md.plane_soff : md.stencil_off, plane ? md.plane_K : h.K,
                       md.rowptr, md.cols, near_of<T>(md), x, ldx, y, ldy, h.n,
                       (T)(h.alpha * h.k * kEta0), (T)(1.0 / (h.k * h.k)),
                       (T)((1.0 - h.alpha) * kEta0));
  };
  // right-hand sides in groups of 4, then the 1 to 3 left over in one group
  auto groups = [&](auto cf_) {
    constexpr bool CF = decltype(cf_)::value;
    const int left = nrhs % 4, r_left = nrhs - left;
    if (r_left > 0) launch(k_interp_near<T, TX, TY, 4, CF>, 0, r_left / 4);
    if (left == 3)
      launch(k_interp_near<T, TX, TY, 3, CF>, r_left, 1);
    else if (left == 2)
      launch(k_interp_near<T, TX, TY, 2, CF>, r_left, 1);
    else if (left == 1 && !plane && h.n <= (h.K >= 64 ? kFewRows : kFewRowsLow))
      launch(k_interp_near<T, TX, TY, 1, CF, 32>, r_left, 1, 32);
    else if (left == 1)
      launch(k_interp_near<T, TX, TY, 1, CF>, r_left, 1);
  };
  // several right-hand sides: x transposed by the projection
  auto multi = [&](auto cf_, auto lr_) {
    constexpr bool CF = decltype(cf_)::value;
    constexpr int LR = decltype(lr_)::value;
    const cx<T> *xt = transposed_x<T, TX>(pl, md, nrhs, x, ldx, false, s);
    hipLaunchKernelGGL((k_interp_multi<T, TY, LR, CF>),
                       dim3(launch_blocks(h.n, kMultiRows), (nrhs + LR - 1) / LR),
                       dim3(kMultiThreads), 0, s, phi, nrhs,
                       plane ? plane_lam_of<T>(md) : lam_of<T>(md), cf ? curl_of<T>(md) : nullptr,
                       plane ? md.plane_anchor : md.anchor_lin,
                       plane ? md.plane_soff : md.stencil_off, plane ? md.plane_K : h.K, md.rowptr,
                       md.cols, near_of<T>(md), xt, y, ldy, h.n, (T)(h.alpha * h.k * kEta0),
                       (T)(1.0 / (h.k * h.k)), (T)((1.0 - h.alpha) * kEta0));
  };
  auto all = [&](auto cf_) {
    const int LR = multi_lanes<T>(md, nrhs);
    if (LR == 16)
      multi(cf_, std::integral_constant<int, 16>{});
    else if (LR == 8)
      multi(cf_, std::integral_constant<int, 8>{});
    else if (lone_rows(md, nrhs) && nrhs % 2 == 0)
      launch(k_interp_near<T, TX, TY, 2, decltype(cf_)::value, 32>, 0, nrhs / 2, 32);
    else if (lone_rows(md, nrhs))
      launch(k_interp_near<T, TX, TY, 1, decltype(cf_)::value>, 0, nrhs);
    else
      groups(cf_);
  };
  if (cf)
    all(std::true_type{});
  else
    all(std::false_type{});
  LAUNCHCHECK();
  if (ev) HIPCHECK(hipEventRecord(ev[7], s));
}

void assign_lanes(Plan *pl, const std::vector<double> &cost) {
  const int K = std::min(pl->nmesh, kMaxLanes);
  pl->nlanes = K;
  if (K > 1) {
    HIPCHECK(hipEventCreateWithFlags(&pl->lane_fork, hipEventDisableTiming));
    for (int l = 1; l < K; ++l) {
      HIPCHECK(hipStreamCreateWithFlags(&pl->lane_stream[l], hipStreamNonBlocking));
      HIPCHECK(hipEventCreateWithFlags(&pl->lane_join[l], hipEventDisableTiming));
    }
  }
  std::vector<int> order(pl->nmesh);
  for (int i = 0; i < pl->nmesh; ++i) order[i] = i;
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return cost[a] > cost[b]; });
  std::vector<double> load(K, 0.0);
  for (int i : order) {
    int l = 0;
    for (int j = 1; j < K; ++j)
      if (load[j] < load[l]) l = j;
    pl->mesh[i].lane = l;
    load[l] += cost[i];
  }
}

void release_lanes(Plan *pl) {
  for (int l = 1; l < kMaxLanes; ++l) {
    if (pl->lane_stream[l]) {
      (void)hipStreamSynchronize(pl->lane_stream[l]);
      (void)hipStreamDestroy(pl->lane_stream[l]);
    }
    if (pl->lane_join[l]) (void)hipEventDestroy(pl->lane_join[l]);
    pl->lane_stream[l] = nullptr;
    pl->lane_join[l] = nullptr;
  }
  if (pl->lane_fork) (void)hipEventDestroy(pl->lane_fork);
  pl->lane_fork = nullptr;
  pl->nlanes = 1;
}

void matvec_plan(Plan *pl, aim_precision prec, int nrhs, const void *x, void *y, hipStream_t s,
                 hipEvent_t *ev, const std::vector<char> *mesh_on) {
  const int64_t ld = pl->n_total;
  const bool lanes = pl->nlanes > 1 && !ev;
  if (lanes) {
    HIPCHECK(hipEventRecord(pl->lane_fork, s));
    for (int l = 1; l < pl->nlanes; ++l) HIPCHECK(hipStreamWaitEvent(pl->lane_stream[l], pl->lane_fork, 0));
  }
  int mi = 0;
  for (auto &md : pl->mesh) {
    if (mesh_on && !(*mesh_on)[mi]) {
      ++mi;
      continue;
    }
    const hipStream_t st = (lanes && md.lane > 0) ? pl->lane_stream[md.lane] : s;
    hipEvent_t *e = ev ? ev + (size_t)mi * (AIM_NSTAGE + 1) : nullptr;
    if (prec == AIM_FP64)
      matvec_mesh<double, double, double>(pl, md, nrhs, (const double2 *)x + md.offset, ld,
                                          (double2 *)y + md.offset, ld, st, e);
    else if (prec == AIM_MIXED)
      matvec_mesh<float, float, float>(pl, md, nrhs, (const float2 *)x + md.offset, ld,
                                       (float2 *)y + md.offset, ld, st, e);
    else
      matvec_mesh<float, double, double>(pl, md, nrhs, (const double2 *)x + md.offset, ld,
                                         (double2 *)y + md.offset, ld, st, e);
    ++mi;
  }
  if (lanes)
    for (int l = 1; l < pl->nlanes; ++l) {
      HIPCHECK(hipEventRecord(pl->lane_join[l], pl->lane_stream[l]));
      HIPCHECK(hipStreamWaitEvent(s, pl->lane_join[l], 0));
    }
}

template <typename T>
void copy_far_stage(Plan *pl, MeshDev &md, int nrhs, int stage, void *out, hipStream_t s) {
  const HostPlan &h = md.hp;
  const int prec = sizeof(T) == 8 ? 0 : 1;
  const int Nx = h.grid[0], Ny = h.grid[1], Nz = h.grid[2];
  const int Py = h.pad[1], Pz = h.pad[2];
  const int64_t F = 4 * (int64_t)nrhs;
  const int blk = kGridBlock<T>;
  const int64_t V2 = (int64_t)Nx * Py * ((Pz + blk - 1) / blk * blk);
  if (thin_layout<T>(Pz) && stage >= 2 && stage <= 5) {  // [F][Pz][A] -> [F][A][Pz]
    const int64_t A = (stage == 3 || stage == 4) ? (int64_t)Nx * Py : (int64_t)Nx * Ny;
    const int64_t tot = F * A * Pz;
    hipLaunchKernelGGL((k_kz_inner<T>), dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s,
                       (const cx<T> *)pl->work[md.lane][prec][(stage == 3 || stage == 4) ? 2 : 1],
                       (cx<T> *)out, F, A, Pz);
    LAUNCHCHECK();
    return;
  }
  if (stage == 3 || stage == 4) {
    const int64_t tot = F * Nx * Py * Pz;
    hipLaunchKernelGGL((k_unblock<T>), dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s,
                       (const cx<T> *)pl->work[md.lane][prec][2], (cx<T> *)out, F, Nx, Py, Pz, blk, V2);
    LAUNCHCHECK();
    return;
  }
  if (stage == 2 || stage == 5) {  // drop the row padding
    const int Pzs = (Pz + blk - 1) / blk * blk;
    HIPCHECK(hipMemcpy2DAsync(out, sizeof(cx<T>) * Pz, pl->work[md.lane][prec][1], sizeof(cx<T>) * Pzs,
                              sizeof(cx<T>) * Pz, (size_t)(F * Nx * Ny), hipMemcpyDeviceToDevice, s));
    return;
  }
  // stage 1: the projected source grid; stage 6: the propagated fields
  HIPCHECK(hipMemcpyAsync(out, stage == 1 ? md.src[prec] : pl->work[md.lane][prec][0],
                          sizeof(cx<T>) * F * Nx * Ny * Nz, hipMemcpyDeviceToDevice, s));
}
template void copy_far_stage<double>(Plan *, MeshDev &, int, int, void *, hipStream_t);
template void copy_far_stage<float>(Plan *, MeshDev &, int, int, void *, hipStream_t);

namespace {
// out[(f A + a) Z + z] = in[f fs + a as + z zs] (inspection)
template <typename T>
__global__ void k_view_copy(const cx<T> *__restrict__ in, cx<T> *__restrict__ out, int64_t F,
                            int64_t A, int64_t Z, int64_t fs, int64_t as, int64_t zs) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= F * A * Z) return;
  const int64_t z = t % Z, a = (t / Z) % A, f = t / (Z * A);
  out[t] = in[f * fs + a * as + z * zs];
}
}  // namespace

template <typename T>
void copy_stage_view(const StageView &v, void *out, hipStream_t s) {
  const int64_t tot = v.F * v.A * v.Z;
  const unsigned blocks = (unsigned)((tot + 255) / 256);
  if (v.kind == 1) {
    hipLaunchKernelGGL((k_view_copy<T>), dim3(blocks), dim3(256), 0, s, (const cx<T> *)v.p,
                       (cx<T> *)out, v.F, v.A, v.Z, v.fs, v.as, v.zs);
  } else if (v.kind == 2) {
    hipLaunchKernelGGL((k_unblock<T>), dim3(blocks), dim3(256), 0, s, (const cx<T> *)v.p,
                       (cx<T> *)out, v.F, v.Nx, v.Py, (int)v.Z, v.blk, v.fstride);
  } else {
    throw Error(AIM_ERR_ARG, "the product has no such stage for this mesh");
  }
  LAUNCHCHECK();
}
template void copy_stage_view<double>(const StageView &, void *, hipStream_t);
template void copy_stage_view<float>(const StageView &, void *, hipStream_t);

void autotune_mesh(Plan *pl, MeshDev &md, hipStream_t s) {
  const int64_t n = md.hp.n;
  // right-hand sides of the timed products (the caller's hint, else one)
  const int nr = std::max(1, (pl->params.tuning >> 16) & 0xff);
  hipEvent_t e0, e1;
  HIPCHECK(hipEventCreate(&e0));
  HIPCHECK(hipEventCreate(&e1));
  void *x = nullptr;
  try {
    x = dev_alloc(pl, sizeof(double2) * n * nr);
    HIPCHECK(hipMemsetAsync(x, 0, sizeof(double2) * n * nr, s));
    // the stages first .. stop alone (zero grids stay zero), with r right-hand sides
    auto time_stages = [&](int prec, int first, int stop, int r) {
      for (int rep = 0; rep < 4; ++rep) {  // first repetition is a warm-up
        if (rep == 1) HIPCHECK(hipEventRecord(e0, s));
        if (prec == 0)
          far_stages<double, double>(pl, md, r, (const double2 *)x, n, stop, s, nullptr, false,
                                     nullptr, first);
        else
          far_stages<float, double>(pl, md, r, (const double2 *)x, n, stop, s, nullptr, false,
                                    nullptr, first);
      }
      HIPCHECK(hipEventRecord(e1, s));
      HIPCHECK(hipEventSynchronize(e1));
      float ms = 0;
      HIPCHECK(hipEventElapsedTime(&ms, e0, e1));
      return ms;
    };
    // projection gather: occupied nodes per wave, with the most right-hand sides it
    // takes on any number of rows if nr are more (k_anterp_multi has no such variants)
    for (int prec = 0; prec < 2; ++prec) {
      if (prec == 1 && !pl->mixed) break;
      float best = 0;
      int choice = kGatherNpwCand[1];
      for (int c = 0; c < 3; ++c) {
        md.gather_npw[prec] = kGatherNpwCand[c];
        const float ms = time_stages(prec, 1, 1, std::min(nr, kMultiFrom - 1));
        if (c == 0 || ms < best) {
          best = ms;
          choice = kGatherNpwCand[c];
        }
      }
      md.gather_npw[prec] = choice;
    }
    // whether every product runs plane by plane
    auto all_planes = [&](int prec) {
      return plane_by_plane(md, prec, 1) && md.plane_fft[prec].hi == INT64_MAX;
    };
    // projection fused with the forward z pass, which one right-hand side alone takes
    for (int prec = 0; prec < 2; ++prec) {
      if (prec == 1 && !pl->mixed) break;
      const bool thin = prec == 0 ? thin_layout<double>(md.hp.pad[2]) : thin_layout<float>(md.hp.pad[2]);
      if (thin || all_planes(prec) || !fft_anterp_fused(md.plan[2])) {
        md.fuse_proj[prec] = 0;
        continue;
      }
      float best = 0;
      int choice = 0;
      for (int v = 0; v < 2; ++v) {
        md.fuse_proj[prec] = v;
        const float ms = time_stages(prec, 1, 2, 1);
        if (v == 0 || ms < best) {
          best = ms;
          choice = v;
        }
      }
      md.fuse_proj[prec] = choice;
    }
    // tile rows of the x pass and of the strided y passes, each pass timed alone
    // (timing the whole far part for all four combinations, and for the pipelined
    // y / x / y passes, took 107 ms of the 8-lambda sphere's set-up): 64-byte rows
    // halve a work-group's LDS tile, so more work-groups fit a CU, at the cost of
    // half-cache-line accesses. A variant must beat 128-byte rows by 3%, the
    // timing spread of products of one right-hand side; by 1% where several are
    // timed. The passes are pipelined over field groups only where the caller
    // asks for it: sequential passes were faster everywhere that was measured
    // (8-lambda sphere: 0.676 ms against 0.688 and 0.738 in 2 and 4 groups).
    const int rows = (pl->params.tuning >> 8) & 0xff;   // 1: 128-byte, 2: 64-byte rows everywhere
    const int groups = pl->params.tuning & 0xff;
    const float margin = nr > 1 ? 0.99f : 0.97f;
    for (int prec = 0; prec < 2; ++prec) {
      if (prec == 1 && !pl->mixed) break;
      const bool thin =
          md.planar_z >= 0 ||
          (prec == 0 ? thin_layout<double>(md.hp.pad[2]) : thin_layout<float>(md.hp.pad[2]));
      md.xy_groups[prec] = 1;
      md.x_row[prec] = md.y_row[prec] = rows == 2 ? 64 : 128;
      if (rows == 0 && !all_planes(prec)) {
        const float x128 = time_stages(prec, 4, 4, nr);
        md.x_row[prec] = 64;
        if (time_stages(prec, 4, 4, nr) >= margin * x128) md.x_row[prec] = 128;
        if (!thin) {  // (the y lines of the thin layouts are contiguous)
          const float y128 = time_stages(prec, 3, 3, nr) + time_stages(prec, 5, 5, nr);
          md.y_row[prec] = 64;
          if (time_stages(prec, 3, 3, nr) + time_stages(prec, 5, 5, nr) >= margin * y128)
            md.y_row[prec] = 128;
        }
      }
      if (groups > 0 && !thin && xy_pipeline_available(md.plan[0], md.plan[1]))
        md.xy_groups[prec] = groups;
    }
    // every buffer of a product with up to nr right-hand sides, so that none is
    // allocated by the first one (which may be captured into a graph): those of nr
    // and of the most below that whose passes are the others (separate or plane by plane)
    for (int prec = 0; prec < 2; ++prec) {
      if (prec == 1 && !pl->mixed) break;
      auto reserve = [&](int r) {
        if (prec == 0)
          far_stages<double, double>(pl, md, r, nullptr, n, 6, s, nullptr, false, nullptr, 7);
        else
          far_stages<float, double>(pl, md, r, nullptr, n, 6, s, nullptr, false, nullptr, 7);
      };
      reserve(nr);
      int other = nr - 1;
      while (other > 0 && plane_by_plane(md, prec, other) == plane_by_plane(md, prec, nr)) --other;
      if (other > 0) reserve(other);
    }
  } catch (...) {
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (x) dev_free(pl, x);
    throw;
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  dev_free(pl, x);
}

template void far_stages<double, double>(Plan *, MeshDev &, int, const double2 *, int64_t, int,
                                         hipStream_t, hipEvent_t *, bool, StageView *, int);
template void far_stages<float, float>(Plan *, MeshDev &, int, const float2 *, int64_t, int,
                                       hipStream_t, hipEvent_t *, bool, StageView *, int);
template void far_stages<float, double>(Plan *, MeshDev &, int, const double2 *, int64_t, int,
                                        hipStream_t, hipEvent_t *, bool, StageView *, int);
template void matvec_mesh<double, double, double>(Plan *, MeshDev &, int, const double2 *, int64_t,
                                                  double2 *, int64_t, hipStream_t, hipEvent_t *);
template void matvec_mesh<float, float, float>(Plan *, MeshDev &, int, const float2 *, int64_t,
                                               float2 *, int64_t, hipStream_t, hipEvent_t *);
template void matvec_mesh<float, double, double>(Plan *, MeshDev &, int, const double2 *, int64_t,
                                                 double2 *, int64_t, hipStream_t, hipEvent_t *);

}  // namespace aim
