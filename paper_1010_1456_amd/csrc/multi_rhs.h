// Projection, and interpolation with the near product, for several right-hand
// sides: a lane per right-hand side.
//
// x is first transposed to [n][R] (in the product's arithmetic), so that the R
// values of one basis are adjacent, as the R x 4 fields of a grid node already
// are; 8 or 16 lanes (LR) then hold one right-hand side each, so that a gather is
// one run of LR values instead of 64 scattered ones. Half a wave takes a node
// (row): its 32 / LR groups of lanes walk every (32 / LR)-th entry and add their
// sums by exchanges in a fixed order (a group alone per row waits on a chain four
// times as long, and a whole wave per row leaves most of it idle: 4-lambda CFIE
// sphere, 16 right-hand sides, c64, with 8 near sums per row: 64 + 118 us and 87 + 110
// against 70 + 101).
// The entries, columns and weights, the same for all right-hand sides, are staged
// through LDS, and results leave through LDS so that stores run along nodes
// (rows). Bound by the latency of those gathers and the L1 traffic of the fields
// (27 x 512 bytes per row and 16 right-hand sides). One right-hand side per launch
// row in the projection and four in the interpolation took 94 + 183 us there (now 71 +
// 114), and 227 + 360 in FP64 at third order on the 2.7-lambda sphere (now 73 + 162).
#pragma once

#include "aim_internal.h"

namespace aim {
namespace {

constexpr int kMultiThreads = 256;
constexpr int kMultiRows = kMultiThreads / 32;  // nodes (rows) per work-group
// Partial sums per lane: of the near product 16 per row, of some 5 entries each, added
// in pairs, the last two to the far part. With 8 in float the product's error against
// FP64 is 1.04e-7 on the 2-lambda sphere (16 right-hand sides) where 32 lanes per row,
// one right-hand side at a time, have 0.978e-7; with 16 it is 0.930e-7 (0.977e-7 where
// the near sum is complete before it meets the far part, which it partly cancels), and
// the interpolation takes 114 us on the 4-lambda sphere (8: 117). FP64, 8 and 16 and
// those 32 lanes: 1.66e-16, 1.53e-16 and 1.56e-16 (1-lambda sphere, this kernel alone),
// 203 and 201 us.
template <int SEG>
constexpr int near_sums() {
  return 16 / SEG;
}
// of the stencil and the projection (float 8 per row; with 16 the interpolation takes
// 150 us there, in FP64 with 8 271)
template <typename T, int SEG>
constexpr int stencil_sums() {
  return sizeof(T) == 4 ? 8 / SEG : 2;
}

// xt[i R + r] = x[r ldx + i]
template <typename T, typename TX>
__global__ void __launch_bounds__(kMultiThreads)
    k_transpose_x(const cx<TX> *__restrict__ x, int64_t ldx, int R, int64_t n,
                  cx<T> *__restrict__ xt) {
  __shared__ cx<T> tile[64][17];
  const int64_t i0 = (int64_t)blockIdx.x * 64;
  const int r0 = blockIdx.y * 16;
  const int li = threadIdx.x & 63;
  for (int r = threadIdx.x >> 6; r < 16; r += kMultiThreads / 64)
    if (r0 + r < R && i0 + li < n) {
      const cx<TX> v = x[(int64_t)(r0 + r) * ldx + i0 + li];
      tile[li][r].x = (T)v.x;
      tile[li][r].y = (T)v.y;
    }
  __syncthreads();
  const int r = threadIdx.x & 15;
  for (int i = threadIdx.x >> 4; i < 64; i += kMultiThreads / 16)
    if (r0 + r < R && i0 + i < n) xt[(i0 + i) * R + r0 + r] = tile[i][r];
}

// Projection of right-hand sides blockIdx.y LR .. onto occupied nodes: as
// k_anterp_gather over occ / occ_ptr.
template <typename T>
constexpr int gather_chunk() {  // entries staged at a time
  return sizeof(T) == 4 ? 768 : 384;
}
template <typename T, int LR>
__global__ void __launch_bounds__(kMultiThreads)
    k_anterp_multi(const cx<T> *__restrict__ xt, int R, const int32_t *__restrict__ occ_ptr,
                   const int32_t *__restrict__ occ, const int32_t *__restrict__ ent_col,
                   const T *__restrict__ lamT, cx<T> *__restrict__ grid, int64_t n_occ,
                   int64_t Vg) {
  constexpr int SEG = 32 / LR, NB = kMultiRows, C = gather_chunk<T>();
  constexpr int kOut = 4 * LR * (NB + 1);  // [4 LR fields][NB nodes], padded
  constexpr size_t kStage = C * (4 * sizeof(T) + sizeof(int32_t)), kBytes = kOut * sizeof(cx<T>);
  __shared__ __align__(16) unsigned char lds[kStage > kBytes ? kStage : kBytes];
  T *wl = reinterpret_cast<T *>(lds);  // [C][4]
  int32_t *cl = reinterpret_cast<int32_t *>(wl + 4 * C);
  const int r = threadIdx.x % LR, seg = threadIdx.x / LR % SEG, g = threadIdx.x / 32;
  const int64_t v0 = (int64_t)blockIdx.x * NB, vend = min(v0 + NB, n_occ);
  const bool ok = v0 + g < n_occ;
  const int e0 = ok ? occ_ptr[v0 + g] : 0, e1 = ok ? occ_ptr[v0 + g + 1] : 0;
  const int b0 = occ_ptr[v0], b1 = occ_ptr[vend];
  const int rr = blockIdx.y * LR + r;
  const cx<T> *xr = xt + (rr < R ? rr : R - 1);
  constexpr int NS = stencil_sums<T, SEG>();
  T a[NS][4][2];
#pragma unroll
  for (int j = 0; j < NS; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q) a[j][q][0] = a[j][q][1] = 0;
  for (int c0 = b0; c0 < b1; c0 += C) {
    const int cnt = min(C, b1 - c0);
    __syncthreads();
    for (int i = threadIdx.x; i < cnt; i += kMultiThreads) cl[i] = ent_col[c0 + i];
    for (int i = threadIdx.x; i < 4 * cnt; i += kMultiThreads) wl[i] = lamT[4 * (int64_t)c0 + i];
    __syncthreads();
    const int hi = min(e1 - c0, cnt);
    auto add = [&](T(&s)[4][2], int k, cx<T> xv) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        s[q][0] += wl[4 * k + q] * xv.x;
        s[q][1] += wl[4 * k + q] * xv.y;
      }
    };
    int k = max(e0 - c0, 0) + seg;
    for (; k + (NS - 1) * SEG < hi; k += NS * SEG) {
      cx<T> xv[NS];
#pragma unroll
      for (int j = 0; j < NS; ++j) xv[j] = xr[(int64_t)cl[k + j * SEG] * R];
#pragma unroll
      for (int j = 0; j < NS; ++j) add(a[j], k + j * SEG, xv[j]);
    }
#pragma unroll
    for (int j = 0; j < NS - 1; ++j)
      if (k + j * SEG < hi) add(a[j], k + j * SEG, xr[(int64_t)cl[k + j * SEG] * R]);
  }
#pragma unroll
  for (int h = NS / 2; h > 0; h /= 2)
#pragma unroll
    for (int j = 0; j < h; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        a[j][q][0] += a[j + h][q][0];
        a[j][q][1] += a[j + h][q][1];
      }
#pragma unroll
  for (int off = LR; off < 32; off <<= 1)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      a[0][q][0] += __shfl_xor(a[0][q][0], off, 64);
      a[0][q][1] += __shfl_xor(a[0][q][1], off, 64);
    }
  __syncthreads();
  cx<T> *out = reinterpret_cast<cx<T> *>(lds);
  if (seg == 0)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      out[(4 * r + q) * (NB + 1) + g].x = a[0][q][0];
      out[(4 * r + q) * (NB + 1) + g].y = a[0][q][1];
    }
  __syncthreads();
  const int i = threadIdx.x % NB;  // node of the store
  if (v0 + i >= n_occ) return;
  const int64_t node = occ[v0 + i];
  const int f0 = blockIdx.y * 4 * LR;
  for (int f = threadIdx.x / NB; f < 4 * LR; f += 32)
    if (f0 + f < 4 * R) grid[(int64_t)(f0 + f) * Vg + node] = out[f * (NB + 1) + i];
}

// Interpolation and near product of right-hand sides blockIdx.y LR ..: as
// k_interp_near.
template <typename T>
constexpr int near_chunk() {  // entries staged at a time
  return sizeof(T) == 4 ? 1024 : 640;
}
constexpr int kWeightLds = 14 * 1024;  // stencil weights staged at a time, bytes
template <typename T, typename TY, int LR, bool CF>
__global__ void __launch_bounds__(kMultiThreads)
    k_interp_multi(const cx<T> *__restrict__ phi, int R, const T *__restrict__ lam,
                   const T *__restrict__ curl, const int32_t *__restrict__ anchor_lin,
                   const int32_t *__restrict__ soff, int K, const int32_t *__restrict__ rowptr,
                   const int32_t *__restrict__ cols, const cx<T> *__restrict__ nearv,
                   const cx<T> *__restrict__ xt, cx<TY> *__restrict__ y, int64_t ldy, int64_t n,
                   T keta, T inv_k2, T eta_h) {
  using V = cx<T>;
  constexpr int SEG = 32 / LR, RB = kMultiRows, C = near_chunk<T>();  // rows, entries
  constexpr int Q = CF ? 7 : 4;                               // weights per node
  constexpr int UC0 = kWeightLds / (RB * Q * (int)sizeof(T));
  constexpr int UC = UC0 < 216 ? UC0 : 216;  // nodes of weights staged
  static_assert(UC >= 1, "weight staging");
  constexpr size_t kStage = C * (sizeof(V) + sizeof(int32_t));
  constexpr size_t kOut = (size_t)LR * (RB + 1) * sizeof(cx<TY>);
  constexpr size_t kMost = kStage > kOut ? kStage : kOut;
  __shared__ __align__(16) unsigned char lds[kMost > kWeightLds ? kMost : kWeightLds];
  __shared__ int32_t sl[UC];
  const int r = threadIdx.x % LR, seg = threadIdx.x / LR % SEG, g = threadIdx.x / 32;
  const int64_t m0 = (int64_t)blockIdx.x * RB, mend = min(m0 + RB, n);
  const bool ok = m0 + g < n;
  const int64_t m = ok ? m0 + g : n - 1;
  const int rr = blockIdx.y * LR + r, rc = rr < R ? rr : R - 1;
  const int e0 = rowptr[m], e1 = rowptr[m + 1], b0 = rowptr[m0], b1 = rowptr[mend];
  const V *ph = phi + ((int64_t)anchor_lin[m] * R + rc) * 4;
  constexpr int NN = near_sums<SEG>(), NF = stencil_sums<T, SEG>();  // far and near sums per lane
  V far[NF], fk[NF], nr[NN];
#pragma unroll
  for (int j = 0; j < NF; ++j) far[j].x = far[j].y = fk[j].x = fk[j].y = 0;
#pragma unroll
  for (int j = 0; j < NN; ++j) nr[j].x = nr[j].y = 0;
  // stencil: weights [q][rows][UC] of UC nodes at a time
  T *wl = reinterpret_cast<T *>(lds);
  for (int u0 = 0; u0 < K; u0 += UC) {
    const int uc = min(UC, K - u0);
    __syncthreads();
    for (int i = threadIdx.x; i < RB * 4 * uc; i += kMultiThreads) {
      const int u = i % uc, row = i / uc / 4, q = i / uc % 4;
      const int64_t mm = min(m0 + row, n - 1);
      wl[(row * Q + q) * UC + u] = lam[(mm * 4 + q) * K + u0 + u];
    }
    if (CF)
      for (int i = threadIdx.x; i < RB * 3 * uc; i += kMultiThreads) {
        const int u = i % uc, row = i / uc / 3, q = i / uc % 3;
        const int64_t mm = min(m0 + row, n - 1);
        wl[(row * Q + 4 + q) * UC + u] = curl[(mm * 3 + q) * K + u0 + u];
      }
    for (int i = threadIdx.x; i < uc; i += kMultiThreads) sl[i] = soff[u0 + i];
    __syncthreads();
    const T *w = wl + g * Q * UC;
    auto add = [&](V &f, V &c, int u) {
      const V *p = ph + (int64_t)sl[u] * (4 * R);
      const V p0 = p[0], p1 = p[1], p2 = p[2], p3 = p[3];
      const T l0 = w[u], l1 = w[UC + u], l2 = w[2 * UC + u], l3 = inv_k2 * w[3 * UC + u];
      f.x += l0 * p0.x + l1 * p1.x + l2 * p2.x - l3 * p3.x;
      f.y += l0 * p0.y + l1 * p1.y + l2 * p2.y - l3 * p3.y;
      if (CF) {
        const T w0 = w[4 * UC + u], w1 = w[5 * UC + u], w2 = w[6 * UC + u];
        c.x += w0 * p0.x + w1 * p1.x + w2 * p2.x;
        c.y += w0 * p0.y + w1 * p1.y + w2 * p2.y;
      }
    };
    int u = seg;
    for (; u + (NF - 1) * SEG < uc; u += NF * SEG)
#pragma unroll
      for (int j = 0; j < NF; ++j) add(far[j], fk[j], u + j * SEG);
#pragma unroll
    for (int j = 0; j < NF - 1; ++j)
      if (u + j * SEG < uc) add(far[j], fk[j], u + j * SEG);
  }
  auto halve = [&](V *v, int h) {  // v[j] += v[j + h], j < h
#pragma unroll
    for (int j = 0; j < h; ++j) {
      v[j].x += v[j + h].x;
      v[j].y += v[j + h].y;
    }
  };
#pragma unroll
  for (int h = NF / 2; h > 0; h /= 2) halve(far, h), halve(fk, h);
  // near zone: entries of the work-group's rows, C at a time
  V *zl = reinterpret_cast<V *>(lds);
  int32_t *cl = reinterpret_cast<int32_t *>(zl + C);
  for (int c0 = b0; c0 < b1; c0 += C) {
    const int cnt = min(C, b1 - c0);
    __syncthreads();
    for (int i = threadIdx.x; i < cnt; i += kMultiThreads) {
      zl[i] = nearv[c0 + i];
      cl[i] = cols[c0 + i];
    }
    __syncthreads();
    const int hi = min(e1 - c0, cnt);
    int k = max(e0 - c0, 0) + seg;
    for (; k + (NN - 1) * SEG < hi; k += NN * SEG) {
      V xv[NN];
#pragma unroll
      for (int j = 0; j < NN; ++j) xv[j] = xt[(int64_t)cl[k + j * SEG] * R + rc];
#pragma unroll
      for (int j = 0; j < NN; ++j) {
        const V z = zl[k + j * SEG];
        nr[j].x += z.x * xv[j].x - z.y * xv[j].y;
        nr[j].y += z.x * xv[j].y + z.y * xv[j].x;
      }
    }
#pragma unroll
    for (int j = 0; j < NN - 1; ++j)
      if (k + j * SEG < hi) {
        const V xv = xt[(int64_t)cl[k + j * SEG] * R + rc], z = zl[k + j * SEG];
        nr[j].x += z.x * xv.x - z.y * xv.y;
        nr[j].y += z.x * xv.y + z.y * xv.x;
      }
  }
#pragma unroll
  for (int h = NN / 2; h >= 2; h /= 2) halve(nr, h);
  V acc;
  acc.x = -keta * far[0].y - (CF ? eta_h * fk[0].x : (T)0);  // j k eta * far
  acc.y = keta * far[0].x - (CF ? eta_h * fk[0].y : (T)0);
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    acc.x += nr[j].x;
    acc.y += nr[j].y;
  }
#pragma unroll
  for (int off = LR; off < 32; off <<= 1) {
    acc.x += __shfl_xor(acc.x, off, 64);
    acc.y += __shfl_xor(acc.y, off, 64);
  }
  cx<TY> o;
  o.x = (TY)acc.x;
  o.y = (TY)acc.y;
  __syncthreads();
  cx<TY> *out = reinterpret_cast<cx<TY> *>(lds);  // [LR][RB + 1]
  if (seg == 0) out[r * (RB + 1) + g] = o;
  __syncthreads();
  const int i = threadIdx.x % RB;
  if (threadIdx.x < LR * RB && m0 + i < n && blockIdx.y * LR + threadIdx.x / RB < R)
    y[(int64_t)(blockIdx.y * LR + threadIdx.x / RB) * ldy + m0 + i] =
        out[(threadIdx.x / RB) * (RB + 1) + i];
}

}  // namespace
}  // namespace aim
