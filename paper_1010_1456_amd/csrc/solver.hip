// Restarted GMRES with right Jacobi preconditioning (the matvec's caller).
//
// The paper solves with a diagonal preconditioner and stops on the relative
// RMS residual (Section 2.2). Here every (mesh, plane wave) pair is its own
// system; all systems advance in lock-step so one batched AIM product serves
// them all. Arnoldi runs in FP64 on the device (classical Gram-Schmidt, two
// passes), and so do the Givens rotations and the residual estimate; the host
// only polls the per-system active flags every few iterations. The steps
// between two polls are captured once into a HIP graph and replayed (the
// launch sequence of a segment depends only on its step range, the precision
// and the buffers, which persist in the plan across solves). For AIM_MIXED the
// inner solves use the c64 operator on c128 Krylov vectors, inside an FP64
// iterative-refinement loop r = b - A64 x that decides convergence.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <complex>
#include <map>
#include <tuple>
#include <type_traits>

#include "aim_internal.h"

namespace aim {

namespace {

constexpr int kRed = 256;

__device__ inline double2 block_sum2(double a, double b) {
  __shared__ double sa[kRed / 64], sb[kRed / 64];
  for (int off = 32; off > 0; off >>= 1) {
    a += __shfl_xor(a, off, 64);
    b += __shfl_xor(b, off, 64);
  }
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    sa[w] = a;
    sb[w] = b;
  }
  __syncthreads();
  double ra = 0, rb = 0;
  if (threadIdx.x == 0)
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) {
      ra += sa[i];
      rb += sb[i];
    }
  return make_double2(ra, rb);
}

// One pass over the Krylov basis of the Gram-Schmidt step: with SUB, w -= V h
// (h[i S + s], or the sum of the np partials of an earlier pass in hpart, then also
// put into, or with `second` added to, column j of H); with DOTS, the partial dot
// products V_i^H w of the (new) w into part[(i S + s) np_stride + blockIdx.x]; with NORM, the partial |w|^2 of the new
// w into npart[s kNormParts + blockIdx.x]. Classical Gram-Schmidt twice is then
// three passes over V instead of four, the middle one (SUB and DOTS) keeping its
// tile of V in registers between the two uses.
//
// Bound by the read of V (N nv 16 bytes, from HBM or the last-level cache). A
// work-group's 256 threads are 16 rows x 16 vector groups: thread (lr, g) holds
// rows lr + 16 k (k < RP) of vectors g + 16 t (t < SLOTS), all loads of a tile
// in flight at once, so that also a basis of a few thousand rows fills the chip.
// With a thread per row (subtraction) or per 8 rows and 8 vectors (dots) the
// 16-lambda plate's steps (N = 61 920, 50 vectors on average) had 242 and 217
// work-groups on 256 CUs and took 16 and 22 us a pass, at 3.1 and 2.3 TB/s.
constexpr int kTileLanes = 16;  // row lanes, and vector groups, of a work-group
constexpr int kNormParts = 1024;  // upper bound of the grid's x extent
template <int SLOTS, int RP, bool SUB, bool DOTS, bool NORM>
__global__ void __launch_bounds__(256)
    k_basis_pass(const double2 *__restrict__ V, double2 *__restrict__ w, int64_t ld,
                 int64_t vstride, int64_t lo, int64_t n, int nv, int sys0, int S,
                 const double2 *__restrict__ h, const double2 *__restrict__ hpart, int np,
                 bool second, double2 *__restrict__ H, int m, int j, int64_t np_stride,
                 double2 *__restrict__ part, double *__restrict__ npart) {
  constexpr int ROWS = kTileLanes * RP;
  __shared__ double2 hs[SUB ? SLOTS * 16 : 1];
  __shared__ double2 red[SUB ? 2 : 1][4][ROWS];
  const int r = blockIdx.y, s = sys0 + r;
  const int lr = threadIdx.x & 15, g = threadIdx.x >> 4;
  const int wave = threadIdx.x >> 6;
  V += (int64_t)r * ld + lo;
  w += (int64_t)r * ld + lo;
  if (SUB) {
    for (int i = threadIdx.x; i < SLOTS * 16; i += 256) {
      double2 c = make_double2(0.0, 0.0);
      if (i < nv && np > 0) {
        for (int p = 0; p < np; ++p) {
          const double2 q = hpart[((int64_t)i * S + s) * np_stride + p];
          c.x += q.x;
          c.y += q.y;
        }
        if (blockIdx.x == 0) {
          double2 *hc = &H[((int64_t)s * (m + 1) + i) * m + j];
          *hc = second ? make_double2(hc->x + c.x, hc->y + c.y) : c;
        }
      } else if (i < nv) {
        c = h[(int64_t)i * S + s];
      }
      hs[i] = c;
    }
    __syncthreads();
  }
  double2 acc[DOTS ? SLOTS : 1];
  double nrm = 0.0;
#pragma unroll
  for (int t = 0; t < (DOTS ? SLOTS : 1); ++t) acc[t] = make_double2(0.0, 0.0);
  int par = 0;
  for (int64_t row0 = (int64_t)blockIdx.x * ROWS; row0 < n; row0 += (int64_t)gridDim.x * ROWS) {
    double2 v[SLOTS][RP], wv[RP];
#pragma unroll
    for (int t = 0; t < SLOTS; ++t)
#pragma unroll
      for (int k = 0; k < RP; ++k) {
        const int64_t row = row0 + lr + 16 * k;
        const int i = g + 16 * t;
        v[t][k] = (i < nv && row < n) ? V[(int64_t)i * vstride + row] : make_double2(0.0, 0.0);
      }
#pragma unroll
    for (int k = 0; k < RP; ++k) {
      const int64_t row = row0 + lr + 16 * k;
      wv[k] = row < n ? w[row] : make_double2(0.0, 0.0);
    }
    if (SUB) {
      double2 p[RP];
#pragma unroll
      for (int k = 0; k < RP; ++k) p[k] = make_double2(0.0, 0.0);
#pragma unroll
      for (int t = 0; t < SLOTS; ++t) {
        const double2 c = hs[g + 16 * t];
#pragma unroll
        for (int k = 0; k < RP; ++k) {
          p[k].x += c.x * v[t][k].x - c.y * v[t][k].y;
          p[k].y += c.x * v[t][k].y + c.y * v[t][k].x;
        }
      }
      // over the 16 vector groups: 4 in each wave, then the 4 waves (the buffer
      // of the tile before last is free: every thread has passed its barrier)
#pragma unroll
      for (int off = 16; off < 64; off <<= 1)
#pragma unroll
        for (int k = 0; k < RP; ++k) {
          p[k].x += __shfl_xor(p[k].x, off, 64);
          p[k].y += __shfl_xor(p[k].y, off, 64);
        }
      if ((g & 3) == 0)
#pragma unroll
        for (int k = 0; k < RP; ++k) red[par][wave][lr + 16 * k] = p[k];
      __syncthreads();
#pragma unroll
      for (int k = 0; k < RP; ++k) {
        double2 q = red[par][0][lr + 16 * k];
#pragma unroll
        for (int u = 1; u < 4; ++u) {
          q.x += red[par][u][lr + 16 * k].x;
          q.y += red[par][u][lr + 16 * k].y;
        }
        wv[k].x -= q.x;
        wv[k].y -= q.y;
        const int64_t row = row0 + lr + 16 * k;
        if (g == 0 && row < n) w[row] = wv[k];
      }
      par ^= 1;
    }
    if (NORM)
#pragma unroll
      for (int k = 0; k < RP; ++k) nrm += wv[k].x * wv[k].x + wv[k].y * wv[k].y;
    if (DOTS)
#pragma unroll
      for (int t = 0; t < SLOTS; ++t)
#pragma unroll
        for (int k = 0; k < RP; ++k) {
          acc[t].x += v[t][k].x * wv[k].x + v[t][k].y * wv[k].y;
          acc[t].y += v[t][k].x * wv[k].y - v[t][k].y * wv[k].x;
        }
  }
  for (int off = 1; off < 16; off <<= 1) {  // over the 16 row lanes
    if (NORM) nrm += __shfl_xor(nrm, off, 64);
    if (DOTS)
#pragma unroll
      for (int t = 0; t < SLOTS; ++t) {
        acc[t].x += __shfl_xor(acc[t].x, off, 64);
        acc[t].y += __shfl_xor(acc[t].y, off, 64);
      }
  }
  if (NORM && threadIdx.x == 0) npart[(int64_t)s * kNormParts + blockIdx.x] = nrm;
  if (DOTS && lr == 0)
#pragma unroll
    for (int t = 0; t < SLOTS; ++t) {
      const int i = g + 16 * t;
      if (i < nv) part[((int64_t)i * S + s) * np_stride + blockIdx.x] = acc[t];
    }
}
// Up to this many partials per sum are added by the next pass itself: a launch of
// its own for them costs more where the basis is short (1-lambda plate, 4 partials:
// 40 -> 35 us per step and product; the passes then write alternate halves of part)
constexpr int kInlineParts = 16;
// work-groups per system of a pass over n rows with R right-hand sides: one per
// 64-row tile up to about 8 per CU over all systems
int64_t basis_groups(int64_t n, int R) {
  const int64_t most = std::min<int64_t>(kNormParts, std::max<int64_t>(64, 2048 / R));
  return std::max<int64_t>(1, std::min<int64_t>(most, (n + 63) / 64));
}

// out[i S + s] = sum_{p < np} part[(i S + s) np_stride + p], fixed order;
// blockIdx.x = i, blockIdx.y = s - sys0. With add (the second pass), the sum of
// both passes goes to column j of H as well. (A work-group per sum: with a wave the
// up to 1024 partials came 16 loads deep, 5.8 us on the 16-lambda plate, now 3.6.)
__global__ void __launch_bounds__(kRed)
    k_part_reduce(const double2 *part, int64_t np_stride, int np, int sys0, int S, double2 *out,
                  const double2 *add, double2 *H, int m, int j) {
  const int s = sys0 + blockIdx.y;
  const int64_t row = (int64_t)blockIdx.x * S + s;
  const double2 *pp = part + row * np_stride;
  double a = 0, b = 0;
  for (int q = threadIdx.x; q < np; q += kRed) {
    a += pp[q].x;
    b += pp[q].y;
  }
  const double2 t = block_sum2(a, b);
  if (threadIdx.x == 0) {
    out[row] = t;
    if (add)
      H[((int64_t)s * (m + 1) + blockIdx.x) * m + j] = make_double2(add[row].x + t.x, add[row].y + t.y);
  }
}

// part[s kNormParts + blockIdx.x] = sum |w|^2 over the block's rows of system
// s (grid-stride); k_norm_reduce adds the partials in a fixed order
__global__ void __launch_bounds__(kRed)
    k_norm2_part(const double2 *w, int64_t ld, int64_t lo, int64_t hi, int sys0, double *part) {
  const int r = blockIdx.y;
  double a = 0;
  for (int64_t n = lo + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; n < hi;
       n += (int64_t)gridDim.x * blockDim.x) {
    const double2 p = w[(int64_t)r * ld + n];
    a += p.x * p.x + p.y * p.y;
  }
  const double2 t = block_sum2(a, 0.0);
  if (threadIdx.x == 0) part[(int64_t)(sys0 + r) * kNormParts + blockIdx.x] = t.x;
}
__global__ void __launch_bounds__(64)
    k_norm_reduce(const double *part, int np, int sys0, double *nrm) {
  const int s = sys0 + blockIdx.x;
  double a = 0;
  for (int q = threadIdx.x; q < np; q += 64) a += part[(int64_t)s * kNormParts + q];
  for (int off = 32; off > 0; off >>= 1) a += __shfl_xor(a, off, 64);
  if (threadIdx.x == 0) nrm[s] = a;
}

// out[r][row] = w[r][row] / sqrt(nrm[s]) (0 if nrm == 0)
__global__ void k_normalize(const double2 *w, double2 *out, int64_t ld, int64_t lo, int64_t hi,
                            int sys0, const double *nrm) {
  const int r = blockIdx.y;
  const int64_t n = lo + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= hi) return;
  const double s = nrm[sys0 + r];
  const double inv = s > 0 ? 1.0 / sqrt(s) : 0.0;
  const double2 p = w[(int64_t)r * ld + n];
  out[(int64_t)r * ld + n] = make_double2(p.x * inv, p.y * inv);
}

// The end of an Arnoldi step in one launch: the squared norm of w from the last
// basis pass' partials (every work-group adds them in the same order;
// work-group 0 stores it for the Givens kernel), v_{j+1} =
// w / |w| into out, and the next step's preconditioned vector
// z = dinv v_{j+1} (what k_precond would compute from out).
__global__ void __launch_bounds__(kRed)
    k_normalize_next(const double2 *w, double2 *out, double2 *z, const double2 *dinv, int64_t ld,
                     int64_t lo, int64_t hi, int sys0, const double *part, int np, double *nrm) {
  __shared__ double snrm;
  const int r = blockIdx.y;
  const int s = sys0 + r;
  const int64_t n = lo + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  double2 p = make_double2(0.0, 0.0), d = p;
  if (n < hi) {  // in flight with the partials
    p = w[(int64_t)r * ld + n];
    d = dinv[n];
  }
  double a = 0;
  for (int q = threadIdx.x; q < np; q += kRed) a += part[(int64_t)s * kNormParts + q];
  const double2 t = block_sum2(a, 0.0);
  if (threadIdx.x == 0) {
    snrm = t.x;
    if (blockIdx.x == 0) nrm[s] = t.x;
  }
  __syncthreads();
  if (n >= hi) return;
  const double sv = snrm;
  const double inv = sv > 0 ? 1.0 / sqrt(sv) : 0.0;
  const double2 v = make_double2(p.x * inv, p.y * inv);
  out[(int64_t)r * ld + n] = v;
  z[(int64_t)r * ld + n] = make_double2(v.x * d.x - v.y * d.y, v.x * d.y + v.y * d.x);
}

// Sum over a wave, the same in every lane: lane permutations within rows of 16
// (DPP: quad swaps, mirrors of 8 and 16 lanes), then the four rows' sums.
template <int CTRL>
__device__ __forceinline__ double add_dpp(double v) {
  return v + __hiloint2double(
                 __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true),
                 __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ double wave_sum(double v) {
  v = add_dpp<0xB1>(v);
  v = add_dpp<0x4E>(v);
  v = add_dpp<0x141>(v);
  v = add_dpp<0x140>(v);
  auto row = [&](int l) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                            __builtin_amdgcn_readlane(__double2loint(v), l));
  };
  return (row(0) + row(16)) + (row(32) + row(48));
}

// The whole Gram-Schmidt step of a small mesh (n <= 256 rows, at most 16 T
// vectors) in one launch: both passes, the norm, v_{j+1} and the next z, by one
// work-group of 16 waves per system. A wave holds vectors wave + 16 t in registers
// (lane + 64 k the rows), so the basis is read once and the dot products stay
// within the wave; the subtraction's sums over vectors go through LDS. The launches
// are what a step costs here (about 4 us each, whatever they do): 4 to 6 of them
// become one.
constexpr int kSmallRows = 256, kSmallWaves = 16;
constexpr int kSmallVectors = 64;  // (96 need 128 registers and spill: 21 us, the six launches 20)
template <int T>
__global__ void __launch_bounds__(64 * kSmallWaves)
    k_arnoldi_small(double2 *V, const double2 *w, double2 *z, const double2 *dinv, int64_t ld,
                    int64_t vstride, int64_t lo, int n, int j, int sys0, int S, double2 *H, int m,
                    double *nrm) {
  constexpr int NK = kSmallRows / 64;
  __shared__ double2 ws[kSmallRows], red[kSmallWaves][kSmallRows];
  const int r = blockIdx.x, s = sys0 + r, nv = j + 1;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double2 *Vr = V + (int64_t)r * ld + lo;
  const int64_t base = (int64_t)r * ld + lo;
  double2 v[T][NK], h[T];
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int i = wave + kSmallWaves * t;
    h[t] = make_double2(0.0, 0.0);
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      const int row = lane + 64 * k;
      v[t][k] = (i < nv && row < n) ? Vr[(int64_t)i * vstride + row] : make_double2(0.0, 0.0);
    }
  }
  if (tid < kSmallRows) ws[tid] = tid < n ? w[base + tid] : make_double2(0.0, 0.0);
  __syncthreads();
  for (int pass = 0; pass < 2; ++pass) {
    double2 y[NK], p[NK];
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      y[k] = ws[lane + 64 * k];
      p[k] = make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int t = 0; t < T; ++t) {
      double a = 0, b = 0;
#pragma unroll
      for (int k = 0; k < NK; ++k) {
        a += v[t][k].x * y[k].x + v[t][k].y * y[k].y;
        b += v[t][k].x * y[k].y - v[t][k].y * y[k].x;
      }
      const double2 c = make_double2(wave_sum(a), wave_sum(b));
      h[t].x += c.x;
      h[t].y += c.y;
#pragma unroll
      for (int k = 0; k < NK; ++k) {
        p[k].x += c.x * v[t][k].x - c.y * v[t][k].y;
        p[k].y += c.x * v[t][k].y + c.y * v[t][k].x;
      }
    }
#pragma unroll
    for (int k = 0; k < NK; ++k) red[wave][lane + 64 * k] = p[k];
    __syncthreads();
    if (tid < kSmallRows) {
      double2 a = ws[tid];
#pragma unroll
      for (int q = 0; q < kSmallWaves; ++q) {
        a.x -= red[q][tid].x;
        a.y -= red[q][tid].y;
      }
      ws[tid] = a;
    }
    __syncthreads();
  }
  if (lane == 0)
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int i = wave + kSmallWaves * t;
      if (i < nv) H[((int64_t)s * (m + 1) + i) * m + j] = h[t];
    }
  double a = 0;  // |w|^2, by every wave in the same order
#pragma unroll
  for (int k = 0; k < NK; ++k) {
    const double2 y = ws[lane + 64 * k];
    a += y.x * y.x + y.y * y.y;
  }
  a = wave_sum(a);
  if (tid == 0) nrm[s] = a;
  const double inv = a > 0 ? 1.0 / sqrt(a) : 0.0;
  if (tid < n) {
    const double2 u = make_double2(ws[tid].x * inv, ws[tid].y * inv), d = dinv[lo + tid];
    Vr[(int64_t)nv * vstride + tid] = u;
    z[base + tid] = make_double2(u.x * d.x - u.y * d.y, u.x * d.y + u.y * d.x);
  }
}

// z[r][row] = v[r][row] / d[row]
__global__ void k_precond(const double2 *v, double2 *z, const double2 *dinv, int64_t ld, int R) {
  const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= ld) return;
  const double2 d = dinv[n];
  for (int r = 0; r < R; ++r) {
    const double2 p = v[(int64_t)r * ld + n];
    z[(int64_t)r * ld + n] = make_double2(p.x * d.x - p.y * d.y, p.x * d.y + p.y * d.x);
  }
}

// x[r][row] += dinv[row] * sum_i y[i*S + s] V[i][r][row]
__global__ void k_update_x(const double2 *V, double2 *x, const double2 *dinv, int64_t ld,
                           int64_t vstride, int64_t lo, int64_t hi, int nv_max, const int *nv_sys,
                           int sys0, int S, const double2 *y) {
  const int r = blockIdx.y;
  const int64_t n = lo + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= hi) return;
  const int nv = min(nv_max, nv_sys[sys0 + r]);
  double ax = 0, ay = 0;
  for (int i = 0; i < nv; ++i) {
    const double2 c = y[(int64_t)i * S + sys0 + r];
    const double2 p = V[(int64_t)i * vstride + (int64_t)r * ld + n];
    ax += c.x * p.x - c.y * p.y;
    ay += c.x * p.y + c.y * p.x;
  }
  const double2 d = dinv[n];
  double2 xv = x[(int64_t)r * ld + n];
  xv.x += ax * d.x - ay * d.y;
  xv.y += ax * d.y + ay * d.x;
  x[(int64_t)r * ld + n] = xv;
}

// r = b - r_in (in place on r: r = b - Ax)
__global__ void k_residual(const double2 *b, double2 *ax, int64_t count) {
  const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= count) return;
  const double2 p = b[n], q = ax[n];
  ax[n] = make_double2(p.x - q.x, p.y - q.y);
}

__global__ void k_axpy_real(double2 *x, const double2 *d, int64_t count) {
  const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= count) return;
  x[n].x += d[n].x;
  x[n].y += d[n].y;
}

__global__ void k_inv_diag(const double2 *zd, double2 *dinv, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double2 d = zd[i];
  const double m = d.x * d.x + d.y * d.y;
  dinv[i] = make_double2(d.x / m, -d.y / m);
}

unsigned nblk(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }
unsigned red_blocks(int64_t n) {
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>(kNormParts, (n + kRed - 1) / kRed));
}

struct Ctx {
  Plan *pl;
  hipStream_t s;
  int R;  // right-hand sides per mesh
  int S;  // systems = nmesh * R
  int64_t ld;
  double2 *dinv;
  // meshes with a system still iterating: the Arnoldi steps skip the others'
  // products and Gram-Schmidt work (their systems are inactive, so nothing
  // reads what those steps would have written); empty = every mesh
  std::vector<char> on;
  bool mesh_on(int mi) const { return on.empty() || on[mi]; }
};

// y = A x with the operator of the given precision on c128 vectors
void apply(Ctx &c, aim_precision prec, const double2 *x, double2 *y) {
  matvec_plan(c.pl, prec == AIM_FP64 ? AIM_FP64 : AIM_MIXED_IO64, c.R, x, y, c.s, nullptr,
              c.on.empty() ? nullptr : &c.on);
}

// nrm[s] = |v_s|^2 for every system, on the device (partials, fixed order)
void norms_dev(Ctx &c, const double2 *v, double *part, double *nrm) {
  int mi = 0;
  for (auto &md : c.pl->mesh) {
    const unsigned nb = red_blocks(md.hp.n);
    hipLaunchKernelGGL(k_norm2_part, dim3(nb, c.R), dim3(kRed), 0, c.s, v, c.ld, md.offset,
                       md.offset + md.hp.n, mi * c.R, part);
    LAUNCHCHECK();
    hipLaunchKernelGGL(k_norm_reduce, dim3(c.R), dim3(64), 0, c.s, part, (int)nb, mi * c.R, nrm);
    LAUNCHCHECK();
    ++mi;
  }
}
// per-system squared norms of v (host result)
void norms(Ctx &c, const double2 *v, double *part, double *nrm, std::vector<double> &out) {
  norms_dev(c, v, part, nrm);
  out.resize(c.S);
  HIPCHECK(hipMemcpyAsync(out.data(), nrm, sizeof(double) * c.S, hipMemcpyDeviceToHost, c.s));
  HIPCHECK(hipStreamSynchronize(c.s));
}

// ---- device-side Givens rotations and back substitution (one thread per
// system). Complex values as double2.
__device__ inline double2 cmul_(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ inline double2 cconjmul_(double2 a, double2 b) {  // conj(a) * b
  return make_double2(a.x * b.x + a.y * b.y, a.x * b.y - a.y * b.x);
}

struct GmresDev {
  double2 *H;      // [S][(m+1) m], column j of system s at H[s][i*m + j]
  double2 *cs, *sn;  // [S][m]
  double2 *g;      // [S][m+1]
  int *active;     // [S]
  int *poll;       // [S] the same for the host (pinned), which polls it
  int *its;        // [S] iterations counted
  int *jend;       // [S] columns of the current cycle
  double *tol_abs;  // [S] stop when |g_{j+1}| <= tol_abs
};

// The new Hessenberg columns j0 .. j1-1 (at most kCheckEvery) of every active
// system, in H as the Gram-Schmidt passes left them, with nrm[j S + s] = |w|^2
// of each: one 64-lane work-group per system and lane c on column j0 + c. The
// rotations known before j0 are applied to all columns at once, then each column
// in turn forms its own, which the later ones apply; the system stops at the
// first column whose residual estimate |g_{j+1}| meets the tolerance, or breaks
// down. The chain of dependent rotations, about 60 ns each, bounds it: one column
// at a time it took 8.1 us per step of the 16-lambda plate's solve, after which
// the next product had to wait. LDS: (kCheckEvery (m + 2) + 2m) complex values.
constexpr int kCheckEvery = 8;  // iterations between convergence checks on the host
__device__ inline void rotate(double2 c, double2 s, double2 &hi, double2 &hn) {
  // [hi; hn] <- [conj(c) hi + conj(s) hn; -s hi + c hn]
  const double2 t0 = cconjmul_(c, hi), t1 = cconjmul_(s, hn);
  const double2 u0 = cmul_(s, hi), u1 = cmul_(c, hn);
  hi = make_double2(t0.x + t1.x, t0.y + t1.y);
  hn = make_double2(u1.x - u0.x, u1.y - u0.y);
}
__global__ void __launch_bounds__(64)
    k_givens(GmresDev d, const double *nrm, int j0, int j1, int m, int S) {
  const int s = blockIdx.x;
  if (!d.active[s]) return;  // uniform over the work-group
  extern __shared__ double2 gsh[];
  __shared__ int stop;
  const int nc = j1 - j0, L = m + 2;  // rows of a column in LDS (odd stride for even m)
  double2 *cl = gsh + kCheckEvery * L, *sl = cl + m;
  double2 *Hs = d.H + (int64_t)s * (m + 1) * m;
  double2 *cs = d.cs + (int64_t)s * m, *sn = d.sn + (int64_t)s * m;
  for (int c = 0; c < nc; ++c) {
    for (int i = threadIdx.x; i <= j0 + c; i += 64) gsh[c * L + i] = Hs[i * m + j0 + c];
    if (threadIdx.x == 0)
      gsh[c * L + j0 + c + 1] = make_double2(sqrt(nrm[(int64_t)(j0 + c) * S + s]), 0.0);
  }
  for (int i = threadIdx.x; i < j0; i += 64) {
    cl[i] = cs[i];
    sl[i] = sn[i];
  }
  if (threadIdx.x == 0) stop = 0;
  __syncthreads();
  const int c = threadIdx.x;
  double2 *col = gsh + c * L;
  if (c < nc)
    for (int i = 0; i < j0; ++i) rotate(cl[i], sl[i], col[i], col[i + 1]);
  int last = 0;  // columns completed
  for (int t = 0; t < nc; ++t) {
    const int j = j0 + t;
    if (c == t) {
      double2 *g = d.g + (int64_t)s * (m + 1);
      const double2 a = col[j];
      const double h1 = col[j + 1].x;  // |w|, untouched by the rotations before j
      const double den = sqrt(a.x * a.x + a.y * a.y + h1 * h1);
      const double2 rc = den == 0.0 ? make_double2(1.0, 0.0) : make_double2(a.x / den, a.y / den);
      const double2 rs = den == 0.0 ? make_double2(0.0, 0.0) : make_double2(h1 / den, 0.0);
      cs[j] = cl[j] = rc;
      sn[j] = sl[j] = rs;
      col[j] = make_double2(den, 0.0);
      col[j + 1] = make_double2(0.0, 0.0);
      const double2 gj = g[j];
      const double2 gn = cmul_(rs, gj);
      g[j + 1] = make_double2(-gn.x, -gn.y);
      g[j] = cconjmul_(rc, gj);
      d.its[s] += 1;
      d.jend[s] = j + 1;
      const double res = sqrt(gn.x * gn.x + gn.y * gn.y);
      if (res <= d.tol_abs[s] || den == 0.0) {
        d.active[s] = 0;
        d.poll[s] = 0;
        stop = 1;
      }
    }
    __syncthreads();
    last = t + 1;
    if (stop) break;
    if (c > t && c < nc) rotate(cl[j], sl[j], col[j], col[j + 1]);
  }
  __syncthreads();
  for (int q = 0; q < last; ++q)
    for (int i = threadIdx.x; i <= j0 + q + 1; i += 64) Hs[i * m + j0 + q] = gsh[q * L + i];
}

// y = H^-1 g on the jend x jend upper triangle (y stored [i][s] like h); one wave
// per system, lane l with rows l + 64 q. Columns are taken from the last: the lane
// that holds row i has y_i, which all lanes take off their rows above it, so the
// chain per column is a division and a lane broadcast, and eight columns are loaded
// ahead of it. (Row by row, with a sum over the lanes and a barrier each, 100
// columns took 72 us.)
constexpr int kBackRows = 4;  // 64 rows each: restart <= 200
__global__ void __launch_bounds__(64) k_backsub(GmresDev d, double2 *y, int m, int S) {
  const int s = blockIdx.x, lane = threadIdx.x;
  const int n = d.jend[s];
  const double2 *Hs = d.H + (int64_t)s * (m + 1) * m;
  const double2 *gs = d.g + (int64_t)s * (m + 1);
  double2 g[kBackRows], inv[kBackRows];  // right-hand side; conj(h_kk) / |h_kk|^2
#pragma unroll
  for (int q = 0; q < kBackRows; ++q) {
    const int k = lane + 64 * q;
    g[q] = inv[q] = make_double2(0.0, 0.0);
    if (k < n) {
      g[q] = gs[k];
      const double2 h = Hs[k * m + k];
      const double dd = h.x * h.x + h.y * h.y;
      if (dd != 0.0) inv[q] = make_double2(h.x / dd, -h.y / dd);  // else y_k = 0
    }
  }
#pragma unroll
  for (int b = kBackRows - 1; b >= 0; --b) {  // columns 64 b .. 64 b + 63
    for (int i1 = min(n, 64 * b + 64); i1 > 64 * b; i1 -= 8) {
      double2 h[8][kBackRows];
#pragma unroll
      for (int c = 0; c < 8; ++c)
#pragma unroll
        for (int q = 0; q <= b; ++q) {
          const int i = i1 - 1 - c, k = lane + 64 * q;
          h[c][q] = (i >= 64 * b && k < i) ? Hs[k * m + i] : make_double2(0.0, 0.0);
        }
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const int i = i1 - 1 - c;
        if (i < 64 * b) break;
        const double2 mine = cmul_(g[b], inv[b]);
        auto at = [&](double v) {
          return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), i & 63),
                                  __builtin_amdgcn_readlane(__double2loint(v), i & 63));
        };
        const double2 yi = make_double2(at(mine.x), at(mine.y));
        if (lane == 0) y[(int64_t)i * S + s] = yi;
#pragma unroll
        for (int q = 0; q <= b; ++q) {
          const double2 t = cmul_(h[c][q], yi);
          g[q].x -= t.x;
          g[q].y -= t.y;
        }
      }
    }
  }
}

struct Work {
  double2 *V = nullptr;  // (m+1) x R x ld
  double2 *z = nullptr, *w = nullptr;
  double2 *h1 = nullptr, *h2 = nullptr, *y = nullptr;
  double *nrm = nullptr;       // per system
  double *step_nrm = nullptr;  // [m][S]: |w|^2 of each Arnoldi step
  double2 *part = nullptr;  // dot-product partials [(m+1) S][np_stride]
  int64_t np_stride = 0;
  double *npart = nullptr;  // norm partials [S][kNormParts]
  GmresDev dev{};
};

}  // namespace

// Buffers, stream and captured graphs of the solver, kept in the plan for
// the shape (right-hand sides per mesh R, restart m) of the last solve.
struct SolverState {
  int R = 0, m = 0;
  Work wk;
  double2 *dinv = nullptr;  // Jacobi: 1 / diag(Z^MOM)
  std::vector<void *> bufs;
  int *poll = nullptr;  // pinned: the systems still active, written by k_givens
  hipStream_t stream = nullptr;
  hipEvent_t entry = nullptr;
  // (precision, j0, j1, meshes still iterating as bits)
  std::map<std::tuple<int, int, int, uint32_t>, hipGraphExec_t> graphs;
  uint64_t gen = 0;       // plan work-buffer generation the graphs were captured with
  bool warm[2] = {false, false};  // a direct step of this precision ran on these buffers
};

namespace {

void drop_graphs(SolverState &st) {
  for (auto &g : st.graphs) (void)hipGraphExecDestroy(g.second);
  st.graphs.clear();
}

SolverState &solver_state(Plan *pl, int R, int m) {
  if (!pl->solver) pl->solver = new SolverState();
  SolverState &st = *pl->solver;
  if (!st.stream) {
    HIPCHECK(hipStreamCreateWithFlags(&st.stream, hipStreamNonBlocking));
    HIPCHECK(hipEventCreateWithFlags(&st.entry, hipEventDisableTiming));
  }
  if (st.R == R && st.m == m) return st;
  HIPCHECK(hipStreamSynchronize(st.stream));
  drop_graphs(st);
  for (void *p : st.bufs) dev_free(pl, p);
  st.bufs.clear();
  if (st.poll) HIPCHECK(hipHostFree(st.poll));
  st.poll = nullptr;
  st.R = st.m = 0;
  st.warm[0] = st.warm[1] = false;
  auto alloc = [&](size_t bytes) {
    void *p = dev_alloc(pl, bytes);
    st.bufs.push_back(p);
    return p;
  };
  const int S = pl->nmesh * R;
  const int64_t ld = pl->n_total, cnt = (int64_t)R * ld;
  Work &wk = st.wk;
  wk.V = (double2 *)alloc(sizeof(double2) * (size_t)(m + 1) * cnt);
  wk.z = (double2 *)alloc(sizeof(double2) * cnt);
  wk.w = (double2 *)alloc(sizeof(double2) * cnt);
  wk.h1 = (double2 *)alloc(sizeof(double2) * (size_t)(m + 1) * S);
  wk.h2 = (double2 *)alloc(sizeof(double2) * (size_t)(m + 1) * S);
  wk.y = (double2 *)alloc(sizeof(double2) * (size_t)(m + 1) * S);
  wk.nrm = (double *)alloc(sizeof(double) * S);
  wk.step_nrm = (double *)alloc(sizeof(double) * (size_t)m * S);
  wk.np_stride = 2 * kInlineParts;
  for (auto &md : pl->mesh) wk.np_stride = std::max(wk.np_stride, basis_groups(md.hp.n, R));
  wk.part = (double2 *)alloc(sizeof(double2) * (size_t)(m + 1) * S * wk.np_stride);
  wk.npart = (double *)alloc(sizeof(double) * (size_t)S * kNormParts);
  wk.dev.H = (double2 *)alloc(sizeof(double2) * (size_t)S * (m + 1) * m);
  wk.dev.cs = (double2 *)alloc(sizeof(double2) * (size_t)S * m);
  wk.dev.sn = (double2 *)alloc(sizeof(double2) * (size_t)S * m);
  wk.dev.g = (double2 *)alloc(sizeof(double2) * (size_t)S * (m + 1));
  wk.dev.active = (int *)alloc(sizeof(int) * S);
  HIPCHECK(hipHostMalloc((void **)&st.poll, sizeof(int) * S,
                         hipHostMallocMapped | hipHostMallocCoherent));
  HIPCHECK(hipHostGetDevicePointer((void **)&wk.dev.poll, st.poll, 0));
  wk.dev.its = (int *)alloc(sizeof(int) * S);
  wk.dev.jend = (int *)alloc(sizeof(int) * S);
  wk.dev.tol_abs = (double *)alloc(sizeof(double) * S);
  st.dinv = (double2 *)alloc(sizeof(double2) * ld);
  for (auto &md : pl->mesh) {
    hipLaunchKernelGGL(k_inv_diag, dim3(nblk(md.hp.n, 256)), dim3(256), 0, st.stream, md.zdiag,
                       st.dinv + md.offset, md.hp.n);
    LAUNCHCHECK();
  }
  st.R = R;
  st.m = m;
  return st;
}

// One Arnoldi step j of every system: w = A D^-1 V[j], two classical
// Gram-Schmidt passes, V[j+1] = w / |w|, Hessenberg column j.
void arnoldi_step(Ctx &c, aim_precision prec, Work &wk, int j, int m) {
  const int S = c.S, R = c.R;
  const int64_t ld = c.ld, vstride = (int64_t)R * ld;
  if (j == 0) {  // later steps find z = dinv v_j left by the previous step
    hipLaunchKernelGGL(k_precond, dim3(nblk(ld, 256)), dim3(256), 0, c.s, wk.V + j * vstride, wk.z,
                       c.dinv, ld, R);
    LAUNCHCHECK();
  }
  apply(c, prec, wk.z, wk.w);
  int mi = 0;
  for (auto &md : c.pl->mesh) {
    if (!c.mesh_on(mi)) {
      ++mi;
      continue;
    }
    const int64_t n = md.hp.n;
    const int nb = (int)basis_groups(n, R), nv = j + 1, sys0 = mi * R;
    if (n <= kSmallRows && nv <= kSmallVectors) {
      auto small = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(R), dim3(64 * kSmallWaves), 0, c.s, wk.V, wk.w, wk.z, c.dinv,
                           ld, vstride, md.offset, (int)n, j, sys0, S, wk.dev.H, m,
                           wk.step_nrm + (int64_t)j * S);
        LAUNCHCHECK();
      };
      if (nv <= 16)
        small(k_arnoldi_small<1>);
      else if (nv <= 32)
        small(k_arnoldi_small<2>);
      else
        small(k_arnoldi_small<4>);
      ++mi;
      continue;
    }
    const int np = nb <= kInlineParts ? nb : 0;
    double2 *const part2 = np ? wk.part + kInlineParts : wk.part;
    auto pass = [&](auto kern, const double2 *h, const double2 *from, double2 *to, bool second) {
      hipLaunchKernelGGL(kern, dim3((unsigned)nb, R), dim3(256), 0, c.s, wk.V, wk.w, ld, vstride,
                         md.offset, n, nv, sys0, S, h, from, np, second, wk.dev.H, m, j,
                         wk.np_stride, to, wk.npart);
      LAUNCHCHECK();
    };
    auto reduce = [&](double2 *h, const double2 *add) {
      if (np) return;
      hipLaunchKernelGGL(k_part_reduce, dim3(nv, R), dim3(kRed), 0, c.s, wk.part, wk.np_stride, nb,
                         sys0, S, h, add, wk.dev.H, m, j);
      LAUNCHCHECK();
    };
    // slots: the smallest tile that holds the nv vectors
    auto passes = [&](auto slots_, auto rp_) {
      constexpr int SL = decltype(slots_)::value, RP = decltype(rp_)::value;
      pass(k_basis_pass<SL, RP, false, true, false>, nullptr, nullptr, wk.part, false);
      reduce(wk.h1, nullptr);
      pass(k_basis_pass<SL, RP, true, true, false>, wk.h1, wk.part, part2, false);
      reduce(wk.h2, wk.h1);
      pass(k_basis_pass<SL, RP, true, false, true>, wk.h2, part2, nullptr, true);
    };
    if (nv <= 16)
      passes(std::integral_constant<int, 1>{}, std::integral_constant<int, 4>{});
    else if (nv <= 32)
      passes(std::integral_constant<int, 2>{}, std::integral_constant<int, 4>{});
    else if (nv <= 64)
      passes(std::integral_constant<int, 4>{}, std::integral_constant<int, 4>{});
    else if (nv <= 112)
      passes(std::integral_constant<int, 7>{}, std::integral_constant<int, 4>{});
    else
      passes(std::integral_constant<int, 13>{}, std::integral_constant<int, 2>{});
    hipLaunchKernelGGL(k_normalize_next, dim3(nblk(n, 256), R), dim3(256), 0, c.s, wk.w,
                       wk.V + (j + 1) * vstride, wk.z, c.dinv, ld, md.offset, md.offset + n, sys0,
                       wk.npart, nb, wk.step_nrm + (int64_t)j * S);
    LAUNCHCHECK();
    ++mi;
  }
}

// Steps j0 .. j1-1 and their columns' rotations.
void arnoldi_segment(Ctx &c, aim_precision prec, Work &wk, int j0, int j1, int m) {
  for (int j = j0; j < j1; ++j) arnoldi_step(c, prec, wk, j, m);
  hipLaunchKernelGGL(k_givens, dim3(c.S), dim3(64),
                     sizeof(double2) * (kCheckEvery * ((size_t)m + 2) + 2 * (size_t)m), c.s, wk.dev,
                     wk.step_nrm, j0, j1, m, c.S);
  LAUNCHCHECK();
}

// Steps j0 .. j1-1 as one HIP graph: captured on first use, replayed after.
void run_segment_graph(Plan *pl, SolverState &st, Ctx &c, aim_precision prec, int j0, int j1) {
  if (pl->work_gen != st.gen) {  // a grid work buffer moved since the capture
    drop_graphs(st);
    st.gen = pl->work_gen;
  }
  uint32_t bits = 0;
  for (int i = 0; i < c.pl->nmesh; ++i)
    if (c.mesh_on(i)) bits |= 1u << i;
  const auto key = std::make_tuple((int)prec, j0, j1, bits);
  auto it = st.graphs.find(key);
  if (it == st.graphs.end()) {
    HIPCHECK(hipStreamBeginCapture(c.s, hipStreamCaptureModeThreadLocal));
    hipGraph_t g = nullptr;
    try {
      arnoldi_segment(c, prec, st.wk, j0, j1, st.m);
    } catch (...) {
      (void)hipStreamEndCapture(c.s, &g);
      if (g) (void)hipGraphDestroy(g);
      throw;
    }
    HIPCHECK(hipStreamEndCapture(c.s, &g));
    hipGraphExec_t ex = nullptr;
    const hipError_t e = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    HIPCHECK(e);
    it = st.graphs.emplace(key, ex).first;
  }
  HIPCHECK(hipGraphLaunch(it->second, c.s));
}

// Solve A d = rhs (d starts at 0) for every system to a relative residual
// tol_s (estimated by the Arnoldi recurrence), restarted every m steps; a
// low-precision run also stops a system whose true residual has reached the
// operator's rounding floor (see the restart check). The
// Arnoldi step, the rotations and the residual estimate stay on the device;
// the host reads the active flags every kCheckEvery iterations. Returns the
// iterations used (lock-step count); `its` per system, `nprod` products.
int gmres_run(Ctx &c, SolverState &st, aim_precision prec, bool graphs, const double2 *rhs,
              double2 *d, const std::vector<double> &rhs_norm2, const std::vector<double> &tol_s,
              int max_iter, std::vector<int> &its, int &nprod) {
  Work &wk = st.wk;
  const int m = st.m;
  const int S = c.S, R = c.R;
  const int64_t ld = c.ld, vstride = (int64_t)R * ld, cnt = vstride;
  const int pi = prec == AIM_FP64 ? 0 : 1;
  HIPCHECK(hipMemsetAsync(d, 0, sizeof(double2) * cnt, c.s));
  std::vector<char> done(S, 0);
  for (int s = 0; s < S; ++s)
    if (rhs_norm2[s] == 0.0) done[s] = 1;
  int total = 0;
  std::vector<double> r2, prev(S, 0.0);
  bool first_cycle = true;
  std::vector<int> act(S), itd(S), jendh(S, m);
  HIPCHECK(hipMemcpyAsync(wk.dev.its, its.data(), sizeof(int) * S, hipMemcpyHostToDevice, c.s));
  // meshes with a system for which flag[s] is set
  auto meshes_of = [&](const auto &flag) {
    std::vector<char> on(c.pl->nmesh, 0);
    for (int s = 0; s < S; ++s)
      if (flag[s]) on[s / R] = 1;
    return on;
  };
  std::vector<char> notdone(S);
  while (true) {
    for (int s = 0; s < S; ++s) notdone[s] = !done[s];
    c.on = meshes_of(notdone);
    // residual of the current iterate: r = rhs - A d (rhs itself on the first cycle)
    if (first_cycle) {
      HIPCHECK(hipMemcpyAsync(wk.w, rhs, sizeof(double2) * cnt, hipMemcpyDeviceToDevice, c.s));
    } else {
      apply(c, prec, d, wk.w);
      ++nprod;
      hipLaunchKernelGGL(k_residual, dim3(nblk(cnt, 256)), dim3(256), 0, c.s, rhs, wk.w, cnt);
      LAUNCHCHECK();
    }
    const bool restarted = !first_cycle;
    first_cycle = false;
    norms(c, wk.w, wk.npart, wk.nrm, r2);
    bool all = true;
    for (int s = 0; s < S; ++s) {
      if (!done[s] && r2[s] <= tol_s[s] * tol_s[s] * rhs_norm2[s]) done[s] = 1;
      // Low-precision operator at its rounding floor: the last cycle's
      // estimate met the tolerance before the restart length, yet the true
      // residual of this operator did not even halve. Further cycles only
      // chase rounding noise; the FP64 refinement around this run continues.
      if (!done[s] && restarted && prec != AIM_FP64 && jendh[s] < m && r2[s] > 0.25 * prev[s])
        done[s] = 1;
      prev[s] = r2[s];
      all &= (bool)done[s];
    }
    if (all || total >= max_iter) break;
    // V[0] = r / |r|; cycle state on the device
    {
      int mi = 0;
      for (auto &md : c.pl->mesh) {
        hipLaunchKernelGGL(k_normalize, dim3(nblk(md.hp.n, 256), R), dim3(256), 0, c.s, wk.w, wk.V,
                           ld, md.offset, md.offset + md.hp.n, mi * R, wk.nrm);
        LAUNCHCHECK();
        ++mi;
      }
    }
    std::vector<double2> g0((size_t)S * (m + 1), make_double2(0, 0));
    std::vector<double> tabs(S);
    for (int s = 0; s < S; ++s) {
      st.poll[s] = act[s] = !done[s];  // (the stream is synchronised: no kernel writes it now)
      g0[(size_t)s * (m + 1)] = make_double2(std::sqrt(r2[s]), 0.0);
      tabs[s] = tol_s[s] * std::sqrt(rhs_norm2[s]);
    }
    std::vector<int> zero(S, 0);
    HIPCHECK(hipMemcpyAsync(wk.dev.g, g0.data(), sizeof(double2) * g0.size(), hipMemcpyHostToDevice, c.s));
    HIPCHECK(hipMemcpyAsync(wk.dev.active, act.data(), sizeof(int) * S, hipMemcpyHostToDevice, c.s));
    HIPCHECK(hipMemcpyAsync(wk.dev.tol_abs, tabs.data(), sizeof(double) * S, hipMemcpyHostToDevice, c.s));
    HIPCHECK(hipMemcpyAsync(wk.dev.jend, zero.data(), sizeof(int) * S, hipMemcpyHostToDevice, c.s));
    // segments of kCheckEvery steps between polls of the active flags; a full
    // segment (or the cycle's last) is a graph once this precision has run
    // directly on the current buffers (so no buffer is allocated in a capture)
    c.on = meshes_of(act);
    for (int j = 0; j < m && total < max_iter;) {
      const int j1 = std::min({j + kCheckEvery, m, j + (max_iter - total)});
      const bool whole = (j1 - j == kCheckEvery) || j1 == m;
      if (graphs && whole && st.warm[pi]) {
        run_segment_graph(c.pl, st, c, prec, j, j1);
      } else {
        arnoldi_segment(c, prec, wk, j, j1, m);
        st.warm[pi] = true;
      }
      nprod += j1 - j;
      total += j1 - j;
      j = j1;
      HIPCHECK(hipStreamSynchronize(c.s));
      bool any = false;
      for (int s = 0; s < S; ++s) any |= (bool)(act[s] = st.poll[s]);
      if (!any) break;
      c.on = meshes_of(act);
    }
    // d += D^-1 V y, y = H^-1 g per system (systems done before the cycle: jend = 0)
    hipLaunchKernelGGL(k_backsub, dim3(S), dim3(64), 0, c.s, wk.dev, wk.y, m, S);
    LAUNCHCHECK();
    {
      int mi = 0;
      for (auto &md : c.pl->mesh) {
        hipLaunchKernelGGL(k_update_x, dim3(nblk(md.hp.n, 256), R), dim3(256), 0, c.s, wk.V, d,
                           c.dinv, ld, vstride, md.offset, md.offset + md.hp.n, m, wk.dev.jend,
                           mi * R, S, wk.y);
        LAUNCHCHECK();
        ++mi;
      }
    }
    HIPCHECK(hipMemcpyAsync(jendh.data(), wk.dev.jend, sizeof(int) * S, hipMemcpyDeviceToHost, c.s));
    HIPCHECK(hipStreamSynchronize(c.s));
  }
  HIPCHECK(hipMemcpyAsync(itd.data(), wk.dev.its, sizeof(int) * S, hipMemcpyDeviceToHost, c.s));
  HIPCHECK(hipStreamSynchronize(c.s));
  for (int s = 0; s < S; ++s) its[s] = itd[s];
  c.on.clear();  // later products (the outer residual) cover every mesh
  return total;
}

}  // namespace

void solver_release(Plan *pl) {
  if (!pl || !pl->solver) return;
  SolverState &st = *pl->solver;
  if (st.stream) (void)hipStreamSynchronize(st.stream);
  drop_graphs(st);
  for (void *p : st.bufs) dev_free(pl, p);
  if (st.poll) (void)hipHostFree(st.poll);
  if (st.entry) (void)hipEventDestroy(st.entry);
  if (st.stream) (void)hipStreamDestroy(st.stream);
  delete pl->solver;
  pl->solver = nullptr;
}

aim_status gmres_solve(Plan *pl, aim_precision prec, int R, const aim_planewave *waves,
                       const aim_solve_opts &o, double2 *x, aim_solve_stats *st, hipStream_t caller) {
  auto t0 = std::chrono::steady_clock::now();
  const int S = pl->nmesh * R;
  const int m = o.restart;
  const int64_t ld = pl->n_total;
  const int64_t cnt = (int64_t)R * ld;
  const bool graphs = !(o.flags & AIM_SOLVE_NO_GRAPH);
  SolverState &ss = solver_state(pl, R, m);
  // the solve runs on the solver's own stream (capturable), after the
  // caller's stream has reached this call; it ends synchronised
  const hipStream_t s = ss.stream;
  HIPCHECK(hipEventRecord(ss.entry, caller));
  HIPCHECK(hipStreamWaitEvent(s, ss.entry, 0));
  Work &wk = ss.wk;
  std::vector<void *> tmp;
  auto alloc = [&](size_t bytes) {
    void *p = dev_alloc(pl, bytes);
    tmp.push_back(p);
    return p;
  };
  aim_status result = AIM_OK;
  try {
    double2 *b = (double2 *)alloc(sizeof(double2) * cnt);
    double2 *r = (double2 *)alloc(sizeof(double2) * cnt);
    double2 *dd = (double2 *)alloc(sizeof(double2) * cnt);
    for (auto &md : pl->mesh) excitation_mesh(pl, md, R, waves, b + md.offset, ld, s);
    Ctx c{pl, s, R, S, ld, ss.dinv};
    std::vector<double> b2, r2;
    norms(c, b, wk.npart, wk.nrm, b2);
    if (!o.warm_start) HIPCHECK(hipMemsetAsync(x, 0, sizeof(double2) * cnt, s));
    std::vector<int> its(S, 0);
    int n_low = 0, n64 = 0, total = 0;
    const double tol = o.tol;
    // residual r = b - A64 x
    auto residual = [&]() {
      apply(c, AIM_FP64, x, r);
      ++n64;
      hipLaunchKernelGGL(k_residual, dim3(nblk(cnt, 256)), dim3(256), 0, s, b, r, cnt);
      LAUNCHCHECK();
      norms(c, r, wk.npart, wk.nrm, r2);
    };
    if (prec == AIM_FP64) {
      if (o.warm_start) {
        residual();
      } else {
        HIPCHECK(hipMemcpyAsync(r, b, sizeof(double2) * cnt, hipMemcpyDeviceToDevice, s));
        r2 = b2;
      }
      std::vector<double> tol_s(S);
      for (int i = 0; i < S; ++i) tol_s[i] = r2[i] > 0 ? tol * std::sqrt(b2[i] / r2[i]) : 1.0;
      total += gmres_run(c, ss, AIM_FP64, graphs, r, dd, r2, tol_s, o.max_iter, its, n64);
      hipLaunchKernelGGL(k_axpy_real, dim3(nblk(cnt, 256)), dim3(256), 0, s, x, dd, cnt);
      LAUNCHCHECK();
      residual();
    } else {
      residual();
      for (int outer = 0; outer < 20; ++outer) {
        bool all = true;
        for (int i = 0; i < S; ++i) all &= (b2[i] == 0 || r2[i] <= tol * tol * b2[i]);
        if (all || total >= o.max_iter) break;
        std::vector<double> tol_s(S);
        for (int i = 0; i < S; ++i) {
          // reach the outer tolerance with margin, but not below what c64 arithmetic resolves
          double want = r2[i] > 0 ? 0.5 * tol * std::sqrt(b2[i] / r2[i]) : 1.0;
          tol_s[i] = std::max(want, 2e-6);
        }
        total += gmres_run(c, ss, AIM_MIXED, graphs, r, dd, r2, tol_s, o.max_iter - total, its,
                           n_low);
        hipLaunchKernelGGL(k_axpy_real, dim3(nblk(cnt, 256)), dim3(256), 0, s, x, dd, cnt);
        LAUNCHCHECK();
        residual();
      }
    }
    double secs = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    bool all_ok = true;
    for (int i = 0; i < S; ++i) {
      double rel = b2[i] > 0 ? std::sqrt(r2[i] / b2[i]) : 0.0;
      if (!(rel <= tol)) all_ok = false;
    }
    if (st) {  // one entry per system (mesh, wave), mesh-major
      for (int sidx = 0; sidx < S; ++sidx) {
        aim_solve_stats q{};
        const double rel = b2[sidx] > 0 ? std::sqrt(r2[sidx] / b2[sidx]) : 0.0;
        q.iterations = its[sidx];
        q.residual = rel;
        q.converged = rel <= tol ? 1 : 0;
        q.matvec_low = n_low;
        q.matvec_fp64 = n64;
        q.seconds = secs;
        st[sidx] = q;
      }
    }
    result = all_ok ? AIM_OK : AIM_ERR_NOCONV;
  } catch (...) {
    (void)hipStreamSynchronize(s);
    for (void *p : tmp) dev_free(pl, p);
    throw;
  }
  HIPCHECK(hipStreamSynchronize(s));
  for (void *p : tmp) dev_free(pl, p);
  return result;
}

}  // namespace aim
