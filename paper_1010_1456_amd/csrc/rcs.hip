// Bistatic radar cross section sigma_theta_theta (FP64).
//
// The paper measures accuracy through the VV bistatic RCS over the sphere of
// directions (Section 2.2, eq. 1). With J = sum_n I_n f_n, the radiation
// vector is N(r_hat) = int J exp(+j k r_hat . r') dS' and, for a unit incident
// field, sigma_tt = (k eta)^2 / (4 pi) |theta_hat . N|^2.
//
// On a triangle with centroid c the current is J = g (r - c) + c0 with the
// complex scalar g = sum_i s_i l_i I_i / (2A) over its basis functions and
// c0 = sum_i s_i l_i I_i (c - v_i) / (2A), and the 7 points of the rule lie at
// c + gamma (3 (v_i - c)) with gamma = 1/3 - a, 1/3 - b (and c itself). So
//   theta_hat . N_T = A e^{j k r_hat . c} [(theta_hat . c0) S + g T / k],
//   S = w_c + sum_{gamma, i} w e^{j gamma p_i},
//   T = sum_{gamma, i} w gamma q_i e^{j gamma p_i},
// p_i = 3 k r_hat . (v_i - c), q_i = 3 k theta_hat . (v_i - c): S, T and the
// phase of c are shared by all right-hand sides, each of which then costs 14
// multiply-adds per triangle and direction.
#include <algorithm>
#include <cmath>
#include <mutex>

#include "aim_internal.h"
#include "fft_core.h"
#include "geom_device.h"
#include "turns.h"

namespace aim {
using namespace geo;

namespace {

// Partial sums of the allocation-free RCS: one array per GPU for the whole
// process, kRcsScratchElems double2 (16 MiB). Host code never passes this
// name to a kernel (on the host it is only a stand-in): it uses the device
// address looked up by rcs_scratch_init.
static __device__ __align__(256) double2 scratch[kRcsScratchElems];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

// Since p_1 + p_2 + p_3 = 0, S and T are functions of a = (p_1^2 + p_2^2 +
// p_3^2) / 2 and b = p_1 p_2 p_3 alone (Newton's identities): the power sums are
// P_n = sum_{2i+3j=n} n (i+j-1)!/(i! j!) a^i b^j (Waring's formula), and
//   S = sum_n (j^n / n!) kappa_n P_n,  kappa_n = sum_gamma w gamma^n.
// T is S's derivative along the change of p by q, times -j. The series through
// n = 14 leaves less than 1e-16 of S and 1e-15 of T's terms while
// |gamma_a p_i| <= 1/2 (kSeriesMax; a lambda/9 mesh has 0.3 to 0.4): 45
// multiply-adds in place of six sines and cosines.
constexpr int kSeriesDegree = 14;
constexpr double kSeriesMax = 0.5;
constexpr double kGa = 1.0 / 3.0 - kQa, kGb = 1.0 / 3.0 - kQb;
constexpr double kappa(int n) {
  double x = kWa, y = kWb;
  for (int i = 0; i < n; ++i) {
    x *= kGa;
    y *= kGb;
  }
  return x + y;
}
// coefficient of a^i b^j in the real (j even) or imaginary (j odd) part of S
constexpr double series_coef(int i, int j) {
  const int n = 2 * i + 3 * j;
  if (n == 0) return 1.0;
  double c = kappa(n) * n / (i + j);  // kappa n (i+j-1)!/(i! j!) / n!
  for (int m = 2; m <= i + j; ++m) c *= m;
  for (int m = 2; m <= i; ++m) c /= m;
  for (int m = 2; m <= j; ++m) c /= m;
  for (int m = 2; m <= n; ++m) c /= m;
  return (n / 2) % 2 ? -c : c;
}
// The constants of both series, read with scalar loads where they are used: as
// literals the compiler moves them all out of the triangle loop into vector
// registers, and spills (54 of 128 for one right-hand side).
struct RcsConst {
  TurnsConst turns;
  double a[5][8];  // series_coef(i, j) as a[j][i]
  constexpr RcsConst() : turns{}, a{} {
    for (int j = 0; j < 5; ++j)
      for (int i = 0; i < 8; ++i) a[j][i] = series_coef(i, j);
  }
};
__constant__ constexpr RcsConst kRcsConst{};
using RcsConstPtr = const __attribute__((address_space(4))) RcsConst *;  // scalar loads

// A_j(a) = sum_i coef(i, j) a^i (DER 0) or its derivative (DER 1)
template <int J, int DER>
__device__ __forceinline__ double series_poly(RcsConstPtr k, double a) {
  constexpr int imax = (kSeriesDegree - 3 * J) / 2;
  double v = (DER ? imax : 1) * k->a[J][imax];
  fftc::static_for<imax - DER>([&](auto i_) AIM_AI {
    constexpr int i = imax - 1 - decltype(i_)::value;
    v = fma(v, a, (DER ? i : 1) * k->a[J][i]);
  });
  return v;
}

// A triangle as the part kernel reads it from LDS (doubles): centroid in
// wavelengths (0-2), 3 k (v_1 - c) (3-5), 3 k (v_2 - c) (6-8), 1 if its
// |gamma_a p| can exceed kSeriesMax (9); then per right-hand side A c0 (6,
// interleaved) and A g / k (2).
constexpr int kTriGeom = 10, kTriRhs = 8;

struct FarMesh {
  const int32_t *tris;
  const double *verts;
  const int32_t *tri_basis;
  const double *len;
  int64_t nt;
  double k;
  // k / 6 pi and what its rounding leaves: a relative error there turns the phases of
  // all triangles together
  double third_hi, third_lo;
};

__device__ __forceinline__ void load_tri(const FarMesh &fm, int64_t tri, D3 *T) {
  for (int c = 0; c < 3; ++c) T[c] = vtx(fm.verts, fm.tris[3 * tri + c]);
}
// (k / 6 pi) (a + b + c), rounded once: rounding the sum would give all triangles of a
// grid line the same error
__device__ __forceinline__ double centroid_turns(const FarMesh &fm, double a, double b, double c) {
  const double s = a + b, u = s - a, e = (a - (s - u)) + (b - u);
  const double t = s + c, v = t - s, f = (s - (t - v)) + (c - v);
  return fma(fm.third_hi, t, fma(fm.third_hi, e + f, fm.third_lo * t));
}
__device__ __forceinline__ void stage_geometry(const FarMesh &fm, int64_t tri, double *o) {
  D3 c = d3(0, 0, 0), p1 = c, p2 = c;
  double coarse = 0.0;
  if (tri < fm.nt) {
    D3 T[3];
    load_tri(fm, tri, T);
    c = d3(centroid_turns(fm, T[0].x, T[1].x, T[2].x), centroid_turns(fm, T[0].y, T[1].y, T[2].y),
           centroid_turns(fm, T[0].z, T[1].z, T[2].z));
    p1 = fm.k * ((T[1] - T[0]) + (T[1] - T[2]));
    p2 = fm.k * ((T[2] - T[0]) + (T[2] - T[1]));
    const double m = fmax(fmax(dot(p1, p1), dot(p2, p2)), dot(p1 + p2, p1 + p2));
    constexpr double lim = kSeriesMax / kGa;
    coarse = m > lim * lim ? 1.0 : 0.0;
  }
  o[0] = c.x, o[1] = c.y, o[2] = c.z;
  o[3] = p1.x, o[4] = p1.y, o[5] = p1.z;
  o[6] = p2.x, o[7] = p2.y, o[8] = p2.z;
  o[9] = coarse;
}
__device__ __forceinline__ void stage_current(const FarMesh &fm, int64_t tri, const double2 *xr,
                                              double *o) {
  double cr[3] = {0, 0, 0}, ci[3] = {0, 0, 0}, gr = 0, gi = 0;
  if (tri < fm.nt) {
    D3 T[3];
    load_tri(fm, tri, T);
    // 3 (c - v_i) from edges, not from c: its rounding is that of the coordinates
    const D3 e1 = T[1] - T[0], e2 = T[2] - T[0];
    const D3 d3c[3] = {e1 + e2, e2 - 2.0 * e1, e1 - 2.0 * e2};
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const int code = fm.tri_basis[3 * tri + i];
      if (code < 0) continue;
      const int64_t n = code >> 1;
      // A f_n = (s l / 2) (r - v_i) on this triangle, v_i the free vertex
      const double f = ((code & 1) ? -0.5 : 0.5) * fm.len[n];
      const double2 I = xr[n];
      const D3 d = d3c[i];
      const double fr = f * I.x, fi = f * I.y;
      cr[0] += d.x * fr, ci[0] += d.x * fi;
      cr[1] += d.y * fr, ci[1] += d.y * fi;
      cr[2] += d.z * fr, ci[2] += d.z * fi;
      gr += fr, gi += fi;
    }
  }
  for (int q = 0; q < 3; ++q) o[2 * q] = cr[q] * (1.0 / 3.0), o[2 * q + 1] = ci[q] * (1.0 / 3.0);
  o[6] = gr / fm.k, o[7] = gi / fm.k;
}

// part[(r ndir + d) nchunk + blockIdx.y] = theta_hat . N of the chunk's
// triangles, r = RB blockIdx.z + r0 .. + RB - 1 (those below nrhs).
//
// Bound by FP64 issue: 114 + 14 RB multiply-adds per triangle and direction. A
// lane owns kDirs directions (their unit vectors and sums stay in registers), a
// work-group 64 kDirs directions; its waves take the triangles of a batch in
// turn, read from LDS at a wave-uniform address, and add their sums through LDS
// at the end. Two directions per lane halve those broadcast reads, which cost
// as much as four multiply-adds per double, and share the series' constants.
// Summing the 7 points of every triangle separately, with the library sincos of
// each and once more for every right-hand side, took 9.6 ms per call on the
// 4-lambda sphere (36 980 triangles, 16 380 directions, one current) and 58 ms
// on the 8-lambda plate (10 368 triangles, 16 currents); this takes 3.0 and 2.6
// ms (2.2 and 1.6 ms is the multiply-adds' time at the FP64 vector rate).
constexpr int kRcsWaves = 4;
constexpr int kDirs = 2;
constexpr int kDirGroup = 64 * kDirs;
template <int RB>
constexpr int rcs_batch() {  // triangles in LDS at a time
  return RB <= 4 ? 64 : 32;
}
template <int RB>
__global__ void __launch_bounds__(64 * kRcsWaves, RB <= 4 ? 4 : (RB <= 8 ? 3 : 2))
    k_rcs_part(FarMesh fm, const double2 *__restrict__ x, int64_t ldx, int r0, int nrhs,
               int64_t per_chunk, const double *__restrict__ theta, int ntheta,
               const double *__restrict__ phi, int nphi, int nchunk, double2 *__restrict__ part) {
  r0 += RB * blockIdx.z;
  constexpr int TB = rcs_batch<RB>(), REC = kTriGeom + kTriRhs * RB;
  constexpr int kRed = 2 * kRcsWaves * kDirGroup;  // the final sums' exchange
  __shared__ __align__(16) double lds[TB * REC > kRed ? TB * REC : kRed];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t ndir = (int64_t)ntheta * nphi;
  const int64_t d0 = (int64_t)blockIdx.x * kDirGroup + lane;
  D3 rh[kDirs], th[kDirs];
  double ar[kDirs][RB], ai[kDirs][RB];
#pragma unroll
  for (int q = 0; q < kDirs; ++q) {
    const int64_t d = d0 + 64 * q < ndir ? d0 + 64 * q : ndir - 1;
    double st, ct, sp, cp;
    sincos(theta[d / nphi], &st, &ct);
    sincos(phi[d % nphi], &sp, &cp);
    rh[q] = d3(st * cp, st * sp, ct);
    th[q] = d3(ct * cp, ct * sp, -st);
#pragma unroll
    for (int r = 0; r < RB; ++r) ar[q][r] = ai[q][r] = 0.0;
  }
  const int64_t t0 = (int64_t)blockIdx.y * per_chunk;
  const int64_t t1 = min(t0 + per_chunk, fm.nt);
  for (int64_t b0 = t0; b0 < t1; b0 += TB) {
    __syncthreads();
    for (int i = threadIdx.x; i < TB * (RB + 1); i += 64 * kRcsWaves) {
      const int tl = i % TB, what = i / TB;
      const int64_t tri = b0 + tl < t1 ? b0 + tl : fm.nt;  // past the chunk: zeros
      if (what == 0)
        stage_geometry(fm, tri, &lds[tl * REC]);
      else
        stage_current(fm, r0 + what - 1 < nrhs ? tri : fm.nt, x + (int64_t)(r0 + what - 1) * ldx,
                      &lds[tl * REC + kTriGeom + kTriRhs * (what - 1)]);
    }
    __syncthreads();
    const int tend = (int)min((int64_t)TB, t1 - b0);
    for (int tl = wave; tl < tend; tl += kRcsWaves) {
      const double *rec = &lds[tl * REC];
      RcsConstPtr kc = (RcsConstPtr)&kRcsConst;
      asm volatile("" : "+s"(kc));  // a new value each time: no load is moved out of the loop
      const D3 c = d3(rec[0], rec[1], rec[2]);
      const D3 v1 = d3(rec[3], rec[4], rec[5]), v2 = d3(rec[6], rec[7], rec[8]);
      const bool coarse = __builtin_amdgcn_readfirstlane(__double2hiint(rec[9])) != 0;
      double sr[kDirs], si[kDirs], tr[kDirs], ti[kDirs];  // e^{j k r_hat . c} (S, T)
#pragma unroll
      for (int q = 0; q < kDirs; ++q) {
        const double p1 = dot(rh[q], v1), p2 = dot(rh[q], v2);
        const double q1 = dot(th[q], v1), q2 = dot(th[q], v2);
        double S_r, S_i, T_r, T_i;
        if (!coarse) {
          const double s = p1 + p2, m = p1 * p2, u = q1 + q2;
          const double dm = p1 * q2 + q1 * p2;
          const double a = s * s - m, b = -m * s;
          const double da = 2.0 * s * u - dm, db = -(dm * s + m * u);
          const double b2 = b * b;
          const double A0 = series_poly<0, 0>(kc, a), A1 = series_poly<1, 0>(kc, a);
          const double A2 = series_poly<2, 0>(kc, a), A3 = series_poly<3, 0>(kc, a);
          const double A4 = series_poly<4, 0>(kc, a);
          S_r = A0 + b2 * (A2 + b2 * A4);
          S_i = b * (A1 + b2 * A3);
          const double fa_r = series_poly<0, 1>(kc, a) +
                              b2 * (series_poly<2, 1>(kc, a) + b2 * series_poly<4, 1>(kc, a));
          const double fa_i = b * (series_poly<1, 1>(kc, a) + b2 * series_poly<3, 1>(kc, a));
          const double fb_r = b * (2.0 * A2 + b2 * (4.0 * A4));
          const double fb_i = A1 + b2 * (3.0 * A3);
          T_r = fa_i * da + fb_i * db;  // -j (f_a da + f_b db)
          T_i = -(fa_r * da + fb_r * db);
        } else {
          S_r = kWc, S_i = 0.0, T_r = 0.0, T_i = 0.0;
#pragma unroll 1
          for (int i = 0; i < 6; ++i) {
            const double g = i < 3 ? kGa : kGb, w = i < 3 ? kWa : kWb;
            const int v = i % 3;
            const double p = v == 0 ? p1 : (v == 1 ? p2 : -(p1 + p2));
            const double t = v == 0 ? q1 : (v == 1 ? q2 : -(q1 + q2));
            double sn, cs;
            sincos_turns(&kc->turns, p * (g * (0.5 / 3.14159265358979323846)), sn, cs);
            S_r += w * cs, S_i += w * sn;
            T_r += (w * g * t) * cs, T_i += (w * g * t) * sn;
          }
        }
        double sn, cs;
        sincos_turns(&kc->turns, dot(rh[q], c), sn, cs);
        sr[q] = cs * S_r - sn * S_i, si[q] = cs * S_i + sn * S_r;
        tr[q] = cs * T_r - sn * T_i, ti[q] = cs * T_i + sn * T_r;
      }
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        const double *o = rec + kTriGeom + kTriRhs * r;
        const double xr = o[0], xi = o[1], yr = o[2], yi = o[3], zr = o[4], zi = o[5];
        const double gr = o[6], gi = o[7];
#pragma unroll
        for (int q = 0; q < kDirs; ++q) {
          const double cr = th[q].x * xr + th[q].y * yr + th[q].z * zr;
          const double ci = th[q].x * xi + th[q].y * yi + th[q].z * zi;
          ar[q][r] += cr * sr[q] - ci * si[q] + gr * tr[q] - gi * ti[q];
          ai[q][r] += cr * si[q] + ci * sr[q] + gr * ti[q] + gi * tr[q];
        }
      }
    }
  }
  // the waves' sums, in wave order, one right-hand side at a time
  double2 *red = reinterpret_cast<double2 *>(lds);  // [kRcsWaves][kDirGroup]
#pragma unroll
  for (int r = 0; r < RB; ++r) {
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kDirs; ++q)
      red[wave * kDirGroup + 64 * q + lane] = make_double2(ar[q][r], ai[q][r]);
    __syncthreads();
    const int64_t d = (int64_t)blockIdx.x * kDirGroup + threadIdx.x;
    if (threadIdx.x < kDirGroup && d < ndir && r0 + r < nrhs) {
      double2 a = red[threadIdx.x];
      for (int w = 1; w < kRcsWaves; ++w) {
        a.x += red[w * kDirGroup + threadIdx.x].x;
        a.y += red[w * kDirGroup + threadIdx.x].y;
      }
      part[((int64_t)(r0 + r) * ndir + d) * nchunk + blockIdx.y] = a;
    }
  }
}

// sigma[rr ndir + d] = scale |sum over chunks of part|^2: `lanes` (a power of two up to
// 64) lanes per slot take every lanes-th chunk and add their sums by exchanges
__global__ void __launch_bounds__(256)
    k_rcs_reduce(const double2 *part, int nchunk, int64_t count, int lanes, double scale,
                 double *sigma) {
  const int lane = threadIdx.x & (lanes - 1);
  const int64_t step = (int64_t)gridDim.x * (256 / lanes);
  for (int64_t t = (int64_t)blockIdx.x * (256 / lanes) + threadIdx.x / lanes; t < count; t += step) {
    double a = 0, b = 0;
    for (int c = lane; c < nchunk; c += lanes) {
      const double2 v = part[t * nchunk + c];
      a += v.x;
      b += v.y;
    }
    for (int off = 1; off < lanes; off <<= 1) {
      a += __shfl_xor(a, off, 64);
      b += __shfl_xor(b, off, 64);
    }
    if (lane == 0) sigma[t] = scale * (a * a + b * b);
  }
}

}  // namespace

void rcs_prepare_mesh(Plan *pl, MeshDev &md, hipStream_t s) {
  const HostPlan &h = md.hp;
  std::vector<int32_t> tb(3 * h.nt, -1);
  for (int64_t n = 0; n < h.n; ++n) {
    for (int side = 0; side < 2; ++side) {
      const int64_t t = side == 0 ? h.tp[n] : h.tm[n];
      const int32_t fv = side == 0 ? h.vp[n] : h.vm[n];
      for (int i = 0; i < 3; ++i)
        if (h.tris[3 * t + i] == fv) tb[3 * t + i] = (int32_t)((n << 1) | side);
    }
  }
  md.tri_basis = (int32_t *)dev_alloc(pl, sizeof(int32_t) * tb.size());
  HIPCHECK(hipMemcpyAsync(md.tri_basis, tb.data(), sizeof(int32_t) * tb.size(),
                          hipMemcpyHostToDevice, s));
  HIPCHECK(hipStreamSynchronize(s));  // tb is a host temporary
}

void rcs_scratch_init() {
  int dev = 0;
  HIPCHECK(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) throw Error(AIM_ERR_ARG, "device index out of range");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[dev]) return;
  void *p = nullptr;
  HIPCHECK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
  if (!p) throw Error(AIM_ERR_HIP, "no device address for the RCS scratch array");
  g_scratch_ptr[dev] = p;
}

void *rcs_scratch_ptr(int device) {
  if (device < 0 || device >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  return g_scratch_ptr[device];
}

// How the part kernel's work is split: triangle chunks, at most `most` (partial sums
// per direction and right-hand side), and right-hand sides per work-group. Many
// directions: chunks of at least two batches, for several rounds of the chip
// (kRcsGroups). Where those are fewer than kRcsFew work-groups the time is one
// work-group's chain: chunks down to kRcsLeast triangles, and right-hand sides in
// smaller groups until there are kRcsSplit (1 direction, 1, 9 and 17 right-hand sides,
// us: 162 triangles 28, 62 and 89 -> 13, 13 and 13; 16 820 triangles 48, 105 and 144 ->
// 26, 55 and 70; 324 directions there 83, 163 and 223 -> 45, 122 and 170; kRcsSplit
// 1024: 17 right-hand sides and 324 directions on those 200; 8-lambda plate, 1 369
// directions: 2 right-hand sides 94 -> 157 with it). The sums of many chunks are then
// added by a wave per slot (a lane each took 20 us there for 600 chunks).
constexpr int64_t kRcsGroups = 4096, kRcsFew = 1024, kRcsSplit = 512, kRcsLeast = 16;
struct RcsSplit {
  int64_t nchunk;
  int rb;
};
static RcsSplit rcs_split(int64_t nt, int64_t ndir, int nrhs, int64_t most) {
  auto up = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
  const int64_t dirs = up(ndir, kDirGroup), groups = dirs * up(nrhs, 16);
  int64_t n = std::min(up(kRcsGroups, groups), up(nt, 128));
  int rb = 16;
  if (groups * n < kRcsFew) {
    n = std::min(std::max<int64_t>(kRcsFew / groups, 1), up(nt, kRcsLeast));
    while (rb > 1 && dirs * n * up(nrhs, rb) < kRcsSplit) rb /= 2;
  }
  n = std::max<int64_t>(std::min({n, most, (int64_t)65535}), 1);
  return {n, rb};
}

// Partial sums into part, then sigma (all device memory). Of 16 right-hand sides per
// work-group, the rest takes the smallest kernel that holds them (one with an unused
// right-hand side or three costs 14 multiply-adds each, a second launch 114).
static void rcs_launch(MeshDev &md, int nrhs, const double2 *x, int64_t ldx, int ntheta,
                       const double *theta, int nphi, const double *phi, double *sigma,
                       double2 *part, RcsSplit split, hipStream_t s) {
  const HostPlan &h = md.hp;
  const int64_t nchunk = split.nchunk;
  const int64_t ndir = (int64_t)ntheta * nphi, groups = (ndir + kDirGroup - 1) / kDirGroup;
  if (groups > INT32_MAX) throw Error(AIM_ERR_ARG, "rcs: too many directions");
  const int64_t per_chunk = (h.nt + nchunk - 1) / nchunk;
  const long double third = (long double)h.k / (6.0L * 3.141592653589793238462643383279502884L);
  const FarMesh fm{md.tris, md.verts, md.tri_basis, md.len, h.nt, h.k,
                   (double)third, (double)(third - (long double)(double)third)};
  constexpr int kMostZ = 32768;
  for (int r0 = 0; r0 < nrhs;) {
    const int left = nrhs - r0;
    auto go = [&](auto kern, int rb, int z) {
      z = std::min(z, kMostZ);
      hipLaunchKernelGGL(kern, dim3((unsigned)groups, (unsigned)nchunk, z), dim3(64 * kRcsWaves),
                         0, s, fm, x, ldx, r0, nrhs, per_chunk, theta, ntheta, phi, nphi,
                         (int)nchunk, part);
      r0 += std::min(left, z * rb);
    };
    const int rb = left < split.rb ? left : split.rb;
    if (rb == 1)
      go(k_rcs_part<1>, 1, left);
    else if (rb == 2)
      go(k_rcs_part<2>, 2, (left + 1) / 2);
    else if (rb <= 4)
      go(k_rcs_part<4>, 4, (left + 3) / 4);
    else if (rb <= 8)
      go(k_rcs_part<8>, 8, (left + 7) / 8);
    else
      go(k_rcs_part<16>, 16, std::max(left / 16, 1));
    LAUNCHCHECK();
  }
  const double keta = h.k * kEta0;
  const int64_t slots = ndir * nrhs;
  int lanes = 1;
  while (lanes < 64 && lanes < nchunk) lanes *= 2;
  hipLaunchKernelGGL(k_rcs_reduce, dim3(loop_blocks(slots * lanes, 256)), dim3(256), 0, s, part,
                     (int)nchunk, slots, lanes, keta * keta / (4.0 * kPi), sigma);
  LAUNCHCHECK();
}

void rcs_mesh(Plan *pl, MeshDev &md, int nrhs, const double2 *x, int64_t ldx, int ntheta,
              const double *theta, int nphi, const double *phi, double *sigma, hipStream_t s) {
  std::vector<void *> tmp;
  auto alloc = [&](size_t bytes) {
    void *p = dev_alloc(pl, bytes);
    tmp.push_back(p);
    return p;
  };
  try {
    double *dth = (double *)alloc(sizeof(double) * ntheta);
    double *dph = (double *)alloc(sizeof(double) * nphi);
    const int64_t ndir = (int64_t)ntheta * nphi;
    double *dsig = (double *)alloc(sizeof(double) * ndir * nrhs);
    HIPCHECK(hipMemcpyAsync(dth, theta, sizeof(double) * ntheta, hipMemcpyHostToDevice, s));
    HIPCHECK(hipMemcpyAsync(dph, phi, sizeof(double) * nphi, hipMemcpyHostToDevice, s));
    const RcsSplit split = rcs_split(md.hp.nt, ndir, nrhs, INT32_MAX);
    double2 *part = (double2 *)alloc(sizeof(double2) * (size_t)ndir * nrhs * split.nchunk);
    rcs_launch(md, nrhs, x, ldx, ntheta, dth, nphi, dph, dsig, part, split, s);
    HIPCHECK(hipMemcpyAsync(sigma, dsig, sizeof(double) * ndir * nrhs, hipMemcpyDeviceToHost, s));
    HIPCHECK(hipStreamSynchronize(s));
  } catch (...) {
    for (void *p : tmp) dev_free(pl, p);
    throw;
  }
  for (void *p : tmp) dev_free(pl, p);
}

void rcs_mesh_noalloc(MeshDev &md, int nrhs, const double2 *x, int64_t ldx, int ntheta,
                      const double *theta, int nphi, const double *phi, double *sigma,
                      double2 *part, hipStream_t s) {
  const int64_t ndir = (int64_t)ntheta * nphi;
  const int64_t slots = ndir * nrhs;  // partial sums needed per chunk
  if (slots > kRcsScratchElems)
    throw Error(AIM_ERR_ARG, "aim_rcs_noalloc: ntheta * nphi * nrhs = " + std::to_string(slots) +
                                 " exceeds its fixed scratch of " +
                                 std::to_string(kRcsScratchElems) + " partial sums");
  // as many chunks as aim_rcs uses, fewer if the scratch cannot hold them
  rcs_launch(md, nrhs, x, ldx, ntheta, theta, nphi, phi, sigma, part,
             rcs_split(md.hp.nt, ndir, nrhs, kRcsScratchElems / slots), s);
}

}  // namespace aim
