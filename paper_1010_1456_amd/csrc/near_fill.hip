// Near-zone fill (FP64): Z^near = Z^MOM - Z^grid on the near pairs of every row.
//
// Entry (m, n) of Z^MOM needs the integrals over 2 x 2 triangle pairs, and the
// ~80 bases near m share ~65 triangles; entry (m, n) of Z^grid is Lambda_m^T g
// Lambda_n on two stencils, and the stencils near m share ~220 grid nodes. So a
// work-group takes one row and computes each triangle pair, and the field of
// basis m at each grid node, once.
#include <algorithm>
#include <cmath>

#include "aim_internal.h"
#include "geom_device.h"
#include "turns.h"

namespace aim {
using namespace geo;

namespace {

// constants read with scalar loads where they are used: the series of sine and
// cosine, and the 7-point rule (barycentric coordinates and weight)
struct FillConst {
  TurnsConst turns;
  double rule[7][4];
  constexpr FillConst() : turns{}, rule{} {
    for (int p = 0; p < 7; ++p) {
      const double a = p == 0 ? 1.0 / 3.0 : (p < 4 ? kQa : kQb);
      for (int c = 0; c < 3; ++c) rule[p][c] = a;
      if (p > 0) rule[p][(p - 1) % 3] = 1.0 - 2.0 * a;
      rule[p][3] = p == 0 ? kWc : (p < 4 ? kWa : kWb);
    }
  }
};
__constant__ constexpr FillConst kFill{};
using FillPtr = const __attribute__((address_space(4))) FillConst *;

// g at integer offsets 0 <= (i, j, l) < dim, rows along l
struct Dim3 {
  int x, y, z;
};
__global__ void k_green_table(double2 *tab, Dim3 dim, double k, double h) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= dim.x * dim.y * dim.z) return;
  const int i = t / (dim.y * dim.z), j = (t / dim.z) % dim.y, l = t % dim.z;
  tab[t] = green(k, h * sqrt((double)i * i + (double)j * j + (double)l * l));
}

__global__ void k_to_float2(const double2 *in, float2 *out, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = make_float2((float)in[i].x, (float)in[i].y);
}

struct C3 {  // complex 3-vector
  D3 re, im;
};

// One point p of the outer 7-point rule on test triangle Tm (area Am, free
// vertex pm, normal nm): w_p A_m times the integrand of the combined-field
// entry against the three source functions r' - v_i of triangle Tn (area An).
//   EFIE: int [(r - pm).(r' - v_i) - 4/k^2] G dS'
//         = a.(V + (r - v_i) J0) - (4/k^2) J0, a = r - pm, J0 = int G, V = int (r' - r) G
//   MFIE: [a x nm].[J x (r - v_i)], J = int grad_r G dS' (grad G is parallel to
//         r - r', so the source factor r' - v_i becomes r - v_i); zero for
//         coplanar triangles
// Touching triangles (a shared vertex): G's static part, and the first two terms
// of grad G in powers of R, -(r - r')/(4 pi R^3) and -k^2 (r - r')/(8 pi R), in
// closed form, the smooth rest, (exp(-jkR) - 1)/R and (d/R) k^2/(4 pi) phi(kR),
// phi(x) = (1 - (1 + j x) exp(-j x))/x^2 + 1/2 (series below x = 1e-2), by the
// inner rule. Returns out_i = cE EFIE_i - cH MFIE_i (+ cH/2 Gram_i if same).
struct PairScale {
  double k, cE, cH;  // j cE: alpha j k eta; cH: (1 - alpha) eta
};
template <bool CF>
__device__ __forceinline__ void pair_point(const PairScale &sc, int p, const D3 *Tm, double Am,
                                           D3 pm, const D3 *Tn, double An, bool touch, bool same,
                                           double *out /* 3 x (re, im) */) {
  constexpr double inv4pi = 0.25 / 3.14159265358979323846;
  FillPtr kc = (FillPtr)&kFill;
  const double k = sc.k, kturn = sc.k * (0.5 / 3.14159265358979323846);
  const D3 rp = kc->rule[p][0] * Tm[0] + kc->rule[p][1] * Tm[1] + kc->rule[p][2] * Tm[2];
  double j0r = 0.0, j0i = 0.0;
  C3 V{d3(0, 0, 0), d3(0, 0, 0)}, J{d3(0, 0, 0), d3(0, 0, 0)};
  if (touch) {
    D3 Iv, G1;
    triangle_statics<CF>(Tn, rp, j0r, Iv, G1);
    j0r *= inv4pi;
    V.re = inv4pi * Iv;
    if (CF) J.re = inv4pi * G1 + (0.5 * k * k * inv4pi) * Iv;
  }
#pragma unroll 1
  for (int q = 0; q < 7; ++q) {
    asm volatile("" : "+s"(kc));  // a new value each time: no load is moved out of the loop
    const D3 dv = kc->rule[q][0] * Tn[0] + kc->rule[q][1] * Tn[1] + kc->rule[q][2] * Tn[2] - rp;
    const double R2 = dot(dv, dv);
    const double ri = R2 > 0.0 ? rsqrt(R2) : 0.0, x = k * (R2 * ri);
    double sn, cs;
    sincos_turns(&kc->turns, kturn * (R2 * ri), sn, cs);
    const double aw = An * kc->rule[q][3] * inv4pi;
    double er, ei, gr = 0, gi = 0;  // G and the radial factor of grad_r G along r' - r
    if (!touch) {
      er = cs * ri;
      ei = -sn * ri;
      if (CF) {  // (1 + j k R) exp(-j k R) / R^3
        const double c = ri * ri * ri;
        gr = c * (cs + x * sn);
        gi = c * (x * cs - sn);
      }
    } else {
      er = (cs - 1.0) * ri;
      ei = R2 > 0.0 ? -sn * ri : -k;
      if (CF) {
        double pr, pi;
        if (x < 1e-2) {
          const double x2 = x * x;
          pr = x2 / 8.0 - x2 * x2 / 144.0;
          pi = x / 3.0 - x2 * x / 30.0;
        } else {
          const double ix = 1.0 / (x * x);
          pr = (1.0 - (cs + x * sn)) * ix + 0.5;
          pi = -(x * cs - sn) * ix;
        }
        const double c = -k * k * ri;
        gr = c * pr;
        gi = c * pi;
      }
    }
    er *= aw, ei *= aw;
    j0r += er, j0i += ei;
    V.re = V.re + er * dv;
    V.im = V.im + ei * dv;
    if (CF) {
      gr *= aw, gi *= aw;
      J.re = J.re + gr * dv;
      J.im = J.im + gi * dv;
    }
  }
  const D3 a = rp - pm;
  const double w = kc->rule[p][3] * Am;
  const double c4 = 4.0 / (k * k);
  const double vr = dot(a, V.re) - c4 * j0r, vi = dot(a, V.im) - c4 * j0i;
  D3 xr = d3(0, 0, 0), xi = xr;
  if (CF) {
    const D3 nm = tri_normal(Tm);
    if (!same && !coplanar(Tm, Tn)) {  // [a x nm].[J x b] = b.[(a x nm) x J]
      const D3 t = cross(a, nm);
      xr = cross(t, J.re);
      xi = cross(t, J.im);
    }
  }
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const D3 b = rp - Tn[i];
    const double ab = dot(a, b);
    const double Er = vr + ab * j0r, Ei = vi + ab * j0i;
    double zr = -sc.cE * Ei, zi = sc.cE * Er;
    if (CF) {
      zr -= sc.cH * dot(b, xr);
      zi -= sc.cH * dot(b, xi);
      if (same) zr += 0.5 * sc.cH * ab;
    }
    out[2 * i] = w * zr;
    out[2 * i + 1] = w * zi;
  }
}

// Z^MOM of row m = row0 + blockIdx.x into nearv, its diagonal entry also into zdiag.
// The triangles of a batch of entries are collected in a hash table in LDS; each
// (triangle, side of m) pair is then integrated by 8 lanes, one outer point each
// (the eighth idles), touching pairs first so that their long path shares few
// waves; at the end each entry adds its four pairs. Bound by FP64 issue (7 x 7
// points of about 80 instructions per pair). One thread per entry, with every
// pair integrated by each of the up to 9 entries that need it and the EFIE and
// MFIE terms apart, took (with the grid part below) 213 ms on the 8-lambda CFIE
// sphere (18.4 M entries), 36.9 ms on the 16-lambda plate (4.4 M) and 2.35 s on
// the 128-lambda plate (285 M); both kernels now take 20, 3.7 and 224 ms, two
// thirds of it here. (A register bound of 168, three waves per SIMD, spills and
// gains nothing.)
constexpr int kMomThreads = 128;
constexpr int kMomBatch = 128;  // entries per batch
constexpr int kMomTris = 96;    // distinct triangles per batch (a batch with more is halved)
constexpr int kMomSlots = 512;  // hash slots, at least twice the references
template <bool CF>
__global__ void __launch_bounds__(kMomThreads)
    k_near_mom(const int32_t *__restrict__ rwg, const double *__restrict__ len,
               const double *__restrict__ area, const int32_t *__restrict__ tris,
               const double *__restrict__ verts, const int32_t *__restrict__ rowptr,
               const int32_t *__restrict__ cols, PairScale sc, int64_t row0,
               double2 *__restrict__ nearv, double2 *__restrict__ zdiag) {
  __shared__ int key[kMomSlots];
  __shared__ unsigned short dense[kMomSlots], ref[2 * kMomBatch], task[2 * kMomTris];
  __shared__ int ids[kMomTris];
  __shared__ double2 val[2 * kMomTris * 3];
  __shared__ int count, ntouch, nplain;
  const int64_t m = row0 + blockIdx.x;
  const int tid = threadIdx.x;
  const int e0 = rowptr[m], e1 = rowptr[m + 1];
  int tm[2], vm[2][3];
  for (int s = 0; s < 2; ++s) {
    tm[s] = rwg[4 * m + s];
    for (int c = 0; c < 3; ++c) vm[s][c] = tris[3 * (int64_t)tm[s] + c];
  }
  const double lm = len[m];
  int batch = kMomBatch;
  for (int e = e0; e < e1;) {
    const int eb = min(batch, e1 - e);
    for (int i = tid; i < kMomSlots; i += kMomThreads) key[i] = -1;
    if (tid == 0) count = ntouch = nplain = 0;
    __syncthreads();
    for (int i = tid; i < 2 * eb; i += kMomThreads) {
      const int t = rwg[4 * (int64_t)cols[e + (i >> 1)] + (i & 1)];
      unsigned h = ((unsigned)t * 2654435761u) >> 23;  // 9 bits
      while (true) {
        const int old = atomicCAS(&key[h], -1, t);
        if (old == -1 || old == t) break;
        h = (h + 1) & (kMomSlots - 1);
      }
      ref[i] = (unsigned short)h;
    }
    __syncthreads();
    for (int i = tid; i < kMomSlots; i += kMomThreads)
      if (key[i] >= 0) {
        const int d = atomicAdd(&count, 1);
        dense[i] = (unsigned short)d;
        if (d < kMomTris) ids[d] = key[i];
      }
    __syncthreads();
    const int nt = count;
    if (nt > kMomTris) {  // (uniform) fewer entries: one alone has two triangles
      batch = (eb + 1) / 2;
      __syncthreads();
      continue;
    }
    for (int i = tid; i < 2 * nt; i += kMomThreads) {
      const int s = i & 1;
      const int32_t *vn = &tris[3 * (int64_t)ids[i >> 1]];
      bool touch = false;
      for (int c = 0; c < 3; ++c) {
        const int v = vn[c];
        touch |= v == vm[s][0] || v == vm[s][1] || v == vm[s][2];
      }
      const int at = touch ? atomicAdd(&ntouch, 1) : 2 * nt - 1 - atomicAdd(&nplain, 1);
      task[at] = (unsigned short)i;
    }
    __syncthreads();
    const int nto = ntouch;
    for (int g = tid >> 3; g < 2 * nt; g += kMomThreads / 8) {
      const int i = task[g], s = i & 1, p = tid & 7;
      const int tn = ids[i >> 1];
      double out[6] = {0, 0, 0, 0, 0, 0};
      if (p < 7) {
        D3 Tm[3], Tn[3];
        const int fv = rwg[4 * m + 2 + s];
        const int t = s ? tm[1] : tm[0];
        for (int c = 0; c < 3; ++c) {
          Tm[c] = vtx(verts, s ? vm[1][c] : vm[0][c]);
          Tn[c] = vtx(verts, tris[3 * (int64_t)tn + c]);
        }
        pair_point<CF>(sc, p, Tm, area[t], vtx(verts, fv), Tn, area[tn], g < nto, t == tn, out);
      }
      for (int off = 1; off < 8; off <<= 1)  // the 7 points, fixed order
#pragma unroll
        for (int c = 0; c < 6; ++c) out[c] += __shfl_xor(out[c], off, 8);
      if (p < 3)
        val[3 * i + p] = p == 0 ? make_double2(out[0], out[1])
                                : (p == 1 ? make_double2(out[2], out[3]) : make_double2(out[4], out[5]));
    }
    __syncthreads();
    for (int i = tid; i < eb; i += kMomThreads) {
      const int64_t n = cols[e + i];
      double zr = 0.0, zi = 0.0;
      for (int q = 0; q < 2; ++q) {  // side of n
        const int d = dense[ref[2 * i + q]];
        const int tn = ids[d], fv = rwg[4 * n + 2 + q];
        const int32_t *vn = &tris[3 * (int64_t)tn];
        const int loc = fv == vn[0] ? 0 : (fv == vn[1] ? 1 : 2);
        for (int s = 0; s < 2; ++s) {
          // s_m s_n l_m l_n / (4 A_m A_n)
          const double f = (q == s ? 0.25 : -0.25) * lm * len[n] / (area[tm[s]] * area[tn]);
          const double2 v = val[3 * (2 * d + s) + loc];
          zr += f * v.x;
          zi += f * v.y;
        }
      }
      nearv[e + i] = make_double2(zr, zi);
      if (n == m) zdiag[m] = make_double2(zr, zi);
    }
    __syncthreads();
    e += eb;
  }
}

// Z^grid of row m = row0 + blockIdx.x subtracted from nearv. The grid nodes on the
// stencils of the row's entries are marked in the box of nodes around m's
// stencil (reach R per axis), numbered, and the four fields of basis m there,
//   Phi_q(w) = sum_u c_q[u] g(|w - u|),  q = x, y, z, div,
// c_q = j alpha k eta Lambda_q - (1 - alpha) eta W_q (the curl weights, combined
// field only), c_div = -j (alpha eta / k) Lambda_div, are formed once in LDS,
// kGridNodes at a time; entry (m, n) is then sum_{q, v} Phi_q Lambda_nq[v], a
// half-wave per entry (lanes along the stencil: coalesced weights). About 220 x
// 27 node pairs per row instead of 80 x 27 x 27. Bound by FP64 issue.
// Stencils are m1 nodes per axis: the in-plane one (m1.z = 1) for a scatterer
// in one grid plane, whose other weights are zero.
constexpr int kGridThreads = 256;
constexpr int kGridNodes = 256;
// largest box (node map of 32 KB) and LDS in all of the per-row kernel: second-order
// stencils fit up to a reach of 11 nodes (92 KB, 44 of them the table), in one grid
// plane up to 55 (94 KB)
constexpr int kGridCells = 16384;
constexpr size_t kGridLds = 96 * 1024;
struct GridNear {
  const int32_t *anchor3;
  const double *lam, *curl;
  const double2 *gtab;  // dim gd
  Dim3 m1, R, W, gd;    // stencil, reach, box 2 R + m1, table R + m1
  double cE, cD, cH;    // alpha k eta, alpha eta / k, (1 - alpha) eta
};
template <bool CF>
__global__ void __launch_bounds__(kGridThreads)
    k_near_grid(GridNear gn, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ cols,
                int64_t row0, double2 *__restrict__ nearv) {
  extern __shared__ __align__(16) unsigned char grid_lds[];
  double2 *phi = reinterpret_cast<double2 *>(grid_lds);  // [kGridNodes][4]
  double2 *gt = phi + 4 * kGridNodes;                    // the table
  const int ng = gn.gd.x * gn.gd.y * gn.gd.z, ncell = gn.W.x * gn.W.y * gn.W.z;
  unsigned short *node = reinterpret_cast<unsigned short *>(gt + ng);  // [kGridNodes] cells
  unsigned short *map = node + kGridNodes;                             // [ncell] number + 1
  __shared__ int wsum[kGridThreads / 64], total;
  const int64_t m = row0 + blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int e0 = rowptr[m], e1 = rowptr[m + 1];
  const int K = gn.m1.x * gn.m1.y * gn.m1.z;
  // an entry's stencil corner in the box (0 along z for the in-plane stencil)
  const int ox = gn.R.x - gn.anchor3[3 * m], oy = gn.R.y - gn.anchor3[3 * m + 1];
  const int oz = gn.m1.z > 1 ? gn.R.z - gn.anchor3[3 * m + 2] : 0;
  auto corner = [&](int64_t n) {
    const int32_t *a = gn.anchor3 + 3 * n;
    return ((a[0] + ox) * gn.W.y + a[1] + oy) * gn.W.z + (gn.m1.z > 1 ? a[2] + oz : 0);
  };
  auto stencil = [&](int v) {
    const int vi = v / (gn.m1.y * gn.m1.z), vj = (v / gn.m1.z) % gn.m1.y, vk = v % gn.m1.z;
    return (vi * gn.W.y + vj) * gn.W.z + vk;
  };
  for (int i = tid; i < ng; i += kGridThreads) gt[i] = gn.gtab[i];
  for (int i = tid; i < ncell; i += kGridThreads) map[i] = 0;
  __syncthreads();
  const int hl = tid & 31, half = tid >> 5;
  for (int e = e0 + half; e < e1; e += kGridThreads / 32) {
    const int c = corner(cols[e]);
    for (int v = hl; v < K; v += 32) map[c + stencil(v)] = 1;
  }
  __syncthreads();
  // number the marked cells in order: each thread a run of cells
  const int per = (ncell + kGridThreads - 1) / kGridThreads;
  const int c0 = min(tid * per, ncell), c1 = min(c0 + per, ncell);
  int mine = 0;
  for (int c = c0; c < c1; ++c) mine += map[c];
  int scan = mine;
  for (int off = 1; off < 64; off <<= 1) {
    const int o = __shfl_up(scan, off, 64);
    if (lane >= off) scan += o;
  }
  if (lane == 63) wsum[wave] = scan;
  __syncthreads();
  int first = scan - mine;
  for (int w = 0; w < wave; ++w) first += wsum[w];
  if (tid == kGridThreads - 1) total = first + mine;
  {
    int k = first;
    for (int c = c0; c < c1; ++c)
      if (map[c]) map[c] = (unsigned short)(++k);
  }
  __syncthreads();
  const double *lm = gn.lam + m * 4 * K, *wm = CF ? gn.curl + m * 3 * K : nullptr;
  for (int base = 0; base < total; base += kGridNodes) {
    for (int c = c0; c < c1; ++c) {
      const int k = (int)map[c] - 1 - base;
      if (k >= 0 && k < kGridNodes) node[k] = (unsigned short)c;
    }
    __syncthreads();
    const int nn = min(kGridNodes, total - base);
    for (int i = tid; i < nn; i += kGridThreads) {
      const int c = node[i];
      const int wx = c / (gn.W.y * gn.W.z) - gn.R.x, wy = (c / gn.W.z) % gn.W.y - gn.R.y;
      const int wz = c % gn.W.z - gn.R.z;
      double2 f[4] = {{0, 0}, {0, 0}, {0, 0}, {0, 0}};
      int u = 0;
      for (int ux = 0; ux < gn.m1.x; ++ux) {
        const int gx = abs(wx - ux) * gn.gd.y;
        for (int uy = 0; uy < gn.m1.y; ++uy) {
          const int gy = (gx + abs(wy - uy)) * gn.gd.z;
          for (int uz = 0; uz < gn.m1.z; ++uz, ++u) {
            const double2 g = gt[gy + abs(wz - uz)];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const double ci = (q < 3 ? gn.cE : -gn.cD) * lm[q * K + u];
              f[q].x -= ci * g.y;
              f[q].y += ci * g.x;
              if (CF && q < 3) {
                const double cr = gn.cH * wm[q * K + u];
                f[q].x -= cr * g.x;
                f[q].y -= cr * g.y;
              }
            }
          }
        }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) phi[4 * i + q] = f[q];
    }
    __syncthreads();
    for (int e = e0 + half; e < e1; e += kGridThreads / 32) {
      const int64_t n = cols[e];
      const int c = corner(n);
      const double *ln = gn.lam + n * 4 * K;
      double zr = 0.0, zi = 0.0;
      for (int v = hl; v < K; v += 32) {
        const int k = (int)map[c + stencil(v)] - 1 - base;
        if (k < 0 || k >= kGridNodes) continue;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const double2 f = phi[4 * k + q];
          const double l = ln[q * K + v];
          zr += f.x * l;
          zi += f.y * l;
        }
      }
      for (int off = 16; off > 0; off >>= 1) {
        zr += __shfl_xor(zr, off, 32);
        zi += __shfl_xor(zi, off, 32);
      }
      if (hl == 0) {
        const double2 z = nearv[e];
        nearv[e] = make_double2(z.x - zr, z.y - zi);
      }
    }
    __syncthreads();
  }
}

// The same subtraction one thread per entry by the double sum over the two
// stencils, for near zones whose box of nodes and table do not fit LDS (kGridCells,
// kGridLds); the table may be large.
template <bool CF>
__global__ void __launch_bounds__(128)
    k_near_grid_direct(GridNear gn, const int32_t *__restrict__ rowptr,
                       const int32_t *__restrict__ cols, int64_t row0,
                       double2 *__restrict__ nearv) {
  const int64_t m = row0 + blockIdx.x;
  const int K = gn.m1.x * gn.m1.y * gn.m1.z;
  const double *lm = gn.lam + m * 4 * K, *wm = CF ? gn.curl + m * 3 * K : nullptr;
  const int32_t *am = gn.anchor3 + 3 * m;
  for (int e = rowptr[m] + threadIdx.x; e < rowptr[m + 1]; e += blockDim.x) {
    const int64_t n = cols[e];
    const int32_t *an = gn.anchor3 + 3 * n;
    const int dx = am[0] - an[0], dy = am[1] - an[1], dz = gn.m1.z > 1 ? am[2] - an[2] : 0;
    const double *ln = gn.lam + n * 4 * K;
    double zr = 0.0, zi = 0.0;
    for (int v = 0; v < K; ++v) {
      const int vi = v / (gn.m1.y * gn.m1.z), vj = (v / gn.m1.z) % gn.m1.y, vk = v % gn.m1.z;
      const double l[4] = {ln[v], ln[K + v], ln[2 * K + v], ln[3 * K + v]};
      int u = 0;
      for (int ux = 0; ux < gn.m1.x; ++ux)
        for (int uy = 0; uy < gn.m1.y; ++uy)
          for (int uz = 0; uz < gn.m1.z; ++uz, ++u) {
            const double2 g = gn.gtab[(abs(dx + ux - vi) * gn.gd.y + abs(dy + uy - vj)) * gn.gd.z +
                                      abs(dz + uz - vk)];
            double ci = -gn.cD * lm[3 * K + u] * l[3], cr = 0.0;
            for (int q = 0; q < 3; ++q) {
              ci += gn.cE * lm[q * K + u] * l[q];
              if (CF) cr -= gn.cH * wm[q * K + u] * l[q];
            }
            zr += cr * g.x - ci * g.y;
            zi += cr * g.y + ci * g.x;
          }
    }
    const double2 z = nearv[e];
    nearv[e] = make_double2(z.x - zr, z.y - zi);
  }
}

}  // namespace

void near_fill_mesh(Plan *pl, MeshDev &md, const double *area, const int32_t *anchor3,
                    hipStream_t s) {
  const HostPlan &h = md.hp;
  const int64_t n = h.n;
  md.near64 = (double2 *)dev_alloc(pl, sizeof(double2) * std::max<int64_t>(h.nnz, 1));
  md.zdiag = (double2 *)dev_alloc(pl, sizeof(double2) * n);
  const bool cf = h.cfie;
  const PairScale sc{h.k, h.alpha * h.k * kEta0, (1.0 - h.alpha) * kEta0};
  auto mom = [&](auto kern) {
    for_launches(n, [&](int64_t row0, unsigned rows) {
      hipLaunchKernelGGL(kern, dim3(rows), dim3(kMomThreads), 0, s, md.rwg, md.len, area, md.tris,
                         md.verts, md.rowptr, md.cols, sc, row0, md.near64, md.zdiag);
      LAUNCHCHECK();
    });
  };
  if (cf)
    mom(k_near_mom<true>);
  else
    mom(k_near_mom<false>);

  const bool plane = md.planar_z >= 0;
  GridNear gn{};
  gn.anchor3 = anchor3;
  gn.lam = plane ? md.plane_lam64 : md.lam64;
  gn.curl = md.curl64;
  gn.cE = sc.cE;
  gn.cD = h.alpha * kEta0 / h.k;
  gn.cH = sc.cH;
  // anchors of near pairs differ by at most the near radius in cells, rounded
  // up: rounding or flooring a coordinate moves a difference d to at most
  // ceil(d) (one more if d is an integer missed by rounding), and clamping to
  // the grid does not grow it
  const int M1 = h.order + 1;
  const double cells = std::floor(h.r_near / h.h + 1e-6) + 1.0;
  int *R[3] = {&gn.R.x, &gn.R.y, &gn.R.z}, *W[3] = {&gn.W.x, &gn.W.y, &gn.W.z};
  int *gd[3] = {&gn.gd.x, &gn.gd.y, &gn.gd.z}, *m1[3] = {&gn.m1.x, &gn.m1.y, &gn.m1.z};
  for (int c = 0; c < 3; ++c) {
    const bool flat = plane && c == 2;
    *m1[c] = flat ? 1 : M1;
    *R[c] = flat ? 0 : (int)std::min<double>(cells, h.grid[c] - M1);
    *W[c] = 2 * *R[c] + *m1[c];
    *gd[c] = *R[c] + *m1[c];
  }
  const int64_t ng = (int64_t)gn.gd.x * gn.gd.y * gn.gd.z;
  const int64_t ncell = (int64_t)gn.W.x * gn.W.y * gn.W.z;
  if (ng > INT32_MAX / 2) throw Error(AIM_ERR_ARG, "near zone too large for 32-bit indexing");
  double2 *gtab = (double2 *)dev_alloc(pl, sizeof(double2) * ng);
  gn.gtab = gtab;
  hipLaunchKernelGGL(k_green_table, dim3((unsigned)((ng + 255) / 256)), dim3(256), 0, s, gtab,
                     gn.gd, h.k, h.h);
  LAUNCHCHECK();
  const size_t lds = sizeof(double2) * (4 * kGridNodes + ng) +
                     sizeof(unsigned short) * (kGridNodes + (size_t)ncell);
  if (ncell <= kGridCells && lds <= kGridLds) {
    auto go = [&](auto kern) {
      for_launches(n, [&](int64_t row0, unsigned rows) {
        hipLaunchKernelGGL(kern, dim3(rows), dim3(kGridThreads), lds, s, gn, md.rowptr, md.cols,
                           row0, md.near64);
        LAUNCHCHECK();
      });
    };
    if (cf)
      go(k_near_grid<true>);
    else
      go(k_near_grid<false>);
  } else {
    auto go = [&](auto kern) {
      for_launches(n, [&](int64_t row0, unsigned rows) {
        hipLaunchKernelGGL(kern, dim3(rows), dim3(128), 0, s, gn, md.rowptr, md.cols, row0,
                           md.near64);
        LAUNCHCHECK();
      });
    };
    if (cf)
      go(k_near_grid_direct<true>);
    else
      go(k_near_grid_direct<false>);
  }
  if (pl->mixed) {
    md.near32 = (float2 *)dev_alloc(pl, sizeof(float2) * std::max<int64_t>(h.nnz, 1));
    if (h.nnz > 0) {
      hipLaunchKernelGGL(k_to_float2, dim3((unsigned)((h.nnz + 255) / 256)), dim3(256), 0, s,
                         md.near64, md.near32, h.nnz);
      LAUNCHCHECK();
    }
  }
  HIPCHECK(hipStreamSynchronize(s));
  dev_free(pl, gtab);
}

}  // namespace aim
