// Operator set-up on the GPU (FP64): projection weights, grid Green's
// function spectrum, near-zone matrix, plane-wave right-hand sides.
#include <algorithm>
#include <cmath>
#include <cstring>

#include "aim_internal.h"
#include "fft_map.h"
#include "geom_device.h"

namespace aim {
using namespace geo;

namespace {

// Lambda[n][q][u] = sum_{T+-} A_T sum_p w_p F_q(r_p) l_u(r_p), q = x, y, z, div.
__global__ void k_projection(const int32_t *rwg, const double *len, const double *area,
                             const int32_t *tris, const double *verts, const int32_t *anchor3,
                             int64_t n, int M, double x0, double y0, double z0, double h,
                             double *lam) {
  const int K = (M + 1) * (M + 1) * (M + 1);
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n * K) return;
  const int64_t b = t / K;
  const int u = (int)(t - b * K);
  const int ui = u / ((M + 1) * (M + 1)), uj = (u / (M + 1)) % (M + 1), uk = u % (M + 1);
  const double ax = anchor3[3 * b], ay = anchor3[3 * b + 1], az = anchor3[3 * b + 2];
  double acc[4] = {0, 0, 0, 0};
  for (int side = 0; side < 2; ++side) {
    D3 T[3], pf;
    double A, s, l;
    basis_side(rwg, len, area, tris, verts, b, side, T, &A, &pf, &s, &l);
    const double cf = s * l / (2.0 * A);
    const double dv = s * l / A;
    for (int p = 0; p < 7; ++p) {
      double w;
      const D3 r = quad_point(T, p, &w);
      const double xi[3] = {(r.x - x0) / h - ax, (r.y - y0) / h - ay, (r.z - z0) / h - az};
      const int sel[3] = {ui, uj, uk};
      double lw = 1.0;
      for (int d = 0; d < 3; ++d) {
        double v = 1.0;
        for (int m = 0; m <= M; ++m)
          if (m != sel[d]) v *= (xi[d] - m) / (double)(sel[d] - m);
        lw *= v;
      }
      const double aw = A * w * lw;
      acc[0] += aw * cf * (r.x - pf.x);
      acc[1] += aw * cf * (r.y - pf.y);
      acc[2] += aw * cf * (r.z - pf.z);
      acc[3] += aw * dv;
    }
  }
  for (int q = 0; q < 4; ++q) lam[(b * 4 + q) * K + u] = acc[q];
}

// l_s(xi) and its derivative for the nodes 0..M
__device__ inline void lagrange_and_deriv(double xi, int s, int M, double *l, double *dl) {
  double v = 1.0, dv = 0.0;
  for (int m = 0; m <= M; ++m) {
    if (m == s) continue;
    const double f = 1.0 / (double)(s - m);
    dv = dv * (xi - m) * f + v * f;  // product rule, factor by factor
    v *= (xi - m) * f;
  }
  *l = v;
  *dl = dv;
}

// Curl weights of the combined field: W[n][e][u] = sum_{T+-} A_T sum_p w_p
// (t(r_p) x grad l_u(r_p))_e with t = f_n x n_T, so that sum_{e,u} W_e[u]
// A_e[u] = int t . curl A for the interpolant of a grid field A.
__global__ void k_curl_projection(const int32_t *rwg, const double *len, const double *area,
                                  const int32_t *tris, const double *verts, const int32_t *anchor3,
                                  int64_t n, int M, double x0, double y0, double z0, double h,
                                  double *curl) {
  const int K = (M + 1) * (M + 1) * (M + 1);
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n * K) return;
  const int64_t b = t / K;
  const int u = (int)(t - b * K);
  const int sel[3] = {u / ((M + 1) * (M + 1)), (u / (M + 1)) % (M + 1), u % (M + 1)};
  const double ax = anchor3[3 * b], ay = anchor3[3 * b + 1], az = anchor3[3 * b + 2];
  D3 acc = d3(0, 0, 0);
  for (int side = 0; side < 2; ++side) {
    D3 T[3], pf;
    double A, s, l;
    basis_side(rwg, len, area, tris, verts, b, side, T, &A, &pf, &s, &l);
    const D3 nt = tri_normal(T);
    const double cf = s * l / (2.0 * A);
    for (int p = 0; p < 7; ++p) {
      double w;
      const D3 r = quad_point(T, p, &w);
      const double xi[3] = {(r.x - x0) / h - ax, (r.y - y0) / h - ay, (r.z - z0) / h - az};
      double L[3], D[3];
      for (int d = 0; d < 3; ++d) lagrange_and_deriv(xi[d], sel[d], M, &L[d], &D[d]);
      const D3 g = (1.0 / h) * d3(D[0] * L[1] * L[2], L[0] * D[1] * L[2], L[0] * L[1] * D[2]);
      const D3 tv = cross(cf * (r - pf), nt);
      acc = acc + (A * w) * cross(tv, g);
    }
  }
  curl[(b * 3 + 0) * K + u] = acc.x;
  curl[(b * 3 + 1) * K + u] = acc.y;
  curl[(b * 3 + 2) * K + u] = acc.z;
}

// (high orders of large meshes have more weights than a launch has threads)
__global__ void k_to_float(const double *in, float *out, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    out[i] = (float)in[i];
}

// g on the circulant embedding [Px][Py][Pz]: index i folds to min(i, P - i)
__global__ void k_embed_green(double2 *out, int Px, int Py, int Pz, int Nx, int Ny, int Nz,
                              double k, double h) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t tot = (int64_t)Px * Py * Pz;
  if (t >= tot) return;
  const int kk = (int)(t % Pz);
  const int jj = (int)((t / Pz) % Py);
  const int ii = (int)(t / ((int64_t)Py * Pz));
  const int fi = min(ii, Px - ii), fj = min(jj, Py - jj), fk = min(kk, Pz - kk);
  double2 v = make_double2(0.0, 0.0);
  if (fi < Nx && fj < Ny && fk < Nz) {
    const double R = h * sqrt((double)fi * fi + (double)fj * fj + (double)fk * fk);
    v = green(k, R);
  }
  out[t] = v;
}

// z range of the grid planes holding a non-zero projection weight (one atomic
// per wave: one per weight, 1.5 M of them on the 4-lambda sphere, queued on the
// two addresses for 0.54 ms)
__global__ void k_lam_zrange(const double *lam, const int32_t *anchor3, int64_t n, int M,
                             int *zr) {
  const int K = (M + 1) * (M + 1) * (M + 1);
  int lo = INT32_MAX, hi = INT32_MIN;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n * K;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t b = t / K;
    const int u = (int)(t - b * K);
    bool nz = false;
    for (int q = 0; q < 4; ++q) nz |= lam[(b * 4 + q) * K + u] != 0.0;
    if (!nz) continue;
    const int z = anchor3[3 * b + 2] + u % (M + 1);
    lo = min(lo, z);
    hi = max(hi, z);
  }
  for (int off = 32; off > 0; off >>= 1) {
    lo = min(lo, __shfl_xor(lo, off, 64));
    hi = max(hi, __shfl_xor(hi, off, 64));
  }
  if ((threadIdx.x & 63) == 0 && lo <= hi) {
    atomicMin(&zr[0], lo);
    atomicMax(&zr[1], hi);
  }
}

// in-plane weights: plane_lam[b][q][ui (M+1) + uj] = lam[b][q][u] with u's
// z index on the plane
__global__ void k_lam_plane(const double *lam, const int32_t *anchor3, int64_t n, int M, int zp,
                            double *plane_lam) {
  const int K = (M + 1) * (M + 1) * (M + 1), K2 = (M + 1) * (M + 1);
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n * K2) return;
  const int64_t b = t / K2;
  const int u2 = (int)(t - b * K2);
  const int uk = zp - anchor3[3 * b + 2];  // in 0..M: the plane holds the basis' weights
  for (int q = 0; q < 4; ++q)
    plane_lam[(b * 4 + q) * K2 + u2] = lam[(b * 4 + q) * K + u2 * (M + 1) + uk];
}

// 2-D spectrum of g(x, y, 0) from the stored 3-D octant: the inverse z
// transform at z = 0 is the sum over kz, i.e. over the folded kz with
// multiplicity 2 except kz = 0 and kz = Pz/2 (the normalisation carries over:
// octant / (Px Py Pz) summed over kz = 2-D spectrum / (Px Py))
__global__ void k_ghat_zsum(const double2 *oct, double2 *out, int Hx, int Hy, int Hz, int Pz) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)Hx * Hy) return;
  double2 acc = make_double2(0.0, 0.0);
  for (int z = 0; z < Hz; ++z) {
    const double m = (z == 0 || 2 * z == Pz) ? 1.0 : 2.0;
    const double2 v = oct[t * Hz + z];
    acc.x += m * v.x;
    acc.y += m * v.y;
  }
  out[t] = acc;
}

// the octant kz-outer: out[(kz Hx + kx) Hy + ky] = oct[(kx Hy + ky) Hz + kz]
template <typename V>
__global__ void k_octant_planes(const V *oct, V *out, int Hx, int Hy, int Hz) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t plane = (int64_t)Hx * Hy;
  if (t >= plane * Hz) return;
  out[t] = oct[(t % plane) * Hz + t / plane];
}

__global__ void k_extract_octant(const double2 *full, double2 *oct, int Py, int Pz, int Hx, int Hy,
                                 int Hz, double scale) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t tot = (int64_t)Hx * Hy * Hz;
  if (t >= tot) return;
  const int kk = (int)(t % Hz);
  const int jj = (int)((t / Hz) % Hy);
  const int ii = (int)(t / ((int64_t)Hy * Hz));
  double2 v = full[((int64_t)ii * Py + jj) * Pz + kk];
  oct[t] = make_double2(v.x * scale, v.y * scale);
}

__global__ void k_excitation(const int32_t *rwg, const double *len, const double *area,
                             const int32_t *tris, const double *verts, int64_t n, double k,
                             const double *wv /* per wave: khat(3), pol(3) */, int nw,
                             double alpha, bool cfie, double2 *b, int64_t ldb) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n * nw) return;
  const int w = (int)(t / n);
  const int64_t m = t - (int64_t)w * n;
  const D3 kh = d3(wv[6 * w], wv[6 * w + 1], wv[6 * w + 2]);
  const D3 ph = d3(wv[6 * w + 3], wv[6 * w + 4], wv[6 * w + 5]);
  const D3 hd = cross(kh, ph);  // eta H_inc direction
  double vr = 0.0, vi = 0.0;
  for (int side = 0; side < 2; ++side) {
    D3 T[3], pf;
    double A, s, l;
    basis_side(rwg, len, area, tris, verts, m, side, T, &A, &pf, &s, &l);
    const double cf = s * l / (2.0 * A);
    // tested field direction: p_hat (EFIE); alpha p_hat + (1 - alpha) n x (k_hat x p_hat) (CFIE)
    const D3 dir = cfie ? alpha * ph + (1.0 - alpha) * cross(tri_normal(T), hd) : ph;
    for (int p = 0; p < 7; ++p) {
      double wq;
      const D3 r = quad_point(T, p, &wq);
      const double fp = cf * dot(r - pf, dir);
      double sn, cs;
      sincos(k * dot(kh, r), &sn, &cs);  // exp(-j k khat.r)
      vr += A * wq * fp * cs;
      vi -= A * wq * fp * sn;
    }
  }
  b[(int64_t)w * ldb + m] = make_double2(vr, vi);
}

int blocks_for(int64_t n, int t) { return (int)((n + t - 1) / t); }

}  // namespace

template <typename T>
static T *upload(Plan *pl, const T *host, size_t count, hipStream_t s) {
  T *d = (T *)dev_alloc(pl, count * sizeof(T));
  HIPCHECK(hipMemcpyAsync(d, host, count * sizeof(T), hipMemcpyHostToDevice, s));
  return d;
}

static void twiddles(Plan *pl, int P, double2 **d64, float2 **d32, hipStream_t s) {
  std::vector<double2> w(P);
  std::vector<float2> wf(P);
  for (int e = 0; e < P; ++e) {
    long double a = -2.0L * 3.141592653589793238462643383279502884L * (long double)e / (long double)P;
    long double c = cosl(a), sn = sinl(a);
    w[e] = make_double2((double)c, (double)sn);
    wf[e] = make_float2((float)c, (float)sn);
  }
  *d64 = upload(pl, w.data(), P, s);
  *d32 = pl->mixed ? upload(pl, wf.data(), P, s) : nullptr;
  HIPCHECK(hipStreamSynchronize(s));  // host vectors go out of scope
}

void setup_mesh_device(Plan *pl, MeshDev &md, hipStream_t s) {
  const HostPlan &h = md.hp;
  const int M = h.order, K = h.K;
  const int64_t n = h.n;
  double t_phase = wall_ms();
  auto phase_done = [&](int which) {  // the stream is synchronised at each phase end
    const double t = wall_ms();
    md.setup_ms[which] = t - t_phase;
    t_phase = t;
  };
  // geometry and tables
  md.verts = upload(pl, h.verts.data(), h.verts.size(), s);
  md.tris = upload(pl, h.tris.data(), h.tris.size(), s);
  double *area = upload(pl, h.area.data(), h.area.size(), s);
  std::vector<int32_t> rwg(4 * n);
  std::vector<int32_t> alin(n);
  for (int64_t i = 0; i < n; ++i) {
    rwg[4 * i] = h.tp[i];
    rwg[4 * i + 1] = h.tm[i];
    rwg[4 * i + 2] = h.vp[i];
    rwg[4 * i + 3] = h.vm[i];
    alin[i] = (int32_t)(((int64_t)h.anchor[3 * i] * h.grid[1] + h.anchor[3 * i + 1]) * h.grid[2] +
                        h.anchor[3 * i + 2]);
  }
  md.rwg = upload(pl, rwg.data(), rwg.size(), s);
  md.len = upload(pl, h.len.data(), h.len.size(), s);
  md.anchor_lin = upload(pl, alin.data(), alin.size(), s);
  int32_t *anchor3 = upload(pl, h.anchor.data(), h.anchor.size(), s);
  std::vector<int32_t> soff(K);
  for (int u = 0; u < K; ++u) {
    int ui = u / ((M + 1) * (M + 1)), uj = (u / (M + 1)) % (M + 1), uk = u % (M + 1);
    soff[u] = (ui * h.grid[1] + uj) * h.grid[2] + uk;
  }
  md.stencil_off = upload(pl, soff.data(), soff.size(), s);
  HIPCHECK(hipStreamSynchronize(s));

  // projection weights
  md.lam64 = (double *)dev_alloc(pl, sizeof(double) * n * 4 * K);
  hipLaunchKernelGGL(k_projection, dim3(blocks_for(n * K, 256)), dim3(256), 0, s, md.rwg, md.len,
                     area, md.tris, md.verts, anchor3, n, M, h.x0[0], h.x0[1], h.x0[2], h.h,
                     md.lam64);
  LAUNCHCHECK();
  if (pl->mixed) {
    md.lam32 = (float *)dev_alloc(pl, sizeof(float) * n * 4 * K);
    hipLaunchKernelGGL(k_to_float, dim3(loop_blocks(n * 4 * K, 256)), dim3(256), 0, s, md.lam64,
                       md.lam32, n * 4 * K);
    LAUNCHCHECK();
  }
  if (h.cfie) {  // curl weights of the MFIE part
    md.curl64 = (double *)dev_alloc(pl, sizeof(double) * n * 3 * K);
    hipLaunchKernelGGL(k_curl_projection, dim3(blocks_for(n * K, 256)), dim3(256), 0, s, md.rwg,
                       md.len, area, md.tris, md.verts, anchor3, n, M, h.x0[0], h.x0[1], h.x0[2],
                       h.h, md.curl64);
    LAUNCHCHECK();
    if (pl->mixed) {
      md.curl32 = (float *)dev_alloc(pl, sizeof(float) * n * 3 * K);
      hipLaunchKernelGGL(k_to_float, dim3(loop_blocks(n * 3 * K, 256)), dim3(256), 0, s, md.curl64,
                         md.curl32, n * 3 * K);
      LAUNCHCHECK();
    }
  }

  // a flat scatterer lying in one grid plane: every projection weight on
  // that plane (exactly: the off-plane Lagrange factors vanish), so the
  // propagation and the interpolation reduce to the plane
  {
    int zr_h[2] = {INT32_MAX, INT32_MIN};
    int *zr = upload(pl, zr_h, 2, s);
    hipLaunchKernelGGL(k_lam_zrange, dim3(std::min(blocks_for(n * K, 256), 2048)), dim3(256), 0, s, md.lam64,
                       anchor3, n, M, zr);
    LAUNCHCHECK();
    HIPCHECK(hipMemcpyAsync(zr_h, zr, sizeof(zr_h), hipMemcpyDeviceToHost, s));
    HIPCHECK(hipStreamSynchronize(s));
    dev_free(pl, zr);
    md.planar_z = (n > 0 && zr_h[0] == zr_h[1]) ? zr_h[0] : -1;
  }
  if (md.planar_z >= 0) {
    // in-plane stencils: (M+1)^2 weights per component, plane-linear anchors
    const int K2 = (M + 1) * (M + 1);
    md.plane_lam64 = (double *)dev_alloc(pl, sizeof(double) * n * 4 * K2);
    hipLaunchKernelGGL(k_lam_plane, dim3(blocks_for(n * K2, 256)), dim3(256), 0, s, md.lam64,
                       anchor3, n, M, md.planar_z, md.plane_lam64);
    LAUNCHCHECK();
    if (pl->mixed) {
      md.plane_lam32 = (float *)dev_alloc(pl, sizeof(float) * n * 4 * K2);
      hipLaunchKernelGGL(k_to_float, dim3(loop_blocks(n * 4 * K2, 256)), dim3(256), 0, s,
                         md.plane_lam64, md.plane_lam32, n * 4 * K2);
      LAUNCHCHECK();
    }
    std::vector<int32_t> a2(n), so2(K2);
    for (int64_t i = 0; i < n; ++i) a2[i] = h.anchor[3 * i] * h.grid[1] + h.anchor[3 * i + 1];
    for (int u = 0; u < K2; ++u) so2[u] = (u / (M + 1)) * h.grid[1] + u % (M + 1);
    md.plane_anchor = upload(pl, a2.data(), a2.size(), s);
    md.plane_soff = upload(pl, so2.data(), so2.size(), s);
    md.plane_K = K2;
  }

  for (int d = 0; d < 3; ++d)
    if (!fft_plan_for(h.pad[d], &md.plan[d])) throw Error(AIM_ERR_ARG, "unsupported FFT length");
  choose_plane_fft(pl, md);
  node_tables_mesh(pl, md, s);
  phase_done(AIM_SETUP_PROJECTION);

  // twiddles, Green's spectrum octant
  for (int d = 0; d < 3; ++d) {
    md.H[d] = h.pad[d] / 2 + 1;
    twiddles(pl, h.pad[d], &md.tw64[d], &md.tw32[d], s);
  }
  {
    const int Px = h.pad[0], Py = h.pad[1], Pz = h.pad[2];
    const int64_t tot = (int64_t)Px * Py * Pz;
    double2 *e0 = (double2 *)dev_alloc(pl, sizeof(double2) * tot);
    double2 *e1 = (double2 *)dev_alloc(pl, sizeof(double2) * tot);
    hipLaunchKernelGGL(k_embed_green, dim3(blocks_for(tot, 256)), dim3(256), 0, s, e0, Px, Py, Pz,
                       h.grid[0], h.grid[1], h.grid[2], h.k, h.h);
    LAUNCHCHECK();
    fft_pass_contig(e0, e1, md.plan[2], Pz, Pz, (int64_t)Px * Py, fftk::contig_map(Pz),
                    fftk::contig_map(Pz), false, md.tw64[2], s);
    const fftk::LineMap my = fftk::plain_map((int64_t)Py * Pz, Pz);
    const fftk::LineMap mx = fftk::plain_map(0, (int64_t)Py * Pz);
    fft_pass_strided(e1, e0, md.plan[1], Py, Py, Px, Pz, my, my, false, md.tw64[1], 128, s);
    fft_pass_strided(e0, e1, md.plan[0], Px, Px, 1, (int64_t)Py * Pz, mx, mx, false, md.tw64[0],
                     128, s);
    const int64_t noct = (int64_t)md.H[0] * md.H[1] * md.H[2];
    md.ghat64 = (double2 *)dev_alloc(pl, sizeof(double2) * noct);
    hipLaunchKernelGGL(k_extract_octant, dim3(blocks_for(noct, 256)), dim3(256), 0, s, e1,
                       md.ghat64, Py, Pz, md.H[0], md.H[1], md.H[2], 1.0 / (double)tot);
    LAUNCHCHECK();
    if (pl->mixed) {
      md.ghat32 = (float2 *)dev_alloc(pl, sizeof(float2) * noct);
      hipLaunchKernelGGL(k_to_float, dim3(loop_blocks(2 * noct, 256)), dim3(256), 0, s,
                         (const double *)md.ghat64, (float *)md.ghat32, 2 * noct);
      LAUNCHCHECK();
    }
    auto planes = [&](auto *oct, auto *&out) {
      using V = std::remove_reference_t<decltype(*oct)>;
      out = (V *)dev_alloc(pl, sizeof(V) * noct);
      hipLaunchKernelGGL((k_octant_planes<V>), dim3(blocks_for(noct, 256)), dim3(256), 0, s, oct,
                         out, md.H[0], md.H[1], md.H[2]);
      LAUNCHCHECK();
    };
    if (md.planar_z < 0 && md.plane_fft[0].any()) planes(md.ghat64, md.ghatp64);
    if (md.planar_z < 0 && md.plane_fft[1].any()) planes(md.ghat32, md.ghatp32);
    HIPCHECK(hipStreamSynchronize(s));
    dev_free(pl, e0);
    dev_free(pl, e1);
  }
  if (md.planar_z >= 0) {
    const int64_t n2 = (int64_t)md.H[0] * md.H[1];
    md.ghat2d64 = (double2 *)dev_alloc(pl, sizeof(double2) * n2);
    hipLaunchKernelGGL(k_ghat_zsum, dim3(blocks_for(n2, 256)), dim3(256), 0, s, md.ghat64,
                       md.ghat2d64, md.H[0], md.H[1], md.H[2], h.pad[2]);
    LAUNCHCHECK();
    if (pl->mixed) {
      md.ghat2d32 = (float2 *)dev_alloc(pl, sizeof(float2) * n2);
      hipLaunchKernelGGL(k_to_float, dim3(loop_blocks(2 * n2, 256)), dim3(256), 0, s,
                         (const double *)md.ghat2d64, (float *)md.ghat2d32, 2 * n2);
      LAUNCHCHECK();
    }
    HIPCHECK(hipStreamSynchronize(s));
  }
  phase_done(AIM_SETUP_GREEN);

  near_pattern_mesh(pl, md, s);
  near_fill_mesh(pl, md, area, anchor3, s);
  phase_done(AIM_SETUP_NEAR_FILL);
  dev_free(pl, anchor3);
  md.area = area;  // kept for excitation and RCS
  rcs_prepare_mesh(pl, md, s);
}

void excitation_mesh(Plan *pl, MeshDev &md, int nw, const aim_planewave *w, double2 *b,
                     int64_t ldb, hipStream_t s) {
  (void)pl;
  std::vector<double> wv(6 * nw);
  for (int i = 0; i < nw; ++i) {
    const double st = std::sin(w[i].theta), ct = std::cos(w[i].theta);
    const double sp = std::sin(w[i].phi), cp = std::cos(w[i].phi);
    // k_hat = -r_hat; p_hat = theta_hat or phi_hat
    wv[6 * i + 0] = -st * cp;
    wv[6 * i + 1] = -st * sp;
    wv[6 * i + 2] = -ct;
    if (w[i].pol == 0) {
      wv[6 * i + 3] = ct * cp;
      wv[6 * i + 4] = ct * sp;
      wv[6 * i + 5] = -st;
    } else {
      wv[6 * i + 3] = -sp;
      wv[6 * i + 4] = cp;
      wv[6 * i + 5] = 0.0;
    }
  }
  double *dwv = upload(pl, wv.data(), wv.size(), s);
  const int64_t n = md.hp.n;
  hipLaunchKernelGGL(k_excitation, dim3(blocks_for(n * nw, 256)), dim3(256), 0, s, md.rwg, md.len,
                     md.area, md.tris, md.verts, n, md.hp.k, dwv, nw, md.hp.alpha, md.hp.cfie, b,
                     ldb);
  LAUNCHCHECK();
  HIPCHECK(hipStreamSynchronize(s));
  dev_free(pl, dwv);
}

}  // namespace aim
