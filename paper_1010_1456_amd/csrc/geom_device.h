// Device-side geometry helpers: the 7-point triangle rule, RWG evaluation,
// closed-form static potentials of a triangle (used by the set-up kernels).
#pragma once

#include <hip/hip_runtime.h>

namespace aim {
namespace geo {

// Radon's 7-point rule (degree 5): barycentric points and weights (sum 1).
// a = (6 - sqrt 15)/21, b = (6 + sqrt 15)/21, w_a = (155 - sqrt 15)/1200,
// w_b = (155 + sqrt 15)/1200, centre weight 9/40.
constexpr double kQa = 0.10128650732345633880098736191512;
constexpr double kQb = 0.47014206410511508977044120951345;
constexpr double kWa = 0.12593918054482715259568394550018;
constexpr double kWb = 0.13239415278850618073764938783315;
constexpr double kWc = 0.225;

__host__ __device__ inline void quad_bary(int p, double &l0, double &l1, double &l2, double &w) {
  const double c = 1.0 / 3.0;
  switch (p) {
    case 0: l0 = c; l1 = c; l2 = c; w = kWc; break;
    case 1: l0 = 1.0 - 2.0 * kQa; l1 = kQa; l2 = kQa; w = kWa; break;
    case 2: l0 = kQa; l1 = 1.0 - 2.0 * kQa; l2 = kQa; w = kWa; break;
    case 3: l0 = kQa; l1 = kQa; l2 = 1.0 - 2.0 * kQa; w = kWa; break;
    case 4: l0 = 1.0 - 2.0 * kQb; l1 = kQb; l2 = kQb; w = kWb; break;
    case 5: l0 = kQb; l1 = 1.0 - 2.0 * kQb; l2 = kQb; w = kWb; break;
    default: l0 = kQb; l1 = kQb; l2 = 1.0 - 2.0 * kQb; w = kWb; break;
  }
}

struct D3 {
  double x, y, z;
};
__host__ __device__ inline D3 d3(double x, double y, double z) { return D3{x, y, z}; }
__host__ __device__ inline D3 operator+(D3 a, D3 b) { return d3(a.x + b.x, a.y + b.y, a.z + b.z); }
__host__ __device__ inline D3 operator-(D3 a, D3 b) { return d3(a.x - b.x, a.y - b.y, a.z - b.z); }
__host__ __device__ inline D3 operator*(double s, D3 a) { return d3(s * a.x, s * a.y, s * a.z); }
__host__ __device__ inline double dot(D3 a, D3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__host__ __device__ inline D3 cross(D3 a, D3 b) {
  return d3(a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x);
}
__host__ __device__ inline double norm(D3 a) { return sqrt(dot(a, a)); }

__host__ __device__ inline D3 vtx(const double *verts, int v) {
  return d3(verts[3 * (int64_t)v], verts[3 * (int64_t)v + 1], verts[3 * (int64_t)v + 2]);
}

__host__ __device__ inline D3 quad_point(const D3 *T, int p, double *w) {
  double l0, l1, l2;
  quad_bary(p, l0, l1, l2, *w);
  return l0 * T[0] + l1 * T[1] + l2 * T[2];
}

// R + l computed without cancellation (R^2 = l^2 + R0^2)
__host__ __device__ inline double r_plus_l(double R, double l, double R0sq) {
  return l >= 0.0 ? R + l : R0sq / (R - l);
}

// Closed-form integrals over a planar triangle T at the observation point r
// (Wilton et al. 1984; Graglia 1993): I1 = int_T 1/|r - r'| dS', Iv = int_T
// (r' - r)/|r - r'| dS' and, with GRAD, G1 = int_T grad_r 1/|r - r'| dS': its
// in-plane part by the divergence theorem (minus the edge integrals of 1/R along
// the outward edge normals: - sum_i u_i f_i), its normal part the d-derivative of
// I1, -sign(d) times the solid angle of T seen from r (the arctan sum), zero in
// the plane of T.
template <bool GRAD>
__device__ inline void triangle_statics(const D3 *T, D3 r, double &I1, D3 &Iv, D3 &G1) {
  D3 n = cross(T[1] - T[0], T[2] - T[0]);
  n = (1.0 / norm(n)) * n;
  const double d = dot(r - T[0], n);
  const double ad = fabs(d);
  const D3 rho = r - d * n;
  double acc1 = 0.0, omega = 0.0;
  D3 accv = d3(0, 0, 0), accg = d3(0, 0, 0);
  D3 a = T[0], b = T[1], c = T[2];
#pragma unroll 1
  for (int e = 0; e < 3; ++e) {
    D3 lhat = b - a;
    lhat = (1.0 / norm(lhat)) * lhat;
    const D3 uhat = cross(lhat, n);
    const double t0 = dot(a - rho, uhat);
    const double lp = dot(b - rho, lhat);
    const double lm = dot(a - rho, lhat);
    const double R0sq = t0 * t0 + d * d;
    const double Rp = sqrt(lp * lp + R0sq);
    const double Rm = sqrt(lm * lm + R0sq);
    double f = 0.0;
    if (R0sq > 0.0) {
      f = log(r_plus_l(Rp, lp, R0sq) / r_plus_l(Rm, lm, R0sq));
      if (d != 0.0)  // else the arctans are multiplied by zero
        omega += atan2(t0 * lp, R0sq + ad * Rp) - atan2(t0 * lm, R0sq + ad * Rm);
    }
    acc1 += t0 * f;
    accv = accv + (0.5 * (R0sq * f + lp * Rp - lm * Rm)) * uhat;
    if (GRAD) accg = accg - f * uhat;
    const D3 t = a;  // the next edge
    a = b;
    b = c;
    c = t;
  }
  acc1 -= ad * omega;
  I1 = acc1;
  Iv = accv - (d * acc1) * n;
  if (GRAD) G1 = accg - (d > 0.0 ? omega : -omega) * n;
}

// side 0 / 1 (T+ / T-) of basis n: its triangle's corners and area, the free
// vertex, the sign and the edge length
__device__ inline void basis_side(const int32_t *rwg, const double *len, const double *area,
                                  const int32_t *tris, const double *verts, int64_t n, int side,
                                  D3 *T, double *A, D3 *free_v, double *s, double *l) {
  const int t = rwg[4 * n + side];
  const int fv = rwg[4 * n + 2 + side];
  for (int c = 0; c < 3; ++c) T[c] = vtx(verts, tris[3 * (int64_t)t + c]);
  *A = area[t];
  *free_v = vtx(verts, fv);
  *s = side == 0 ? 1.0 : -1.0;
  *l = len[n];
}

// unit normal (v1 - v0) x (v2 - v0) of a triangle
__device__ inline D3 tri_normal(const D3 *T) {
  const D3 c = cross(T[1] - T[0], T[2] - T[0]);
  return (1.0 / norm(c)) * c;
}

// grid Green's function exp(-jkR)/(4 pi R), 0 at R = 0
__device__ inline double2 green(double k, double R) {
  if (R == 0.0) return make_double2(0.0, 0.0);
  double sn, cs;
  sincos(k * R, &sn, &cs);
  const double g = 0.25 / (3.14159265358979323846 * R);
  return make_double2(g * cs, -g * sn);
}

// true if every vertex of Tn lies in the plane of Tm (relative tolerance
// 1e-12 of the longer first edge): then the MFIE pair term vanishes
__host__ __device__ inline bool coplanar(const D3 *Tm, const D3 *Tn) {
  D3 n = cross(Tm[1] - Tm[0], Tm[2] - Tm[0]);
  n = (1.0 / norm(n)) * n;
  const double sc = fmax(norm(Tm[1] - Tm[0]), norm(Tn[1] - Tn[0]));
  for (int v = 0; v < 3; ++v)
    if (fabs(dot(Tn[v] - Tm[0], n)) > 1e-12 * sc) return false;
  return true;
}

}  // namespace geo
}  // namespace aim
