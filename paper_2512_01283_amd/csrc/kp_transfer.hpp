// kp_transfer.hpp -- device code shared by the transport (kp_kernels.hip) and
// the imaging (kp_image.hip) kernels: complex arithmetic, extinction
// coefficients, the composite mesh and the tally's per-cell block; and the
// Appendix A cell solution of peel-off.
#pragma once
#include "kp_device.hpp"
#include "kp_internal.hpp"

namespace kp {

template <typename R> struct Cx { R re, im; };
template <typename R> __device__ __forceinline__ Cx<R> cmul(Cx<R> a, Cx<R> b) {
  return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
template <typename R> __device__ __forceinline__ Cx<R> cmulc(Cx<R> a, Cx<R> b) {  // a * conj(b)
  return {a.re * b.re + a.im * b.im, a.im * b.re - a.re * b.im};
}
template <typename R> __device__ __forceinline__ Cx<R> cadd(Cx<R> a, Cx<R> b) {
  return {a.re + b.re, a.im + b.im};
}
template <typename R> __device__ __forceinline__ R cabs2(Cx<R> a) { return a.re * a.re + a.im * a.im; }
template <typename R> __device__ __forceinline__ Cx<R> cscale(Cx<R> a, R s) { return {a.re * s, a.im * s}; }

// e^z and (e^z - 1) / z of z = x + i y.  Where |z|^2 would leave the type's normal
// range (a ray through a cell's edge has no length in it; FP32 exponents of a
// medium's thin wings) the quotient is its limit 1 + z / 2, whose next term z^2 / 6
// is far below rounding there.
template <typename R> __device__ __forceinline__ void cx_exp_phi(R x, R y, Cx<R>& ez, Cx<R>& phi) {
  const R ex = k_exp(x), cy = k_cos(y), sy = k_sin(y), sh = k_sin((R)0.5 * y);
  ez = {ex * cy, ex * sy};
  const Cx<R> em1{k_expm1(x) * cy - (R)2 * sh * sh, ex * sy};
  const R den = x * x + y * y;
  if (den < (sizeof(R) == 4 ? (R)1e-30 : (R)1e-280)) phi = {(R)1 + (R)0.5 * x, (R)0.5 * y};
  else phi = {(em1.re * x + em1.im * y) / den, (em1.im * x - em1.re * y) / den};
}

// Dimensionless extinction coefficients for a direction with cos(theta') =
// ct to the grain axis (dipole: cross sections from Im of the
// polarizability, normalised by the orientation average).
template <typename R, bool SPHERE>
__device__ __forceinline__ void alphas(const DustDev& D, R ct, R& a1, R& a2, R& a3) {
  if (SPHERE) { a1 = (R)1; a2 = (R)0; a3 = (R)0; return; }
  R cth = (R)D.ap_im * ct * ct + (R)D.aa_im * (sizeof(R) == 4 ? ((R)1 - ct) * ((R)1 + ct) : (R)1 - ct * ct);
  R cph = (R)D.ap_im;
  a1 = (cth + cph) * (R)D.inv2cavg;
  a2 = (cth - cph) * (R)D.inv2cavg;
  a3 = (R)D.alpha3_scale * a2;
}

// ---------------------------------------------------------------------------
// Composite mesh with static refinement (Sec. 2: the mesh the packets
// cross).  Inside a leaf block the cell walk is the uniform one; leaving it,
// the point is expressed in finest-cell units (exact on the crossed face,
// since cell edges are powers of two of the finest one), its finest cell
// taken with the face rule (a coordinate on a face belongs to the cell the
// direction points into), and the leaf holding that cell found by
// descending from its root block.
// ---------------------------------------------------------------------------
__device__ __forceinline__ long long finest_cell(double t, double n) {
  const double fl = floor(t);
  long long X = (long long)fl;
  if (fl == t && n < 0.0) X -= 1;
  return X;
}

__device__ __forceinline__ int mesh_find(const MeshDev& m, const long long X[3]) {
  const long long full = (long long)m.block << m.max_level;
  const long long r0 = X[0] / full, r1 = X[1] / full, r2 = X[2] / full;
  int node = (int)(r0 + (long long)m.rx * (r1 + (long long)m.ry * r2));
  long long o0 = r0 * full, o1 = r1 * full, o2 = r2 * full, size = full;
  for (int c = m.child[node]; c >= 0; c = m.child[node]) {
    size >>= 1;
    int oct = 0;
    if (X[0] - o0 >= size) { oct |= 1; o0 += size; }
    if (X[1] - o1 >= size) { oct |= 2; o1 += size; }
    if (X[2] - o2 >= size) { oct |= 4; o2 += size; }
    node = c + oct;
  }
  return m.leaf_of_node[node];
}

// A ray (direction om) in leaf `leaf` at local cell ci, fraction f whose
// index on some axis left the leaf: the leaf beyond (leaf, lvl, ci, f
// updated), or false if the ray left the domain.
__device__ __forceinline__ bool mesh_ray_cross(const MeshDev& m, int& leaf, int& lvl, int ci[3], double f[3],
                                               const double om[3]) {
  const int4 o = reinterpret_cast<const int4*>(m.leaf_org)[leaf];
  const double sz = (double)(1ll << (m.max_level - o.w));
  const long long X0[3] = {o.x, o.y, o.z};
  double t[3];
  long long X[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    t[k] = (double)X0[k] + ((double)ci[k] + f[k]) * sz;
    X[k] = finest_cell(t[k], om[k]);
    if (X[k] < 0 || X[k] >= m.nfine[k]) return false;
  }
  leaf = mesh_find(m, X);
  const int4 o1 = reinterpret_cast<const int4*>(m.leaf_org)[leaf];
  lvl = o1.w;
  const int sh = m.max_level - lvl;
  const long long X1[3] = {o1.x, o1.y, o1.z};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const long long i = (X[k] - X1[k]) >> sh;
    ci[k] = (int)i;
    f[k] = fmin(1.0, fmax(0.0, (t[k] - (double)X1[k]) / (double)(1ll << sh) - (double)i));
  }
  return true;
}

// Components of the tally kept per cell and the per-cell stride in doubles:
// spheres never create circular polarisation from unpolarised light, so the
// antisymmetric (V) part of the coherency is identically zero.
// Per-cell tally block of TS doubles (one 64- or 128-byte aligned block):
// slots [0, NC) the coherency sums.  For non-spherical grains slots NC..NC+3 hold
// the unit quaternion (w, x, y, z) of the cell's grain frame, formed once per run
// from the alignment direction (eq. grain-quaternion) instead of at every step and
// scattering.  The density comes from the compact FP32 array (64 MB at 256^3, which
// stays in the caches), asked for on entering the cell: an empty cell, half of a
// disk's grid, then touches no block (aligned slab 18.1 -> 15.7 ms, batched disk
// 27.6 -> 25.2, aligned 256^3 disk 12.6 -> 12.1 against the density in the block;
// asking for the next cell's quaternion early too: 16.3, 26.4, 12.4).
template <bool SPHERE> struct TallyShape {
  static constexpr int NC = SPHERE ? 6 : 9;
  static constexpr int TS = SPHERE ? 8 : 16;
  static constexpr int QUAT = NC;
  static constexpr bool HAS_B = !SPHERE;  // grain quaternion in slots NC..NC+3
};

// ---------------------------------------------------------------------------
// Peel-off: the Appendix A solution in its eigenbasis (step 2 has its own form of
// it, dichroic_cell in kp_image.hip).
// ---------------------------------------------------------------------------
__device__ __forceinline__ void appA_eigen(double a1, double a2, double a3, double dtau,
                                           const double src[4], double s[4]) {
  const double a = a1 + a2, b = a1 - a2;
  const double A = s[0] + s[1], B = s[0] - s[1];
  const double SA = src[0] + src[1], SB = src[0] - src[1];
  const double An = A * exp(-a * dtau) + SA * dtau * phi1(a * dtau);
  const double Bn = B * exp(-b * dtau) + SB * dtau * phi1(b * dtau);
  double Un, Vn;
  if (a3 == 0.0) {
    const double e = exp(-a1 * dtau), g = dtau * phi1(a1 * dtau);
    Un = s[2] * e + src[2] * g;
    Vn = s[3] * e + src[3] * g;
  } else {
    // U + iV relaxes as exp(-(a1 - i a3) tau) toward the stationary state
    Cx<double> ez, phic;
    cx_exp_phi(-a1 * dtau, a3 * dtau, ez, phic);
    const Cx<double> Z{s[2], s[3]}, SZ{src[2], src[3]};
    const Cx<double> Zn = cadd(cmul(Z, ez), cscale(cmul(SZ, phic), dtau));
    Un = Zn.re; Vn = Zn.im;
  }
  s[0] = 0.5 * (An + Bn);
  s[1] = 0.5 * (An - Bn);
  s[2] = Un;
  s[3] = Vn;
}

}  // namespace kp
