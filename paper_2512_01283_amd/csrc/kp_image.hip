// kp_image.hip -- gfx950 kernels of the deterministic imaging ray-march (step
// 2) of Yang & Wang, arXiv:2512.01283, Sec. 2.3 and Appendix A.
#include <type_traits>

#include "kp_transfer.hpp"

namespace kp {

namespace {

// a . C b for a symmetric matrix C (xx yy zz xy xz yz) is m . C with
// m = sym(a, b): the cell's six numbers against six constants of the camera
struct Sym6 {
  double m[6];
  __device__ __forceinline__ void set(const V3<double>& a, const V3<double>& b) {
    m[0] = a.x * b.x; m[1] = a.y * b.y; m[2] = a.z * b.z;
    m[3] = a.x * b.y + a.y * b.x; m[4] = a.x * b.z + a.z * b.x; m[5] = a.y * b.z + a.z * b.y;
  }
  __device__ __forceinline__ double dot(const double C[6]) const {
    return m[0] * C[0] + m[1] * C[1] + m[2] * C[2] + m[3] * C[3] + m[4] * C[4] + m[5] * C[5];
  }
};

// Camera constants of a ray: its basis and the maps of a cell's coherency to
// r11 + r22, r11 - r22 and r12 of an isotropic scatterer.
struct Camera {
  V3<double> om, e1, e2;
  Sym6 sum, dif, mix;
  __device__ __forceinline__ void set(const ViewDev& v) {
    om = {v.ox, v.oy, v.oz};
    e1 = {v.tx, v.ty, v.tz};
    e2 = {v.px, v.py, v.pz};
    Sym6 a, b;
    a.set(e1, e1);
    b.set(e2, e2);
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      // the off-diagonal numbers of C appear twice in e C e, and set() counts both
      sum.m[k] = a.m[k] + b.m[k];
      dif.m[k] = a.m[k] - b.m[k];
    }
    mix.set(e1, e2);
  }
};

// One dichroic cell (Appendix A) along the ray: b the grain axis (norm 1
// within rounding of its FP32 components, ib2 = 1 / b.b), S the source per unit
// length (camera basis), tl the path length in it, dtau its extinction at the
// orientation average, eB the thermal source per unit optical depth.  In the
// eigenbasis A = I + Q, B = I - Q, U + iV of the grain frame, whose Q axis is the
// projection of b on the sky: the rotation from the camera's basis needs
// only b . e1 and b . e2.
__device__ __forceinline__ void dichroic_cell(const DustDev& D, double b1, double b2, double bo, double ib2, double tl,
                                              double dtau, double eB, const double S[4], double st[4]) {
  const double q = b1 * b1 + b2 * b2;
  double c2 = 1.0, s2 = 0.0;
  if (q > KP_POLE2) {
    const double iq = 1.0 / q;
    c2 = (b1 * b1 - b2 * b2) * iq;
    s2 = 2.0 * b1 * b2 * iq;
  }
  const double ct2 = bo * bo * ib2;
  const double cth = D.ap_im * ct2 + D.aa_im * (1.0 - ct2);
  const double a1 = (cth + D.ap_im) * D.inv2cavg, a2 = (cth - D.ap_im) * D.inv2cavg;
  const double a3 = D.alpha3_scale * a2;
  const double Qg = c2 * st[1] + s2 * st[2], Ug = c2 * st[2] - s2 * st[1];
  const double S1 = c2 * S[1] + s2 * S[2], S2 = c2 * S[2] - s2 * S[1];
  const double ed = eB * dtau;
  const double a = a1 + a2, b = a1 - a2;
  double An, Bn, Un, Vn, E, P;
  exp_phi(a * dtau, E, P);
  An = (st[0] + Qg) * E + ((S[0] + S1) * tl + ed * a) * P;
  exp_phi(b * dtau, E, P);
  Bn = (st[0] - Qg) * E + ((S[0] - S1) * tl + ed * b) * P;
  if (a3 == 0.0) {
    exp_phi(a1 * dtau, E, P);
    Un = Ug * E + S2 * tl * P;
    Vn = st[3] * E + S[3] * tl * P;
  } else {
    // U + iV relaxes as exp(-(a1 - i a3) tau) toward the stationary state
    Cx<double> ez, phic;
    cx_exp_phi(-a1 * dtau, a3 * dtau, ez, phic);
    const Cx<double> Zn = cadd(cmul(Cx<double>{Ug, st[3]}, ez), cscale(cmul(Cx<double>{S2, S[3]}, phic), tl));
    Un = Zn.re;
    Vn = Zn.im;
  }
  st[0] = 0.5 * (An + Bn);
  const double Qn = 0.5 * (An - Bn);
  st[1] = c2 * Qn - s2 * Un;
  st[2] = s2 * Qn + c2 * Un;
  st[3] = Vn;
}

// Stokes source toward the camera of dipole grains (axis b) whose incident
// coherency is C9: rho'_ij = h_i . C conj(h_j) with h_i = a_perp e_i +
// (a_par - a_perp)(b . e_i) b, written in the three products C needs with b:
// g = Re C b, z = Im C b = b x w (w the imaginary parts), b . g.
__device__ __forceinline__ void dipole_source(const double C9[9], const Camera& cam, const DustDev& D,
                                              const V3<double>& b, double b1, double b2, double ib2, double pf,
                                              double S[4]) {
  const double dr = D.aa_re - D.ap_re, di = D.aa_im - D.ap_im;
  const double P = D.ap_re * D.ap_re + D.ap_im * D.ap_im;
  // a_perp conj(a_par - a_perp), |a_par - a_perp|^2
  const double kr = (D.ap_re * dr + D.ap_im * di) * ib2, ki = (D.ap_im * dr - D.ap_re * di) * ib2;
  const V3<double> g{C9[0] * b.x + C9[3] * b.y + C9[4] * b.z, C9[3] * b.x + C9[1] * b.y + C9[5] * b.z,
                     C9[4] * b.x + C9[5] * b.y + C9[2] * b.z};
  const V3<double> w{C9[6], C9[7], C9[8]};
  const V3<double> z = cross(b, w);
  const double T = (dr * dr + di * di) * ib2 * ib2 * dot(b, g);
  const double u1 = dot(cam.e1, g), u2 = dot(cam.e2, g), v1 = dot(cam.e1, z), v2 = dot(cam.e2, z);
  const double x1 = kr * u1 - ki * v1, x2 = kr * u2 - ki * v2;
  const double y1 = kr * v1 + ki * u1, y2 = kr * v2 + ki * u2;
  const double d1 = b1 * (2.0 * x1 + T * b1), d2 = b2 * (2.0 * x2 + T * b2);
  S[0] = pf * (P * cam.sum.dot(C9) + d1 + d2);
  S[1] = pf * (P * cam.dif.dot(C9) + d1 - d2);
  S[2] = 2.0 * pf * (P * cam.mix.dot(C9) + b2 * x1 + b1 * x2 + T * b1 * b2);
  S[3] = -2.0 * pf * (P * dot(w, cam.om) + b2 * y1 - b1 * y2);
}

}  // namespace

// ---------------------------------------------------------------------------
// Step 2 (Sec. 2.3): one lane per (wavelength, view, pixel).  The ray enters
// the grid box from the far side and is marched cell by cell toward the
// camera; each cell applies the Appendix A solution with the cell's
// extinction for the camera direction and the scattering source formed from
// the coherency tally (or a caller-given per-view source).  FP64 throughout.
// A wavefront takes 8 x 8 pixels and a 256-thread block 16 x 16, so that rays
// marching together cross the same cells' lines; a map that is no multiple of them
// is packed without gaps (image_pixel), small ones share wavefronts (MULTI):
// padded to 16 x 16, images of 17 x 17 pixels took 1.8 ms instead of 0.6 (64^3 sphere,
// 64 views, 32 wavelengths), of 4096 x 1 with 8 views 414 us instead of 90.  Consecutive
// blocks, which the hardware deals out over the 8 XCDs, are regrouped so that one XCD's
// L2 serves neighbouring tiles.  A cell costs six numbers against the camera's constants
// (spheres) or three products with its grain axis (dichroic grains), one
// exponential per eigenvalue and no division by the density; what then bounds
// a large grid are the L2's misses on the tally's 64-byte sectors (50 G/s: little of
// the grid is crossed twice by one camera's rays).  So the grain axis comes from the
// tally's block, whose second sector the coherency reads anyway, where step 1 of
// the same call wrote it (three more gathers otherwise: 6.2 ms instead of 3.2 for
// the aligned 256^3 disk and 8 views), and spheres run two blocks per CU (see
// launch_image).  Before, with complex 3 x 3 products, three divisions, six
// exponentials and the grain's quaternion per cell, VALU issue took 0.6 of the
// cycles: 256^3 disk, 8 views 2.74 -> 1.94 ms; aligned 7.9 -> 3.2; 150^3 x 8
// wavelengths x 16 views 24.6 -> 10.9; 128^3 aligned slab, 4 views 0.97 -> 0.39; 32^3
// sphere, one view 0.086 -> 0.043.  Asking for the next cell's source one step
// early (a two-cell pipeline) measured 2.3 ms and 6.4 ms: it adds lines in flight, and
// it is their reuse that is short.
// ---------------------------------------------------------------------------
template <bool ALIGNED, bool SPHERE, bool USER_S, bool MESH, bool MULTI>
__global__ void __launch_bounds__(256) k_image(ImageArgs a) {
  // No fused multiply-adds in the geometry: a ray that grazes a cell face (a
  // pixel centre on a face, drifting off it by ~1e-16 per cell) then takes the
  // face-side decisions of a plain (unfused) evaluation of the same expressions.
#pragma clang fp contract(off)
  static_assert(!(ALIGNED && SPHERE), "the extinction of spheres is scalar");
  const uint64_t npix = (uint64_t)a.npx * a.npy;
  uint32_t blk = blockIdx.x;
  if (blk < gridDim.x - gridDim.x % 8u) blk = (blk & 7u) * (gridDim.x / 8u) + (blk >> 3);
  const uint32_t wave =
      (uint32_t)__builtin_amdgcn_readfirstlane((int)(blk * (blockDim.x >> 6) + (threadIdx.x >> 6)));
  // the (wavelength, view) map of this lane's pixel and the pixel's place in it
  uint32_t map, px = threadIdx.x & 63u;
  if (MULTI) {
    px += 64u * wave;
    map = px / (uint32_t)npix;
    px -= map * (uint32_t)npix;
  } else {
    const uint32_t per = ((uint32_t)npix + 63u) >> 6;
    map = wave / per;
    px += 64u * (wave - map * per);
  }
  const int lam = (int)(map / (uint32_t)a.n_views), v = (int)(map - (uint32_t)lam * (uint32_t)a.n_views);
  if (lam >= a.n_lambda || px >= npix) return;
  int ix, iy;
  image_pixel(px, (uint32_t)a.npx, (uint32_t)a.npy, ix, iy);
  const ViewDev vw = a.views[v];
  const DustDev& D = a.dust[lam];
  const double W = vw.half_width;
  const double xp = -W + (ix + 0.5) * (2.0 * W / a.npx);
  const double yp = -W + (iy + 0.5) * (2.0 * W / a.npy);
  const double P0[3] = {xp * vw.px - yp * vw.tx, xp * vw.py - yp * vw.ty, xp * vw.pz - yp * vw.tz};
  const double om[3] = {vw.ox, vw.oy, vw.oz};
  const double lo[3] = {a.x0, a.y0, a.z0};
  const int nn[3] = {a.nx, a.ny, a.nz};
  double sn = -__builtin_huge_val(), sf = __builtin_huge_val();
  bool miss = false;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    if ((a.boundary >> k) & 1) continue;  // the periodic copies fill the axis
    const double hi = lo[k] + nn[k] * a.dx;
    if (om[k] != 0.0) {
      const double s1 = (lo[k] - P0[k]) / om[k], s2 = (hi - P0[k]) / om[k];
      sn = fmax(sn, fmin(s1, s2));
      sf = fmin(sf, fmax(s1, s2));
    } else if (P0[k] < lo[k] || P0[k] >= hi) {
      miss = true;
    }
  }
  double st[4] = {0.0, 0.0, 0.0, 0.0};
  if (!miss && sn < sf) {
    int ci[3];
    double f[3];
    // composite mesh: the leaf block of the ray and its level
    int leaf = 0, lvl = 0;
    const MeshDev& m = a.mesh;
    const uint64_t B = MESH ? (uint64_t)m.block : 0;
    if (MESH) {
      // the entry point in finest cells, clamped into the domain
      double t[3];
      long long X[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        t[k] = (P0[k] + sn * om[k] - lo[k]) / m.fine;
        X[k] = (long long)floor(t[k]);
        X[k] = X[k] < 0 ? 0 : (X[k] > m.nfine[k] - 1 ? m.nfine[k] - 1 : X[k]);
      }
      leaf = mesh_find(m, X);
      const int4 org = reinterpret_cast<const int4*>(m.leaf_org)[leaf];
      lvl = org.w;
      const int sh = m.max_level - lvl;
      const long long X0[3] = {org.x, org.y, org.z};
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const long long i = (X[k] - X0[k]) >> sh;
        ci[k] = (int)i;
        f[k] = fmin(1.0, fmax(0.0, (t[k] - (double)X0[k]) / (double)(1ll << sh) - (double)i));
      }
    }
#pragma unroll
    for (int k = 0; k < 3 && !MESH; ++k) {
      const double t = (P0[k] + sn * om[k] - lo[k]) / a.dx;
      const double fl = floor(t);
      if ((a.boundary >> k) & 1) {
        const long long n = nn[k], i = (long long)fl;
        ci[k] = (int)(((i % n) + n) % n);
        f[k] = fmin(1.0, fmax(0.0, t - fl));
        continue;
      }
      int i = (int)fl;
      i = i < 0 ? 0 : (i > nn[k] - 1 ? nn[k] - 1 : i);
      ci[k] = i;
      f[k] = fmin(1.0, fmax(0.0, t - (double)i));
    }
    Camera cam;
    cam.set(vw);
    const double pfac = SPHERE ? D.pfac * (D.ap_re * D.ap_re + D.ap_im * D.ap_im) : D.pfac;
    double clen = MESH ? ldexp(a.dx, -lvl) : a.dx;
    double inv_vol = 1.0 / (clen * clen * clen);
    // per axis: the face coordinate ahead, the step, the reciprocal direction
    // (kept finite: that of a subnormal component overflows, and a ray that starts
    // on the face ahead of it has no length left, not 0 times infinity)
    double face[3], rom[3];
    int stp[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      face[k] = om[k] > 0.0 ? 1.0 : 0.0;
      stp[k] = om[k] > 0.0 ? 1 : -1;
      rom[k] = om[k] != 0.0 ? fmin(1.7976931348623157e308, fmax(-1.7976931348623157e308, 1.0 / om[k])) : 0.0;
    }
    const double eBf = D.ka_cell / D.ke_cell;
    auto flat = [&]() {
      return MESH ? (uint64_t)leaf * B * B * B + (uint64_t)ci[0] + B * ((uint64_t)ci[1] + B * ci[2])
                  : (uint64_t)((uint32_t)ci[0] + (uint32_t)a.nx * ((uint32_t)ci[1] + (uint32_t)a.ny * (uint32_t)ci[2]));
    };
    uint64_t cn = flat();
    float rho_n = a.rho[cn];
    while (true) {
      // this cell; its density was loaded one step ago
      const uint64_t c = cn;
      const double rho = (double)rho_n;
      const uint64_t sl = tally_slot(c, ci[0], ci[1], ci[2], MESH ? 0 : a.tbx, a.tby);
      const double clen_c = clen, inv_vol_c = inv_vol;
      double t[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) t[k] = om[k] != 0.0 ? (face[k] - f[k]) * rom[k] : __builtin_huge_val();
      // the exit face: the smallest distance, the lowest axis of equal ones
      const bool ax0 = t[0] <= t[1] && t[0] <= t[2], ax1 = !ax0 && t[1] <= t[2], ax2 = !ax0 && !ax1;
      const double tb = ax0 ? t[0] : (ax1 ? t[1] : t[2]);
      f[0] = ax0 ? 1.0 - face[0] : fmin(1.0, fmax(0.0, f[0] + tb * om[0]));
      f[1] = ax1 ? 1.0 - face[1] : fmin(1.0, fmax(0.0, f[1] + tb * om[1]));
      f[2] = ax2 ? 1.0 - face[2] : fmin(1.0, fmax(0.0, f[2] + tb * om[2]));
      ci[0] += ax0 ? stp[0] : 0;
      ci[1] += ax1 ? stp[1] : 0;
      ci[2] += ax2 ? stp[2] : 0;
      const int cx = ax0 ? ci[0] : (ax1 ? ci[1] : ci[2]);  // the index that moved
      bool left;
      if (MESH) {
        left = false;
        if (cx < 0 || cx >= (int)B) {
          // the leaf beyond the block face, if the ray does not leave the domain
          left = !mesh_ray_cross(m, leaf, lvl, ci, f, om);
          if (!left) {
            clen = ldexp(a.dx, -lvl);
            inv_vol = 1.0 / (clen * clen * clen);
          }
        }
      } else {
        const int n = ax0 ? nn[0] : (ax1 ? nn[1] : nn[2]);
        left = cx < 0 || cx >= n;
        if (a.boundary != 0 && left && ((a.boundary >> (ax0 ? 0 : (ax1 ? 1 : 2))) & 1)) {
          const int wrapped = cx < 0 ? n - 1 : 0;
          if (ax0) ci[0] = wrapped;
          else if (ax1) ci[1] = wrapped;
          else ci[2] = wrapped;
          left = false;
        }
      }
      if (!left) {
        cn = flat();
        rho_n = a.rho[cn];
      }
      if (rho > 0.0) {
        const double tl = tb * clen_c, dtau = rho * D.kext * tl;
        // the dust's thermal emission per unit optical depth,
        // (kappa_abs / kappa_ext) (alpha1, alpha2, 0, 0) B in the grain-frame
        // basis of the ray (eq. polarized-rt)
        const double eB = a.em_B ? eBf * (double)a.em_B[(uint64_t)lam * a.ncell + c] : 0.0;
        double S[4];
        double C9[9] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        const double pf = pfac * inv_vol_c;
        if (USER_S) {
          const double* Sv = a.user_S + (((uint64_t)lam * a.nslot + sl) * a.n_views + v) * 4;
          S[0] = Sv[0]; S[1] = Sv[1]; S[2] = Sv[2]; S[3] = Sv[3];
        } else {
          const double* T = a.tally + ((uint64_t)lam * a.nslot + sl) * TallyShape<SPHERE>::TS;
#pragma unroll
          for (int k = 0; k < TallyShape<SPHERE>::NC; ++k) C9[k] = T[k];
        }
        if (SPHERE) {
          double E, P;
          exp_phi(dtau, E, P);
          if (!USER_S) {
            S[0] = pf * cam.sum.dot(C9);
            S[1] = pf * cam.dif.dot(C9);
            S[2] = 2.0 * pf * cam.mix.dot(C9);
            S[3] = 0.0;
          }
          const double tP = tl * P;
          st[0] = fma(st[0], E, fma(S[0], tP, eB * dtau * P));
#pragma unroll
          for (int k = 1; k < (USER_S ? 4 : 3); ++k) st[k] = fma(st[k], E, S[k] * tP);
        } else {
          V3<double> b{0.0, 0.0, 1.0};
          double ib2 = 1.0;
          if (ALIGNED && a.axis_in_tally) {
            // the grain frame's z axis, from the block the coherency came from
            const double* q = a.tally + ((uint64_t)lam * a.nslot + sl) * TallyShape<SPHERE>::TS + TallyShape<SPHERE>::QUAT;
            b = grain_axis(Quat<double>{q[0], q[1], q[2], q[3]});
          } else if (ALIGNED) {
            b = V3<double>{(double)a.bx[c], (double)a.by[c], (double)a.bz[c]};
            ib2 = 1.0 / dot(b, b);
          }
          const double b1 = dot(b, cam.e1), b2 = dot(b, cam.e2), bo = dot(b, cam.om);
          if (!USER_S) dipole_source(C9, cam, D, b, b1, b2, ib2, pf, S);
          dichroic_cell(D, b1, b2, bo, ib2, tl, dtau, eB, S, st);
        }
      }
      if (left) break;
    }
  }
  double* out = a.images + (((uint64_t)lam * a.n_views + v) * 4) * npix + (uint64_t)iy * a.npx + ix;
#pragma unroll
  for (int k = 0; k < 4; ++k) out[(uint64_t)k * npix] = st[k];
}

template <bool U, bool M, bool X>
static void launch_image_one(const ImageArgs& a, bool aligned, bool sphere, dim3 grid, int bs, hipStream_t s) {
  // On a uniform grid spheres' registers would let four blocks run per CU;
  // their rays then cross 4 MB of the tally per step on each XCD, all of its L2, and a
  // line is gone before the neighbouring rays reach it.  Half a CU's LDS, not
  // used, keeps it at two blocks: 256^3 disk 2.62 (four), 2.28 (three), 1.94 ms
  // (two), 2.40 (one).  The limit is for the largest grids, whose time it is about:
  // uniform spheres, 8 views of 256^2, with it and without, 256^3 1.97 and 2.44 ms,
  // 192^3 1.03 and 1.11, 160^3 0.76 and 0.73, 128^3 0.57 and 0.52, 64^3 0.29 and 0.23,
  // and with 8 wavelengths 128^3 4.5 and 3.3.
  const size_t lds = sphere && !U && !M && !X && bs == 256 ? size_t(80) << 10 : 0;
  if (sphere) hipLaunchKernelGGL((k_image<false, true, U, M, X>), grid, dim3(bs), lds, s, a);
  else if (aligned) hipLaunchKernelGGL((k_image<true, false, U, M, X>), grid, dim3(bs), 0, s, a);
  else hipLaunchKernelGGL((k_image<false, false, U, M, X>), grid, dim3(bs), 0, s, a);
}

hipError_t launch_image(const ImageArgs& a, bool aligned, bool sphere, bool user_source, bool mesh, hipStream_t s) {
  const uint64_t npix = (uint64_t)a.npx * a.npy, maps = (uint64_t)a.n_views * a.n_lambda;
  const bool multi = image_multi(npix);
  const uint64_t waves = image_waves(npix, maps);
  // few wavefronts go one to a block, so that they spread over the CUs
  const int bs = waves < 1024 ? 64 : 256;
  const uint64_t blocks = (waves * 64 + bs - 1) / bs;
  if (blocks > 0x7fffffffull) return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks);
  auto go = [&](auto x) {
    constexpr bool X = decltype(x)::value;
    if (user_source && mesh) launch_image_one<true, true, X>(a, aligned, sphere, grid, bs, s);
    else if (user_source) launch_image_one<true, false, X>(a, aligned, sphere, grid, bs, s);
    else if (mesh) launch_image_one<false, true, X>(a, aligned, sphere, grid, bs, s);
    else launch_image_one<false, false, X>(a, aligned, sphere, grid, bs, s);
  };
  if (multi) go(std::true_type{});
  else go(std::false_type{});
  return hipGetLastError();
}

}  // namespace kp
