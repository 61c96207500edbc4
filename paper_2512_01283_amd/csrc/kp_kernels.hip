// kp_kernels.hip -- gfx950 kernels of the polarized Monte Carlo transport
// (step 1) of Yang & Wang, arXiv:2512.01283, Sec. 2.2-2.3 and Appendix A (step 2
// is in kp_image.hip).
//
// Step 1 is a persistent packet-per-lane loop: every lane of a 64-wide
// wavefront carries one photon packet and advances it by one cell segment per
// iteration (plus the scattering event that may end the segment); lanes whose
// packet ended are refilled from a global work counter for several of them at a
// time (ids handed out by lane rank), so long and short paths do not idle a
// wavefront.  Packets are independent: each draws from its own Philox stream
// (key (seed, wavelength), counter (packet, block, 0, 0)), so the schedule never
// changes a packet's path.
//
// The scattering-source tally of step 1 is kept as the incident coherency of
// each cell (3x3 Hermitian, 9 reals): because every scatterer here is a
// dipole, the source toward any camera is a fixed linear map of it (formed in
// step 2), so one tally serves all views and wavelengths' views at 9 FP64
// atomics per segment instead of 4 per view (6 when no circular polarisation
// can arise, i.e. for spheres).  Segments are staged in LDS, those of one lane in
// the same cell added up there while its entry is staged (multiple scattering
// inside a thick cell then costs few atomics), and flushed cooperatively by the
// whole wavefront: one atomic instruction carries the contiguous components of
// ~7-10 cells, each cell's block aligned to one cache line (64 B for 6 reals,
// 128 B for 9) -- memory-side FP64 atomics are charged per line request, so this
// is ~5x cheaper than one cell per lane.
#include "kp_transfer.hpp"

namespace kp {

enum : uint32_t {
  EV_SCATTER = 1, END_ESCAPE = 2, EV_RR_SURVIVE = 3, END_RR_KILL = 4, END_BUDGET = 5,
  END_NUMERIC = 6
};

__device__ __forceinline__ uint64_t fnv_u32(uint64_t h, uint32_t v) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    h ^= (v >> (8 * k)) & 0xffu;
    h *= 1099511628211ull;
  }
  return h;
}
__device__ __forceinline__ uint64_t hash_event(uint64_t h, uint32_t kind, uint64_t cell) {
  return fnv_u32(fnv_u32(h, kind), (uint32_t)cell);
}

template <typename R>
struct Packet {
  // Geometry is FP64 in every variant: position inside the cell (cell units),
  // direction and remaining scattering depth.  A packet's path is sensitive
  // to them well beyond their own size -- a scattering depth off by 3e-7
  // moves a scattering point inside a tenuous cell (rho kappa dx ~ 1e-3) by
  // 3e-4 cell, which a later cell of optical depth 1e3 turns into a 0.3 %
  // weight error -- so only the polarisation arithmetic runs in R.
  double fx, fy, fz;
  double nx, ny, nz;
  double rnx, rny, rnz;  // 1 / n per axis (inf for a zero component), set with n
  double tau;
  R I, Q, U, V;       // Stokes vector in the lab basis of n
  R w0;               // initial weight
  R tau_path;         // sum of |continuous extinction exponent| along the path
  double e_abs;
  double ks, ke;      // per-wavelength kappa_sca and kappa_ext times the cell size, held
  R ka;               // in registers (no dependent load per step); ka = kappa_abs dx
  float rho;          // density of the current cell when the grid holds it (loaded on
                      // entering the cell, one step before its use)
  uint32_t last;      // cell of the last step (~0: none)
  int ci, cj, ck;
  int leaf, lvl;      // composite mesh: the leaf block (ci..ck local to it) and its level
  int events, steps, lam;
};

// The part of a packet's state that only scattering, roulette and its start
// and end touch, in LDS (one lane per column, so a wavefront's access to one
// field is conflict-free): kept in registers it costs the step's kernels a
// wave per SIMD.
struct Cold {
  uint64_t pid[64], hash[64];
  double e_scat[64], e_gain[64];
  float u[8][64];     // uniforms of the last two Philox blocks: draw d at u[d & 7]
                      // (23 bits and a half: exact in FP32)
  uint32_t draw[64];  // uniforms consumed
  uint32_t blk[64];   // the newest block in u (~0: none)
  uint32_t trials[64], rr[64];
};
struct ColdRef {
  Cold& c;
  int l;
  __device__ __forceinline__ uint64_t& pid() const { return c.pid[l]; }
  __device__ __forceinline__ uint64_t& hash() const { return c.hash[l]; }
  __device__ __forceinline__ double& e_scat() const { return c.e_scat[l]; }
  __device__ __forceinline__ double& e_gain() const { return c.e_gain[l]; }
  __device__ __forceinline__ uint32_t& draw() const { return c.draw[l]; }
  __device__ __forceinline__ uint32_t& blk() const { return c.blk[l]; }
  __device__ __forceinline__ uint32_t& trials() const { return c.trials[l]; }
  __device__ __forceinline__ uint32_t& rr() const { return c.rr[l]; }
  __device__ __forceinline__ float& u(uint32_t d) const { return c.u[d & 7u][l]; }
};

// block b of the packet's stream, unless it is the newest one already
__device__ __forceinline__ void need_block(const ColdRef& k, uint32_t b, uint64_t seed, int lam) {
  if (b != k.blk()) {
    uint64_t w[4];
    philox4x64_10(k.pid(), (uint64_t)b, 0ull, 0ull, seed, (uint64_t)lam, w);
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) k.u(4 * b + i) = word_uniform<float>(w[i]);
    k.blk() = b;
  }
}

__device__ __forceinline__ float next_uniform(const ColdRef& k, uint64_t seed, int lam) {
  const uint32_t d = k.draw();
  k.draw() = d + 1;
  need_block(k, d >> 2, seed, lam);
  return k.u(d);
}

// The next four uniforms, draws d .. d + 3, in one visit of the generator
// (they lie in at most two blocks, of which the older is in u already); the
// caller consumes three or four of them, so that the blocks held always
// cover the next draw.
__device__ __forceinline__ void next_four(const ColdRef& k, uint32_t d, uint64_t seed, int lam, float u[4]) {
  need_block(k, (d + 3) >> 2, seed, lam);
#pragma unroll
  for (uint32_t i = 0; i < 4; ++i) u[i] = k.u(d + i);
}

// Isotropic direction from two uniforms: mu = 2 u0 - 1, azimuth 2 pi u1.
template <typename R>
__device__ __forceinline__ void isotropic_dir(Packet<R>& p, double u0, double u1) {
  const double mu = 2.0 * u0 - 1.0;
  const double s = sqrt(fmax(0.0, 1.0 - mu * mu));
  double sp, cp;
  sincospi(2.0 * u1, &sp, &cp);
  p.nx = s * cp; p.ny = s * sp; p.nz = mu;
}

// The cell emitting a packet of the dust's thermal emission: the first cell
// whose running luminosity sum exceeds u L.  The guide table brackets it:
// entry k - 1 (or cell 0) from below and entry k + 1 from above, k =
// floor(u ncell), so the search spans only the cells between two guide
// points.
__device__ __forceinline__ uint64_t emission_cell(const double* F, const uint32_t* G, uint64_t ncell,
                                                  double u) {
  const double t = u * F[ncell - 1];
  uint64_t k = (uint64_t)(u * (double)ncell);
  if (k > ncell - 1) k = ncell - 1;
  uint64_t lo = k > 0 ? (uint64_t)G[k - 1] : 0ull, hi = (uint64_t)G[k + 1];
  while (lo < hi) {
    const uint64_t mid = lo + ((hi - lo) >> 1);
    if (t < F[mid]) hi = mid; else lo = mid + 1;
  }
  return lo;
}

// the packet at finest-unit position t in finest cell X: leaf, local cell,
// fractions, and the cell-length constants of the leaf's level
template <typename R>
__device__ __forceinline__ void mesh_place(Packet<R>& p, const TransportArgs& a, const double t[3],
                                           const long long X[3]) {
  const MeshDev& m = a.mesh;
  const int j = mesh_find(m, X);
  const int4 o = reinterpret_cast<const int4*>(m.leaf_org)[j];
  const int sh = m.max_level - o.w;
  const double s = (double)(1ll << sh);
  p.leaf = j;
  p.lvl = o.w;
  const long long i0 = (X[0] - o.x) >> sh, i1 = (X[1] - o.y) >> sh, i2 = (X[2] - o.z) >> sh;
  p.ci = (int)i0; p.cj = (int)i1; p.ck = (int)i2;
  p.fx = fmin(1.0, fmax(0.0, (t[0] - (double)o.x) / s - (double)i0));
  p.fy = fmin(1.0, fmax(0.0, (t[1] - (double)o.y) / s - (double)i1));
  p.fz = fmin(1.0, fmax(0.0, (t[2] - (double)o.z) / s - (double)i2));
  const DustDev& D = a.dust[p.lam];
  const double sc = ldexp(1.0, -o.w);
  p.ks = D.ks_cell * sc;
  p.ke = D.ke_cell * sc;
  p.ka = (R)(D.ka_cell * sc);
}

// after a face crossing moved a local index out of the leaf block: the leaf
// beyond, or true if the packet left the domain
template <typename R>
__device__ bool mesh_cross(Packet<R>& p, const TransportArgs& a) {
  const MeshDev& m = a.mesh;
  const int4 o = reinterpret_cast<const int4*>(m.leaf_org)[p.leaf];
  const double s = (double)(1ll << (m.max_level - o.w));
  const double t[3] = {(double)o.x + ((double)p.ci + p.fx) * s, (double)o.y + ((double)p.cj + p.fy) * s,
                       (double)o.z + ((double)p.ck + p.fz) * s};
  const double n[3] = {p.nx, p.ny, p.nz};
  long long X[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    X[k] = finest_cell(t[k], n[k]);
    if (X[k] < 0 || X[k] >= m.nfine[k]) return true;
  }
  mesh_place(p, a, t, X);
  return false;
}

// flat index of the packet's cell
template <bool MESH, typename R>
__device__ __forceinline__ uint64_t cell_index(const Packet<R>& p, const TransportArgs& a) {
  if (MESH) {
    const uint64_t B = (uint64_t)a.mesh.block;
    return (uint64_t)p.leaf * B * B * B + (uint64_t)p.ci + B * ((uint64_t)p.cj + B * (uint64_t)p.ck);
  }
  return (uint64_t)p.ci + (uint64_t)a.nx * ((uint64_t)p.cj + (uint64_t)a.ny * p.ck);
}

// Emission (Sec. 2.2).  Point sources: isotropic direction (or the pencil
// direction), an unpolarised Stokes vector of weight lum/N, and the cell
// holding the source (a coordinate on a face belongs to the cell the
// direction points into).  Thermal emission of the dust (the alpha_abs B
// term of eq. polarized-rt): the cell drawn by luminosity 4 pi rho kappa_abs
// B V, the position uniform in it, an isotropic direction and the Stokes
// vector w (alpha1, alpha2, 0, 0) in the grain-frame basis of the direction
// (the dichroism of absorption is that of extinction), carried to the lab
// basis; its mean over directions is w.  Draws: cell, three coordinates,
// two for the direction.  Then an exponential scattering depth.  Returns
// false if a point source lies outside the grid.
template <typename R, bool ALIGNED, bool SPHERE, bool MESH>
__device__ bool init_packet(Packet<R>& p, const ColdRef& k, uint64_t g, const TransportArgs& a) {
  int lo = 0, hi = a.n_lambda - 1;
  while (lo < hi) {  // last wavelength whose first index <= g
    int mid = (lo + hi + 1) >> 1;
    if (a.dust[mid].first <= g) lo = mid; else hi = mid - 1;
  }
  p.lam = lo;
  k.pid() = g - a.dust[lo].first;
  k.blk() = 0xffffffffu;
  p.w0 = (R)a.dust[lo].w0;
  p.ks = a.dust[lo].ks_cell;
  p.ke = a.dust[lo].ke_cell;
  p.ka = (R)a.dust[lo].ka_cell;
  p.e_abs = 0.0;
  k.e_scat() = 0.0;
  k.e_gain() = 0.0;
  p.tau_path = (R)0;
  p.events = 0; p.steps = 0;
  k.trials() = 0;
  k.rr() = 0;
  k.hash() = 14695981039346656037ull;
  p.last = 0xffffffffu;
  // the draws of the start: for thermal emission the cell and three
  // coordinates first, then two for the direction and one for the depth
  float ue[4] = {0.f, 0.f, 0.f, 0.f}, us[4];
  uint32_t d0 = 0;
  if (a.src_kind == 2) {
    next_four(k, 0, a.seed, lo, ue);
    d0 = 4;
  }
  next_four(k, d0, a.seed, lo, us);
  k.draw() = d0 + 3;
  const double u0 = (double)us[0], u1 = (double)us[1];
  bool in = true;
  if (a.src_kind == 2) {
    const uint64_t c = emission_cell(a.em_cdf + (uint64_t)lo * a.ncell,
                                     a.em_guide + (uint64_t)lo * (a.ncell + 1), a.ncell,
                                     (double)ue[0]);
    if (MESH) {
      // cell c of the mesh: leaf c / block^3, local cell x fastest; the
      // cell-length constants of the leaf's level
      const uint64_t Bm = (uint64_t)a.mesh.block, r = c % (Bm * Bm * Bm);
      p.leaf = (int)(c / (Bm * Bm * Bm));
      p.ci = (int)(r % Bm);
      p.cj = (int)((r / Bm) % Bm);
      p.ck = (int)(r / (Bm * Bm));
      p.lvl = a.mesh.leaf_org[4 * p.leaf + 3];
      const double sc = ldexp(1.0, -p.lvl);
      p.ks = a.dust[lo].ks_cell * sc;
      p.ke = a.dust[lo].ke_cell * sc;
      p.ka = (R)(a.dust[lo].ka_cell * sc);
    } else {
      p.ci = (int)(c % (uint64_t)a.nx);
      p.cj = (int)((c / (uint64_t)a.nx) % (uint64_t)a.ny);
      p.ck = (int)(c / ((uint64_t)a.nx * (uint64_t)a.ny));
    }
    p.fx = (double)ue[1];
    p.fy = (double)ue[2];
    p.fz = (double)ue[3];
    isotropic_dir(p, u0, u1);
    const double w = a.dust[lo].w0;
    if (SPHERE) {
      p.I = (R)w; p.Q = (R)0; p.U = (R)0; p.V = (R)0;
    } else {
      const V3<double> nd{p.nx, p.ny, p.nz};
      V3<double> ngd = nd;
      double c2 = 1.0, s2 = 0.0;
      if (ALIGNED) {
        const Quat<double> qd = grain_quat(V3<double>{(double)a.bx[c], (double)a.by[c], (double)a.bz[c]});
        ngd = to_grain(qd, nd);
        eta2(qd, nd, ngd, c2, s2);
      }
      double a1, a2, a3;
      alphas<double, SPHERE>(a.dust[lo], ngd.z, a1, a2, a3);
      p.I = (R)(w * a1); p.Q = (R)(c2 * w * a2); p.U = (R)(s2 * w * a2); p.V = (R)0;
    }
    p.rho = a.rho[c];
  } else {
    if (a.src_kind == 1) {
      p.nx = a.dx_; p.ny = a.dy_; p.nz = a.dz_;
    } else {
      isotropic_dir(p, u0, u1);
    }
    p.I = p.w0; p.Q = (R)0; p.U = (R)0; p.V = (R)0;
    const double pos[3] = {a.sx, a.sy, a.sz}, org[3] = {a.x0, a.y0, a.z0};
    const double dir[3] = {p.nx, p.ny, p.nz};
    if (MESH) {
      // the finest cell holding the source (face rule), then its leaf
      double t[3];
      long long X[3];
      in = true;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        t[k] = (pos[k] - org[k]) / a.mesh.fine;
        X[k] = finest_cell(t[k], dir[k]);
        in = in && X[k] >= 0 && X[k] < a.mesh.nfine[k];
      }
      if (in) mesh_place(p, a, t, X);
      p.rho = in ? a.rho[cell_index<true>(p, a)] : 0.f;
      p.rnx = 1.0 / p.nx; p.rny = 1.0 / p.ny; p.rnz = 1.0 / p.nz;
      p.tau = -log((double)us[2]);
      return in;
    }
    int ci[3];
    double fr[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      double t = (pos[k] - org[k]) / a.dx;
      double fl = floor(t);
      double f = t - fl;
      int i = (int)fl;
      if (f == 0.0 && dir[k] < 0.0) { i -= 1; f = 1.0; }
      ci[k] = i;
      fr[k] = f;
    }
    const int nn[3] = {a.nx, a.ny, a.nz};
#pragma unroll
    for (int k = 0; k < 3; ++k)  // a periodic axis holds every coordinate
      if ((a.boundary >> k) & 1) ci[k] = ((ci[k] % nn[k]) + nn[k]) % nn[k];
    p.ci = ci[0]; p.cj = ci[1]; p.ck = ci[2];
    p.fx = fr[0]; p.fy = fr[1]; p.fz = fr[2];
    in = p.ci >= 0 && p.ci < a.nx && p.cj >= 0 && p.cj < a.ny && p.ck >= 0 && p.ck < a.nz;
    p.rho = in ? a.rho[(uint64_t)p.ci + (uint64_t)a.nx * ((uint64_t)p.cj + (uint64_t)a.ny * p.ck)] : 0.f;
  }
  p.rnx = 1.0 / p.nx; p.rny = 1.0 / p.ny; p.rnz = 1.0 / p.nz;
  p.tau = -log((double)us[2]);
  return in;
}

// Coherency contribution of a segment-integrated Stokes vector J (lab basis of
// n): sum_ab rho_ab e_a e_b^T with rho = 1/2 [[I+Q, U-iV],[U+iV, I-Q]],
// e1 = theta_hat(n), e2 = phi_hat(n), times the weight w.  Output order: real
// xx yy zz xy xz yz, imaginary yz zx xy (the antisymmetric part equals
// -V/2 [n]_x in this basis).
// With e1 = (nz cos p, nz sin p, -sin t), e2 = (-sin p, cos p, 0) every
// product of two basis components is written with cos^2 p, sin^2 p,
// cos p sin p (from n by one reciprocal of nx^2 + ny^2) and sin t cos p = nx,
// sin t sin p = ny: no square root per step.  At the pole (phi = 0) cos p = 1
// and sin t = sqrt(nx^2 + ny^2).  Jp, Jm: J_I + J_Q and J_I - J_Q.  Every sum of
// two products is written as one product and one fused multiply-add, so that
// a kernel's FP32 results do not depend on which of the two the compiler fuses
// in the code around it.
template <typename R, int NC>
__device__ __forceinline__ void coherency(const V3<R>& n, R Jp, R Jm, R JU, R JV, R w,
                                          R out[NC]) {
#pragma clang fp contract(off)
  const R r2 = k_fma(n.y, n.y, n.x * n.x);
  R px, py, cc, ss, cs;  // sin t cos p, sin t sin p, cos^2 p, sin^2 p, cos p sin p
  if (r2 <= (R)KP_POLE2) {
    px = k_sqrt(r2); py = (R)0; cc = (R)1; ss = (R)0; cs = (R)0;
  } else {
    const R ir = (R)1 / r2;
    px = n.x; py = n.y; cc = n.x * n.x * ir; ss = n.y * n.y * ir; cs = n.x * n.y * ir;
  }
  const R a = (R)0.5 * Jp * w, b = (R)0.5 * Jm * w, u = (R)0.5 * JU * w;
  const R v = (R)-0.5 * JV * w;
  const R an = a * n.z, an2 = an * n.z, un = u * n.z, un2 = un + un;
  out[0] = k_fma(-un2, cs, k_fma(b, ss, an2 * cc));
  out[1] = k_fma(un2, cs, k_fma(an2, ss, b * cc));
  out[2] = a * r2;
  out[3] = k_fma(k_fma(an, n.z, -b), cs, un * (cc - ss));
  out[4] = k_fma(u, py, -an * px);
  out[5] = k_fma(-an, py, -(u * px));
  if (NC > 6) {
    out[NC > 6 ? 6 : 0] = v * n.x;
    out[NC > 7 ? 7 : 0] = v * n.y;
    out[NC > 8 ? 8 : 0] = v * n.z;
  }
}

// The grain-frame quaternion of a cell: from its tally block, or formed from
// the alignment direction when the block does not hold it.
template <bool ALIGNED, bool SPHERE>
__device__ __forceinline__ Quat<double> cell_quat(const TransportArgs& a, const double* blk, uint64_t c) {
  using TSh = TallyShape<SPHERE>;
  if (TSh::HAS_B) return Quat<double>{blk[TSh::QUAT], blk[TSh::QUAT + 1], blk[TSh::QUAT + 2], blk[TSh::QUAT + 3]};
  return grain_quat(V3<double>{(double)a.bx[c], (double)a.by[c], (double)a.bz[c]});
}

template <typename R>
__device__ __forceinline__ Quat<R> quat_cast(const Quat<double>& q) {
  return Quat<R>{(R)q.w, (R)q.x, (R)q.y, (R)q.z};
}

// Tally flush, wave-cooperative and deferred.  A lane's tallied segment is
// staged as (key, NC values) in its wavefront's LDS area (wave_stage), or,
// when it lies in the cell of the lane's last entry and that is still there,
// added to it (a drain forgets the entries: a lane that stays in a cell across one
// adds a second line, 1 % more lines on the disk and up to 2.3 times as many in a
// scattering sphere of depth 100, for the 12-18 registers a sum of its own takes);
// when the area may not hold another full wavefront of entries, wave_drain
// adds all staged entries to the tally: lane L adds component L % NC of entry
// L / NC, so one atomic instruction covers 64 / NC whole cells.  Deferring
// matters on gfx9: atomics without return still count in vmcnt, and the next
// density load's wait (vmcnt(0)) would otherwise wait every iteration for the
// last flush's read-modify-writes to reach memory; drained every few
// iterations, that latency is exposed once per drain.  Both must be reached by
// all lanes of the wavefront; `staged` is the same in every lane.
template <int NC>
__device__ __forceinline__ int wave_stage_new(bool need, int64_t key, const double acc[NC], double* sv, long long* sk,
                                              int lane, int& staged, int& slot) {
  const unsigned long long mask = __ballot(need);
  if (mask == 0ull) return 0;
  if (need) {
    slot = staged + __popcll(mask & ((1ull << lane) - 1ull));
#pragma unroll
    for (int k = 0; k < NC; ++k) sv[slot * NC + k] = acc[k];
    sk[slot] = key;
  }
  const int n = __popcll(mask);
  staged += n;
  return n;
}
template <int NC, typename R>
__device__ __forceinline__ int wave_stage(bool has, int64_t key, const R cc[NC], double* sv, long long* sk, int lane,
                                          int& staged, int64_t& last_key, int& slot) {
  const bool same = has && slot >= 0 && key == last_key;
  if (same) {
#pragma unroll
    for (int k = 0; k < NC; ++k) sv[slot * NC + k] += (double)cc[k];
  }
  double v[NC];
#pragma unroll
  for (int k = 0; k < NC; ++k) v[k] = (double)cc[k];
  if (has) last_key = key;
  return wave_stage_new<NC>(has && !same, key, v, sv, sk, lane, staged, slot);
}

template <int NC, int TS>
__device__ __forceinline__ void wave_drain(double* tally, double* sv, long long* sk, int lane, int& staged) {
  const int n = staged;
  if (n == 0) return;
  staged = 0;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  constexpr int G = 64 / NC;
  constexpr int U = 4;  // rounds whose LDS reads are issued before one wait
  const int slot = lane / NC, k = lane - slot * NC;
  if (slot < G) {
    for (int base = 0; base < n; base += U * G) {
      double v[U];
      long long key_r[U];
      // reads of entries beyond n stay inside the staged entries (index
      // clamped to n - 1) and their atomics are masked below
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = min(base + u * G + slot, n - 1);
        v[u] = sv[e * NC + k];
        key_r[u] = sk[e];
      }
      // keep every key read ahead of the branches below (one LDS wait
      // for all of them instead of one per round)
#pragma unroll
      for (int u = 0; u < U; ++u) asm volatile("" : : "v"(key_r[u]));
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (base + u * G + slot < n && v[u] != 0.0)
          unsafeAtomicAdd(tally + (uint64_t)key_r[u] * TS + k, v[u]);
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The same for the packets of a pencil beam, which all cross the same cells, those
// that started together at the same time: each group of NC lanes takes a run
// of consecutive entries and adds those of one cell up before they go to memory.
// The beam's lines are otherwise what bounds such a run, the more so the more
// wavefronts contend for them: 64-cell column, 3e5 packets, 5.4, 6.3 and 7.2 ms
// with one, two and three blocks per CU, so 0.85 ms; a beam across a 64^3 sphere of
// depth 1, where most entries are scattered light's, 5.8 -> 3.5, of depth 20 21.6.
// Returns the blocks added.
template <int NC, int TS>
__device__ __forceinline__ int wave_drain_runs(double* tally, const double* sv, const long long* sk, int lane,
                                               int& staged) {
  const int n = staged;
  if (n == 0) return 0;
  staged = 0;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  constexpr int G = 64 / NC;
  constexpr int U = 4;  // entries whose LDS reads are issued before one wait
  const int slot = lane / NC, k = lane - slot * NC, per = (n + G - 1) / G;
  const int end = slot < G ? min(n, (slot + 1) * per) : 0;
  int blocks = 0;
  long long cur = -1;
  double sum = 0.0;
  for (int i = 0; i < per; i += U) {
    double v[U];
    long long key[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = min(slot * per + i + u, n - 1);
      v[u] = sv[e * NC + (slot < G ? k : 0)];
      key[u] = sk[e];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool have = i + u < per && slot * per + i + u < end;
      const bool out = have && key[u] != cur && cur >= 0;
      blocks += __popcll(__ballot(out && k == 0));
      if (out && sum != 0.0) unsafeAtomicAdd(tally + (uint64_t)cur * TS + k, sum);
      if (have) {
        sum = key[u] == cur ? sum + v[u] : v[u];
        cur = key[u];
      }
    }
  }
  blocks += __popcll(__ballot(cur >= 0 && k == 0));
  if (cur >= 0 && sum != 0.0) unsafeAtomicAdd(tally + (uint64_t)cur * TS + k, sum);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  return blocks;
}

// Spherical grains' scattering in real arithmetic: the Jones matrix J_ij =
// f_i . e_j of a proposal (e_i the bases of the incident direction, f_i of the
// proposed one), the intensity it scatters from the incident coherency
// (r11, r22, r12) divided by pf, and the scattered state.  Circular polarisation does
// not arise (reals only).  As in coherency(), every rounding is written out.
template <typename R>
struct SphereJones {
  R J11, J12, J21, J22;
  __device__ __forceinline__ R set(R mu, R smu, R cph, R sph, R cpn, R spn, R stn, R nz, R r11, R r22, R r12) {
#pragma clang fp contract(off)
    const R e1x = nz * cpn, e1y = nz * spn;
    const R f1x = mu * cph, f1y = mu * sph;
    J11 = k_fma(stn, smu, k_fma(e1x, f1x, e1y * f1y));
    J12 = k_fma(cpn, f1y, -(spn * f1x));
    J21 = k_fma(e1y, cph, -(e1x * sph));
    J22 = k_fma(cpn, cph, spn * sph);
    const R C = k_fma(J21, J22, J11 * J12);
    const R A = k_fma(J21, J21, J11 * J11), B = k_fma(J22, J22, J12 * J12);
    return k_fma(r12, C + C, k_fma(r11, A, r22 * B));
  }
  // (I, Q, U) scattered, times pf, from the incident coherency
  __device__ __forceinline__ void state(R pf, R r11, R r22, R r12, R& So, R& Qo, R& Uo) const {
#pragma clang fp contract(off)
    const R T11 = k_fma(r11, J11, r12 * J12), T12 = k_fma(r22, J12, r12 * J11);
    const R T21 = k_fma(r11, J21, r12 * J22), T22 = k_fma(r22, J22, r12 * J21);
    const R p11 = J11 * T11 + J12 * T12, p22 = J21 * T21 + J22 * T22;
    const R p12 = J21 * T11 + J22 * T12;
    So = (p22 + p11) * pf;
    Qo = (p11 - p22) * pf;
    Uo = (pf + pf) * p12;
  }
};

// Scattering event (Sec. 2.2; rejection sampling of Sec. 3): incident state
// carried into the grain frame, proposals uniform on the sphere there
// (cos, azimuth, acceptance: three uniforms per trial), accepted when
// u * bound <= [P s]_I, output rescaled to the scattered power, then carried
// back to the lab frame.  Returns false on a numerical failure.
template <typename R, bool ALIGNED, bool SPHERE>
__device__ bool scatter(Packet<R>& p, const ColdRef& k, const Quat<R>& q, const Quat<double>& qd,
                        const DustDev& D, uint64_t seed, float& u_tau) {
  const V3<R> n{(R)p.nx, (R)p.ny, (R)p.nz};
  V3<R> ng = n;
  R c2 = (R)1, s2 = (R)0;
  R cpn, spn, stn;
  if (ALIGNED) {
    // The grain-frame direction and its azimuth are formed in FP64: for a
    // packet moving nearly along the grain axis the transverse components
    // are small differences of order-one terms, which FP32 resolves only to
    // ~1e-7 absolute, i.e. to a basis angle error of ~1e-7 / sin(theta').
    const V3<double> nd{p.nx, p.ny, p.nz};
    const V3<double> ngd = to_grain(qd, nd);
    double cpd, spd, std_;
    azimuth(ngd, cpd, spd, std_);
    ng = V3<R>{(R)ngd.x, (R)ngd.y, (R)ngd.z};
    cpn = (R)cpd;
    spn = (R)spd;
    stn = (R)std_;
    eta2(q, n, ng, c2, s2);
  } else {
    azimuth(ng, cpn, spn, stn);
  }
  const R I = p.I, V = p.V;
  const R Qg = ALIGNED ? c2 * p.Q + s2 * p.U : p.Q, Ug = ALIGNED ? -s2 * p.Q + c2 * p.U : p.U;
  V3<R> e1, e2;
  e1 = {ng.z * cpn, ng.z * spn, -stn};
  e2 = {-spn, cpn, (R)0};
  const R r11 = (R)0.5 * (I + Qg), r22 = (R)0.5 * (I - Qg);
  const Cx<R> r12{(R)0.5 * Ug, (R)-0.5 * V};
  const R pf = (R)D.pfac;
  const R bound = (R)D.bound_fac * I;
  const R tol = sizeof(R) == 4 ? (R)1e-4 : (R)1e-12;
  const Cx<R> ap{(R)D.ap_re, (R)D.ap_im};
  const Cx<R> dd{(R)(D.aa_re - D.ap_re), (R)(D.aa_im - D.ap_im)};
  Cx<R> J11, J12, J21, J22;
  SphereJones<R> js;
  R mu = 0, smu = 0, cph = 1, sph = 0, Iout = 0, umu = 0, uph = 0;
  bool ok = false;
  uint32_t d = k.draw();
  int trial = 0;
  for (; trial < 100000; ++trial) {
    float u[4];  // a trial's three, and the depth's once it is accepted
    next_four(k, d, seed, p.lam, u);
    d += 3;
    umu = (R)u[0];
    mu = (R)2 * umu - (R)1;
    uph = (R)u[1];
    R ua = (R)u[2];
    u_tau = u[3];
    // 1 - mu^2 as (1 - mu)(1 + mu): both factors are exact, so sin theta'
    // keeps full relative precision near the grain axis in FP32
    smu = sizeof(R) == 4 ? k_sqrt(fmax((R)0, ((R)1 - mu) * ((R)1 + mu))) : k_sqrt(fmax((R)0, (R)1 - mu * mu));
    k_sincospi((R)2 * uph, &sph, &cph);
    if (smu * smu <= (R)KP_POLE2) { cph = (R)1; sph = (R)0; }
    if (SPHERE) {
      Iout = js.set(mu, smu, cph, sph, cpn, spn, stn, ng.z, r11, r22, r12.re) * pf;
    } else {
      const V3<R> f1{mu * cph, mu * sph, -smu}, f2{-sph, cph, (R)0};
      const R D11 = dot(f1, e1), D12 = dot(f1, e2), D21 = dot(f2, e1), D22 = dot(f2, e2);
      J11 = cadd(cscale(ap, D11), cscale(dd, smu * stn));
      J12 = cscale(ap, D12);
      J21 = cscale(ap, D21);
      J22 = cscale(ap, D22);
      Iout = pf * (cabs2(J11) * r11 + cabs2(J12) * r22 + (R)2 * cmulc(cmul(J11, r12), J12).re +
                   cabs2(J21) * r11 + cabs2(J22) * r22 + (R)2 * cmulc(cmul(J21, r12), J22).re);
    }
    if (!(Iout <= bound * ((R)1 + tol))) { ++trial; break; }
    if (ua * bound <= Iout) { ok = true; break; }
  }
  k.trials() += (uint32_t)trial + (ok ? 1u : 0u);
  if (!ok) return false;
  k.draw() = d + 1;
  // full scattered state rho' = J rho J^dagger in the natural basis of mg
  R So, Qo, Uo, Vo = (R)0;
  if (SPHERE) {
    js.state(pf, r11, r22, r12.re, So, Qo, Uo);
  } else {
    const Cx<R> r21{r12.re, -r12.im};
    const Cx<R> T11 = cadd(cscale(J11, r11), cmul(J12, r21));
    const Cx<R> T12 = cadd(cmul(J11, r12), cscale(J12, r22));
    const Cx<R> T21 = cadd(cscale(J21, r11), cmul(J22, r21));
    const Cx<R> T22 = cadd(cmul(J21, r12), cscale(J22, r22));
    const R p11 = cmulc(T11, J11).re + cmulc(T12, J12).re;
    const R p22 = cmulc(T21, J21).re + cmulc(T22, J22).re;
    const Cx<R> p12 = cadd(cmulc(T11, J21), cmulc(T12, J22));
    So = pf * (p11 + p22);
    Qo = pf * (p11 - p22);
    Uo = pf * (R)2 * p12.re;
    Vo = pf * (R)-2 * p12.im;
  }
  // scattered power: sum_k |a_k|^2 C_kk / N_P with C_zz = r11 sin^2(theta'_n)
  R sig = I;
  if (!SPHERE) {
    R czz = r11 * stn * stn;
    sig = (R)D.ap2_np * (I - czz) + (R)D.aa2_np * czz;
  }
  R scale = sig / So;
  So = sig; Qo *= scale; Uo *= scale; Vo *= scale;
  if (sizeof(R) == 4) {
    // In FP32 the scattered state of a direction of near-zero scattered
    // intensity is a difference of terms of size I, so rounding can leave it
    // outside |P| <= I (one packet of 1.5e8 on a 256^3 disk: |P| = 1.0008 I,
    // after which the next event's bound check fails); it is projected back
    // onto the cone.
    const R p2 = k_fma(Vo, Vo, k_fma(Qo, Qo, Uo * Uo));
    if (p2 > So * So) {
      const R f = So / k_sqrt(p2);
      Qo *= f; Uo *= f; Vo *= f;
    }
  }
  // the accepted direction itself is formed in FP64 from the same uniforms
  const double mud = 2.0 * (double)umu - 1.0;
  const double smud = sqrt(fmax(0.0, 1.0 - mud * mud));
  double sphd, cphd;
  sincospi(2.0 * (double)uph, &sphd, &cphd);
  if (smud * smud <= KP_POLE2) { cphd = 1.0; sphd = 0.0; }
  const V3<double> mgd{smud * cphd, smud * sphd, mud};
  V3<double> md = mgd;
  R cm = (R)1, sm = (R)0;
  if (ALIGNED) {
    md = from_grain(qd, mgd);
    eta2(q, V3<R>{(R)md.x, (R)md.y, (R)md.z}, V3<R>{(R)mgd.x, (R)mgd.y, (R)mgd.z}, cm, sm);
  }
  p.nx = md.x; p.ny = md.y; p.nz = md.z;
  p.rnx = 1.0 / p.nx; p.rny = 1.0 / p.ny; p.rnz = 1.0 / p.nz;
  k.e_scat() += (double)(sig - I);
  p.I = So;
  p.Q = cm * Qo - sm * Uo;
  p.U = sm * Qo + cm * Uo;
  p.V = Vo;
  return true;
}

// ---------------------------------------------------------------------------
// Tabulated scattering (Sec. 2.2: optical properties given as interpolation
// tables).  The table holds the scattering-plane elements S11 S12 S22 S33
// S34 S44 of randomly oriented grains, normalised so that S11 integrates to 1
// over solid angle, at scattering angles uniform on [0, pi]; values are linear
// in cos Theta between nodes.  FP64 throughout.
// ---------------------------------------------------------------------------
// The nodes come from the device arrays of a wavelength (the node interval by
// the guide's entry for the cos Theta bin) or from a block's copy in LDS (by the
// FP32 inverse cosine: no read on the dependency chain); either is then moved
// to the interval holding mu.
struct TabNodes {
  const double* Z;       // [n][6]
  const double* M;       // [n]
  const int32_t* guide;  // [G] (device arrays)
  int n, G;
};
__device__ __forceinline__ TabNodes tab_nodes(const DustDev& D) {
  return TabNodes{D.tab, D.tab_mu, D.tab_guide, D.tab_n, D.tab_g};
}
template <bool LDS>
__device__ __forceinline__ void tab_eval(const TabNodes& T, double mu, double z[6]) {
  const int n = T.n;
  mu = fmin(1.0, fmax(-1.0, mu));
  int j;
  if (LDS) {
    j = (int)(acosf((float)mu) * ((float)(n - 1) * 0.31830988618f));
    j = j < 0 ? 0 : (j > n - 2 ? n - 2 : j);
  } else {
    int b = (int)((1.0 - mu) * (0.5 * (double)T.G));
    b = b < 0 ? 0 : (b > T.G - 1 ? T.G - 1 : b);
    j = T.guide[b];
  }
  const double* M = T.M;
  while (j < n - 2 && mu < M[j + 1]) ++j;
  while (j > 0 && mu > M[j]) --j;
  const double ma = M[j], mb = M[j + 1];
  const double t = ma > mb ? (ma - mu) / (ma - mb) : 0.0;
  const double* Z = T.Z + 6 * j;
#pragma unroll
  for (int k = 0; k < 6; ++k) z[k] = (1.0 - t) * Z[k] + t * Z[6 + k];
}

// P(m; n) s per unit solid angle: s in the lab basis of n, the result in the
// basis (tm, pm) of m.  The scattering plane's normal is e = n x m / |n x m|
// (phi_hat of n when m = +-n); with a = m . theta_hat_n, b = m . phi_hat_n
// (|n x m|^2 = a^2 + b^2) the rotation into the plane basis (e x n, e) is
// cos 2psi = (a^2 - b^2) / |n x m|^2, sin 2psi = 2ab / |n x m|^2, and the
// rotation out of (e x m, e) into (tm, pm) is by -chi with
// cos 2chi = ((n.tm)^2 - (n.pm)^2) / |n x m|^2, sin 2chi = 2 (n.tm)(n.pm) /
// |n x m|^2: no square root or angle is formed.
template <bool LDS>
__device__ __forceinline__ void tab_toward(const TabNodes& T, const V3<double>& n, const double s[4],
                                           const V3<double>& m, const V3<double>& tm,
                                           const V3<double>& pm, double out[4]) {
  const double ct = dot(n, tm), cp = dot(n, pm);
  const double w2 = ct * ct + cp * cp, r2 = n.x * n.x + n.y * n.y;
  double c2p = 1.0, s2p = 0.0, c2c, s2c;
  if (w2 > 1e-24 && r2 > KP_POLE2) {
    // a and b times sin theta of n, so that n's basis is not needed
    const double a = n.z * (m.x * n.x + m.y * n.y) - r2 * m.z, b = m.y * n.x - m.x * n.y;
    const double iq = 1.0 / (r2 * w2), iw = r2 * iq;
    c2p = (a * a - b * b) * iq;
    s2p = 2.0 * a * b * iq;
    c2c = (ct * ct - cp * cp) * iw;
    s2c = 2.0 * ct * cp * iw;
  } else {
    V3<double> thn, phn;
    basis(n, thn, phn);
    const double a = dot(m, thn), b = dot(m, phn);
    const double v2 = a * a + b * b;
    if (v2 > 1e-24) {
      const double iw = 1.0 / v2;
      c2p = (a * a - b * b) * iw;
      s2p = 2.0 * a * b * iw;
      c2c = (ct * ct - cp * cp) * iw;
      s2c = 2.0 * ct * cp * iw;
    } else {
      const double cc = dot(phn, pm), ss = -dot(phn, tm);
      c2c = cc * cc - ss * ss;
      s2c = 2.0 * cc * ss;
    }
  }
  const double Qp = c2p * s[1] + s2p * s[2], Up = -s2p * s[1] + c2p * s[2];
  double z[6];
  tab_eval<LDS>(T, dot(n, m), z);
  const double I = z[0] * s[0] + z[1] * Qp, Q = z[1] * s[0] + z[2] * Qp;
  const double U = z[3] * Up + z[4] * s[3], V = -z[4] * Up + z[5] * s[3];
  out[0] = I;
  out[1] = c2c * Q - s2c * U;
  out[2] = s2c * Q + c2c * U;
  out[3] = V;
}

// Scattering event of tabulated grains: envelope rejection.  Per trial four
// uniforms: the node interval by the envelope's cumulative mass (the larger
// S11 of its two nodes times the interval's width in cos Theta), cos Theta
// uniform inside it, the azimuth, and acceptance of u * max S11 (I + |P_lin|)
// <= the scattered I.  The total scattered power does not depend on the
// polarisation, so the scattered state is rescaled to the incident I.
template <typename R>
__device__ bool scatter_tab(Packet<R>& p, const ColdRef& k, const DustDev& D, uint64_t seed, float& u_tau) {
  const V3<double> n{p.nx, p.ny, p.nz};
  V3<double> th, ph;
  basis(n, th, ph);
  const double s[4] = {(double)p.I, (double)p.Q, (double)p.U, (double)p.V};
  const double plin = sqrt(s[1] * s[1] + s[2] * s[2]);
  const int nt = D.tab_n;
  const double* cum = D.tab_cum;
  const double total = cum[nt - 1];
  for (int trial = 0; trial < 100000; ++trial) {
    float u[4];
    next_four(k, k.draw(), seed, p.lam, u);
    k.draw() += 4;
    k.trials()++;
    const double u1 = (double)u[0], u2 = (double)u[1], u3 = (double)u[2], u4 = (double)u[3];
    // the first interval whose cumulative envelope mass exceeds u1 * total
    const double target = u1 * total;
    int lo = 0, hi = nt - 2;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (cum[mid + 1] > target) hi = mid;
      else lo = mid + 1;
    }
    const int j = lo;
    const double ma = D.tab_mu[j], mb = D.tab_mu[j + 1];
    const double mu = ma + u2 * (mb - ma);
    double sp, cp;
    sincospi(2.0 * u3, &sp, &cp);
    const double st = sqrt(fmax(0.0, 1.0 - mu * mu));
    V3<double> m{mu * n.x + st * (cp * th.x + sp * ph.x), mu * n.y + st * (cp * th.y + sp * ph.y),
                 mu * n.z + st * (cp * th.z + sp * ph.z)};
    const double inm = 1.0 / sqrt(dot(m, m));
    m = V3<double>{m.x * inm, m.y * inm, m.z * inm};
    V3<double> tm, pm;
    basis(m, tm, pm);
    double o[4];
    tab_toward<false>(tab_nodes(D), n, s, m, tm, pm, o);
    const double env = fmax(D.tab[6 * j], D.tab[6 * (j + 1)]) * (s[0] + plin);
    if (!(o[0] <= env * (1.0 + 1e-9))) return false;
    if (u4 * env <= o[0]) {
      const double scale = s[0] / o[0];
      p.nx = m.x; p.ny = m.y; p.nz = m.z;
      p.rnx = 1.0 / p.nx; p.rny = 1.0 / p.ny; p.rnz = 1.0 / p.nz;
      const R Io = (R)(o[0] * scale);
      k.e_scat() += (double)(Io - p.I);
      p.I = Io;
      p.Q = (R)(o[1] * scale);
      p.U = (R)(o[2] * scale);
      p.V = (R)(o[3] * scale);
      u_tau = next_uniform(k, seed, p.lam);
      return true;
    }
  }
  return false;
}

constexpr int TAB_LVL_SHIFT = 47, TAB_LAM_SHIFT = 52;
constexpr int TAB_CAP = 96;  // staged entries per wavefront (tabulated grains)

// e^-x and (1 - e^-x) / x
__device__ __forceinline__ void cell_exp(double x, double& E, double& P) { exp_phi(x, E, P); }
__device__ __forceinline__ void cell_exp(float x, float& E, float& P) {
  E = k_exp(-x);
  P = phi1(x);
}

// One loop iteration: one cell segment (Sec. 2.2: cell-to-cell traversal,
// exponential scattering depth, continuous extinction across the segment by
// the analytic cell solution of Appendix A, tally of the segment into the
// scattering source of Sec. 2.3), then a scattering event or the crossing
// into the next cell (Russian roulette follows in the caller).  Returns 0 or
// an end kind.
template <typename R, bool ALIGNED, bool SPHERE, bool TAB, bool MESH>
__device__ uint32_t step(Packet<R>& p, const ColdRef& kc, const TransportArgs& a, uint64_t hot_base,
                         bool& has, int64_t& key, R cc[TallyShape<SPHERE>::NC], bool& pending) {
  constexpr int NC = TallyShape<SPHERE>::NC;
  static_assert(!TAB || (SPHERE && !ALIGNED), "tabulated grains have scalar extinction");
  const uint64_t c = cell_index<MESH>(p, a);
  const int ci0 = p.ci, cj0 = p.cj, ck0 = p.ck, lvl0 = MESH ? p.lvl : 0;
  p.last = (uint32_t)c;
  if (p.events >= a.max_events || p.steps >= KP_MAX_STEPS) {
    kc.hash() = hash_event(kc.hash(), END_BUDGET, c);
    return END_BUDGET;
  }
  // the cell's grain frame, asked for before the geometry that does not need it
  const double rhod = (double)p.rho;
  const uint64_t sl = tally_slot(c, p.ci, p.cj, p.ck, MESH ? 0 : a.tbx, a.tby);
  Quat<double> qd{1.0, 0.0, 0.0, 0.0};
  if (ALIGNED && !SPHERE && rhod > 0.0)
    qd = cell_quat<ALIGNED, SPHERE>(a, a.tally + ((uint64_t)p.lam * a.nslot + sl) * TallyShape<SPHERE>::TS, c);
  const double inf = __builtin_huge_val();
  const double dnx = p.nx, dny = p.ny, dnz = p.nz;
  // distances to the exit faces (reciprocals of n formed when n changes)
  double tx = dnx > 0.0 ? (1.0 - p.fx) * p.rnx : (dnx < 0.0 ? -p.fx * p.rnx : inf);
  double ty = dny > 0.0 ? (1.0 - p.fy) * p.rny : (dny < 0.0 ? -p.fy * p.rny : inf);
  double tz = dnz > 0.0 ? (1.0 - p.fz) * p.rnz : (dnz < 0.0 ? -p.fz * p.rnz : inf);
  double td = tx;
  int axis = 0;
  if (ty < td) { td = ty; axis = 1; }
  if (tz < td) { td = tz; axis = 2; }
  if (!(td < inf)) return END_NUMERIC;
  const DustDev& D = a.dust[p.lam];
  const double kbd = rhod * p.ks;
  double tld;
  bool scat;
  if (kbd > 0.0 && p.tau < kbd * td) { tld = p.tau / kbd; scat = true; }
  else { tld = td; p.tau -= kbd * td; scat = false; }
  const R rho = (R)rhod, kb = (R)kbd, tl = (R)tld;
  p.steps++;
  if (rho > (R)0 && tl > (R)0) {
    const V3<R> n{(R)p.nx, (R)p.ny, (R)p.nz};
    const R Ib = p.I;
    R JI, JQ, JU, JV, Jp, Jm;  // Jp, Jm: J_I + J_Q, J_I - J_Q
    if (SPHERE && !ALIGNED) {
      // spheres: extinction is the scalar absorption e^{-rho kappa_abs l}
      const R m1 = rho * p.ka;
      const R E = k_exp(-m1 * tl), G = tl * phi1(m1 * tl);
      p.tau_path += m1 * tl;
      JI = p.I * G; JQ = p.Q * G; JU = p.U * G; JV = p.V * G;
      Jp = k_fma(p.I, G, JQ);
      Jm = k_fma(p.I, G, -JQ);
      p.I *= E; p.Q *= E; p.U *= E; p.V *= E;
    } else {
      // The exponents are differences of two cell-scale optical depths
      // (rho kappa_ext alpha vs rho kappa_sca, each up to ~1e3 per cell), so
      // the grain-frame direction, the alphas and the exponents are formed in
      // FP64; the exponentials and the Stokes arithmetic run in R.
      const V3<double> nd{p.nx, p.ny, p.nz};
      double ctd = nd.z, c2d = 1.0, s2d = 0.0;
      if (ALIGNED) {
        const V3<double> b = grain_axis(qd);
        ctd = dot(b, nd);
        eta2_axis(b, nd, c2d, s2d);
      }
      const R c2 = (R)c2d, s2 = (R)s2d;
      double a1, a2, a3;
      alphas<double, SPHERE>(D, ctd, a1, a2, a3);
      const double ked = rhod * p.ke;
      const double xAd = (ked * (a1 + a2) - kbd) * tld, xBd = (ked * (a1 - a2) - kbd) * tld;
      const double xUd = (ked * a1 - kbd) * tld, yd = ked * a3 * tld;
      const R xA = (R)xAd, xB = (R)xBd, xU = (R)xUd;
      p.tau_path += (R)fabs(xUd);
      const R Qg = c2 * p.Q + s2 * p.U, Ug = -s2 * p.Q + c2 * p.U;
      const R A = p.I + Qg, B = p.I - Qg;
      R gA, gB, eA, eB;
      cell_exp(xA, eA, gA);
      cell_exp(xB, eB, gB);
      gA *= tl;
      gB *= tl;
      R JUg, JVg, Un, Vn;
      if (yd == 0.0) {
        R gU, eU;
        cell_exp(xU, eU, gU);
        gU *= tl;
        JUg = Ug * gU; JVg = p.V * gU;
        Un = Ug * eU; Vn = p.V * eU;
      } else {
        // U + iV evolves as exp((-mU + i w) s)
        Cx<R> ez, phic;
        cx_exp_phi(-xU, (R)yd, ez, phic);
        const Cx<R> Z{Ug, p.V};
        const Cx<R> JZ = cscale(cmul(Z, phic), tl), Zn = cmul(Z, ez);
        JUg = JZ.re; JVg = JZ.im; Un = Zn.re; Vn = Zn.im;
      }
      const R JA = A * gA, JB = B * gB, An = A * eA, Bn = B * eB;
      const R JQg = (R)0.5 * (JA - JB), Qn = (R)0.5 * (An - Bn);
      JI = (R)0.5 * (JA + JB);
      JQ = c2 * JQg - s2 * JUg;
      JU = s2 * JQg + c2 * JUg;
      JV = JVg;
      Jp = JI + JQ;
      Jm = JI - JQ;
      p.I = (R)0.5 * (An + Bn);
      p.Q = c2 * Qn - s2 * Un;
      p.U = s2 * Qn + c2 * Un;
      p.V = Vn;
    }
    p.e_abs += (double)(Ib - p.I);
    if (kb > (R)0) {
      if (TAB) {
        // tabulated grains: the segment's Stokes integral itself (in the lab
        // basis of n), projected on every camera when it is flushed
        cc[0] = JI * kb; cc[1] = JQ * kb; cc[2] = JU * kb; cc[3] = JV * kb;
      } else {
        coherency<R, NC>(n, Jp, Jm, JU, JV, kb, cc);
      }
      uint64_t slot = (uint64_t)p.lam * a.nslot + sl;
      if (!MESH) {
        // a cell of the box around the source: this wavefront's copy of it
        const uint32_t hx = hot_index(ci0, a.hot_x), hy = hot_index(cj0, a.hot_y), hz = hot_index(ck0, a.hot_z);
        if ((hx | hy | hz) < (uint32_t)HOT_SIDE)
          slot = hot_base + (uint64_t)((uint32_t)p.lam * HOT_CELLS + (hx + HOT_SIDE * (hy + HOT_SIDE * hz)));
      }
      if (TAB) slot |= (uint64_t)p.lam << TAB_LAM_SHIFT | (MESH ? (uint64_t)lvl0 << TAB_LVL_SHIFT : 0ull);
      key = (int64_t)slot;
      has = true;
    }
  }
  if (!(p.I > (R)0)) {
    // the weight underflowed in a very thick absorbing segment: the packet is
    // absorbed (a non-finite weight is reported as a numerical failure)
    if (!isfinite(p.I)) return END_NUMERIC;
    kc.hash() = hash_event(kc.hash(), END_RR_KILL, c);
    return END_RR_KILL;
  }
  if (scat) {
    // the scattering event itself runs in scatter_step(), possibly a few
    // iterations later together with other lanes of the wavefront
    p.fx = fmin(1.0, fmax(0.0, p.fx + tld * dnx));
    p.fy = fmin(1.0, fmax(0.0, p.fy + tld * dny));
    p.fz = fmin(1.0, fmax(0.0, p.fz + tld * dnz));
    pending = true;
    return 0;
  } else {
    if (axis != 0) p.fx = fmin(1.0, fmax(0.0, p.fx + td * dnx));
    if (axis != 1) p.fy = fmin(1.0, fmax(0.0, p.fy + td * dny));
    if (axis != 2) p.fz = fmin(1.0, fmax(0.0, p.fz + td * dnz));
    bool out;
    // leaving through an open face ends the packet; a periodic face brings
    // it back through the opposite one; on a mesh, leaving the leaf block
    // moves it into the leaf beyond
    const int nbx = MESH ? a.mesh.block : a.nx, nby = MESH ? a.mesh.block : a.ny;
    const int nbz = MESH ? a.mesh.block : a.nz;
    if (axis == 0) {
      if (dnx > 0.0) { p.ci++; p.fx = 0.0; } else { p.ci--; p.fx = 1.0; }
      out = p.ci < 0 || p.ci >= nbx;
    } else if (axis == 1) {
      if (dny > 0.0) { p.cj++; p.fy = 0.0; } else { p.cj--; p.fy = 1.0; }
      out = p.cj < 0 || p.cj >= nby;
    } else {
      if (dnz > 0.0) { p.ck++; p.fz = 0.0; } else { p.ck--; p.fz = 1.0; }
      out = p.ck < 0 || p.ck >= nbz;
    }
    // the boundary mask is the same for every lane: open grids skip the wrap
    if (!MESH && a.boundary != 0 && out && ((a.boundary >> axis) & 1)) {
      if (axis == 0) p.ci = p.ci < 0 ? a.nx - 1 : 0;
      else if (axis == 1) p.cj = p.cj < 0 ? a.ny - 1 : 0;
      else p.ck = p.ck < 0 ? a.nz - 1 : 0;
      out = false;
    }
    if (MESH && out) out = mesh_cross(p, a);
    if (out) {
      kc.hash() = hash_event(kc.hash(), END_ESCAPE, c);
      return END_ESCAPE;
    }
    // the next step's density, in flight while this iteration finishes
    p.rho = a.rho[cell_index<MESH>(p, a)];
  }
  return 0;
}

// Stokes vector scattered toward a camera (basis e1 = theta_hat, e2 = phi_hat
// of its direction) by a dipole whose incident coherency is C9 (real xx yy
// zz xy xz yz, imaginary yz zx xy): rho'_ij = h_i^T C conj(h_j) with h_i =
// alpha e_i and the lab polarizability alpha = a_perp 1 + (a_par - a_perp)
// b b^T (b the grain axis), times pf.
template <bool SPHERE>
__device__ __forceinline__ void source_toward(const double C9[9], const Quat<double>& q, const DustDev& D,
                                              const V3<double>& e1, const V3<double>& e2, double pf,
                                              double S[4]) {
  const double Cr[3][3] = {{C9[0], C9[3], C9[4]}, {C9[3], C9[1], C9[5]}, {C9[4], C9[5], C9[2]}};
  const double i6 = C9[6], i7 = C9[7], i8 = C9[8];
  const double Ci[3][3] = {{0.0, i8, -i7}, {-i8, 0.0, i6}, {i7, -i6, 0.0}};
  Cx<double> h1[3], h2[3];
  const double ev1[3] = {e1.x, e1.y, e1.z}, ev2[3] = {e2.x, e2.y, e2.z};
  if (SPHERE) {
#pragma unroll
    for (int k = 0; k < 3; ++k) { h1[k] = {ev1[k], 0.0}; h2[k] = {ev2[k], 0.0}; }
  } else {
    const V3<double> b = from_grain(q, V3<double>{0.0, 0.0, 1.0});
    const double bv[3] = {b.x, b.y, b.z};
    const double b1 = dot(b, e1), b2 = dot(b, e2);
    const Cx<double> ap{D.ap_re, D.ap_im}, dd{D.aa_re - D.ap_re, D.aa_im - D.ap_im};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      h1[k] = cadd(cscale(ap, ev1[k]), cscale(dd, b1 * bv[k]));
      h2[k] = cadd(cscale(ap, ev2[k]), cscale(dd, b2 * bv[k]));
    }
  }
  // g_j = C conj(h_j)
  Cx<double> g1[3], g2[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    g1[k] = {0.0, 0.0};
    g2[k] = {0.0, 0.0};
#pragma unroll
    for (int l = 0; l < 3; ++l) {
      const Cx<double> C{Cr[k][l], Ci[k][l]};
      g1[k] = cadd(g1[k], cmulc(C, h1[l]));
      g2[k] = cadd(g2[k], cmulc(C, h2[l]));
    }
  }
  double r11 = 0.0, r22 = 0.0;
  Cx<double> r12{0.0, 0.0};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    r11 += cmul(h1[k], g1[k]).re;
    r22 += cmul(h2[k], g2[k]).re;
    r12 = cadd(r12, cmul(h1[k], g2[k]));
  }
  S[0] = pf * (r11 + r22);
  S[1] = pf * (r11 - r22);
  S[2] = pf * 2.0 * r12.re;
  S[3] = -pf * 2.0 * r12.im;
}

// Peel-off imaging at a scattering event (the Monte Carlo imaging that Sec.
// 2.3 sets two-step imaging against): for every camera, the Stokes vector the
// event scatters toward it per unit solid angle (from the packet's incident
// coherency, as step 2 forms its source from the tallied one), carried to
// the grid's edge through the Appendix A extinction of every cell on the way
// (no source), added to the pixel the event projects to, per unit pixel
// area.  FP64; open boundaries.
template <typename R, bool ALIGNED, bool SPHERE, bool TAB, bool MESH>
__device__ void peel_off(const Packet<R>& p, const TransportArgs& a, const Quat<double>& q_ev,
                         const DustDev& D) {
  double C9[9];
  const double s_in[4] = {(double)p.I, (double)p.Q, (double)p.U, (double)p.V};
  if (!TAB) coherency<double, 9>(V3<double>{p.nx, p.ny, p.nz}, s_in[0] + s_in[1], s_in[0] - s_in[1], s_in[2], s_in[3], 1.0, C9);
  double X[3] = {a.x0 + ((double)p.ci + p.fx) * a.dx, a.y0 + ((double)p.cj + p.fy) * a.dx,
                 a.z0 + ((double)p.ck + p.fz) * a.dx};
  if (MESH) {
    // the event's position from its leaf's corner, in finest cells
    const int4 o = reinterpret_cast<const int4*>(a.mesh.leaf_org)[p.leaf];
    const double sz = (double)(1ll << (a.mesh.max_level - o.w));
    X[0] = a.x0 + ((double)o.x + ((double)p.ci + p.fx) * sz) * a.mesh.fine;
    X[1] = a.y0 + ((double)o.y + ((double)p.cj + p.fy) * sz) * a.mesh.fine;
    X[2] = a.z0 + ((double)o.z + ((double)p.ck + p.fz) * sz) * a.mesh.fine;
  }
  const int nn[3] = {a.nx, a.ny, a.nz};
  for (int v = 0; v < a.n_views; ++v) {
    const ViewDev vw = a.views[v];
    const double W = vw.half_width;
    const double xi = X[0] * vw.px + X[1] * vw.py + X[2] * vw.pz;
    const double yi = -(X[0] * vw.tx + X[1] * vw.ty + X[2] * vw.tz);
    const double fxp = (xi + W) / (2.0 * W / a.npx), fyp = (yi + W) / (2.0 * W / a.npy);
    if (!(fxp >= 0.0 && fxp < (double)a.npx && fyp >= 0.0 && fyp < (double)a.npy)) continue;
    const int ix = (int)fxp, iy = (int)fyp;
    const V3<double> Om{vw.ox, vw.oy, vw.oz};
    double st[4];
    if (TAB)
      tab_toward<false>(tab_nodes(D), V3<double>{p.nx, p.ny, p.nz}, s_in, Om, V3<double>{vw.tx, vw.ty, vw.tz},
                 V3<double>{vw.px, vw.py, vw.pz}, st);
    else
      source_toward<SPHERE>(C9, q_ev, D, V3<double>{vw.tx, vw.ty, vw.tz}, V3<double>{vw.px, vw.py, vw.pz},
                            D.pfac, st);
    const double om[3] = {vw.ox, vw.oy, vw.oz};
    int ci[3] = {p.ci, p.cj, p.ck};
    double f[3] = {p.fx, p.fy, p.fz};
    int leaf = MESH ? p.leaf : 0, lvl = MESH ? p.lvl : 0;
    const uint64_t Bm = MESH ? (uint64_t)a.mesh.block : 0;
    while (true) {
      double tb = __builtin_huge_val();
      int axis = -1;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        double t;
        if (om[k] > 0.0) t = (1.0 - f[k]) / om[k];
        else if (om[k] < 0.0) t = -f[k] / om[k];
        else continue;
        if (t < tb) { tb = t; axis = k; }
      }
      if (axis < 0) break;
      const uint64_t c = MESH ? (uint64_t)leaf * Bm * Bm * Bm + (uint64_t)ci[0] + Bm * ((uint64_t)ci[1] + Bm * ci[2])
                              : (uint64_t)ci[0] + (uint64_t)a.nx * ((uint64_t)ci[1] + (uint64_t)a.ny * ci[2]);
      const double rho = (double)a.rho[c];
      if (rho > 0.0 && tb > 0.0) {
        const double dtau = rho * D.kext * tb * (MESH ? ldexp(a.dx, -lvl) : a.dx);
        if (SPHERE && !ALIGNED) {
          const double E = exp(-dtau);
#pragma unroll
          for (int k = 0; k < 4; ++k) st[k] *= E;
        } else {
          const double* blk =
              a.tally + ((uint64_t)p.lam * a.nslot + tally_slot(c, ci[0], ci[1], ci[2], MESH ? 0 : a.tbx, a.tby)) *
                            TallyShape<SPHERE>::TS;
          Quat<double> qc{1.0, 0.0, 0.0, 0.0};
          if (ALIGNED) qc = cell_quat<ALIGNED, SPHERE>(a, blk, c);
          V3<double> og = Om;
          double c2 = 1.0, s2 = 0.0;
          if (ALIGNED) {
            og = to_grain(qc, Om);
            eta2(qc, Om, og, c2, s2);
          }
          double a1, a2, a3;
          alphas<double, SPHERE>(D, og.z, a1, a2, a3);
          double sg[4] = {st[0], c2 * st[1] + s2 * st[2], -s2 * st[1] + c2 * st[2], st[3]};
          const double zero[4] = {0.0, 0.0, 0.0, 0.0};
          appA_eigen(a1, a2, a3, dtau, zero, sg);
          st[0] = sg[0];
          st[1] = c2 * sg[1] - s2 * sg[2];
          st[2] = s2 * sg[1] + c2 * sg[2];
          st[3] = sg[3];
        }
      }
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if (k != axis) f[k] = fmin(1.0, fmax(0.0, f[k] + tb * om[k]));
      if (om[axis] > 0.0) { ci[axis]++; f[axis] = 0.0; } else { ci[axis]--; f[axis] = 1.0; }
      if (MESH) {
        if ((ci[axis] < 0 || ci[axis] >= (int)Bm) && !mesh_ray_cross(a.mesh, leaf, lvl, ci, f, om)) break;
        continue;
      }
      if (ci[axis] < 0 || ci[axis] >= nn[axis]) break;
    }
    const double area = (2.0 * W / a.npx) * (2.0 * W / a.npy);
    double* out = a.peel + (((uint64_t)p.lam * a.n_views + v) * 4) * ((uint64_t)a.npx * a.npy) +
                  (uint64_t)iy * a.npx + ix;
#pragma unroll
    for (int k = 0; k < 4; ++k) unsafeAtomicAdd(out + (uint64_t)k * a.npx * a.npy, st[k] / area);
  }
}

// Per-view flush of tabulated grains (the scattering source S of Sec. 2.3,
// eq. scat-disc-sum, one Stokes vector per camera): each staged entry holds
// the segment's weighted Stokes integral (lab basis of its direction) and the
// direction.  The wavefront takes the (entry, camera) pairs 64 at a time, one
// per lane, and projects the entry on the camera with the table; the four
// components then go through the wavefront's LDS area `sp` (64 x 4 doubles)
// so that each atomic instruction writes 64 consecutive doubles: the pairs of
// one entry are adjacent in S[lambda][cell][view][4], so an instruction
// covers whole 128-byte lines (two per entry with 8 cameras) instead of
// putting one component of every pair on its own line -- the drain is bound
// by the L2's atomic line requests, and this cuts them four-fold.  Reached by
// all lanes of the wavefront.  The source is per unit volume of the entry's
// cell: on a composite mesh a cell of level l has (dx 2^-l)^3.
//
// A key holds the tally slot, and above it the cell's mesh level and the
// wavelength.
//
// Where they fit (launch_transport) the tables of all wavelengths and the camera
// directions are read from the block's LDS: the drain then makes no load from
// memory, whose wait would also be for the atomics of the round before (gfx9
// counts both in vmcnt).  128^3 disk, 181 nodes, 8 cameras, 2e6 packets: 34.1 ms
// with the tables in memory, 21.8 in LDS (31.4 and 30.1 with one and two pairs per
// lane and round from memory but without the 64-bit divisions and the square
// root and quotient of n's basis); 9.5e7 entries x 4 lines at the L2's 2.35e10 atomics/s
// are 16 ms.
template <bool MESH, bool LDS>
__device__ __forceinline__ void wave_drain_views(const TransportArgs& a, double* sv, long long* sk, double* sp,
                                                 long long* sa, const double* tab, int lane, int& staged) {
  constexpr int NV = 7;  // staged values per entry: weighted J (4) and n (3)
  const int n = staged;
  if (n == 0) return;
  staged = 0;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const int nv = a.n_views;
  const int items = n * nv;  // at most TAB_CAP x 4096
  const float rnv = 1.0f / (float)nv;
  const double inv_vol = 1.0 / (a.dx * a.dx * a.dx);
  const double* cams = tab + (6 * a.n_lambda + 1) * a.tab_n;
  for (int base = 0; base < items; base += 64) {
    const int it = base + lane;
    if (it < items) {
      int e = (int)((float)it * rnv), v = it - e * nv;
      if (v < 0) { --e; v += nv; }
      if (v >= nv) { ++e; v -= nv; }
      const double* x = sv + e * NV;
      const uint64_t key = (uint64_t)sk[e];
      const uint64_t slot = key & ((1ull << TAB_LVL_SHIFT) - 1ull);
      const int lam = (int)(key >> TAB_LAM_SHIFT);
      const double s_in[4] = {x[0], x[1], x[2], x[3]};
      const V3<double> d{x[4], x[5], x[6]};
      double st[4];
      if (LDS) {
        const double* c = cams + 9 * v;
        const TabNodes T{tab + 6 * a.tab_n * lam, tab + 6 * a.tab_n * a.n_lambda, nullptr, a.tab_n, 0};
        tab_toward<true>(T, d, s_in, V3<double>{c[0], c[1], c[2]}, V3<double>{c[3], c[4], c[5]},
                         V3<double>{c[6], c[7], c[8]}, st);
      } else {
        const ViewDev& vw = a.views[v];
        tab_toward<false>(tab_nodes(a.dust[lam]), d, s_in, V3<double>{vw.ox, vw.oy, vw.oz},
                          V3<double>{vw.tx, vw.ty, vw.tz}, V3<double>{vw.px, vw.py, vw.pz}, st);
      }
      const double iv = MESH ? ldexp(inv_vol, 3 * (int)((key >> TAB_LVL_SHIFT) & 31u)) : inv_vol;
#pragma unroll
      for (int k = 0; k < 4; ++k) sp[4 * lane + k] = st[k] * iv;
      sa[lane] = (long long)((slot * (uint64_t)nv + (uint64_t)v) * 4);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int d = 64 * j + lane;      // component d & 3 of pair d >> 2 of this round
      if (base + (d >> 2) < items) {
        const double val = sp[d];
        if (val != 0.0) unsafeAtomicAdd(a.tally + sa[d >> 2] + (d & 3), val);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

// Scattering event at the packet's current position (Sec. 2.2), the next
// scattering depth.
template <typename R, bool ALIGNED, bool SPHERE, bool PEEL, bool TAB, bool MESH>
__device__ uint32_t scatter_step(Packet<R>& p, const ColdRef& k, const TransportArgs& a) {
  const uint64_t c = cell_index<MESH>(p, a);
  const DustDev& D = a.dust[p.lam];
  Quat<R> q{(R)1, (R)0, (R)0, (R)0};
  Quat<double> qd{1.0, 0.0, 0.0, 0.0};
  if (ALIGNED) {
    const double* blk =
        a.tally + ((uint64_t)p.lam * a.nslot + tally_slot(c, p.ci, p.cj, p.ck, MESH ? 0 : a.tbx, a.tby)) *
                      TallyShape<SPHERE>::TS;
    qd = cell_quat<ALIGNED, SPHERE>(a, blk, c);
    q = quat_cast<R>(qd);
  }
  if (PEEL) peel_off<R, ALIGNED, SPHERE, TAB, MESH>(p, a, qd, D);
  float u_tau;
  if (TAB) {
    if (!scatter_tab<R>(p, k, D, a.seed, u_tau)) return END_NUMERIC;
  } else if (!scatter<R, ALIGNED, SPHERE>(p, k, q, qd, D, a.seed, u_tau)) {
    return END_NUMERIC;
  }
  p.events++;
  k.hash() = hash_event(k.hash(), EV_SCATTER, c);
  p.tau = -log((double)u_tau);
  return 0;
}

// Russian roulette after a segment or an event in the packet's cell (reading
// R8); the cell index is formed only when the check draws
template <bool MESH, typename R>
__device__ uint32_t roulette(Packet<R>& p, const ColdRef& k, const TransportArgs& a) {
  if (!isfinite(p.I)) return END_NUMERIC;
  if (a.rr_wmin > 0.0 && p.I < (R)a.rr_wmin * p.w0) {
    const uint64_t cn = cell_index<MESH>(p, a);
    const R u = (R)next_uniform(k, a.seed, p.lam);
    if (u < (R)a.rr_psurv) {
      const R before = p.I, inv = (R)1 / (R)a.rr_psurv;
      p.I *= inv; p.Q *= inv; p.U *= inv; p.V *= inv;
      k.e_gain() += (double)(p.I - before);
      k.rr()++;
      k.hash() = hash_event(k.hash(), EV_RR_SURVIVE, cn);
    } else {
      k.hash() = hash_event(k.hash(), END_RR_KILL, cn);
      return END_RR_KILL;
    }
  }
  return 0;
}

// stats slots in LDS
enum { SC_STEPS, SC_SCAT, SC_TRIALS, SC_KILL, SC_SURV, SC_ESC, SC_BUDGET, SC_NUM, SC_PACK, SC_FLUSH, SC_N };
enum { SE_EMIT, SE_ESC, SE_ABS, SE_KILL, SE_GAIN, SE_BUDGET, SE_SCAT, SE_N };

template <typename R>
__device__ void finish(const Packet<R>& p, const ColdRef& k, uint32_t end, const TransportArgs& a,
                       unsigned long long* sc, double* se) {
  atomicAdd(&sc[SC_STEPS], (unsigned long long)p.steps);
  atomicAdd(&sc[SC_SCAT], (unsigned long long)p.events);
  atomicAdd(&sc[SC_TRIALS], (unsigned long long)k.trials());
  atomicAdd(&sc[SC_PACK], 1ull);
  if (k.rr()) atomicAdd(&sc[SC_SURV], (unsigned long long)k.rr());
  if (end != END_NUMERIC) {
    atomicAdd(&se[SE_ABS], p.e_abs);
    atomicAdd(&se[SE_SCAT], k.e_scat());
    if (k.e_gain() != 0.0) atomicAdd(&se[SE_GAIN], k.e_gain());
  }
  switch (end) {
    case END_ESCAPE: atomicAdd(&sc[SC_ESC], 1ull); atomicAdd(&se[SE_ESC], (double)p.I); break;
    case END_RR_KILL: atomicAdd(&sc[SC_KILL], 1ull); atomicAdd(&se[SE_KILL], (double)p.I); break;
    case END_BUDGET: atomicAdd(&sc[SC_BUDGET], 1ull); atomicAdd(&se[SE_BUDGET], (double)p.I); break;
    default: atomicAdd(&sc[SC_NUM], 1ull); break;
  }
  const uint64_t pid = k.pid();
  if (a.trace_count && (pid % a.trace_stride) == 0 && pid / a.trace_stride < a.trace_count) {
    TraceDev& t = a.traces[(uint64_t)p.lam * a.trace_count + pid / a.trace_stride];
    t.packet = pid;
    t.end_kind = (int32_t)end;
    t.events = p.events;
    t.steps = p.steps;
    t.last_cell = p.last == 0xffffffffu ? -1ll : (int64_t)p.last;
    t.n[0] = (double)p.nx; t.n[1] = (double)p.ny; t.n[2] = (double)p.nz;
    t.stokes[0] = (double)p.I; t.stokes[1] = (double)p.Q;
    t.stokes[2] = (double)p.U; t.stokes[3] = (double)p.V;
    t.hash = k.hash();
    t.tau_path = (double)p.tau_path;
  }
}

// The kernel's arguments read again from its argument segment, for the paths
// that few iterations take (start, scattering, end of a packet): their
// arguments are then loaded there instead of being held in scalar registers
// (and spilled to vector ones) through the whole loop.
__device__ __forceinline__ TransportArgs reload_args(int varying) {
  const __attribute__((address_space(4))) char* p =
      (const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr();
  asm("" : "+s"(p) : "s"(varying));
  TransportArgs r;
  __builtin_memcpy(&r, p, sizeof r);
  return r;
}

template <typename R, bool ALIGNED, bool SPHERE, bool PEEL, bool TAB, bool MESH, bool BEAM>
__device__ __forceinline__ void transport_body(const TransportArgs& a) {
  constexpr int NC = TallyShape<SPHERE>::NC, TS = TallyShape<SPHERE>::TS;
  __shared__ unsigned long long sc[SC_N];
  __shared__ double se[SE_N];
  // flush staging, one area of FLUSH_CAP entries per wavefront (28 KB per
  // block for spheres, 41 KB for aligned grains; tabulated grains' entries are
  // the segment's Stokes integral and direction, 7 values).  A wavefront
  // drains its area once it holds more than FLUSH_CAP - 64 entries (a stage
  // adds at most 64).  With the cold state (21 KB) three blocks of spheres and two
  // of aligned grains fit a CU; caps of 96 and 150 measured 1-3 % and 5 % slower on
  // the disk.
  constexpr int NSV = TAB ? 7 : NC;
  constexpr int FLUSH_CAP = TAB ? TAB_CAP : 128;
  static_assert(FLUSH_CAP > 64, "an area must take a wavefront's entries");
  __shared__ double s_val[4 * FLUSH_CAP * NSV];
  // tabulated grains: per wavefront the projections of one drain round
  __shared__ double s_proj[TAB ? 4 * 256 : 1];
  __shared__ long long s_addr[TAB ? 4 * 64 : 1];
  __shared__ long long s_key[4 * FLUSH_CAP];
  __shared__ Cold s_cold[4];
  // tabulated grains: the tables' nodes (contiguous on the device) and the
  // camera directions (launch_transport)
  extern __shared__ double s_tab[];
  if (TAB && a.tab_lds) {
    static_assert(!TAB || sizeof(s_val) + sizeof(s_proj) + sizeof(s_addr) + sizeof(s_key) + sizeof(s_cold) + 256 +
                                  8 * TAB_LDS_MAX <= 80 * 1024, "two blocks per CU");
    const int nt = (6 * a.n_lambda + 1) * a.tab_n;
    for (int i = (int)threadIdx.x; i < nt; i += (int)blockDim.x) s_tab[i] = a.dust[0].tab[i];
    for (int i = (int)threadIdx.x; i < 9 * a.n_views; i += (int)blockDim.x)
      s_tab[nt + i] = (&a.views[i / 9].ox)[i % 9];
  }
  if (threadIdx.x < SC_N) sc[threadIdx.x] = 0ull;
  if (threadIdx.x < SE_N) se[threadIdx.x] = 0.0;
  __syncthreads();

  const int lane = (int)__lane_id();
  const int wv = (int)(threadIdx.x >> 6);
  double* sv = s_val + wv * FLUSH_CAP * NSV;
  double* sp = s_proj + (TAB ? wv * 256 : 0);
  long long* sa = s_addr + (TAB ? wv * 64 : 0);
  long long* sk = s_key + wv * FLUSH_CAP;
  const ColdRef kc{s_cold[wv], lane};
  int staged = 0;  // entries in this wavefront's staging area (uniform)
  Packet<R> p;
  bool active = false, exhausted = false, pending = false;
  int waited = 0;
  int64_t last_key = -1;  // key and staging slot of this lane's last entry (slot -1: drained)
  int slot = -1;
  // first slot of this wavefront's copy of the cells around the source
  const uint64_t hot_base =
      a.hot_copies ? (uint64_t)a.n_lambda * (a.nslot + (uint64_t)HOT_CELLS * ((blockIdx.x * 4u + wv) % (uint32_t)a.hot_copies))
                   : 0;
  unsigned long long flushes = 0;  // tally cells flushed by this wavefront

  // Packet ids reserved by this wavefront, [wnext, wend) (uniform).  With
  // spherical grains a step is short and every wavefront refills its idle
  // lanes often: taking ids one refill at a time from the one counter all
  // wavefronts share serialised them on that counter (disk 256^3, 1e8
  // packets: 1371 ms), taking WAVE_CHUNK at a time does not (860 ms).  The
  // aligned-grain kernels contend less and measured slower with the reserve
  // (batched workload 718 -> 744 ms in FP64, 449 -> 494 ms in FP32), so they
  // take exactly the ids they need.
  constexpr bool CHUNKED = SPHERE;
  constexpr unsigned long long WAVE_CHUNK = 64;
  // Lanes refilled together: a start costs ~900 instructions (Philox, sines, a
  // logarithm, divisions) whatever the number of lanes that run it, and lanes that
  // wait for one are idle.  One lane at a time: aligned disk +9 %.  8 and 16 lanes,
  // whole calls: aligned slab 16.51, 16.73 ms; aligned disk 15.59, 15.78; 8
  // wavelengths 35.51, 35.70; mesh 41.08, 41.35; spherical disk 9.27, 9.28, at 1e8
  // packets 609.9, 607.4.
  constexpr int REFILL_BATCH = 8;
  // a refill hands up to 64 idle lanes ids from one new chunk
  static_assert(WAVE_CHUNK >= 64, "a chunk must cover a whole wavefront");
  unsigned long long wnext = 0, wend = 0;
  // A run of fewer packets than the chip has lanes gives each wavefront only
  // `lanes` of them (launch_transport's caller): the time is then the longest
  // packet's, whose every iteration also runs the paths that the wavefront's other
  // packets take (4000 packets in a 32^3 sphere: 0.61 ms with full wavefronts, 0.43
  // with two packets each; 2e4 in a refined sphere 1.41, 1.01).  The scattering batch
  // is that share of its setting, and a share of what still moves at the end.
  const int lanes = a.lanes;
  const unsigned long long chunk = lanes < 64 ? (unsigned long long)lanes : WAVE_CHUNK;
  // refill at this many packets or fewer: 0 once no ids are left (one threshold: a
  // condition of two keeps 30 more registers alive)
  int refill_at = lanes - max(1, REFILL_BATCH * lanes >> 6);
  bool global_done = false;  // the global counter has passed the total
  uint32_t ended = 0;        // this lane's packet has ended (its end kind), not yet reported
  while (true) {
    // Ended packets are reported (finish) and their lanes refilled for
    // REFILL_BATCH lanes of the wavefront at a time, or when no lane is left to
    // move: both run once for all of them instead of once per packet.
    const int nactive = __popcll(__ballot(active));
    if (nactive <= refill_at) {
      if (ended) {
        finish(p, kc, ended, reload_args(nactive), sc, se);
        ended = 0;
      }
      if (exhausted) break;  // nothing moves (nactive == 0) and no ids are left
      const unsigned long long idle = __ballot(!active && lane < lanes);
      const unsigned long long nidle = (unsigned long long)__popcll(idle);
      const int leader = __ffsll((unsigned long long)idle) - 1;
      bool have;
      unsigned long long g;
      const unsigned long long r = (unsigned long long)__popcll(idle & ((1ull << lane) - 1ull));
      if (CHUNKED) {
        const unsigned long long rem = wend - wnext;
        const bool refill = rem < nidle && !global_done;
        unsigned long long base = 0;
        if (refill) {
          if (lane == leader) base = atomicAdd(a.counter, chunk);
          // the leader's value, as a wave-uniform (scalar) value
          const unsigned lo = __builtin_amdgcn_readlane((unsigned)base, leader);
          const unsigned hi = __builtin_amdgcn_readlane((unsigned)(base >> 32), leader);
          base = ((unsigned long long)hi << 32) | lo;
          if (base + chunk >= a.total) global_done = true;
        }
        have = r < rem || refill;
        g = r < rem ? wnext + r : base + (r - rem);
        if (refill) {
          wnext = base + (nidle - rem);
          wend = base + chunk;
        } else {
          wnext += nidle < rem ? nidle : rem;
        }
        if (global_done && (wnext >= wend || wnext >= a.total)) exhausted = true;
      } else {
        unsigned long long base = 0;
        if (lane == leader) base = atomicAdd(a.counter, nidle);
        base = __shfl(base, leader);
        have = true;
        g = base + r;
        if (base + nidle >= a.total) exhausted = true;
      }
      if (exhausted) refill_at = 0;
      if (!active && lane < lanes && have && g < a.total) {
        const bool in = init_packet<R, ALIGNED, SPHERE, MESH>(p, kc, g, reload_args(nactive));
        atomicAdd(&se[SE_EMIT], (double)p.I);  // the emitted intensity
        if (in) active = true;
        else ended = END_ESCAPE;
      }
      continue;
    }
    bool has = false, check = false;
    int64_t key = -1;
    R cc[NC];
    if (active && !pending) {
      ended = step<R, ALIGNED, SPHERE, TAB, MESH>(p, kc, a, hot_base, has, key, cc, pending);
      check = !ended && !pending;
    }
    if (TAB) {
      // tabulated grains: every segment is staged with its direction (a
      // segment's projection on the cameras depends on it)
      const double e7[7] = {(double)cc[0], (double)cc[1], (double)cc[2], (double)cc[3], p.nx, p.ny, p.nz};
      flushes += wave_stage_new<7>(has, key, e7, sv, sk, lane, staged, slot);
      if (staged > FLUSH_CAP - 64) {
        if (a.tab_lds) wave_drain_views<MESH, true>(a, sv, sk, sp, sa, s_tab, lane, staged);
        else wave_drain_views<MESH, false>(a, sv, sk, sp, sa, s_tab, lane, staged);
      }
    } else {
      const int added = wave_stage<NC, R>(has, key, cc, sv, sk, lane, staged, last_key, slot);
      if (!BEAM) flushes += added;
      if (staged > FLUSH_CAP - 64) {
        if (BEAM) flushes += wave_drain_runs<NC, TS>(a.tally, sv, sk, lane, staged);
        else wave_drain<NC, TS>(a.tally, sv, sk, lane, staged);
        slot = -1;
      }
    }
    // Scattering events are run for the parked lanes together once enough
    // of them wait (or one has waited long enough, or nothing else can
    // move): the rejection loop then runs for many lanes at once instead of
    // stalling the wavefront for one lane at a time.
    const unsigned long long pm = __ballot(pending);
    if (pm) {
      ++waited;
      const unsigned long long movable = __ballot(active && !ended && !pending);
      const int batch = events_together(a.scatter_batch, lanes, nactive, exhausted, PEEL);
      if (__popcll(pm) >= batch || waited >= a.scatter_wait || movable == 0ull) {
        waited = 0;
        if (pending) {
          pending = false;
          ended = scatter_step<R, ALIGNED, SPHERE, PEEL, TAB, MESH>(p, kc, reload_args(nactive));
          check = !ended;
        }
      }
    }
    if (check) ended = roulette<MESH>(p, kc, a);
    if (ended) active = false;
  }
  if (TAB && a.tab_lds) wave_drain_views<MESH, true>(a, sv, sk, sp, sa, s_tab, lane, staged);
  else if (TAB) wave_drain_views<MESH, false>(a, sv, sk, sp, sa, s_tab, lane, staged);
  else if (BEAM) flushes += wave_drain_runs<NC, TS>(a.tally, sv, sk, lane, staged);
  else wave_drain<NC, TS>(a.tally, sv, sk, lane, staged);
  if (lane == 0) atomicAdd(&sc[SC_FLUSH], flushes);
  __syncthreads();
  if (threadIdx.x < SC_N) atomicAdd(&(&a.stats->cell_steps)[threadIdx.x], sc[threadIdx.x]);
  if (threadIdx.x < SE_N) unsafeAtomicAdd(&(&a.stats->e_emitted)[threadIdx.x], se[threadIdx.x]);
}

// The persistent transport kernels.  VALU issue and its latency bound them
// (disk: VALU busy 0.72 of the cycles at two waves per SIMD, aligned grains
// 0.45 at one), beside the L2's line atomics, so registers are what the body is
// written for: with the rarely touched state in LDS (Cold), the arguments of
// the rare paths read again where they are used (reload_args) and machine
// LICM off (it would hold the literals of every path in registers across the
// loop), the sphere kernel takes 127 registers (253 before), tables 193, the mesh
// 161 and the FP64 kernel of aligned grains 201 (361), none with a spill:
// three waves per SIMD for spheres and the mesh and two for aligned grains in FP64
// (which spilled 50-190 registers at two before).  256^3 disk, 1e6 packets:
// 8.44 -> 7.17 ms, 3e7: 213.5 -> 173.0 ms; aligned grains, 1e6: 21.9 -> 13.4 ms;
// refined sphere, 2e6: 37.3 -> 31.7 ms.  Four waves per SIMD for spheres measured
// 7.29 / 177.7 ms, and any spill costs more than a wave gains (47 spilled
// registers at four waves: 15.5 ms).  PEEL adds peel-off imaging at every
// scattering event (a separate instantiation); its FP64 body keeps the
// registers it needs, at one wave.
template <bool ALIGNED, bool SPHERE, bool PEEL, bool TAB, bool MESH, bool BEAM>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
k_transport32(TransportArgs a) {
  transport_body<float, ALIGNED, SPHERE, PEEL, TAB, MESH, BEAM>(a);
}
template <bool ALIGNED, bool SPHERE, bool PEEL, bool TAB, bool MESH, bool BEAM>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(PEEL ? 1 : 2)))
k_transport64(TransportArgs a) {
  transport_body<double, ALIGNED, SPHERE, PEEL, TAB, MESH, BEAM>(a);
}

// ---------------------------------------------------------------------------
// utility kernels
// ---------------------------------------------------------------------------
__global__ void k_fill_zero(uint64_t* p, uint64_t nwords, unsigned char* tail, int ntail) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nwords; i += stride)
    p[i] = 0ull;
  if (blockIdx.x == 0 && (int)threadIdx.x < ntail) tail[threadIdx.x] = 0;
}

// Tally blocks of non-spherical grains before a transport run: coherency slots
// zero and the grain-frame quaternion of the alignment direction (identity
// without one) in the four slots after them, for every (wavelength, cell) at its
// tally slot; the rest of each block, and the padding slots of the bricks (never
// read), zero.  A wavefront takes 64 consecutive slots (a brick): each lane forms one
// cell's quaternion, they meet in LDS, and the 64 blocks are written for every
// wavelength in consecutive 16-byte stores.  Bound by the
// writes: 2.1 GB (256^3) in 2.09 ms with one thread per double, five of sixteen
// forming the quaternion, 0.52 ms so.
constexpr int TI_NC = TallyShape<false>::NC, TI_TS = TallyShape<false>::TS;
__global__ void __launch_bounds__(256) k_tally_init(double* tally, const float* bx, const float* by, const float* bz,
                                                    uint64_t ncell, int n_lambda, uint64_t nslot,
                                                    int nx, int ny, int tbx, int tby) {
  __shared__ double held[4][64 * 4];
  const int lane = (int)(threadIdx.x & 63u);
  double* h = held[threadIdx.x >> 6];
  const uint64_t cxy = (uint64_t)nx * (uint64_t)ny;
  const uint64_t nz = tbx ? ncell / cxy : 0;
  const uint64_t groups = (nslot + 63) / 64, stride = (uint64_t)gridDim.x * 4;
  for (uint64_t g = (uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6); g < groups; g += stride) {
    // the cell of this lane's slot (the inverse of tally_slot), if it is one
    uint64_t c = g * 64 + (uint64_t)lane;
    bool valid = c < ncell;
    if (tbx) {
      const uint64_t t = g / (uint64_t)tbx;
      const uint64_t i = (g - t * (uint64_t)tbx) * 4 + (uint64_t)(lane & 3);
      const uint64_t j = (t % (uint64_t)tby) * 4 + (uint64_t)((lane >> 2) & 3);
      const uint64_t k = (t / (uint64_t)tby) * 4 + (uint64_t)(lane >> 4);
      valid = i < (uint64_t)nx && j < (uint64_t)ny && k < nz;
      c = i + (uint64_t)nx * j + cxy * k;
    }
    Quat<double> q{0.0, 0.0, 0.0, 0.0};
    if (valid) {
      q = Quat<double>{1.0, 0.0, 0.0, 0.0};
      if (bx) q = grain_quat(V3<double>{(double)bx[c], (double)by[c], (double)bz[c]});
    }
    h[4 * lane] = q.w;
    h[4 * lane + 1] = q.x;
    h[4 * lane + 2] = q.y;
    h[4 * lane + 3] = q.z;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int it = 0; it < 64 * TI_TS / 128; ++it) {
      const int o = 2 * (64 * it + lane), cell = o / TI_TS, k = o % TI_TS;
      double v[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int m = k + u - TI_NC;
        v[u] = m >= 0 && m < 4 ? h[4 * cell + (m < 0 ? 0 : (m > 3 ? 3 : m))] : 0.0;
      }
      if (g * 64 + (uint64_t)cell < nslot)
        for (int lam = 0; lam < n_lambda; ++lam)
          *reinterpret_cast<double2*>(tally + ((uint64_t)lam * nslot + g * 64) * TI_TS + o) = double2{v[0], v[1]};
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

// The cells of the box around the source: their copies added to the tally.  One
// thread per (wavelength, cell, component); fixed order.
__global__ void k_hot_sum(double* tally, uint64_t nslot, int n_lambda, int copies, int ts, int nc, int hx, int hy,
                          int hz, int nx, int ny, int nz, int tbx, int tby) {
  const int per = HOT_CELLS * nc;
  const int t = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  const int lam = t / per, r = t - lam * per;
  if (lam >= n_lambda) return;
  const int w = r / nc, k = r - w * nc;
  const int i = hx + (w % HOT_SIDE), j = hy + (w / HOT_SIDE) % HOT_SIDE, l = hz + w / (HOT_SIDE * HOT_SIDE);
  if (i < 0 || j < 0 || l < 0 || i >= nx || j >= ny || l >= nz) return;
  const double* h = tally + ((uint64_t)n_lambda * nslot + (uint64_t)lam * HOT_CELLS + w) * ts + k;
  double s = 0.0;
  for (int m = 0; m < copies; ++m) s += h[(uint64_t)m * n_lambda * HOT_CELLS * ts];
  const uint64_t c = (uint64_t)i + (uint64_t)nx * ((uint64_t)j + (uint64_t)ny * (uint64_t)l);
  if (s != 0.0) tally[((uint64_t)lam * nslot + tally_slot(c, i, j, l, tbx, tby)) * ts + k] += s;
}

__global__ void k_validate(const float* rho, const float* bx, const float* by, const float* bz,
                           uint64_t n, unsigned long long* bad) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  unsigned long long nbad = 0;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const float r = rho[i];
    if (!(r >= 0.0f) || !isfinite(r)) nbad++;
    if (bx) {
      const double b2 = (double)bx[i] * bx[i] + (double)by[i] * by[i] + (double)bz[i] * bz[i];
      if (!(fabs(sqrt(b2) - 1.0) <= 1e-5)) nbad++;
    }
  }
  if (nbad) atomicAdd(bad, nbad);
}

// ---------------------------------------------------------------------------
// Thermal emission tables (set-up of the dust's emission, Sec. 2.2): for one
// wavelength the running sum F of the cell luminosities fac rho B (fac =
// 4 pi kappa_abs dx^3) over the cells in flat order, and its guide table.
// On a composite mesh (lorg non-null: leaf origins and levels, b3 = block^3
// cells per leaf) a cell's luminosity carries its own volume, 2^-3 level of
// a root cell's.  Blocks of EM_CHUNK cells; thread t of a block sums EM_PER
// consecutive cells.
// ---------------------------------------------------------------------------
constexpr int EM_THREADS = 256;
constexpr int EM_PER = 16;
constexpr uint64_t EM_CHUNK = (uint64_t)EM_THREADS * EM_PER;

__device__ __forceinline__ double em_lum(const float* rho, const float* B, double fac, const int32_t* lorg,
                                         uint64_t b3, uint64_t c) {
  const double l = fac * (double)rho[c] * (double)B[c];
  return lorg ? ldexp(l, -3 * lorg[4 * (c / b3) + 3]) : l;
}

__device__ __forceinline__ double em_thread_sum(const float* rho, const float* B, double fac,
                                                const int32_t* lorg, uint64_t b3, uint64_t first,
                                                uint64_t ncell) {
  double sum = 0.0;
  for (int k = 0; k < EM_PER; ++k) {
    const uint64_t c = first + k;
    if (c < ncell) sum += em_lum(rho, B, fac, lorg, b3, c);
  }
  return sum;
}

// exclusive scan of one value per thread over a block of EM_THREADS
__device__ __forceinline__ double em_block_exclusive(double v, double* sh, double* total) {
  const int t = threadIdx.x;
  sh[t] = v;
  __syncthreads();
  for (int off = 1; off < EM_THREADS; off <<= 1) {
    const double add = t >= off ? sh[t - off] : 0.0;
    __syncthreads();
    sh[t] += add;
    __syncthreads();
  }
  const double incl = sh[t];
  *total = sh[EM_THREADS - 1];
  __syncthreads();
  return incl - v;
}

__global__ void __launch_bounds__(EM_THREADS)
k_em_partial(const float* rho, const float* B, double fac, const int32_t* lorg, uint64_t b3, uint64_t ncell,
             double* partial) {
  __shared__ double sh[EM_THREADS];
  const uint64_t first = (uint64_t)blockIdx.x * EM_CHUNK + (uint64_t)threadIdx.x * EM_PER;
  double total;
  em_block_exclusive(em_thread_sum(rho, B, fac, lorg, b3, first, ncell), sh, &total);
  if (threadIdx.x == 0) partial[blockIdx.x] = total;
}

// one block: block totals -> exclusive block offsets, in place
__global__ void __launch_bounds__(EM_THREADS) k_em_offsets(double* partial, uint64_t nb) {
  __shared__ double sh[EM_THREADS];
  const uint64_t per = (nb + EM_THREADS - 1) / EM_THREADS;
  const uint64_t b0 = (uint64_t)threadIdx.x * per;
  double sum = 0.0;
  for (uint64_t b = b0; b < b0 + per && b < nb; ++b) sum += partial[b];
  double total;
  double run = em_block_exclusive(sum, sh, &total);
  for (uint64_t b = b0; b < b0 + per && b < nb; ++b) {
    const double v = partial[b];
    partial[b] = run;
    run += v;
  }
}

__global__ void __launch_bounds__(EM_THREADS)
k_em_cdf(const float* rho, const float* B, double fac, const int32_t* lorg, uint64_t b3, uint64_t ncell,
         const double* offsets, double* cdf) {
  __shared__ double sh[EM_THREADS];
  const uint64_t first = (uint64_t)blockIdx.x * EM_CHUNK + (uint64_t)threadIdx.x * EM_PER;
  double total;
  double run = offsets[blockIdx.x] +
               em_block_exclusive(em_thread_sum(rho, B, fac, lorg, b3, first, ncell), sh, &total);
  for (int k = 0; k < EM_PER; ++k) {
    const uint64_t c = first + k;
    if (c < ncell) {
      run += em_lum(rho, B, fac, lorg, b3, c);
      cdf[c] = run;
    }
  }
}

// guide[k] = the first cell whose running sum exceeds L k / ncell
// (k < ncell); guide[ncell] = the last cell
__global__ void k_em_guide(const double* cdf, uint64_t ncell, uint32_t* guide) {
  const uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k > ncell) return;
  if (k == ncell) { guide[k] = (uint32_t)(ncell - 1); return; }
  const double T = cdf[ncell - 1] * ((double)k / (double)ncell);
  uint64_t lo = 0, hi = ncell - 1;
  while (lo < hi) {
    const uint64_t mid = lo + ((hi - lo) >> 1);
    if (T < cdf[mid]) hi = mid; else lo = mid + 1;
  }
  guide[k] = (uint32_t)lo;
}

uint64_t emission_blocks(uint64_t ncell) { return (ncell + EM_CHUNK - 1) / EM_CHUNK; }

hipError_t launch_emission_table(const float* rho, const float* B, double fac, const int32_t* leaf_org,
                                 uint64_t block3, uint64_t ncell, double* partial, double* cdf, uint32_t* guide,
                                 hipStream_t s) {
  const uint64_t nb = emission_blocks(ncell);
  hipLaunchKernelGGL(k_em_partial, dim3((unsigned)nb), dim3(EM_THREADS), 0, s, rho, B, fac, leaf_org, block3,
                     ncell, partial);
  hipLaunchKernelGGL(k_em_offsets, dim3(1), dim3(EM_THREADS), 0, s, partial, nb);
  hipLaunchKernelGGL(k_em_cdf, dim3((unsigned)nb), dim3(EM_THREADS), 0, s, rho, B, fac, leaf_org, block3, ncell,
                     (const double*)partial, cdf);
  hipLaunchKernelGGL(k_em_guide, dim3((unsigned)((ncell + 1 + 255) / 256)), dim3(256), 0, s,
                     (const double*)cdf, ncell, guide);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
// A pencil beam's runs have kernels with a drain of their own (wave_drain_runs; as a
// branch of the others' it made the mesh's 4 % slower), except with peel-off, whose
// events take the time, and tabulated grains, whose drains are per camera.
static bool beam_kernel(int src_kind, bool peel, bool tab) { return src_kind == 1 && !peel && !tab; }

template <bool A, bool S, bool T, bool M>
static void launch_one(const TransportArgs& a, bool fp64, bool peel, int blocks, int bs, hipStream_t s) {
  const size_t lds = (size_t)a.tab_lds * 8;
  if constexpr (!T) {
    if (beam_kernel(a.src_kind, peel, T)) {
      if (fp64) hipLaunchKernelGGL((k_transport64<A, S, false, T, M, true>), dim3(blocks), dim3(bs), lds, s, a);
      else hipLaunchKernelGGL((k_transport32<A, S, false, T, M, true>), dim3(blocks), dim3(bs), lds, s, a);
      return;
    }
  }
  if (fp64 && peel) hipLaunchKernelGGL((k_transport64<A, S, true, T, M, false>), dim3(blocks), dim3(bs), lds, s, a);
  else if (fp64) hipLaunchKernelGGL((k_transport64<A, S, false, T, M, false>), dim3(blocks), dim3(bs), lds, s, a);
  else if (peel) hipLaunchKernelGGL((k_transport32<A, S, true, T, M, false>), dim3(blocks), dim3(bs), lds, s, a);
  else hipLaunchKernelGGL((k_transport32<A, S, false, T, M, false>), dim3(blocks), dim3(bs), lds, s, a);
}

hipError_t launch_transport(const TransportArgs& a, bool fp64, bool aligned, bool sphere, bool peel, bool tab,
                            bool mesh, int blocks, int block_size, hipStream_t s) {
  if (mesh && tab) {
    launch_one<false, true, true, true>(a, fp64, peel, blocks, block_size, s);
  } else if (mesh) {
    if (aligned && sphere) launch_one<true, true, false, true>(a, fp64, peel, blocks, block_size, s);
    else if (aligned) launch_one<true, false, false, true>(a, fp64, peel, blocks, block_size, s);
    else if (sphere) launch_one<false, true, false, true>(a, fp64, peel, blocks, block_size, s);
    else launch_one<false, false, false, true>(a, fp64, peel, blocks, block_size, s);
  } else if (tab) {
    launch_one<false, true, true, false>(a, fp64, peel, blocks, block_size, s);
  } else if (aligned && sphere) {
    launch_one<true, true, false, false>(a, fp64, peel, blocks, block_size, s);
  } else if (aligned) {
    launch_one<true, false, false, false>(a, fp64, peel, blocks, block_size, s);
  } else if (sphere) {
    launch_one<false, true, false, false>(a, fp64, peel, blocks, block_size, s);
  } else {
    launch_one<false, false, false, false>(a, fp64, peel, blocks, block_size, s);
  }
  return hipGetLastError();
}

template <bool A, bool S, bool PL, bool T, bool M, bool B>
static int occ_one(bool fp64, int bs, size_t lds) {
  int n = 0;
  const hipError_t e = fp64 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_transport64<A, S, PL, T, M, B>, bs, lds)
                            : hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_transport32<A, S, PL, T, M, B>, bs, lds);
  return e == hipSuccess ? n : 0;
}

template <bool A, bool S, bool T, bool M>
static int occ_peel(bool fp64, bool peel, bool beam, int bs, size_t lds = 0) {
  if constexpr (!T)
    if (beam) return occ_one<A, S, false, T, M, true>(fp64, bs, lds);
  return peel ? occ_one<A, S, true, T, M, false>(fp64, bs, lds) : occ_one<A, S, false, T, M, false>(fp64, bs, lds);
}

int transport_max_blocks_per_cu(bool fp64, bool aligned, bool sphere, bool peel, bool tab, bool mesh,
                                int src_kind, int block_size, int tab_lds) {
  const bool beam = beam_kernel(src_kind, peel, tab);
  const size_t lds = (size_t)tab_lds * 8;
  if (mesh && tab) return occ_peel<false, true, true, true>(fp64, peel, beam, block_size, lds);
  if (mesh) {
    if (aligned && sphere) return occ_peel<true, true, false, true>(fp64, peel, beam, block_size);
    if (aligned) return occ_peel<true, false, false, true>(fp64, peel, beam, block_size);
    if (sphere) return occ_peel<false, true, false, true>(fp64, peel, beam, block_size);
    return occ_peel<false, false, false, true>(fp64, peel, beam, block_size);
  }
  if (tab) return occ_peel<false, true, true, false>(fp64, peel, beam, block_size, lds);
  if (aligned && sphere) return occ_peel<true, true, false, false>(fp64, peel, beam, block_size);
  if (aligned) return occ_peel<true, false, false, false>(fp64, peel, beam, block_size);
  if (sphere) return occ_peel<false, true, false, false>(fp64, peel, beam, block_size);
  return occ_peel<false, false, false, false>(fp64, peel, beam, block_size);
}

hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t s) {
  if (bytes == 0) return hipSuccess;
  const uint64_t nwords = bytes / 8;
  const int ntail = (int)(bytes % 8);
  uint64_t blocks = (nwords + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (blocks == 0) blocks = 1;
  hipLaunchKernelGGL(k_fill_zero, dim3((unsigned)blocks), dim3(256), 0, s, (uint64_t*)p, nwords,
                     (unsigned char*)p + nwords * 8, ntail);
  return hipGetLastError();
}

hipError_t launch_tally_init(double* tally, const float* bx, const float* by,
                             const float* bz, uint64_t ncell, int n_lambda, bool sphere, uint64_t nslot, int nx,
                             int ny, int tbx, int tby, hipStream_t s) {
  if (sphere) return launch_fill_zero(tally, (size_t)n_lambda * nslot * tally_stride(true) * sizeof(double), s);
  uint64_t blocks = (nslot + 255) / 256;
  if (blocks > 16384) blocks = 16384;
  hipLaunchKernelGGL(k_tally_init, dim3((unsigned)blocks), dim3(256), 0, s, tally, bx, by, bz, ncell, n_lambda,
                     nslot, nx, ny, tbx, tby);
  return hipGetLastError();
}

hipError_t launch_hot_sum(const TransportArgs& a, int ts, int nc, hipStream_t s) {
  const int n = a.n_lambda * HOT_CELLS * nc;  // below HOT_BYTES / 8
  hipLaunchKernelGGL(k_hot_sum, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a.tally, a.nslot, a.n_lambda,
                     a.hot_copies, ts, nc, a.hot_x, a.hot_y, a.hot_z, a.nx, a.ny, a.nz, a.tbx, a.tby);
  return hipGetLastError();
}

hipError_t launch_validate(const float* rho, const float* bx, const float* by, const float* bz,
                           uint64_t n, unsigned long long* bad, hipStream_t s) {
  uint64_t blocks = (n + 255) / 256;
  if (blocks > 16384) blocks = 16384;
  if (blocks == 0) blocks = 1;
  hipLaunchKernelGGL(k_validate, dim3((unsigned)blocks), dim3(256), 0, s, rho, bx, by, bz, n, bad);
  return hipGetLastError();
}

}  // namespace kp
