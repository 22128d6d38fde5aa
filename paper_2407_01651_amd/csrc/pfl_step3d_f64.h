// Fused 3D time step in FP64 (the parity form): D3Q19 flow, D3Q7 bubble phase,
// order parameter, solute and heat, advanced by one step in one launch.  The
// scheme is the FP32-compute step's (pfl_step3d_impl.h): the same column of
// nodes marching through z with LDS rings of planes, the same stencils and
// closed-form collisions.
//
// What differs is what a thread holds between pulling its node's populations
// and finishing the node: not the populations but the moments the collisions
// need, nine of the 19 flow populations and four of each seven.  (The
// FP32-compute forms are built with reassociation, so that any change of their
// source changes their rounding; they keep populations.)
#pragma once
#include "pfl_step3d.h"

namespace pfl {

namespace {

// Moments of a node's flow populations: momentum, sum of the moving ones (the
// pressure's) and the five traceless stresses; of a 7-velocity set: sum and
// flux.
struct NsMom {
  double j[3], s9, s11, sxy, syz, sxz, sum;
};
struct ScMom {
  double d, J[3];
};
__device__ __forceinline__ void ns_momentum(const double (&f)[19], double (&j)[3]) {
  using L = Lat<19>;
  j[0] = j[1] = j[2] = 0.0;
#pragma unroll
  for (int i = 0; i < 19; ++i) {
    if (L::c[i][0]) j[0] += L::c[i][0] * f[i];
    if (L::c[i][1]) j[1] += L::c[i][1] * f[i];
    if (L::c[i][2]) j[2] += L::c[i][2] * f[i];
  }
}
__device__ __forceinline__ void ns_moments(const double (&f)[19], NsMom& m) {
  using L = Lat<19>;
  ns_momentum(f, m.j);
  m.sum = m.s9 = m.s11 = m.sxy = m.syz = m.sxz = 0.0;
#pragma unroll
  for (int i = 1; i < 19; ++i) {
    const int cx = L::c[i][0], cy = L::c[i][1], cz = L::c[i][2];
    m.sum += f[i];
    m.s9 += (double)(2 * cx * cx - cy * cy - cz * cz) * f[i];
    m.s11 += (double)(cy * cy - cz * cz) * f[i];
    m.sxy += (double)(cx * cy) * f[i];
    m.syz += (double)(cy * cz) * f[i];
    m.sxz += (double)(cx * cz) * f[i];
  }
}
__device__ __forceinline__ double sc_sum(const double (&f)[7]) {
  double d = 0.0;
#pragma unroll
  for (int i = 0; i < 7; ++i) d += f[i];
  return d;
}
__device__ __forceinline__ void sc_moments(const double (&f)[7], ScMom& m) {
  m.d = sc_sum(f);
#pragma unroll
  for (int a = 0; a < 3; ++a) m.J[a] = f[1 + 2 * a] - f[2 + 2 * a];
}

// U from psi and C.
__device__ __forceinline__ double u_of(const KP<double>& K, double psi, double C) {
  return (C * rcp(1.0 - K.k1 * ((psi + 1.0) * 0.5)) - 1.0) * K.inv_k1;
}

// Flow quantities at one LDS position of a plane (node or ring 1) that the own
// node's collision takes too: grad phi, k_s mu, 1 / sqrt(|grad phi|^2 + delta).
struct FlowKept {
  double g[3], ksmu, inv;
};
// The quantities that follow from phi and psi alone.
struct FlowPoint {
  double sharp, chi, rho;
};
__device__ __forceinline__ FlowPoint flow_point(const KP<double>& K, double phi, double psi) {
  FlowPoint o;
  const double dw = (1.0 - phi) * phi;
  o.sharp = K.sharp * (dw > 0.0 ? dw : 0.0);
  o.chi = clamp01((psi + 1.0) * 0.5);
  o.rho = K.rho_g + K.drho * phi;
  return o;
}
// (y, x) in ring-1 plane coordinates; ph: the phi planes below, at and above;
// psi of the position.  Without the bubble phase phi = 1 and the stencils vanish.
template <bool NS, bool PHI, int R>
__device__ __forceinline__ void flow_kept(const KP<double>& K, const double* const ph[3], double phi, double psi,
                                          int y, int x, FlowKept& o) {
  using PR = Pl<double, R>;
  constexpr int d = R - 1;
  double lap = 0.0;
  o.g[0] = o.g[1] = o.g[2] = 0.0;
  if constexpr (PHI) {
    grad19p<double, PR>(ph, y + d, x + d, o.g);
    lap = lap19p<double, PR>(ph, y + d, x + d);
  }
  o.inv = rsq(o.g[0] * o.g[0] + o.g[1] * o.g[1] + o.g[2] * o.g[2] + K.dn);
  o.ksmu = 0.0;
  if constexpr (NS) {
    const double one_m = 1.0 - phi;
    const double f1p = 0.5 * one_m * phi * (1.0 - 2.0 * phi);
    const double ps1 = psi + 1.0;
    const double f3p = -2.0 * K.beta_inter * one_m * ps1 * ps1;
    o.ksmu = K.k_s * (f1p + f3p - K.Wphi2 * lap);
  }
}
// D_phi and the velocity without the mass-flux force at a position of momentum j.
__device__ __forceinline__ void dv_of(const KP<double>& K, const FlowKept& f, double phi, double psi,
                                      const double (&j)[3], double (&D)[3], double (&v0)[3]) {
  const FlowPoint q = flow_point(K, phi, psi);
  const double s = (1.0 - q.chi) * rcp(q.rho);
  const double Fb[3] = {0.0, -(q.rho - K.rho_l) * K.g, 0.0};
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    D[a] = K.M_phi * (f.g[a] - q.sharp * (f.g[a] * f.inv));
    v0[a] = s * (j[a] + 0.5 * (f.ksmu * f.g[a] + Fb[a]));
  }
}

// Temperature of a node: H = c_p theta - c_p^s h with sum g = rho H; rho, c_p,
// k_T linear in phi between gas and liquid (liquid = solid = 1); s_th the heat
// relaxation rate from k_T.
__device__ __forceinline__ void heat_of(const KP<double>& K, double phi, double h, double H, double& theta, double& s_th) {
  s_th = K.s_th;
  if (K.varheat) {
    const double rh = K.th_rho_g + (1.0 - K.th_rho_g) * phi;
    const double cp = K.th_cp_g + (1.0 - K.th_cp_g) * phi;
    const double kh = K.th_k_g + (1.0 - K.th_k_g) * phi;
    theta = (H + rh * h) / (rh * cp);
    s_th = rcp(K.alpha_cs * kh + 0.5);
  } else {
    theta = H + h;
  }
}

// Anisotropy, kinetics and source of psi at a node.
struct PsiNode {
  double invp, a_s, as2, Nv[3], lin, an, S, rate;
};
__device__ __forceinline__ void psi_node(const DevParams& P, const KP<double>& K, const double (&gp)[3],
                                         const double (&gU)[3], double cth, double sth, double phi, double psi,
                                         double theta, double U, PsiNode& o) {
  const double dn = K.dn;
  o.invp = rsq(gp[0] * gp[0] + gp[1] * gp[1] + gp[2] * gp[2] + dn);
  // cubic anisotropy in the crystal frame (rotation about z):
  // a_s = 1 + eps (4 S4 - 3 G^2) / (G + delta)^2, N' = G a_s d a_s / d g'
  const double r[3] = {cth * gp[0] + sth * gp[1], -sth * gp[0] + cth * gp[1], gp[2]};
  const double r2[3] = {r[0] * r[0], r[1] * r[1], r[2] * r[2]};
  const double G = r2[0] + r2[1] + r2[2];
  const double S4 = r2[0] * r2[0] + r2[1] * r2[1] + r2[2] * r2[2];
  const double invGd = rcp(G + dn);
  const double inv2 = invGd * invGd;
  const double eps = K.eps4;
  o.a_s = 1.0 + eps * (4.0 * S4 - 3.0 * G * G) * inv2;
  const double pre = 4.0 * eps * G * o.a_s * inv2 * invGd;
  double Nr[3];
#pragma unroll
  for (int a = 0; a < 3; ++a)
    Nr[a] = pre * r[a] * (4.0 * r2[a] * G + (4.0 * r2[a] - 3.0 * G) * dn - 4.0 * S4);
  o.Nv[0] = cth * Nr[0] - sth * Nr[1];
  o.Nv[1] = sth * Nr[0] + cth * Nr[1];
  o.Nv[2] = Nr[2];
  o.as2 = o.a_s * o.a_s;

  o.lin = 1.0 + K.k1 * U;
  const double F = K.inv_Le + K.Mcinf * (o.lin > 0.0 ? o.lin : 0.0);
  const double gFs = o.lin > 0.0 ? K.Mcinf * K.k1 : 0.0;
  const double om = 1.0 - phi;
  const double ps1 = psi + 1.0;
  const double f2p = 0.5 * (1.0 - psi) * ps1 * (-2.0 * psi);
  const double f3psi = 2.0 * K.beta_inter * om * om * ps1;
  const double s1m = (1.0 - psi) * ps1;
  const double pprime = 30.0 / 32.0 * s1m * s1m;
  const double Qpsi = -(f2p + f3psi + K.lam * pprime * (theta + K.Mcinf * U));
  // rewritten form: a_n = a_s^2, F(U) in D_psi and S_psi with the
  // grad F term; form for Le = O(1): a_n = a_s^2 F(U) (Appendix B)
  double D_psi;
  if (P.le1) {
    o.S = Qpsi * K.inv_tau0;
    D_psi = K.d_psi * o.as2;
    o.an = o.as2 * F;
  } else {
    const double invF = rcp(F);
    double gdot = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) gdot += gFs * gU[a] * (o.as2 * gp[a] + o.Nv[a]);
    o.S = K.d_psi * invF * invF * gdot + Qpsi * invF * K.inv_tau0;
    D_psi = K.d_psi * o.as2 * invF;
    o.an = o.as2;
  }
  o.rate = rcp(D_psi * (1.0 / Lat<7>::cs2) + 0.5);
}

// The populations of an axis of a 7-velocity set are an even part plus or
// minus an odd one: put(0, rest), put(1 + 2 a, even + odd[a]), put(2 + 2 a, even - odd[a]).
template <class Put>
__device__ __forceinline__ void put7(double rest, double even, const double (&odd)[3], Put&& put) {
  put(0, rest);
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    put(1 + 2 * a, even + odd[a]);
    put(2 + 2 * a, even - odd[a]);
  }
}
constexpr double W7_0 = Lat<7>::w[0], W7_1 = Lat<7>::w[1], W7_C = Lat<7>::w[1] / Lat<7>::cs2;

// CAC collision: equilibrium w phi (1 + c.v/cs2), whose flux is phi v; the
// source's flux fl = d(phi v)/dt + sharpening.
template <class Put>
__device__ __forceinline__ void collide_phi(const KP<double>& K, const ScMom& m, const double (&phiv)[3],
                                            const double (&prev)[3], double sharp, const double (&n)[3], Put&& put) {
  const double r = 1.0 - K.s_phi;
  double odd[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const double fl = (phiv[a] - prev[a]) + Lat<7>::cs2 * sharp * n[a];
    odd[a] = W7_C * phiv[a] + 0.5 * r * (m.J[a] - phiv[a]) + (0.5 * W7_C + 0.25 * r) * fl;
  }
  put7(W7_0 * m.d, W7_1 * m.d, odd, put);
}
// AAC collision f* before the time stretch; G_i = -w_i c_i.N / a_s^2.
template <class Put>
__device__ __forceinline__ void collide_psi(const DevParams& P, const ScMom& m, const PsiNode& q, double Sprev,
                                            Put&& put) {
  const double inv_as2 = P.le1 ? rcp(q.as2) : rcp(q.an);
  const double even = m.d + q.S + 0.5 * (q.S - Sprev);
  double odd[3];
#pragma unroll
  for (int a = 0; a < 3; ++a)
    odd[a] = 0.5 * (1.0 - q.rate) * m.J[a] - (1.0 - 0.5 * q.rate) * W7_1 * q.Nv[a] * inv_as2;
  put7(W7_0 * even, W7_1 * even, odd, put);
}
// Collision of the solute or heat set with equilibrium flux B, its change dB
// since the last step and rate s1.
template <class Put>
__device__ __forceinline__ void collide_flux(double rest, double even, const ScMom& m, const double (&B)[3],
                                             const double (&dB)[3], double s1, Put&& put) {
  double odd[3];
#pragma unroll
  for (int a = 0; a < 3; ++a)
    odd[a] = W7_C * B[a] + 0.5 * (1.0 - s1) * (m.J[a] - B[a]) + (1.0 - 0.5 * s1) * W7_C * dB[a];
  put7(rest, even, odd, put);
}

// Velocity, forces and pressure of a node from its moments and forces.
struct Flow {
  double v[3], F[3], gr[3], p, rho;
};
__device__ __forceinline__ void flow_node_state(const KP<double>& K, const NsMom& m, const FlowKept& k, const FlowPoint& q,
                                                const double (&dv)[3], Flow& o) {
  using L = Lat<19>;
  o.rho = q.rho;
  const double Fb[3] = {0.0, -(q.rho - K.rho_l) * K.g, 0.0};
  const double onechi = 1.0 - q.chi, irho = rcp(q.rho);
  double vv = 0.0, vg = 0.0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    // mass-flux force: (1/cs2) sum_i w_i (c_i . D(x + c_i)) v0_b(x + c_i) = 3 dv
    const double Fs = k.ksmu * k.g[a], Fm = K.drho * 3.0 * dv[a];
    const double rv = m.j[a] + 0.5 * (Fs + Fb[a] + Fm);
    o.v[a] = onechi * rv * irho;
    o.F[a] = Fs + Fb[a] + Fm - 2.0 * q.chi * rv;
    o.gr[a] = K.drho * k.g[a];
    vv += o.v[a] * o.v[a];
    vg += o.v[a] * o.gr[a];
  }
  o.p = L::cs2 / (1.0 - L::w[0]) * (m.sum + 0.5 * vg - q.rho * (L::w[0] * 1.5 * vv));
}

// NS collision: f* = feq + F/2 + (1 - s_nu) P_s (f - feq + F/2), P_s the
// orthogonal projector on the five traceless stress moments
// 2cx^2 - cy^2 - cz^2, cy^2 - cz^2, cx cy, cy cz, cx cz (squared norms over
// D3Q19: 36, 12, 4, 4, 4), in moment form: D3Q19 is 4th-order isotropic, so
// each traceless stress moment T of f^eq + F/2 is rho T:vv + T:(vF + cs2 v
// grad(rho)) symmetrised; for i > 0 f_i^eq + F_i/2 = w_i [A + c.v (3 rho + 4.5
// (rho c.v + c.F) + 1.5 c.grad(rho)) + 1.5 c.F] with A = 3p - 1.5 rho v.v -
// 1.5 v.F, and w_0 A - 3p at rest.  Opposite populations share their even and
// odd parts: put(i, own, opposite).
template <class Put>
__device__ __forceinline__ void collide_ns(const KP<double>& K, const NsMom& m, const Flow& o, double phi, Put&& put) {
  using L = Lat<19>;
  const double rho = o.rho;
  const double nu = (K.mu_g + (K.mu_l - K.mu_g) * phi) * rcp(rho);
  const double r = 1.0 - rcp(nu * 3.0 + 0.5);
  const double vx = o.v[0], vy = o.v[1], vz = o.v[2], Fx = o.F[0], Fy = o.F[1], Fz = o.F[2];
  const double gx = o.gr[0], gy = o.gr[1], gz = o.gr[2];
  const double vv = vx * vx + vy * vy + vz * vz;
  const double vF = vx * Fx + vy * Fy + vz * Fz;
  const double A = 3.0 * o.p - 1.5 * rho * vv - 1.5 * vF;
  constexpr double c3 = 1.0 / 3, c6 = 1.0 / 6;
  const double q9 = (r * (1.0 / 36)) * (m.s9 - rho * (2.0 * vx * vx - vy * vy - vz * vz) +
                                        (2.0 * vx * Fx - vy * Fy - vz * Fz) + c3 * (2.0 * vx * gx - vy * gy - vz * gz));
  const double q11 = (r * (1.0 / 12)) * (m.s11 - rho * (vy * vy - vz * vz) + (vy * Fy - vz * Fz) + c3 * (vy * gy - vz * gz));
  const double qxy = (r * 0.25) * (m.sxy - rho * vx * vy + 0.5 * (vx * Fy + vy * Fx) + c6 * (vx * gy + vy * gx));
  const double qyz = (r * 0.25) * (m.syz - rho * vy * vz + 0.5 * (vy * Fz + vz * Fy) + c6 * (vy * gz + vz * gy));
  const double qxz = (r * 0.25) * (m.sxz - rho * vx * vz + 0.5 * (vx * Fz + vz * Fx) + c6 * (vx * gz + vz * gx));
  const double rho3 = 3.0 * rho;
  put(0, L::w[0] * A - 3.0 * o.p, L::w[0] * A - 3.0 * o.p);
#pragma unroll
  for (int i = 1; i < 19; i += 2) {
    const int cx = L::c[i][0], cy = L::c[i][1], cz = L::c[i][2];
    const double w = L::w[i];
    const double cv = cx * vx + cy * vy + cz * vz;
    const double cF = cx * Fx + cy * Fy + cz * Fz;
    const double cg = cx * gx + cy * gy + cz * gz;
    const double even = w * (A + cv * (4.5 * (rho * cv + cF) + 1.5 * cg)) +
                        ((double)(2 * cx * cx - cy * cy - cz * cz) * q9 + (double)(cy * cy - cz * cz) * q11 +
                         (double)(cx * cy) * qxy + (double)(cy * cz) * qyz + (double)(cx * cz) * qxz);
    const double odd = w * (cv * rho3 + 1.5 * cF);
    put(i, even + odd, even - odd);
    put(i + 1, even - odd, even + odd);
  }
}
static_assert([] {
  for (int i = 1; i < 19; i += 2)
    if (Lat<19>::opp[i] != i + 1) return false;
  return true;
}(), "opposite flow populations are neighbours");

// What a population that leaves the node across a side becomes when stored:
// bits of the sides crossed by direction (dx, dy, dz) at node (x, y, z).
__device__ __forceinline__ bool leaves(const DevParams& P, int sides, int x, int y, int z, int dx, int dy, int dz) {
  return (dx > 0 && x == P.nx - 1 && ((sides >> 3) & 1)) || (dx < 0 && x == 0 && (sides & 1)) ||
         (dy > 0 && y == P.ny - 1 && ((sides >> 4) & 1)) || (dy < 0 && y == 0 && ((sides >> 1) & 1)) ||
         (dz > 0 && z == P.nz - 1 && ((sides >> 5) & 1)) || (dz < 0 && z == 0 && ((sides >> 2) & 1));
}
// Stored value of a 7-velocity population: by anti-bounce-back to the value
// zeta where it leaves across a far-field side (far: the grid has them and
// the node may touch one).
__device__ __forceinline__ double stored7(const DevParams& P, bool far, int x, int y, int z, int i, double f, double zeta) {
  using L = Lat<7>;
  if (far && leaves(P, P.far, x, y, z, L::c[i][0], L::c[i][1], L::c[i][2])) return 2.0 * L::w[i] * zeta - f;
  return f;
}
// Stored value of a flow population.  Velocity and pressure sides
// (non-equilibrium extrapolation, Sec. 3 boundary paragraph): the slot of
// population i leaving across one holds what the node pulls back along
// j = opp(i) next step, its own f*_j (opp) plus f^eq_j(p, rho, v_in) -
// f^eq_j(p, rho, v) (velocity side) or f^eq_j(0, rho, v) - f^eq_j(p, rho, v) =
// -w_j p / cs2 (pressure side); a velocity side takes precedence where both
// are crossed.
__device__ __forceinline__ double stored19(const DevParams& P, bool sides, int x, int y, int z, int i, double f, double opp,
                                           const Flow& o) {
  using L = Lat<19>;
  if (!sides) return f;
  const int dx = L::c[i][0], dy = L::c[i][1], dz = L::c[i][2], j = L::opp[i];
  if (leaves(P, P.vel, x, y, z, dx, dy, dz)) {
    double cb = 0.0, cv = 0.0, bb = 0.0, vv = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      cb += L::c[j][a] * P.vin[a];
      cv += L::c[j][a] * o.v[a];
      bb += P.vin[a] * P.vin[a];
      vv += o.v[a] * o.v[a];
    }
    return opp + o.rho * L::w[j] * ((cb - cv) * 3.0 + (cb * cb - cv * cv) * 4.5 - (bb - vv) * 1.5);
  }
  if (leaves(P, P.pres, x, y, z, dx, dy, dz)) return opp - L::w[j] * o.p * 3.0;
  return f;
}

// One macro plane k of the node at idx (put_macros writes them all).
__device__ __forceinline__ void put_macro(const DevParams& P, double* mout, long long idx, int k, double v) {
  if (!((P.mmask >> k) & 1u)) return;
  const long long at = (long long)__popc(P.mmask & ((1u << k) - 1u)) * P.N + idx;
  if (P.mf32) ((float*)mout)[at] = (float)v;
  else mout[at] = v;
}

// The column of a workgroup.
template <int R>
struct Column {
  using T = Col3<double>;
  int bx0, by0, z0, z1;
  bool fast_xy;
  __device__ __forceinline__ explicit Column(const DevParams& P) {
    const int gtx = (P.nx + T::TX - 1) / T::TX, gty = (P.ny + T::TY - 1) / T::TY;
    const int zc = P.zc, nch = (P.nz + zc - 1) / zc;
    const int lt = logical_tile(blockIdx.x, gtx * gty * nch);
    bx0 = (lt % gtx) * T::TX;
    by0 = ((lt / gtx) % gty) * T::TY;
    z0 = (lt / (gtx * gty)) * zc;
    z1 = z0 + zc < P.nz ? z0 + zc : P.nz;
    // pulls of every position the tile loads stay inside the domain in x and
    // y; at plane p they stay inside in z when 1 <= p <= nz - 2
    fast_xy = P.plane32 && bx0 >= R + 1 && by0 >= R + 1 && bx0 + T::TX + R + 1 <= P.nx && by0 + T::TY + R + 1 <= P.ny;
  }
  __device__ __forceinline__ bool fast(const DevParams& P, int p) const { return fast_xy && p >= 1 && p + 2 <= P.nz; }
  // node whose values tile position (tx, ty) of plane p holds
  __device__ __forceinline__ void source(const DevParams& P, bool f, int tx, int ty, int p, int (&g)[3]) const {
    g[0] = bx0 + tx;
    g[1] = by0 + ty;
    g[2] = p;
    if (!f) {
      g[0] = map_coord(g[0], P.nx, P.wall[0]);
      g[1] = map_coord(g[1], P.ny, P.wall[1]);
      g[2] = map_coord(g[2], P.nz, P.wall[2]);
    }
  }
  // tile position (in a plane with R2 rings) of ring position r: the R2 top
  // rows, the R2 bottom rows, then the side columns
  template <int R2>
  __device__ static __forceinline__ int ring_pos(int r) {
    using PL = Pl<double, R2>;
    if (r < R2 * PL::X) return r;
    if (r < 2 * R2 * PL::X) return (PL::Y - R2) * PL::X + (r - R2 * PL::X);
    const int q = r - 2 * R2 * PL::X, c = q % (2 * R2);
    return (R2 + q / (2 * R2)) * PL::X + (c < R2 ? c : PL::X - 2 * R2 + c);
  }
  // whether plane p's tile position (tx, ty) is a ghost across an odd number of
  // far-field sides: psi and U are odd there about psi_l = -1 and U = 0 (each
  // crossing mirrors once)
  __device__ __forceinline__ bool far_ghost(const DevParams& P, int tx, int ty, int p) const {
    const int gx = bx0 + tx, gy = by0 + ty;
    const bool fx = gx < 0 ? far_side(P, 0, true) : gx >= P.nx && far_side(P, 0, false);
    const bool fy = gy < 0 ? far_side(P, 1, true) : gy >= P.ny && far_side(P, 1, false);
    const bool fz = p < 0 ? far_side(P, 2, true) : p >= P.nz && far_side(P, 2, false);
    return fx ^ fy ^ fz;
  }
};

// Signs of D_phi and v0 at tile position (rx, ry) (ring-1 coordinates) of plane
// q, and the position m they are formed at: a ghost across a wall takes its
// mirror node's values, D (x) v0 odd across the wall (D takes minus the value
// once per wall crossed, v0 the value); across a symmetry plane the ghost is
// the mirror image (the normal components of D and v0 change sign).  flip_z: q
// is a ghost plane of a side in z.  Returns false beyond the first ghost.
template <bool SYM>
__device__ __forceinline__ bool dv_mirror(const DevParams& P, int bx0, int by0, int rx, int ry, int q, bool flip_z,
                                          int (&m)[2], double& sgn, double (&sc)[3]) {
  const int g[2] = {bx0 + rx - 1, by0 + ry - 1}, n[2] = {P.nx, P.ny};
  m[0] = rx;
  m[1] = ry;
  sgn = sc[0] = sc[1] = sc[2] = 1.0;
  bool ok = true;
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    if (P.wall[a] && (g[a] < 0 || g[a] >= n[a])) {
      if (g[a] == -1) m[a] += 1; else if (g[a] == n[a]) m[a] -= 1; else ok = false;
      if (SYM && sym_side(P, a, g[a] < 0)) sc[a] = -sc[a]; else sgn = -sgn;
    }
  }
  if (flip_z) {
    if (SYM && sym_side(P, 2, q < 0)) sc[2] = -sc[2]; else sgn = -sgn;
  }
  return ok;
}

// The mass-flux force of the own node at plane z is the divergence
// (1/cs2) sum_i w_i (c_i . D(x + c_i)) v0(x + c_i) over the planes z - 1, z,
// z + 1.  Each plane's D and v0 are in LDS once, right after they are
// formed; the own thread then adds that plane's terms to the sums of the
// nodes below (c_i,z = +1), at (c_i,z = 0) and above it (c_i,z = -1).
__device__ __forceinline__ void div_part(const double* s_D, const double* s_v0, int ly, int lx, double (&up)[3],
                                         double (&mid)[3], double (&dn)[3]) {
  using L = Lat<19>;
  using P1 = Pl<double, 1>;
#pragma unroll
  for (int b = 0; b < 3; ++b) up[b] = mid[b] = dn[b] = 0.0;
#pragma unroll
  for (int i = 1; i < 19; ++i) {
    const int q1 = P1::at(ly + 1 + L::c[i][1], lx + 1 + L::c[i][0]);
    double cD = 0.0;
    if (L::c[i][0]) cD += L::c[i][0] * s_D[q1];
    if (L::c[i][1]) cD += L::c[i][1] * s_D[P1::N + q1];
    if (L::c[i][2]) cD += L::c[i][2] * s_D[2 * P1::N + q1];
    const double wc = L::w[i] * cD;
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      const double term = wc * s_v0[b * P1::N + q1];
      if (L::c[i][2] > 0) up[b] += term;
      else if (L::c[i][2] < 0) dn[b] += term;
      else mid[b] += term;
    }
  }
}

// One node per thread; a thread holds its own node's moments from phase A (the
// pull) to the plane's phase C.  psi, C, theta and the flow are pulled one
// plane ahead (two planes held), phi two with the mass-flux force (three
// planes).  A population is pulled once; phase C reads only the history and
// the psi values of the time-stretched store.  At one wave per SIMD the kernel
// is bound by the latency of its loads, so those of a plane are issued
// together.  256^3 coupled: 5.50 ms with kept populations, 5.13 with moments,
// 5.08 with the flow quantities kept from phase B, 4.72 with the loads
// issued together.
template <int FIELDS, bool SYM, bool STREAM>
__global__ __launch_bounds__(Col3<double>::NT, FIELDS == 31 ? 1 : 2) void step3d_f64_kernel(const DevParams P, const double* __restrict__ fin,
                                                                        double* __restrict__ fout, double* hist,
                                                                        double* __restrict__ mout, int mode) {
  constexpr bool NS = FIELDS & F_NS, PHI = FIELDS & F_PHI, PSI = FIELDS & F_PSI;
  constexpr bool CC = FIELDS & F_C, TH = FIELDS & F_TH;
  constexpr bool FLOWX = NS && PHI;
  constexpr int R = FLOWX ? 2 : 1;
  constexpr int AHEAD = FLOWX ? 2 : 1;     // phi runs this many planes ahead
  constexpr int NT = Col3<double>::NT, TX = Col3<double>::TX;
  // general pulls by selects (256^3 coupled 4.67 -> 4.54 ms a step, 96^3 corner
  // 117 -> 111 us), but not for a flow without the bubble phase, which is faster
  // with branches (160 x 150^2 with psi and heat 463 us a step; selects 466).  The
  // FP32-compute forms, built with reassociation, would round differently.
  constexpr bool SEL = !NS || PHI;
  using ST = double;
  using PR = Pl<double, R>;
  using P1 = Pl<double, 1>;
  // LDS plane slots.  Phase C of plane t reads the psi and U planes t - 1, t,
  // t + 1 (and phi without the mass-flux force); phase A of plane t + 1, which a
  // thread may reach while others are still in that phase C (no barrier between
  // them), writes psi, U (phi) at t + 2.  With the mass-flux force phi is read
  // in phase B only, at t, t + 1, t + 2 (t - 1, t, t + 1 for the ghost plane
  // beyond a high side), which a barrier separates from the next phase A.
  constexpr int NPH = 4, NPS = 4;
  const KP<double>& K = P.kd;
  const ArgLines<double> args;

  __shared__ double s_phi[NPH * PR::N];
  __shared__ double s_psi[NPS * P1::N];
  __shared__ double s_U[CC ? NPS * P1::N : 1];
  __shared__ double s_j[NS ? 3 * P1::N : 1];
  // D_phi and v0 of the plane formed last, tile + ring 1: [component][position]
  __shared__ double s_D[FLOWX ? 3 * P1::N : 1];
  __shared__ double s_v0[FLOWX ? 3 * P1::N : 1];

  const int tid = threadIdx.x, lx = tid % TX, ly = tid / TX;
  const Column<R> col(P);
  const int x = col.bx0 + lx, y = col.by0 + ly;
  const bool own_xy = x < P.nx && y < P.ny;
  const long long N = P.N;
  const bool zwall = P.wall[2] != 0, first = P.first != 0;

  const double* fin_ns = fin + (size_t)(NS ? P.o_ns : 0) * (size_t)N;
  const double* fin_phi = fin + (size_t)(PHI ? P.o_phi : 0) * (size_t)N;
  const double* fin_psi = fin + (size_t)(PSI ? P.o_psi : 0) * (size_t)N;
  const double* fin_c = fin + (size_t)(CC ? P.o_c : 0) * (size_t)N;
  const double* fin_th = fin + (size_t)(TH ? P.o_th : 0) * (size_t)N;

  args.settle();
  ScMom ph0{}, ph1{}, ph2{};                // phi at planes t, t + 1, t + 2
  NsMom nsA{}, nsB{};                       // planes t (this step's phase C), t + 1
  ScMom psA{}, psB{}, cA{}, cB{}, thA{}, thB{};
  FlowKept flA{}, flB{};
  double rph[7], rps[7], rc[7], rns[19], rth[7];   // own populations of the plane being pulled

  // ---- phase A
  auto pull_phi = [&](int p) {
    if constexpr (PHI) {
      const bool fast = col.fast(P, p);
      int g[3];
      col.source(P, fast, lx, ly, p, g);
      pull3<7, ST, double, SYM, SEL>(fast, fin_phi, P, g[0], g[1], g[2], rph);
    }
  };
  auto pull_rest = [&](int p) {
    const bool fast = col.fast(P, p);
    int g[3];
    col.source(P, fast, lx, ly, p, g);
    auto all = [&](auto f) {
      constexpr bool F = decltype(f)::value;
      if constexpr (PSI) pull3<7, ST, double, SYM, SEL>(F, fin_psi, P, g[0], g[1], g[2], rps);
      if constexpr (CC) pull3<7, ST, double, SYM, SEL>(F, fin_c, P, g[0], g[1], g[2], rc);
      if constexpr (NS) pull3<19, ST, double, SYM, SEL>(F, fin_ns, P, g[0], g[1], g[2], rns);
      if constexpr (TH) pull3<7, ST, double, SYM, SEL>(F, fin_th, P, g[0], g[1], g[2], rth);
    };
    if (fast) all(std::true_type{});
    else all(std::false_type{});
  };
  auto own_phi = [&](int p) {
    if constexpr (PHI) sc_moments(rph, ph2);
    s_phi[ring_slot(p, NPH) * PR::N + PR::at(ly + R, lx + R)] = PHI ? ph2.d : 1.0;
  };
  // the ring positions of phi go to the last threads, those of the others to
  // the first, so that few waves do both
  auto ring_phi = [&](int p) {
    const bool fast = col.fast(P, p);
    double* dst = s_phi + ring_slot(p, NPH) * PR::N;
    for (int r = NT - 1 - tid; r < PR::N - NT; r += NT) {
      const int k = Column<R>::template ring_pos<R>(r);
      double phi = 1.0;
      if constexpr (PHI) {
        int g[3];
        col.source(P, fast, k % PR::X - R, k / PR::X - R, p, g);
        double f[7];
        pull3<7, ST, double, SYM, SEL>(fast, fin_phi, P, g[0], g[1], g[2], f);
        phi = sc_sum(f);
      }
      dst[k] = phi;
    }
  };
  auto put_rest = [&](int p, int k, double psi, double C, const double (&j)[3]) {
    double U = CC ? u_of(K, psi, C) : K.U0;
    if (SYM && P.far && !col.fast(P, p) && col.far_ghost(P, k % P1::X - 1, k / P1::X - 1, p)) {
      psi = -2.0 - psi;
      U = -U;
    }
    const int at = ring_slot(p, NPS) * P1::N + k;
    s_psi[at] = psi;
    if constexpr (CC) s_U[at] = U;
    if constexpr (NS) {
#pragma unroll
      for (int a = 0; a < 3; ++a) s_j[a * P1::N + k] = j[a];
    }
  };
  auto own_rest = [&](int p) {
    if constexpr (PSI) sc_moments(rps, psB);
    if constexpr (CC) sc_moments(rc, cB);
    if constexpr (TH) sc_moments(rth, thB);
    if constexpr (NS) ns_moments(rns, nsB);
    put_rest(p, P1::at(ly + 1, lx + 1), PSI ? psB.d : -1.0, cB.d, nsB.j);
  };
  auto ring_rest = [&](int p) {
    const bool fast = col.fast(P, p);
    for (int r = tid; r < P1::N - NT; r += NT) {
      const int k = Column<R>::template ring_pos<1>(r);
      int g[3];
      col.source(P, fast, k % P1::X - 1, k / P1::X - 1, p, g);
      double fp[7], fc[7], fn[19], j[3] = {0.0, 0.0, 0.0};
      auto all = [&](auto f) {
        constexpr bool F = decltype(f)::value;
        if constexpr (PSI) pull3<7, ST, double, SYM, SEL>(F, fin_psi, P, g[0], g[1], g[2], fp);
        if constexpr (CC) pull3<7, ST, double, SYM, SEL>(F, fin_c, P, g[0], g[1], g[2], fc);
        if constexpr (NS) pull3<19, ST, double, SYM, SEL>(F, fin_ns, P, g[0], g[1], g[2], fn);
      };
      if (fast) all(std::true_type{});
      else all(std::false_type{});
      if constexpr (NS) ns_momentum(fn, j);
      double psi = -1.0, C = 0.0;
      if constexpr (PSI) psi = sc_sum(fp);
      if constexpr (CC) C = sc_sum(fc);
      put_rest(p, k, psi, C, j);
    }
  };
  auto phi_planes = [&](int p, const double* pl[3]) {
#pragma unroll
    for (int c = 0; c < 3; ++c) pl[c] = s_phi + ring_slot(p - 1 + c, NPH) * PR::N;
  };
  // ---- phase B: D_phi and v0 of plane q on the tile and ring 1, from the
  // flow quantities at plane m (q itself, or the plane q mirrors in z)
  auto form_dv = [&](int q, int m, bool flip_z) {
    const double* ph[3];
    phi_planes(m, ph);
    const double* ps = s_psi + ring_slot(m, NPS) * P1::N;
    constexpr int NPASS = 1 + (P1::N - NT + NT - 1) / NT;
#pragma unroll 1
    for (int it = 0; it < NPASS; ++it) {
      const int r = tid + (it - 1) * NT;
      if (it > 0 && r >= P1::N - NT) break;
      const int k = it == 0 ? P1::at(ly + 1, lx + 1) : Column<R>::template ring_pos<1>(r);
      int mm[2];
      double sgn, sc[3], D[3] = {0.0, 0.0, 0.0}, v0[3] = {0.0, 0.0, 0.0};
      if (dv_mirror<SYM>(P, col.bx0, col.by0, k % P1::X, k / P1::X, q, flip_z, mm, sgn, sc)) {
        const int at = P1::at(mm[1], mm[0]);
        const double phi = ph[1][PR::at(mm[1] + R - 1, mm[0] + R - 1)], psi = ps[at];
        const double j[3] = {s_j[at], s_j[P1::N + at], s_j[2 * P1::N + at]};
        FlowKept f;
        flow_kept<NS, PHI, R>(K, ph, phi, psi, mm[1], mm[0], f);
        dv_of(K, f, phi, psi, j, D, v0);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          D[a] *= sgn * sc[a];
          v0[a] *= sc[a];
        }
        if (it == 0) flB = f;
      }
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        s_D[a * P1::N + k] = D[a];
        s_v0[a * P1::N + k] = v0[a];
      }
    }
  };
  double dv_t[3] = {0.0, 0.0, 0.0}, dv_t1[3] = {0.0, 0.0, 0.0};   // divergence sums at planes t, t + 1

  // phi planes z0 - 2, z0 - 1 before the march when phi runs two planes ahead
  if constexpr (FLOWX) {
    for (int p = col.z0 - 2; p < col.z0; ++p) {
      pull_phi(p);
      ring_phi(p);
      own_phi(p);
    }
    ph1 = ph2;
  }
  for (int t = col.z0 - 2; t < col.z1; ++t) {
    // history, grain id and the stored psi of the time-stretched store of the
    // own node at plane t: issued first, used in phase C
    const long long idx = ((long long)t * P.ny + y) * P.nx + x;
    const uint32_t byte = (uint32_t)idx * 8u;
    const bool stepped = t >= col.z0 && own_xy;
    double h_psi = 0.0, h_S = 0.0, h_pv[3] = {0.0, 0.0, 0.0}, h_B[3] = {0.0, 0.0, 0.0}, h_Hv[3] = {0.0, 0.0, 0.0}, old[7];
    int gid = 0;
    if (stepped) {
      const double* hsrc = P.hist_src ? (const double*)P.hist_src : hist;
      auto hld = [&](int plane) -> double {
        if (P.plane32) return *(const double*)((const char*)(hsrc + (size_t)plane * (size_t)N) + byte);
        return hsrc[(long long)plane * N + idx];
      };
      if (PSI) gid = P.grain[idx];
      if (mode == 0) {
        if constexpr (PSI) {
#pragma unroll
          for (int i = 0; i < 7; ++i) old[i] = fin_psi[idx + (long long)i * N];
        }
        if (!first) {
          if constexpr (PSI) { h_psi = hld(P.h_psi); h_S = hld(P.h_S); }
#pragma unroll
          for (int a = 0; a < 3; ++a) {
            if constexpr (PHI) h_pv[a] = hld(P.h_phiv + a);
            if constexpr (CC) h_B[a] = hld(P.h_B + a);
            if constexpr (TH) h_Hv[a] = hld(P.h_Hv + a);
          }
        }
      }
    }
    pull_phi(t + AHEAD);
    pull_rest(t + 1);
    ring_phi(t + AHEAD);
    ring_rest(t + 1);
    own_phi(t + AHEAD);
    own_rest(t + 1);
    __syncthreads();
    double dv_t2[3] = {0.0, 0.0, 0.0};       // the own node at plane t + 2
    if constexpr (FLOWX) {
      const int q = t + 1;
      double up[3], mid[3], dn[3];
      if (zwall && q == 0) {
        // the ghost plane -1 (plane t): its terms reach plane t + 1 = 0
        form_dv(-1, 0, true);
        __syncthreads();
        if (own_xy) {
          div_part(s_D, s_v0, ly, lx, up, mid, dn);
#pragma unroll
          for (int b = 0; b < 3; ++b) dv_t1[b] += dn[b];
        }
        __syncthreads();
      }
      if (!zwall || (q >= 0 && q < P.nz)) form_dv(q, q, false);   // a ghost plane waits for its mirror
      if (zwall && q == P.nz) form_dv(q, P.nz - 1, true);
      __syncthreads();
      if (own_xy && (!zwall || (q >= 0 && q <= P.nz))) {
        div_part(s_D, s_v0, ly, lx, up, mid, dn);
#pragma unroll
        for (int b = 0; b < 3; ++b) {
          dv_t[b] += up[b];
          dv_t1[b] += mid[b];
          dv_t2[b] = dn[b];
        }
      }
    }
    // ---- phase C: the rest of the step at the own node of plane t
    if (stepped) {
      auto node = [&]() {
        const bool fast = col.fast(P, t);
        const bool far = SYM && !fast && P.far, nee = SYM && !fast && (P.vel | P.pres);
        const double phi = PHI ? ph0.d : 1.0, psi = PSI ? psA.d : -1.0, C = cA.d, H = thA.d;
        const double h = (psi + 1.0) * 0.5;
        const double U = CC ? u_of(K, psi, C) : K.U0;
        double theta = K.theta0, s_th = K.s_th;
        if constexpr (TH) heat_of(K, phi, h, H, theta, s_th);
        const FlowPoint fp = flow_point(K, phi, psi);
        if constexpr (!FLOWX) {
          const double* ph[3];
          phi_planes(t, ph);
          flow_kept<NS, PHI, R>(K, ph, phi, psi, ly + 1, lx + 1, flA);
        }
        const double n[3] = {flA.g[0] * flA.inv, flA.g[1] * flA.inv, flA.g[2] * flA.inv};
        Flow fl{};
        if constexpr (NS) flow_node_state(K, nsA, flA, fp, dv_t, fl);
        if (mode == 1) {
          const double m9[9] = {phi, psi, C, theta, U, fl.p, fl.v[0], fl.v[1], fl.v[2]};
          put_macros(P, mout, idx, m9);
          return;
        }
        double gp[3] = {0.0, 0.0, 0.0}, gU[3] = {0.0, 0.0, 0.0};
        const double* psp[3];
        const double* Up[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          psp[c] = s_psi + ring_slot(t - 1 + c, NPS) * P1::N;
          Up[c] = s_U + (CC ? ring_slot(t - 1 + c, NPS) * P1::N : 0);
        }
        if constexpr (PSI) grad19p<double, P1>(psp, ly + 1, lx + 1, gp);
        if constexpr (CC) grad19p<double, P1>(Up, ly + 1, lx + 1, gU);
        PsiNode pn{};
        if constexpr (PSI || CC)
          psi_node(P, K, gp, gU, P.grain_cs[2 * gid], P.grain_cs[2 * gid + 1], phi, psi, theta, U, pn);

        // one address form for every grid: a uniform plane base and one 64-bit
        // shift-add per store (a run-time choice of a 32-bit byte offset keeps
        // both forms in registers: psi + C + theta 215 -> 286)
        auto st = [&](int plane, double v) {
          put<STREAM, double>(fout + (long long)plane * N + idx, v);
        };
        auto hst = [&](int plane, double v) {
          put<STREAM, double>(hist + (long long)plane * N + idx, v);
        };
        if constexpr (NS)
          collide_ns(K, nsA, fl, phi, [&](int i, double f, double opp) {
            st(P.o_ns + i, stored19(P, nee, x, y, t, i, f, opp, fl));
          });
        if constexpr (PHI) {
          const double phiv[3] = {phi * fl.v[0], phi * fl.v[1], phi * fl.v[2]};
          collide_phi(K, ph0, phiv, first ? phiv : h_pv, fp.sharp, n, [&](int i, double f) { st(P.o_phi + i, f); });
#pragma unroll
          for (int a = 0; a < 3; ++a) hst(P.h_phiv + a, phiv[a]);
        }
        if constexpr (PSI) {
          // time-stretched store: the population i at x + c_i before this step is the
          // stored value of plane i at x itself (pull form; across a side it is the
          // own f_opp(i), pulled from that same slot)
          const double inv_an = rcp(pn.an);
          collide_psi(P, psA, pn, first ? pn.S : h_S, [&](int i, double f) {
            st(P.o_psi + i, (stored7(P, far, x, y, t, i, f, -1.0) - (1.0 - pn.an) * old[i]) * inv_an);
          });
        }
        if constexpr (CC) {
          const double q = clamp01((1.0 - psi) * 0.5), om = 1.0 - phi;
          const double at = -K.aW0 * pn.a_s * pn.lin * (psi - (first ? psi : h_psi));
          const double DqC = K.D * q * C;
          const double jv = DqC * K.sharp * (om > 0.0 ? om : 0.0);
          const double invm = rcp(1.0 - K.k1 * h);
          const double dr = DqC * K.k1 * invm * invm * 0.5;
          double B[3], dB[3];
#pragma unroll
          for (int a = 0; a < 3; ++a) {
            B[a] = C * fl.v[a] - dr * gp[a] + K.k1 * (at * gp[a] * pn.invp + jv * n[a]);
            dB[a] = B[a] - (first ? B[a] : h_B[a]);
          }
          const double s1 = rcp(K.D * q * invm * (1.0 / Lat<7>::cs2) + 0.5);
          collide_flux(W7_0 * C, W7_1 * C, cA, B, dB, s1, [&](int i, double f) {
            st(P.o_c + i, stored7(P, far, x, y, t, i, f, 1.0));
          });
#pragma unroll
          for (int a = 0; a < 3; ++a) hst(P.h_B + a, B[a]);
        }
        if constexpr (TH) {
          double Hv[3], dHv[3];
#pragma unroll
          for (int a = 0; a < 3; ++a) {
            Hv[a] = H * fl.v[a];
            dHv[a] = Hv[a] - (first ? Hv[a] : h_Hv[a]);
          }
          // H (the sum of g) is rho times the model's H: the rest equilibrium is
          // rho H + (w - 1) theta
          collide_flux(H + (W7_0 - 1.0) * theta, W7_1 * theta, thA, Hv, dHv, s_th, [&](int i, double f) {
            st(P.o_th + i, stored7(P, far, x, y, t, i, f, K.theta0));
          });
#pragma unroll
          for (int a = 0; a < 3; ++a) hst(P.h_Hv + a, Hv[a]);
        }
        if constexpr (PSI) {
          hst(P.h_psi, psi);
          hst(P.h_S, pn.S);
        }
      };
      node();
    }
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      dv_t[b] = dv_t1[b];
      dv_t1[b] = dv_t2[b];
    }
    if constexpr (FLOWX) { ph0 = ph1; ph1 = ph2; }
    else ph0 = ph2;
    flA = flB;
    nsA = nsB;
    psA = psB;
    cA = cB;
    thA = thB;
    // no barrier here: the next phase A writes slots this phase C does not
    // read (the slot counts above), the D_phi/v0 plane is read before the
    // barrier after phase B, and the momentum plane only in phase B
  }
}

template <int FIELDS, bool SYM, bool STREAM>
hipError_t launch_step3d_f64_k(const DevParams& Pc, const void* fin, void* fout, void* hist, double* mout, int mode,
                               hipStream_t s) {
  using T = Col3<double>;
  const auto kernel = step3d_f64_kernel<FIELDS, SYM, STREAM>;
  static const int per_cu = blocks_per_cu(kernel, T::NT);
  DevParams P = Pc;
  const long long cols = (long long)((P.nx + T::TX - 1) / T::TX) * ((P.ny + T::TY - 1) / T::TY);
  if (P.zc <= 0) P.zc = chunk_planes(cols, P.nz, (long long)P.cus * per_cu);
  const long long tiles = cols * ((P.nz + P.zc - 1) / P.zc);
  hipLaunchKernelGGL(kernel, dim3((unsigned)tiles), dim3(T::NT), 0, s, P, (const double*)fin, (double*)fout,
                     (double*)hist, mout, mode);
  return hipGetLastError();
}

template <int FIELDS>
hipError_t launch_step3d_f64(const DevParams& P, const void* fin, void* fout, void* hist, double* mout, int mode,
                             hipStream_t s) {
  const bool sym = P.sym || P.far;
  if (sym && P.nt) return launch_step3d_f64_k<FIELDS, true, true>(P, fin, fout, hist, mout, mode, s);
  if (sym) return launch_step3d_f64_k<FIELDS, true, false>(P, fin, fout, hist, mout, mode, s);
  if (P.nt) return launch_step3d_f64_k<FIELDS, false, true>(P, fin, fout, hist, mout, mode, s);
  return launch_step3d_f64_k<FIELDS, false, false>(P, fin, fout, hist, mout, mode, s);
}

}  // namespace

}  // namespace pfl
