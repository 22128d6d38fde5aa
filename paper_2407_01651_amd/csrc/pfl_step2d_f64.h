// Fused 2D time step in FP64 (the parity form): one launch advances every
// active population set by one step.  The scheme, the tiles and the phases
// are the FP32-compute step's (pfl_step2d_impl.h): moments of a tile and its
// halo in LDS, D_phi (x) v0 on the tile and one ring, the rest of the step at
// the own node.
//
// What differs is what a thread holds between the phases: not its node's
// populations but the moments the collisions need (five of the nine flow
// populations, three of each five), and the stored psi populations of the
// time-stretched store come from memory, where the tile's pulls have just
// brought them, instead of five LDS planes.  (The FP32-compute forms are
// built with reassociation, so that any change of their source changes their
// rounding; they keep populations.)
#pragma once
#include "pfl_kernels.h"
#include "pfl_step2d.h"

namespace pfl {

namespace {

// Moments of a node's flow populations: momentum, the traceless stresses
// c_x^2 - c_y^2 and c_x c_y, the sum of the moving populations; of a scalar
// set: sum and flux.
struct NsMom2 {
  double j[2], s1, s2, sum;
};
struct ScMom2 {
  double d, J[2];
};
__device__ __forceinline__ void ns_momentum2(const double (&f)[9], double (&j)[2]) {
  using L = Lat<9>;
  j[0] = j[1] = 0.0;
#pragma unroll
  for (int i = 1; i < 9; ++i) {
    if (L::c[i][0]) j[0] += L::c[i][0] * f[i];
    if (L::c[i][1]) j[1] += L::c[i][1] * f[i];
  }
}
__device__ __forceinline__ void ns_moments2(const double (&f)[9], NsMom2& m) {
  using L = Lat<9>;
  ns_momentum2(f, m.j);
  m.s1 = m.s2 = m.sum = 0.0;
#pragma unroll
  for (int i = 1; i < 9; ++i) {
    const int cx = L::c[i][0], cy = L::c[i][1];
    m.sum += f[i];
    if (cx * cx != cy * cy) m.s1 += (double)(cx * cx - cy * cy) * f[i];
    if (cx * cy) m.s2 += (double)(cx * cy) * f[i];
  }
}
template <int Q>
__device__ __forceinline__ double sc_sum2(const double (&f)[Q]) {
  double d = 0.0;
#pragma unroll
  for (int i = 0; i < Q; ++i) d += f[i];
  return d;
}
template <int Q>
__device__ __forceinline__ void sc_moments2(const double (&f)[Q], ScMom2& m) {
  using L = Lat<Q>;
  m.d = sc_sum2<Q>(f);
  m.J[0] = m.J[1] = 0.0;
#pragma unroll
  for (int i = 1; i < Q; ++i) {
    if (L::c[i][0]) m.J[0] += L::c[i][0] * f[i];
    if (L::c[i][1]) m.J[1] += L::c[i][1] * f[i];
  }
}

// Collision of a scalar set that relaxes its flux moments, in even and odd parts
// of opposite populations: put(0, rest), and for c_i and its opposite
// w_i even +- c_i.F, with F the flux over the set's squared norm: for any vector
// A, w_i c_i.A / cs2 has flux A, so an equilibrium flux E and a flux deviation D
// give w_i c_i.E / cs2 + c_i.D / norm.
template <int Q, class Put>
__device__ __forceinline__ void put_set(double rest, double even, const double (&E)[2], const double (&D)[2], Put&& put) {
  using L = Lat<Q>;
  put(0, rest);
#pragma unroll
  for (int i = 1; i < Q; ++i) {
    if (L::opp[i] < i) continue;
    const double cE = L::c[i][0] * E[0] + L::c[i][1] * E[1], cD = L::c[i][0] * D[0] + L::c[i][1] * D[1];
    const double e = L::w[i] * even, o = (L::w[i] / L::cs2) * cE + (1.0 / L::flux_norm) * cD;
    put(i, e + o);
    put(L::opp[i], e - o);
  }
}

// One thread per node of the tile (StepTile).  Large grids are bound by HBM at
// the waves the registers allow, small ones by the chain of latencies from the
// pulls to the stores, so a thread issues its own pulls and its halo
// position's together.  The choice between the interior and the general form of
// the pulls is made once around them all: made for each set, the compiler waits
// for one set's loads before it issues the next one's (registers of the form
// not taken), and the kernel takes 165 VGPRs instead of 139.  With the crystal
// angle read ahead of the barriers: 128^2 coupled 10.9 -> 8.9 us a step, 200 x
// 400 column 18.1 -> 16.9, 500 x 333 coupled 21.1 -> 18.9, 2048^2 548 -> 540.
template <int FIELDS, int QP, bool SYM, bool STREAM>
__global__ __launch_bounds__((StepTile<FIELDS, double>::N))
void step2d_f64_kernel(const DevParams P, const double* __restrict__ fin, double* __restrict__ fout, double* hist,
                       double* __restrict__ mout, int mode) {
  constexpr bool NS = FIELDS & F_NS, PHI = FIELDS & F_PHI, PSI = FIELDS & F_PSI;
  constexpr bool CC = FIELDS & F_C, TH = FIELDS & F_TH;
  constexpr bool FLOWX = NS && PHI;          // mass-flux force needs D_phi (x) v0 on ring 1
  constexpr int R = FLOWX ? 2 : 1;
  constexpr int STX = StepTile<FIELDS, double>::X, STY = StepTile<FIELDS, double>::Y, SNT = STX * STY;
  constexpr int RX = STX + 2 * R, RY = STY + 2 * R;
  using ST = double;
  using LN = Lat<9>;
  using LS = Lat<5>;
  using LP = Lat<QP>;
  // The time-stretched store needs f_i(x + c_i) from before the step.  In pull
  // form that is the stored value of plane i at x itself (across a side it is
  // the own f_opp(i), pulled from that same slot).  With the mass-flux force the
  // kernel loads it again, from lines its pulls have just brought, since LDS
  // bounds the workgroups on a unit (2048^2 coupled: 1183 -> 1098 us for two
  // steps); the others, with LDS to spare, take it from the tile's pulled
  // populations (2048^2 psi + C 873 -> 823 us for four).
  constexpr bool OLDS = PSI && !FLOWX;
  const KP<double>& K = P.kd;
  const ArgLines<double> args;

  __shared__ double s_phi[RY][RX];
  __shared__ double s_psi[RY][RX];
  __shared__ double s_U[CC ? RY : 1][CC ? RX : 1];
  __shared__ double s_jx[NS ? RY : 1][NS ? RX : 1];
  __shared__ double s_jy[NS ? RY : 1][NS ? RX : 1];
  // psi populations of the tile and ring 1 (see OLDS)
  __shared__ double s_fps[OLDS ? 5 : 1][OLDS ? RY : 1][OLDS ? RX : 1];
  __shared__ double s_X[FLOWX ? 4 : 1][FLOWX ? RY : 1][FLOWX ? RX : 1];

  const int tid = threadIdx.x;
  const int lx = tid % STX, ly = tid / STX;
  const int gtx = (P.nx + STX - 1) / STX;
  const int lt = logical_tile(blockIdx.x, gtx * ((P.ny + STY - 1) / STY));
  const int bx0 = (lt % gtx) * STX, by0 = (lt / gtx) * STY;
  const int x = bx0 + lx, y = by0 + ly;
  const bool own = x < P.nx && y < P.ny;
  const long long N = P.N, idx = (long long)y * P.nx + x;
  // every pull of the tile and its halo stays inside the domain
  const bool fast = P.fast && bx0 >= R + 1 && by0 >= R + 1 && bx0 + STX + R + 1 <= P.nx && by0 + STY + R + 1 <= P.ny;
  const bool first = P.first != 0;
  const int ry = ly + R, rx = lx + R;

  const double* fin_ns = fin + (long long)(NS ? P.o_ns : 0) * N;
  const double* fin_phi = fin + (long long)(PHI ? P.o_phi : 0) * N;
  const double* fin_psi = fin + (long long)(PSI ? P.o_psi : 0) * N;
  const double* fin_c = fin + (long long)(CC ? P.o_c : 0) * N;
  const double* fin_th = fin + (long long)(TH ? P.o_th : 0) * N;

  // ---- phase A: moments of the tile and its halo.  Positions past the domain
  // hold the node they map to; across an odd number of far-field sides psi and U
  // are odd about psi_l = -1 and U = 0 (each crossing mirrors once).
  auto put_node = [&](int py, int px, double phi, double psi, double C, double jx, double jy, bool ring1) {
    s_phi[py][px] = phi;
    if (!ring1) return;
    double U = 0.0;
    if constexpr (CC) U = (C * rcp(1.0 - K.k1 * ((psi + 1.0) * 0.5)) - 1.0) * K.inv_k1;
    if (SYM && !fast && P.far) {
      const int gx = bx0 + px - R, gy = by0 + py - R;
      const bool fx = gx < 0 ? far_side(P, 0, true) : gx >= P.nx && far_side(P, 0, false);
      const bool fy = gy < 0 ? far_side(P, 1, true) : gy >= P.ny && far_side(P, 1, false);
      if (fx != fy) {
        psi = -2.0 - psi;
        U = -U;
      }
    }
    s_psi[py][px] = psi;
    if constexpr (CC) s_U[py][px] = U;
    if constexpr (NS) {
      s_jx[py][px] = jx;
      s_jy[py][px] = jy;
    }
  };
  NsMom2 mn{};
  ScMom2 mph{}, mps{}, mc{}, mth{};
  int gid = 0;
  auto phase_a = [&](auto interior) {
    constexpr bool IN = decltype(interior)::value;
    int gx = x, gy = y;
    if constexpr (!IN) {
      gx = map_coord(x, P.nx, P.wall[0]);
      gy = map_coord(y, P.ny, P.wall[1]);
    }
    double fn[9], fph[QP], fps[5], fc[5], fth[5];
    if constexpr (PSI) gid = P.grain[(long long)gy * P.nx + gx];
    if constexpr (PHI) pull<QP, ST, double, SYM>(IN, fin_phi, P, gx, gy, fph);
    if constexpr (NS) pull<9, ST, double, SYM>(IN, fin_ns, P, gx, gy, fn);
    if constexpr (PSI) pull<5, ST, double, SYM>(IN, fin_psi, P, gx, gy, fps);
    if constexpr (CC) pull<5, ST, double, SYM>(IN, fin_c, P, gx, gy, fc);
    if constexpr (TH) pull<5, ST, double, SYM>(IN, fin_th, P, gx, gy, fth);
    constexpr int NH = RX * RY - SNT;
    for (int k = tid; k < NH; k += SNT) {
      int px, py;
      halo_pos<R, STX, STY>(k, px, py);
      const bool ring1 = px >= R - 1 && px <= RX - R && py >= R - 1 && py <= RY - R;
      int hx = bx0 + px - R, hy = by0 + py - R;
      if constexpr (!IN) {
        hx = map_coord(hx, P.nx, P.wall[0]);
        hy = map_coord(hy, P.ny, P.wall[1]);
      }
      double phi = 1.0, psi = -1.0, C = 0.0, j[2] = {0.0, 0.0};
      double hph[QP], hps[5], hc[5], hn[9];
      if constexpr (PHI) pull<QP, ST, double, SYM>(IN, fin_phi, P, hx, hy, hph);
      if (ring1) {
        if constexpr (PSI) pull<5, ST, double, SYM>(IN, fin_psi, P, hx, hy, hps);
        if constexpr (CC) pull<5, ST, double, SYM>(IN, fin_c, P, hx, hy, hc);
        if constexpr (NS) pull<9, ST, double, SYM>(IN, fin_ns, P, hx, hy, hn);
        if constexpr (PSI) psi = sc_sum2<5>(hps);
        if constexpr (OLDS) {
#pragma unroll
          for (int i = 0; i < 5; ++i) s_fps[i][py][px] = hps[i];
        }
        if constexpr (CC) C = sc_sum2<5>(hc);
        if constexpr (NS) ns_momentum2(hn, j);
      }
      if constexpr (PHI) phi = sc_sum2<QP>(hph);
      put_node(py, px, phi, psi, C, j[0], j[1], ring1);
    }
    if constexpr (PHI) sc_moments2<QP>(fph, mph);
    if constexpr (NS) ns_moments2(fn, mn);
    if constexpr (PSI) sc_moments2<5>(fps, mps);
    if constexpr (OLDS) {
#pragma unroll
      for (int i = 0; i < 5; ++i) s_fps[i][ry][rx] = fps[i];
    }
    if constexpr (CC) sc_moments2<5>(fc, mc);
    if constexpr (TH) sc_moments2<5>(fth, mth);
    put_node(ry, rx, PHI ? mph.d : 1.0, PSI ? mps.d : -1.0, mc.d, mn.j[0], mn.j[1], true);
  };
  args.settle();
  if (fast) phase_a(std::true_type{});
  else phase_a(std::false_type{});
  // history, the grain's angle and the stored psi of the time-stretched store:
  // issued before the barriers, used after them
  double h_psi = 0.0, h_S = 0.0, h_pv[2] = {0.0, 0.0}, h_B[2] = {0.0, 0.0}, h_Hv[2] = {0.0, 0.0}, old[5];
  double cth = 1.0, sth = 0.0;
  if constexpr (PSI || CC) {
    cth = P.grain_cs[2 * gid];
    sth = P.grain_cs[2 * gid + 1];
  }
  if (own) {
    const double* hsrc = (P.hist_src ? (const double*)P.hist_src : hist) + idx;
    if (mode == 0) {
      if constexpr (PSI && !OLDS) {
#pragma unroll
        for (int i = 0; i < 5; ++i) old[i] = fin_psi[(long long)i * N + idx];
      }
      if (!first) {
        if constexpr (PSI) { h_psi = hsrc[(long long)P.h_psi * N]; h_S = hsrc[(long long)P.h_S * N]; }
#pragma unroll
        for (int a = 0; a < 2; ++a) {
          if constexpr (PHI) h_pv[a] = hsrc[(long long)(P.h_phiv + a) * N];
          if constexpr (CC) h_B[a] = hsrc[(long long)(P.h_B + a) * N];
          if constexpr (TH) h_Hv[a] = hsrc[(long long)(P.h_Hv + a) * N];
        }
      }
    }
  }
  __syncthreads();

  // ---- phase B: D_phi (x) v0 on the tile and ring 1 (mass-flux force).  Ghosts
  // across a wall take minus the value at their mirror node; across a symmetry
  // plane the mirror image: the off-diagonal components (one index along the
  // normal) change sign.
  FlowNode<double> fo;
  if constexpr (FLOWX) {
    auto form_X = [&](int py, int px, FlowNode<double>& h) {
      const int g[2] = {bx0 + px - R, by0 + py - R}, n[2] = {P.nx, P.ny};
      int m[2] = {px, py};
      double sgn = 1.0, sod = 1.0;
      bool ok = true;
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        if (P.wall[a] && (g[a] < 0 || g[a] >= n[a])) {
          if (g[a] == -1) m[a] += 1; else if (g[a] == n[a]) m[a] -= 1; else ok = false;
          if (SYM && sym_side(P, a, g[a] < 0)) sod = -sod; else sgn = -sgn;
        }
      }
      double X[4] = {0.0, 0.0, 0.0, 0.0};
      if (ok) {
        flow_node<NS, PHI, double, RX>(K, s_phi, s_psi, s_jx, s_jy, m[1], m[0], h);
        X[0] = sgn * h.Dx * h.v0x;
        X[1] = sgn * sod * h.Dx * h.v0y;
        X[2] = sgn * sod * h.Dy * h.v0x;
        X[3] = sgn * h.Dy * h.v0y;
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) s_X[c][py][px] = X[c];
    };
    form_X(ry, rx, fo);
    for (int k = tid; k < (STX + 2) * (STY + 2) - SNT; k += SNT) {
      int px, py;
      halo_pos<1, STX, STY>(k, px, py);
      FlowNode<double> h;
      form_X(py + R - 1, px + R - 1, h);
    }
    __syncthreads();
  } else {
    if (own) flow_node<NS, PHI, double, RX>(K, s_phi, s_psi, s_jx, s_jy, ry, rx, fo);
  }
  if (!own) return;

  // ---- phase C: the rest of the step at the own node
  const double phi = PHI ? mph.d : 1.0, psi = PSI ? mps.d : -1.0, C = mc.d, H = mth.d;
  const double h = (psi + 1.0) * 0.5;
  double U = K.U0;
  if constexpr (CC) U = (C * rcp(1.0 - K.k1 * h) - 1.0) * K.inv_k1;
  // temperature: H = c_p theta - c_p^s h with sum g = rho H; rho, c_p, k_T
  // linear in phi between gas and liquid (liquid = solid = 1); s_th the heat
  // relaxation rate from k_T
  double theta = K.theta0, s_th = K.s_th;
  if constexpr (TH) {
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
  double gp[2] = {0.0, 0.0}, gU[2] = {0.0, 0.0};
  if constexpr (PSI) grad9<double, RX>(s_psi, ry, rx, gp[0], gp[1]);
  if constexpr (CC) grad9<double, RX>(s_U, ry, rx, gU[0], gU[1]);

  // velocity, forces, pressure
  double v[2] = {0.0, 0.0}, F[2] = {0.0, 0.0}, gr[2] = {0.0, 0.0}, Fm[2] = {0.0, 0.0}, p = 0.0;
  const double rho = fo.rho;
  if constexpr (NS) {
    if constexpr (FLOWX) {
      // (div X)_b = 3 sum_i w_i sum_a c_ia X_ab(x + c_i), X = D (x) v0
      constexpr double w1 = 1.0 / 9, w2 = 1.0 / 36;
      auto Xs = [&](int c, int dy, int dx) { return s_X[c][ry + dy][rx + dx]; };
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        // a = x components (X0: D_x v0_x, X1: D_x v0_y); a = y (X2, X3)
        const double ax = w1 * (Xs(b, 0, 1) - Xs(b, 0, -1)) +
                          w2 * ((Xs(b, 1, 1) - Xs(b, 1, -1)) + (Xs(b, -1, 1) - Xs(b, -1, -1)));
        const double ay = w1 * (Xs(2 + b, 1, 0) - Xs(2 + b, -1, 0)) +
                          w2 * ((Xs(2 + b, 1, 1) + Xs(2 + b, 1, -1)) - (Xs(2 + b, -1, -1) + Xs(2 + b, -1, 1)));
        Fm[b] = K.drho * 3.0 * (ax + ay);
      }
    }
    const double Fs[2] = {fo.Fsx, fo.Fsy}, Fb[2] = {0.0, -(rho - K.rho_l) * K.g};
    const double onechi = 1.0 - fo.chi, irho = rcp(rho);
    gr[0] = K.drho * fo.gx;
    gr[1] = K.drho * fo.gy;
    double vv = 0.0, vg = 0.0;
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const double rv = mn.j[a] + 0.5 * (Fs[a] + Fb[a] + Fm[a]);
      v[a] = onechi * rv * irho;
      F[a] = Fs[a] + Fb[a] + Fm[a] - 2.0 * fo.chi * rv;
      vv += v[a] * v[a];
      vg += v[a] * gr[a];
    }
    p = LN::cs2 / (1.0 - LN::w[0]) * (mn.sum + 0.5 * vg - rho * (LN::w[0] * 1.5 * vv));
  }

  // the step's stencil results, for an adjoint sweep that does not redo them
  if (P.tape) {
    double* t = (double*)P.tape + idx;
    const double tv[TAPE_PLANES] = {fo.gx, fo.gy, fo.lap, gp[0], gp[1], gU[0], gU[1], Fm[0], Fm[1]};
#pragma unroll
    for (int k = 0; k < TAPE_PLANES; ++k) t[(long long)k * N] = tv[k];
  }
  if (mode == 1) {
    const double m9[9] = {phi, psi, C, theta, U, p, v[0], v[1], 0.0};
    put_macros(P, mout, idx, m9);
    return;
  }

  auto st = [&](double* at, double val) { put<STREAM, double>(at, val); };
  auto hst2 = [&](int plane, double v0, double v1) {
    double* at = hist + (long long)plane * N + idx;
    st(at, v0);
    st(at + N, v1);
  };
  // whether direction (dx, dy) leaves the node across one of the sides m (bits as DevParams::sym)
  auto leaves = [&](int m, int dx, int dy) {
    return (dx > 0 && x == P.nx - 1 && ((m >> 3) & 1)) || (dx < 0 && x == 0 && (m & 1)) ||
           (dy > 0 && y == P.ny - 1 && ((m >> 4) & 1)) || (dy < 0 && y == 0 && ((m >> 1) & 1));
  };
  // stored value of a 5-velocity population: by anti-bounce-back to zeta across a far-field side
  const bool far = SYM && !fast && P.far;
  auto stored5 = [&](int i, double f, double zeta) {
    return far && leaves(P.far, LS::c[i][0], LS::c[i][1]) ? 2.0 * LS::w[i] * zeta - f : f;
  };

  // ---- NS collision in moment form: f* = feq + F/2 + (1 - s_nu) P_s (f - feq +
  // F/2), P_s the orthogonal projector on c_x^2 - c_y^2 and c_x c_y.  On the
  // 4th-order isotropic lattice the traceless stress moments of f^eq and of F/2 are
  // rho T:vv and T:(vF + cs2 v grad(rho)) (symmetrised), and for i > 0
  // f_i^eq + F_i/2 = w_i [A + c.v (3 rho + 4.5 (rho c.v + c.F) + 1.5 c.grad(rho)) + 1.5 c.F]
  // with A = 3p - 1.5 rho v.v - 1.5 v.F; f_0^eq + F_0/2 = w_0 A - 3p.
  if constexpr (NS) {
    const Planes<9, double> out(fout + (long long)P.o_ns * N + idx, N);
    const double nu = (K.mu_g + (K.mu_l - K.mu_g) * phi) * rcp(rho);
    const double r = 1.0 - rcp(nu * 3.0 + 0.5);
    const double vx = v[0], vy = v[1], Fx = F[0], Fy = F[1], grx = gr[0], gry = gr[1];
    const double vv = vx * vx + vy * vy, vF = vx * Fx + vy * Fy;
    const double A = 3.0 * p - 1.5 * rho * vv - 1.5 * vF;
    const double q1 = 0.25 * r * (mn.s1 - rho * (vx * vx - vy * vy) + (vx * Fx - vy * Fy) + (1.0 / 3) * (vx * grx - vy * gry));
    const double q2 = 0.25 * r * (mn.s2 - rho * vx * vy + 0.5 * (vx * Fy + vy * Fx) + (1.0 / 6) * (vx * gry + vy * grx));
    const double rho3 = 3.0 * rho;
    // Velocity and pressure sides (non-equilibrium extrapolation, Sec. 3
    // boundary paragraph): the slot of population i leaving across one holds
    // what the node pulls back along j = opp(i) on the next step, its own f*_j
    // plus f^eq_j(p, rho, v_in) - f^eq_j(p, rho, v) (velocity side) or
    // f^eq_j(0, rho, v) - f^eq_j(p, rho, v) = -w_j p / cs2 (pressure side);
    // a velocity side takes precedence where both are crossed.
    const bool nee = SYM && !fast && (P.vel | P.pres);
    auto put_ns = [&](int i, double f, double opp) {
      const int dx = LN::c[i][0], dy = LN::c[i][1], j = LN::opp[i];
      if (nee && leaves(P.vel, dx, dy)) {
        const double cx = LN::c[j][0], cy = LN::c[j][1], bx = P.vin[0], by = P.vin[1];
        const double cb = cx * bx + cy * by, cv = cx * vx + cy * vy;
        f = opp + rho * LN::w[j] * ((cb - cv) * 3.0 + (cb * cb - cv * cv) * 4.5 - (bx * bx + by * by - vv) * 1.5);
      } else if (nee && leaves(P.pres, dx, dy)) {
        f = opp - LN::w[j] * p * 3.0;
      }
      st(out.at[i], f);
    };
    put_ns(0, LN::w[0] * A - 3.0 * p, 0.0);
#pragma unroll
    for (int i = 1; i < 9; ++i) {
      if (LN::opp[i] < i) continue;
      const int cx = LN::c[i][0], cy = LN::c[i][1];
      const double w = LN::w[i], cv = cx * vx + cy * vy, cF = cx * Fx + cy * Fy, cg = cx * grx + cy * gry;
      const double even = w * (A + cv * (4.5 * (rho * cv + cF) + 1.5 * cg)) + ((double)(cx * cx - cy * cy) * q1 + (double)(cx * cy) * q2);
      const double odd = w * (cv * rho3 + 1.5 * cF);
      put_ns(i, even + odd, even - odd);
      put_ns(LN::opp[i], even - odd, even + odd);
    }
  }

  // ---- CAC collision: equilibrium w phi (1 + c.v/cs2), whose flux is phi v;
  // source flux fl = d(phi v)/dt + sharpening
  if constexpr (PHI) {
    const double n[2] = {fo.nx, fo.ny}, r = 1.0 - K.s_phi;
    double E[2], D[2], pvs[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const double pv = phi * v[a], prev = first ? pv : h_pv[a];
      const double fl = (pv - prev) + LP::cs2 * fo.sharp * n[a];
      E[a] = pv + 0.5 * fl;
      D[a] = r * (mph.J[a] - pv) + 0.5 * r * fl;
      pvs[a] = pv;
    }
    hst2(P.h_phiv, pvs[0], pvs[1]);
    const Planes<QP, double> out(fout + (long long)P.o_phi * N + idx, N);
    put_set<QP>(LP::w[0] * phi, phi, E, D, [&](int i, double f) { st(out.at[i], f); });
  }

  // ---- anisotropy, kinetics and source of psi
  double a_s = 1.0, lin = 0.0;
  const double invp = rsq(gp[0] * gp[0] + gp[1] * gp[1] + K.dn);
  if constexpr (PSI || CC) {
    // cubic anisotropy in the crystal frame of the nearest seed:
    // a_s = 1 + eps (4 S4 - 3 G^2) / (G + delta)^2, N' = G a_s d a_s / d g'
    const double dn = K.dn;
    const double rx_ = cth * gp[0] + sth * gp[1], ry_ = -sth * gp[0] + cth * gp[1];
    const double rx2 = rx_ * rx_, ry2 = ry_ * ry_;
    const double G = rx2 + ry2, S4 = rx2 * rx2 + ry2 * ry2;
    const double invGd = rcp(G + dn), inv2 = invGd * invGd, eps = K.eps4;
    a_s = 1.0 + eps * (4.0 * S4 - 3.0 * G * G) * inv2;
    const double pre = 4.0 * eps * G * a_s * inv2 * invGd;
    const double Nrx = pre * rx_ * (4.0 * rx2 * G + (4.0 * rx2 - 3.0 * G) * dn - 4.0 * S4);
    const double Nry = pre * ry_ * (4.0 * ry2 * G + (4.0 * ry2 - 3.0 * G) * dn - 4.0 * S4);
    const double Nv[2] = {cth * Nrx - sth * Nry, sth * Nrx + cth * Nry};
    const double as2 = a_s * a_s;
    lin = 1.0 + K.k1 * U;
    const double Fu = K.inv_Le + K.Mcinf * (lin > 0.0 ? lin : 0.0);
    const double gFs = lin > 0.0 ? K.Mcinf * K.k1 : 0.0;
    const double om = 1.0 - phi, ps1 = psi + 1.0;
    const double f2p = 0.5 * (1.0 - psi) * ps1 * (-2.0 * psi);
    const double f3psi = 2.0 * K.beta_inter * om * om * ps1;
    const double s1m = (1.0 - psi) * ps1;
    const double Qpsi = -(f2p + f3psi + K.lam * (30.0 / 32.0 * s1m * s1m) * (theta + K.Mcinf * U));
    // rewritten form: a_n = a_s^2, F(U) in D_psi and S_psi with the grad F
    // term; form for Le = O(1): a_n = a_s^2 F(U) (Appendix B)
    double S_psi, D_psi, an;
    if (P.le1) {
      S_psi = Qpsi * K.inv_tau0;
      D_psi = K.d_psi * as2;
      an = as2 * Fu;
    } else {
      const double invF = rcp(Fu);
      const double gdot = gFs * gU[0] * (as2 * gp[0] + Nv[0]) + gFs * gU[1] * (as2 * gp[1] + Nv[1]);
      S_psi = K.d_psi * invF * invF * gdot + Qpsi * invF * K.inv_tau0;
      D_psi = K.d_psi * as2 * invF;
      an = as2;
    }
    // ---- AAC collision with the time-stretched store; G_i = -w_i c_i.N / a_s^2
    if constexpr (PSI) {
      if constexpr (OLDS) {
#pragma unroll
        for (int i = 0; i < 5; ++i) {
          const int dx = LS::c[i][0], dy = LS::c[i][1];
          const bool across = !fast && ((P.wall[0] && (x + dx < 0 || x + dx >= P.nx)) ||
                                        (P.wall[1] && (y + dy < 0 || y + dy >= P.ny)));
          // both read, one taken (a choice between the two addresses came out of the
          // compiler with one of them undefined on edge tiles)
          const double here = s_fps[LS::opp[i]][ry][rx], there = s_fps[i][ry + dy][rx + dx];
          old[i] = across ? here : there;
        }
      }
      const double rate = rcp(D_psi * 3.0 + 0.5), inv_an = rcp(an);
      const double inv_as2 = P.le1 ? rcp(as2) : inv_an;
      const double even = psi + S_psi + 0.5 * (S_psi - (first ? S_psi : h_S));
      const double g = -(1.0 - 0.5 * rate) * inv_as2 * LS::cs2;
      const double E[2] = {g * Nv[0], g * Nv[1]}, D[2] = {(1.0 - rate) * mps.J[0], (1.0 - rate) * mps.J[1]};
      const Planes<5, double> out(fout + (long long)P.o_psi * N + idx, N);
      put_set<5>(LS::w[0] * even, even, E, D, [&](int i, double f) {
        st(out.at[i], (stored5(i, f, -1.0) - (1.0 - an) * old[i]) * inv_an);
      });
      st(hist + (long long)P.h_psi * N + idx, psi);
      st(hist + (long long)P.h_S * N + idx, S_psi);
    }
  }

  // ---- solute collision
  if constexpr (CC) {
    const double q = clamp01((1.0 - psi) * 0.5), om = 1.0 - phi;
    const double at = -K.aW0 * a_s * lin * (psi - (first ? psi : h_psi));
    const double DqC = K.D * q * C;
    const double jv = DqC * K.sharp * (om > 0.0 ? om : 0.0);   // sqrt(2 beta_phi)/W_phi (phi_l - phi)+
    const double invm = rcp(1.0 - K.k1 * h);
    const double dr = DqC * K.k1 * invm * invm * 0.5;          // grad h = grad psi / 2
    const double s1 = rcp(K.D * q * invm * 3.0 + 0.5);
    const double n[2] = {fo.nx, fo.ny};
    double E[2], D[2], Bs[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const double B = C * v[a] - dr * gp[a] + K.k1 * (at * (gp[a] * invp) + jv * n[a]);
      E[a] = B + (1.0 - 0.5 * s1) * (B - (first ? B : h_B[a]));
      D[a] = (1.0 - s1) * (mc.J[a] - B);
      Bs[a] = B;
    }
    hst2(P.h_B, Bs[0], Bs[1]);
    const Planes<5, double> out(fout + (long long)P.o_c * N + idx, N);
    put_set<5>(LS::w[0] * C, C, E, D, [&](int i, double f) { st(out.at[i], stored5(i, f, 1.0)); });
  }

  // ---- heat collision; H (the sum of g) is rho times the model's H: the rest
  // equilibrium is rho H + (w - 1) theta
  if constexpr (TH) {
    double E[2], D[2], Hvs[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const double Hv = H * v[a];
      E[a] = Hv + (1.0 - 0.5 * s_th) * (Hv - (first ? Hv : h_Hv[a]));
      D[a] = (1.0 - s_th) * (mth.J[a] - Hv);
      Hvs[a] = Hv;
    }
    hst2(P.h_Hv, Hvs[0], Hvs[1]);
    const Planes<5, double> out(fout + (long long)P.o_th * N + idx, N);
    put_set<5>(H + (LS::w[0] - 1.0) * theta, theta, E, D, [&](int i, double f) { st(out.at[i], stored5(i, f, K.theta0)); });
  }
}

template <int FIELDS, int QP>
hipError_t launch_step2d_f64(const DevParams& P, const void* fin, void* fout, void* hist, double* mout, int mode,
                             hipStream_t s) {
  using T = StepTile<FIELDS, double>;
  const dim3 grid(((P.nx + T::X - 1) / T::X) * ((P.ny + T::Y - 1) / T::Y));
  const bool sym = P.sym || P.far;
#define PFL_LAUNCH2(SYMV, NTV)                                                                     \
  hipLaunchKernelGGL((step2d_f64_kernel<FIELDS, QP, SYMV, NTV>), grid, dim3(T::N), 0, s, P,        \
                     (const double*)fin, (double*)fout, (double*)hist, mout, mode)
  if (sym && P.nt) PFL_LAUNCH2(true, true);
  else if (sym) PFL_LAUNCH2(true, false);
  else if (P.nt) PFL_LAUNCH2(false, true);
  else PFL_LAUNCH2(false, false);
#undef PFL_LAUNCH2
  return hipGetLastError();
}

}  // namespace

}  // namespace pfl
