// 3D step building blocks shared by the FP64 step and the FP32-compute one:
// column tile, pulls (general and plane-base addressing), isotropic D3Q19
// stencils on LDS planes, the flow quantities of one position and the choice
// of z planes per workgroup.
#pragma once
#include "pfl_kernels.h"
#include "pfl_util.h"

namespace pfl {

namespace {

// Column tile: 32 x 8 nodes, 256 threads (rows of 32 nodes keep each wave's
// loads and stores in whole or half 128-byte lines).  FP64 runs one wave per
// SIMD either way; against 32 x 4 the taller column spreads the ring pulls
// over more nodes (coupled 256^3 FP64 2.65k -> 2.75k MLUPS) and fits the
// LDS (55 KB).
template <class CT>
struct Col3 {
  static constexpr int TX = 32, TY = sizeof(CT) == 8 ? 8 : 16;
  static constexpr int NT = TX * TY;
};

// One LDS plane of the tile plus R rings in x and y.
template <class CT, int R>
struct Pl {
  static constexpr int X = Col3<CT>::TX + 2 * R, Y = Col3<CT>::TY + 2 * R;
  static constexpr int N = X * Y;
  __device__ static constexpr int at(int y, int x) { return y * X + x; }
};

// Ring slot of plane p among n slots.
__device__ __forceinline__ int ring_slot(int p, int n) {
  const int s = p % n;
  return s < 0 ? s + n : s;
}

// Pull the stored values of one set at node (x, y, z), general addressing:
// periodic wrap, half-way bounce-back at a wall or specular reflection at a
// symmetry plane on each axis, from per-axis source offsets computed once
// per node.
// SEL: addresses by selects instead of branches, so that the loads of a set
// leave together.
template <int Q, class ST, class CT, bool SYM, bool SEL>
__device__ __forceinline__ void pull3_general(const typename Store<ST>::raw* __restrict__ base,
                                              const DevParams& P, int x, int y, int z, CT f[Q]) {
  using L = Lat<Q>;
  AxisSrc ax, ay, az;
  axis_src(x, P.nx, P.wall[0], SYM && sym_side(P, 0, true), SYM && sym_side(P, 0, false), 1, ax);
  axis_src(y, P.ny, P.wall[1], SYM && sym_side(P, 1, true), SYM && sym_side(P, 1, false), P.nx, ay);
  axis_src(z, P.nz, P.wall[2], SYM && sym_side(P, 2, true), SYM && sym_side(P, 2, false), P.nx * P.ny, az);
  const int m = SYM ? sym_touch(P, x, y, z) : 0;
  const long long own = ((long long)z * P.ny + y) * P.nx + x;
  const long long N = P.N;
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    const int cx = L::c[i][0] + 1, cy = L::c[i][1] + 1, cz = L::c[i][2] + 1;
    const bool b = ax.wall[cx] || ay.wall[cy] || az.wall[cz];
    long long e;
    if constexpr (SEL) {
      const int off = b ? 0 : ax.off[cx] + ay.off[cy] + az.off[cz];
      const long long plane = SYM ? (long long)(b ? L::opp[i] : pulled_population<Q>(i, m)) * N
                                  : (b ? L::opp[i] * N : i * N);
      e = plane + own + off;
    } else {
      const int j = SYM ? pulled_population<Q>(i, m) : i;
      e = b ? (long long)L::opp[i] * N + own : (long long)j * N + (own + ax.off[cx] + ay.off[cy] + az.off[cz]);
    }
    f[i] = Store<ST>::template ld<CT>(base + e);
  }
}

// Pull at a node whose sources x - c_i all lie inside the domain: a 64-bit
// plane base per population and one 32-bit in-plane byte offset (the source
// node's offset is non-negative and below N S < 2^32).
template <int Q, class ST, class CT>
__device__ __forceinline__ void pull3_fast(const typename Store<ST>::raw* __restrict__ base,
                                           const DevParams& P, uint32_t nbyte, CT f[Q]) {
  using L = Lat<Q>;
  constexpr uint32_t S = sizeof(typename Store<ST>::raw);
  const uint32_t sxy = (uint32_t)P.nx * (uint32_t)P.ny;
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    const uint32_t shift = ((uint32_t)L::c[i][0] + (uint32_t)L::c[i][1] * (uint32_t)P.nx +
                            (uint32_t)L::c[i][2] * sxy) * S;
    f[i] = Store<ST>::template ld<CT>(at_byte<ST>(base + (size_t)i * (size_t)P.N, nbyte - shift));
  }
}

template <int Q, class ST, class CT, bool SYM = false, bool SEL = false>
__device__ __forceinline__ void pull3(bool fast, const typename Store<ST>::raw* __restrict__ base,
                                      const DevParams& P, int x, int y, int z, CT f[Q]) {
  if (fast) {
    const uint32_t nbyte = (uint32_t)((z * P.ny + y) * P.nx + x) * (uint32_t)sizeof(typename Store<ST>::raw);
    pull3_fast<Q, ST, CT>(base, P, nbyte, f);
  } else {
    pull3_general<Q, ST, CT, SYM, SEL>(base, P, x, y, z, f);
  }
}

// Isotropic D3Q19 gradient (1/cs2) sum_i w_i c_i f(x + c_i) and Laplacian
// (2/cs2) sum_i w_i [f(x + c_i) - f(x)] from three LDS planes (below, at,
// above the node), (y, x) in the plane geometry PL.
template <class CT, class PL>
__device__ __forceinline__ void grad19p(const CT* const pl[3], int y, int x, CT g[3]) {
  using L = Lat<19>;
  CT a0 = CT(0), a1 = CT(0), a2 = CT(0);
#pragma unroll
  for (int i = 1; i < 19; ++i) {
    const CT v = CT(L::w[i]) * pl[L::c[i][2] + 1][PL::at(y + L::c[i][1], x + L::c[i][0])];
    if (L::c[i][0]) a0 += CT(L::c[i][0]) * v;
    if (L::c[i][1]) a1 += CT(L::c[i][1]) * v;
    if (L::c[i][2]) a2 += CT(L::c[i][2]) * v;
  }
  g[0] = CT(3) * a0;
  g[1] = CT(3) * a1;
  g[2] = CT(3) * a2;
}
template <class CT, class PL>
__device__ __forceinline__ CT lap19p(const CT* const pl[3], int y, int x) {
  using L = Lat<19>;
  const CT c = pl[1][PL::at(y, x)];
  CT a = CT(0);
#pragma unroll
  for (int i = 1; i < 19; ++i) a += CT(L::w[i]) * (pl[L::c[i][2] + 1][PL::at(y + L::c[i][1], x + L::c[i][0])] - c);
  return CT(6) * a;
}

// z planes per workgroup of a launch whose columns number cols and of which
// slots workgroups run at once.  A chunk of zc planes costs its zc iterations
// and two more that only fill the rings, so a launch of r full rounds costs
// r (zc + 2) with the chunk that makes the rounds full, zc = ceil(nz / (r
// slots / cols)).  The smallest cost wins; within 1% the shorter chunk does
// (256^3 FP64: 128 planes in two rounds against 256 in one, 3.06k against
// 3.02k MLUPS).  Measured, one chunk length of 128 planes before, against this
// rule: 96^3 FP64 psi + C + theta 1055 -> 138 us a step (14 chunks of 7),
// 90 x 70 x 50 FP32 650 -> 71 us (17 of 3), 160^3 FP16 coupled 2023 -> 597 us
// (5 of 32); between its minima the step time follows the cost within 10%.
inline int chunk_planes(long long cols, int nz, long long slots) {
  const long long r0 = (cols + slots - 1) / slots;
  int best = nz;
  double cost = 0.0;
  for (long long r = r0; r < r0 + 16; ++r) {
    const long long n = r * slots / cols;             // chunks per column, at least 1
    const int zc = (int)((nz + n - 1) / n);
    const double c = (double)r * (zc + 2);
    if (r == r0 || c < cost) cost = c;
    if (c <= 1.01 * cost) best = zc;
    if (zc == 1) break;
  }
  return best;
}

// Workgroups of nt threads of a kernel that a compute unit holds at once, a
// property of the compiled kernel.
template <class K>
int blocks_per_cu(K kernel, int nt) {
  int n = 0;
  const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, nt, 0);
  return e == hipSuccess && n > 0 ? n : 1;
}

}  // namespace

}  // namespace pfl
