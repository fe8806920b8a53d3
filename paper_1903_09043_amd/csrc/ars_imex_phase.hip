// ars_imex_phase.hip -- what surrounds the solve of an implicit acoustic step
// (the scheme: ars_imex.hip) whose axes are all periodic or walled at both
// ends: the system before it, the transport and update behind it.
//
// Every pass here is bound by memory, so what counts is how many fields are
// moved and how often.  On such axes no ghost value is needed but the
// primitives' (a periodic neighbour is a cell, a wall face carries no flow),
// which leaves six passes:
//   prim    state -> primitives with ghosts (no copy of the state, none of
//           the values that follow from others in one product);
//   diss    acoustic dissipation of every face, the only thing of the
//           explicit faces that the implicit step needs: the source S is
//           formed where it is used;
//   vel     velocities that a Pi gives, at the cells (before the solve with
//           Pi = p^n, behind it with the solution);
//   rows    r = b - A p^n as -F(p^n), F the inhomogeneous operator (the large
//           terms of b and of A p^n cancel inside the face differences),
//           b = r + A p^n for its norm alone, the coefficients, the zeroed
//           vectors, both sums and the coefficients' ranges;
//   cell    implicit faces, acoustic cell values;
//   update  all fluxes of a cell and its new state, in place: a cell reads
//           only its own state.
// The general path (outflow ends) passes through padded copies of Pi, two
// applications of the operator, stored explicit faces and stored fluxes
// instead, some 25 launches.  Against that path, us: before the solve 235 -> 80
// (1024^2) and 260 -> 92 (96^3), behind it 155 -> 76 and 255 -> 130; a whole
// step 0.80 -> 0.56 ms and 1.55 -> 1.26 ms.  update has the longest way to the
// memory's rate (76 us at 96^3: 64 + 42 values gathered a cell at two waves a
// SIMD); each flux is formed by both of its cells.
// Blocks are handed to the eight XCDs in turn; block_of gives each XCD one run
// of consecutive cells, so that a stencil's rows meet in one L2.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "ars_imex_phase.h"
#include "ars_internal.h"
#include "ars_ref.h"

namespace ars {

namespace {

constexpr int BS = 256;
constexpr int R_DISS = 3;  // slot of a face field (R_FACE + 4 a) that holds the dissipation

__device__ __forceinline__ unsigned block_of() { return (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3); }

// Blocks for n elements, a multiple of eight (block_of).
unsigned blocks8(long long n) { return (unsigned)(((n + BS - 1) / BS + 7) / 8 * 8); }

__device__ __forceinline__ int axis_of(int DIM, int t) { return t == DIM - 1 ? 2 : t; }

// Offsets of the neighbours k - 1 and k + 1 of coordinate k on an axis of m
// cells and stride st: periodic images; on a walled axis the cell itself takes
// the place of a missing one (the ghost Pi of the homogeneous operator).
__device__ __forceinline__ void near(int k, int m, long long st, bool wall, long long& om, long long& op) {
  om = k > 0 ? -st : (wall ? 0 : (m - 1) * st);
  op = k + 1 < m ? st : (wall ? 0 : -(m - 1) * st);
}

// A cell of the grid: unpadded index c, padded index q.
struct Cell {
  int k[3];  // x, y, z
  long long c, q;
};
template <int DIM>
__device__ __forceinline__ Cell cell_of(const Params& P, const RefGrid& G, unsigned c) {
  Cell o;
  coords32(c, (unsigned)P.nx, (unsigned)P.ny, o.k[0], o.k[1], o.k[2]);
  o.c = c;
  o.q = G.pad(o.k[0] + 2, DIM == 3 ? o.k[1] + 2 : 0, o.k[2] + 2);
  return o;
}

// S of the vertical face between padded cells l (vertical index lz) and r.
__device__ __forceinline__ double source(const Params& P, double rhoL, double rhoR, int lz) {
  return (-0.5 * (rhoL + rhoR)) * (phi_at(P, lz + 1 - 2) - phi_at(P, lz - 2));
}

template <int DIM>
__global__ __launch_bounds__(BS) void k_imex_prim(Params P, RefGrid G, const double* __restrict__ U,
                                                  double* __restrict__ W) {
  const long long i = (long long)block_of() * BS + threadIdx.x;
  if (i >= G.npad) return;
  constexpr int NV = DIM + 2;
  int qx, qy, qz;
  decode(G, i, qx, qy, qz);
  const int cx = resolve_lat(qx - 2, P.nx, P.bcx);
  const int cy = DIM == 3 ? resolve_lat(qy - 2, P.ny, P.bcy) : 0;
  int kz = qz - 2, ghost = -1;
  if (kz < 0 || kz >= P.nz) {
    const int side = kz < 0 ? 0 : 1;
    if (P.bcz[side] == BC_WALL) {
      ghost = side;
      kz = side == 0 ? 0 : P.nz - 1;
    } else {
      kz = resolve_lat(kz, P.nz, P.bcz);
    }
  }
  const long long cell = cx + (long long)P.nx * (cy + (long long)P.ny * kz);
  double b[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) b[v] = U[cell + v * P.ncell];
  Prim<DIM> q = cons_to_prim<DIM>(P, b);
  if (ghost >= 0) q = wall_ghost<DIM>(P, q, ghost, phi_at(P, ghost == 0 ? -1 : P.nz) - phi_at(P, kz));
  const long long n = G.npad;
  W[R_RHO * n + i] = q.rho;
  W[R_R * n + i] = q.r;
#pragma unroll
  for (int k = 0; k < DIM; ++k) W[ufield(DIM, k) * n + i] = q.u[k];
  W[R_P * n + i] = q.p;
  W[R_RC * n + i] = q.rc;
  W[R_IC * n + i] = q.ic;
  W[R_IRC * n + i] = q.irc;
  if (P.diss) W[R_T * n + i] = q.T;
}

// (a_j theta_j / 2)(u^n_R - u^n_L) of every face between padded cells.
template <int DIM, bool LM>
__global__ __launch_bounds__(BS) void k_imex_diss(Params P, RefGrid G, double* __restrict__ W) {
  const long long i = (long long)block_of() * BS + threadIdx.x;
  if (i >= G.npad) return;
  int qx, qy, qz;
  decode(G, i, qx, qy, qz);
  const int qd[3] = {qx, qy, qz}, Pd[3] = {G.Px, G.Py, G.Pz};
  const long long n = G.npad;
  double d[DIM];
#pragma unroll
  for (int t = 0; t < DIM; ++t) {
    const int a = axis_of(DIM, t);
    d[t] = 0.0;
    if (qd[a] + 1 >= Pd[a]) continue;
    const long long j = i + astride(G, a);
    const double uL = W[ufield(DIM, t) * n + i], uR = W[ufield(DIM, t) * n + j];
    const double am = P.K * dmax2(W[R_RC * n + i], W[R_RC * n + j]);
    double theta = 1.0;
    if (LM) {
      double us = 0.0;  // the explicit u* of t^n
      if (!ref_wall(P, a, qz)) {
        const double S = a == 2 ? source(P, W[R_RHO * n + i], W[R_RHO * n + j], qz) : 0.0;
        us = 0.5 * (uL + uR) -
             ((W[R_P * n + j] - W[R_P * n + i]) - S) * (P.hK * dmin2(W[R_IRC * n + i], W[R_IRC * n + j]));
      }
      theta = dmin2(fabs(us) * dmin2(W[R_IC * n + i], W[R_IC * n + j]), 1.0);
    }
    d[t] = ((0.5 * am) * theta) * (uR - uL);
  }
#pragma unroll
  for (int t = 0; t < DIM; ++t) W[(R_FACE + 4 * axis_of(DIM, t) + R_DISS) * n + i] = d[t];
}

// u = u^n - lambda tau ([Pi*] - S-bar) at the cells; Pi = p^n of the workspace
// (FIRST) or x.
template <int DIM, bool FIRST>
__global__ __launch_bounds__(BS) void k_imex_vel(Params P, RefGrid G, const double* __restrict__ W,
                                                 const double* __restrict__ x, const double* __restrict__ d_dt,
                                                 double* __restrict__ ext) {
  const long long cc = (long long)block_of() * BS + threadIdx.x;
  if (cc >= P.ncell) return;
  const Cell o = cell_of<DIM>(P, G, (unsigned)cc);
  const long long n = G.npad, q = o.q;
  const double* p = W + R_P * n;
  const double dt = *d_dt, tau = W[R_R * n + q], pc = p[q];
  const int m[3] = {P.nx, P.ny, P.nz};
  const long long cs[3] = {1, P.nx, (long long)P.nx * P.ny};
  const double xc = FIRST ? pc : x[o.c];
  double u[DIM];
#pragma unroll
  for (int t = 0; t < DIM; ++t) {
    const int a = axis_of(DIM, t);
    const long long e = astride(G, a);
    double xm, xp;
    if (FIRST) {
      xm = p[q - e];
      xp = p[q + e];
    } else {
      const bool wall = a == 2 && P.bcz[0] == BC_WALL;
      long long om, op;
      near(o.k[a], m[a], cs[a], wall, om, op);
      xm = x[o.c + om];
      xp = x[o.c + op];
      if (wall && o.k[2] == 0) xm = xc + (p[q - e] - pc);
      if (wall && o.k[2] == P.nz - 1) xp = xc + (p[q + e] - pc);
    }
    const double* d = W + (R_FACE + 4 * a + R_DISS) * n;
    const double pp = 0.5 * (xc + xp) - d[q];
    const double pm = 0.5 * (xm + xc) - d[q - e];
    double dpi = pp - pm;
    if (a == 2) {
      const double rho = W[R_RHO * n + q];
      dpi = dpi - 0.5 * (source(P, rho, W[R_RHO * n + q + e], o.k[2] + 2) +
                         source(P, W[R_RHO * n + q - e], rho, o.k[2] + 1));
    }
    u[t] = W[ufield(DIM, t) * n + q] - ((dt / P.dx[a]) * tau) * dpi;
  }
#pragma unroll
  for (int t = 0; t < DIM; ++t) ext[t * n + q] = u[t];
}

// Sums and extremes of a block, rows k of part (gridDim.x values a row).
__device__ __forceinline__ double wave_add(double v) {
#pragma unroll
  for (int m = 32; m > 0; m >>= 1) v = v + __shfl_xor(v, m, 64);
  return v;
}

// The system: r, x, coefficients, zeroed vectors; block sums of (b, b) and
// (r, r), then the smallest and largest of the three coefficients.
template <int DIM>
__global__ __launch_bounds__(BS) void k_imex_rows(Params P, RefGrid G, const double* __restrict__ W,
                                                  const double* __restrict__ ext, const double* __restrict__ d_dt,
                                                  ImexSystem S) {
  const long long n = G.npad;
  const double* p = W + R_P * n;
  const double* ti = W + R_R * n;
  const double* ii = W + R_IRC * n;
  const double dt = *d_dt;
  const int m[3] = {P.nx, P.ny, P.nz};
  double bb = 0.0, rr = 0.0;
  const double inf = __builtin_huge_val();
  double lo[3] = {inf, inf, inf}, hi[3] = {0.0, 0.0, 0.0};
  // one run of consecutive cells a block
  const long long run = ((P.ncell + gridDim.x - 1) / gridDim.x + BS - 1) / BS * BS;
  const long long c0 = (long long)block_of() * run, c1 = c0 + run < P.ncell ? c0 + run : P.ncell;
  for (long long cc = c0 + threadIdx.x; cc < c1; cc += BS) {
    const Cell o = cell_of<DIM>(P, G, (unsigned)cc);
    const long long q = o.q;
    const double pc = p[q], tc = ti[q], ic = ii[q];
    double div = 0.0, hom = 0.0;
#pragma unroll
    for (int t = 0; t < DIM; ++t) {
      const int a = axis_of(DIM, t);
      const long long e = astride(G, a);
      const bool wall = a == 2 && P.bcz[0] == BC_WALL;
      const bool first = wall && o.k[2] == 0, last = wall && o.k[2] == P.nz - 1;
      const double lam = dt / P.dx[a];
      long long om, op, om2, op2, skip;
      near(o.k[a], m[a], e, wall, om, op);
      {  // the neighbours' neighbours
        const int km = o.k[a] > 0 ? o.k[a] - 1 : (wall ? 0 : m[a] - 1);
        const int kp = o.k[a] + 1 < m[a] ? o.k[a] + 1 : (wall ? m[a] - 1 : 0);
        near(km, m[a], e, wall, om2, skip);
        near(kp, m[a], e, wall, skip, op2);
      }
      const double hm = P.hK * dmin2(ii[q + om], ic), hp = P.hK * dmin2(ic, ii[q + op]);
      const double* u = ext + t * n;
      double Sm = 0.0, Sp = 0.0;
      if (a == 2) {
        const double rho = W[R_RHO * n + q];
        Sm = source(P, W[R_RHO * n + q - e], rho, o.k[2] + 1);
        Sp = source(P, rho, W[R_RHO * n + q + e], o.k[2] + 2);
      }
      const double uc = u[q], pm = p[q + om], pp = p[q + op];
      const double usm = first ? 0.0 : 0.5 * (u[q + om] + uc) - ((pc - pm) - Sm) * hm;
      const double usp = last ? 0.0 : 0.5 * (uc + u[q + op]) - ((pp - pc) - Sp) * hp;
      div = div + lam * (usp - usm);
      // homogeneous operator on p^n
      const double vm = -(lam * ti[q + om]) * (0.5 * (pc - p[q + om + om2]));
      const double vc = -(lam * tc) * (0.5 * (pp - pm));
      const double vp = -(lam * ti[q + op]) * (0.5 * (p[q + op + op2] - pc));
      const double hsm = first ? 0.0 : 0.5 * (vm + vc) - (pc - pm) * hm;
      const double hsp = last ? 0.0 : 0.5 * (vc + vp) - (pp - pc) * hp;
      hom = hom + lam * (hsp - hsm);
    }
    const double v[3] = {ic * W[R_IC * n + q], tc, ic};
    const double r = -div;
    const double b = r + (pc * v[0] + hom);
    rr = rr + r * r;
    bb = bb + b * b;
    S.x[cc] = pc;
    S.r[cc] = r;
    S.p[cc] = 0.0;
    S.v[cc] = 0.0;
    S.irc2[cc] = v[0];
    S.tau[cc] = v[1];
    S.irc[cc] = v[2];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      lo[k] = v[k] < lo[k] ? v[k] : lo[k];
      hi[k] = v[k] > hi[k] ? v[k] : hi[k];
    }
  }
  __shared__ double sh[8][BS / 64];
  const int w = threadIdx.x >> 6;
  const double val[8] = {wave_add(bb),       wave_add(rr),     -wave_max(-lo[0]), wave_max(hi[0]),
                         -wave_max(-lo[1]), wave_max(hi[1]), -wave_max(-lo[2]), wave_max(hi[2])};
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int k = 0; k < 8; ++k) sh[k][w] = val[k];
  }
  __syncthreads();
  if (threadIdx.x < 8) {
    const int k = threadIdx.x;
    double a = sh[k][0];
    for (int i = 1; i < BS / 64; ++i) {
      const double o = sh[k][i];
      a = k < 2 ? a + o : (k & 1 ? larger(a, o) : -larger(-a, -o));
    }
    S.part[k * gridDim.x + blockIdx.x] = a;
  }
}

// The blocks' rows, one wave each, and the time step, for the host.
__global__ __launch_bounds__(512) void k_imex_begin_final(const double* __restrict__ part, int nb,
                                                          const double* __restrict__ d_dt, double* __restrict__ bb_rr,
                                                          double* __restrict__ range_dt) {
  const int k = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const double sign = k >= 2 && !(k & 1) ? -1.0 : 1.0;
  const double* row = part + k * nb;
  if (k < 2) {
    double s = 0.0;
    for (int i = lane; i < nb; i += 64) s = s + row[i];
    s = wave_add(s);
    if (lane == 0) bb_rr[k] = s;
  } else {
    double v = sign * row[0];
    for (int i = lane; i < nb; i += 64) v = larger(v, sign * row[i]);
    v = wave_max(v);
    if (lane == 0) range_dt[k - 2] = sign * v;
  }
  if (threadIdx.x == 0) range_dt[6] = *d_dt;
}

// Implicit u* and Pi* of a cell's faces and its acoustic values: the +faces
// (and the bottom wall's) and b~ into the workspace.
template <int DIM>
__global__ __launch_bounds__(BS) void k_imex_cells(Params P, RefGrid G, const double* __restrict__ U,
                                                   double* __restrict__ W, const double* __restrict__ ext,
                                                   const double* __restrict__ x, const double* __restrict__ d_dt,
                                                   Control* ctl) {
  const long long cc = (long long)block_of() * BS + threadIdx.x;
  if (cc >= P.ncell) return;
  constexpr int NV = DIM + 2;
  const Cell o = cell_of<DIM>(P, G, (unsigned)cc);
  const long long n = G.npad, q = o.q, sz = astride(G, 2);
  const double* p = W + R_P * n;
  const double* ii = W + R_IRC * n;
  const double dt = *d_dt, xc = x[o.c], ic = ii[q], rho = W[R_RHO * n + q];
  const int m[3] = {P.nx, P.ny, P.nz};
  const long long cs[3] = {1, P.nx, (long long)P.nx * P.ny};
  const bool wallz = P.bcz[0] == BC_WALL;
  const bool first = wallz && o.k[2] == 0, last = wallz && o.k[2] == P.nz - 1;
  const double Sm = source(P, W[R_RHO * n + q - sz], rho, o.k[2] + 1);
  const double Sp = source(P, rho, W[R_RHO * n + q + sz], o.k[2] + 2);
  double Lc = 1.0, Am[DIM], AE = 0.0, us[DIM], pi[DIM], pib = 0.0;
#pragma unroll
  for (int t = 0; t < DIM; ++t) {
    const int a = axis_of(DIM, t);
    const long long e = astride(G, a);
    const bool wall = a == 2 && wallz;
    const double lam = dt / P.dx[a];
    long long om, op, qm, qp;
    near(o.k[a], m[a], cs[a], wall, om, op);
    near(o.k[a], m[a], e, wall, qm, qp);
    double xm = x[o.c + om], xp = x[o.c + op];
    if (a == 2 && first) xm = xc + (p[q - e] - p[q]);
    if (a == 2 && last) xp = xc + (p[q + e] - p[q]);
    const double* u = ext + t * n;
    const double* d = W + (R_FACE + 4 * a + R_DISS) * n;
    const double uc = u[q];
    double dm = xc - xm, dp = xp - xc;
    if (a == 2) {
      dm = dm - Sm;
      dp = dp - Sp;
    }
    const double usm = a == 2 && first ? 0.0 : 0.5 * (u[q + qm] + uc) - dm * (P.hK * dmin2(ii[q + qm], ic));
    const double usp = a == 2 && last ? 0.0 : 0.5 * (uc + u[q + qp]) - dp * (P.hK * dmin2(ic, ii[q + qp]));
    const double pim = 0.5 * (xm + xc) - d[q - e];
    const double pip = 0.5 * (xc + xp) - d[q];
    us[t] = usp;
    pi[t] = pip;
    if (a == 2) pib = pim;
    Lc = Lc + lam * (usp - usm);
    double dpi = pip - pim;
    if (a == 2) dpi = dpi - 0.5 * (Sp + Sm);
    Am[t] = lam * dpi;
    const double Pp = pip * usp, Pm = pim * usm;
    const double term = lam * (Pp - Pm);
    AE = (t == 0) ? term : AE + term;
  }
  const double iL = rcp_nr(Lc);
  const double calE = U[(NV - 1) * P.ncell + o.c] + rho * phi_at(P, o.k[2]);
  double bt[NV];
  bt[0] = rho * iL;
#pragma unroll
  for (int k = 0; k < DIM; ++k) bt[1 + k] = (U[(1 + k) * P.ncell + o.c] - Am[k]) * iL;
  bt[NV - 1] = (calE - AE) * iL;
#pragma unroll
  for (int v = 0; v < NV; ++v) W[(R_BT + v) * n + q] = bt[v];
#pragma unroll
  for (int t = 0; t < DIM; ++t) {
    double* f = W + (R_FACE + 4 * axis_of(DIM, t)) * n;
    f[q] = us[t];
    f[n + q] = pi[t];
  }
  if (first) {
    double* f = W + (R_FACE + 4 * 2) * n;
    f[q - sz] = 0.0;
    f[n + q - sz] = pib;
  }
  if (!(Lc > 0.0)) {
    atomicOr(&ctl->fault, 1u);
    atomicMin(&ctl->fault_cell, (unsigned long long)o.c);
  }
}

// Value of the field at f, byte offset o: a scalar base and one 32-bit offset
// register a location (OFF = unsigned, while a field's bytes fit 32 bits), where
// 64-bit addresses are two registers for every field and location (the 3D
// viscous update then spills 800 bytes at three waves a SIMD).
template <typename OFF>
__device__ __forceinline__ double at(const double* __restrict__ f, OFF o) {
  return *(const double*)((const char*)f + o);
}

// Total flux of the face (a, i | i + e): the transport from the face's u*, Pi*
// (at f) and b~ of its two cells, and the viscous and heat fluxes on the
// padded primitives.  Offsets in bytes, e[b] the axes' strides.  Both cells of
// a face form it with this expression.
template <int DIM, bool DISS, typename OFF>
__device__ __forceinline__ void imex_flux(const Params& P, long long n, const double* __restrict__ W, const OFF* e,
                                          int t, OFF f, OFF left, OFF right, OFF i, bool wall, double* Gv) {
  constexpr int NV = DIM + 2;
  const int a = axis_of(DIM, t);
  const OFF j = i + e[t];
  const double us = at(W + (R_FACE + 4 * a) * n, f), pi = at(W + (R_FACE + 4 * a + 1) * n, f);
  if (wall) {
#pragma unroll
    for (int v = 0; v < NV; ++v) Gv[v] = 0.0;
  } else {
    const OFF up = us >= 0.0 ? left : right;
#pragma unroll
    for (int v = 0; v < NV - 1; ++v) Gv[v] = at(W + (R_BT + v) * n, up) * us;
    Gv[NV - 1] = (at(W + (R_BT + NV - 1) * n, up) + pi) * us;
  }
  Gv[1 + t] = Gv[1 + t] + pi;
  if (DISS) {
    double g[DIM][DIM];  // g[b][k]: derivative along axis b of u_k
#pragma unroll
    for (int b = 0; b < DIM; ++b) {
      const int ab = axis_of(DIM, b);
#pragma unroll
      for (int k = 0; k < DIM; ++k) {
        const double* u = W + ufield(DIM, k) * n;
        g[b][k] = b == t ? (at(u, j) - at(u, i)) * P.idx[a]
                         : ((at<OFF>(u, i + e[b]) - at<OFF>(u, i - e[b])) +
                            (at<OFF>(u, j + e[b]) - at<OFF>(u, j - e[b]))) * P.qidx[ab];
      }
    }
    double div = g[0][0];
#pragma unroll
    for (int b = 1; b < DIM; ++b) div = div + g[b][b];
    double Wk = 0.0;
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
      double s = P.mu * (g[t][k] + g[k][t]);
      if (k == t) s = s + P.eta * div;
      const double* u = W + ufield(DIM, k) * n;
      const double uf = 0.5 * (at(u, i) + at(u, j));
      Wk = (k == 0) ? s * uf : Wk + s * uf;
      Gv[1 + k] = Gv[1 + k] - s;
    }
    const double* T = W + R_T * n;
    const double Q = -(P.kappa * ((at(T, j) - at(T, i)) * P.idx[a]));
    Gv[NV - 1] = (Gv[NV - 1] - Wk) + Q;
  }
}

template <int DIM, bool DISS, typename OFF>
__global__ __launch_bounds__(BS, 2) void k_imex_update(Params P, RefGrid G, double* U, const double* __restrict__ W,
                                                       const double* __restrict__ d_dt, Control* ctl) {
  const long long cc = (long long)block_of() * BS + threadIdx.x;
  if (cc >= P.ncell) return;
  constexpr int NV = DIM + 2;
  const Cell o = cell_of<DIM>(P, G, (unsigned)cc);
  const long long n = G.npad;
  const OFF q = (OFF)(8 * o.q);
  OFF e[DIM];
#pragma unroll
  for (int t = 0; t < DIM; ++t) e[t] = (OFF)(8 * astride(G, axis_of(DIM, t)));
  const double dt = *d_dt;
  const double phic = phi_at(P, o.k[2]);
  const int m[3] = {P.nx, P.ny, P.nz};
  const bool wallz = P.bcz[0] == BC_WALL;
  double nb[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) nb[v] = U[v * P.ncell + o.c];
  nb[NV - 1] = nb[NV - 1] + nb[0] * phic;
#pragma unroll
  for (int t = 0; t < DIM; ++t) {
    const int a = axis_of(DIM, t);
    const bool first = a == 2 && wallz && o.k[2] == 0, last = a == 2 && wallz && o.k[2] == P.nz - 1;
    const double lam = dt / P.dx[a];
    const OFF span = (OFF)(m[a] - 1) * e[t];
    const OFF qm = o.k[a] > 0 ? q - e[t] : q + span, qp = o.k[a] + 1 < m[a] ? q + e[t] : q - span;
    double Gp[NV], Gm[NV];
    imex_flux<DIM, DISS, OFF>(P, n, W, e, t, q, q, qp, q, last, Gp);
    imex_flux<DIM, DISS, OFF>(P, n, W, e, t, first ? q - e[t] : qm, qm, q, q - e[t], first, Gm);
#pragma unroll
    for (int v = 0; v < NV; ++v) nb[v] = nb[v] - lam * (Gp[v] - Gm[v]);
  }
  const double* rf = W + R_RHO * n;
  const double rho = at(rf, q);
  const double sb = 0.5 * (source(P, rho, at<OFF>(rf, q + e[DIM - 1]), o.k[2] + 2) +
                           source(P, at<OFF>(rf, q - e[DIM - 1]), rho, o.k[2] + 1));
  nb[DIM] = nb[DIM] + (dt / P.dx[2]) * sb;
  nb[NV - 1] = nb[NV - 1] - nb[0] * phic;
#pragma unroll
  for (int v = 0; v < NV; ++v) U[v * P.ncell + o.c] = nb[v];
  const Prim<DIM> qn = cons_to_prim<DIM>(P, nb);
  double kin = nb[1] * qn.u[0];
#pragma unroll
  for (int k = 1; k < DIM; ++k) kin = kin + nb[1 + k] * qn.u[k];
  const bool ok = (nb[0] > 0.0) && (qn.p > 0.0) && isfinite(nb[0]) && isfinite(qn.p) && isfinite(kin);
  if (!ok) {
    atomicOr(&ctl->fault, 1u);
    atomicMin(&ctl->fault_cell, (unsigned long long)o.c);
  }
}

template <int DIM, typename OFF>
void update_t(const Params& P, const RefGrid& G, double* U, const double* W, const double* d_dt, Control* ctl,
              hipStream_t s) {
  const dim3 g(blocks8(P.ncell));
  if (P.diss)
    hipLaunchKernelGGL((k_imex_update<DIM, true, OFF>), g, dim3(BS), 0, s, P, G, U, W, d_dt, ctl);
  else
    hipLaunchKernelGGL((k_imex_update<DIM, false, OFF>), g, dim3(BS), 0, s, P, G, U, W, d_dt, ctl);
}

template <int DIM>
hipError_t begin_t(const Params& P, const double* U, double* W, double* ext, const double* d_dt, const ImexSystem& S,
                   hipStream_t s) {
  const RefGrid G = make_grid(P);
  const unsigned np = blocks8(G.npad), nc = blocks8(P.ncell);
  const unsigned nr = std::min(nc, (unsigned)IMEX_BEGIN_BLOCKS);
  hipLaunchKernelGGL(k_imex_prim<DIM>, dim3(np), dim3(BS), 0, s, P, G, U, W);
  if (P.low_mach)
    hipLaunchKernelGGL((k_imex_diss<DIM, true>), dim3(np), dim3(BS), 0, s, P, G, W);
  else
    hipLaunchKernelGGL((k_imex_diss<DIM, false>), dim3(np), dim3(BS), 0, s, P, G, W);
  hipLaunchKernelGGL((k_imex_vel<DIM, true>), dim3(nc), dim3(BS), 0, s, P, G, W, nullptr, d_dt, ext);
  hipLaunchKernelGGL(k_imex_rows<DIM>, dim3(nr), dim3(BS), 0, s, P, G, W, ext, d_dt, S);
  hipLaunchKernelGGL(k_imex_begin_final, dim3(1), dim3(512), 0, s, S.part, (int)nr, d_dt, S.bb_rr, S.range_dt);
  return hipGetLastError();
}

template <int DIM>
hipError_t finish_t(const Params& P, double* U, double* W, double* ext, const double* x, const double* d_dt,
                    Control* ctl, hipStream_t s) {
  const RefGrid G = make_grid(P);
  const unsigned nc = blocks8(P.ncell);
  hipLaunchKernelGGL((k_imex_vel<DIM, false>), dim3(nc), dim3(BS), 0, s, P, G, W, x, d_dt, ext);
  hipLaunchKernelGGL(k_imex_cells<DIM>, dim3(nc), dim3(BS), 0, s, P, G, U, W, ext, x, d_dt, ctl);
  if ((unsigned long long)G.npad * 8 <= 0xffffffffull)
    update_t<DIM, unsigned>(P, G, U, W, d_dt, ctl, s);
  else
    update_t<DIM, long long>(P, G, U, W, d_dt, ctl, s);
  return hipGetLastError();
}

}  // namespace

hipError_t imex_begin(const Params& P, const double* U, double* W, double* ext, const double* d_dt,
                      const ImexSystem& S, hipStream_t s) {
  return P.dim == 3 ? begin_t<3>(P, U, W, ext, d_dt, S, s) : begin_t<2>(P, U, W, ext, d_dt, S, s);
}

hipError_t imex_finish(const Params& P, double* U, double* W, double* ext, const double* x, const double* d_dt,
                       Control* ctl, hipStream_t s) {
  return P.dim == 3 ? finish_t<3>(P, U, W, ext, x, d_dt, ctl, s) : finish_t<2>(P, U, W, ext, x, d_dt, ctl, s);
}

}  // namespace ars
