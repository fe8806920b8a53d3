// ars_imex.hip -- implicit acoustic (IMEX) step of the all-regime scheme:
// the further work the paper names in its Conclusion (solve the acoustic
// part implicitly to lift the acoustic CFL condition, keeping the
// well-balanced gravity source).  The paper prints no scheme; the reading:
// Sec. 2.1.2's acoustic step with its interface values taken at the END of
// the step (backward Euler on the linear relaxation system at frozen
// a, S, theta of t^n).  Unknowns per interior cell i: Pi_i and the normal
// velocities u_{d,i}; with lambda_d = dt / dx_d,
//   u*_j  = (u_L + u_R)/2 - (Pi_R - Pi_L - S_j) / (2 a_j)       (0 at walls)
//   Pi*_j = (Pi_L + Pi_R)/2 - (a_j theta_j / 2)(u^n_R - u^n_L)
//   u_{d,i} = u^n_{d,i} - lambda_d tau_i ([Pi*]_{d,i} - S-bar_{d,i})
//   Pi_i    = p_i - rho_i c_i^2 sum_d lambda_d [u*]_{d,i}
// (the pressure row is the Lagrangian update linearised through the
// equation of state; the acoustic dissipation of Pi* acts on u^n, so the
// velocity rows are explicit in Pi and u is eliminated: the system is for
// Pi alone, its rows scaled by 1 / (rho c^2)).  Ghost cells take the boundary rules of the explicit
// step applied to the unknowns (periodic images, outflow copies; at walls
// Pi_g = Pi_i + (p_g - p_i)^n and the reflected velocity).  The implicit
// (u*, Pi*) then replace the explicit ones in the acoustic cell values,
// the transport, the update and the relaxation, which are the explicit
// step's (the dissipative fluxes stay explicit).
//
// GPU layout: the reference step's padded workspace (primitives, explicit
// faces for a, S, theta, then the implicit faces, L, b~, fluxes), padded
// extensions of Pi and of the velocities it gives, and the vectors of an
// Krylov solver on the N unknowns Pi: conjugate gradients when every axis is
// periodic or walled at both ends (the operator is then symmetric positive
// definite), plain or preconditioned by the constant-coefficient operator's
// inverse (ars_trig.hip), BiCGSTAB otherwise (outflow).  With conjugate
// gradients the system is formed and the step finished by the passes of
// ars_imex_phase.hip.  For BiCGSTAB the operator is applied
// matrix-free: one kernel extends Pi to the ghost cells, one forms the
// velocities of every padded cell from the Pi* of its two faces per axis
// (ghosts by the boundary rules), one forms every row from the u* of the
// two faces of each axis.  Dot products are two-level reductions in a
// fixed order (deterministic); the iteration's scalars stay on the device
// and the host reads the residual norm every few iterations.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "../../include/ars.h"
#include "ars_dev.h"
#include "ars_imex_phase.h"
#include "ars_internal.h"
#include "ars_ref.h"
#include "ars_trig.h"

namespace ars {

namespace {

constexpr int DOT_BLOCKS = 1024;
constexpr int CG_BLOCKS = 1024;  // blocks of the CG kernels (<= the partial-sum slots)
constexpr int BS = 256;
constexpr int CG_CHECK = 16;  // CG iterations between host reads of the residual
// scalar slots of the iteration
enum { SC_RHO_OLD = 0, SC_ALPHA, SC_OMEGA, SC_RHO_NEW, SC_RV, SC_TS, SC_TT, SC_RR, SC_BB,
       SC_CG_RR,      // (r, r) of CG iterations 0, 2, 4, ... (SC_CG_RR + 1: 1, 3, 5, ...)
       SC_CG_CHK = 11,
       SC_RANGE = 16,  // smallest and largest 1/(rho c^2), tau, 1/(rho c)
       SC_DT = 22, SC_N = 32 };

struct ImexLayout {
  RefGrid G;
  long long n;      // unknowns: Pi of every interior cell
  double* W;        // reference workspace
  double* ext;      // (D + 1) padded fields: Pi, u_0..u_{D-1}
  double* x;        // solution
  double* r;
  double* rh;       // shadow residual
  double* p;
  double* v;
  double* sv;
  double* t;
  double* b;
  double* r2;       // CG: the second residual and product of the ping-pong
  double* q2;
  double* part;     // partial sums (one per block of a reduction; CG: up to two sets of four)
  double* sc;       // scalars
};

ImexLayout layout_of(const Params& P, void* work) {
  ImexLayout L;
  L.G = make_grid(P);
  const int D = P.dim;
  L.n = P.ncell;
  char* w = (char*)work;
  size_t off = 0;
  auto take = [&](size_t count) {
    double* q = (double*)(w + off);
    off += ((count * sizeof(double) + 255) / 256) * 256;
    return q;
  };
  L.W = take((size_t)R_NFIELD * L.G.npad);
  L.ext = take((size_t)(D + 1) * L.G.npad);
  L.x = take(L.n);
  L.r = take(L.n);
  L.rh = take(L.n);
  L.p = take(L.n);
  L.v = take(L.n);
  L.sv = take(L.n);
  L.t = take(L.n);
  L.b = take(L.n);
  L.r2 = take(L.n);
  L.q2 = take(L.n);
  L.part = take(8 * (CG_BLOCKS > DOT_BLOCKS ? CG_BLOCKS : DOT_BLOCKS));
  L.sc = take(SC_N);
  return L;
}

__device__ __forceinline__ int comp_axis(int DIM, int a) { return a == 2 ? DIM - 1 : a; }

// Interior source cell of a padded cell (periodic image, outflow copy, or
// the interior neighbour of a wall ghost: wall = 0 bottom, 1 top, -1 none).
template <int DIM>
__device__ __forceinline__ void source_cell(const Params& P, int qx, int qy, int qz, int& cx, int& cy, int& kz,
                                            int& wall) {
  cx = resolve_lat(qx - 2, P.nx, P.bcx);
  cy = (DIM == 3) ? resolve_lat(qy - 2, P.ny, P.bcy) : 0;
  kz = qz - 2;
  wall = -1;
  if (kz < 0 || kz >= P.nz) {
    const int side = kz < 0 ? 0 : 1;
    if (P.bcz[side] == BC_WALL) {
      wall = side;
      kz = side == 0 ? 0 : P.nz - 1;
    } else {
      kz = resolve_lat(kz, P.nz, P.bcz);
    }
  }
}

// Padded extension of Pi (cst: with the wall ghosts' hydrostatic offset).
template <int DIM>
__global__ void k_schur_extP(Params P, RefGrid G, const double* __restrict__ W, const double* __restrict__ x, int cst,
                             double* __restrict__ ext) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= G.npad) return;
  int qx, qy, qz, cx, cy, kz, wall;
  decode(G, i, qx, qy, qz);
  source_cell<DIM>(P, qx, qy, qz, cx, cy, kz, wall);
  const long long n = G.npad;
  double Pi = x[cx + (long long)P.nx * (cy + (long long)P.ny * kz)];
  if (wall >= 0 && cst) {
    const long long qi = G.pad(qx, qy, wall == 0 ? 2 : P.nz + 1);
    Pi = Pi + (W[R_P * n + i] - W[R_P * n + qi]);
  }
  ext[i] = Pi;
}

// Acoustic dissipation term of Pi* on face (a, l | l + e_a), on the
// velocities of t^n: (a_j theta_j / 2)(u^n_R - u^n_L).
template <int DIM, bool LM>
__device__ __forceinline__ double dissip_n(const Params& P, const RefGrid& G, const double* __restrict__ W,
                                           long long l, int a) {
  const long long n = G.npad;
  const long long r = l + astride(G, a);
  const double am = P.K * dmax2(W[R_RC * n + l], W[R_RC * n + r]);
  double theta = 1.0;
  if (LM) {
    const double use = W[(R_FACE + 4 * a) * n + l];  // explicit u* of t^n
    theta = dmin2(fabs(use) * dmin2(W[R_IC * n + l], W[R_IC * n + r]), 1.0);
  }
  const int uf = ufield(DIM, a == 2 ? DIM - 1 : a);
  return ((0.5 * am) * theta) * (W[uf * n + r] - W[uf * n + l]);
}

// Velocities of every padded cell from Pi (its source cell's velocity
// rows, then the ghost rule): u = cst u^n - lambda tau ([Pi*] - cst S-bar).
template <int DIM, bool LM>
__global__ void k_schur_u(Params P, RefGrid G, const double* __restrict__ W, const double* __restrict__ d_dt, int cst,
                          double* __restrict__ ext) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= G.npad) return;
  int qx, qy, qz, cx, cy, kz, wall;
  decode(G, i, qx, qy, qz);
  source_cell<DIM>(P, qx, qy, qz, cx, cy, kz, wall);
  const long long n = G.npad;
  const long long q = G.pad(cx + 2, DIM == 3 ? cy + 2 : 0, kz + 2);  // padded index of the source cell
  const double dt = *d_dt;
  const int axes[3] = {0, DIM == 3 ? 1 : 2, 2};
#pragma unroll
  for (int t = 0; t < DIM; ++t) {
    const int a = axes[t];
    const long long e = astride(G, a);
    double pp = 0.5 * (ext[q] + ext[q + e]);
    double pm = 0.5 * (ext[q - e] + ext[q]);
    double dpi;
    if (cst) {
      pp = pp - dissip_n<DIM, LM>(P, G, W, q, a);
      pm = pm - dissip_n<DIM, LM>(P, G, W, q - e, a);
      dpi = pp - pm;
      if (a == 2) dpi = dpi - 0.5 * (W[(R_FACE + 4 * a + 3) * n + q] + W[(R_FACE + 4 * a + 3) * n + q - e]);
    } else {
      dpi = pp - pm;
    }
    const int k = comp_axis(DIM, a);
    double u = (cst ? W[ufield(DIM, k) * n + q] : 0.0) - ((dt / P.dx[a]) * W[R_R * n + q]) * dpi;
    if (wall >= 0 && (P.noslip || k == DIM - 1)) u = -u;
    ext[(1 + k) * n + i] = u;
  }
}

// Implicit u* of face (a, l | l + e_a) from the extensions.
template <int DIM>
__device__ __forceinline__ double ustar_imp(const Params& P, const RefGrid& G, const double* __restrict__ W,
                                            const double* __restrict__ ext, long long l, int lz, int a, int cst) {
  if (ref_wall(P, a, lz)) return 0.0;
  const long long n = G.npad;
  const long long r = l + astride(G, a);
  const int k = comp_axis(DIM, a);
  const double h2a = P.hK * dmin2(W[R_IRC * n + l], W[R_IRC * n + r]);  // 1 / (2a)
  const double S = (a == 2 && cst) ? W[(R_FACE + 4 * a + 3) * n + l] : 0.0;
  return 0.5 * (ext[(1 + k) * n + l] + ext[(1 + k) * n + r]) - ((ext[r] - ext[l]) - S) * h2a;
}

// Rows of the system for Pi at every interior cell, scaled by 1/(rho c^2):
// y = (Pi - cst p) / (rho c^2) + sum_d lambda_d [u*]_d.
template <int DIM>
__global__ void k_schur_rows(Params P, RefGrid G, const double* __restrict__ W, const double* __restrict__ ext,
                             const double* __restrict__ d_dt, const double* __restrict__ x, int cst,
                             double* __restrict__ y) {
  const long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= P.ncell) return;
  int cxx, cyy, czz;
  coords32((unsigned)c, (unsigned)P.nx, (unsigned)P.ny, cxx, cyy, czz);
  const long long q = G.pad(cxx + 2, DIM == 3 ? cyy + 2 : 0, czz + 2);
  const long long n = G.npad;
  const double dt = *d_dt;
  const int axes[3] = {0, DIM == 3 ? 1 : 2, 2};
  double div = 0.0;
#pragma unroll
  for (int t = 0; t < DIM; ++t) {
    const int a = axes[t];
    const double usp = ustar_imp<DIM>(P, G, W, ext, q, czz + 2, a, cst);
    const double usm = ustar_imp<DIM>(P, G, W, ext, q - astride(G, a), czz + 2 - (a == 2), a, cst);
    div = div + (dt / P.dx[a]) * (usp - usm);
  }
  const double rc2 = W[R_RC * n + q] * W[R_C * n + q];  // rho c^2
  y[c] = (x[c] - (cst ? W[R_P * n + q] : 0.0)) / rc2 + div;
}

// Implicit faces of every padded face into the workspace (u*, Pi*, Pi* u*;
// S untouched); every thread reads only its own faces' explicit u* (for
// theta) before overwriting them.
template <int DIM, bool LM>
__global__ void k_imex_faces(Params P, RefGrid G, double* __restrict__ W, const double* __restrict__ ext) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= G.npad) return;
  int qx, qy, qz;
  decode(G, i, qx, qy, qz);
  const long long n = G.npad;
  const int axes[3] = {0, DIM == 3 ? 1 : 2, 2};
  double us[3], pi[3];
  bool has[3];
#pragma unroll
  for (int t = 0; t < DIM; ++t) {
    const int a = axes[t];
    const int qa = a == 0 ? qx : (a == 1 ? qy : qz);
    const int Pa = a == 0 ? G.Px : (a == 1 ? G.Py : G.Pz);
    has[t] = qa + 1 < Pa;
    us[t] = pi[t] = 0.0;
    if (has[t]) {
      us[t] = ustar_imp<DIM>(P, G, W, ext, i, qz, a, 1);
      pi[t] = 0.5 * (ext[i] + ext[i + astride(G, a)]) - dissip_n<DIM, LM>(P, G, W, i, a);
    }
  }
#pragma unroll
  for (int t = 0; t < DIM; ++t) {
    if (!has[t]) continue;
    const int f = R_FACE + 4 * axes[t];
    W[(f + 0) * n + i] = us[t];
    W[(f + 1) * n + i] = pi[t];
    W[(f + 2) * n + i] = pi[t] * us[t];
  }
}

// Acoustic cell values L, S-bar, b~ (Sec. 2.1.2) from the stored faces.
template <int DIM>
__global__ void k_imex_cell(Params P, RefGrid G, const double* __restrict__ d_dt, double* __restrict__ W) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= G.npad) return;
  constexpr int NV = DIM + 2;
  int qx, qy, qz;
  decode(G, i, qx, qy, qz);
  const bool cell = qx >= 1 && qx < G.Px - 1 && qz >= 1 && qz < G.Pz - 1 && (DIM == 2 || (qy >= 1 && qy < G.Py - 1));
  if (!cell) return;
  const long long n = G.npad;
  const double dt = *d_dt;
  const int axes[3] = {0, DIM == 3 ? 1 : 2, 2};
  double Lc = 1.0, Am[3], AE = 0.0;
  const long long sz = astride(G, 2);
  const double sb = 0.5 * (W[(R_FACE + 4 * 2 + 3) * n + i] + W[(R_FACE + 4 * 2 + 3) * n + i - sz]);
#pragma unroll
  for (int t = 0; t < DIM; ++t) {
    const int a = axes[t];
    const int f = R_FACE + 4 * a;
    const long long m = i - astride(G, a);
    const double lam = dt / P.dx[a];
    Lc = Lc + lam * (W[f * n + i] - W[f * n + m]);
    double dpi = W[(f + 1) * n + i] - W[(f + 1) * n + m];
    if (a == 2) dpi = dpi - sb;
    Am[t] = lam * dpi;
    const double term = lam * (W[(f + 2) * n + i] - W[(f + 2) * n + m]);
    AE = (t == 0) ? term : AE + term;
  }
  const double rho = W[R_CONS * n + i];
  const double calE = W[(R_CONS + NV - 1) * n + i] + rho * phi_at(P, qz - 2);
  const double iL = rcp_nr(Lc);
  W[R_L * n + i] = Lc;
  W[R_SB * n + i] = sb;
  W[R_BT * n + i] = rho * iL;
#pragma unroll
  for (int k = 0; k < DIM; ++k) W[(R_BT + 1 + k) * n + i] = (W[(R_CONS + 1 + k) * n + i] - Am[k]) * iL;
  W[(R_BT + NV - 1) * n + i] = (calE - AE) * iL;
}

// ------------------------------------------------------------ BiCGSTAB ----
__global__ void k_dot_partial(const double* __restrict__ a, const double* __restrict__ b, long long n,
                              double* __restrict__ part) {
  __shared__ double sh[BS];
  double s = 0.0;
  for (long long i = (long long)blockIdx.x * BS + threadIdx.x; i < n; i += (long long)gridDim.x * BS)
    s = s + a[i] * b[i];
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int w = BS / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) sh[threadIdx.x] = sh[threadIdx.x] + sh[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

__global__ void k_dot_final(const double* __restrict__ part, int nb, double* __restrict__ out) {
  __shared__ double sh[BS];
  double s = 0.0;
  for (int i = threadIdx.x; i < nb; i += BS) s = s + part[i];
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int w = BS / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) sh[threadIdx.x] = sh[threadIdx.x] + sh[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = sh[0];
}

// r = b - r (r holds A x on entry); rh = r; p = v = 0; scalars start.
__global__ void k_bicg_start(long long n, const double* __restrict__ b, double* __restrict__ r, double* __restrict__ rh,
                             double* __restrict__ p, double* __restrict__ v, double* __restrict__ sc) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0) {
    sc[SC_RHO_OLD] = 1.0;
    sc[SC_ALPHA] = 1.0;
    sc[SC_OMEGA] = 1.0;
  }
  if (i >= n) return;
  const double ri = b[i] - r[i];
  r[i] = ri;
  rh[i] = ri;
  p[i] = 0.0;
  v[i] = 0.0;
}

// p = r + beta (p - omega v),  beta = (rho_new / rho_old) (alpha / omega)
__global__ void k_bicg_p(long long n, const double* __restrict__ r, const double* __restrict__ v,
                         double* __restrict__ p, const double* __restrict__ sc) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double den = sc[SC_RHO_OLD] * sc[SC_OMEGA];
  const double beta = den != 0.0 ? (sc[SC_RHO_NEW] * sc[SC_ALPHA]) / den : 0.0;
  p[i] = r[i] + beta * (p[i] - sc[SC_OMEGA] * v[i]);
}

// alpha = rho_new / (rh, v), 0 at a breakdown
__device__ __forceinline__ double bicg_alpha(const double* sc) {
  return sc[SC_RV] != 0.0 ? sc[SC_RHO_NEW] / sc[SC_RV] : 0.0;
}

// s = r - alpha v
__global__ void k_bicg_s(long long n, const double* __restrict__ r, const double* __restrict__ v,
                         double* __restrict__ s, double* __restrict__ sc) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const double alpha = bicg_alpha(sc);
  if (i >= n) return;
  s[i] = r[i] - alpha * v[i];
}

// x += alpha p + omega s;  r = s - omega t;  omega = (t, s) / (t, t)
__global__ void k_bicg_xr(long long n, const double* __restrict__ p, const double* __restrict__ s,
                          const double* __restrict__ t, double* __restrict__ x, double* __restrict__ r,
                          double* __restrict__ sc) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const double alpha = bicg_alpha(sc);
  const double omega = sc[SC_TT] > 0.0 ? sc[SC_TS] / sc[SC_TT] : 0.0;
  if (i < n) {
    x[i] = x[i] + alpha * p[i] + omega * s[i];
    r[i] = s[i] - omega * t[i];
  }
}

// alpha, omega and rho_old of this iteration for the next one's beta (a
// kernel of its own: k_bicg_xr's threads read the previous values)
__global__ void k_bicg_scalars(double* __restrict__ sc) {
  if (threadIdx.x == 0) {
    sc[SC_ALPHA] = bicg_alpha(sc);
    sc[SC_OMEGA] = sc[SC_TT] > 0.0 ? sc[SC_TS] / sc[SC_TT] : 0.0;
    sc[SC_RHO_OLD] = sc[SC_RHO_NEW];
  }
}

// Conjugate gradients (every axis periodic or walled at both ends: the
// eliminated operator is symmetric positive definite, diag(1/(rho c^2)) +
// lambda^2 K^T tau K + lambda G^T (1/(2a)) G with K the central difference
// of the two face averages and G the face difference.  At a wall the ghost
// Pi is the wall cell's, so the wall face's Pi* is that cell's Pi, and the
// wall face's u* is 0; the ghost velocity feeds nothing else, and the
// operator stays symmetric.  Outflow copies make u* at the boundary face
// the edge cell's velocity, which breaks the symmetry: BiCGSTAB there.)
// The operator is a star stencil of radius 2 on the unknowns (neighbour
// indices wrapped on periodic axes, clamped on walled ones).  An
// iteration is one kernel (k_cg_iter_2d over LDS tiles, k_cg_iter_3d over
// columns of cells): it applies the previous iteration's update of x and r,
// forms p and q = A p on the fly and leaves the block sums of both.  The
// preconditioned iteration takes two streaming kernels: (1) p = z + beta p_old
// and q = A p (k_cg_apply), (2) x += alpha p, r -= alpha q (k_cg_xr).
// Each kernel starts by adding the
// block sums it needs itself, every block in the same fixed order (so every
// block forms the same alpha and beta bit for bit, and no one-block launch
// sits between kernels).  A last-block-arrives reduction would need
// device-scope fences (one per block, an L2 write-back each on a part whose
// XCDs have L2s of their own), which cost far more.

// Index offsets of the neighbours k - 2, k - 1, k + 1, k + 2 of coordinate
// k on an axis of m >= 2 cells and stride st: periodic images, or on a
// walled axis the nearest interior cell (the ghost Pi is the wall cell's).
__device__ __forceinline__ void nb_offsets(int k, int m, int st, bool wall, int& om2, int& om1, int& op1, int& op2) {
  if (wall) {
    om2 = ((k >= 2 ? k - 2 : 0) - k) * st;
    om1 = ((k >= 1 ? k - 1 : 0) - k) * st;
    op1 = ((k + 1 < m ? k + 1 : m - 1) - k) * st;
    op2 = ((k + 2 < m ? k + 2 : m - 1) - k) * st;
  } else {
    om2 = (k >= 2 ? -2 : m - 2) * st;
    om1 = (k >= 1 ? -1 : m - 1) * st;
    op1 = (k + 1 < m ? 1 : 1 - m) * st;
    op2 = (k + 2 < m ? 2 : 2 - m) * st;
  }
}

// Block sum of s in a fixed order (a butterfly within each wave, then the
// waves' sums in order); every thread gets it.  The caller separates two
// calls with a barrier.
__device__ __forceinline__ double block_sum(double s) {
  __shared__ double sh[BS / 64];
#pragma unroll
  for (int m = 32; m > 0; m >>= 1) s = s + __shfl_xor(s, m, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
  __syncthreads();
  double t = sh[0];
#pragma unroll
  for (int w = 1; w < BS / 64; ++w) t = t + sh[w];
  return t;
}

// Sum of a reduction's block sums in a fixed order, in one block (thread 0
// holds it).
__device__ __forceinline__ double sum_parts(const double* __restrict__ part, int nb) {
  double s = 0.0;
  for (int i = threadIdx.x; i < nb; i += BS) s = s + part[i];
  return block_sum(s);
}

// beta = (r, r) / (r, r) of the previous iteration (0 in the first) from
// the nb block sums of (r, r); every block adds them in the same order, and
// block 0 keeps this iteration's (r, r) for the next one and for alpha.
__device__ __forceinline__ double cg_beta(const double* __restrict__ part_rr, int nb, double* __restrict__ sc, int it) {
  double beta = 0.0;
  if (it > 0) {
    const double rr = sum_parts(part_rr, nb);
    const double old = sc[SC_CG_RR + ((it - 1) & 1)];
    beta = old != 0.0 ? rr / old : 0.0;
    if (blockIdx.x == 0 && threadIdx.x == 0) sc[SC_CG_RR + (it & 1)] = rr;
    __syncthreads();
  }
  return beta;
}

// Work units of k_cg_apply: BS consecutive cells (a unit per x row left 160 of
// 256 lanes idle on rows of 96: 28.6 us an iteration at 96^3 against 25.7, a
// step at 32^3 0.80 against 0.56 ms); each block takes a contiguous run of
// units, and the runs of the blocks one XCD receives (blocks go to the XCDs in
// turn) are contiguous, so the rows a row's stencil reaches are mostly read
// through the same L2.
// Cell indices are 32-bit (the host takes this path below 2^31 cells).
template <int DIM>
__global__ __launch_bounds__(BS) void k_cg_apply(Params P, const double* __restrict__ d_dt, const double* __restrict__ r,
                                                 const double* __restrict__ pold, double* __restrict__ pnew,
                                                 const double* __restrict__ tau, const double* __restrict__ irc,
                                                 const double* __restrict__ irc2, double* __restrict__ q,
                                                 const double* __restrict__ part_rr, int nb_rr,
                                                 double* __restrict__ part_pq, double* __restrict__ sc, int it,
                                                 int wallmask) {
  const double beta = cg_beta(part_rr, nb_rr, sc, it);
  const double dt = *d_dt;
  const int axes[3] = {0, DIM == 3 ? 1 : 2, 2};
  const int ext[3] = {P.nx, P.ny, P.nz};
  const int str[3] = {1, P.nx, P.nx * P.ny};
  double lam[DIM];
#pragma unroll
  for (int t = 0; t < DIM; ++t) lam[t] = dt / P.dx[axes[t]];
  const double hK = P.hK;
  const int units = (int)((P.ncell + BS - 1) / BS);
  const unsigned G = gridDim.x, b = blockIdx.x;
  const unsigned lw = (G % 8 == 0) ? (b % 8) * (G / 8) + b / 8 : b;
  const int u0 = (int)((long long)units * lw / G), u1 = (int)((long long)units * (lw + 1) / G);
  double s = 0.0;
  for (int u = u0; u < u1; ++u) {
    const unsigned cu = (unsigned)u * BS + threadIdx.x;
    if (cu >= (unsigned)P.ncell) continue;
    const int c = (int)cu;
    int crd[3];
    coords32(cu, (unsigned)P.nx, (unsigned)P.ny, crd[0], crd[1], crd[2]);
    const double P0 = r[c] + beta * pold[c];
    const double t0 = tau[c], i0 = irc[c];
    double div = 0.0;
#pragma unroll
    for (int t = 0; t < DIM; ++t) {
      const int a = axes[t];
      const bool wall = (wallmask >> a) & 1;
      int om2, om1, op1, op2;
      nb_offsets(crd[a], ext[a], str[a], wall, om2, om1, op1, op2);
      const double Pm2 = r[c + om2] + beta * pold[c + om2];
      const double Pm1 = r[c + om1] + beta * pold[c + om1];
      const double Pp1 = r[c + op1] + beta * pold[c + op1];
      const double Pp2 = r[c + op2] + beta * pold[c + op2];
      // velocities of the cells c - e, c, c + e: u = -lambda tau [Pi*],
      // [Pi*] = (Pi_{+1} - Pi_{-1}) / 2 of the cell's neighbours
      const double um = -(lam[t] * tau[c + om1]) * (0.5 * (P0 - Pm2));
      const double uc = -(lam[t] * t0) * (0.5 * (Pp1 - Pm1));
      const double up = -(lam[t] * tau[c + op1]) * (0.5 * (Pp2 - P0));
      // u* of the faces c - e | c and c | c + e (0 on a wall face)
      double usm = 0.5 * (um + uc) - (P0 - Pm1) * (hK * dmin2(irc[c + om1], i0));
      double usp = 0.5 * (uc + up) - (Pp1 - P0) * (hK * dmin2(i0, irc[c + op1]));
      if (wall && crd[a] == 0) usm = 0.0;
      if (wall && crd[a] == ext[a] - 1) usp = 0.0;
      div = div + lam[t] * (usp - usm);
    }
    const double y = P0 * irc2[c] + div;
    pnew[c] = P0;
    q[c] = y;
    s = s + P0 * y;
  }
  const double tot = block_sum(s);
  if (threadIdx.x == 0) part_pq[blockIdx.x] = tot;
}

// The 2D product goes through LDS: a tile of CT_X x CT_Z cells stages p
// with its halo of 2 (periodic images or, on a walled axis, the wall cell),
// and tau and 1/(rho c) with their halo of 1, so each value is read from
// memory once per tile instead of once per stencil point (29 loads a cell
// become about 8).  Tiles in row-major order, a contiguous run per block
// and the blocks of one XCD together, as above.
constexpr int CT_X = 64, CT_Z = 16;
constexpr int CP_X = CT_X + 4, CP_Z = CT_Z + 4;  // p with halo 2
constexpr int CC_X = CT_X + 2, CC_Z = CT_Z + 2;  // tau, 1/(rho c) with halo 1
static_assert((CT_X * CT_Z) % BS == 0 && CT_X % 64 == 0, "tile rows are whole waves");

// One whole CG iteration in 2D, i >= 0, in one kernel.  From the previous
// iteration's r, q = A p and p (stencil reads through the LDS tile) and the
// block sums of its (p, q), (r, q), (q, q), (r, r): alpha = (r, r) / (p, q),
// the new (r, r) = (r, r) - 2 alpha (r, q) + alpha^2 (q, q) (the expansion
// of |r - alpha q|^2 over one step from exact sums: no drift accumulates),
// beta = new (r, r) / (r, r); then at every cell r' = r - alpha q,
// p' = r' + beta p, x += alpha p (own cells), q' = A p', and the block sums
// of (p', q'), (r', q'), (q', q') and the exact (r', r').  Iteration 0 takes
// alpha = beta = 0 (r' = r, p' = r).  Four sums per block in the layout
// part[k * pstride + block].
template <int NT>
__device__ __forceinline__ void block_sum4(double (&v)[4]) {
  __shared__ double sh4[4][NT / 64];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) v[k] = v[k] + __shfl_xor(v[k], m, 64);
  }
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int k = 0; k < 4; ++k) sh4[k][threadIdx.x >> 6] = v[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    double t = sh4[k][0];
#pragma unroll
    for (int w = 1; w < NT / 64; ++w) t = t + sh4[k][w];
    v[k] = t;
  }
}

enum { CGS_PQ = 0, CGS_RQ, CGS_QQ, CGS_RR };

// alpha and beta of an iteration from the previous one's block sums.
template <int NT>
__device__ __forceinline__ void cg_scalars(const double* __restrict__ pprev, int pstride, double& alpha,
                                           double& beta) {
  double v[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    double a = 0.0;
    for (int i = threadIdx.x; i < (int)gridDim.x; i += NT) a = a + pprev[k * pstride + i];
    v[k] = a;
  }
  block_sum4<NT>(v);
  const double rr = v[CGS_RR];
  alpha = v[CGS_PQ] != 0.0 ? rr / v[CGS_PQ] : 0.0;
  const double rrn = (rr - 2.0 * alpha * v[CGS_RQ]) + (alpha * alpha) * v[CGS_QQ];
  beta = rr != 0.0 ? rrn / rr : 0.0;
  __syncthreads();
}

__global__ __launch_bounds__(BS) void k_cg_iter_2d(Params P, const double* __restrict__ d_dt,
                                                   const double* __restrict__ rin, const double* __restrict__ qin,
                                                   const double* __restrict__ pin, double* __restrict__ rout,
                                                   double* __restrict__ qout, double* __restrict__ pout,
                                                   double* __restrict__ x, const double* __restrict__ tau,
                                                   const double* __restrict__ irc, const double* __restrict__ irc2,
                                                   const double* __restrict__ pprev, double* __restrict__ pcur,
                                                   int pstride, int it, int wallmask) {
  __shared__ double sP[CP_Z][CP_X];
  __shared__ double sT[CC_Z][CC_X];
  __shared__ double sI[CC_Z][CC_X];
  __shared__ double sR[CT_Z][CT_X];
  __shared__ int colm[CP_X];
  __shared__ int rowm[CP_Z];
  double alpha = 0.0, beta = 0.0;
  if (it > 0) cg_scalars<BS>(pprev, pstride, alpha, beta);
  const double dt = *d_dt;
  const double lx = dt / P.dx[0], lz = dt / P.dx[2], hK = P.hK;
  const int nx = P.nx, nz = P.nz;
  const bool wx = wallmask & 1, wz = (wallmask >> 2) & 1;
  const int tx = (nx + CT_X - 1) / CT_X;
  const int tiles = tx * ((nz + CT_Z - 1) / CT_Z);
  const unsigned G = gridDim.x, b = blockIdx.x;
  const unsigned lw = (G % 8 == 0) ? (b % 8) * (G / 8) + b / 8 : b;
  const int t0 = (int)((long long)tiles * lw / G), t1 = (int)((long long)tiles * (lw + 1) / G);
  const int tid = threadIdx.x;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  for (int t = t0; t < t1; ++t) {
    const int x0 = (t % tx) * CT_X, z0 = (t / tx) * CT_Z;
    if (tid < CP_X) {
      const int v = x0 + tid - 2;
      int g = v % nx;
      g = g < 0 ? g + nx : g;
      colm[tid] = wx ? (v < 0 ? 0 : (v < nx ? v : nx - 1)) : g;
    } else if (tid < CP_X + CP_Z) {
      const int v = z0 + (tid - CP_X) - 2;
      int g = v % nz;
      g = g < 0 ? g + nz : g;
      rowm[tid - CP_X] = (wz ? (v < 0 ? 0 : (v < nz ? v : nz - 1)) : g) * nx;
    }
    __syncthreads();
    for (int e = tid; e < CP_X * CP_Z; e += BS) {
      const int j = e / CP_X, i = e - j * CP_X;
      const int idx = rowm[j] + colm[i];
      const double pp = pin[idx];
      const double rv = rin[idx] - alpha * qin[idx];
      const double pv = rv + beta * pp;
      sP[j][i] = pv;
      if (j >= 2 && j < CT_Z + 2 && i >= 2 && i < CT_X + 2 && x0 + i - 2 < nx && z0 + j - 2 < nz) {
        rout[idx] = rv;
        pout[idx] = pv;
        x[idx] = x[idx] + alpha * pp;
        sR[j - 2][i - 2] = rv;
        acc[CGS_RR] = acc[CGS_RR] + rv * rv;
      }
    }
    for (int e = tid; e < CC_X * CC_Z; e += BS) {
      const int j = e / CC_X, i = e - j * CC_X;
      const int idx = rowm[j + 1] + colm[i + 1];
      sT[j][i] = tau[idx];
      sI[j][i] = irc[idx];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < CT_X * CT_Z / BS; ++k) {
      const int e = tid + k * BS;
      const int i = e % CT_X, j = e / CT_X;
      const int gx = x0 + i, gz = z0 + j;
      if (gx < nx && gz < nz) {
        const double P0 = sP[j + 2][i + 2], t0c = sT[j + 1][i + 1], i0 = sI[j + 1][i + 1];
        double div = 0.0;
        {  // x: velocities of the cells c - e, c, c + e, then u* of the two faces
          const double Pm2 = sP[j + 2][i], Pm1 = sP[j + 2][i + 1], Pp1 = sP[j + 2][i + 3], Pp2 = sP[j + 2][i + 4];
          const double um = -(lx * sT[j + 1][i]) * (0.5 * (P0 - Pm2));
          const double uc = -(lx * t0c) * (0.5 * (Pp1 - Pm1));
          const double up = -(lx * sT[j + 1][i + 2]) * (0.5 * (Pp2 - P0));
          double usm = 0.5 * (um + uc) - (P0 - Pm1) * (hK * dmin2(sI[j + 1][i], i0));
          double usp = 0.5 * (uc + up) - (Pp1 - P0) * (hK * dmin2(i0, sI[j + 1][i + 2]));
          if (wx && gx == 0) usm = 0.0;
          if (wx && gx == nx - 1) usp = 0.0;
          div = div + lx * (usp - usm);
        }
        {  // z
          const double Pm2 = sP[j][i + 2], Pm1 = sP[j + 1][i + 2], Pp1 = sP[j + 3][i + 2], Pp2 = sP[j + 4][i + 2];
          const double um = -(lz * sT[j][i + 1]) * (0.5 * (P0 - Pm2));
          const double uc = -(lz * t0c) * (0.5 * (Pp1 - Pm1));
          const double up = -(lz * sT[j + 2][i + 1]) * (0.5 * (Pp2 - P0));
          double usm = 0.5 * (um + uc) - (P0 - Pm1) * (hK * dmin2(sI[j][i + 1], i0));
          double usp = 0.5 * (uc + up) - (Pp1 - P0) * (hK * dmin2(i0, sI[j + 2][i + 1]));
          if (wz && gz == 0) usm = 0.0;
          if (wz && gz == nz - 1) usp = 0.0;
          div = div + lz * (usp - usm);
        }
        const int c = gz * nx + gx;
        const double y = P0 * irc2[c] + div;
        qout[c] = y;
        acc[CGS_PQ] = acc[CGS_PQ] + P0 * y;
        acc[CGS_RQ] = acc[CGS_RQ] + sR[j][i] * y;
        acc[CGS_QQ] = acc[CGS_QQ] + y * y;
      }
    }
    __syncthreads();  // the next tile overwrites the LDS
  }
  block_sum4<BS>(acc);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < 4; ++k) pcur[k * pstride + blockIdx.x] = acc[k];
  }
}

// The same iteration in 3D: a unit is a 32 x 16 column of cells over zc planes,
// one thread a column.  A column's own values of five planes stay in
// registers; a plane's p, tau and 1/(rho c) go to LDS for the lateral
// neighbours, with the halo (2 for p, 1 for the others, no corners) read by
// 192 of the 512 threads; two LDS planes in turn, one barrier a plane, the
// next plane's loads in flight meanwhile.  Memory bounds it: 11 values a cell
// are read or written, and some 4 more for the halo (loads two planes ahead
// change nothing).  Against k_cg_apply and k_cg_xr, which read 41 and 4 values
// a cell in two launches, us an iteration: 32^3 14, 13; 96^3 38, 30; 128^3
// 69, 47; 200^3 342, 221.
constexpr int C3_X = 32, C3_Y = 16, C3_T = C3_X * C3_Y;
constexpr int C3_PX = C3_X + 4, C3_PY = C3_Y + 4;

__device__ __forceinline__ int image_of(int v, int n, bool wall) {
  if (wall) return v < 0 ? 0 : (v < n ? v : n - 1);
  const int g = v % n;
  return g < 0 ? g + n : g;
}

__global__ __launch_bounds__(C3_T) void k_cg_iter_3d(Params P, const double* __restrict__ d_dt,
                                                     const double* __restrict__ rin, const double* __restrict__ qin,
                                                     const double* __restrict__ pin, double* __restrict__ rout,
                                                     double* __restrict__ qout, double* __restrict__ pout,
                                                     double* __restrict__ x, const double* __restrict__ tau,
                                                     const double* __restrict__ irc, const double* __restrict__ irc2,
                                                     const double* __restrict__ pprev, double* __restrict__ pcur,
                                                     int pstride, int it, int wallmask, int zc) {
  __shared__ double sP[2][C3_PY * C3_PX];
  __shared__ double sT[2][C3_PY * C3_PX];
  __shared__ double sI[2][C3_PY * C3_PX];
  double alpha = 0.0, beta = 0.0;
  if (it > 0) cg_scalars<C3_T>(pprev, pstride, alpha, beta);
  const double dt = *d_dt, hK = P.hK;
  const double lx = dt / P.dx[0], ly = dt / P.dx[1], lz = dt / P.dx[2];
  const int nx = P.nx, ny = P.ny, nz = P.nz, nxy = nx * ny;
  const bool wx = wallmask & 1, wy = (wallmask >> 1) & 1, wz = (wallmask >> 2) & 1;
  const int ntx = (nx + C3_X - 1) / C3_X, nty = (ny + C3_Y - 1) / C3_Y, nch = (nz + zc - 1) / zc;
  const long long units = (long long)ntx * nty * nch;
  const unsigned G = gridDim.x, b = blockIdx.x;
  const unsigned lw = (G % 8 == 0) ? (b % 8) * (G / 8) + b / 8 : b;
  const long long u0 = units * lw / G, u1 = units * (lw + 1) / G;
  const int tid = threadIdx.x, tx = tid % C3_X, ty = tid / C3_X;
  const int pos = (ty + 2) * C3_PX + tx + 2;
  // halo position of this thread: rows -2, -1, C3_Y, C3_Y + 1, then columns;
  // tau and 1/(rho c) at the inner ones
  int hx = tx, hy = ty;
  bool inner = false;
  const bool halo = tid < 4 * (C3_X + C3_Y);
  if (tid < 4 * C3_X) {
    const int k = tid / C3_X;
    hy = k < 2 ? k - 2 : C3_Y + k - 2;
    inner = k == 1 || k == 2;
  } else if (halo) {
    const int h = tid - 4 * C3_X, k = h / C3_Y;
    hy = h % C3_Y;
    hx = k < 2 ? k - 2 : C3_X + k - 2;
    inner = k == 1 || k == 2;
  }
  const int hpos = (hy + 2) * C3_PX + hx + 2;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  int s = 0;
  for (long long u = u0; u < u1; ++u) {
    const int tile = (int)(u / nch), z0 = (int)(u - (long long)tile * nch) * zc, z1 = min(z0 + zc, nz);
    const int x0 = (tile % ntx) * C3_X, y0 = (tile / ntx) * C3_Y;
    const int gx = x0 + tx, gy = y0 + ty;
    const bool in = gx < nx && gy < ny;
    const int col = image_of(gx, nx, wx) + nx * image_of(gy, ny, wy);
    const int hcol = image_of(x0 + hx, nx, wx) + nx * image_of(y0 + hy, ny, wy);
    // loads of step v: r, q, p (and x) of plane v, tau and 1/(rho c) of v - 1,
    // the halo and 1/(rho c^2) of v - 2
    double nr, nq, np, nX = 0.0, nt = 0.0, ni = 0.0, nc = 0.0, hr = 0.0, hq = 0.0, hp = 0.0, ht = 0.0, hi = 0.0;
    auto load = [&](int v) __attribute__((always_inline)) {
      const int i = image_of(v, nz, wz) * nxy + col;
      nr = rin[i];
      nq = qin[i];
      np = pin[i];
      if (v >= z0 && v < z1) nX = x[i];
      if (v >= z0) {
        const int j = image_of(v - 1, nz, wz) * nxy + col;
        nt = tau[j];
        ni = irc[j];
      }
      if (v >= z0 + 2) {
        const int z = (v - 2) * nxy;
        nc = irc2[z + col];
        if (halo) {
          hr = rin[z + hcol];
          hq = qin[z + hcol];
          hp = pin[z + hcol];
          if (inner) {
            ht = tau[z + hcol];
            hi = irc[z + hcol];
          }
        }
      }
    };
    load(z0 - 2);
    double p0 = 0, p1 = 0, p2 = 0, p3 = 0, p4 = 0;  // p of planes v - 4 .. v
    double r2 = 0, r3 = 0, r4 = 0;                  // r of planes v - 2 .. v
    double t1 = 0, t2 = 0, t3 = 0, i1 = 0, i2 = 0, i3 = 0;  // of planes v - 3 .. v - 1
    for (int v = z0 - 2; v <= z1 + 1; ++v) {
      const double pold = np, xo = nX, ic2 = nc;
      p0 = p1; p1 = p2; p2 = p3; p3 = p4;
      r2 = r3; r3 = r4;
      t1 = t2; t2 = t3; i1 = i2; i2 = i3;
      t3 = nt; i3 = ni;
      r4 = nr - alpha * nq;
      p4 = r4 + beta * pold;
      const int z = v - 2;
      if (z >= z0) {
        sP[s][pos] = p2;
        sT[s][pos] = t2;
        sI[s][pos] = i2;
        if (halo) {
          sP[s][hpos] = (hr - alpha * hq) + beta * hp;
          if (inner) {
            sT[s][hpos] = ht;
            sI[s][hpos] = hi;
          }
        }
      }
      if (v <= z1) load(v + 1);
      if (v >= z0 && v < z1 && in) {
        const int i = v * nxy + col;
        rout[i] = r4;
        pout[i] = p4;
        x[i] = xo + alpha * pold;
        acc[CGS_RR] = acc[CGS_RR] + r4 * r4;
      }
      if (z < z0) continue;
      __syncthreads();
      // velocities of the cells c - e, c, c + e of an axis, then u* of the two
      // faces (0 on a wall face)
      auto axis = [&](double lam, double Pm2, double Pm1, double Pp1, double Pp2, double tm, double tp, double im,
                      double ip, bool first, bool last) __attribute__((always_inline)) {
        const double um = -(lam * tm) * (0.5 * (p2 - Pm2));
        const double uc = -(lam * t2) * (0.5 * (Pp1 - Pm1));
        const double up = -(lam * tp) * (0.5 * (Pp2 - p2));
        double usm = 0.5 * (um + uc) - (p2 - Pm1) * (hK * dmin2(im, i2));
        double usp = 0.5 * (uc + up) - (Pp1 - p2) * (hK * dmin2(i2, ip));
        if (first) usm = 0.0;
        if (last) usp = 0.0;
        return lam * (usp - usm);
      };
      double div = 0.0;
      div = div + axis(lx, sP[s][pos - 2], sP[s][pos - 1], sP[s][pos + 1], sP[s][pos + 2], sT[s][pos - 1],
                       sT[s][pos + 1], sI[s][pos - 1], sI[s][pos + 1], wx && gx == 0, wx && gx == nx - 1);
      div = div + axis(ly, sP[s][pos - 2 * C3_PX], sP[s][pos - C3_PX], sP[s][pos + C3_PX], sP[s][pos + 2 * C3_PX],
                       sT[s][pos - C3_PX], sT[s][pos + C3_PX], sI[s][pos - C3_PX], sI[s][pos + C3_PX],
                       wy && gy == 0, wy && gy == ny - 1);
      div = div + axis(lz, p0, p1, p3, p4, t1, t3, i1, i3, wz && z == 0, wz && z == nz - 1);
      if (in) {
        const double y = p2 * ic2 + div;
        qout[z * nxy + col] = y;
        acc[CGS_PQ] = acc[CGS_PQ] + p2 * y;
        acc[CGS_RQ] = acc[CGS_RQ] + r2 * y;
        acc[CGS_QQ] = acc[CGS_QQ] + y * y;
      }
      s ^= 1;
    }
  }
  block_sum4<C3_T>(acc);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < 4; ++k) pcur[k * pstride + blockIdx.x] = acc[k];
  }
}

// alpha = (r, r) / (p, q), every block adding the block sums of (p, q) in
// the same order; then x += alpha p, r -= alpha q and the block sums of
// the new (r, r).
__global__ __launch_bounds__(BS) void k_cg_xr(long long n, const double* __restrict__ p, const double* __restrict__ q,
                                              double* __restrict__ x, double* __restrict__ r,
                                              const double* __restrict__ part_pq, int nb_pq,
                                              double* __restrict__ part_rr, const double* __restrict__ sc, int it) {
  const double pq = sum_parts(part_pq, nb_pq);
  const double alpha = pq != 0.0 ? sc[SC_CG_RR + (it & 1)] / pq : 0.0;
  __syncthreads();
  double s = 0.0;
  for (long long i = (long long)blockIdx.x * BS + threadIdx.x; i < n; i += (long long)gridDim.x * BS) {
    x[i] = x[i] + alpha * p[i];
    const double ri = r[i] - alpha * q[i];
    r[i] = ri;
    s = s + ri * ri;
  }
  const double tot = block_sum(s);
  if (threadIdx.x == 0) part_rr[blockIdx.x] = tot;
}

// (r, r) of the last iteration, for the host's convergence test.
__global__ __launch_bounds__(BS) void k_cg_check(const double* __restrict__ part_rr, int nb, double* __restrict__ sc) {
  const double rr = sum_parts(part_rr, nb);
  if (threadIdx.x == 0) sc[SC_CG_CHK] = rr;
}

// x0 = p^n of every interior cell.
template <int DIM>
__global__ void k_imex_x0(Params P, RefGrid G, const double* __restrict__ W, double* __restrict__ x) {
  const long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= P.ncell) return;
  int cxx, cyy, czz;
  coords32((unsigned)c, (unsigned)P.nx, (unsigned)P.ny, cxx, cyy, czz);
  x[c] = W[R_P * G.npad + G.pad(cxx + 2, DIM == 3 ? cyy + 2 : 0, czz + 2)];
}

__global__ void k_fill0(long long n, double* __restrict__ a) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) a[i] = 0.0;
}

__global__ void k_neg(long long n, double* __restrict__ a) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) a[i] = -a[i];
}

__global__ void k_add_t(double* __restrict__ t, const double* __restrict__ dt) {
  if (threadIdx.x == 0) *t = *t + *dt;
}

unsigned nblk(long long n) { return (unsigned)((n + BS - 1) / BS); }

template <int DIM>
struct Imex {
  const Params& P;
  ImexLayout L;
  hipStream_t s;
  const double* d_dt;

  hipError_t apply(const double* xin, double* y, int cst) {
    const unsigned np = nblk(L.G.npad);
    hipLaunchKernelGGL(k_schur_extP<DIM>, dim3(np), dim3(BS), 0, s, P, L.G, L.W, xin, cst, L.ext);
    if (P.low_mach)
      hipLaunchKernelGGL((k_schur_u<DIM, true>), dim3(np), dim3(BS), 0, s, P, L.G, L.W, d_dt, cst, L.ext);
    else
      hipLaunchKernelGGL((k_schur_u<DIM, false>), dim3(np), dim3(BS), 0, s, P, L.G, L.W, d_dt, cst, L.ext);
    hipLaunchKernelGGL(k_schur_rows<DIM>, dim3(nblk(P.ncell)), dim3(BS), 0, s, P, L.G, L.W, L.ext, d_dt, xin, cst, y);
    return hipGetLastError();
  }
  void dot(const double* a, const double* b, int slot) {
    hipLaunchKernelGGL(k_dot_partial, dim3(DOT_BLOCKS), dim3(BS), 0, s, a, b, L.n, L.part);
    hipLaunchKernelGGL(k_dot_final, dim3(1), dim3(BS), 0, s, L.part, DOT_BLOCKS, L.sc + slot);
  }
  int read(int slot, double* h) {
    if (hipMemcpyAsync(h, L.sc + slot, sizeof(double), hipMemcpyDeviceToHost, s) != hipSuccess) return ARS_EDEVICE;
    return hipStreamSynchronize(s) == hipSuccess ? ARS_OK : ARS_EDEVICE;
  }

  // Solve the implicit system of the state whose primitives and explicit
  // faces are in the workspace; returns iterations in *its.
  int solve(double tol, int max_iter, int* its) {
    const unsigned nb = nblk(L.n);
    // b = -F(0); x0 = explicit values; r = b - L x0
    hipLaunchKernelGGL(k_fill0, dim3(nb), dim3(BS), 0, s, L.n, L.t);
    if (apply(L.t, L.b, 1) != hipSuccess) return ARS_EDEVICE;
    hipLaunchKernelGGL(k_neg, dim3(nb), dim3(BS), 0, s, L.n, L.b);
    hipLaunchKernelGGL(k_imex_x0<DIM>, dim3(nblk(P.ncell)), dim3(BS), 0, s, P, L.G, L.W, L.x);
    if (apply(L.x, L.r, 0) != hipSuccess) return ARS_EDEVICE;
    hipLaunchKernelGGL(k_bicg_start, dim3(nb), dim3(BS), 0, s, L.n, L.b, L.r, L.rh, L.p, L.v, L.sc);
    dot(L.b, L.b, SC_BB);
    double bb = 0.0;
    if (read(SC_BB, &bb) != ARS_OK) return ARS_EDEVICE;
    const double target = tol * tol * (bb > 0.0 ? bb : 1.0);
    // the explicit pressure may already solve the system (an equilibrium)
    dot(L.r, L.r, SC_RR);
    double rr0 = 0.0;
    if (read(SC_RR, &rr0) != ARS_OK) return ARS_EDEVICE;
    if (!std::isfinite(rr0)) return ARS_ENOCONV;
    if (rr0 <= target) {
      if (its) *its = 0;
      return ARS_OK;
    }
    int it = 0;
    for (; it < max_iter; ++it) {
      dot(L.rh, L.r, SC_RHO_NEW);
      hipLaunchKernelGGL(k_bicg_p, dim3(nb), dim3(BS), 0, s, L.n, L.r, L.v, L.p, L.sc);
      if (apply(L.p, L.v, 0) != hipSuccess) return ARS_EDEVICE;
      dot(L.rh, L.v, SC_RV);
      hipLaunchKernelGGL(k_bicg_s, dim3(nb), dim3(BS), 0, s, L.n, L.r, L.v, L.sv, L.sc);
      if (apply(L.sv, L.t, 0) != hipSuccess) return ARS_EDEVICE;
      dot(L.t, L.sv, SC_TS);
      dot(L.t, L.t, SC_TT);
      hipLaunchKernelGGL(k_bicg_xr, dim3(nb), dim3(BS), 0, s, L.n, L.p, L.sv, L.t, L.x, L.r, L.sc);
      hipLaunchKernelGGL(k_bicg_scalars, dim3(1), dim3(64), 0, s, L.sc);
      if (it % 4 == 3 || it + 1 == max_iter) {
        dot(L.r, L.r, SC_RR);
        double rr = 0.0;
        if (read(SC_RR, &rr) != ARS_OK) return ARS_EDEVICE;
        if (!std::isfinite(rr)) return ARS_ENOCONV;
        if (rr <= target) {
          ++it;
          break;
        }
      }
    }
    if (its) *its = it;
    if (it >= max_iter) {
      double rr = 0.0;
      if (read(SC_RR, &rr) != ARS_OK) return ARS_EDEVICE;
      if (!(rr <= target)) return ARS_ENOCONV;
    }
    return hipGetLastError() == hipSuccess ? ARS_OK : ARS_EDEVICE;
  }

  // Conjugate gradients on the same system of the state U (every axis periodic
  // or walled; imex_begin forms it).  The BiCGSTAB-only vectors hold the
  // coefficients (rh: tau, sv: 1/(rho c), t: 1/(rho c^2)) and, in b, the
  // second p.
  int solve_cg(const double* U, double tol, int max_iter, int* its) {
    const unsigned nb = nblk(L.n);
    // bit a: the physical axis a is walled at both ends (a configuration
    // admits walls on the vertical axis only; the products take the mask
    // per axis all the same)
    const int wallmask = (P.bcx[0] == BC_WALL ? 1 : 0) | (DIM == 3 && P.bcy[0] == BC_WALL ? 2 : 0) |
                         (P.bcz[0] == BC_WALL ? 4 : 0);
    const unsigned gb = nb < (unsigned)CG_BLOCKS ? nb : (unsigned)CG_BLOCKS;
    static_assert(SC_CG_RR == SC_BB + 1 && SC_DT == SC_RANGE + 6 && IMEX_BEGIN_BLOCKS <= CG_BLOCKS, "imex_begin");
    const ImexSystem S{L.x, L.r, L.p, L.v, L.rh, L.sv, L.t, L.part, L.sc + SC_BB, L.sc + SC_RANGE};
    if (imex_begin(P, U, L.W, L.ext, d_dt, S, s) != hipSuccess) return ARS_EDEVICE;
    double h[SC_N];
    if (hipMemcpyAsync(h, L.sc, SC_N * sizeof(double), hipMemcpyDeviceToHost, s) != hipSuccess) return ARS_EDEVICE;
    if (hipStreamSynchronize(s) != hipSuccess) return ARS_EDEVICE;
    const double bb = h[SC_BB], rr0 = h[SC_CG_RR];
    const double target = tol * tol * (bb > 0.0 ? bb : 1.0);
    if (!std::isfinite(rr0)) return ARS_ENOCONV;
    if (rr0 <= target) {
      if (its) *its = 0;
      return ARS_OK;
    }
    TrigCoef tc;
    if (prefer_trig(h, std::sqrt(rr0 / target), max_iter, &tc)) return iterate_trig(target, max_iter, its, tc, gb, wallmask);
    return iterate_cg(target, max_iter, its, wallmask);
  }

  // Scratch of the trigonometric preconditioner: the reference workspace from
  // L on holds nothing while the system is solved (cell values, fluxes).
  double* trig_scratch() { return L.W + (size_t)R_L * L.G.npad; }
  size_t trig_room() const { return (size_t)(R_NFIELD - R_L) * L.G.npad; }

  // Whether conjugate gradients with the trigonometric preconditioner
  // (ars_trig.hip) take less time than without, for a reduction of the
  // residual by `red`, from what both need at most: with the condition
  // number k of the iterated operator, log(2 red) / log((sqrt k + 1) /
  // (sqrt k - 1)) iterations.  Preconditioned, k is at most the largest
  // max/min ratio of the three coefficients (the reference values are their
  // geometric means).  Without, k is the largest eigenvalue over the smallest
  // and the bound more than what is seen (736 against 2300 at acoustic CFL 275
  // on the 1024^2 vortex, 75 against 130 at CFL 30 on 64^2), so 0.4 of it is
  // taken, and half a block of CG_CHECK iterations for the late read of the
  // residual.  Time per iteration as measured (with the host's
  // reads): without, 12.9 us at 64^2, 13.2 at 512^2, 27.8 at 1024^2 in 2D and
  // 13 us at 32^3, 30 at 96^3, 221 at 200^3; with, 68 us at 64^2 (the transforms'
  // launches, product, updates and a read of the residual), 330 at 1024^2, where
  // the expression below gives 341: TRIG_RATE counts a transform as the full
  // product of 2 n flop a value, which its half products do in 52 us (41 TF/s
  // so counted) where 62 are allowed, so near the line the plain iteration is
  // taken.  Boxes with ny nz beyond 2^21 have not been run with it.
  bool prefer_trig(const double* h, double red, int max_iter, TrigCoef* tc) const {
    const double n = (double)L.n;
    if (P.nx > TRIG_MAXN || P.ny > TRIG_MAXN || P.nz > TRIG_MAXN || (long long)P.ny * P.nz > (1 << 21) ||
        trig_scratch_doubles(P) > trig_room())
      return false;
    double ratio = 1.0, ref[3];
    for (int k = 0; k < 3; ++k) {
      const double lo = h[SC_RANGE + 2 * k], hi = h[SC_RANGE + 2 * k + 1];
      if (!(lo > 0.0) || !std::isfinite(hi)) return false;
      ratio = std::fmax(ratio, hi / lo);
      ref[k] = std::sqrt(lo * hi);
    }
    *tc = TrigCoef{ref[0], ref[1], ref[2]};
    double top = h[SC_RANGE + 1];
    for (int a = 0; a < 3; ++a) {
      if (a == 1 && DIM == 2) continue;
      const double lam = h[SC_DT] / P.dx[a];
      top += lam * lam * h[SC_RANGE + 3] + 4.0 * lam * P.hK * h[SC_RANGE + 5];
    }
    auto most = [&](double k) {
      const double s = std::sqrt(k);
      return s > 1.0 + 1e-12 ? std::log(2.0 * red) / std::log((s + 1.0) / (s - 1.0)) : 1.0;
    };
    const double with = 2.0 + most(ratio), without = 8.0 + 0.4 * most(top / h[SC_RANGE]);
    if (with > 0.5 * max_iter) return false;
    const double TRIG_RATE = 35e6, MEM = 3.7e6;  // flop and bytes per us
    double t_with = 35.0 + n * 150.0 / MEM;
    for (int a = 0; a < 3; ++a) {
      if (a == 1 && DIM == 2) continue;
      const double len = a == 0 ? P.nx : (a == 1 ? P.ny : P.nz);
      t_with += 2.0 * std::fmax(6.0, 2.0 * n * len / TRIG_RATE + n * 16.0 / MEM);
    }
    const double t_without = DIM == 2 ? std::fmax(12.5, 3.0 + n * 24e-6) : std::fmax(11.5, 9.0 + n * 23e-6);
    return 20.0 + with * t_with < without * t_without;
  }

  // Preconditioned conjugate gradients: z = M^-1 r, then k_cg_apply with z in
  // the place of r (p = z + beta p_old, q = A p; its beta and alpha come from
  // the sums of (r, z)) and k_cg_xr; the host reads (r, r) every iteration,
  // of which there are few.
  int iterate_trig(double target, int max_iter, int* its, const TrigCoef& tc, unsigned gb, int wallmask) {
    const int ps = CG_BLOCKS > DOT_BLOCKS ? CG_BLOCKS : DOT_BLOCKS;
    double* const part_pq = L.part;
    double* const part_rr = L.part + ps;
    double* const part_rz = L.part + 2 * ps;
    double* w = trig_scratch();
    if (trig_setup(P, tc, d_dt, w, s) != hipSuccess) return ARS_EDEVICE;
    double* pv[2] = {L.p, L.b};  // p = 0 on entry, so the first p is z
    for (int it = 0; it < max_iter; ++it) {
      const double* z = nullptr;
      if (trig_solve(P, tc, L.r, w, &z, s) != hipSuccess) return ARS_EDEVICE;
      hipLaunchKernelGGL(k_dot_partial, dim3(DOT_BLOCKS), dim3(BS), 0, s, L.r, z, L.n, part_rz);
      if (it == 0) hipLaunchKernelGGL(k_dot_final, dim3(1), dim3(BS), 0, s, part_rz, DOT_BLOCKS, L.sc + SC_CG_RR);
      hipLaunchKernelGGL(k_cg_apply<DIM>, dim3(gb), dim3(BS), 0, s, P, d_dt, z, pv[it & 1], pv[(it + 1) & 1], L.rh,
                         L.sv, L.t, L.v, part_rz, DOT_BLOCKS, part_pq, L.sc, it, wallmask);
      hipLaunchKernelGGL(k_cg_xr, dim3(gb), dim3(BS), 0, s, L.n, pv[(it + 1) & 1], L.v, L.x, L.r, part_pq, (int)gb,
                         part_rr, L.sc, it);
      hipLaunchKernelGGL(k_cg_check, dim3(1), dim3(BS), 0, s, part_rr, (int)gb, L.sc);
      double rr = 0.0;
      if (read(SC_CG_CHK, &rr) != ARS_OK) return ARS_EDEVICE;
      if (its) *its = it + 1;
      if (!std::isfinite(rr)) return ARS_ENOCONV;
      if (rr <= target) return hipGetLastError() == hipSuccess ? ARS_OK : ARS_EDEVICE;
    }
    return ARS_ENOCONV;
  }

  // One kernel an iteration (k_cg_iter_2d, k_cg_iter_3d).  Iteration i reads the
  // residual, product and direction of set (i + 1) & 1 and writes set i & 1
  // (set 1 starts as r0, 0, 0: imex_begin zeroed p and v), and its four
  // block sums go to sum set i & 1.
  int iterate_cg(double target, int max_iter, int* its, int wallmask) {
    unsigned ga = 1;
    int zc = 1;
    if (DIM == 2) {
      const long long tiles = (long long)((P.nx + CT_X - 1) / CT_X) * ((P.nz + CT_Z - 1) / CT_Z);
      ga = tiles < CG_BLOCKS ? (unsigned)tiles : (unsigned)CG_BLOCKS;
    } else {
      // planes a unit: the fewest for the busiest CU, a unit costing 1.5 more
      // for its halo planes; at most two workgroups are resident per CU
      const long long tiles = (long long)((P.nx + C3_X - 1) / C3_X) * ((P.ny + C3_Y - 1) / C3_Y);
      double best = 1e300;
      for (int ch = 1; ch <= P.nz && (ch == 1 || tiles * ch <= 512); ++ch) {
        const int c = (P.nz + ch - 1) / ch;
        const long long units = tiles * ((P.nz + c - 1) / c);
        const double cost = (double)((units + 255) / 256) * (c + 1.5);
        if (cost < best) {
          best = cost;
          zc = c;
          ga = (unsigned)std::min(512LL, units);
        }
      }
    }
    const int ps = CG_BLOCKS > DOT_BLOCKS ? CG_BLOCKS : DOT_BLOCKS;
    double* R[2] = {L.r2, L.r};
    double* Q[2] = {L.q2, L.v};
    double* Pv[2] = {L.b, L.p};
    double* S[2] = {L.part, L.part + 4 * ps};
    // kernel i applies the update of iteration i - 1 and starts its own; the
    // 2D count is of kernels, the 3D count of updates
    const int lead = DIM == 3 ? 1 : 0;
    int it = 0;  // iterations counted
    double rr = 0.0;
    for (int k = 0; it < max_iter; ++k) {
      const int o = k & 1, in = o ^ 1;
      if (DIM == 2)
        hipLaunchKernelGGL(k_cg_iter_2d, dim3(ga), dim3(BS), 0, s, P, d_dt, R[in], Q[in], Pv[in], R[o], Q[o], Pv[o],
                           L.x, L.rh, L.sv, L.t, S[in], S[o], ps, k, wallmask);
      else
        hipLaunchKernelGGL(k_cg_iter_3d, dim3(ga), dim3(C3_T), 0, s, P, d_dt, R[in], Q[in], Pv[in], R[o], Q[o],
                           Pv[o], L.x, L.rh, L.sv, L.t, S[in], S[o], ps, k, wallmask, zc);
      it = k + 1 - lead;
      if (it > 0 && (it % CG_CHECK == 0 || it == max_iter)) {
        hipLaunchKernelGGL(k_cg_check, dim3(1), dim3(BS), 0, s, S[o] + CGS_RR * ps, (int)ga, L.sc);
        if (read(SC_CG_CHK, &rr) != ARS_OK) return ARS_EDEVICE;
        if (!std::isfinite(rr)) return ARS_ENOCONV;
        if (rr <= target) break;
      }
    }
    if (its) *its = it;
    if (!(rr <= target)) return ARS_ENOCONV;
    return hipGetLastError() == hipSuccess ? ARS_OK : ARS_EDEVICE;
  }

  // The rest of the step with the implicit faces of x.
  hipError_t finish(double* Uout, Control* ctl) {
    const unsigned np = nblk(L.G.npad);
    hipLaunchKernelGGL(k_schur_extP<DIM>, dim3(np), dim3(BS), 0, s, P, L.G, L.W, L.x, 1, L.ext);
    if (P.low_mach) {
      hipLaunchKernelGGL((k_schur_u<DIM, true>), dim3(np), dim3(BS), 0, s, P, L.G, L.W, d_dt, 1, L.ext);
      hipLaunchKernelGGL((k_imex_faces<DIM, true>), dim3(np), dim3(BS), 0, s, P, L.G, L.W, L.ext);
    } else {
      hipLaunchKernelGGL((k_schur_u<DIM, false>), dim3(np), dim3(BS), 0, s, P, L.G, L.W, d_dt, 1, L.ext);
      hipLaunchKernelGGL((k_imex_faces<DIM, false>), dim3(np), dim3(BS), 0, s, P, L.G, L.W, L.ext);
    }
    hipLaunchKernelGGL(k_imex_cell<DIM>, dim3(np), dim3(BS), 0, s, P, L.G, d_dt, L.W);
    if (hipGetLastError() != hipSuccess) return hipErrorUnknown;
    return launch_ref_finish(P, L.W, Uout, d_dt, ctl, s);
  }
};

}  // namespace

size_t imex_workspace_bytes(const Params& P) {
  RefGrid G = make_grid(P);
  const long long n = P.ncell;
  auto al = [](size_t b) { return ((b + 255) / 256) * 256; };
  size_t s = al((size_t)R_NFIELD * G.npad * sizeof(double)) + al((size_t)(P.dim + 1) * G.npad * sizeof(double));
  s += 10 * al((size_t)n * sizeof(double));
  s += al(8 * (CG_BLOCKS > DOT_BLOCKS ? CG_BLOCKS : DOT_BLOCKS) * sizeof(double)) + al(SC_N * sizeof(double));
  return s;
}

template <int DIM>
static int imex_steps(const Params& P, double* d_state, double* d_tmp, Control* ctl, void* wimex, int nsteps,
                      const double* d_dt_sched, double* d_t, double tol, int max_iter, int* h_iters, hipStream_t s) {
  Imex<DIM> M{P, layout_of(P, wimex), s, nullptr};
  int total = 0;
  double* src = d_state;
  double* dst = d_tmp;
  // conjugate gradients, and the step in place, where the operator is
  // symmetric: every axis periodic or walled at both ends
  auto sym = [](const int* bc) {
    return (bc[0] == BC_PERIODIC && bc[1] == BC_PERIODIC) || (bc[0] == BC_WALL && bc[1] == BC_WALL);
  };
  const bool symmetric = sym(P.bcx) && sym(P.bcz) && (DIM == 2 || sym(P.bcy)) && P.nx >= 2 && P.nz >= 2 &&
                         (DIM == 2 || P.ny >= 2) && P.ncell < (1LL << 31) - (long long)BS;
  for (int st = 0; st < nsteps; ++st) {
    M.d_dt = d_dt_sched + st;
    int its = 0, rc;
    if (symmetric) {
      rc = M.solve_cg(d_state, tol, max_iter, &its);
    } else {
      if (launch_ref_forward(P, src, M.L.W, M.d_dt, s) != hipSuccess) return ARS_EDEVICE;
      rc = M.solve(tol, max_iter, &its);
    }
    total += its;
    if (rc != ARS_OK) {
      if (h_iters) *h_iters = total;
      return rc;
    }
    if (symmetric) {
      if (imex_finish(P, d_state, M.L.W, M.L.ext, M.L.x, M.d_dt, ctl, s) != hipSuccess) return ARS_EDEVICE;
    } else {
      if (M.finish(dst, ctl) != hipSuccess) return ARS_EDEVICE;
      std::swap(src, dst);
    }
    if (d_t) hipLaunchKernelGGL(k_add_t, dim3(1), dim3(64), 0, s, d_t, M.d_dt);
  }
  if (src != d_state &&
      hipMemcpyAsync(d_state, src, (size_t)(P.dim + 2) * P.ncell * sizeof(double), hipMemcpyDeviceToDevice, s) !=
          hipSuccess)
    return ARS_EDEVICE;
  if (h_iters) *h_iters = total;
  return hipGetLastError() == hipSuccess ? ARS_OK : ARS_EDEVICE;
}

int step_imex(const Params& P, double* d_state, double* d_tmp, Control* ctl, void* wimex, int nsteps,
              const double* d_dt_sched, double* d_t, double tol, int max_iter, int* h_iters, hipStream_t s) {
  return P.dim == 3 ? imex_steps<3>(P, d_state, d_tmp, ctl, wimex, nsteps, d_dt_sched, d_t, tol, max_iter, h_iters, s)
                    : imex_steps<2>(P, d_state, d_tmp, ctl, wimex, nsteps, d_dt_sched, d_t, tol, max_iter, h_iters, s);
}

}  // namespace ars
