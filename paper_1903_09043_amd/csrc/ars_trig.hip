// ars_trig.hip -- trigonometric preconditioner of the implicit acoustic
// system of ars_step_imex.
//
// With constant coefficients (1/(rho c^2), tau, 1/(rho c) of one reference
// state) the operator of that system is diagonal in real trigonometric modes:
// on a periodic axis of n cells in cas(2 pi k j / n) (cas = cos + sin, the
// Hartley kernel; theta_k = 2 pi k / n), on an axis walled at both ends in
// cos(pi k (j + 1/2) / n) (theta_k = pi k / n: the ghost Pi of a wall is the
// wall cell's, its even extension), with the eigenvalue
//   1/(rho c^2) + sum_d [ lambda_d^2 tau sin^2 theta_d
//                         + lambda_d (0.5/K) (1/(rho c)) 4 sin^2(theta_d / 2) ].
// M^-1 r is then one transform per axis, a division and the transforms back.
// In the low-Mach flows the implicit step is made for, the coefficients vary
// by Ma^2 and the system is solved in two or three iterations whatever the
// acoustic CFL number; the caller weighs it against plain iterations by the
// coefficients' range.
//
// A transform of any length is a product with an orthonormal n x n matrix,
// whose entries come from sincospi at an exponent reduced exactly in
// integers, and runs on the FP64 matrix cores: v_mfma_f64_16x16x4f64, a wave
// accumulating 32 x 32 outputs (4 operand loads for 4 matrix instructions of
// 32 cycles), four waves a 64 x 64 tile, both operands staged in LDS 32 deep
// and the next stage's global loads in flight behind the present one's
// products.  The pitch of 81 doubles serves both stores (along the tile and
// across it) and the operand reads of both forms without bank conflicts
// (one lane in 32 excepted).
// Measured on the Mach 1e-3 vortex at acoustic CFL 275, 1024^2 (one
// implicit step, residual 1e-10): 736 plain iterations, 20.5 ms; one
// preconditioned iteration, 0.81 ms.  What bounds it: the matrix
// instructions (4 products of 2.1 GFLOP) and the set-up around the solve.
#include <algorithm>

#include "ars_trig.h"

namespace ars {

namespace {

typedef double dbl4 __attribute__((ext_vector_type(4)));

constexpr int TM = 64, TN = 64, TK = 32;  // tile of the product: TM x TN outputs, TK deep
constexpr int PITCH = 81;

struct Axis {
  int n;         // cells
  bool wall;     // cosine modes (else Hartley)
  size_t fwd;    // offset of G[x][k]: weight of input x in output k
  size_t inv;    // offset of G^T (the same where G is symmetric)
  size_t eig;    // offset of the n eigenvalue parts
};

struct Plan {
  Axis a[3];  // x, y (n = 1 in 2D), z
  size_t f0, f1, total;
};

Plan plan_of(const Params& P) {
  Plan p{};
  size_t off = 0;
  auto take = [&](size_t count) {
    const size_t o = off;
    off += (count + 31) / 32 * 32;
    return o;
  };
  const int n[3] = {P.nx, P.dim == 3 ? P.ny : 1, P.nz};
  const int* bc[3] = {P.bcx, P.bcy, P.bcz};
  for (int d = 0; d < 3; ++d) {
    Axis& A = p.a[d];
    A.n = n[d];
    A.wall = bc[d][0] == BC_WALL;
    A.fwd = take((size_t)A.n * A.n);
    A.inv = A.wall ? take((size_t)A.n * A.n) : A.fwd;
    A.eig = take((size_t)A.n);
  }
  p.f0 = take((size_t)P.ncell);
  p.f1 = take((size_t)P.ncell);
  p.total = off;
  return p;
}

// Orthonormal matrix of one axis, G[x][k] (and its transpose for walls), and
// the axis' part of the eigenvalues.
__global__ void __launch_bounds__(256) k_trig_axis(int n, int wall, double dx, double hK, TrigCoef c,
                                                   const double* __restrict__ d_dt, double* __restrict__ G,
                                                   double* __restrict__ GT, double* __restrict__ eig) {
  const double lam = *d_dt / dx;
  const int stride = gridDim.x * 256;
  const double norm = sqrt((wall ? 2.0 : 1.0) / (double)n);
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n * n; i += stride) {
    const int x = i / n, k = i - x * n;
    double s, co, g;
    if (wall) {
      // cos(pi k (2 x + 1) / (2 n)), the exponent mod 4 n
      const int m = (int)(((long long)k * (2 * x + 1)) % (4 * n));
      sincospi((double)m / (double)(2 * n), &s, &co);
      g = k == 0 ? sqrt(1.0 / (double)n) : norm * co;
      GT[(size_t)k * n + x] = g;
    } else {
      const int m = (int)(((long long)k * x) % n);
      sincospi(2.0 * (double)m / (double)n, &s, &co);
      g = norm * (co + s);
    }
    G[i] = g;
  }
  for (int k = blockIdx.x * 256 + threadIdx.x; k < n; k += stride) {
    double s, co, sh, ch;
    const double th = (wall ? 1.0 : 2.0) * (double)k / (double)n;  // theta / pi
    sincospi(th, &s, &co);
    sincospi(0.5 * th, &sh, &ch);
    eig[k] = (lam * lam) * c.tau * (s * s) + lam * (hK * c.irc) * (4.0 * (sh * sh));
  }
}

// Eigenvalues at an output of the last forward transform: Y is divided by
// base + e_row part + e_col parts.
struct Scale {
  double base;
  const double* ez;  // by the row of the product (null: no scaling)
  const double* ex;  // by column % nx
  const double* ey;  // by column / nx (null in 2D)
  int nx;
};

// LEFT: Y[b][k][c] = sum_x G[x][k] X[b][x][c] (M = K = n, columns c < C).
// Right (x axis): Y[r][k] = sum_x X[r][x] G[x][k] (M = rows, K = n, columns k).
template <bool LEFT, bool SCALE>
__global__ void __launch_bounds__(256) k_trig_mul(int n, int M, int C, const double* __restrict__ G,
                                                  const double* __restrict__ X, double* __restrict__ Y, Scale sc) {
  __shared__ double sA[TK * PITCH];
  __shared__ double sB[TK * PITCH];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c0 = blockIdx.x * TN, m0 = blockIdx.y * TM;
  const long long batch = (long long)blockIdx.z * M * C;
  X += batch;
  Y += batch;
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
  const int i = lane & 15, q = lane >> 4;
  // operands of one stage: A (TM x TK) and B (TK x TN), 8 values a thread each
  double ra[8], rb[8];
  auto fetch = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      {  // B: rows along K, threads along the columns
        const int k = k0 + (tid >> 6) + 4 * t, c = c0 + (tid & 63);
        const double* src = LEFT ? X : G;
        rb[t] = (k < n && c < C) ? src[(long long)k * C + c] : 0.0;
      }
      if (LEFT) {  // A[m][k] = G[k][m]: threads along m
        const int k = k0 + (tid >> 6) + 4 * t, m = m0 + (tid & 63);
        ra[t] = (k < n && m < M) ? G[(long long)k * n + m] : 0.0;
      } else {  // A[m][k] = X[m][k]: threads along k
        const int k = k0 + (tid & 31), m = m0 + (tid >> 5) + 8 * t;
        ra[t] = (k < n && m < M) ? X[(long long)m * n + k] : 0.0;
      }
    }
  };
  dbl4 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = dbl4{0.0, 0.0, 0.0, 0.0};
  fetch(0);
  for (int k0 = 0; k0 < n; k0 += TK) {
    __syncthreads();  // the stage before has been read
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      sB[((tid >> 6) + 4 * t) * PITCH + (tid & 63)] = rb[t];
      if (LEFT)
        sA[((tid >> 6) + 4 * t) * PITCH + (tid & 63)] = ra[t];
      else
        sA[(tid & 31) * PITCH + (tid >> 5) + 8 * t] = ra[t];
    }
    __syncthreads();
    if (k0 + TK < n) fetch(k0 + TK);
#pragma unroll
    for (int k = 0; k < TK; k += 4) {
      double a[2], b[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        a[j] = sA[(k + q) * PITCH + wm + 16 * j + i];
        b[j] = sB[(k + q) * PITCH + wn + 16 * j + i];
      }
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v) acc[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b[v], acc[u][v], 0, 0, 0);
    }
  }
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + wm + 16 * u + q + 4 * r, c = c0 + wn + 16 * v + i;
        if (m >= M || c >= C) continue;
        double y = acc[u][v][r];
        if (SCALE) {
          const int cy = c / sc.nx, cx = c - cy * sc.nx;
          double e = sc.base + sc.ez[m] + sc.ex[cx];
          if (sc.ey) e = e + sc.ey[cy];
          y = y / e;
        }
        Y[(long long)m * C + c] = y;
      }
}

template <bool LEFT, bool SCALE>
hipError_t multiply(int n, int M, int C, int batches, const double* G, const double* X, double* Y, const Scale& sc,
                    hipStream_t s) {
  const dim3 g((unsigned)((C + TN - 1) / TN), (unsigned)((M + TM - 1) / TM), (unsigned)batches);
  hipLaunchKernelGGL((k_trig_mul<LEFT, SCALE>), g, dim3(256), 0, s, n, M, C, G, X, Y, sc);
  return hipGetLastError();
}

}  // namespace

size_t trig_scratch_doubles(const Params& P) { return plan_of(P).total; }

hipError_t trig_setup(const Params& P, const TrigCoef& c, const double* d_dt, double* w, hipStream_t s) {
  const Plan p = plan_of(P);
  for (int d = 0; d < 3; ++d) {
    const Axis& A = p.a[d];
    if (d == 1 && P.dim == 2) continue;
    const unsigned nb = (unsigned)std::min(1024, (A.n * A.n + 255) / 256);
    hipLaunchKernelGGL(k_trig_axis, dim3(nb), dim3(256), 0, s, A.n, A.wall ? 1 : 0, P.dx[d], P.hK, c, d_dt, w + A.fwd,
                       w + A.inv, w + A.eig);
  }
  return hipGetLastError();
}

hipError_t trig_solve(const Params& P, const TrigCoef& c, const double* r, double* w, const double** z,
                      hipStream_t s) {
  const Plan p = plan_of(P);
  const Axis &ax = p.a[0], &ay = p.a[1], &az = p.a[2];
  const int plane = P.nx * P.ny, rows = P.ny * P.nz;
  double* f[2] = {w + p.f0, w + p.f1};
  const double* src = r;
  int t = 0;
  const Scale none{};
  auto step = [&](hipError_t e) {
    src = f[t];
    t ^= 1;
    return e;
  };
  hipError_t e = step(multiply<false, false>(ax.n, rows, ax.n, 1, w + ax.fwd, src, f[t], none, s));
  if (e == hipSuccess && P.dim == 3)
    e = step(multiply<true, false>(ay.n, ay.n, P.nx, P.nz, w + ay.fwd, src, f[t], none, s));
  const Scale sc{c.irc2, w + az.eig, w + ax.eig, P.dim == 3 ? w + ay.eig : nullptr, P.nx};
  if (e == hipSuccess) e = step(multiply<true, true>(az.n, az.n, plane, 1, w + az.fwd, src, f[t], sc, s));
  if (e == hipSuccess) e = step(multiply<true, false>(az.n, az.n, plane, 1, w + az.inv, src, f[t], none, s));
  if (e == hipSuccess && P.dim == 3)
    e = step(multiply<true, false>(ay.n, ay.n, P.nx, P.nz, w + ay.inv, src, f[t], none, s));
  if (e == hipSuccess) e = step(multiply<false, false>(ax.n, rows, ax.n, 1, w + ax.inv, src, f[t], none, s));
  *z = src;
  return e;
}

}  // namespace ars
