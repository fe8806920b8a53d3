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
// integers.  Both kernels have a mirror symmetry (cas: x and n - x; cos: x and
// n - 1 - x), which splits the product into two of half the length each way,
// one on the sums and one on the differences of mirror images, so half the
// operations are left: a stage of the product forms them on its way to LDS,
// and the two accumulators give two outputs as their sum and difference (or,
// for cosine modes, the even and the odd modes).
// The products run on the FP64 matrix cores: v_mfma_f64_16x16x4f64, four waves
// a tile, the operands staged in LDS 32 deep and the loads of two stages in
// flight behind the present one's products.  A tile is 32 x 32 pairs, one pair
// of accumulators a wave (as 64 x 64 outputs of the full product, 1024^2 gave
// each CU one workgroup).  The pitch of 49 doubles serves both stores (along
// the tile and across it) and the operand reads of both forms: no bank
// conflicts counted.
// Measured, a transform of one axis of 1024^2: 61 to 67 us as a full product, 58
// as half products in stages of 16, 52 in stages of 32; matrix cores busy for
// 37k of the 85k cycles a CU works.  No further gain from scalar bases with
// 32-bit offsets for the loads (50 us) or eight waves on the halves of a stage
// (50 us): what is left is neither address arithmetic nor too few waves.
// The Mach 1e-3 vortex at acoustic CFL 275, 1024^2 (one implicit step, residual
// 1e-10): 736 plain iterations, 20.5 ms; one preconditioned iteration, 0.51 ms,
// of which the four transforms take 0.21.
#include <algorithm>

#include "ars_trig.h"

namespace ars {

namespace {

typedef double dbl4 __attribute__((ext_vector_type(4)));

constexpr int TM = 32, TN = 32, TK = 32;  // tile of the product: TM x TN pairs, TK deep
constexpr int PITCH = 49;

// A transform: which inputs meet in pair k, which outputs come of pair m.
enum Form {
  HARTLEY,  // inputs k and n - k, outputs m and n - m
  COS_FWD,  // inputs k and n - 1 - k, outputs 2 m and 2 m + 1
  COS_INV   // inputs 2 k and 2 k + 1, outputs m and n - 1 - m
};

struct Axis {
  int n;         // cells
  int h;         // pairs: n / 2 + 1 (cas), (n + 1) / 2 (cos)
  bool wall;     // cosine modes (else Hartley)
  size_t fwd;    // offset of the forward matrices: two of h x h, [input pair][output pair]
  size_t inv;    // of the inverse's (the same for cas)
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
    A.h = A.wall ? (A.n + 1) / 2 : A.n / 2 + 1;
    A.fwd = take((size_t)2 * A.h * A.h);
    A.inv = A.wall ? take((size_t)2 * A.h * A.h) : A.fwd;
    A.eig = take((size_t)A.n);
  }
  p.f0 = take((size_t)P.ncell);
  p.f1 = take((size_t)P.ncell);
  p.total = off;
  return p;
}

// The two half matrices of one axis, G[pair of x][pair of k], their transposes
// GT for walls, and the axis' part of the eigenvalues.
__global__ void __launch_bounds__(256) k_trig_axis(int n, int h, int wall, double dx, double hK, TrigCoef c,
                                                   const double* __restrict__ d_dt, double* __restrict__ G,
                                                   double* __restrict__ GT, double* __restrict__ eig) {
  const double lam = *d_dt / dx;
  const int stride = gridDim.x * 256;
  const int hh = h * h;
  const double norm = sqrt((wall ? 2.0 : 1.0) / (double)n);
  for (int i = blockIdx.x * 256 + threadIdx.x; i < hh; i += stride) {
    const int x = i / h, k = i - x * h;
    double s, co;
    if (wall) {
      // cos(pi k' (2 x + 1) / (2 n)) of k' = 2 k and 2 k + 1, the exponent mod 4 n
      double g[2];
#pragma unroll
      for (int o = 0; o < 2; ++o) {
        const int m = (int)(((long long)(2 * k + o) * (2 * x + 1)) % (4 * n));
        sincospi((double)m / (double)(2 * n), &s, &co);
        g[o] = 2 * k + o == 0 ? sqrt(1.0 / (double)n) : (2 * k + o < n ? norm * co : 0.0);
        G[o * hh + i] = g[o];
        GT[o * hh + k * h + x] = g[o];
      }
    } else {
      const int m = (int)(((long long)k * x) % n);
      sincospi(2.0 * (double)m / (double)n, &s, &co);
      G[i] = norm * co;
      G[hh + i] = norm * s;
    }
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

// LEFT: Y[b][k][c] = sum_x G[x][k] X[b][x][c], the pairs of k along the rows of
// a tile, columns c < C.  Right (x axis): Y[r][k] = sum_x X[r][x] G[x][k], the
// pairs of k along the columns, rows r < R.
template <bool LEFT, int FORM, bool SCALE>
__global__ void __launch_bounds__(256) k_trig_mul(int n, int h, int R, int C, const double* __restrict__ G,
                                                  const double* __restrict__ X, double* __restrict__ Y, Scale sc) {
  __shared__ double sA[2][TK * PITCH];  // of the sums and of the differences
  __shared__ double sB[2][TK * PITCH];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // the pairs along y: the grid's other sides end at 2^16 - 1
  const int c0 = (LEFT ? blockIdx.x : blockIdx.y) * TN, m0 = (LEFT ? blockIdx.y : blockIdx.x) * TM;
  const long long batch = (long long)blockIdx.z * n * C;  // right: one batch
  const int hh = h * h;
  X += batch;
  Y += batch;
  const int wm = (wave >> 1) * 16, wn = (wave & 1) * 16;
  const int i = lane & 15, q = lane >> 4;
  // A stage's operands as they come from memory, NT values of each of the two
  // a thread: of G the two matrices, of X the two inputs of a pair (added only
  // on their way to LDS, or the loads would be waited for where they start).
  // Addresses past an end are those of its last element, and a pair past the
  // last counts as zero.
  constexpr int NT = TK * TM / 256;
  struct Stage {
    double g[2][NT], x[2][NT];
  };
  const int r32 = tid >> 5, l32 = tid & 31;
  const int gi = (LEFT ? m0 : c0) + l32;  // the thread's output pair of G
  const int gc = gi < h ? gi : h - 1;
  const int xc = c0 + l32 < C ? c0 + l32 : C - 1;  // LEFT: its column of X
  auto first = [&](int k) __attribute__((always_inline)) { return FORM == COS_INV ? 2 * k : k; };
  auto second = [&](int k) __attribute__((always_inline)) {
    return FORM == COS_INV ? 2 * k + 1 : (FORM == HARTLEY ? n - k : n - 1 - k);
  };
  auto fetch = [&](int k0, Stage& S) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int kg = k0 + r32 + 8 * t < h ? k0 + r32 + 8 * t : h - 1;
      S.g[0][t] = G[kg * h + gc];
      S.g[1][t] = G[hh + kg * h + gc];
      int k = LEFT ? kg : (k0 + l32 < h ? k0 + l32 : h - 1);
      const int m = m0 + r32 + 8 * t < R ? m0 + r32 + 8 * t : R - 1;  // right: row of X
      const double* base = LEFT ? X + xc : X + (long long)m * n;
      const long long st = LEFT ? C : 1;
      const int ia = first(k), ib = second(k);
      S.x[0][t] = base[ia * st];
      S.x[1][t] = base[(ib < n ? ib : ia) * st];
    }
  };
  dbl4 acc[2] = {dbl4{0.0, 0.0, 0.0, 0.0}, dbl4{0.0, 0.0, 0.0, 0.0}};
  auto stage = [&](int k0, Stage& S) __attribute__((always_inline)) {
    __syncthreads();  // the stage before has been read
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int kx = LEFT ? k0 + r32 + 8 * t : k0 + l32;
      const bool two = second(kx) < n && second(kx) != first(kx);
      const double a = kx < h ? S.x[0][t] : 0.0, b = kx < h && two ? S.x[1][t] : 0.0;
      const double e = FORM == COS_INV ? a : a + b;
      const double o = FORM == COS_INV ? b : (two ? a - b : 0.0);
      const int at = (r32 + 8 * t) * PITCH + l32, tr = l32 * PITCH + r32 + 8 * t;
      (LEFT ? sA : sB)[0][at] = S.g[0][t];
      (LEFT ? sA : sB)[1][at] = S.g[1][t];
      (LEFT ? sB : sA)[0][LEFT ? at : tr] = e;
      (LEFT ? sB : sA)[1][LEFT ? at : tr] = o;
    }
    __syncthreads();
    // two stages ahead and always (past the end: the last element again), so that
    // the counted waits for one stage leave the other's loads in flight
    fetch(k0 + 2 * TK, S);
#pragma unroll
    for (int k = 0; k < TK; k += 4)
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        const double a = sA[g][(k + q) * PITCH + wm + i], b = sB[g][(k + q) * PITCH + wn + i];
        acc[g] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc[g], 0, 0, 0);
      }
  };
  Stage s0, s1;
  fetch(0, s0);
  fetch(TK, s1);
  int k0 = 0;
  for (; k0 + TK < h; k0 += 2 * TK) {
    stage(k0, s0);
    stage(k0 + TK, s1);
  }
  if (k0 < h) stage(k0, s0);
  auto store = [&](int m, int c, double y) __attribute__((always_inline)) {
    if (SCALE) {
      const int cy = c / sc.nx, cx = c - cy * sc.nx;
      double e = sc.base + sc.ez[m] + sc.ex[cx];
      if (sc.ey) e = e + sc.ey[cy];
      y = y / e;
    }
    Y[(long long)m * C + c] = y;
  };
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int m = m0 + wm + q + 4 * r, c = c0 + wn + i;
    const int p = LEFT ? m : c;  // output pair
    if (p >= h || (LEFT ? c >= C : m >= R)) continue;
    const int oa = FORM == COS_FWD ? 2 * p : p;
    const int ob = FORM == COS_FWD ? 2 * p + 1 : (FORM == HARTLEY ? n - p : n - 1 - p);
    const double ya = FORM == COS_FWD ? acc[0][r] : acc[0][r] + acc[1][r];
    const double yb = FORM == COS_FWD ? acc[1][r] : acc[0][r] - acc[1][r];
    store(LEFT ? oa : m, LEFT ? c : oa, ya);
    if (ob < n && ob != oa) store(LEFT ? ob : m, LEFT ? c : ob, yb);
  }
}

// The transform of axis A; LEFT: columns C and batches, right: R rows.
template <bool LEFT, bool SCALE>
hipError_t multiply(const Axis& A, bool inverse, int R, int C, int batches, const double* w, const double* X,
                    double* Y, const Scale& sc, hipStream_t s) {
  static_assert(TM == TN, "the grid below");
  const dim3 g((unsigned)(((LEFT ? C : R) + TM - 1) / TM), (unsigned)((A.h + TM - 1) / TM), (unsigned)batches);
  const double* G = w + (inverse ? A.inv : A.fwd);
  if (!A.wall)
    hipLaunchKernelGGL((k_trig_mul<LEFT, HARTLEY, SCALE>), g, dim3(256), 0, s, A.n, A.h, R, C, G, X, Y, sc);
  else if (!inverse)
    hipLaunchKernelGGL((k_trig_mul<LEFT, COS_FWD, SCALE>), g, dim3(256), 0, s, A.n, A.h, R, C, G, X, Y, sc);
  else
    hipLaunchKernelGGL((k_trig_mul<LEFT, COS_INV, SCALE>), g, dim3(256), 0, s, A.n, A.h, R, C, G, X, Y, sc);
  return hipGetLastError();
}

}  // namespace

size_t trig_scratch_doubles(const Params& P) { return plan_of(P).total; }

hipError_t trig_setup(const Params& P, const TrigCoef& c, const double* d_dt, double* w, hipStream_t s) {
  const Plan p = plan_of(P);
  for (int d = 0; d < 3; ++d) {
    const Axis& A = p.a[d];
    if (d == 1 && P.dim == 2) continue;
    const unsigned nb = (unsigned)std::min(1024, (A.h * A.h + 255) / 256);
    hipLaunchKernelGGL(k_trig_axis, dim3(nb), dim3(256), 0, s, A.n, A.h, A.wall ? 1 : 0, P.dx[d], P.hK, c, d_dt,
                       w + A.fwd, w + A.inv, w + A.eig);
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
  const Scale sc{c.irc2, w + az.eig, w + ax.eig, P.dim == 3 ? w + ay.eig : nullptr, P.nx};
  hipError_t e = step(multiply<false, false>(ax, false, rows, ax.n, 1, w, src, f[t], none, s));
  if (e == hipSuccess && P.dim == 3)
    e = step(multiply<true, false>(ay, false, 0, P.nx, P.nz, w, src, f[t], none, s));
  if (e == hipSuccess) e = step(multiply<true, true>(az, false, 0, plane, 1, w, src, f[t], sc, s));
  if (e == hipSuccess) e = step(multiply<true, false>(az, true, 0, plane, 1, w, src, f[t], none, s));
  if (e == hipSuccess && P.dim == 3)
    e = step(multiply<true, false>(ay, true, 0, P.nx, P.nz, w, src, f[t], none, s));
  if (e == hipSuccess) e = step(multiply<false, false>(ax, true, rows, ax.n, 1, w, src, f[t], none, s));
  *z = src;
  return e;
}

}  // namespace ars
