// ars_reduce.hip -- reductions around the step: the CFL rate of a state
// (time-step kernel), control-block preparation, dt finalisation and the
// diagnostics of Sec. 4 (deterministic two-level sums).
#include "ars_dev.h"
#include "ars_internal.h"

namespace ars {

template <int DIM>
__global__ void __launch_bounds__(256) k_rate(Params P, const double* __restrict__ U, RateMax* slot) {
  constexpr int NV = DIM + 2;
  __shared__ double red[4];
  double m = 0.0;
  for (long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x; c < P.ncell;
       c += (long long)gridDim.x * blockDim.x) {
    double b[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) b[v] = U[c + v * P.ncell];
    const Prim<DIM> q = cons_to_prim<DIM>(P, b);
    const double l = cell_rate<DIM>(P, q);
    m = l > m ? l : m;
  }
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    double mm = red[0];
    for (int w = 1; w < 4; ++w) mm = red[w] > mm ? red[w] : mm;
    atomic_max_rate(slot, mm);
  }
}

hipError_t launch_rate_reduce(const Params& P, const double* U, RateMax* slot, hipStream_t s) {
  long long nb = (P.ncell + 255) / 256;
  if (nb > 2048) nb = 2048;
  if (P.dim == 3)
    hipLaunchKernelGGL(k_rate<3>, dim3((unsigned)nb), dim3(256), 0, s, P, U, slot);
  else
    hipLaunchKernelGGL(k_rate<2>, dim3((unsigned)nb), dim3(256), 0, s, P, U, slot);
  return hipGetLastError();
}

// mode 0: clear the rate maxima; mode 2: clear the fault latch.  A kernel, not
// a memset, so the call can sit inside a captured graph.
__global__ void __launch_bounds__(RATE_WORDS) k_ctl_prep(Control* ctl, int mode) {
  if (mode == 0) {
    for (int i = 0; i < 3; ++i) ctl->lammax[i].w[threadIdx.x] = 0ull;
  }
  if (mode == 2 && threadIdx.x == 0) {
    ctl->fault = 0u;
    ctl->fault_cell = ~0ull;
  }
}

hipError_t launch_ctl_prep(Control* ctl, int mode, hipStream_t s) {
  hipLaunchKernelGGL(k_ctl_prep, dim3(1), dim3(RATE_WORDS), 0, s, ctl, mode);
  return hipGetLastError();
}

// The next step's dt, and the rate maxima back to zero: every call leaves them
// so for the next one, which then needs no kernel of its own in front of its
// first step (1.5 us of a one-step call's 12).
__global__ void __launch_bounds__(RATE_WORDS) k_dt_finish(double cfl, Control* ctl, int slot, double* d_dt) {
  const double r = rate_of(&ctl->lammax[slot]);  // one wave: read before it clears
  if (threadIdx.x == 0) *d_dt = cfl / r;
  for (int i = 0; i < 3; ++i) ctl->lammax[i].w[threadIdx.x] = 0ull;
}

hipError_t launch_dt_finish(const Params& P, Control* ctl, int slot, double* d_dt, hipStream_t s) {
  hipLaunchKernelGGL(k_dt_finish, dim3(1), dim3(RATE_WORDS), 0, s, P.cfl, ctl, slot, d_dt);
  return hipGetLastError();
}

// Sum (or largest) of a wave in a fixed order, in every lane: a butterfly.
template <bool MAX>
__device__ __forceinline__ double wave_total(double v) {
#pragma unroll
  for (int m = 32; m > 0; m >>= 1) {
    const double o = __shfl_xor(v, m, 64);
    v = MAX ? larger(v, o) : v + o;
  }
  return v;
}

// Sum of a block of 256 in a fixed order (the waves' butterflies, then the
// four waves in order), in thread 0.
__device__ __forceinline__ double block_total(double v) {
  __shared__ double sh[4];
  v = wave_total<false>(v);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  return ((sh[0] + sh[1]) + sh[2]) + sh[3];
}

// ---------------------------------------------------------------- diagnostics
// partials: field f of block b at [f * DIAG_NB + b]:
//  0 mass, 1-3 mom, 4 e_total, 5 e_kin, 6 e_int, 7 e_grav, 8 sum|u|,
//  9 max|u|, 10 max Mach, 11 bottom wall flux sum, 12 top wall flux sum
constexpr int DIAG_NB = 1024;
constexpr int DIAG_NF = 16;

size_t diag_partial_bytes(const Params&) { return (size_t)DIAG_NB * DIAG_NF * sizeof(double); }

template <int DIM>
__global__ void __launch_bounds__(256) k_diag_partial(Params P, const double* __restrict__ U, double* partials) {
  constexpr int NV = DIM + 2;
  __shared__ double sh[4][13];
  double acc[DIAG_NF];
#pragma unroll
  for (int i = 0; i < DIAG_NF; ++i) acc[i] = 0.0;
  const unsigned plane = (unsigned)P.nx * (unsigned)P.ny;  // at most 2^31 cells
  for (unsigned c = blockIdx.x * 256u + threadIdx.x; c < (unsigned)P.ncell; c += gridDim.x * 256u) {
    double b[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) b[v] = U[c + v * P.ncell];
    const Prim<DIM> q = cons_to_prim<DIM>(P, b);
    const int kz = (int)(c / plane);
    const double phi = phi_at(P, kz);
    double kin = 0.0, uu = 0.0;
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
      kin += 0.5 * b[1 + k] * q.u[k];
      uu += q.u[k] * q.u[k];
    }
    const double um = sqrt(uu);
    acc[0] += b[0];
    acc[1] += b[1];
    acc[2] += b[2];
    if (DIM == 3) acc[3] += b[3];
    acc[4] += b[NV - 1] + b[0] * phi;
    acc[5] += kin;
    acc[6] += b[NV - 1] - kin;
    acc[7] += b[0] * phi;
    acc[8] += um;
    acc[9] = um > acc[9] ? um : acc[9];
    const double ma = um / q.c;
    acc[10] = ma > acc[10] ? ma : acc[10];
    if (kz == 0) acc[11] += 2.0 * (0.5 * P.Tw2[0] - q.T) / P.dx[2];
    if (kz == P.nz - 1) acc[12] += 2.0 * (q.T - 0.5 * P.Tw2[1]) / P.dx[2];
  }
  // block reduction in a fixed order: the waves' butterflies, then the four
  // waves in order (13 trees through LDS, 17 barriers each: 26.8 us at 128^3,
  // 22.0 so, 3.8 TB/s)
#pragma unroll
  for (int f = 0; f < 13; ++f) {
    const double v = (f == 9 || f == 10) ? wave_total<true>(acc[f]) : wave_total<false>(acc[f]);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6][f] = v;
  }
  __syncthreads();
  const int f = threadIdx.x;
  if (f < 13) {
    double v = sh[0][f];
    for (int w = 1; w < 4; ++w) v = (f == 9 || f == 10) ? larger(v, sh[w][f]) : v + sh[w][f];
    partials[f * DIAG_NB + blockIdx.x] = v;
  }
}

// One wave per field; the fault latch goes along (bits in out[13], out[14]),
// so that the host reads everything at once.
__global__ void __launch_bounds__(13 * 64) k_diag_final(int nblocks, const double* partials, const Control* ctl,
                                                        double* out) {
  const int f = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const bool mx = f == 9 || f == 10;
  double a = 0.0;
  for (int b = lane; b < nblocks; b += 64) {
    const double x = partials[f * DIAG_NB + b];
    a = mx ? larger(a, x) : a + x;
  }
  a = mx ? wave_total<true>(a) : wave_total<false>(a);
  if (lane == 0) out[f] = a;
  if (threadIdx.x == 0) {
    out[13] = __longlong_as_double((long long)ctl->fault);
    out[14] = __longlong_as_double((long long)ctl->fault_cell);
  }
}

// ------------------------------------------------- kinetic-energy objective
// KE = sum_cells (1/2) sum_k m_k u_k dV; optional gradient dKE/dU:
// d/drho = -|u|^2 dV / 2, d/dm_k = u_k dV, d/dE = 0.
template <int DIM>
__global__ void __launch_bounds__(256) k_ke(Params P, double dV, const double* __restrict__ U,
                                           double* __restrict__ grad, double* partials) {
  constexpr int NV = DIM + 2;
  double acc = 0.0;
  for (long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x; c < P.ncell;
       c += (long long)gridDim.x * blockDim.x) {
    const double rho = U[c];
    const double r = 1.0 / rho;
    double kin = 0.0, uu = 0.0;
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
      const double m = U[c + (1 + k) * P.ncell];
      const double u = m * r;
      kin = (k == 0) ? m * u : kin + m * u;
      uu = (k == 0) ? u * u : uu + u * u;
      if (grad) grad[c + (1 + k) * P.ncell] = u * dV;
    }
    acc += 0.5 * kin;
    if (grad) {
      grad[c] = -0.5 * uu * dV;
      grad[c + (NV - 1) * P.ncell] = 0.0;
    }
  }
  acc = block_total(acc);
  if (threadIdx.x == 0) partials[blockIdx.x] = acc;
}

// Sum of the blocks' partials times `scale` (one thread adding 1024 of them
// was 39 us of a kinetic energy's 55 at 128^3).
__global__ void __launch_bounds__(256) k_sum_final(int nb, double scale, const double* __restrict__ partials,
                                                   double* __restrict__ out) {
  double a = 0.0;
  for (int b = threadIdx.x; b < nb; b += 256) a += partials[b];
  a = block_total(a);
  if (threadIdx.x == 0) *out = a * scale;
}

hipError_t launch_ke(const Params& P, const double* U, double* grad, double* partials, double* out, hipStream_t s) {
  double dV = P.dx[0] * P.dx[2];
  if (P.dim == 3) dV = P.dx[0] * P.dx[1] * P.dx[2];
  long long nb = (P.ncell + 255) / 256;
  if (nb > DIAG_NB) nb = DIAG_NB;
  if (P.dim == 3)
    hipLaunchKernelGGL(k_ke<3>, dim3((unsigned)nb), dim3(256), 0, s, P, dV, U, grad, partials);
  else
    hipLaunchKernelGGL(k_ke<2>, dim3((unsigned)nb), dim3(256), 0, s, P, dV, U, grad, partials);
  hipLaunchKernelGGL(k_sum_final, dim3(1), dim3(256), 0, s, (int)nb, dV, partials, out);
  return hipGetLastError();
}

// ------------------------------------------------ Nusselt-number objective
// Nu = C sum_cols 2 (T_w - T_0)/dz (bottom) or C sum_cols 2 (T_{n-1} - T_w)/dz
// (top), C = depth / (dT ncol); optional gradient dNu/dU (zero except on the
// wall-adjacent plane): with T = (gamma-1)(E - kin) / rho,
// dT/dE = (gamma-1)/rho, dT/dm_k = -(gamma-1) u_k / rho,
// dT/drho = (gamma-1)|u|^2/(2 rho) - T/rho.
template <int DIM>
__global__ void __launch_bounds__(256) k_nu(Params P, int side, double C, const double* __restrict__ U,
                                           double* __restrict__ grad, double* partials) {
  constexpr int NV = DIM + 2;
  const long long plane = (long long)P.nx * P.ny;
  const long long base = side == 0 ? 0 : plane * (P.nz - 1);
  const double sgn = side == 0 ? -1.0 : 1.0;  // d(flux)/dT of the wall-adjacent cell
  const double Tw = 0.5 * P.Tw2[side];
  double acc = 0.0;
  for (long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x; c < plane;
       c += (long long)gridDim.x * blockDim.x) {
    const long long i = base + c;
    double b[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) b[v] = U[i + v * P.ncell];
    const Prim<DIM> q = cons_to_prim<DIM>(P, b);
    const double f = side == 0 ? 2.0 * (Tw - q.T) / P.dx[2] : 2.0 * (q.T - Tw) / P.dx[2];
    acc += f;
    if (grad) {
      const double dNdT = C * (sgn * 2.0 / P.dx[2]);
      double uu = 0.0;
#pragma unroll
      for (int k = 0; k < DIM; ++k) {
        uu += q.u[k] * q.u[k];
        grad[i + (1 + k) * P.ncell] = dNdT * (-(P.gm1 * q.u[k]) * q.r);
      }
      grad[i] = dNdT * ((0.5 * (P.gm1 * uu)) * q.r - q.T * q.r);
      grad[i + (NV - 1) * P.ncell] = dNdT * (P.gm1 * q.r);
    }
  }
  acc = block_total(acc);
  if (threadIdx.x == 0) partials[blockIdx.x] = acc;
}

__global__ void __launch_bounds__(256) k_fill(double* p, long long n, double v) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
    p[i] = v;
}

hipError_t launch_nusselt(const Params& P, int side, double C, const double* U, double* grad, double* partials,
                          double* out, hipStream_t s) {
  const long long plane = (long long)P.nx * P.ny;
  long long nb = (plane + 255) / 256;
  if (nb > DIAG_NB) nb = DIAG_NB;
  if (grad) {
    const long long n = (long long)(P.dim + 2) * P.ncell;
    long long fb = (n + 255) / 256;
    if (fb > 4096) fb = 4096;
    hipLaunchKernelGGL(k_fill, dim3((unsigned)fb), dim3(256), 0, s, grad, n, 0.0);
  }
  if (P.dim == 3)
    hipLaunchKernelGGL(k_nu<3>, dim3((unsigned)nb), dim3(256), 0, s, P, side, C, U, grad, partials);
  else
    hipLaunchKernelGGL(k_nu<2>, dim3((unsigned)nb), dim3(256), 0, s, P, side, C, U, grad, partials);
  hipLaunchKernelGGL(k_sum_final, dim3(1), dim3(256), 0, s, (int)nb, C, partials, out);
  return hipGetLastError();
}

hipError_t launch_diag(const Params& P, const double* U, double* partials, const Control* ctl, double* out,
                       hipStream_t s) {
  long long nb = (P.ncell + 255) / 256;
  if (nb > DIAG_NB) nb = DIAG_NB;
  if (P.dim == 3)
    hipLaunchKernelGGL(k_diag_partial<3>, dim3((unsigned)nb), dim3(256), 0, s, P, U, partials);
  else
    hipLaunchKernelGGL(k_diag_partial<2>, dim3((unsigned)nb), dim3(256), 0, s, P, U, partials);
  hipLaunchKernelGGL(k_diag_final, dim3(1), dim3(13 * 64), 0, s, (int)nb, partials, ctl, out);
  return hipGetLastError();
}

}  // namespace ars
