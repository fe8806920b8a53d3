// ars_spectrum.hip -- kinetic-energy spectrum of one horizontal plane, the
// diagnostic of the 3D Rayleigh-Benard runs (Sec. 4.5, 3D case).
//
// For w_c = sqrt(rho) u_c on the plane at vertical index kz (every velocity
// component), W_c(k) = sum_x w_c(x) exp(-2 pi i k.x / n) and
//   E(s) = sum_{k : round(|k|) = s} sum_c |W_c(k)|^2 / (2 N^2),
// k integer wave vectors in the FFT order (k_j = j for j < (n+1)/2, else
// j - n), N the cell count of the plane; sum_s E(s) is then the plane mean of
// rho |u|^2 / 2 (Parseval).  In 2D the plane is a line along x.
//
// The plane is real, so W_c(-k) is the conjugate of W_c(k): only the columns
// 0 <= k_x <= n_x / 2 are formed, and those with a distinct mirror image
// count twice.  When both sides are powers of two the transforms are FFTs in
// LDS: a row as the half-length transform of its even and odd elements, then
// one workgroup per column, which also forms the power and its shells' sums
// (three launches).  Otherwise it is a dense DFT, rows then columns, and a
// DFT is a matrix product: the row transform is W (n_y x n_x) times the
// twiddle matrix, the column transform the n_y x n_y twiddle matrix times X,
// so both run on the FP64 matrix cores (v_mfma_f64_16x16x4f64: one wave
// accumulates a 16 x 16 tile over K in steps of 4).  The twiddle matrices
// are never stored: entry (k, x) is read from an LDS table of
// exp(-2 pi i j / n) at j = k x mod n, the exponent carried exactly in
// integers.
//
// Along a column the shell number does not fall with |k_y| and never skips
// one, so a column's share of a shell is the sum of one run of consecutive
// |k_y|, kept at [k_x][s - k_x]; a last small kernel adds the columns.  All
// orders are fixed: the result is deterministic.  256 x 256, three
// components: 28.5 us a call with full complex rows, one radix-2 stage a
// barrier and a walk of the whole plane's annulus per shell (w 3.0, rows 6.7,
// columns 10.8, shells 11.8 us); 15.7 now (rows 5.7, columns 7.2, sum 3.4: each
// a chain of barriers at one workgroup per CU).
#include <algorithm>

#include "ars_dev.h"
#include "ars_internal.h"

namespace ars {

constexpr int SPEC_MAXN = 2048;

// tw[j] = exp(-2 pi i j / n), j < n, cos in tw[0..n), -sin in tw[n..2n).
__device__ __forceinline__ void fill_twiddles(double* tw, int n) {
  for (int j = threadIdx.x; j < n; j += blockDim.x) {
    double s, c;
    sincospi(2.0 * (double)j / (double)n, &s, &c);
    tw[j] = c;
    tw[n + j] = -s;
  }
}

typedef double dbl4 __attribute__((ext_vector_type(4)));

// One 16 x 16 x 4 FP64 matrix step: C (16 x 16) += A (16 x 4) B (4 x 16).
// Lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16]; it holds
// C[l / 16 + 4 r][l % 16] in element r.
__device__ __forceinline__ dbl4 mma16(double a, double b, dbl4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// w_c = sqrt(rho) u_c on the plane, W[c][y][x].
__global__ void __launch_bounds__(256) k_spec_w(Params P, const double* __restrict__ U, int kz,
                                                double* __restrict__ W) {
  const long long N = (long long)P.nx * P.ny;
  const long long base = (long long)kz * N;
  for (long long f = (long long)blockIdx.x * blockDim.x + threadIdx.x; f < N * P.dim;
       f += (long long)gridDim.x * blockDim.x) {
    const int c = (int)(f / N);
    const long long i = f - c * N;
    const double rho = U[base + i];
    const double m = U[(long long)(1 + c) * P.ncell + base + i];
    W[f] = sqrt(rho) * (m / rho);
  }
}

// Row transforms X_c = W_c T_x, T_x(x, k) = exp(-2 pi i k x / n_x): block
// (kx group of 64, row tile of 16, component c), wave w the 16 x 16 tile of
// rows y0.. and wave numbers k0 = 64 bx + 16 w ..; real and imaginary
// parts in two accumulators; X_c[y][k], k <= n_x / 2.  Out-of-range rows,
// columns and K entries contribute zeros.  STATE: the block forms its rows of w
// from the state in LDS, behind the twiddles; W then is the density's plane.
template <bool STATE>
__global__ void __launch_bounds__(256) k_spec_rows(Params P, const double* __restrict__ W, double* __restrict__ Xr,
                                                   double* __restrict__ Xi) {
  extern __shared__ double tw[];
  const int nx = P.nx, ny = P.ny, kn = nx / 2 + 1, c = blockIdx.z;
  fill_twiddles(tw, nx);
  const int pitch = nx | 1;  // odd: the 16 rows of an operand read fall on different banks
  if (STATE) {
    const int rows = min(16, ny - (int)blockIdx.y * 16);
    const double* rho = W + (long long)blockIdx.y * 16 * nx;
    const double* mom = rho + (long long)(1 + c) * P.ncell;
    for (int f = threadIdx.x; f < rows * nx; f += 256) {
      const int r = f / nx;
      tw[2 * nx + r * pitch + (f - r * nx)] = sqrt(rho[f]) * (mom[f] / rho[f]);
    }
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i = lane & 15, q = lane >> 4;
  const int y0 = blockIdx.y * 16, k0 = blockIdx.x * 64 + wave * 16;
  const int y = y0 + i, k = k0 + i;  // A row of this lane, B column of this lane
  const double* Wr = W + ((long long)c * ny + (y < ny ? y : 0)) * nx;
  const double* own = tw + 2 * nx + i * pitch;
  const int dk = (int)((4LL * k) % nx);
  int e = (int)(((long long)k * q) % nx);  // k x mod n_x at x = q
  dbl4 ar = {0.0, 0.0, 0.0, 0.0}, ai = {0.0, 0.0, 0.0, 0.0};
  // K in blocks of 8 steps: all operand loads of a block are issued before
  // its 16 matrix steps
  for (int x0 = 0; x0 < nx; x0 += 32) {
    double a[8], br[8], bi[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int x = x0 + 4 * j + q;
      const bool in = x < nx;
      a[j] = (in && y < ny) ? (STATE ? own[x] : Wr[x]) : 0.0;
      br[j] = (in && k < kn) ? tw[e] : 0.0;
      bi[j] = (in && k < kn) ? tw[nx + e] : 0.0;
      e += dk;
      if (e >= nx) e -= nx;
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      ar = mma16(a[j], br[j], ar);
      ai = mma16(a[j], bi[j], ai);
    }
  }
  const int kc = k0 + i;  // output column of this lane
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int yo = y0 + q + 4 * r;
    if (yo < ny && kc < kn) {
      const long long o = ((long long)c * ny + yo) * kn + kc;
      Xr[o] = ar[r];
      Xi[o] = ai[r];
    }
  }
}

// Column transforms Y_c = T_y X_c, T_y(ky, y) = exp(-2 pi i ky y / n_y),
// and Pc[c][k][ky] = |Y_c(ky, k)|^2: block (k group of 64, ky tile of 16,
// component c), wave w the 16 x 16 tile of ky0.. and k0 = 64 bx + 16 w ..
__global__ void __launch_bounds__(256) k_spec_cols(Params P, const double* __restrict__ Xr,
                                                   const double* __restrict__ Xi, double* __restrict__ Pc) {
  extern __shared__ double tw[];
  const int ny = P.ny, kn = P.nx / 2 + 1, c = blockIdx.z;
  fill_twiddles(tw, ny);
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i = lane & 15, q = lane >> 4;
  const int ky0 = blockIdx.y * 16, k0 = blockIdx.x * 64 + wave * 16;
  const int ky = ky0 + i, k = k0 + i;  // A row (ky) and B column (k) of this lane
  const long long o = (long long)c * ny * kn;
  const int dky = (int)((4LL * ky) % ny);
  int e = (int)(((long long)ky * q) % ny);  // ky y mod n_y at y = q
  dbl4 yr = {0.0, 0.0, 0.0, 0.0}, yi = {0.0, 0.0, 0.0, 0.0};
  for (int y0 = 0; y0 < ny; y0 += 32) {
    double tr[8], ti[8], xr[8], xi[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int y = y0 + 4 * j + q;
      const bool in = y < ny;
      tr[j] = (in && ky < ny) ? tw[e] : 0.0;
      ti[j] = (in && ky < ny) ? tw[ny + e] : 0.0;
      const bool bk = in && k < kn;
      xr[j] = bk ? Xr[o + (long long)y * kn + k] : 0.0;
      xi[j] = bk ? Xi[o + (long long)y * kn + k] : 0.0;
      e += dky;
      if (e >= ny) e -= ny;
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      // (tr + i ti)(xr + i xi)
      yr = mma16(tr[j], xr[j], yr);
      yr = mma16(-ti[j], xi[j], yr);
      yi = mma16(tr[j], xi[j], yi);
      yi = mma16(ti[j], xr[j], yi);
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int kyo = ky0 + q + 4 * r;
    if (kyo < ny && k < kn) Pc[o + (long long)k * ny + kyo] = yr[r] * yr[r] + yi[r] * yi[r];
  }
}

// round(sqrt(k^2 + j^2)): v is an integer, so it lies above (s + 1/2)^2 where
// it exceeds s^2 + s, and no bound is ever met exactly.
__device__ __forceinline__ int shell_of(int k, int j) {
  const int v = k * k + j * j;
  int s = (int)sqrtf((float)v);
  while (s * s > v) --s;
  while ((s + 1) * (s + 1) <= v) ++s;
  return s + (v > s * s + s ? 1 : 0);
}

// One column's shares of the shells: pw its n powers in FFT order (LDS), sum
// 2 (n / 2 + 1) doubles of LDS, part[s - k] the share of shell s.  The thread at
// the first |ky| of a shell adds its run.  The caller has synchronised.
__device__ __forceinline__ void shell_shares(const double* pw, double* sum, int n, int nx, int k, double* part) {
  const int h = n / 2;
  int* shell = (int*)(sum + h + 1);
  for (int j = threadIdx.x; j <= h; j += blockDim.x) {
    sum[j] = (j > 0 && 2 * j != n) ? pw[j] + pw[n - j] : pw[j];
    shell[j] = shell_of(k, j);
  }
  __syncthreads();
  const double w = (k == 0 || 2 * k == nx) ? 1.0 : 2.0;  // the column -k
  for (int j = threadIdx.x; j <= h; j += blockDim.x) {
    const int s = shell[j];
    if (j > 0 && shell[j - 1] == s) continue;
    double a = sum[j];
    for (int i = j + 1; i <= h && shell[i] == s; ++i) a += sum[i];
    part[s - k] = w * a;
  }
}

// Dense path: block k takes column k's powers, the components added in order.
__global__ void __launch_bounds__(256) k_spec_part(Params P, const double* __restrict__ Pc,
                                                   double* __restrict__ part) {
  extern __shared__ double sm[];
  const int n = P.ny, k = blockIdx.x, kn = gridDim.x;
  for (int y = threadIdx.x; y < n; y += blockDim.x) {
    double p = 0.0;
    for (int c = 0; c < P.dim; ++c) p = p + Pc[((long long)c * kn + k) * n + y];
    sm[y] = p;
  }
  __syncthreads();
  shell_shares(sm, sm + n, n, P.nx, k, part + (long long)k * (n / 2 + 1));
}

// E(s): the columns' shares of shell s, k <= s <= shell_of(k, n_y / 2), each
// lane its columns in order, then the lanes; one wave per shell.
__global__ void __launch_bounds__(64) k_spec_final(Params P, const double* __restrict__ part, double* __restrict__ E) {
  const int hx = P.nx / 2, hy = P.ny / 2, s = blockIdx.x;
  const double N = (double)((long long)P.nx * P.ny);
  double a = 0.0;
  for (int k = threadIdx.x; k <= hx && k <= s; k += 64)
    if (s - k <= hy && shell_of(k, hy) >= s) a += part[(long long)k * (hy + 1) + (s - k)];
#pragma unroll
  for (int m = 32; m > 0; m >>= 1) a = a + __shfl_xor(a, m, 64);
  if (threadIdx.x == 0) E[s] = a / (2.0 * N * N);
}

// ---------------------------------------------------------------- FFT path
constexpr int FFT_LDS_DOUBLES = 8192;  // 64 KB of dynamic LDS

__device__ __forceinline__ int bit_reverse(int x, int logn) {
  return logn ? (int)(__brev((unsigned)x) >> (32 - logn)) : 0;
}

// tw[j] = exp(-2 pi i j / n) for j < n / 2: cos in tw[0..n/2), -sin in
// tw[n/2..n).
__device__ __forceinline__ void fill_half_twiddles(double* tw, int n) {
  const int h = n / 2;
  for (int j = threadIdx.x; j < h; j += blockDim.x) {
    double sn, cs;
    sincospi(2.0 * (double)j / (double)n, &sn, &cs);
    tw[j] = cs;
    tw[h + j] = -sn;
  }
}

// cnt transforms of m = 2^logm points in LDS, one after the other, loaded in
// bit-reversed order; tw the half table of n >= m points.  Two radix-2 stages
// at a time (a first one alone if logm is odd), since a stage's barrier and
// LDS round trip cost more than its arithmetic: X_i, X_j <- X_i + w X_j,
// X_i - w X_j with w = exp(-2 pi i k / len).  Synchronised on return.
__device__ void fft_stages(double* re, double* im, const double* tw, int n, int logm, int cnt) {
  const int hn = n / 2, m = 1 << logm;
  int lh = logm & 1;
  if (lh) {
    for (int b = threadIdx.x; b < cnt * (m / 2); b += blockDim.x) {
      const double ar = re[2 * b], ai = im[2 * b], br = re[2 * b + 1], bi = im[2 * b + 1];
      re[2 * b] = ar + br;
      im[2 * b] = ai + bi;
      re[2 * b + 1] = ar - br;
      im[2 * b + 1] = ai - bi;
    }
    __syncthreads();
  }
  for (; lh < logm; lh += 2) {
    const int half = 1 << lh;
    const int st = n >> (lh + 2);  // exp(-2 pi i k / (4 half)) = table entry k st
    for (int b = threadIdx.x; b < cnt * (m / 4); b += blockDim.x) {
      const int k = b & (half - 1), i0 = ((b >> lh) << (lh + 2)) + k;  // (4 half divides m)
      const int i1 = i0 + half, i2 = i1 + half, i3 = i2 + half;
      const double ur = tw[2 * k * st], ui = tw[hn + 2 * k * st];  // of length 2 half
      const double vr = tw[k * st], vi = tw[hn + k * st];          // of length 4 half
      const double x1r = re[i1], x1i = im[i1], x3r = re[i3], x3i = im[i3];
      const double t1r = ur * x1r - ui * x1i, t1i = ur * x1i + ui * x1r;
      const double t3r = ur * x3r - ui * x3i, t3i = ur * x3i + ui * x3r;
      const double x0r = re[i0], x0i = im[i0], x2r = re[i2], x2i = im[i2];
      const double a0r = x0r + t1r, a0i = x0i + t1i, a1r = x0r - t1r, a1i = x0i - t1i;
      const double a2r = x2r + t3r, a2i = x2i + t3i, a3r = x2r - t3r, a3i = x2i - t3i;
      const double s2r = vr * a2r - vi * a2i, s2i = vr * a2i + vi * a2r;
      // exp(-2 pi i (k + half) / (4 half)) = -i times that of k
      const double q3r = vr * a3r - vi * a3i, q3i = vr * a3i + vi * a3r;
      re[i0] = a0r + s2r;
      im[i0] = a0i + s2i;
      re[i2] = a0r - s2r;
      im[i2] = a0i - s2i;
      re[i1] = a1r + q3i;
      im[i1] = a1i - q3r;
      re[i3] = a1r - q3i;
      im[i3] = a1i + q3r;
    }
    __syncthreads();
  }
}

// Row transforms of w_c = sqrt(rho) u_c, X_c[k][y], k <= n / 2: block (nr rows
// from y0, component c).  With z = w(2 p) + i w(2 p + 1) and Z its transform
// of m = n / 2 points, E = (Z(k) + Z*(m - k)) / 2, O = (Z(k) - Z*(m - k)) / 2i,
// X(k) = E + exp(-2 pi i k / n) O.
__global__ void __launch_bounds__(256) k_fft_rows(Params P, int logx, int nr, const double* __restrict__ U, int kz,
                                                  double* __restrict__ Xr, double* __restrict__ Xi) {
  extern __shared__ double sm[];
  const int n = P.nx, m = n / 2, ny = P.ny, y0 = blockIdx.x * nr, c = blockIdx.y;
  const double* rho = U + (long long)kz * n * ny;
  const double* mom = rho + (long long)(1 + c) * P.ncell;
  const long long o = (long long)c * (m + 1) * ny;
  if (n == 1) {
    if (threadIdx.x < nr && y0 + (int)threadIdx.x < ny) {
      const int y = y0 + (int)threadIdx.x;
      Xr[o + y] = sqrt(rho[y]) * (mom[y] / rho[y]);
      Xi[o + y] = 0.0;
    }
    return;
  }
  double* tw = sm;
  double* re = sm + n;
  double* im = re + nr * m;
  for (int e = threadIdx.x; e < nr * m; e += blockDim.x) {
    const int r = e >> (logx - 1), p = e & (m - 1);
    const int j = r * m + bit_reverse(p, logx - 1);
    double w0 = 0.0, w1 = 0.0;
    if (y0 + r < ny) {
      const long long i = (long long)(y0 + r) * n + 2 * p;
      const double r0 = rho[i], r1 = rho[i + 1], m0 = mom[i], m1 = mom[i + 1];
      w0 = sqrt(r0) * (m0 / r0);
      w1 = sqrt(r1) * (m1 / r1);
    }
    re[j] = w0;
    im[j] = w1;
  }
  fill_half_twiddles(tw, n);
  __syncthreads();
  fft_stages(re, im, tw, n, logx - 1, nr);
  for (int e = threadIdx.x; e < nr * (m + 1); e += blockDim.x) {
    const int k = e / nr, r = e - k * nr, y = y0 + r;
    if (y >= ny) continue;
    const int a = r * m + (k & (m - 1)), b = r * m + ((m - k) & (m - 1));
    const double er = 0.5 * (re[a] + re[b]), ei = 0.5 * (im[a] - im[b]);
    const double dr = 0.5 * (im[a] + im[b]), di = -0.5 * (re[a] - re[b]);
    const double wr = k < m ? tw[k] : -1.0, wi = k < m ? tw[m + k] : 0.0;
    Xr[o + (long long)k * ny + y] = er + (wr * dr - wi * di);
    Xi[o + (long long)k * ny + y] = ei + (wr * di + wi * dr);
  }
}

// Column transforms, power and shell shares: block k takes column k, nc
// components at a time.
__global__ void __launch_bounds__(256) k_fft_cols(Params P, int logy, int nc, const double* __restrict__ Xr,
                                                  const double* __restrict__ Xi, double* __restrict__ part) {
  extern __shared__ double sm[];
  const int n = P.ny, k = blockIdx.x, kn = gridDim.x;
  double* tw = sm;
  double* pw = sm + n;
  double* re = pw + n;
  double* im = re + nc * n;
  for (int c0 = 0; c0 < P.dim; c0 += nc) {
    const int cnt = min(nc, P.dim - c0);
    for (int e = threadIdx.x; e < cnt * n; e += blockDim.x) {
      const int c = e >> logy, y = e & (n - 1);
      const long long i = ((long long)(c0 + c) * kn + k) * n + y;
      const int j = c * n + bit_reverse(y, logy);
      re[j] = Xr[i];
      im[j] = Xi[i];
    }
    if (c0 == 0) fill_half_twiddles(tw, n);
    __syncthreads();
    fft_stages(re, im, tw, n, logy, cnt);
    for (int y = threadIdx.x; y < n; y += blockDim.x) {
      double p = c0 ? pw[y] : 0.0;
      for (int c = 0; c < cnt; ++c) p = p + (re[c * n + y] * re[c * n + y] + im[c * n + y] * im[c * n + y]);
      pw[y] = p;
    }
    __syncthreads();
  }
  shell_shares(pw, re, n, P.nx, k, part + (long long)k * (n / 2 + 1));
}

static int log2_exact(int n) {
  int l = 0;
  while ((1 << l) < n) ++l;
  return (1 << l) == n ? l : -1;
}

int spectrum_shells(const Params& P) {
  const double hx = (double)(P.nx / 2), hy = (double)(P.ny / 2);
  return (int)llrint(sqrt(hx * hx + hy * hy)) + 1;
}

size_t spectrum_work_bytes(const Params& P) {
  const size_t N = (size_t)P.nx * (size_t)P.ny;
  return (size_t)(4 * P.dim) * N * sizeof(double);
}

bool spectrum_supported(const Params& P) { return P.nx <= SPEC_MAXN && P.ny <= SPEC_MAXN; }

// Work: X_c (2 dim planes of at most N), then the columns' shell shares
// ((n_x / 2 + 1)(n_y / 2 + 1) <= N); the dense path also w_c, and its powers
// where w_c was.
hipError_t launch_spectrum(const Params& P, const double* U, int kz, double* E, void* work, hipStream_t s) {
  const long long N = (long long)P.nx * P.ny;
  double* Wp = (double*)work;
  double* Xr = Wp + (long long)P.dim * N;
  double* Xi = Xr + (long long)P.dim * N;
  double* part = Xi + (long long)P.dim * N;
  const unsigned kn = (unsigned)(P.nx / 2 + 1);
  const int lx = log2_exact(P.nx), ly = log2_exact(P.ny);
  if (lx >= 0 && ly >= 0) {
    // nr rows a block: their values of one k are adjacent in X
    int nr = 4;
    while (nr > 1 && P.nx + nr * P.nx > FFT_LDS_DOUBLES) nr /= 2;
    const int nc = (2 + 2 * P.dim) * P.ny <= FFT_LDS_DOUBLES ? P.dim : 1;
    hipLaunchKernelGGL(k_fft_rows, dim3((unsigned)((P.ny + nr - 1) / nr), (unsigned)P.dim), dim3(256),
                       (size_t)(P.nx + nr * P.nx) * sizeof(double), s, P, lx, nr, U, kz, Xr, Xi);
    hipLaunchKernelGGL(k_fft_cols, dim3(kn), dim3(256), (size_t)(2 + 2 * nc) * P.ny * sizeof(double), s, P, ly, nc,
                       Xr, Xi, part);
  } else {
    const dim3 g((kn + 63) / 64, (unsigned)((P.ny + 15) / 16), (unsigned)P.dim);
    // twiddles and 16 rows of w; where they fit (up to 455 cells), w needs no
    // launch of its own, of which a small plane's call consists: us a call with
    // and without one 100 x 60 24.2, 20.2; 130 x 130 29.6, 28.1; 250 x 249 41.9,
    // 40.4 (formed by every wave of a row in registers: 24.0 at 100 x 60)
    const size_t own = ((size_t)2 * P.nx + 16 * (size_t)(P.nx | 1)) * sizeof(double);
    const size_t lds = (size_t)2 * P.nx * sizeof(double);
    if (own <= FFT_LDS_DOUBLES * sizeof(double)) {
      hipLaunchKernelGGL(k_spec_rows<true>, g, dim3(256), own, s, P, U + (long long)kz * N, Xr, Xi);
    } else {
      const long long nb = std::min((N * P.dim + 255) / 256, 4096LL);
      hipLaunchKernelGGL(k_spec_w, dim3((unsigned)nb), dim3(256), 0, s, P, U, kz, Wp);
      hipLaunchKernelGGL(k_spec_rows<false>, g, dim3(256), lds, s, P, Wp, Xr, Xi);
    }
    hipLaunchKernelGGL(k_spec_cols, g, dim3(256), (size_t)2 * P.ny * sizeof(double), s, P, Xr, Xi, Wp);
    hipLaunchKernelGGL(k_spec_part, dim3(kn), dim3(256), (size_t)(P.ny + 2 * (P.ny / 2 + 1)) * sizeof(double), s, P, Wp,
                       part);
  }
  hipLaunchKernelGGL(k_spec_final, dim3((unsigned)spectrum_shells(P)), dim3(64), 0, s, P, part, E);
  return hipGetLastError();
}

}  // namespace ars
