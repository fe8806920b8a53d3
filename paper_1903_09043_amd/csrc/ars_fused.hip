// ars_fused.hip -- fused explicit step of the all-regime, well-balanced
// scheme (arXiv 1903.09043, eq. all_regime_scheme with the dissipative
// fluxes of Sec. 2.2 and the relaxation step of Sec. 2.1.4) for gfx950.
//
// Design (MI355X-first, not the paper's flat Kokkos loop):
//  * One workgroup owns a tile of TX x TY columns (2D: TX columns) plus a
//    2-cell halo and marches along the vertical (gravity) axis.  The stencil
//    of one update is the radius-2 diamond (the upwinded transport value
//    b~ of a neighbour needs all faces of that neighbour), so the halo is 2.
//  * The vertical neighbours live in registers (a rolling window of planes).
//    2D: a row segment is one wave and its neighbours the lanes beside (DPP
//    moves).  3D: lateral neighbours are exchanged through LDS once per plane:
//      XA  acoustic fields (rho c, c, p, u_lat) of the newest plane p
//      V   u, T of plane p-1 (viscous stencil), DZ  u(p) - u(p-2)
//      F   own +x/+y acoustic faces (u*, Pi*, Pi* u*) of plane p
//      B   transported values b~ of plane p-1
//      GX  own +x/+y total face fluxes of plane p-1
//    Per plane: faces at p, acoustic cell values at p-1, fluxes at p-1 and
//    the update of plane p-2; 2 barriers per plane.
//  * Every face is evaluated once; the only HBM traffic is the read of U^n
//    and the write of U^{n+1} (plus halo re-reads that hit L2).
//  * Epilogue: the rate of the NEW state for the next CFL time step is
//    reduced (one wave: DPP moves; several: LDS) to one atomicMax per
//    workgroup, spread over 64 words, so dt never leaves the device and n steps
//    need no host synchronisation.
//  * No MFMA: nothing here is a contraction.

#include <algorithm>
#include <numeric>

#include "ars_fused.h"

namespace ars {

template <int DIM, bool LM, bool DISS, bool NC, int EX, int EY, bool SPLIT>
__global__ void __launch_bounds__(EX* EY) k_step_fused(Params P, const double* __restrict__ Uin,
                                                       double* __restrict__ Uout, StepIO io) {
  constexpr int NPOS = EX * EY;
  using Ly = FusedLayout<DIM>;
  __shared__ double sm[DIM == 3 ? Ly::TOTAL * NPOS : 1];  // 2D exchanges through registers
  constexpr int NW = (NPOS + 63) / 64;  // waves (the last one partial if 64 does not divide NPOS)

  const int tid = threadIdx.x;
  // Time step of this step.  2D: loaded here and used behind the first state
  // loads, t and the log written behind the march, whose latency is the step's.
  // 3D: all of that first, and dt / dx in scalar registers: the 3D march has no
  // vector registers to spare (10 spilled with the loads in flight together, 7
  // with the time step first, 6 so).  us a step with a given dt, in that order:
  // 8^3 13.5, 12.8, 13.0; 32^3 13.9, 13.4, 13.3; 128^3 103.2, 102.3, 101.9; 512 x
  // 512 x 4 75.8, 75.2, 74.1.
  RateLoad rate{};
  double dt_given = 0.0;
  if (io.rate_in)
    rate.load(io.rate_in);
  else
    dt_given = *io.dt_in;
  double dt = 0.0, lam[3] = {0.0, 0.0, 0.0};
  auto take_dt = [&]() __attribute__((always_inline)) {
    dt = io.rate_in ? P.cfl / rate.max() : dt_given;
    lam[0] = dt / P.dx[0];
    lam[1] = (DIM == 3) ? dt / P.dx[1] : 0.0;
    lam[2] = dt / P.dx[2];
  };
  auto book = [&]() __attribute__((always_inline)) {
    if (blockIdx.x != 0) return;
    static_assert(NPOS >= RATE_WORDS, "one thread clears one word");
    if (io.clear_slot && tid < RATE_WORDS) io.clear_slot->w[tid] = 0ull;
    if (tid == 0) {
      if (io.t) *io.t = *io.t + dt;
      if (io.dt_log) *io.dt_log = dt;
    }
  };
  if (DIM == 3) {
    take_dt();
    book();
#pragma unroll
    for (int a = 0; a < 3; ++a) lam[a] = lane_value(lam[a], 0);
  }
  auto lam_of = [&](double& lamx, double& lamy, double& lamz) __attribute__((always_inline)) {
    if (DIM == 2) take_dt();
    lamx = lam[0];
    lamy = lam[1];
    lamz = lam[2];
  };

  // Persistent schedule: every workgroup takes one contiguous share of the
  // (tile, plane) pairs; those of one XCD are neighbours in space, so halo
  // re-reads hit that XCD's L2.
  const unsigned G = gridDim.x, b = blockIdx.x;
  // 2D: a G that 8 does not divide in launch order; the host avoids it where it
  // counts (64 x 32: 40 ns of a step's 6.7 us for the few scalar instructions
  // more; 60 x 7000, with the copy of an odd step count: 27.9 us, 28.8 by XCD)
  const unsigned lw = DIM == 3 ? xcd_share(b, G) : (G % 8 == 0) ? (b % 8) * (G / 8) + b / 8 : b;
  unsigned cur, stop;
  share_of<DIM == 3>(io.shares, lw, (unsigned)P.nz, cur, stop);
  double lmax = 0.0;
  unsigned long long badcell = ~0ull;
  while (cur < stop) {
    const int tile = (int)(cur / (unsigned)P.nz);
    const int z0 = (int)(cur - (unsigned)tile * (unsigned)P.nz);
    const int z1 = (int)min((unsigned)P.nz, (unsigned)z0 + (stop - cur));
    cur += z1 - z0;
    const int tx = (DIM == 3) ? tile % io.ntx : tile * EY + (int)threadIdx.x / EX;
    const int ty = (DIM == 3) ? tile / io.ntx : 0;
    march_tile<DIM, LM, DISS, NC, EX, EY, SPLIT>(P, Uin, Uout, sm, tx, ty, 0, z0, z1, lam_of, lmax, badcell);
  }

  if (DIM == 2) book();

  // ---- workgroup reduction of the new-state rate, fault latch --------------
  if (badcell != ~0ull) {
    atomicOr(&io.ctl->fault, 1u);
    atomicMin(&io.ctl->fault_cell, badcell);
  }
  if (io.rate_out) {
    double m;
    if (NW == 1) {
      m = wave_max(lmax);  // no barrier, no LDS: the tail of a one-wave workgroup is on every 2D step
    } else {
      // every position's rate to wave 0 through LDS (free after the march)
      __syncthreads();
      sm[tid] = lmax;
      __syncthreads();
      m = 0.0;
      if (tid < 64) {
        for (int j = tid; j < NPOS; j += 64) m = larger(m, sm[j]);
        m = wave_max(m);
      }
    }
    if (tid == 0) atomic_max_rate(io.rate_out, m);
  }
}

// --------------------------------------------------------------------------
// Host-side launch
// --------------------------------------------------------------------------
Shares shares_of(long long tiles, int nz, long long most, long long least, int halo) {
  const long long total = tiles * nz;
  auto run = [](long long groups, long long chunks, long long pairs) {
    Shares s{};
    s.groups = (unsigned)groups;
    s.chunks = (unsigned)chunks;
    s.share = (unsigned)(pairs / chunks);
    s.extra = (unsigned)(pairs % chunks);
    s.step = (unsigned)((((pairs % chunks) << 32) + chunks - 1) / chunks);
    return s;
  };
  const long long g = std::max(1ll, std::min((total + least - 1) / least, most));
  const long long longest = (total + g - 1) / g;
  const bool aligned = total % g == 0 && (nz % longest == 0 || longest % nz == 0);
  const long long marches = aligned ? (longest + nz - 1) / nz : 1 + (longest + nz - 2) / nz;
  const long long c = std::min((long long)nz, std::min(most / tiles, std::max(1ll, nz / least)));
  if (c < 1 || (nz + c - 1) / c + halo > longest + halo * marches) return run(g, g, total);
  return run(tiles * c, c, nz);
}

// Resident workgroups per CU of one kernel.
template <int DIM, bool LM, bool DISS, bool NC, int EX, int EY, bool SPLIT>
static int resident() {
  static int occ = 0;
  if (occ == 0) {
    int o = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&o, k_step_fused<DIM, LM, DISS, NC, EX, EY, SPLIT>, EX * EY, 0) !=
            hipSuccess ||
        o < 1)
      o = 1;
    occ = o;
  }
  return occ;
}

template <int DIM, bool LM, bool DISS, bool NC, int EX, int EY>
static hipError_t launch_fused_t(const Params& P, const double* Uin, double* Uout, StepIO io, const TileShape& ts,
                                 hipStream_t s) {
  constexpr int TX = EX - 4;
  constexpr int TY = (DIM == 3) ? EY - 4 : 1;
  io.ntx = (DIM == 3) ? (P.nx + TX - 1) / TX : (P.nx + TX * EY - 1) / (TX * EY);
  io.nty = (DIM == 3) ? (P.ny + TY - 1) / TY : 1;
  const long long total = (long long)io.ntx * io.nty * P.nz;
  int ncu = ts.num_cu;
  if (ncu <= 0) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || ncu < 1)
      ncu = 256;
  }
  // at most as many workgroups as are resident at once.  2D: the step is the
  // latency of one march and a workgroup is one wave, so there is at most one a
  // SIMD while that takes no longer shares than the default; above that shares
  // of up to 4 planes, and beyond some 12,000 pairs the number of resident waves
  // decides.  Measured, viscous, us a step with a given dt, one wave a SIMD and
  // the shares that go beyond it: 60 x 1100 7.7, 9.8 (shares of 1); 512 x 256
  // (2304 pairs) 9.4, 10.3 (2); 60 x 3000 9.4, 13.1 (2); 60 x 4000 10.8, 14.5 (3);
  // 60 x 5000 12.0, 15.2 (4); 60 x 6000 13.2, 15.0 (4).  Longer shares: 60 x 8000 14.3
  // with 4 planes and with 8; 1024^2 24.2 with 2, 24.1 with 4, 25.2 with 8
  const long long simds = 4ll * ncu;
  const bool own = DIM == 2 && !ts.chosen, alone = own && total <= simds * ts.zchunk;
  const long long least = alone ? 1 : own ? std::min(4, ts.zchunk) : ts.zchunk;
  const long long tiles = (long long)io.ntx * io.nty;
  long long cap = simds;
  if (const long long c = std::min((long long)P.nz, simds / tiles); alone && c > 0) {
    // chunks a tile that make a multiple of 8 workgroups (those of an XCD are
    // then neighbours: 512 x 256, 1017 and 1008 workgroups: 10.6, 9.4 us), if
    // their shares are no longer
    const long long m = 8 / std::gcd(tiles, 8ll), c8 = c / m * m;
    if (c8 > 0 && (P.nz + c8 - 1) / c8 == (P.nz + c - 1) / c) cap = tiles * c8;
  }
  auto shares = [&](int occ) {
    const long long most = (long long)(ts.wg_per_cu > 0 ? ts.wg_per_cu : occ) * ncu;
    return shares_of(tiles, P.nz, alone ? std::min(most, cap) : most, least, 4);
  };
  io.shares = shares(resident<DIM, LM, DISS, NC, EX, EY, false>());
  // the split march where a share has enough steady planes (2D, us a step
  // whole against split: 64 x 32, 5 planes marched: 6.9, 7.3; 1024^2, 10:
  // 24.2, 23.4; 2048 x 1024, 15: 41.2, 38.4)
  const bool split = DIM == 2 && total >= 6ll * io.shares.groups;
  if (split) io.shares = shares(resident<DIM, LM, DISS, NC, EX, EY, DIM == 2>());
  const dim3 grid(io.shares.groups), block(EX * EY);
  if (split)
    hipLaunchKernelGGL((k_step_fused<DIM, LM, DISS, NC, EX, EY, DIM == 2>), grid, block, 0, s, P, Uin, Uout, io);
  else
    hipLaunchKernelGGL((k_step_fused<DIM, LM, DISS, NC, EX, EY, false>), grid, block, 0, s, P, Uin, Uout, io);
  return hipGetLastError();
}

template <int DIM, bool NC, int EX, int EY>
static hipError_t launch_variant(const Params& P, const double* Uin, double* Uout, StepIO io, const TileShape& ts,
                                 hipStream_t s) {
  const bool lm = P.low_mach != 0, ds = P.diss != 0;
  if (lm && ds) return launch_fused_t<DIM, true, true, NC, EX, EY>(P, Uin, Uout, io, ts, s);
  if (lm && !ds) return launch_fused_t<DIM, true, false, NC, EX, EY>(P, Uin, Uout, io, ts, s);
  if (!lm && ds) return launch_fused_t<DIM, false, true, NC, EX, EY>(P, Uin, Uout, io, ts, s);
  return launch_fused_t<DIM, false, false, NC, EX, EY>(P, Uin, Uout, io, ts, s);
}

hipError_t launch_step_fused(const Params& P, const double* Uin, double* Uout, StepIO io, const TileShape& ts,
                             hipStream_t s) {
  if (P.dim == 2)
    return P.nc ? launch_variant<2, true, 64, 1>(P, Uin, Uout, io, ts, s)
                : launch_variant<2, false, 64, 1>(P, Uin, Uout, io, ts, s);
  if (ts.tile3 == 1)
    return P.nc ? launch_variant<3, true, TILE3_EX[1], TILE3_EY[1]>(P, Uin, Uout, io, ts, s)
                : launch_variant<3, false, TILE3_EX[1], TILE3_EY[1]>(P, Uin, Uout, io, ts, s);
  return P.nc ? launch_variant<3, true, TILE3_EX[0], TILE3_EY[0]>(P, Uin, Uout, io, ts, s)
              : launch_variant<3, false, TILE3_EX[0], TILE3_EY[0]>(P, Uin, Uout, io, ts, s);
}

}  // namespace ars
