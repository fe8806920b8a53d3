// ars_imex_phase.h -- what surrounds the solve of an implicit acoustic step
// whose axes are all periodic or walled at both ends (ars_imex_phase.hip).
#pragma once
#include "ars_dev.h"

namespace ars {

// Blocks whose sums and extremes imex_begin leaves in `part` (8 rows).
constexpr int IMEX_BEGIN_BLOCKS = 1024;

// Where imex_begin puts the system: unpadded vectors of P.ncell values.
struct ImexSystem {
  double *x;                // start value p^n
  double *r;                // b - A x
  double *p, *v;            // zeroed
  double *tau, *irc, *irc2; // 1/rho, 1/(rho c), 1/(rho c^2)
  double *part;             // 8 * IMEX_BEGIN_BLOCKS
  double *bb_rr;            // (b, b), (r, r)
  double *range_dt;         // smallest and largest irc2, tau, irc, then dt
};

// Primitives of U into the reference workspace W, velocities into ext (D
// padded fields), the system into S.
hipError_t imex_begin(const Params& P, const double* U, double* W, double* ext, const double* d_dt,
                      const ImexSystem& S, hipStream_t s);

// The step from the solution x, in place on U (W as imex_begin left it up to
// the face fields; the solve may have used what lies behind them).
hipError_t imex_finish(const Params& P, double* U, double* W, double* ext, const double* x, const double* d_dt,
                       Control* ctl, hipStream_t s);

}  // namespace ars
