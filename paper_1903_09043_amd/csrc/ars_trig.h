// ars_trig.h -- trigonometric preconditioner of the implicit acoustic system
// (ars_trig.hip): the operator with its coefficients held constant, inverted
// exactly by real transforms along every axis.
#pragma once
#include "ars_dev.h"

namespace ars {

// Constant coefficients: 1/(rho c^2), tau = 1/rho and 1/(rho c).
struct TrigCoef {
  double irc2, tau, irc;
};

// Largest axis the transforms take (the matrices grow with its square).
constexpr int TRIG_MAXN = 4096;

// Doubles of scratch a problem needs: per axis the transform matrix, its
// transpose where it is not symmetric, and the eigenvalues; two fields.
size_t trig_scratch_doubles(const Params& P);

// Matrices and eigenvalues for the step *d_dt into `scratch`.
hipError_t trig_setup(const Params& P, const TrigCoef& c, const double* d_dt, double* scratch, hipStream_t s);

// z = M^-1 r; z one of the two fields inside `scratch`, returned.
hipError_t trig_solve(const Params& P, const TrigCoef& c, const double* r, double* scratch, const double** z,
                      hipStream_t s);

}  // namespace ars
