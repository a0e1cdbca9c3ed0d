// refine_rule.h -- when the mixed-precision refinement of one right-hand side
// ends (plain C++, shared by the device code and a host test).
#pragma once

namespace tsqr {

constexpr double kEtaMax = 1e-12;   // a refined x whose backward-error bound is above this is flagged (dinfo = -3)

enum RefineState { kRefineGoOn = 0, kRefineConverged = 1, kRefineStalled = 2 };

// A column after `sweeps` earlier sweeps and one whose correction is rel =
// ||dx|| / ||x|| (prev: the sweep before's).  Converged: the error left after
// this correction, estimated as rho ||dx|| with rho = rel / prev the observed
// contraction (at most 1), is below tol ||x|| -- so a sweep whose correction is
// already far below the tolerance is not needed just to confirm it.  Stalled:
// the correction shrank by less than 10 %, or is not a number.
constexpr RefineState refine_state(double rel, double prev, int sweeps, double tol) {
    if ((sweeps >= 1 && rel > 0.9 * prev) || !(rel == rel)) return kRefineStalled;
    const double q = (sweeps >= 1 && prev > 0.0) ? rel / prev : 1.0, rho = q < 1.0 ? q : 1.0;
    return rho * rel <= tol ? kRefineConverged : kRefineGoOn;
}

// Whether the column needs no further sweep.  Its status word is formed from
// the bound of the last residual pass, which comes BEFORE the last correction:
// a first correction at FP32's rounding level, about 1e-7, ends a column by
// rho rel <= 1e-14 on one side of 1e-7 and not on the other, with a residual
// that still holds the whole correction (a bound of some 1e-8 for an x that is
// right to rounding).  So a converged column also waits for a residual pass
// that shows it: eta, the bound, at most half of kEtaMax (half, because the
// status word's own sum runs in another order).  A caller's tolerance above
// kEtaMax asks for less than that, and alone decides.  known: there was a
// residual pass.
constexpr bool refine_done(RefineState state, double tol, bool known, double eta) {
    if (state != kRefineConverged) return state == kRefineStalled;
    return tol > kEtaMax || (known && eta <= 0.5 * kEtaMax);
}

}  // namespace tsqr
