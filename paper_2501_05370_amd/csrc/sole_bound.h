// The distances by which a Langevin chain held by one component is known to stay so (sd_langevin.hip): plain fp32 arithmetic, the
// same on the host.
#pragma once
#include <cmath>

#ifdef __HIP__
#define SOLE_FN __device__ __forceinline__
#else
#define SOLE_FN inline
#endif

struct SoleBound {
  float slack = -1.f;        // how far the state may still move with component `top` alone
  float radius = 0.f;        // of the ball around mu_top
  float rho = 0.f;           // upper bound of |x - mu_top|
  // the state is at (at most) `r` from mu_top
  SOLE_FN void at_distance(float r) {
    rho = r;
    slack = fmaxf(slack, radius - r);      // the better of two bounds; one that is not a number gives way
  }
  SOLE_FN void moved(float by) {
    slack -= by;
    rho += by;
  }
  // A chain may be walked for any number of steps between two looks, each of them below the slack's last bit, so the roundings
  // must not add up.  A window's 64 steps and this one round by 65 of 2^-24 at most, of the slack at the window's start; a factor
  // of 1 - 2^-16 takes that back where the slack fell to a quarter or less slowly, and the windows in which it fell faster
  // leave 65 (1 + 1/4 + ...) 2^-24 = 5.2e-6 of the slack when it was set, which carries a margin of 1e-4.  The distance only
  // grows: the factor covers it.  Per window and not per step: 1.5 % of a run of 1000 coordinates.
  SOLE_FN void window_ended(float by) {
    moved(by);
    slack *= 1.f - 0x1p-16f;
    rho *= 1.f + 0x1p-16f;
  }
};
