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
  // A chain may be walked for any number of steps between two looks, each of them far below the slack's last bit, so the
  // roundings must not add up: with u = 2^-24, (1 + u)^2 (1 - 2u) < 1 and (1 - u)^2 (1 + 4u) > 1.
  SOLE_FN void moved(float by) {
    slack = (slack - by) * (1.f - 0x1p-23f);
    rho = (rho + by) * (1.f + 0x1p-22f);
  }
};
