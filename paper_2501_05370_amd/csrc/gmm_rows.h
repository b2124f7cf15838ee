// Posterior mean of a diagonal Gaussian mixture for one row on one wavefront: shared by the denoiser's
// evaluation of many rows and by the kernel that runs whole chains (sdden_gmm.hip).
//
//   r_m(x)  = softmax_m( log w_m + log N(x; sqrt(ab) mu_m, diag(ab s_m^2 + 1-ab)) )
//   D(x,k)  = sum_m r_m(x) ( mu_m + sqrt(ab) s_m^2 / v_m * (x - sqrt(ab) mu_m) )
//
// Two mappings of the 64 lanes, one per phase.  Logits: lane = part + PARTS * m (component m, PARTS = 64 / Mp lanes
// per component, Mp = M rounded up to a power of two), so a quadratic form ends with log2(PARTS) exchanges.
// Mean: lane = coordinate, a loop over the components whose responsibility is at least 1e-25 (any other moves
// no coordinate by more than 1e-25 of its mean).  A pair of the mean loop recomputes its reciprocal variance,
// which costs less than keeping the 64-lane x NI table of component means in registers and exchanging it: the
// earlier form of this kernel did that and spent 1150 vector instructions per row at M = 32, d = 64 whatever
// the responsibilities were.  Most rows of a chain have one or two live components (the many-component rows
// are those of the first, noisiest steps).
// All arithmetic in fp64.  No workgroup barrier, no LDS exchange.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "sd_lanes.h"

namespace sdgmm {

constexpr int kMaxLaneComponents = 64;   // components one lane each
constexpr int kTabStride = 65;           // LDS table: units per slot (64 lanes + 1 so that both mappings read without conflicts)

struct Model {
  const float2* lane_tab;    // [nslots, 64] (mean, std) in the lane order of the logit phase; (0, 1) where there is no pair
  const float2* row_tab;     // [M, d] (mean, std)
  const double* cst;         // [T, M] log w_m - 1/2 sum_i log v_mi(k)
  const double2* steps;      // [T] (ab, sqrt(ab))
  const float* radius2;      // [M, T] where a component is alone (gmm_radius_kernel)
  int M, d, T;
  int lm;                    // log2 of Mp (PARTS = 64 >> lm)
  int nslots;                // ceil(d / PARTS), from 3 on rounded up to a multiple of 4
};

// The hardware fp64 reciprocal (measured over 10^6 arguments from e^-600 to e^600: within 4.6e-8) and one Newton step:
// relative error below 2.2e-15 in the same measurement.
__device__ __forceinline__ double reciprocal_one_step(double v) {
  const double y = __builtin_amdgcn_rcp(v);
  return y * fma(-v, y, 2.0);
}

// 1/v to fp64 rounding: with e = 1 - v y, y (1 + e + e^2) leaves e^3, for one instruction more than the Newton step.
__device__ __forceinline__ double reciprocal(double v) {
  const double y = __builtin_amdgcn_rcp(v), e = fma(-v, y, 1.0);
  return fma(y, fma(e, e, e), y);
}
template <bool FINE>
__device__ __forceinline__ double reciprocal_of(double v) {
  if constexpr (FINE) return reciprocal(v);
  else return reciprocal_one_step(v);
}

// Which mixtures keep reciprocal variances to fp64 rounding: those of more than 32 components or of more than 32 pairs per
// lane, which have always had them so.  (The others had 4e-14 before they had reciprocal_one_step.)  No fp32 result shows
// the difference: all but 3e-7 of the outputs are the correctly rounded ones with either.
inline bool needs_fine(int M, int d, int lm) { return M > 32 || (static_cast<int64_t>(d) << lm) > 32 * 64; }

// exp(x) for x <= 0; 0 below -64, where exp(x) < 2^-92 adds nothing to a sum that contains exp(0).
// x = n ln2 + f, |f| <= ln2 / 2, and the Taylor polynomial of degree 13 (remainder 4e-18), even and odd halves
// as two chains.  A NaN stays one.
__device__ __forceinline__ double exp_nonpositive(double x) {
  const double n = __builtin_rint(x * 1.4426950408889634);
  double f = fma(-n, 0x1.62e42fefa39efp-1, x);
  f = fma(-n, 0x1.abc9e3b39803fp-56, f);
  const double g = f * f;
  double e = 1.0 / 479001600.0, o = 1.0 / 6227020800.0;
  e = fma(e, g, 1.0 / 3628800.0);  o = fma(o, g, 1.0 / 39916800.0);
  e = fma(e, g, 1.0 / 40320.0);    o = fma(o, g, 1.0 / 362880.0);
  e = fma(e, g, 1.0 / 720.0);      o = fma(o, g, 1.0 / 5040.0);
  e = fma(e, g, 1.0 / 24.0);       o = fma(o, g, 1.0 / 120.0);
  e = fma(e, g, 0.5);              o = fma(o, g, 1.0 / 6.0);
  e = fma(e, g, 1.0);              o = fma(o, g, 1.0);
  const double r = __builtin_amdgcn_ldexp(fma(o, f, e), static_cast<int>(n));
  return x < -64.0 ? 0.0 : r;
}

__device__ __forceinline__ double readlane_f64(double v, int src_lane) {
  const long long bits = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane(static_cast<int>(bits), src_lane);
  const int hi = __builtin_amdgcn_readlane(static_cast<int>(bits >> 32), src_lane);
  return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<unsigned int>(lo));
}

// orders the lanes' LDS accesses of one wavefront for the compiler (the hardware executes them in program order)
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// log w_m - 1/2 sum_i log v_mi(k) of the component this lane holds in the logit phase
__device__ __forceinline__ double lane_constant(const Model& g, int k, int lane) {
  const int m = lane >> (6 - g.lm);
  return m < g.M ? g.cst[static_cast<int64_t>(k) * g.M + m] : 0.0;
}

// From a lane's share of its component's quadratic form to the component's responsibility: sum over the 64 >> LM lanes
// of a component, then softmax over the 2^LM components.
template <int LM>
__device__ __forceinline__ double responsibility(double q, double base, bool live_lane) {
  constexpr int LP = 6 - LM;
  if constexpr (LP >= 1) q += sdlane::lane_xor<1>(q);
  if constexpr (LP >= 2) q += sdlane::lane_xor<2>(q);
  if constexpr (LP >= 3) q += sdlane::lane_xor<4>(q);
  if constexpr (LP >= 4) q += sdlane::lane_xor<8>(q);
  if constexpr (LP >= 5) q = sdlane::pair_sum_rows<16>(q);
  if constexpr (LP >= 6) q = sdlane::pair_sum_rows<32>(q);
  const double logit = live_lane ? base - 0.5 * q : -INFINITY;
  double mx = logit;
  if constexpr (LP < 1) mx = fmax(mx, sdlane::lane_xor<1>(mx));
  if constexpr (LP < 2) mx = fmax(mx, sdlane::lane_xor<2>(mx));
  if constexpr (LP < 3) mx = fmax(mx, sdlane::lane_xor<4>(mx));
  if constexpr (LP < 4) mx = fmax(mx, sdlane::lane_xor<8>(mx));
  if constexpr (LP < 5) mx = sdlane::pair_max_rows<16>(mx);
  if constexpr (LP < 6) mx = sdlane::pair_max_rows<32>(mx);
  const double ex = live_lane ? exp_nonpositive(logit - mx) : 0.0;
  double sum = ex;
  if constexpr (LP < 1) sum += sdlane::lane_xor<1>(sum);
  if constexpr (LP < 2) sum += sdlane::lane_xor<2>(sum);
  if constexpr (LP < 3) sum += sdlane::lane_xor<4>(sum);
  if constexpr (LP < 4) sum += sdlane::lane_xor<8>(sum);
  if constexpr (LP < 5) sum = sdlane::pair_sum_rows<16>(sum);
  if constexpr (LP < 6) sum = sdlane::pair_sum_rows<32>(sum);
  return ex * reciprocal(sum);
}

__device__ __forceinline__ float wave_sum(float v) {
  auto other = [](float u, auto mask) { return __int_as_float(sdlane::lane_xor<decltype(mask)::value>(__float_as_int(u))); };
  v += other(v, std::integral_constant<int, 1>{});
  v += other(v, std::integral_constant<int, 2>{});
  v += other(v, std::integral_constant<int, 4>{});
  v += other(v, std::integral_constant<int, 8>{});
  v += other(v, std::integral_constant<int, 16>{});
  return v + other(v, std::integral_constant<int, 32>{});
}

// The component a chain was last seen with alone, where its state was at the last attempt, and the squared radii (gmm_radius_kernel) of that
// component's balls at 64 steps, one per lane: in a ball nothing is loaded per step.
struct Alone {
  int top = -1;
  float rho2 = 0.f;
  int base = 0;
  float radius2 = 0.f;
  __device__ __forceinline__ void load(const Model& g, int k, int lane) {
    base = k;
    radius2 = g.radius2[static_cast<int64_t>(top) * g.T + min(k + lane, g.T - 1)];
  }
};

// The constants of the steps a chain evaluates, requested one step ahead while it needs them (not in a ball).
struct Constants {
  double cur = 0.0, next = 0.0;
  int cur_k = -1, next_k = -1;
  __device__ __forceinline__ double at(const Model& g, int k, int lane) {
    if (cur_k != k) {
      cur = next_k == k ? next : lane_constant(g, k, lane);
      cur_k = k;
      next_k = min(k + 1, g.T - 1);
      next = lane_constant(g, next_k, lane);
    }
    return cur;
  }
};

// The posterior mean where component `was.top` is alone: its own mean, the same bits as with all responsibilities.  False: it
// is not known to be alone here, and `out` holds nothing.  A squared distance that is not a number is not below the radius.
template <int E, int C, bool LDS, bool FINE>
__device__ __forceinline__ bool mean_of_one(const Model& g, const double2* tab, const float (&x)[C][E], double ab, double sab,
                                            int k, int lane, Alone& was, float (&out)[C][E]) {
  if (was.top < 0) return false;
  const int lp = 6 - g.lm, top = was.top;
  if (static_cast<unsigned>(k - was.base) >= 64u) was.load(g, k, lane);
  const float r2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(was.radius2), k - was.base));
  // Far outside at the last attempt: not worth another one until the radius has come near that distance.  (Taking the distance anew
  // from every evaluation makes more attempts that fail: two models, d = 100, M = 20, 300 chains, 200 steps 990 / 1016 us; no run gained.)
  if (!(r2 > 0.8f * was.rho2)) return false;
  const double om = 1.0 - ab;
  double rho2 = 0.0;
  float2 t[C][E];
  if (!LDS) {
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int i = E * (lane + 64 * c) + e;
        t[c][e] = g.row_tab[static_cast<int64_t>(top) * g.d + (i < g.d ? i : 0)];
      }
  }
#pragma unroll
  for (int c = 0; c < C; ++c)
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int i = E * (lane + 64 * c) + e, ii = i < g.d ? i : 0;
      double mu, s2;
      if (LDS) {
        const double2 u = tab[(ii >> lp) * kTabStride + (ii & ((1 << lp) - 1)) + (top << lp)];
        mu = u.x; s2 = u.y;
      } else {
        mu = t[c][e].x;
        s2 = static_cast<double>(t[c][e].y) * t[c][e].y;
      }
      const double iv = reciprocal_of<FINE>(fma(ab, s2, om));
      const double df = fma(-sab, mu, static_cast<double>(x[c][e]));
      rho2 = i < g.d ? fma(df * df, iv, rho2) : rho2;
      out[c][e] = i < g.d ? static_cast<float>(fma(sab * s2 * iv, df, mu)) : 0.f;
    }
  was.rho2 = wave_sum(static_cast<float>(rho2));
  return __builtin_amdgcn_readfirstlane(was.rho2 < r2 ? 1 : 0) != 0;
}

// Coordinates of a lane: group c, element e -> E * (lane + 64 c) + e.  E * 64 * C >= d.
// ab, sab = sqrt(ab): signal level of the row's step; base = lane_constant of that step.
// `x` holds 0 at coordinates >= d; `xs` is wavefront-private LDS of nslots * PARTS doubles.  `tab` (LDS form only): the
// lane table as (mean, variance) doubles, slot j of lane l at j * kTabStride + l.  AHEAD (not the LDS form): table entries
// are requested a group or more ahead of their use, and a scheduling barrier keeps them there.  Left to itself the compiler
// has one load in flight where registers are short, a memory round trip per entry.  One chain of 64 components, us a step
// with / without: d = 1800 79 / 208, d = 1000 43 / 54; 1000 rows of d = 1000 81 / 157.  Row evaluations of up to 512
// coordinates do without it: the compiler keeps their four loads together, and the registers cost more than the latency
// where many wavefronts share a SIMD (32768 rows, 8 components: d = 200 60 / 58, d = 400 105 / 100).
template <int E, int C, bool LDS, bool AHEAD, bool FINE, bool SHARES = (E * C == 1)>
__device__ __forceinline__ void posterior_mean(const Model& g, const double2* tab, double* xs, const float (&x)[C][E], double ab,
                                               double sab, double base, int lane, float (&out)[C][E], Alone* was = nullptr, int k = 0) {
  const int lp = 6 - g.lm;
  const int parts = 1 << lp, part = lane & (parts - 1), m = lane >> lp;
  const int npad = g.nslots << lp;
  const bool live_lane = m < g.M;
  const double om = 1.0 - ab;
  wave_lds_fence();                        // readers of the previous call are done
#pragma unroll
  for (int c = 0; c < C; ++c)
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int i = E * (lane + 64 * c) + e;
      if (i < npad) xs[i] = static_cast<double>(x[c][e]);
    }
  wave_lds_fence();
  // Quadratic form.  Four pairs share one reciprocal: sum_i n_i / v_i over a common denominator, whose fp64 exponent
  // range holds a product of four variances anywhere in the fp32 range.
  double q = 0.0;
  const double* xp = xs + part;
  auto term = [&](double xj, double mu, double s2, double& v, double& nu) {
    v = fma(ab, s2, om);
    const double df = fma(-sab, mu, xj);                       // a slot past d: 0 - 0
    nu = df * df;
  };
  auto pair = [&](int j, double& v, double& nu) {
    if (LDS) {
      const double2 t = tab[j * kTabStride + lane];
      term(xp[j << lp], t.x, t.y, v, nu);
    } else {
      const float2 t = g.lane_tab[j * 64 + lane];
      term(xp[j << lp], t.x, static_cast<double>(t.y) * t.y, v, nu);
    }
  };
  auto add4 = [&](double v0, double v1, double v2, double v3, double n0, double n1, double n2, double n3) {
    const double n01 = fma(n0, v1, n1 * v0), v01 = v0 * v1, n23 = fma(n2, v3, n3 * v2), v23 = v2 * v3;
    q = fma(fma(n01, v23, n23 * v01), reciprocal_of<FINE>(v01 * v23), q);
  };
  int j = 0;
  if (AHEAD && g.nslots >= 4) {
    float2 t[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) t[i] = g.lane_tab[i * 64 + lane];
    for (; j + 3 < g.nslots; j += 4) {
      const int jn = j + 7 < g.nslots ? j + 4 : j;
      float2 next[4];
      double xj[4], v[4], nu[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) next[i] = g.lane_tab[(jn + i) * 64 + lane];
#pragma unroll
      for (int i = 0; i < 4; ++i) xj[i] = xp[(j + i) << lp];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        term(xj[i], t[i].x, static_cast<double>(t[i].y) * t[i].y, v[i], nu[i]);
        t[i] = next[i];
      }
      add4(v[0], v[1], v[2], v[3], nu[0], nu[1], nu[2], nu[3]);
    }
  }
  for (; !AHEAD && j + 3 < g.nslots; j += 4) {
    double v0, v1, v2, v3, n0, n1, n2, n3;
    pair(j, v0, n0);
    pair(j + 1, v1, n1);
    pair(j + 2, v2, n2);
    pair(j + 3, v3, n3);
    add4(v0, v1, v2, v3, n0, n1, n2, n3);
  }
  for (; j < g.nslots; ++j) {
    double v, nu;
    pair(j, v, nu);
    q = fma(nu, reciprocal_of<FINE>(v), q);
  }
  double r;
  switch (g.lm) {                          // uniform: one jump instead of a branch per exchange level
    case 0: r = responsibility<0>(q, base, live_lane); break;
    case 1: r = responsibility<1>(q, base, live_lane); break;
    case 2: r = responsibility<2>(q, base, live_lane); break;
    case 3: r = responsibility<3>(q, base, live_lane); break;
    case 4: r = responsibility<4>(q, base, live_lane); break;
    case 5: r = responsibility<5>(q, base, live_lane); break;
    default: r = responsibility<6>(q, base, live_lane); break;
  }
  unsigned long long live = __ballot(live_lane && part == 0 && !(r < 1e-25));   // a NaN counts as live and reaches the result

  if (was) {
    const bool one = live != 0 && (live & (live - 1)) == 0;
    const int top = one ? __builtin_ctzll(live) >> lp : -1;
    if (top != was->top) {
      was->top = top;
      was->rho2 = 0.f;
      if (one) was->load(g, k, lane);      // used from the next evaluation on
    }
  }

  if constexpr (SHARES) {
    static_assert(E * C == 1, "a coordinate per lane");
    // Few pairs per lane: every component's share of a coordinate is in the logit phase's lanes already, and adding them up takes
    // log2(Mp) exchanges per pair instead of a loop over the live components; ahead with one pair, or from two live
    // components per pair on.  us of a run, with / without: 4096 chains, d = 3, M = 16, 100 steps 260 / 418; 4096 chains, d = 5,
    // M = 20, 200 steps 714 / 850; 500 chains, d = 8, M = 48, carried, 100 steps 206 / 242; toy runs within 5 %.
    auto sum_of_shares = [&](int s) {
      double mu, s2;
      if (LDS) {
        const double2 t = tab[s * kTabStride + lane];
        mu = t.x; s2 = t.y;
      } else {
        const float2 t = g.lane_tab[s * 64 + lane];
        mu = t.x; s2 = static_cast<double>(t.y) * t.y;
      }
      const double df = fma(-sab, mu, xp[s << lp]);
      double share = r * fma(sab * s2 * reciprocal_of<FINE>(fma(ab, s2, om)), df, mu);
      if (!live_lane || r < 1e-25) share = 0.0;            // a NaN stays
      if (lp < 1) share += sdlane::lane_xor<1>(share);
      if (lp < 2) share += sdlane::lane_xor<2>(share);
      if (lp < 3) share += sdlane::lane_xor<4>(share);
      if (lp < 4) share += sdlane::lane_xor<8>(share);
      if (lp < 5) share = sdlane::pair_sum_rows<16>(share);
      if (lp < 6) share = sdlane::pair_sum_rows<32>(share);
      return share;
    };
    if (g.nslots == 1 || __popcll(live) > 2 * g.nslots) {
      double sum = sum_of_shares(0);
      for (int s = 1; s < g.nslots; ++s) {
        const double next = sum_of_shares(s);
        if ((lane >> lp) == s) sum = next;                 // coordinate `lane` is pair s of the lanes with its part
      }
      out[0][0] = lane < g.d ? static_cast<float>(sum) : 0.f;
      return;
    }
  }

  double acc[C][E];
#pragma unroll
  for (int c = 0; c < C; ++c)
#pragma unroll
    for (int e = 0; e < E; ++e) acc[c][e] = 0.0;
  auto at = [&](int mc, int ii, double& mu, double& s2) {
    if (LDS) {
      const double2 t = tab[(ii >> lp) * kTabStride + (ii & (parts - 1)) + (mc << lp)];
      mu = t.x; s2 = t.y;
    } else {
      const float2 t = g.row_tab[static_cast<int64_t>(mc) * g.d + ii];
      mu = t.x;
      s2 = static_cast<double>(t.y) * t.y;
    }
  };
  auto add_one = [&](int c, int e, double r0, double mu, double s2) {
    const double iv = reciprocal_of<FINE>(fma(ab, s2, om));
    const double df = fma(-sab, mu, static_cast<double>(x[c][e]));
    acc[c][e] = fma(r0, fma(sab * s2 * iv, df, mu), acc[c][e]);
  };
  auto add_four = [&](int c, int e, double r0, double r1, double r2, double r3, double mu0, double mu1, double mu2, double mu3,
                      double s0, double s1, double s2, double s3) {
    const double xi = static_cast<double>(x[c][e]);
    const double v0 = fma(ab, s0, om), v1 = fma(ab, s1, om), v2 = fma(ab, s2, om), v3 = fma(ab, s3, om);
    const double n0 = r0 * s0 * fma(-sab, mu0, xi), n1 = r1 * s1 * fma(-sab, mu1, xi);
    const double n2 = r2 * s2 * fma(-sab, mu2, xi), n3 = r3 * s3 * fma(-sab, mu3, xi);
    const double n01 = fma(n0, v1, n1 * v0), v01 = v0 * v1, n23 = fma(n2, v3, n3 * v2), v23 = v2 * v3;
    acc[c][e] = fma(r0, mu0, acc[c][e]);
    acc[c][e] = fma(r1, mu1, acc[c][e]);
    acc[c][e] = fma(r2, mu2, acc[c][e]);
    acc[c][e] = fma(r3, mu3, acc[c][e]);
    acc[c][e] = fma(sab * fma(n01, v23, n23 * v01), reciprocal_of<FINE>(v01 * v23), acc[c][e]);
  };
  auto request = [&](int mc, int c, float2 (&to)[E]) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int i = E * (lane + 64 * c) + e;
      to[e] = g.row_tab[static_cast<int64_t>(mc) * g.d + (i < g.d ? i : 0)];
    }
  };
  auto var = [](float2 t) { return static_cast<double>(t.y) * t.y; };
  while (live) {                           // uniform: the mask is the same on every lane
    // up to four components at a time over a common denominator, as above; a missing one repeats the last with weight 0
    int bit = __builtin_ctzll(live);
    live &= live - 1;
    const int m0 = bit >> lp;
    const double r0 = readlane_f64(r, bit);
    if (!live) {
      if constexpr (AHEAD) {
        float2 t[3][E];                    // two groups ahead
        request(m0, 0, t[0]);
        if (C > 1) request(m0, 1, t[1]);
#pragma unroll
        for (int c = 0; c < C; ++c) {
          if (c + 2 < C) {
            request(m0, c + 2, t[(c + 2) % 3]);
            __builtin_amdgcn_sched_barrier(0);
          }
#pragma unroll
          for (int e = 0; e < E; ++e) add_one(c, e, r0, t[c % 3][e].x, var(t[c % 3][e]));
        }
      } else {
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
          for (int e = 0; e < E; ++e) {
            const int i = E * (lane + 64 * c) + e;
            double mu, s2;
            at(m0, i < g.d ? i : 0, mu, s2);
            add_one(c, e, r0, mu, s2);
          }
      }
      break;
    }
    bit = __builtin_ctzll(live);
    live &= live - 1;
    const int m1 = bit >> lp;
    const double r1 = readlane_f64(r, bit);
    bit = live ? __builtin_ctzll(live) : bit;
    const int m2 = bit >> lp;
    const double r2 = live ? readlane_f64(r, bit) : 0.0;
    live &= live - 1;
    bit = live ? __builtin_ctzll(live) : bit;
    const int m3 = bit >> lp;
    const double r3 = live ? readlane_f64(r, bit) : 0.0;
    live &= live - 1;
    if constexpr (AHEAD) {
#pragma unroll
      for (int c = 0; c < C; ++c) {        // the four components of a group together
        float2 t[4][E];
        request(m0, c, t[0]);
        request(m1, c, t[1]);
        request(m2, c, t[2]);
        request(m3, c, t[3]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < E; ++e)
          add_four(c, e, r0, r1, r2, r3, t[0][e].x, t[1][e].x, t[2][e].x, t[3][e].x, var(t[0][e]), var(t[1][e]), var(t[2][e]),
                   var(t[3][e]));
      }
    } else {
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const int i = E * (lane + 64 * c) + e, ii = i < g.d ? i : 0;
          double mu0, mu1, mu2, mu3, s0, s1, s2, s3;
          at(m0, ii, mu0, s0);
          at(m1, ii, mu1, s1);
          at(m2, ii, mu2, s2);
          at(m3, ii, mu3, s3);
          add_four(c, e, r0, r1, r2, r3, mu0, mu1, mu2, mu3, s0, s1, s2, s3);
        }
    }
  }
#pragma unroll
  for (int c = 0; c < C; ++c)
#pragma unroll
    for (int e = 0; e < E; ++e) out[c][e] = E * (lane + 64 * c) + e < g.d ? static_cast<float>(acc[c][e]) : 0.f;
}

}  // namespace sdgmm
