// One speculative window of unadjusted Langevin on a Gaussian-mixture energy, fused in one launch.
//
// Paper: Sec. 5 and Alg. "Speculative Sampling for Unadjusted Langevin Diffusion", frozen-gradient
// proxy (grad E^(x_{n+j}) = grad E(x_n)):
//   draft    y~_{j} = y~_{j-1} - gamma g0 + sqrt(2 gamma) z_j,          g0 = grad E(x_n)
//   target   mean     y~_{j-1} - gamma grad E(y~_{j-1})
//   Delta_j = sqrt(gamma/2) (grad E(y~_{j-1}) - g0),  accept iff log u <= min(0, -z.Delta - |Delta|^2/2)
//   reject:  x_out = y~_{j-1} - gamma grad E(y~_{j-1}) + sqrt(2 gamma) (z - 2 (z.Delta/|Delta|^2) Delta)
// with E(x) = -log sum_m w_m N(x; mu_m, s^2 I), grad E = (x - sum_m r_m(x) mu_m) / s^2.
//
// Three kernels.  For d <= 128 several chains share a wavefront (langevin_short_kernel), for d <= 1024 a WAVEFRONT owns a
// chain (langevin_window_wave_kernel), for larger d a workgroup does (langevin_window_kernel).  State, frozen gradient and
// Delta stay in registers, and because the whole chain lives in one place the walk simply stops at the first rejection: no
// work is spent on drafts that would be discarded.  The 16 logits and the two dot products of a position are summed in
// fp64.  The phi^4 lattice energy has kernels of its own at the end of the file.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "sd_internal.h"
#include "sd_lanes.h"
#include "sd_rng.h"
#include "sole_bound.h"

namespace {

constexpr int kMaxGroups = 1024;           // groups of four coordinates a chain may have

struct LangevinArgs {
  const float* x;
  const int32_t* n;
  const int64_t* id;
  const float* means;   // [M,d]
  const float* logw;    // [M]
  float* x_out;
  int32_t* adv;
  uint8_t* rej;
  float *logratio, *logu;
  const int32_t* active;
  int32_t* queue;       // [0]: the wavefront kernel's next chain to hand out; [1]: windows of the longest chain of a run to T
                        // (each zeroed ahead of the launch that uses it)
  int max_windows;      // 1: one window per chain (sd_langevin_window); > 1: windows back to back (sd_langevin_run)
  int32_t* n_out;       // run mode: the step each chain reached
  unsigned long long* counters;   // run mode, optional: sum adv, chain-windows, rejections, launches, sum Kt
  int B, d, K, T, M;
  uint64_t seed;
  double gamma, inv_s2, inv_tau;
};

// v of lane (lane ^ mask), mask a single bit known at compile time after unrolling
__device__ __forceinline__ double dpp_xor(double v, int mask) {
  switch (mask) {
    case 1: return sdlane::lane_xor<1>(v);
    case 2: return sdlane::lane_xor<2>(v);
    case 4: return sdlane::lane_xor<4>(v);
    case 8: return sdlane::lane_xor<8>(v);
    case 16: return sdlane::lane_xor<16>(v);
    default: return sdlane::lane_xor<32>(v);
  }
}

// ---------------------------------------------------------------------------------------------
// While one component holds a state, its logits need not be computed.  The log-odds of component a over m,
//   l_a(x) - l_m(x) = log w_a - log w_m + (|x - mu_m|^2 - |x - mu_a|^2) / 2 s^2,
// are linear in x with slope |mu_a - mu_m| / s^2.  With x0 a state where they were computed, they stay above kSoleGap for
// every m while |x - x0| < min_m (odds_m(x0) - kSoleGap) s^2 / |mu_a - mu_m|; and wherever |x - mu_a| <
// min_m ((|mu_a - mu_m|^2 / 2 s^2 + log w_a - log w_m) - kSoleGap) s^2 / |mu_a - mu_m|, the ball's radius.  All other
// responsibilities are then below e^-60 < 1e-25, which the weighted mean skips and the softmax sum rounds away: the
// responsibility of a is exactly 1, the gradient (x - mu_a) / s^2, the same bits as with all logits.  On mixtures whose
// components lie a few standard deviations per coordinate apart a chain is in a ball almost all the time; elsewhere the
// logits are computed as ever.  Distances walked are bounded from above, radii from below: each in fp32 with a margin (kUp,
// kDown) far above its rounding, and sums of them for any number of steps (sole_bound.h).  Whatever is not a number fails the
// comparison with 0 and takes the long way.
// Where it does not hold: overlapping components, 16 of them, runs of 100 steps, us with the rule in the kernel / before it was:
// 4096 chains, d = 250 672 / 761, d = 1000 1503 / 1928, 300 chains, d = 150 305 / 367 (the wavefront kernel; the other one below).
// ---------------------------------------------------------------------------------------------
constexpr double kSoleGap = 60.0;
constexpr double kSoleEnter = 72.0;        // gap from which the workgroup-per-chain kernel follows one component: not at every flicker
constexpr float kUp = 1.0001f, kDown = 0.9999f;

struct Sole : SoleBound {
  int top = -1;              // component the distances belong to
  __device__ __forceinline__ bool holds() const { return __builtin_amdgcn_readfirstlane(slack > 0.f ? 1 : 0) != 0; }
};

// Sum over the wavefront in fp32, the same bits on every lane.
__device__ __forceinline__ float wave_sum_f32(float v) {
  auto x = [](float u, int mask) {
    const int b = __float_as_int(u);
    return __int_as_float(mask == 1 ? sdlane::lane_xor<1>(b) : mask == 2 ? sdlane::lane_xor<2>(b) : mask == 4 ? sdlane::lane_xor<4>(b)
                          : mask == 8 ? sdlane::lane_xor<8>(b) : mask == 16 ? sdlane::lane_xor<16>(b) : sdlane::lane_xor<32>(b));
  };
  v += x(v, 1);
  v += x(v, 2);
  v += x(v, 4);
  v += x(v, 8);
  v += x(v, 16);
  return v + x(v, 32);
}

// Least value over the other components, lane l speaking for component l >> 2; one that is not a number counts as -inf.
__device__ __forceinline__ float least_of_others(float v, bool other) {
  v = other ? (v == v ? v : -INFINITY) : INFINITY;
  v = fminf(v, __int_as_float(sdlane::lane_xor<4>(__float_as_int(v))));
  v = fminf(v, __int_as_float(sdlane::lane_xor<8>(__float_as_int(v))));
  v = fminf(v, __int_as_float(sdlane::lane_xor<16>(__float_as_int(v))));
  return fminf(v, __int_as_float(sdlane::lane_xor<32>(__float_as_int(v))));
}

// ---------------------------------------------------------------------------------------------
// One WAVEFRONT per chain (d <= 1024 * CPT/4): no workgroup barrier on the walk at all.
// A lane owns CPT groups of four coordinates; the mixture means sit in LDS as fp64, once per workgroup
// (its wavefronts share them; the workgroups stay resident for the whole launch and their
// wavefronts draw chains from a counter).  Logits use  log w_m + (x.mu_m - |mu_m|^2/2)/s^2  (the |x|^2
// term cancels in the softmax), so a position costs two passes over the means: 16 dot products and the
// responsibility-weighted mean.  The 16 per-lane partial dot products are reduced with a transposed
// butterfly (values are exchanged in halves, 17 exchanges instead of 96, all of them DPP moves or row
// swaps in the vector ALU); responsibilities are then broadcast through scalar registers.
// RUN: the chain's windows follow each other inside the kernel (sd_langevin_run).
// ---------------------------------------------------------------------------------------------
// Wavefronts of the one workgroup a CU holds, as many as the registers of CPT groups of coordinates let reside: 2, 3 or 4 per
// SIMD.  16384 chains, d = 250 1.85 ms (2.27 with two per SIMD); 8000 chains, d = 400 1.24 (1.43); with few chains the
// workgroups take a wavefront or two each instead of filling some CUs: 100 chains, d = 201 0.31 (0.40).
constexpr int wave_chains(int cpt) { return cpt <= 2 ? 16 : cpt == 3 ? 12 : 8; }
constexpr int kWaveM = 16;                 // components handled by the transposed reduction

// the steps of reduce16_transposed after the first
template <int N>
__device__ __forceinline__ double reduce8_transposed(double (&a)[N]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) a[i] = sdlane::halving_add<16>(a[i], a[i + 4]);
#pragma unroll
  for (int i = 0; i < 2; ++i) a[i] = sdlane::halving_add<8>(a[i], a[i + 2]);
  a[0] = sdlane::halving_add<4>(a[0], a[1]);
  a[0] += sdlane::lane_xor<2>(a[0]);
  a[0] += sdlane::lane_xor<1>(a[0]);
  return a[0];
}

// in: 16 per-lane partial sums; out: total of value ((lane >> 2) & 15), on every lane
__device__ __forceinline__ double reduce16_transposed(double (&a)[16], int lane) {
  (void)lane;
#pragma unroll
  for (int i = 0; i < 8; ++i) a[i] = sdlane::halving_add<32>(a[i], a[i + 8]);
  return reduce8_transposed(a);
}

__device__ __forceinline__ double readlane_f64(double v, int src_lane) {
  const long long bits = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane(static_cast<int>(bits), src_lane);
  const int hi = __builtin_amdgcn_readlane(static_cast<int>(bits >> 32), src_lane);
  return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<unsigned int>(lo));
}

// Sum over the 16 lanes of a row, the same bits on each.
__device__ __forceinline__ double row_sum(double v) {
  v += sdlane::lane_xor<1>(v);
  v += sdlane::lane_xor<2>(v);
  v += sdlane::lane_xor<4>(v);
  return v + sdlane::lane_xor<8>(v);
}
__device__ __forceinline__ float row_sum(float v) {
  v += __int_as_float(sdlane::lane_xor<1>(__float_as_int(v)));
  v += __int_as_float(sdlane::lane_xor<2>(__float_as_int(v)));
  v += __int_as_float(sdlane::lane_xor<4>(__float_as_int(v)));
  return v + __int_as_float(sdlane::lane_xor<8>(__float_as_int(v)));
}

// Sum over each half of the wavefront.
__device__ __forceinline__ double half_wave_sum(double v) { return sdlane::pair_sum_rows<16>(row_sum(v)); }
__device__ __forceinline__ float half_wave_sum(float v) {
  v = row_sum(v);
  return v + __int_as_float(sdlane::lane_xor<16>(__float_as_int(v)));
}

// sdlane::halving_add in fp32
template <int MASK>
__device__ __forceinline__ float halving_add_f32(float lower, float upper) {
  if constexpr (MASK == 32 || MASK == 16) {
    const sdlane::uint2v r = MASK == 32 ? __builtin_amdgcn_permlane32_swap(__float_as_uint(lower), __float_as_uint(upper), false, false)
                                        : __builtin_amdgcn_permlane16_swap(__float_as_uint(lower), __float_as_uint(upper), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
  } else {
    const bool up = __lane_id() & MASK;
    const float keep = up ? upper : lower, send = up ? lower : upper;
    return keep + __int_as_float(sdlane::lane_xor<MASK>(__float_as_int(send)));
  }
}

// As reduce16_transposed: in 16 per-lane sums, out the total of value ((lane >> 2) & 15).
__device__ __forceinline__ float reduce16_transposed_f32(float (&a)[16]) {
#pragma unroll
  for (int i = 0; i < 8; ++i) a[i] = halving_add_f32<32>(a[i], a[i + 8]);
#pragma unroll
  for (int i = 0; i < 4; ++i) a[i] = halving_add_f32<16>(a[i], a[i + 4]);
#pragma unroll
  for (int i = 0; i < 2; ++i) a[i] = halving_add_f32<8>(a[i], a[i + 2]);
  float v = halving_add_f32<4>(a[0], a[1]);
  v += __int_as_float(sdlane::lane_xor<2>(__float_as_int(v)));
  return v + __int_as_float(sdlane::lane_xor<1>(__float_as_int(v)));
}

struct FourFloats {                        // four floats at any float's address
  float x, y, z, w;
};

// d > 1024: a workgroup per chain, a thread per group of four coordinates (= one Philox block), up to 1024 threads.
// What bounds it is one chain's walk, a serial chain of gradients, and at 1024 threads the issue of its 16 wavefronts.  Hence
// one group per thread; the sums of a position, two to a butterfly, in one exchange over LDS that every wavefront adds up
// itself; buffers that alternate, so one barrier per exchange; the noise drawn while sums settle; uniforms 64 steps at a time.
// Two loops, between which a chain changes with its state (RUN; a single window has the first alone), because the second's
// branches and registers in the first cost a fifth of its time:
//   all logits: 16 squared distances in fp64, whose exchange is a position's first.
//   held by one component: no logits and one exchange.  Where the distances walked no longer prove that it is alone, fp32
//   distances with a bound on their error travel with the sums; what they do not confirm is done the first way.
// LDS: all means lie there as fp32, else (window form; runs whose means do not fit) the first eight, and the first loop has the
// others in registers while it runs: two chains of up to 384 threads share a CU where 16 rows each would not.  Both loops ask
// for the next means before they use the last ones; two pairs ahead, not one or four (5 % more at 320 to 512 threads).
// Whole runs, 60 steps, us (with all means in registers and all logits at every position): components two standard deviations
// per coordinate apart 200 chains, d = 1100, M = 9 156 (229), d = 2500 188 (309), 700 chains, d = 1100, M = 16 474 (627),
// 100 chains, d = 4000, M = 16 286 (520); overlapping components, the same sizes 242 (243), 315 (325), 712 (687), 444 (566).  Windows
// of 8, 600 chains, d = 1100, M = 16 70 us each (94).
// MAXT: bound on the workgroup's threads (512, 768 or 1024: 256, 168 or 128 registers per thread).
// RUN: the chain's windows follow each other inside the kernel, what sd_advance does to the chain between two of them
// included (the state passes through fp32, so the bits are those of separate calls).
template <int MAXT, bool RUN, bool LDS>
__global__ __launch_bounds__(MAXT) void langevin_window_kernel(LangevinArgs p) {
  constexpr int MC = 16, MR = LDS ? MC : MC / 2;           // MR: components in LDS
  constexpr int NW = 16;                       // slots of the sums over wavefronts; those the launch does not have hold 0
  extern __shared__ __align__(16) float4 sh_means[];       // [min(M, MR)][blockDim.x], 0 beyond d
  __shared__ double sh_part[2][NW][MC];
  __shared__ float sh_near[2][NW][MC];
  __shared__ double sh_s[2][2][NW];            // z.Delta, |Delta|^2
  __shared__ float sh_n[2][2][NW];             // |z|^2, |g|^2

  const int b = blockIdx.x;
  const int Bact = p.active ? min(p.B, max(0, *p.active)) : p.B;
  if (b >= Bact) return;                       // uniform over the workgroup
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  int n = __builtin_amdgcn_readfirstlane(p.n[b]);
  const int64_t id = p.id[b];
  const int d = p.d, M = p.M;
  const double gamma = p.gamma, inv_s2 = p.inv_s2;
  const double sq2g = sqrt(2.0 * gamma), sqg2 = sqrt(0.5 * gamma);
  const int my_m = lane >> 2;                  // component whose totals this lane holds after a reduction
  const double my_logw = my_m < M ? static_cast<double>(p.logw[my_m]) : 0.0;

  for (int q = t; q < 2 * NW * MC; q += blockDim.x) {
    (&sh_part[0][0][0])[q] = 0.0;
    (&sh_near[0][0][0])[q] = 0.f;
  }
  if (t < 4 * NW) {
    (&sh_s[0][0][0])[t] = 0.0;
    (&sh_n[0][0][0])[t] = 0.f;
  }

  // ---- my coordinates, my slice of the means (0 beyond d; noise is 0 there too, so state, gradient and Delta stay 0)
  bool own[4];
  double cur[4];                               // y~_{j-1}: the state the target gradient is evaluated at
  const int i0 = 4 * t;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    own[e] = i0 + e < d;
    cur[e] = own[e] ? static_cast<double>(p.x[static_cast<int64_t>(b) * d + i0 + e]) : 0.0;
  }
  auto from_memory = [&](int m) {
    const float* row = p.means + static_cast<int64_t>(m) * d;
    if (own[3]) {
      const FourFloats v = *reinterpret_cast<const FourFloats*>(row + i0);
      return make_float4(v.x, v.y, v.z, v.w);
    }
    return make_float4(own[0] ? row[i0] : 0.f, own[1] ? row[i0 + 1] : 0.f, own[2] ? row[i0 + 2] : 0.f, 0.f);
  };
  const int rows = min(M, MR);                 // in LDS
  for (int m = 0; m < rows; ++m) sh_means[m * blockDim.x + t] = from_memory(m);
  auto mean_at = [&](int m) { return m < rows ? sh_means[m * blockDim.x + t] : from_memory(m); };
  __syncthreads();
  auto draw = [&](int k, float (&z)[4]) {
    sdrng::normal4(p.seed, id, static_cast<uint32_t>(k), sdrng::kStreamNoise, static_cast<uint32_t>(t), z);
#pragma unroll
    for (int e = 0; e < 4; ++e) z[e] = own[e] ? z[e] : 0.f;
  };

  auto square = [](const double (&from)[4], const float4& mu) {            // unowned coordinates contribute 0 - 0
    const double d0 = from[0] - mu.x, d1 = from[1] - mu.y, d2 = from[2] - mu.z, d3 = from[3] - mu.w;
    return fma(d3, d3, fma(d2, d2, fma(d1, d1, d0 * d0)));
  };
  // 16 sums over the workgroup, the lower and the upper half of them already added over half a wavefront: lane l gets that
  // of component l >> 2.  A buffer is written again two calls later, past the barrier of the next one.  Uniform control flow:
  // called by every thread.
  int buf = 0;
  auto total = [&](double (&q)[MC / 2], auto&& meanwhile) {
    const double part = reduce8_transposed(q);
    if ((lane & 3) == 0) sh_part[buf][wave][my_m] = part;
    meanwhile();
    __syncthreads();
    double tot = 0.0;                          // the four lanes of a component add four wavefronts each
#pragma unroll
    for (int w = 0; w < NW; w += 4) tot += sh_part[buf][w + (lane & 3)][my_m];
    tot += sdlane::lane_xor<1>(tot);
    tot += sdlane::lane_xor<2>(tot);
    buf ^= 1;
    return tot;
  };
  auto softmax = [&](double logit, double& mx) {
    mx = logit;
#pragma unroll
    for (int s = 4; s <= 32; s <<= 1) mx = fmax(mx, dpp_xor(mx, s));
    const double ex = my_m < M ? exp(logit - mx) : 0.0;
    double sum = ex;
#pragma unroll
    for (int s = 4; s <= 32; s <<= 1) sum += dpp_xor(sum, s);
    return ex / sum;
  };

  // One pass of either loop below is one position of a window: the gradient at the state (at a window's first position the
  // frozen one, and the position is accepted: Delta = 0), accept test, new state.
  int Kt = max(0, min(p.K, p.T - n)), j = 0, jdone = 0, sbuf = 0;
  bool rejected = false;
  unsigned long long acc_adv = 0, acc_win = 0, acc_rej = 0, acc_kt = 0;
  double g0[4] = {0.0, 0.0, 0.0, 0.0};
  int lu_base = 0;                             // log u of 64 steps, lane l holding step lu_base + l
  bool lu_have = false;
  double lu_batch = 0.0;
  float z[4];

  auto uniforms = [&](int k1) {
    if (!lu_have || k1 - lu_base >= 64) {
      lu_base = k1;
      lu_have = true;
      lu_batch = sdrng::log_uniform(p.seed, id, static_cast<uint32_t>(k1 + lane));
    }
  };
  // Delta and this wavefront's share of z.Delta and |Delta|^2: two sums in one butterfly, the lower half of the wavefront carries
  // the first, the upper half the second
  auto products = [&](const double (&g)[4], double (&dl)[4]) {
    if (j == 0) {
#pragma unroll
      for (int e = 0; e < 4; ++e) g0[e] = g[e];
    }
    double a1 = 0.0, a2 = 0.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      dl[e] = sqg2 * (g[e] - g0[e]);
      a1 = fma(static_cast<double>(z[e]), dl[e], a1);
      a2 = fma(dl[e], dl[e], a2);
    }
    return half_wave_sum(sdlane::halving_add<32>(a1, a2));
  };
  // accept test and new state, from the sums that lie in sh_s[at]
  auto decide = [&](int at, const double (&g)[4], const double (&dl)[4]) {
    const double s_half = row_sum(sh_s[at][lane >> 5][lane & 15]);
    const double S1 = readlane_f64(s_half, 0), S2 = readlane_f64(s_half, 32), lu = readlane_f64(lu_batch, n + j + 1 - lu_base);
    double lr = 0.0, coef = 0.0;
    bool reject = false;
    if (j > 0) {
      lr = (-S1 - 0.5 * S2) * p.inv_tau;
      reject = !(S2 == 0.0 || (lr == lr && lu <= fmin(0.0, lr)));   // a log-ratio that is not a number rejects
      reject = __builtin_amdgcn_readfirstlane(reject ? 1 : 0) != 0;
      coef = S2 > 0.0 ? S1 / S2 : 0.0;
    }
    if (!RUN && t == 0) {
      if (p.logratio) p.logratio[static_cast<int64_t>(b) * p.K + j] = static_cast<float>(lr);
      if (p.logu) p.logu[static_cast<int64_t>(b) * p.K + j] = static_cast<float>(lu);
    }
    if (reject) {
#pragma unroll
      for (int e = 0; e < 4; ++e) cur[e] = cur[e] - gamma * g[e] + sq2g * (static_cast<double>(z[e]) - 2.0 * coef * dl[e]);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) cur[e] = cur[e] - gamma * g0[e] + sq2g * static_cast<double>(z[e]);
    }
    ++j;
    return reject;
  };
  // end of a window (RUN: the next one begins); Kt = 0: the last one
  auto end_window = [&](bool reject) {
    jdone = j;
    rejected = reject;
    n += j;
    acc_adv += j; acc_win += 1; acc_rej += reject ? 1 : 0; acc_kt += Kt;
    j = 0;
    Kt = RUN ? max(0, min(p.K, p.T - n)) : 0;
    if (RUN) {
#pragma unroll
      for (int e = 0; e < 4; ++e) cur[e] = static_cast<double>(static_cast<float>(cur[e]));
    }
  };

  // All branches are uniform: every wavefront holds the same totals.  Kt is uniform; every window advances the chain by at
  // least one step, and each loop takes at least one position.
  while (Kt > 0) {
    // ---- all logits
    float mreg[MR < MC ? MC - MR : 1][4];      // the components that are not in LDS
#pragma unroll
    for (int m = MR; m < MC; ++m) {
      const float4 v = from_memory(min(m, M - 1));
      mreg[m - MR][0] = v.x; mreg[m - MR][1] = v.y; mreg[m - MR][2] = v.z; mreg[m - MR][3] = v.w;
    }
    auto mean = [&](int m) {                   // m is known at compile time; from M on any that exists, which nobody uses
      if (m < MR) return sh_means[min(m, rows - 1) * blockDim.x + t];
#pragma unroll
      for (int e = 0; e < 4; ++e) asm volatile("" : "+v"(mreg[m - MR][e]));        // no converted copies across the walk
      return make_float4(mreg[m - MR][0], mreg[m - MR][1], mreg[m - MR][2], mreg[m - MR][3]);
    };
    bool one = false;                          // the position's state is held by one component
    while (Kt > 0 && !one) {
      uniforms(n + j + 1);
      double q[MC / 2];                        // the first halving step as the sums come, to keep half of them
      float4 lo[2], hi[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        lo[u] = mean(u);
        hi[u] = mean(MC / 2 + u);
      }
#pragma unroll
      for (int m = 0; m < MC / 2; m += 2) {   // two pairs at a time, the next ones on their way
        float4 lo2[2], hi2[2];
        if (m + 2 < MC / 2) {
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            lo2[u] = mean(m + 2 + u);
            hi2[u] = mean(MC / 2 + m + 2 + u);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          q[m + u] = sdlane::halving_add<32>(square(cur, lo[u]), square(cur, hi[u]));
          lo[u] = lo2[u];
          hi[u] = hi2[u];
        }
      }
      const double tot = total(q, [&]() { draw(n + j + 1, z); });          // the noise while the sums settle
      const double logit = my_m < M ? my_logw - 0.5 * tot * inv_s2 : -INFINITY;
      double mx;
      const double r_mine = softmax(logit, mx);            // every wavefront runs it itself
      if (RUN) one = __popcll(__ballot(my_m < M && !(mx - logit > kSoleEnter))) <= 4;
      double g[4], dl[4], bar[4] = {0.0, 0.0, 0.0, 0.0};
      float4 mu[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) mu[u] = mean(u);
#pragma unroll
      for (int m0 = 0; m0 < MC; m0 += 4) {     // four at a time, the next four on their way
        if (m0 >= M) break;
        float4 mu2[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (m0 + 4 < MC) mu2[u] = mean(m0 + 4 + u);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const double r = readlane_f64(r_mine, 4 * (m0 + u));             // uniform: lives in scalar registers
          if (r < 1e-25 || m0 + u >= M) continue;          // moves nothing by more than 1e-25 |mu| (see the wavefront kernel)
          bar[0] = fma(r, static_cast<double>(mu[u].x), bar[0]);
          bar[1] = fma(r, static_cast<double>(mu[u].y), bar[1]);
          bar[2] = fma(r, static_cast<double>(mu[u].z), bar[2]);
          bar[3] = fma(r, static_cast<double>(mu[u].w), bar[3]);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) mu[u] = mu2[u];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) g[e] = (cur[e] - bar[e]) * inv_s2;
      const double both = products(g, dl);
      const int at = sbuf;
      if ((lane & 31) == 0) sh_s[at][lane >> 5][wave] = both;              // last read two rounds ago
      __syncthreads();
      sbuf ^= 1;
      const bool reject = decide(at, g, dl);
      if (reject || j >= Kt) end_window(reject);
    }
    if (!RUN) break;

    // ---- held by one component: looked for with all logits at the first position, then followed
    Sole sole;
    float per_nat = 0.f, norm_top = 0.f;       // s^2 / |mu_top - mu_{my_m}|, at most; |mu_top|
    float4 mt = make_float4(0.f, 0.f, 0.f, 0.f);           // mu_top
    float gn0 = INFINITY;                      // |g0|; a window that is under way has an unknown one
    auto distances = [&](const double (&from)[4], int self) {
      auto dist2 = [&](int m) {
        if (m >= M) return 0.0;
        float4 mu = mean_at(m);
        if (m == self) mu = make_float4(0.f, 0.f, 0.f, 0.f);               // the vector itself in place of its distance from itself
        return square(from, mu);
      };
      double q[MC / 2];
#pragma unroll
      for (int m = 0; m < MC / 2; ++m) {
        const double lower = dist2(m), upper = dist2(m + MC / 2);
        q[m] = sdlane::halving_add<32>(lower, upper);
        __builtin_amdgcn_sched_barrier(0);
      }
      return total(q, []() {});
    };
    auto gradient = [&](double (&g)[4]) {
      const double tot = distances(cur, -1);
      const double logit = my_m < M ? my_logw - 0.5 * tot * inv_s2 : -INFINITY;
      double mx;
      const double r_mine = softmax(logit, mx);
      double bar[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int m = 0; m < MC; ++m) {
        const double r = readlane_f64(r_mine, 4 * m);
        if (r < 1e-25 || m >= M) continue;
        const float4 mu = mean_at(m);
        bar[0] = fma(r, static_cast<double>(mu.x), bar[0]);
        bar[1] = fma(r, static_cast<double>(mu.y), bar[1]);
        bar[2] = fma(r, static_cast<double>(mu.z), bar[2]);
        bar[3] = fma(r, static_cast<double>(mu.w), bar[3]);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) g[e] = (cur[e] - bar[e]) * inv_s2;
      // is the largest logit alone, and how far does that carry?
      const unsigned long long at_max = __ballot(logit == mx && my_m < M);
      const int top = at_max ? __builtin_ctzll(at_max) >> 2 : -1;
      const bool other = my_m < M && my_m != top;
      const double gap = mx - logit - kSoleGap;
      if (top < 0 || __ballot(other && !(gap > 0.0)) != 0ull) return;      // the same in every wavefront
      sole.top = top;
      mt = mean_at(top);
      const double from[4] = {mt.x, mt.y, mt.z, mt.w};
      const double d2 = distances(from, top);              // |mu_top|^2 in its own place
      per_nat = 1.f / (static_cast<float>(inv_s2) * (kUp * static_cast<float>(sqrt(d2))));
      norm_top = kUp * static_cast<float>(sqrt(readlane_f64(d2, 4 * top)));
      const double odds = 0.5 * d2 * inv_s2 + readlane_f64(my_logw, 4 * top) - my_logw - kSoleGap;
      sole.radius = kDown * least_of_others(static_cast<float>(odds) * per_nat, other);
      sole.slack = kDown * least_of_others(static_cast<float>(gap) * per_nat, other);
    };
    draw(n + j + 1, z);
    while (Kt > 0) {                           // with a sole component a position has one barrier
      uniforms(n + j + 1);
      double g[4], dl[4];
      // With `top` alone, or alone at the last state, the gradient is that of one component; in the second case fp32 distances
      // travel with the sums and confirm it.
      const bool look = sole.top < 0, confirm = !look && !sole.holds();
      if (look) {
        gradient(g);
      } else {
        g[0] = (cur[0] - static_cast<double>(mt.x)) * inv_s2;
        g[1] = (cur[1] - static_cast<double>(mt.y)) * inv_s2;
        g[2] = (cur[2] - static_cast<double>(mt.z)) * inv_s2;
        g[3] = (cur[3] - static_cast<double>(mt.w)) * inv_s2;
      }
      const double both = products(g, dl);
      float zz = 0.f, gg = 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        zz = fmaf(z[e], z[e], zz);
        gg = fmaf(static_cast<float>(g[e]), static_cast<float>(g[e]), gg);
      }
      const float norms = half_wave_sum(halving_add_f32<32>(zz, gg));
      const int at = sbuf;
      if ((lane & 31) == 0) {                  // last read two rounds ago
        sh_s[at][lane >> 5][wave] = both;
        sh_n[at][lane >> 5][wave] = norms;
      }
      if (confirm) {
        const float x0 = static_cast<float>(cur[0]), x1 = static_cast<float>(cur[1]);
        const float x2 = static_cast<float>(cur[2]), x3 = static_cast<float>(cur[3]);
        float q[MC];
#pragma unroll
        for (int m = 0; m < MC; ++m) {
          q[m] = 0.f;
          if (m >= M) continue;
          const float4 mu = mean_at(m);
          const float d0 = x0 - mu.x, d1 = x1 - mu.y, d2 = x2 - mu.z, d3 = x3 - mu.w;
          q[m] = fmaf(d3, d3, fmaf(d2, d2, fmaf(d1, d1, d0 * d0)));
        }
        const float part = reduce16_transposed_f32(q);
        if ((lane & 3) == 0) sh_near[at][wave][my_m] = part;
      }
      float z_next[4];
      draw(n + j + 2, z_next);                 // the next position's noise, while the sums settle
      __syncthreads();
      sbuf ^= 1;
      const float n_half = row_sum(sh_n[at][lane >> 5][lane & 15]);
      zz = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(n_half), 0));
      gg = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(n_half), 32));
      if (confirm) {
        float dm = 0.f;
#pragma unroll
        for (int w = 0; w < NW; w += 4) dm += sh_near[at][w + (lane & 3)][my_m];
        dm += __int_as_float(sdlane::lane_xor<1>(__float_as_int(dm)));
        dm += __int_as_float(sdlane::lane_xor<2>(__float_as_int(dm)));
        // error of an fp32 squared distance D: the sum's roundings (30 of 2^-24 D at most) and those of x (2^-24 |x| each way)
        const float is2 = static_cast<float>(inv_s2), dt = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(dm), 4 * sole.top));
        const float rd = __builtin_amdgcn_sqrtf(dm), rt = __builtin_amdgcn_sqrtf(dt);
        const float err = 1e-5f * (dm + dt) + 1e-6f * (norm_top + rt) * (rd + rt);
        const float gap = is2 * (0.5f * (dm - dt) - err) + static_cast<float>(readlane_f64(my_logw, 4 * sole.top) - my_logw - kSoleGap);
        const bool other = my_m < M && my_m != sole.top;
        if (__ballot(other && !(gap > 0.f)) != 0ull) break;                // not so (or not certain): this position the long way
        sole.slack = kDown * least_of_others(gap * per_nat, other);
      }
      const bool first = j == 0;
      const bool reject = decide(at, g, dl);
#pragma unroll
      for (int e = 0; e < 4; ++e) z[e] = z_next[e];
      const float gn = kUp * __builtin_amdgcn_sqrtf(gg);
      if (first) gn0 = gn;
      if (sole.holds()) sole.at_distance(gn * kUp * static_cast<float>(1.0 / inv_s2));
      sole.moved(kUp * (static_cast<float>(gamma) * (reject ? gn : gn0) + static_cast<float>(sq2g) * __builtin_amdgcn_sqrtf(zz)));
      if (reject || j >= Kt) {
        end_window(reject);
        sole.window_ended(6.1e-8f * (norm_top + sole.rho));                // half an fp32 unit of the state's length
      }
      if (sole.top < 0) break;                 // no component is alone
    }
  }

  if (RUN) {
    if (t == 0) {
      if (acc_win == 0) acc_win = 1;           // handed over at T: one window, of no positions
      if (p.counters) {
        atomicAdd(&p.counters[0], acc_adv);
        atomicAdd(&p.counters[1], acc_win);
        atomicAdd(&p.counters[2], acc_rej);
        atomicAdd(&p.counters[4], acc_kt);
      }
      atomicMax(&p.queue[1], static_cast<int32_t>(acc_win));
    }
  } else if (t == 0) {
    p.adv[b] = jdone;
    if (p.rej) p.rej[b] = rejected ? 1 : 0;
    for (int q = jdone; q < p.K; ++q) {        // positions not reached report 0
      if (p.logratio) p.logratio[static_cast<int64_t>(b) * p.K + q] = 0.f;
      if (p.logu) p.logu[static_cast<int64_t>(b) * p.K + q] = 0.f;
    }
  }
  const int64_t row = RUN ? id : b;            // sd_advance leaves a finished chain's state at its id
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (own[e]) p.x_out[row * d + i0 + e] = static_cast<float>(cur[e]);
}

// WHOLE: d is a multiple of 4, so a group of four coordinates is inside d or outside it as a whole (one mask
// per group instead of four).
template <int CPT, bool WHOLE, bool RUN>
__global__ __launch_bounds__(64 * wave_chains(CPT), wave_chains(CPT) / 4) void langevin_window_wave_kernel(LangevinArgs p, int workers) {
  constexpr int kWaveChains = wave_chains(CPT);
  // [kWaveM][256 CPT] as fp64 (rows beyond M and the pad are 0): converted once here instead of once per use --
  // the logit pass is one FMA per table element, and a conversion beside each would be a fifth of all
  // vector instructions of the kernel.  16 x 1024 doubles = 128 KiB: one workgroup of 8 wavefronts per CU.
  extern __shared__ __align__(16) double sh_mu[];
  __shared__ double sh_hn[kWaveM];                         // |mu_m|^2 / 2
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int d = p.d, M = p.M;
  // Rows are read as whole float4s through this view, indexed in units of 16 bytes: with the row stride a
  // run-time number of floats the compiler cannot see that a row starts 16-byte aligned and splits every
  // 128-bit LDS read into 32-bit pairs, which are slower and collide on the banks.
  // Row layout: a row has kRow = 256 * CPT doubles; the four coordinates 4 g .. 4 g + 3 of group g = lane + 64 c
  // sit as two halves, (e = 0, 1) at c * 256 + 2 * lane and (e = 2, 3) at c * 256 + 128 + 2 * lane, so that each
  // of the two 128-bit reads of a group is contiguous over the lanes (conflict-free, and the row stride is a
  // compile-time multiple of 16 bytes).
  constexpr int kRow = 256 * CPT;
  const double2* sh_mu2 = reinterpret_cast<const double2*>(sh_mu);

  for (int idx = t; idx < kWaveM * kRow; idx += 64 * kWaveChains) {
    const int m = idx / kRow, i = idx % kRow;            // i: coordinate
    const int c = i >> 8, ln = (i & 255) >> 2, e = i & 3;
    const int pos = c * 256 + (e < 2 ? 2 * ln + e : 128 + 2 * ln + (e - 2));
    sh_mu[m * kRow + pos] = (m < M && i < d) ? static_cast<double>(p.means[static_cast<int64_t>(m) * d + i]) : 0.0;
  }
  __syncthreads();
  if (wave == 0) {                                         // half squared norms, fp64
    double part[16];
#pragma unroll
    for (int m = 0; m < kWaveM; ++m) {
      double acc = 0.0;
      for (int i = lane; i < kRow; i += 64) {
        const double v = sh_mu[m * kRow + i];
        acc = fma(v, v, acc);
      }
      part[m] = acc;
    }
    const double tot = reduce16_transposed(part, lane);
    if ((lane & 3) == 0) sh_hn[lane >> 2] = 0.5 * tot;
  }
  __syncthreads();                                         // last workgroup-wide barrier
  if (wave >= workers) return;                             // few chains: spread over the CUs, the rest only staged the table

  const int Bact = p.active ? min(p.B, max(0, *p.active)) : p.B;
  const double inv_s2 = p.inv_s2, sq2g = sqrt(2.0 * p.gamma);
  const double per_s2 = p.gamma * inv_s2, to_delta = sqrt(0.5 * p.gamma) * inv_s2;       // Delta = to_delta (s^2 grad - the frozen one)
  const int my_m = lane >> 2;                              // component this lane holds after a reduction
  const double my_logw = my_m < M ? static_cast<double>(p.logw[my_m]) : 0.0;
  const double my_hn = sh_hn[my_m];

  // The workgroup keeps its copy of the means for the whole launch (the table is staged once per resident
  // workgroup, not once per four chains) and its wavefronts, independent from here on, take chains one at a
  // time from a counter: a chain's window ends at its first rejection, so the work per chain varies by an
  // order of magnitude and a fixed split would leave most of the chip waiting for the unluckiest wavefront.
  unsigned long long acc_adv = 0, acc_win = 0, acc_rej = 0, acc_kt = 0;   // run mode: this wavefront's share of the counters
  for (;;) {
  int ticket = 0;
  if (lane == 0) ticket = atomicAdd(&p.queue[0], 1);
  const int b = __builtin_amdgcn_readfirstlane(ticket);
  if (b >= Bact) break;
  int n = __builtin_amdgcn_readfirstlane(p.n[b]);
  const int64_t id = p.id[b];

  bool own[CPT][4];
  double cur[CPT][4];
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    const int i0 = 4 * (lane + 64 * c);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      own[c][e] = c < CPT - 1 || (WHOLE ? i0 < d : i0 + e < d);    // CPT is the smallest that holds d
      cur[c][e] = own[c][e] ? static_cast<double>(p.x[static_cast<int64_t>(b) * d + i0 + e]) : 0.0;
    }
  }

  Sole sole;
  float per_nat = 0.f, norm_top = 0.f;                     // s^2 / |mu_top - mu_{my_m}|, at most; |mu_top|
  float gn = 0.f, last = 0.f;                              // upper bound of |s^2 grad| at hand; the last step's length

  auto norm_of = [&](const double g[CPT][4]) {
    double q = 0.0;
#pragma unroll
    for (int c = 0; c < CPT; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) q = fma(g[c][e], g[c][e], q);
    return kUp * __builtin_amdgcn_sqrtf(wave_sum_f32(static_cast<float>(q)));
  };

  // After the logits of `cur`: is the largest one alone, and how far does that carry?
  auto look_for_sole = [&](double logit, double mx) {
    const unsigned long long at_max = __ballot(logit == mx && my_m < M);
    const int top = at_max ? __builtin_ctzll(at_max) >> 2 : -1;
    const bool other = my_m < M && my_m != top;
    const double gap = mx - logit - kSoleGap;
    sole.slack = -1.f;
    if (top < 0 || __ballot(other && !(gap > 0.0)) != 0ull) return;
    if (top != sole.top) {
      sole.top = top;
      double part[16];
#pragma unroll
      for (int m = 0; m < kWaveM; ++m) part[m] = 0.0;
#pragma unroll 1
      for (int c = 0; c < 2 * CPT; ++c) {
        const double2 a = sh_mu2[top * (kRow / 2) + 64 * c + lane];
#pragma unroll
        for (int m = 0; m < kWaveM; ++m) {
          const double2 v = sh_mu2[m * (kRow / 2) + 64 * c + lane];
          part[m] = fma(a.x - v.x, a.x - v.x, part[m]);
          part[m] = fma(a.y - v.y, a.y - v.y, part[m]);
        }
      }
      const double d2 = reduce16_transposed(part, lane);
      per_nat = 1.f / (static_cast<float>(inv_s2) * (kUp * static_cast<float>(sqrt(d2))));
      norm_top = kUp * static_cast<float>(sqrt(2.0 * sh_hn[top]));
      const double odds = 0.5 * d2 * inv_s2 + readlane_f64(my_logw, 4 * top) - my_logw - kSoleGap;
      sole.radius = kDown * least_of_others(static_cast<float>(odds) * per_nat, other);
    }
    sole.slack = kDown * least_of_others(static_cast<float>(gap) * per_nat, other);
  };

  // s^2 grad E at `cur` for my coordinates: the state's distance from the weighted mean
  auto gradient = [&](double g[CPT][4]) {
    if (RUN && sole.holds()) {
      const int top = __builtin_amdgcn_readfirstlane(sole.top);
#pragma unroll
      for (int c = 0; c < CPT; ++c) {
        const double2 lo = sh_mu2[top * (kRow / 2) + c * 128 + lane], hi = sh_mu2[top * (kRow / 2) + c * 128 + 64 + lane];
        g[c][0] = cur[c][0] - lo.x;
        g[c][1] = cur[c][1] - lo.y;
        g[c][2] = cur[c][2] - hi.x;
        g[c][3] = cur[c][3] - hi.y;
      }
      if (__builtin_amdgcn_readfirstlane(sole.slack < 2.5f * last ? 1 : 0))      // about to run out: where in the ball is it?
        sole.at_distance(norm_of(g));
      gn = sole.rho;
      return;
    }
    int at = lane;                                         // opaque: the table's reads must not leave the walk's loop
    asm volatile("" : "+v"(at));
    double dot[16];
#pragma unroll
    for (int m = 0; m < kWaveM; ++m) dot[m] = 0.0;
#pragma unroll
    for (int c = 0; c < CPT; ++c) {                        // 16 independent accumulation chains; rows are padded with zeros
#pragma unroll
      for (int m = 0; m < kWaveM; ++m) {
        const double2 lo = sh_mu2[m * (kRow / 2) + c * 128 + at], hi = sh_mu2[m * (kRow / 2) + c * 128 + 64 + at];
        dot[m] = fma(cur[c][0], lo.x, dot[m]);
        dot[m] = fma(cur[c][1], lo.y, dot[m]);
        dot[m] = fma(cur[c][2], hi.x, dot[m]);
        dot[m] = fma(cur[c][3], hi.y, dot[m]);
        if (m % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // eight reads in flight: more would not fit the registers
      }
    }
    const double tot = reduce16_transposed(dot, lane);     // x . mu_{my_m}
    double logit = my_m < M ? my_logw + (tot - my_hn) * inv_s2 : -INFINITY;
    double mx = logit;
#pragma unroll
    for (int s = 4; s <= 32; s <<= 1) mx = fmax(mx, dpp_xor(mx, s));
    if (RUN) look_for_sole(logit, mx);
    const double ex = my_m < M ? exp(logit - mx) : 0.0;
    double sum = ex;
#pragma unroll
    for (int s = 4; s <= 32; s <<= 1) sum += dpp_xor(sum, s);
    const double r_mine = ex / sum;
    double bar[CPT][4];
#pragma unroll
    for (int c = 0; c < CPT; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) bar[c][e] = 0.0;
#pragma unroll
    for (int m = 0; m < kWaveM; ++m) {
      const double r = readlane_f64(r_mine, 4 * m);        // uniform: lives in scalar registers
      // a component whose responsibility is below 1e-25 moves no coordinate of the weighted mean by more
      // than 1e-25 |mu|, far below the last bit of anything downstream: its pass over the means is skipped
      // (uniform branch).  Well-separated mixtures leave one or two components per state.
      if (r < 1e-25) continue;
#pragma unroll
      for (int c = 0; c < CPT; ++c) {
        const double2 lo = sh_mu2[m * (kRow / 2) + c * 128 + at], hi = sh_mu2[m * (kRow / 2) + c * 128 + 64 + at];
        bar[c][0] = fma(r, lo.x, bar[c][0]);
        bar[c][1] = fma(r, lo.y, bar[c][1]);
        bar[c][2] = fma(r, hi.x, bar[c][2]);
        bar[c][3] = fma(r, hi.y, bar[c][3]);
      }
    }
#pragma unroll
    for (int c = 0; c < CPT; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) g[c][e] = cur[c][e] - bar[c][e];
    if (RUN) {
      gn = norm_of(g);
      if (sole.holds()) sole.at_distance(gn);
    }
  };

  // One pass of the loop is one position of a window: the gradient at the state (at a window's first position the frozen
  // one, and the position is accepted: Delta = 0), noise, accept test, new state.
  int Kt = max(0, min(p.K, p.T - n)), j = 0, jdone = 0, windows = 0;
  bool rejected = false;
  double g0[CPT][4];
  float gn0 = 0.f;
  // log u of 64 steps, lane l holding step lu_base + l: they are keyed by the step alone, so a batch outlives its window
  int lu_base = 0;
  double lu_batch = 0.0;
  bool lu_have = false;
  while (Kt > 0) {                                         // Kt is uniform over the wavefront; every window advances the chain
    double dl[CPT][4];                                     // s^2 grad at the draft, then its difference from the frozen one
    gradient(dl);
    const int k1 = n + j + 1;                              // step this position produces
    if (!lu_have || k1 - lu_base >= 64) {
      lu_base = k1;
      lu_have = true;
      lu_batch = sdrng::log_uniform(p.seed, id, static_cast<uint32_t>(k1 + lane));
    }
    // the noise is drawn after the gradient, which is the register-hungry part
    // Coordinates past d (the tail of the last group) get no noise: their state starts at 0 and the means table
    // is 0 there, so state, gradients and Delta stay exactly 0 and need no masking anywhere else.
    float z[CPT][4], zn = 0.f;                             // zn: |z|, which the reflection keeps
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      sdrng::normal4(p.seed, id, static_cast<uint32_t>(k1), sdrng::kStreamNoise, static_cast<uint32_t>(lane + 64 * c), z[c]);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        z[c][e] = own[c][e] ? z[c][e] : 0.f;
        if (RUN) zn = fmaf(z[c][e], z[c][e], zn);
      }
    }
    if (RUN) zn = __builtin_amdgcn_sqrtf(wave_sum_f32(zn));
    const double lu = readlane_f64(lu_batch, k1 - lu_base);
    double lr = 0.0, twice = 0.0;
    bool reject = false;
    if (j == 0) {
      gn0 = gn;
#pragma unroll
      for (int c = 0; c < CPT; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) g0[c][e] = dl[c][e];
    } else {
      double a1 = 0.0, a2 = 0.0;
#pragma unroll
      for (int c = 0; c < CPT; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          dl[c][e] -= g0[c][e];
          a1 = fma(static_cast<double>(z[c][e]), dl[c][e], a1);
          a2 = fma(dl[c][e], dl[c][e], a2);
        }
      // both sums in one butterfly: the lower half of the wavefront carries the first, the upper half the second
      const double both = half_wave_sum(sdlane::halving_add<32>(a1, a2));
      const double S1 = to_delta * readlane_f64(both, 0), S2 = to_delta * to_delta * readlane_f64(both, 32);
      lr = (-S1 - 0.5 * S2) * p.inv_tau;
      reject = !(S2 == 0.0 || (lr == lr && lu <= fmin(0.0, lr)));   // a log-ratio that is not a number rejects
      reject = __builtin_amdgcn_readfirstlane(reject ? 1 : 0) != 0;   // all lanes hold the same totals
      twice = S2 > 0.0 ? 2.0 * to_delta * (S1 / S2) : 0.0;
    }
    if (!RUN && lane == 0) {
      if (p.logratio) p.logratio[static_cast<int64_t>(b) * p.K + j] = static_cast<float>(lr);
      if (p.logu) p.logu[static_cast<int64_t>(b) * p.K + j] = static_cast<float>(lu);
    }
    if (RUN) {
      last = kUp * (static_cast<float>(per_s2) * (reject ? gn : gn0) + static_cast<float>(sq2g) * zn);
      sole.moved(last);
    }
    if (reject) {
#pragma unroll
      for (int c = 0; c < CPT; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          cur[c][e] = cur[c][e] - per_s2 * (g0[c][e] + dl[c][e]) + sq2g * (static_cast<double>(z[c][e]) - twice * dl[c][e]);
    } else {
#pragma unroll
      for (int c = 0; c < CPT; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          cur[c][e] = cur[c][e] - per_s2 * g0[c][e] + sq2g * static_cast<double>(z[c][e]);
    }
    ++j;
    if (!reject && j < Kt) continue;

    // end of the window
    jdone = j;
    rejected = reject;
    if (!RUN) break;
    // what sd_advance and the next sd_langevin_window would do: the step count moves on and the state passes
    // through fp32, so a run is bit for bit the window entry point applied again and again
    n += j;
    j = 0;
    ++windows;
    acc_adv += jdone; acc_win += 1; acc_rej += reject ? 1 : 0; acc_kt += Kt;
#pragma unroll
    for (int c = 0; c < CPT; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) cur[c][e] = static_cast<double>(static_cast<float>(cur[c][e]));
    sole.window_ended(6.1e-8f * (norm_top + sole.rho));           // half an fp32 unit of the state's length
    Kt = windows < p.max_windows ? max(0, min(p.K, p.T - n)) : 0;
  }

  if (lane == 0) {
    if (RUN) {
      p.n_out[b] = n;
    } else {
      p.adv[b] = jdone;
      if (p.rej) p.rej[b] = rejected ? 1 : 0;
      for (int q = jdone; q < p.K; ++q) {                  // positions not reached report 0
        if (p.logratio) p.logratio[static_cast<int64_t>(b) * p.K + q] = 0.f;
        if (p.logu) p.logu[static_cast<int64_t>(b) * p.K + q] = 0.f;
      }
    }
  }
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    const int i0 = 4 * (lane + 64 * c);
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (own[c][e]) p.x_out[static_cast<int64_t>(b) * d + i0 + e] = static_cast<float>(cur[c][e]);
  }
  }                                                        // next chain of this wavefront
  if (RUN && p.counters && lane == 0 && acc_win) {
    atomicAdd(&p.counters[0], acc_adv);
    atomicAdd(&p.counters[1], acc_win);
    atomicAdd(&p.counters[2], acc_rej);
    atomicAdd(&p.counters[4], acc_kt);
  }
}

// ---------------------------------------------------------------------------------------------
// Short chains (d <= 128): G lanes per chain, one group of four coordinates each, 64 / G chains per wavefront.
// The wavefront kernel above leaves all but ceil(d / 4) lanes of its 64 idle here and walks one chain at a time.  A step
// of the loop is one position of every chain of the wavefront: its gradient (at a window's first position the frozen
// one), accept test and new state, so chains stay in step whatever their windows; what a chain computes does not depend
// on its neighbours.  The 16 logits are summed transposed over the chain's lanes (16 / G of them per lane), the
// weights come back through a slice of LDS.  Bound by vector instructions at many chains, by one step's latency at few.
// Whole runs, us (before: a wavefront per chain):
//   16384 chains: d = 5, M = 4, 150 steps 401 (3164)   d = 16, M = 16, 100 steps 309 (2421)   d = 60, M = 10, 100 steps
//   616 (2139)   d = 120, M = 16, 100 steps 1119 (2101)
//   2000 chains d = 37, M = 16, 150 steps 344 (520)   100 chains d = 100, M = 8, 150 steps 324 (451)   3 chains d = 3,
//   M = 16, 300 steps 594 (755)
// With the means in LDS, as the wavefront kernel has them, 375 / 354 / 615 / 1142 / 437 / 324 / 940.
// ---------------------------------------------------------------------------------------------
template <int MASK, int TO>
__device__ __forceinline__ double group_max(double v) {
  v = fmax(v, sdlane::lane_xor<MASK>(v));
  if constexpr (2 * MASK < TO) return group_max<2 * MASK, TO>(v);
  else return v;
}
template <int MASK, int TO>
__device__ __forceinline__ double group_add(double v) {     // over the lanes that differ in the bits MASK .. TO / 2
  v += sdlane::lane_xor<MASK>(v);
  if constexpr (2 * MASK < TO) return group_add<2 * MASK, TO>(v);
  else return v;
}
// a[0 .. N) summed over the lanes of a group, transposed: halves exchanged at MASK, MASK / 2, ...
template <int MASK, int N>
__device__ __forceinline__ void reduce_transposed(double (&a)[16]) {
  if constexpr (N > 1) {
#pragma unroll
    for (int i = 0; i < N / 2; ++i) a[i] = sdlane::halving_add<MASK>(a[i], a[i + N / 2]);
  } else {
    a[0] += sdlane::lane_xor<MASK>(a[0]);
  }
  if constexpr (MASK > 1) reduce_transposed<MASK / 2, (N > 1 ? N / 2 : 1)>(a);
}

template <int G, bool RUN>
__global__ __launch_bounds__(256, 2) void langevin_short_kernel(LangevinArgs p) {
  constexpr int CPWV = 64 / G, NV = G < 16 ? 16 / G : 1, PAIR = G == 32 ? 2 : 1;   // G = 32: two lanes hold a logit
  __shared__ __align__(16) double sh_r[4 * CPWV][18];       // a chain's weights (stride 144 B: spread over the banks)
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, sub = lane / G, gl = lane % G;
  const int d = p.d, M = p.M;
  const int slot = wave * CPWV + sub;
  const int Bact = p.active ? min(p.B, max(0, *p.active)) : p.B;
  const int b_raw = blockIdx.x * (4 * CPWV) + slot;
  const bool valid = b_raw < Bact;
  const int b = valid ? b_raw : 0;
  int n = valid ? p.n[b] : p.T;
  const int64_t id = valid ? p.id[b] : 0;
  const double gamma = p.gamma, inv_s2 = p.inv_s2;
  const double sq2g = sqrt(2.0 * gamma), sqg2 = sqrt(0.5 * gamma), inv_sqg2 = 1.0 / sqg2;
  const int my_m = gl / PAIR * NV;                          // first of the NV components whose logits this lane holds
  double my_logw[NV], my_hn[NV];
  // my four coordinates of every mean (0 beyond M and d), in registers: read twice a step, they would be half of its
  // time out of LDS
  double mu[kWaveM][4], hn[16];
#pragma unroll
  for (int m = 0; m < kWaveM; ++m) {
    hn[m] = 0.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int i = 4 * gl + e;
      mu[m][e] = (m < M && i < d) ? static_cast<double>(p.means[static_cast<int64_t>(m) * d + i]) : 0.0;
      hn[m] = fma(mu[m][e], mu[m][e], hn[m]);
    }
  }
  reduce_transposed<G / 2, 16>(hn);
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    my_logw[i] = my_m + i < M ? static_cast<double>(p.logw[my_m + i]) : 0.0;
    my_hn[i] = 0.5 * hn[i];
  }
  bool own[4];
  double cur[4], g0[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    own[e] = 4 * gl + e < d;
    cur[e] = (valid && own[e]) ? static_cast<double>(p.x[static_cast<int64_t>(b) * d + 4 * gl + e]) : 0.0;
  }
  double* r_slot = sh_r[slot];

  // grad E at `cur`; every lane of the wavefront takes part
  auto gradient = [&](double g[4]) {
    auto dot4 = [&](int m) { return fma(cur[3], mu[m][3], fma(cur[2], mu[m][2], fma(cur[1], mu[m][1], cur[0] * mu[m][0]))); };
    double dot[16];
#pragma unroll
    for (int m = 0; m < kWaveM / 2; ++m) {                  // the first halving step as the products come
      const double lower = dot4(m), upper = M > kWaveM / 2 ? dot4(m + kWaveM / 2) : 0.0;
      dot[m] = sdlane::halving_add<G / 2>(lower, upper);
    }
    if constexpr (G > 2) reduce_transposed<G / 4, 8>(dot);
    double logit[NV], mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      logit[i] = my_m + i < M ? my_logw[i] + (dot[i] - my_hn[i]) * inv_s2 : -INFINITY;
      mx = fmax(mx, logit[i]);
    }
    mx = group_max<PAIR, G>(mx);
    if (gl % PAIR == 0) {
#pragma unroll
      for (int i = 0; i < NV; ++i) r_slot[my_m + i] = my_m + i < M ? exp(logit[i] - mx) : 0.0;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // every lane adds the 16 weights itself, in one order whatever G: with it nothing depends on G (the lanes past a
    // short row add zeros to every other sum), so G can follow the number of chains
    double r[16];
#pragma unroll
    for (int m = 0; m < kWaveM; m += 2) {
      const double2 v = *reinterpret_cast<const double2*>(r_slot + m);
      r[m] = v.x;
      r[m + 1] = v.y;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const double sum = (((r[0] + r[1]) + (r[2] + r[3])) + ((r[4] + r[5]) + (r[6] + r[7]))) +
                       (((r[8] + r[9]) + (r[10] + r[11])) + ((r[12] + r[13]) + (r[14] + r[15])));
    const double inv_sum = 1.0 / sum;
    double bar[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int m = 0; m < kWaveM; ++m) {
      const double rm = r[m] * inv_sum;
      if (__ballot(!(rm < 1e-25)) == 0ull) continue;        // negligible as in the wavefront kernel, for every chain here
      const double w = rm < 1e-25 ? 0.0 : rm;
#pragma unroll
      for (int e = 0; e < 4; ++e) bar[e] = fma(w, mu[m][e], bar[e]);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) g[e] = (cur[e] - bar[e]) * inv_s2;
  };

  int Kt = max(0, min(p.K, p.T - n));
  int j = 0, windows = 0, adv = 0;
  bool active = valid && Kt > 0, rejected = false;
  int lu_base = 0;                                          // first absolute step of the uniforms held in lu_batch
  bool lu_have = false;
  double lu_batch = 0.0;
  unsigned long long acc_adv = 0, acc_win = 0, acc_rej = 0, acc_kt = 0;

  // Ends: a step moves every active chain one position on, a window of Kt positions ends after at most Kt steps and
  // advances n by at least 1, and a chain stops at n = T or after max_windows windows.
  while (__ballot(active) != 0ull) {
    double g[4];
    gradient(g);
    if (active) {                                           // the lanes of a chain agree
      const int k1 = n + j + 1;                             // absolute step this position produces
      float z[4];
      sdrng::normal4(p.seed, id, static_cast<uint32_t>(k1), sdrng::kStreamNoise, static_cast<uint32_t>(gl), z);
      if (!lu_have || k1 - lu_base >= G) {
        lu_base = k1;
        lu_have = true;
        lu_batch = sdrng::log_uniform(p.seed, id, static_cast<uint32_t>(k1 + gl));
      }
      const double lu = __shfl(lu_batch, sub * G + (k1 - lu_base), 64);
      double lr = 0.0, dl[4] = {0.0, 0.0, 0.0, 0.0}, coef = 0.0;
      rejected = false;
      if (j == 0) {
#pragma unroll
        for (int e = 0; e < 4; ++e) g0[e] = g[e];
      } else {
        double a1 = 0.0, a2 = 0.0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          z[e] = own[e] ? z[e] : 0.f;
          dl[e] = sqg2 * (g[e] - g0[e]);                    // 0 past d: state and means are 0 there
          a1 = fma(static_cast<double>(z[e]), dl[e], a1);
          a2 = fma(dl[e], dl[e], a2);
        }
        const double S1 = group_add<1, G>(a1), S2 = group_add<1, G>(a2);
        lr = (-S1 - 0.5 * S2) * p.inv_tau;
        rejected = !(S2 == 0.0 || (lr == lr && lu <= fmin(0.0, lr)));   // a log-ratio that is not a number rejects
        coef = S2 > 0.0 ? S1 / S2 : 0.0;
      }
      if (!RUN && gl == 0) {
        if (p.logratio) p.logratio[static_cast<int64_t>(b) * p.K + j] = static_cast<float>(lr);
        if (p.logu) p.logu[static_cast<int64_t>(b) * p.K + j] = static_cast<float>(lu);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (!own[e]) continue;
        if (rejected)                                       // target gradient = g0 + Delta / sqrt(gamma/2)
          cur[e] = cur[e] - gamma * (g0[e] + dl[e] * inv_sqg2) + sq2g * (static_cast<double>(z[e]) - 2.0 * coef * dl[e]);
        else
          cur[e] = cur[e] - gamma * g0[e] + sq2g * static_cast<double>(z[e]);
      }
      ++j;
      if (rejected || j == Kt) {
        adv = j;
        n += j;
        ++windows;
        if (RUN) {                                          // the state passes through fp32, as between separate calls
          acc_adv += j; acc_win += 1; acc_rej += rejected ? 1 : 0; acc_kt += Kt;
#pragma unroll
          for (int e = 0; e < 4; ++e) cur[e] = static_cast<double>(static_cast<float>(cur[e]));
        }
        j = 0;
        Kt = max(0, min(p.K, p.T - n));
        active = RUN && Kt > 0 && windows < p.max_windows;
      }
    }
  }

  if (RUN && p.counters) {                                  // one atomic per wavefront and counter
    unsigned long long c[4] = {acc_adv, acc_win, acc_rej, acc_kt};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      c[q] = gl == 0 ? c[q] : 0ull;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) c[q] += __shfl_xor(c[q], o, 64);
      if (lane == 0 && c[q]) atomicAdd(&p.counters[q == 3 ? 4 : q], c[q]);
    }
  }
  if (!valid) return;
  if (gl == 0) {
    if (RUN) {
      p.n_out[b] = n;
    } else {
      p.adv[b] = adv;
      if (p.rej) p.rej[b] = rejected ? 1 : 0;
      for (int q = adv; q < p.K; ++q) {                     // positions not reached report 0
        if (p.logratio) p.logratio[static_cast<int64_t>(b) * p.K + q] = 0.f;
        if (p.logu) p.logu[static_cast<int64_t>(b) * p.K + q] = 0.f;
      }
    }
  }
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (own[e]) p.x_out[static_cast<int64_t>(b) * d + 4 * gl + e] = static_cast<float>(cur[e]);
}

template <int G>
void launch_short(const LangevinArgs& p, bool run, hipStream_t st) {
  const unsigned grid = static_cast<unsigned>((p.B + 256 / G - 1) / (256 / G));
  if (run) hipLaunchKernelGGL((langevin_short_kernel<G, true>), dim3(grid), dim3(256), 0, st, p);
  else hipLaunchKernelGGL((langevin_short_kernel<G, false>), dim3(grid), dim3(256), 0, st, p);
}

// The chain dispenser starts every launch at zero: a one-thread kernel ahead of the launch (a kernel, not a
// memset, so that the sequence can be captured in a HIP graph), never a rewind at the end of the previous one --
// a launch that does not run to its end must not leave the next call without chains.
__global__ void reset_queue_kernel(int32_t* queue, int slot) { queue[slot] = 0; }

// run to T: a batch stepped window by window makes as many windows as its longest chain, and ends with none active
__global__ void chains_end_kernel(const int32_t* longest, unsigned long long* counters, int32_t* B_active) {
  if (counters) counters[3] += static_cast<unsigned long long>(*longest);
  *B_active = 0;
}

// The workgroup-per-chain kernel at the thread count of the row length.
constexpr int kWideMeansLds = 148 * 1024;  // of 160 KiB; the sums' buffers take 8

template <int MAXT, bool RUN>
void launch_wide(const LangevinArgs& p, dim3 block, hipStream_t st) {
  const dim3 grid(static_cast<unsigned>(p.B));
  const size_t row = sizeof(float4) * block.x, means = row * p.M;
  if constexpr (RUN) {
    if (MAXT <= 512 || means <= kWideMeansLds) {           // 16 rows of up to 512 threads always fit
      hipLaunchKernelGGL((langevin_window_kernel<MAXT, true, true>), grid, block, means, st, p);
      return;
    }
  }
  if constexpr (!RUN || MAXT > 512)
    hipLaunchKernelGGL((langevin_window_kernel<MAXT, RUN, false>), grid, block, std::min(means, 8 * row), st, p);
}

template <int MAXT>
hipError_t prepare_wide() {
  auto allow = [](const void* kernel) { return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kWideMeansLds); };
  hipError_t e = allow(reinterpret_cast<const void*>(&langevin_window_kernel<MAXT, false, false>));
  if (e == hipSuccess) e = allow(reinterpret_cast<const void*>(&langevin_window_kernel<MAXT, true, true>));
  if constexpr (MAXT > 512)
    if (e == hipSuccess) e = allow(reinterpret_cast<const void*>(&langevin_window_kernel<MAXT, true, false>));
  return e;
}

template <bool RUN>
void launch_wide(const LangevinArgs& p, int groups, hipStream_t st) {
  const dim3 block(static_cast<unsigned>((groups + 63) / 64 * 64));
  if (block.x <= 512) launch_wide<512, RUN>(p, block, st);
  else if (block.x <= 768) launch_wide<768, RUN>(p, block, st);
  else launch_wide<1024, RUN>(p, block, st);
}

// run mode: one launch counts as one entry of the `windows` counter
__global__ void bump_launches_kernel(unsigned long long* counters) { counters[3] += 1; }

template <int CPT, bool WHOLE, bool RUN>
hipError_t prepare_wave() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&langevin_window_wave_kernel<CPT, WHOLE, RUN>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024);
}

// prepare_wave<...>() has run for every instantiation when the context was created (sdi::langevin_prepare);
// `resident` = workgroups the chip holds at once (one per CU), from the same call.
template <int CPT, bool WHOLE, bool RUN>
hipError_t launch_wave(const LangevinArgs& p, int resident, hipStream_t st) {
  const size_t shmem = sizeof(double) * kWaveM * static_cast<size_t>(256 * CPT);
  const int per_cu = (p.B + resident - 1) / resident;
  const int workers = per_cu < wave_chains(CPT) ? per_cu : wave_chains(CPT);
  const int groups = (p.B + workers - 1) / workers;
  const unsigned grid = static_cast<unsigned>(groups < resident ? groups : resident);
  hipLaunchKernelGGL(reset_queue_kernel, dim3(1), dim3(1), 0, st, p.queue, 0);
  hipLaunchKernelGGL((langevin_window_wave_kernel<CPT, WHOLE, RUN>), dim3(grid), dim3(64 * wave_chains(CPT)), shmem, st, p, workers);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// phi^4 lattice energy on an L x L periodic grid (Langevin appendix, table of sampling metrics):
//   E(x) = (beta/2) sum over ordered neighbour pairs (x_i - x_j)^2 + sum_i (x_i^2 - 1)^2,
//   grad E_i = 2 beta (4 x_i - four neighbours) + 4 x_i (x_i^2 - 1).
// G lanes work on one chain (G = power of two >= d/4, one Philox block of four sites per lane),
// 64/G chains share a wavefront and 256/G a workgroup.  The chain's state is mirrored in a
// wavefront-private slice of LDS for the neighbour reads; no workgroup barrier is used, since the
// chains of a workgroup leave their walks at different positions.  A wavefront walks until none
// of its chains is alive; a chain that has rejected or finished is masked.
// ---------------------------------------------------------------------------------------------
struct Phi4Args {
  const float* x;
  const int32_t* n;
  const int64_t* id;
  float* x_out;
  int32_t* adv;
  uint8_t* rej;
  float *logratio, *logu;
  const int32_t* active;
  int B, d, L, K, T;
  uint64_t seed;
  double gamma, beta, inv_tau;
  int max_windows;                 // sd_langevin_run_phi4: windows per chain at most
  int32_t* n_out;                  //   the step each chain reached
  unsigned long long* counters;    //   optional: sum adv, chain-windows, rejections, launches, sum Kt
};

template <int G>
__device__ __forceinline__ double group_sum_f64(double v) {
#pragma unroll
  for (int s = G / 2; s >= 1; s >>= 1) v += dpp_xor(v, s);
  return v;
}

template <int G>
__global__ __launch_bounds__(256) void phi4_window_kernel(Phi4Args p) {
  constexpr int CPWV = 64 / G;                       // chains per wavefront
  extern __shared__ __align__(16) double sh_x[];     // [256 / G][d]
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int sub = lane / G, gl = lane % G;
  const int slot = wave * CPWV + sub;
  const int Bact = p.active ? min(p.B, max(0, *p.active)) : p.B;
  const int b_raw = blockIdx.x * (4 * CPWV) + slot;
  const bool valid = b_raw < Bact;
  const int b = valid ? b_raw : 0;
  const int d = p.d, L = p.L;
  const int n = valid ? p.n[b] : 0;
  const int Kt = valid ? max(0, min(p.K, p.T - n)) : 0;
  const int64_t id = valid ? p.id[b] : 0;
  const double gamma = p.gamma, beta2 = 2.0 * p.beta;
  const double sq2g = sqrt(2.0 * gamma), sqg2 = sqrt(0.5 * gamma), inv_sqg2 = 1.0 / sqg2;
  double* xs = sh_x + static_cast<size_t>(slot) * d;

  bool own[4];
  int nb[4][4];
  double cur[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int s = 4 * gl + e;
    own[e] = s < d;
    const int sc = own[e] ? s : 0;
    const int r = sc / L, c = sc % L;
    nb[e][0] = ((r + L - 1) % L) * L + c;
    nb[e][1] = ((r + 1) % L) * L + c;
    nb[e][2] = r * L + (c + L - 1) % L;
    nb[e][3] = r * L + (c + 1) % L;
    cur[e] = (valid && own[e]) ? static_cast<double>(p.x[static_cast<int64_t>(b) * d + s]) : 0.0;
  }

  // grad E at `cur`: mirror the state in LDS, then read the four neighbours.  Writers and readers
  // are lanes of one wavefront and the two accesses are separate instructions in program order.
  auto gradient = [&](double g[4]) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (own[e]) xs[4 * gl + e] = cur[e];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      double v = 0.0;
      if (own[e]) {
        const double s4 = xs[nb[e][0]] + xs[nb[e][1]] + xs[nb[e][2]] + xs[nb[e][3]];
        v = beta2 * (4.0 * cur[e] - s4) + 4.0 * cur[e] * (cur[e] * cur[e] - 1.0);
      }
      g[e] = v;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();                 // reads done before the next mirror overwrites
  };

  double g0[4];
  gradient(g0);

  int jr = -1;
  double lu_batch = 0.0;                             // log u of position (j - j % G) + gl + 1, drawn G positions at a time
  for (int j = 0; j < p.K; ++j) {
    const bool alive = valid && j < Kt && jr < 0;
    if (__ballot(alive) == 0ull) break;              // uniform over the wavefront
    const uint32_t k1 = static_cast<uint32_t>(n + j + 1);
    float z[4];
    sdrng::normal4(p.seed, id, k1, sdrng::kStreamNoise, static_cast<uint32_t>(gl), z);
    if (j % G == 0) lu_batch = sdrng::log_uniform(p.seed, id, static_cast<uint32_t>(n + j + gl + 1));   // j is uniform
    const double lu = __shfl(lu_batch, sub * G + j % G, 64);
    double lr = 0.0, coef = 0.0;
    bool reject = false;
    double dl[4] = {0.0, 0.0, 0.0, 0.0};
    if (j > 0) {                                     // position 1: the target gradient IS g0
      gradient(dl);                                  // every lane of the wavefront takes part
      double a1 = 0.0, a2 = 0.0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        dl[e] = (own[e] && alive) ? sqg2 * (dl[e] - g0[e]) : 0.0;
        a1 = fma(static_cast<double>(z[e]), dl[e], a1);
        a2 = fma(dl[e], dl[e], a2);
      }
      const double S1 = group_sum_f64<G>(a1), S2 = group_sum_f64<G>(a2);
      lr = (-S1 - 0.5 * S2) * p.inv_tau;
      reject = alive && !(S2 == 0.0 || (lr == lr && lu <= fmin(0.0, lr)));
      coef = S2 > 0.0 ? S1 / S2 : 0.0;
    }
    if (alive && gl == 0) {
      if (p.logratio) p.logratio[static_cast<int64_t>(b) * p.K + j] = static_cast<float>(lr);
      if (p.logu) p.logu[static_cast<int64_t>(b) * p.K + j] = static_cast<float>(lu);
    }
    if (alive) {
      if (reject) {
        jr = j;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (own[e])                                // target gradient = g0 + Delta / sqrt(gamma/2)
            cur[e] = cur[e] - gamma * (g0[e] + dl[e] * inv_sqg2) + sq2g * (static_cast<double>(z[e]) - 2.0 * coef * dl[e]);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (own[e]) cur[e] = cur[e] - gamma * g0[e] + sq2g * static_cast<double>(z[e]);
      }
    }
  }

  if (!valid) return;
  const int jdone = jr >= 0 ? jr + 1 : Kt;
  if (gl == 0) {
    p.adv[b] = jdone;
    if (p.rej) p.rej[b] = jr >= 0 ? 1 : 0;
    for (int j = jdone; j < p.K; ++j) {
      if (p.logratio) p.logratio[static_cast<int64_t>(b) * p.K + j] = 0.f;
      if (p.logu) p.logu[static_cast<int64_t>(b) * p.K + j] = 0.f;
    }
  }
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (own[e]) p.x_out[static_cast<int64_t>(b) * d + 4 * gl + e] = static_cast<float>(cur[e]);
}

// Windows back to back for the chains of a wavefront (sd_langevin_run_phi4).  A chain's walk is a sequence of
// steps, each of which costs one gradient at its current state and one draw of noise, whether the step opens a
// window (the gradient is the frozen one and the position is accepted by construction) or tests a draft (the
// gradient gives Delta).  So the 64 / G chains of a wavefront stay in lockstep step by step although their
// windows start and end at different times, and no lane idles before its chain has reached T.
// Noise and uniforms are keyed by chain and absolute step, so the values are those of the window kernel;
// the uniforms are drawn G steps at a time and the batch carries over from one window to the next.  At the end
// of a window the state passes through fp32, as it does between sd_langevin_window_phi4 and the next call:
// the result is bit for bit that of window + advance repeated.
template <int G>
__global__ __launch_bounds__(256) void phi4_run_kernel(Phi4Args p) {
  constexpr int CPWV = 64 / G;
  extern __shared__ __align__(16) double sh_x[];     // [256 / G][d]
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int sub = lane / G, gl = lane % G;
  const int slot = wave * CPWV + sub;
  const int Bact = p.active ? min(p.B, max(0, *p.active)) : p.B;
  const int b_raw = blockIdx.x * (4 * CPWV) + slot;
  const bool valid = b_raw < Bact;
  const int b = valid ? b_raw : 0;
  const int d = p.d, L = p.L;
  int n = valid ? p.n[b] : p.T;
  const int64_t id = valid ? p.id[b] : 0;
  const double gamma = p.gamma, beta2 = 2.0 * p.beta;
  const double sq2g = sqrt(2.0 * gamma), sqg2 = sqrt(0.5 * gamma), inv_sqg2 = 1.0 / sqg2;
  double* xs = sh_x + static_cast<size_t>(slot) * d;

  bool own[4];
  int nb[4][4];
  double cur[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int s = 4 * gl + e;
    own[e] = s < d;
    const int sc = own[e] ? s : 0;
    const int r = sc / L, c = sc % L;
    nb[e][0] = ((r + L - 1) % L) * L + c;
    nb[e][1] = ((r + 1) % L) * L + c;
    nb[e][2] = r * L + (c + L - 1) % L;
    nb[e][3] = r * L + (c + 1) % L;
    cur[e] = (valid && own[e]) ? static_cast<double>(p.x[static_cast<int64_t>(b) * d + s]) : 0.0;
  }

  auto gradient = [&](double g[4]) {               // as in phi4_window_kernel: every lane of the wavefront takes part
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (own[e]) xs[4 * gl + e] = cur[e];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      double v = 0.0;
      if (own[e]) {
        const double s4 = xs[nb[e][0]] + xs[nb[e][1]] + xs[nb[e][2]] + xs[nb[e][3]];
        v = beta2 * (4.0 * cur[e] - s4) + 4.0 * cur[e] * (cur[e] * cur[e] - 1.0);
      }
      g[e] = v;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };

  int Kt = max(0, min(p.K, p.T - n));
  int j = 0, windows = 0;
  bool active = valid && Kt > 0;
  double g0[4] = {0.0, 0.0, 0.0, 0.0};
  int lu_base = 0;                                   // first absolute step of the batch of uniforms held in lu_batch
  bool lu_have = false;
  double lu_batch = 0.0;
  unsigned long long acc_adv = 0, acc_win = 0, acc_rej = 0, acc_kt = 0;

  // Ends: a step moves every active chain forward by one position, a window of Kt positions ends after at
  // most Kt steps and advances n by at least 1, and a chain stops at n = T or after max_windows windows.
  while (__ballot(active) != 0ull) {
    double g[4];
    gradient(g);
    if (active) {                                    // the lanes of a chain agree
      const int k1 = n + j + 1;                      // absolute step this position produces
      float z[4];
      sdrng::normal4(p.seed, id, static_cast<uint32_t>(k1), sdrng::kStreamNoise, static_cast<uint32_t>(gl), z);
      bool ended = false, rejected = false;
      if (j == 0) {                                  // window start: this gradient is the frozen one
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          g0[e] = g[e];
          if (own[e]) cur[e] = cur[e] - gamma * g0[e] + sq2g * static_cast<double>(z[e]);
        }
      } else {
        if (!lu_have || k1 - lu_base >= G) {
          lu_base = k1;
          lu_have = true;
          lu_batch = sdrng::log_uniform(p.seed, id, static_cast<uint32_t>(k1 + gl));
        }
        const double lu = __shfl(lu_batch, sub * G + (k1 - lu_base), 64);
        double dl[4], a1 = 0.0, a2 = 0.0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          dl[e] = own[e] ? sqg2 * (g[e] - g0[e]) : 0.0;
          a1 = fma(static_cast<double>(z[e]), dl[e], a1);
          a2 = fma(dl[e], dl[e], a2);
        }
        const double S1 = group_sum_f64<G>(a1), S2 = group_sum_f64<G>(a2);
        const double lr = (-S1 - 0.5 * S2) * p.inv_tau;
        rejected = !(S2 == 0.0 || (lr == lr && lu <= fmin(0.0, lr)));
        const double coef = S2 > 0.0 ? S1 / S2 : 0.0;
        if (rejected) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (own[e])
              cur[e] = cur[e] - gamma * (g0[e] + dl[e] * inv_sqg2) + sq2g * (static_cast<double>(z[e]) - 2.0 * coef * dl[e]);
          ended = true;
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (own[e]) cur[e] = cur[e] - gamma * g0[e] + sq2g * static_cast<double>(z[e]);
        }
      }
      ++j;
      if (j == Kt) ended = true;
      if (ended) {
        n += j;
        acc_adv += j; acc_win += 1; acc_rej += rejected ? 1 : 0; acc_kt += Kt;
#pragma unroll
        for (int e = 0; e < 4; ++e) cur[e] = static_cast<double>(static_cast<float>(cur[e]));
        ++windows;
        j = 0;
        Kt = max(0, min(p.K, p.T - n));
        active = Kt > 0 && windows < p.max_windows;
      }
    }
  }

  if (!valid) return;
  if (gl == 0) {
    p.n_out[b] = n;
    if (p.counters && acc_win) {
      atomicAdd(&p.counters[0], acc_adv);
      atomicAdd(&p.counters[1], acc_win);
      atomicAdd(&p.counters[2], acc_rej);
      atomicAdd(&p.counters[4], acc_kt);
    }
  }
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (own[e]) p.x_out[static_cast<int64_t>(b) * d + 4 * gl + e] = static_cast<float>(cur[e]);
}

template <int G>
hipError_t launch_phi4_run(const Phi4Args& p, hipStream_t st) {
  constexpr int chains_per_wg = 256 / G;
  const size_t shmem = sizeof(double) * static_cast<size_t>(chains_per_wg) * p.d;
  const unsigned grid = static_cast<unsigned>((p.B + chains_per_wg - 1) / chains_per_wg);
  hipLaunchKernelGGL(phi4_run_kernel<G>, dim3(grid), dim3(256), shmem, st, p);
  return hipGetLastError();
}

template <int G>
hipError_t launch_phi4(const Phi4Args& p, hipStream_t st) {
  constexpr int chains_per_wg = 256 / G;
  const size_t shmem = sizeof(double) * static_cast<size_t>(chains_per_wg) * p.d;
  const unsigned grid = static_cast<unsigned>((p.B + chains_per_wg - 1) / chains_per_wg);
  hipLaunchKernelGGL(phi4_window_kernel<G>, dim3(grid), dim3(256), shmem, st, p);
  return hipGetLastError();
}

}  // namespace

// One-time set-up on the current device, called by sd_create: dynamic-LDS limits of every instantiation of the
// wavefront kernel (so that no launch path carries set-up calls or "already done" flags) and the CU count.
hipError_t sdi::langevin_prepare(int* cus) {
  hipError_t e = hipSuccess;
#define SD_PREP(c_) \
  if (e == hipSuccess) e = prepare_wave<c_, false, false>(); \
  if (e == hipSuccess) e = prepare_wave<c_, false, true>();  \
  if (e == hipSuccess) e = prepare_wave<c_, true, false>();  \
  if (e == hipSuccess) e = prepare_wave<c_, true, true>();
  SD_PREP(1) SD_PREP(2) SD_PREP(3) SD_PREP(4)
#undef SD_PREP
  if (e == hipSuccess) e = prepare_wide<512>();
  if (e == hipSuccess) e = prepare_wide<768>();
  if (e == hipSuccess) e = prepare_wide<1024>();
  int dev = 0, n = 0;
  if (e == hipSuccess) e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev);
  *cus = n > 0 ? n : 256;
  return e;
}

namespace {

// Shared by sd_langevin_window (max_windows = 1) and sd_langevin_run.
int langevin_launch(const char* who, sd_ctx* ctx, int32_t B, const float* x, const int32_t* n,
                    const int64_t* chain_id, const float* means, const float* logw, float comp_std, int32_t M,
                    float gamma, float* x_out, int32_t* adv, uint8_t* rejected, float* logratio, float* logu,
                    int32_t max_windows, int32_t* n_out, int64_t* counters, void* stream) {
  if (M > 16)
    return sdi::fail(ctx->err, SD_ERR_UNSUPPORTED, "%s: at most 16 mixture components (M=%d)", who, M);
  const int groups = (ctx->d + 3) / 4;
  if (groups > kMaxGroups)
    return sdi::fail(ctx->err, SD_ERR_UNSUPPORTED, "%s: d=%d exceeds the register-resident limit of %d", who,
                     ctx->d, 4 * kMaxGroups);
  LangevinArgs p;
  p.x = x; p.n = n; p.id = chain_id; p.means = means; p.logw = logw; p.x_out = x_out; p.adv = adv;
  p.rej = rejected; p.logratio = logratio; p.logu = logu; p.active = ctx->active; p.queue = ctx->dev_queue;
  p.B = B; p.d = ctx->d; p.K = ctx->K; p.T = ctx->T; p.M = M; p.seed = ctx->seed;
  p.gamma = gamma; p.inv_s2 = 1.0 / (static_cast<double>(comp_std) * comp_std); p.inv_tau = 1.0 / ctx->tau;
  p.max_windows = max_windows; p.n_out = n_out; p.counters = reinterpret_cast<unsigned long long*>(counters);
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int dpad = 4 * groups;
  if (groups <= 32) {                       // several chains per wavefront
    const bool run = max_windows > 1;
    // Lanes per chain: the row's groups, but with chains too few for a wavefront on every SIMD up to 16, one logit per
    // lane: a step is then latency, and eight exponentials in a row are a third of it.  Both give the same bits.
    int G = groups <= 2 ? 2 : groups <= 4 ? 4 : groups <= 8 ? 8 : groups <= 16 ? 16 : 32;
    while (G < 16 && static_cast<int64_t>(B) * 2 * G <= 64ll * 4 * ctx->cus) G *= 2;
    if (G == 2) launch_short<2>(p, run, st);
    else if (G == 4) launch_short<4>(p, run, st);
    else if (G == 8) launch_short<8>(p, run, st);
    else if (G == 16) launch_short<16>(p, run, st);
    else launch_short<32>(p, run, st);
    if (run && counters) hipLaunchKernelGGL(bump_launches_kernel, dim3(1), dim3(1), 0, st, p.counters);
    SD_HIP_TRY(ctx->err, hipGetLastError());
    return SD_OK;
  }
  if (dpad <= 1024) {                       // a wavefront per chain, means in LDS (16 rows of doubles, <= 128 KiB)
    hipError_t e;
    const bool whole = ctx->d % 4 == 0;
    const int sel = ((groups + 63) / 64 - 1) * 4 + (whole ? 2 : 0) + (max_windows > 1 ? 1 : 0);
    switch (sel) {
      case 0: e = launch_wave<1, false, false>(p, ctx->cus, st); break;
      case 1: e = launch_wave<1, false, true>(p, ctx->cus, st); break;
      case 2: e = launch_wave<1, true, false>(p, ctx->cus, st); break;
      case 3: e = launch_wave<1, true, true>(p, ctx->cus, st); break;
      case 4: e = launch_wave<2, false, false>(p, ctx->cus, st); break;
      case 5: e = launch_wave<2, false, true>(p, ctx->cus, st); break;
      case 6: e = launch_wave<2, true, false>(p, ctx->cus, st); break;
      case 7: e = launch_wave<2, true, true>(p, ctx->cus, st); break;
      case 8: e = launch_wave<3, false, false>(p, ctx->cus, st); break;
      case 9: e = launch_wave<3, false, true>(p, ctx->cus, st); break;
      case 10: e = launch_wave<3, true, false>(p, ctx->cus, st); break;
      case 11: e = launch_wave<3, true, true>(p, ctx->cus, st); break;
      case 12: e = launch_wave<4, false, false>(p, ctx->cus, st); break;
      case 13: e = launch_wave<4, false, true>(p, ctx->cus, st); break;
      case 14: e = launch_wave<4, true, false>(p, ctx->cus, st); break;
      default: e = launch_wave<4, true, true>(p, ctx->cus, st); break;
    }
    if (e != hipSuccess) return sdi::fail(ctx->err, SD_ERR_HIP, "%s: %s", who, hipGetErrorString(e));
    if (max_windows > 1 && counters) hipLaunchKernelGGL(bump_launches_kernel, dim3(1), dim3(1), 0, st, p.counters);
    return SD_OK;
  }
  if (max_windows > 1)
    return sdi::fail(ctx->err, SD_ERR_UNSUPPORTED, "%s: d=%d is above the 1024 the back-to-back form serves", who, ctx->d);
  launch_wide<false>(p, groups, st);
  SD_HIP_TRY(ctx->err, hipGetLastError());
  return SD_OK;
}

}  // namespace

extern "C" int sd_langevin_window(sd_ctx* ctx, int32_t B, const float* x, const int32_t* n,
                                  const int64_t* chain_id, const float* means, const float* logw,
                                  float comp_std, int32_t M, float gamma, float* x_out, int32_t* adv,
                                  uint8_t* rejected, float* logratio, float* logu, void* stream) {
  if (!ctx) return SD_ERR_ARG;
  if (B < 0 || M <= 0 || !(comp_std > 0.f) || !(gamma > 0.f) ||
      (B > 0 && (!x || !n || !chain_id || !means || !logw || !x_out || !adv)))
    return sdi::fail(ctx->err, SD_ERR_ARG, "sd_langevin_window: bad argument");
  if (B == 0) return SD_OK;
  return langevin_launch("sd_langevin_window", ctx, B, x, n, chain_id, means, logw, comp_std, M, gamma, x_out, adv,
                         rejected, logratio, logu, 1, nullptr, nullptr, stream);
}

extern "C" int sd_langevin_run(sd_ctx* ctx, int32_t B, const float* x, const int32_t* n, const int64_t* chain_id,
                               const float* means, const float* logw, float comp_std, int32_t M, float gamma,
                               int32_t max_windows, float* x_out, int32_t* n_out, int64_t* counters, void* stream) {
  if (!ctx) return SD_ERR_ARG;
  if (B < 0 || M <= 0 || !(comp_std > 0.f) || !(gamma > 0.f) || max_windows < 2 ||
      (B > 0 && (!x || !n || !chain_id || !means || !logw || !x_out || !n_out)))
    return sdi::fail(ctx->err, SD_ERR_ARG, "sd_langevin_run: bad argument (max_windows >= 2)");
  if (B == 0) return SD_OK;
  return langevin_launch("sd_langevin_run", ctx, B, x, n, chain_id, means, logw, comp_std, M, gamma, x_out, nullptr,
                         nullptr, nullptr, nullptr, max_windows, n_out, counters, stream);
}

extern "C" int sd_langevin_chains(sd_ctx* ctx, int32_t B, const float* x, const int32_t* n, const int64_t* chain_id,
                                  const float* means, const float* logw, float comp_std, int32_t M, float gamma,
                                  float* out, int32_t* B_active, int64_t* counters, void* stream) {
  if (!ctx) return SD_ERR_ARG;
  if (B < 0 || M <= 0 || !(comp_std > 0.f) || !(gamma > 0.f) || !B_active ||
      (B > 0 && (!x || !n || !chain_id || !means || !logw || !out)))
    return sdi::fail(ctx->err, SD_ERR_ARG, "sd_langevin_chains: bad argument");
  const int groups = (ctx->d + 3) / 4;
  if (M > 16 || ctx->d <= 1024 || groups > kMaxGroups || ctx->active)
    return sdi::fail(ctx->err, SD_ERR_UNSUPPORTED, "sd_langevin_chains: 1024 < d <= %d, at most 16 components, no device-side count",
                     4 * kMaxGroups);
  LangevinArgs p{};
  p.x = x; p.n = n; p.id = chain_id; p.means = means; p.logw = logw; p.x_out = out; p.queue = ctx->dev_queue;
  p.B = B; p.d = ctx->d; p.K = ctx->K; p.T = ctx->T; p.M = M; p.seed = ctx->seed;
  p.gamma = gamma; p.inv_s2 = 1.0 / (static_cast<double>(comp_std) * comp_std); p.inv_tau = 1.0 / ctx->tau;
  p.counters = reinterpret_cast<unsigned long long*>(counters);
  hipStream_t st = static_cast<hipStream_t>(stream);
  hipLaunchKernelGGL(reset_queue_kernel, dim3(1), dim3(1), 0, st, p.queue, 1);
  if (B > 0) launch_wide<true>(p, groups, st);
  hipLaunchKernelGGL(chains_end_kernel, dim3(1), dim3(1), 0, st, p.queue + 1, p.counters, B_active);
  SD_HIP_TRY(ctx->err, hipGetLastError());
  return SD_OK;
}

extern "C" int sd_langevin_window_phi4(sd_ctx* ctx, int32_t B, const float* x, const int32_t* n,
                                       const int64_t* chain_id, int32_t L, float beta, float gamma, float* x_out,
                                       int32_t* adv, uint8_t* rejected, float* logratio, float* logu, void* stream) {
  if (!ctx) return SD_ERR_ARG;
  if (B < 0 || L < 3 || !(beta >= 0.f) || !(gamma > 0.f) || (B > 0 && (!x || !n || !chain_id || !x_out || !adv)))
    return sdi::fail(ctx->err, SD_ERR_ARG, "sd_langevin_window_phi4: bad argument (L >= 3, beta >= 0, gamma > 0)");
  if (L * L != ctx->d)
    return sdi::fail(ctx->err, SD_ERR_ARG, "sd_langevin_window_phi4: the context's d=%d is not L*L=%d", ctx->d, L * L);
  if (ctx->d > 256)
    return sdi::fail(ctx->err, SD_ERR_UNSUPPORTED, "sd_langevin_window_phi4: grids up to 16 x 16 (d=%d)", ctx->d);
  if (B == 0) return SD_OK;
  Phi4Args p;
  p.x = x; p.n = n; p.id = chain_id; p.x_out = x_out; p.adv = adv; p.rej = rejected; p.logratio = logratio; p.logu = logu;
  p.active = ctx->active; p.B = B; p.d = ctx->d; p.L = L; p.K = ctx->K; p.T = ctx->T; p.seed = ctx->seed;
  p.gamma = gamma; p.beta = beta; p.inv_tau = 1.0 / ctx->tau;
  p.max_windows = 1; p.n_out = nullptr; p.counters = nullptr;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int groups = (ctx->d + 3) / 4;
  hipError_t e;
  if (groups <= 4) e = launch_phi4<4>(p, st);
  else if (groups <= 8) e = launch_phi4<8>(p, st);
  else if (groups <= 16) e = launch_phi4<16>(p, st);
  else if (groups <= 32) e = launch_phi4<32>(p, st);
  else e = launch_phi4<64>(p, st);
  if (e != hipSuccess) return sdi::fail(ctx->err, SD_ERR_HIP, "sd_langevin_window_phi4: %s", hipGetErrorString(e));
  return SD_OK;
}

extern "C" int sd_langevin_run_phi4(sd_ctx* ctx, int32_t B, const float* x, const int32_t* n, const int64_t* chain_id,
                                    int32_t L, float beta, float gamma, int32_t max_windows, float* x_out,
                                    int32_t* n_out, int64_t* counters, void* stream) {
  if (!ctx) return SD_ERR_ARG;
  if (B < 0 || L < 3 || !(beta >= 0.f) || !(gamma > 0.f) || max_windows < 2 ||
      (B > 0 && (!x || !n || !chain_id || !x_out || !n_out)))
    return sdi::fail(ctx->err, SD_ERR_ARG,
                     "sd_langevin_run_phi4: bad argument (L >= 3, beta >= 0, gamma > 0, max_windows >= 2)");
  if (L * L != ctx->d)
    return sdi::fail(ctx->err, SD_ERR_ARG, "sd_langevin_run_phi4: the context's d=%d is not L*L=%d", ctx->d, L * L);
  if (ctx->d > 256)
    return sdi::fail(ctx->err, SD_ERR_UNSUPPORTED, "sd_langevin_run_phi4: grids up to 16 x 16 (d=%d)", ctx->d);
  if (B == 0) return SD_OK;
  Phi4Args p;
  p.x = x; p.n = n; p.id = chain_id; p.x_out = x_out; p.adv = nullptr; p.rej = nullptr; p.logratio = nullptr; p.logu = nullptr;
  p.active = ctx->active; p.B = B; p.d = ctx->d; p.L = L; p.K = ctx->K; p.T = ctx->T; p.seed = ctx->seed;
  p.gamma = gamma; p.beta = beta; p.inv_tau = 1.0 / ctx->tau;
  p.max_windows = max_windows; p.n_out = n_out; p.counters = reinterpret_cast<unsigned long long*>(counters);
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int groups = (ctx->d + 3) / 4;
  hipError_t e;
  if (groups <= 4) e = launch_phi4_run<4>(p, st);
  else if (groups <= 8) e = launch_phi4_run<8>(p, st);
  else if (groups <= 16) e = launch_phi4_run<16>(p, st);
  else if (groups <= 32) e = launch_phi4_run<32>(p, st);
  else e = launch_phi4_run<64>(p, st);
  if (e != hipSuccess) return sdi::fail(ctx->err, SD_ERR_HIP, "sd_langevin_run_phi4: %s", hipGetErrorString(e));
  if (counters) hipLaunchKernelGGL(bump_launches_kernel, dim3(1), dim3(1), 0, st, p.counters);
  return SD_OK;
}
