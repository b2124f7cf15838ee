// Posterior mean of a diagonal-covariance Gaussian mixture under the forward noising
// x_t = sqrt(ab) x0 + sqrt(1-ab) eps -- the analytic stand-in for the target network
// (paper Sec. 3.1 treats the drift as a black box; the low-dimensional mixture study of the
// experiments has this shape) -- and whole chains on it in one launch (sdden_run).  Also the generic
// entry points of sdden.h.
//
// Up to 64 components: one wavefront per row, gmm_rows.h.  More components: the general kernel below.
// All arithmetic in fp64: the rows are few and small, and the responsibilities are
// exponentials of sums of d terms.
#include <algorithm>
#include <cmath>
#include <new>
#include <type_traits>
#include <vector>

#include "gmm_rows.h"
#include "sd_rng.h"
#include "sdden_internal.h"

namespace sdi {
std::string g_den_create_error;
}

namespace {

using sdgmm::reciprocal;

constexpr int kRowsPerBlock = 4;

struct GmmArgs {
  const float* X;
  const int32_t* krow;
  float* out;
  sdgmm::Model g;
  const float *mu, *sd;      // [M,d]  component means and stds        (general kernel only)
  const float *muT, *sdT;    // [d,M]  the same, transposed
  const float* ab;           // [T+1]
  const int32_t* active;
  int rows_per_chain;
  int R;
};

// One wavefront per row (gmm_rows.h), tables from the vector caches: a launch lives too short to pay for a copy in LDS.
// Bound by fp64 issue: 6.5 vector instructions per (component, coordinate) pair of the logit phase, about 11 per
// coordinate and live component.  32768 rows of 64 coordinates and 32 components: 66 us (80 with the component means of
// every row kept in registers and exchanged); 2000 rows of 200 and 48: 33 us (88 with a kernel that had no registers for it).
template <int E, int C, bool FINE>
__global__ __launch_bounds__(64 * kRowsPerBlock) void gmm_rows_kernel(GmmArgs p) {
  extern __shared__ double smem[];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int r = blockIdx.x * kRowsPerBlock + wave;
  const int Ract = sdi::active_rows(p.active, p.rows_per_chain, p.R);
  const int k = r < Ract ? p.krow[r] : -1;
  // masked row (k < 0) or a step the chain does not have; the whole wavefront leaves together, no barriers used
  if (static_cast<unsigned>(k) >= static_cast<unsigned>(p.g.T)) return;
  const float* row = p.X + static_cast<int64_t>(r) * p.g.d;
  const double2 st = p.g.steps[k];
  const double base = sdgmm::lane_constant(p.g, k, lane);
  float x[C][E], y[C][E];
#pragma unroll
  for (int c = 0; c < C; ++c)
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int i = E * (lane + 64 * c) + e;
      x[c][e] = i < p.g.d ? row[i] : 0.f;
    }
  double* xs = smem + static_cast<size_t>(wave) * (p.g.nslots << (6 - p.g.lm));
  sdgmm::posterior_mean<E, C, false, (C > 2), FINE>(p.g, nullptr, xs, x, st.x, st.y, base, lane, y);
  float* o = p.out + static_cast<int64_t>(r) * p.g.d;
#pragma unroll
  for (int c = 0; c < C; ++c)
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int i = E * (lane + 64 * c) + e;
      if (i < p.g.d) o[i] = y[c][e];
    }
}

// One component, whose responsibility is 1: the mean of gmm_rows.h coordinate by coordinate, with the same bits.  A row (or a
// weight) with an infinity or a NaN has no responsibilities and becomes NaN, as there.  Bound by the row's bytes and one round trip:
// 1000 rows of d = 1800 8.0 us (12.3 through gmm_rows_kernel), 32768 rows of d = 400 21 us (46.5).
__global__ __launch_bounds__(64 * kRowsPerBlock) void gmm_one_component_kernel(GmmArgs p) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, d = p.g.d;
  const int r = blockIdx.x * kRowsPerBlock + wave;
  const int Ract = sdi::active_rows(p.active, p.rows_per_chain, p.R);
  const int k = r < Ract ? p.krow[r] : -1;
  if (static_cast<unsigned>(k) >= static_cast<unsigned>(p.g.T)) return;
  const double2 st = p.g.steps[k];
  const double ab = st.x, sab = st.y, om = 1.0 - ab;
  const float* x = p.X + static_cast<int64_t>(r) * d;
  float* o = p.out + static_cast<int64_t>(r) * d;
  bool finite = __builtin_isfinite(p.g.cst[k]);
#pragma unroll 4
  for (int i = lane; i < d; i += 64) {
    const float2 t = p.g.row_tab[i];
    const double mu = t.x, s2 = static_cast<double>(t.y) * t.y;
    const double iv = sdgmm::reciprocal_one_step(fma(ab, s2, om));
    const double df = fma(-sab, mu, static_cast<double>(x[i]));
    finite = finite && __builtin_isfinite(df);
    o[i] = static_cast<float>(fma(sab * s2 * iv, df, mu));
  }
  if (__ballot(!finite) != 0ull)
    for (int i = lane; i < d; i += 64) o[i] = __builtin_nanf("");
}

// More than 64 components.  Phase 1: a lane owns components lane, lane + 64, .. and walks the coordinates (no
// cross-lane reduction for the logits).  Phase 2: a lane owns a coordinate and walks the components.
__global__ __launch_bounds__(64 * kRowsPerBlock) void gmm_many_components_kernel(GmmArgs p) {
  extern __shared__ double smem[];
  const int M = p.g.M, d = p.g.d;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  double* rs = smem + static_cast<size_t>(wave) * (M + d);       // [M] responsibilities
  double* xs = rs + M;                                           // [d] the row
  const int r = blockIdx.x * kRowsPerBlock + wave;
  const int Ract = sdi::active_rows(p.active, p.rows_per_chain, p.R);
  const int k = r < Ract ? p.krow[r] : -1;
  if (static_cast<unsigned>(k) >= static_cast<unsigned>(p.g.T)) return;
  const double ab = p.ab[k];
  const double sab = sqrt(ab), om = 1.0 - ab;
  const float* x = p.X + static_cast<int64_t>(r) * d;
  for (int i = lane; i < d; i += 64) xs[i] = x[i];
  sdgmm::wave_lds_fence();

  double mx = -INFINITY;
  for (int m = lane; m < M; m += 64) {
    double q = 0.0;
    for (int i = 0; i < d; ++i) {
      const double diff = xs[i] - sab * p.muT[static_cast<int64_t>(i) * M + m];
      const double sd = p.sdT[static_cast<int64_t>(i) * M + m];
      const double iv = reciprocal(ab * sd * sd + om);
      q = fma(diff * diff, iv, q);
    }
    const double logit = p.g.cst[static_cast<int64_t>(k) * M + m] - 0.5 * q;
    rs[m] = logit;
    mx = fmax(mx, logit);
  }
  for (int s = 32; s >= 1; s >>= 1) mx = fmax(mx, __shfl_xor(mx, s, 64));
  double sum = 0.0;
  for (int m = lane; m < M; m += 64) {
    const double e = exp(rs[m] - mx);
    rs[m] = e;
    sum += e;
  }
  for (int s = 32; s >= 1; s >>= 1) sum += __shfl_xor(sum, s, 64);
  const double inv = 1.0 / sum;
  sdgmm::wave_lds_fence();

  float* o = p.out + static_cast<int64_t>(r) * d;
  for (int i = lane; i < d; i += 64) {
    const double xi = xs[i];
    double acc = 0.0;
    for (int m = 0; m < M; ++m) {
      if (rs[m] < 1e-25) continue;          // the same for every lane; such a component moves nothing
      const double mu = p.mu[static_cast<int64_t>(m) * d + i];
      const double sd = p.sd[static_cast<int64_t>(m) * d + i];
      const double s2 = sd * sd;
      const double iv = reciprocal(ab * s2 + om);
      acc += rs[m] * (mu + sab * s2 * iv * (xi - sab * mu));
    }
    o[i] = static_cast<float>(acc * inv);
  }
}

// Where one component is alone.  With q_m = |x - sqrt(ab) mu_m|^2 in the metric 1 / v_m(k) and rho^2 = q_a, the triangle
// inequality in the metric of m gives sqrt(q_m) >= D - s rho, D the distance of the two means there and s^2 the largest v_a / v_m:
//   l_a - l_m >= cst_a - cst_m + (D - s rho)^2 / 2 - rho^2 / 2    for rho <= D / s,
// which falls with rho.  The radius of component a at step k is where the least of them reaches kAloneGap: inside, every other
// responsibility is below e^-60 < 1e-25, adds nothing to the mean and nothing to the softmax sum's 53 bits.  Rounded down by
// far more than the arithmetic of either side is off.  One wavefront per (step, component), a lane per other component, once
// per denoiser; also counts the balls that hold a typical state.
constexpr double kAloneGap = 60.0;
__global__ __launch_bounds__(64 * kRowsPerBlock) void gmm_radius_kernel(sdgmm::Model g, float* radius2, int32_t* holds) {
  const int64_t at = static_cast<int64_t>(blockIdx.x) * kRowsPerBlock + (threadIdx.x >> 6);
  if (at >= static_cast<int64_t>(g.T) * g.M) return;
  const int m = threadIdx.x & 63, k = static_cast<int>(at / g.M), a = static_cast<int>(at % g.M);
  const double2 st = g.steps[k];
  const double ab = st.x, om = 1.0 - ab, *cst = g.cst + static_cast<int64_t>(k) * g.M;
  float least = INFINITY;
  if (m < g.M && m != a && cst[m] != -INFINITY) {
    const float2 *pa = g.row_tab + static_cast<int64_t>(a) * g.d, *pm = g.row_tab + static_cast<int64_t>(m) * g.d;
    double d2 = 0.0, s2 = 0.0;
#pragma unroll 4
    for (int i = 0; i < g.d; ++i) {
      const float2 ta = pa[i], tm = pm[i];
      const double iv = reciprocal(fma(ab, static_cast<double>(tm.y) * tm.y, om));
      const double df = st.y * (static_cast<double>(ta.x) - tm.x);
      d2 = fma(df * df, iv, d2);
      s2 = fmax(s2, fma(ab, static_cast<double>(ta.y) * ta.y, om) * iv);
    }
    // the smaller root of c + D^2 / 2 - s D rho + (s^2 - 1) rho^2 / 2, at most D / s; none: positive all the way there
    const double top = 2.0 * (cst[a] - cst[m] - kAloneGap) + d2, sD2 = s2 * d2, disc = sD2 - (s2 - 1.0) * top;
    double rho = disc >= 0.0 ? top / (sqrt(sD2) + sqrt(disc)) : INFINITY;
    rho = fmin(rho, sqrt(d2 / s2));
    least = top > 0.0 ? static_cast<float>(rho) : 0.f;     // also where something is not a number
  }
  for (int o = 32; o >= 1; o >>= 1) least = fminf(least, __shfl_xor(least, o, 64));
  if (m == 0) {
    const float r2 = 0.999f * least * least;
    radius2[static_cast<int64_t>(a) * g.T + k] = r2;
    if (r2 > static_cast<float>(g.d)) atomicAdd(holds, 1);
  }
}

// ---------------------------------------------------------------------------------------------
// Every chain of a batch from its step to T in one launch: one wavefront owns a chain and walks its windows, each of
// which computes what (window-start prediction, draft, batched prediction, verify, advance) computes for it.  Chains
// do not interact, so nothing needs the launches, the compaction and the readback between two windows; and because
// the walk of a window is serial it stops at the first rejection, so a chain costs exactly one target evaluation per
// step it takes (plus the carried one of the efficient frozen drafter) instead of K per window.
// Values: drafts, predictions and states are rounded to fp32 exactly where the separate calls store them; log-ratios
// are fp64 sums of the same terms.
// Measured against windows of separate calls: 4096 chains, d = 64, 32 components, 200 steps 0.87 ms against 4.76; 64 chains,
// d = 2, 8 components, 100 steps 0.11 ms against 1.81 (gmm_window_run_kernel); 300 chains, d = 75, 12 components, a draft model, 60
// steps 0.21 ms against 8.1 (two wavefronts a chain).  The first is bound by fp64 issue, over half of it in the quarter of the steps in
// which many components are live, the others by the latency of one wavefront's step: hence no branch per exchange level, no load and no
// generator pass per step.
// ---------------------------------------------------------------------------------------------
struct RunArgs {
  sdgmm::Model t, q;         // target; draft model of the independent drafter
  const float *y, *Dfz;      // start states; carried predictions (efficient frozen drafter)
  const int32_t* n;
  const int64_t* id;
  float* out;
  const float *a, *c, *sigma;
  int B, K, T;
  int reused, carry_last;    // efficient frozen drafter and its second carry rule
  uint64_t seed;
  double inv_tau;
  unsigned long long* counters;   // optional: sum adv, chain-windows, rejections, windows, sum Kt
  int32_t* longest;               // windows of the chain that needed most (zero on entry)
};

// Standard normals of this lane's coordinates E * (lane + 64 c) + e of the vector keyed (seed, id, k).
// d <= 128 (E < 4): a step needs ceil(d / 4) <= 32 blocks of the generator, so one pass of the 64 lanes draws the noise
// of several steps, a block each, and parks it in wavefront-private LDS; a chain takes its steps in order.  (Drawing
// per step, lanes that share a block would each repeat its ten rounds.)
struct NoiseBatch {
  int base, steps, shift;    // first step held, steps held at a time (64 >> shift), log2 of the blocks a step takes
  __device__ __forceinline__ void init(int d) {
    shift = 0;
    while ((4 << shift) < d) ++shift;
    steps = 64 >> shift;
    base = -64;
  }
};

template <int E, int C>
__device__ __forceinline__ void lane_normals(NoiseBatch& nb, float* zs, uint64_t seed, int64_t id, int k, int lane, float (&z)[C][E]) {
  if constexpr (E == 4) {
#pragma unroll
    for (int c = 0; c < C; ++c)
      sdrng::normal4(seed, id, static_cast<uint32_t>(k), sdrng::kStreamNoise, static_cast<uint32_t>(lane + 64 * c), z[c]);
  } else {
    static_assert(C == 1, "one group of coordinates per lane");
    if (k - nb.base >= nb.steps) {
      nb.base = k;
      float w[4];
      sdrng::normal4(seed, id, static_cast<uint32_t>(k + (lane >> nb.shift)), sdrng::kStreamNoise,
                     static_cast<uint32_t>(lane & ((1 << nb.shift) - 1)), w);
      sdgmm::wave_lds_fence();
      *reinterpret_cast<float4*>(zs + 4 * lane) = make_float4(w[0], w[1], w[2], w[3]);
      sdgmm::wave_lds_fence();
    }
    const int at = ((k - nb.base) << (nb.shift + 2)) + E * lane;       // a step's noise: 4 << shift consecutive floats
    if constexpr (E == 2) {
      const float2 v = *reinterpret_cast<const float2*>(zs + (at & 255));
      z[0][0] = v.x; z[0][1] = v.y;
    } else {
      z[0][0] = zs[at & 255];              // lanes past d read another coordinate's noise, which is not used
    }
  }
}

template <bool LDS>
__device__ __forceinline__ void stage_table(const sdgmm::Model& g, double2* tab) {
  if (!LDS) return;
#pragma unroll 4
  for (int s = threadIdx.x; s < g.nslots * 64; s += blockDim.x) {
    const float2 v = g.lane_tab[s];
    tab[(s >> 6) * sdgmm::kTabStride + (s & 63)] = make_double2(v.x, static_cast<double>(v.y) * v.y);
  }
}

// What a step needs from the per-step tables, 64 steps at a time in the lanes of a wavefront: a chain's evaluations come
// in the order of the steps whatever its windows do, so a step is served by readlane instead of by loads whose latency
// a lone wavefront could not hide.
struct StepBatch {
  int base;                  // first step held; -64 before the first refill
  float a, c, s;
  double inv_s2, log_u;      // 1 / sigma^2; log of the uniform that tests the state the step produces
  double2 t, q;              // (ab, sqrt(ab)) of the target's and the draft model's tables
  __device__ __forceinline__ void refill(const RunArgs& p, bool indep, int k, int64_t id, int lane) {
    base = k;
    const int kk = min(k + lane, p.T - 1);
    a = p.a[kk]; c = p.c[kk]; s = p.sigma[kk];
    const double sg = s;
    inv_s2 = 1.0 / (sg * sg);
    log_u = sdrng::log_uniform(p.seed, id, static_cast<uint32_t>(k + lane + 1));
    t = p.t.steps[kk];
    if (indep) q = p.q.steps[kk];
  }
};

__device__ __forceinline__ float readlane_f32(float v, int src_lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), src_lane));
}

// FINE: reciprocal variances to fp64 rounding (sdgmm::needs_fine); the vector caches' form always has them.
// ALONE: a step is first tried with the component its chain was last seen with alone, which takes no pass over the pairs, no
// exchange of the row and no softmax; about 300 of 550 instructions at 32 pairs per lane, while the attempts and the wider
// loop cost the other steps 4 to 10 %.  Taken where the share of the balls that hold a typical state (radius^2 > d) reaches 0.35 from 24
// pairs per lane on, 0.45 below.  Runs of 100 or 200 steps, with / without it, over the share:
//   28 to 52 pairs  0.16 1.04  0.23 1.08  0.39 0.97  0.40 0.97  0.49 0.81  0.56 0.69  0.62 0.74  0.75 0.59
//   116 pairs       0.46 0.78  0.66 0.58  0.90 0.40
//   4 to 20 pairs   0.12 1.09  0.22 1.05  0.41 1.00  0.46 0.92  0.49 0.90  0.60 0.79  0.70 0.79
//   1 or 2 pairs    0.24 1.09  0.33 1.06  0.59 0.86  0.61 0.91
//   two models      0.16 0.95  0.20 1.10  0.22 1.10  0.41 1.02 and 1.06  0.51 1.01  0.56 0.75  0.61 0.95  0.65 0.91  0.70 0.93 and 1.01
// whether the table lies in LDS or not.  Two models follow the target's share.
// SHARES: the model may have its components' shares added up where they are (sdgmm::posterior_mean): runs that cannot are 1 to 3 %
// faster without that code in the loop: 3000 chains, d = 60, M = 8, 100 steps 248 / 258, 2000 chains, d = 30, M = 20 287 / 294.
// PAIR (INDEP): two wavefronts a chain, one for each model; an instance of its own, because the branches around the two predictions
// cost many chains 4 % (4096 chains, d = 10, M = 12, two models, 100 steps 568 us with them, 542 without).
// DENSE (two models, ALONE, a coordinate per lane): held to the registers of four wavefronts per SIMD, for runs that fill more than
// three: 4096 chains, 60 steps d = 64, M = 32 622 us with it, 730 without, M = 12 346 / 400; 1200 chains 245 / 233.
enum Form { kPlain, kPair, kDense };
template <int E, int C, bool LDS, bool INDEP, bool FINE, bool ALONE, Form FORM, bool SHARES>
__global__ __launch_bounds__(256, FORM == kDense ? 4 : 1) void gmm_run_kernel(RunArgs p) {
  constexpr bool PAIR = FORM == kPair;
  extern __shared__ __align__(16) unsigned char run_smem[];
  __shared__ unsigned long long sh_cnt[4];
  __shared__ int sh_longest;
  double2* tab_t = reinterpret_cast<double2*>(run_smem);
  double2* tab_q = tab_t + (LDS ? p.t.nslots * sdgmm::kTabStride : 0);
  double* xs0 = reinterpret_cast<double*>(tab_q + (LDS && INDEP ? p.q.nslots * sdgmm::kTabStride : 0));
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  int npad = p.t.nslots << (6 - p.t.lm);
  if (INDEP) npad = max(npad, p.q.nslots << (6 - p.q.lm));
  npad = (npad + 1) & ~1;                  // 16-byte pieces
  double* xs = xs0 + static_cast<size_t>(wave) * npad;
  float* zs = reinterpret_cast<float*>(xs0 + static_cast<size_t>(blockDim.x >> 6) * npad) + 256 * wave;   // E < 4 only
  float* both = zs + 256 * ((E < 4 ? 2 : 0) - wave);       // pair: [2][2][64 E C] predictions, buffers that alternate
  int par = 0;
  stage_table<LDS>(p.t, tab_t);
  if (INDEP) stage_table<LDS>(p.q, tab_q);
  if (threadIdx.x < 4) sh_cnt[threadIdx.x] = 0;
  if (threadIdx.x == 0) sh_longest = 0;
  __syncthreads();

  const int b = PAIR ? static_cast<int>(blockIdx.x) : static_cast<int>(blockIdx.x) * static_cast<int>(blockDim.x >> 6) + wave;
  if (b < p.B) {                           // uniform over the wavefront; pair: over the workgroup
    const int d = p.t.d;
    const int64_t id = p.id[b];
    int n = __builtin_amdgcn_readfirstlane(p.n[b]);
    const int n_start = n;
    float y[C][E], d0[C][E];
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int i = E * (lane + 64 * c) + e;
        y[c][e] = i < d ? p.y[static_cast<int64_t>(b) * d + i] : 0.f;
        d0[c][e] = !INDEP && p.reused && i < d ? p.Dfz[static_cast<int64_t>(b) * d + i] : 0.f;
      }
    int windows = 0, rejections = 0;
    long long kt_sum = 0;
    StepBatch sb;
    sb.base = -64;
    NoiseBatch nb;
    nb.init(d);
    sdgmm::Constants cst_t, cst_q;         // ALONE
    // else component constants of the next step to be evaluated, requested one step ahead
    double next_t = ALONE ? 0.0 : sdgmm::lane_constant(p.t, min(n, p.T - 1), lane), next_q = 0.0;
    if (INDEP && !ALONE) next_q = sdgmm::lane_constant(p.q, min(n, p.T - 1), lane);
    sdgmm::Alone alone_t, alone_q;

    while (n < p.T) {                      // every window advances the chain by at least one step
      const int Kt = min(p.K, p.T - n);
      const bool frozen = !INDEP && !p.reused;
      float dr[C][E], dq[C][E];
      int adv = Kt;
      bool rejected = false;
      for (int j = 0; j < Kt; ++j) {
        const int k = n + j;
        if (k - sb.base >= 64) sb.refill(p, INDEP, k, id, lane);
        const int at = k - sb.base;
        const float a = readlane_f32(sb.a, at), cf = readlane_f32(sb.c, at), s = readlane_f32(sb.s, at);
        const double ab = sdgmm::readlane_f64(sb.t.x, at), sab = sdgmm::readlane_f64(sb.t.y, at);
        double base_t = next_t, base_q = next_q;
        if (!ALONE) {
          next_t = sdgmm::lane_constant(p.t, min(k + 1, p.T - 1), lane);
          if (INDEP) next_q = sdgmm::lane_constant(p.q, min(k + 1, p.T - 1), lane);
        }
        float z[C][E], mp[C][E];
        lane_normals<E, C>(nb, zs, p.seed, id, k + 1, lane, z);
        // The step's one target evaluation, at the state it starts from: the frozen prediction of the window (first
        // position of the frozen drafter), else what the draft is tested against.
        if (PAIR && wave == 1) {}          // the other wavefront's
        else if (!ALONE || !sdgmm::mean_of_one<E, C, LDS, FINE>(p.t, tab_t, y, ab, sab, k, lane, alone_t, dq)) {
          if (ALONE) base_t = cst_t.at(p.t, k, lane);
          sdgmm::posterior_mean<E, C, LDS, !LDS, FINE, SHARES>(p.t, tab_t, xs, y, ab, sab, base_t, lane, dq, ALONE ? &alone_t : nullptr, k);
        }
        if (frozen && j == 0) {
#pragma unroll
          for (int c = 0; c < C; ++c)
#pragma unroll
            for (int e = 0; e < E; ++e) d0[c][e] = dq[c][e];
        }
        if (INDEP && !(PAIR && wave == 0)) {       // the draft model's prediction
          const double abq = sdgmm::readlane_f64(sb.q.x, at), sabq = sdgmm::readlane_f64(sb.q.y, at);
          if (!ALONE || !sdgmm::mean_of_one<E, C, LDS, FINE>(p.q, tab_q, y, abq, sabq, k, lane, alone_q, mp)) {
            if (ALONE) base_q = cst_q.at(p.q, k, lane);
            sdgmm::posterior_mean<E, C, LDS, !LDS, FINE, SHARES>(p.q, tab_q, xs, y, abq, sabq, base_q, lane, mp, ALONE ? &alone_q : nullptr, k);
          }
        }
        if (PAIR) {                        // both go on with both: all that follows is the same on the two
          float* mine = both + (par * 2 + wave) * 64 * E * C;
          const float* theirs = both + (par * 2 + 1 - wave) * 64 * E * C;
#pragma unroll
          for (int c = 0; c < C; ++c)
#pragma unroll
            for (int e = 0; e < E; ++e) mine[(c * E + e) * 64 + lane] = wave == 0 ? dq[c][e] : mp[c][e];
          __syncthreads();
#pragma unroll
          for (int c = 0; c < C; ++c)
#pragma unroll
            for (int e = 0; e < E; ++e) {
              const float v = theirs[(c * E + e) * 64 + lane];
              if (wave == 0) mp[c][e] = v;
              else dq[c][e] = v;
            }
          par ^= 1;
        }
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
          for (int e = 0; e < E; ++e) {
            if (INDEP) {
              mp[c][e] = fmaf(a, y[c][e], cf * mp[c][e]);
              dr[c][e] = fmaf(s, z[c][e], mp[c][e]);
            } else {
              dr[c][e] = fmaf(a, y[c][e], fmaf(cf, d0[c][e], s * z[c][e]));
            }
            if (E * (lane + 64 * c) + e >= d) dr[c][e] = 0.f;
          }
        // frozen drafter, first position: draft and target mean are the same, accepted without a test
        if (!frozen || j > 0) {
          double s1 = 0.0, s2 = 0.0;
#pragma unroll
          for (int c = 0; c < C; ++c)
#pragma unroll
            for (int e = 0; e < E; ++e) {
              if (E * (lane + 64 * c) + e >= d) continue;
              double w, dl;                // as in verify_kernel: sigma Z, and (sigma / c) Delta or sigma Delta
              if (INDEP) {
                w = static_cast<double>(dr[c][e]) - static_cast<double>(mp[c][e]);
                dl = static_cast<double>(mp[c][e]) - (static_cast<double>(a) * y[c][e] + static_cast<double>(cf) * dq[c][e]);
              } else {
                w = static_cast<double>(dr[c][e]) - static_cast<double>(a) * y[c][e] - static_cast<double>(cf) * d0[c][e];
                dl = static_cast<double>(d0[c][e]) - static_cast<double>(dq[c][e]);
              }
              s1 = fma(w, dl, s1);
              s2 = fma(dl, dl, s2);
            }
          // both sums in one butterfly: the lower half of the wavefront carries s1, the upper half s2
          double t = sdlane::halving_add<32>(s1, s2);
          if (d > 16 * E) t = sdlane::pair_sum_rows<16>(t);            // lanes past d hold 0
          if (d > 8 * E) t += sdlane::lane_xor<8>(t);
          t += sdlane::lane_xor<4>(t);
          t += sdlane::lane_xor<2>(t);
          t += sdlane::lane_xor<1>(t);
          const double lu = sdgmm::readlane_f64(sb.log_u, at), inv_s2 = sdgmm::readlane_f64(sb.inv_s2, at);
          const double cc = INDEP ? 1.0 : static_cast<double>(cf);
          const double S1 = sdgmm::readlane_f64(t, 0) * cc * inv_s2, S2 = sdgmm::readlane_f64(t, 32) * cc * cc * inv_s2;
          const double lr = (-S1 - 0.5 * S2) * p.inv_tau;
          if (!(S2 == 0.0 || (lr == lr && lu <= fmin(0.0, lr)))) {       // uniform; a log-ratio that is not a number rejects
            const double two_coef = 2.0 * (S2 > 0.0 ? S1 / S2 : 0.0);
#pragma unroll
            for (int c = 0; c < C; ++c)
#pragma unroll
              for (int e = 0; e < E; ++e) {
                if (INDEP) {
                  const double mq = static_cast<double>(a) * y[c][e] + static_cast<double>(cf) * dq[c][e];
                  const double mpd = mp[c][e];
                  y[c][e] = static_cast<float>(mq + (static_cast<double>(dr[c][e]) - mpd) - two_coef * (mpd - mq));
                } else {
                  const double f = static_cast<double>(cf) * (1.0 + two_coef);
                  y[c][e] = static_cast<float>(static_cast<double>(dr[c][e]) -
                                               f * (static_cast<double>(d0[c][e]) - static_cast<double>(dq[c][e])));
                }
                if (E * (lane + 64 * c) + e >= d) y[c][e] = 0.f;
              }
            adv = j + 1;
            rejected = true;
            break;
          }
        }
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
          for (int e = 0; e < E; ++e) y[c][e] = dr[c][e];
      }
      n += adv;
      windows += 1;
      rejections += rejected ? 1 : 0;
      kt_sum += Kt;
      if (!INDEP && p.reused && n < p.T) {
        // the next window's frozen prediction: at the draft state of the step advanced to, or (second rule, after a
        // rejection) the one already at hand for the last state kept
        if (rejected && p.carry_last) {
#pragma unroll
          for (int c = 0; c < C; ++c)
#pragma unroll
            for (int e = 0; e < E; ++e) d0[c][e] = dq[c][e];
        } else {
          if (n - sb.base >= 64) sb.refill(p, INDEP, n, id, lane);
          const int at = n - sb.base;
          const double abn = sdgmm::readlane_f64(sb.t.x, at), sabn = sdgmm::readlane_f64(sb.t.y, at);
          if (!ALONE || !sdgmm::mean_of_one<E, C, LDS, FINE>(p.t, tab_t, dr, abn, sabn, n, lane, alone_t, d0))
            sdgmm::posterior_mean<E, C, LDS, !LDS, FINE, SHARES>(p.t, tab_t, xs, dr, abn, sabn, ALONE ? cst_t.at(p.t, n, lane) : next_t, lane, d0,
                                                         ALONE ? &alone_t : nullptr, n);
        }
      }
    }
    windows = max(windows, 1);             // handed over at T: one window, of no positions, that keeps the state
    const bool writes = !PAIR || wave == 0;
    float* o = p.out + id * d;
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int i = E * (lane + 64 * c) + e;
        if (writes && i < d) o[i] = y[c][e];
      }
    if (writes && lane == 0) {
      atomicAdd(&sh_cnt[0], static_cast<unsigned long long>(n - n_start));
      atomicAdd(&sh_cnt[1], static_cast<unsigned long long>(windows));
      atomicAdd(&sh_cnt[2], static_cast<unsigned long long>(rejections));
      atomicAdd(&sh_cnt[3], static_cast<unsigned long long>(kt_sum));
      atomicMax(&sh_longest, windows);
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    if (p.counters) {
      if (sh_cnt[0]) atomicAdd(p.counters + 0, sh_cnt[0]);
      if (sh_cnt[1]) atomicAdd(p.counters + 1, sh_cnt[1]);
      if (sh_cnt[2]) atomicAdd(p.counters + 2, sh_cnt[2]);
      if (sh_cnt[3]) atomicAdd(p.counters + 4, sh_cnt[3]);
    }
    if (sh_longest) atomicMax(p.longest, sh_longest);
  }
}

// ---------------------------------------------------------------------------------------------
// The same for few chains (frozen and efficient frozen drafter): a workgroup of W wavefronts owns a chain, and what the
// sampling is made for happens inside it.  With the frozen prediction known every draft of the window is, so in one round
// wavefront w predicts (and tests) the w-th position from here; the first rejection, or the end of the window, decides where
// the chain goes on.  One wavefront takes the state behind the window's last draft, which is the next window's start where
// everything is accepted.  A chain then costs a round per W positions and one more after a rejection (the frozen drafter's new
// start) instead of a prediction per position.  Every wavefront holds the chain's state and walks the drafts to its position
// itself (two operations each, noise from a ring in LDS that the wavefronts fill ahead in turn); a round's states, predictions
// and verdicts go through LDS, in buffers that alternate, behind one barrier.  Values and decisions are those of the
// kernel above: same operations on the same numbers.
// Bound by a round's latency, about 2 us: 64 chains of the toy (d = 2, M = 8, K = 4, 3.8 of 4 accepted) 110 us a run, 161 with a
// wavefront a chain; more in GmmDenoiser::run.
// ---------------------------------------------------------------------------------------------
template <int E, bool LDS, bool FINE, bool ALONE, bool SHARES>
__global__ __launch_bounds__(512) void gmm_window_run_kernel(RunArgs p) {
  extern __shared__ __align__(16) unsigned char run_smem[];
  constexpr int kRow = 64 * E;
  const int W = static_cast<int>(blockDim.x >> 6);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int npad = ((p.t.nslots << (6 - p.t.lm)) + 1) & ~1;
  double2* tab = reinterpret_cast<double2*>(run_smem);
  double* xs = reinterpret_cast<double*>(tab + (LDS ? p.t.nslots * sdgmm::kTabStride : 0)) + static_cast<size_t>(w) * npad;
  float* states = reinterpret_cast<float*>(reinterpret_cast<double*>(tab + (LDS ? p.t.nslots * sdgmm::kTabStride : 0)) +
                                           static_cast<size_t>(W) * npad);      // [2][W][kRow]
  float* means = states + 2 * W * kRow;                                         // [2][W][kRow]
  float* ring = means + 2 * W * kRow;                                           // [passes][256]
  __shared__ int verdict[2][8];
  stage_table<LDS>(p.t, tab);

  const int b = blockIdx.x, d = p.t.d;
  const int64_t id = p.id[b];
  int n = __builtin_amdgcn_readfirstlane(p.n[b]);
  const int n_start = n;
  float y[E], d0[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int i = E * lane + e;
    y[e] = i < d ? p.y[static_cast<int64_t>(b) * d + i] : 0.f;
    d0[e] = p.reused && i < d ? p.Dfz[static_cast<int64_t>(b) * d + i] : 0.f;
  }

  // Noise: one pass of a wavefront draws 64 >> shift consecutive steps (E < 4; a block per lane) or one, 256 floats; pass q holds
  // steps q << sh .. and lies in slot q % passes.  Wavefront q % W draws it.  A round that starts at step k0 reads the noise of
  // k0 + 1 .. k0 + W + 1 and ends at k0 + W + 1 at most: what is drawn up to k0 + 2 W + 2 serves the next one whatever it decides,
  // and the slots it takes are those of steps up to k0.
  int shift = 6;                                   // log2 of the blocks a step takes, 64 for E = 4
  if (E < 4) {
    shift = 0;
    while ((4 << shift) < d) ++shift;
  }
  const int sh = 6 - shift, passes = ((2 * W + 1) >> sh) + 2;
  int drawn = (n + 1) >> sh;                       // this wavefront's next pass
  while (drawn % W != w) ++drawn;
  auto draw_up_to = [&](int last_step) {
    for (; drawn <= last_step >> sh; drawn += W) {
      float z[4];
      sdrng::normal4(p.seed, id, static_cast<uint32_t>((drawn << sh) + (lane >> shift)), sdrng::kStreamNoise,
                     static_cast<uint32_t>(lane & ((1 << shift) - 1)), z);
      *reinterpret_cast<float4*>(ring + (drawn % passes) * 256 + 4 * lane) = make_float4(z[0], z[1], z[2], z[3]);
    }
  };
  auto noise = [&](int k, float (&z)[E]) {         // of the step that ends in state k
    const float* pass = ring + ((k >> sh) % passes) * 256;
    const int from = ((k & ((1 << sh) - 1)) << (shift + 2)) + E * lane;
#pragma unroll
    for (int e = 0; e < E; ++e) z[e] = pass[(from + e) & 255];                  // lanes past d: not used
  };
  draw_up_to(n + 2 * W + 2);
  __syncthreads();

  StepBatch sb;
  sb.base = -64 - W;                               // a round looks at steps up to k0 + W + 1
  sdgmm::Alone alone;
  int cst_k = -1;                                  // constants of the step this wavefront is expected to predict next
  double cst = 0.0;
  auto expect = [&](int k) {
    cst_k = min(k, p.T - 1);
    cst = sdgmm::lane_constant(p.t, cst_k, lane);
  };
  auto predict = [&](const float (&x)[E], int k, float (&out)[E]) {
    const int at = k - sb.base;
    const double ab = sdgmm::readlane_f64(sb.t.x, at), sab = sdgmm::readlane_f64(sb.t.y, at);
    float xx[1][E], oo[1][E];
#pragma unroll
    for (int e = 0; e < E; ++e) xx[0][e] = x[e];
    if (!ALONE || !sdgmm::mean_of_one<E, 1, LDS, FINE>(p.t, tab, xx, ab, sab, k, lane, alone, oo))
      sdgmm::posterior_mean<E, 1, LDS, !LDS, FINE, SHARES>(p.t, tab, xs, xx, ab, sab, cst_k == k ? cst : sdgmm::lane_constant(p.t, k, lane), lane, oo,
                                                   ALONE ? &alone : nullptr, k);
#pragma unroll
    for (int e = 0; e < E; ++e) out[e] = oo[0][e];
  };
  auto draft = [&](const float (&x)[E], int k, float (&to)[E]) {               // state k + 1 from state k
    const int at = k - sb.base;
    const float a = readlane_f32(sb.a, at), cf = readlane_f32(sb.c, at), s = readlane_f32(sb.s, at);
    float z[E];
    noise(k + 1, z);
#pragma unroll
    for (int e = 0; e < E; ++e) to[e] = E * lane + e < d ? fmaf(a, x[e], fmaf(cf, d0[e], s * z[e])) : 0.f;
  };
  auto put = [&](float* rows, int par, int r, const float (&v)[E]) {
#pragma unroll
    for (int e = 0; e < E; ++e) rows[(par * W + r) * kRow + E * lane + e] = v[e];
  };
  auto get = [&](const float* rows, int par, int r, float (&v)[E]) {
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = rows[(par * W + r) * kRow + E * lane + e];
  };

  int windows = 0, rejections = 0, j = 0, par = 0;
  long long kt_sum = 0;
  bool have_d0 = p.reused != 0;                    // the window's frozen prediction is known
  bool at_y = false;                               // and is the prediction at y itself: position 0 need not be tested
  auto know_d0_at_y = [&]() {
    bool finite = true;
#pragma unroll
    for (int e = 0; e < E; ++e) finite = finite && __builtin_isfinite(d0[e]);
    have_d0 = true;
    at_y = !p.reused || __ballot(!finite) == 0ull;         // Delta = 0 accepts, a Delta that is not a number does not
  };
  // Ends: a round either finds the frozen prediction, which the next one has, or decides at least one position.
  while (n < p.T) {                                // uniform over the workgroup: every wavefront holds the same numbers
    const int Kt = min(p.K, p.T - n), k0 = n + j;
    if (k0 + W + 1 - sb.base >= 64) sb.refill(p, false, k0, id, lane);
    if (!have_d0) {                                // a window's start
      if (w == 0) {
        float m[E];
        predict(y, n, m);
        put(means, par, 0, m);
      }
      draw_up_to(k0 + 2 * W + 2);
      __syncthreads();
      get(means, par, 0, d0);
      par ^= 1;
      know_d0_at_y();
      continue;
    }
    const int first = j == 0 && at_y ? 1 : 0, pos = j + first + w;             // window position of this wavefront
    float x[E], m[E] = {}, res[E] = {};
#pragma unroll
    for (int e = 0; e < E; ++e) x[e] = y[e];
    bool reject = false;
    if (pos <= Kt) {
      for (int t = j; t < pos; ++t) draft(x, n + t, x);
      if (n + pos < p.T) predict(x, n + pos, m);
#pragma unroll
      for (int e = 0; e < E; ++e) res[e] = x[e];
      if (pos < Kt) {
        const int k = n + pos, at = k - sb.base;
        const float a = readlane_f32(sb.a, at), cf = readlane_f32(sb.c, at);
        float dr[E];
        draft(x, k, dr);
        double s1 = 0.0, s2 = 0.0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
          if (E * lane + e >= d) continue;
          const double u = static_cast<double>(dr[e]) - static_cast<double>(a) * x[e] - static_cast<double>(cf) * d0[e];
          const double dl = static_cast<double>(d0[e]) - static_cast<double>(m[e]);
          s1 = fma(u, dl, s1);
          s2 = fma(dl, dl, s2);
        }
        double t = sdlane::halving_add<32>(s1, s2);
        if (d > 16 * E) t = sdlane::pair_sum_rows<16>(t);
        if (d > 8 * E) t += sdlane::lane_xor<8>(t);
        t += sdlane::lane_xor<4>(t);
        t += sdlane::lane_xor<2>(t);
        t += sdlane::lane_xor<1>(t);
        const double lu = sdgmm::readlane_f64(sb.log_u, at), inv_s2 = sdgmm::readlane_f64(sb.inv_s2, at);
        const double cc = static_cast<double>(cf);
        const double S1 = sdgmm::readlane_f64(t, 0) * cc * inv_s2, S2 = sdgmm::readlane_f64(t, 32) * cc * cc * inv_s2;
        const double lr = (-S1 - 0.5 * S2) * p.inv_tau;
        reject = !(S2 == 0.0 || (lr == lr && lu <= fmin(0.0, lr)));            // a log-ratio that is not a number rejects
        const double f = cc * (1.0 + 2.0 * (S2 > 0.0 ? S1 / S2 : 0.0));
#pragma unroll
        for (int e = 0; e < E; ++e) {
          res[e] = reject ? static_cast<float>(static_cast<double>(dr[e]) -
                                               f * (static_cast<double>(d0[e]) - static_cast<double>(m[e]))) : dr[e];
          if (E * lane + e >= d) res[e] = 0.f;
        }
      }
      put(states, par, w, res);
      put(means, par, w, m);
    }
    if (lane == 0) verdict[par][w] = reject ? 1 : 0;
    expect(j + first + W < Kt ? n + pos + W : n + Kt + 1 + w);                 // where this wavefront goes if all are accepted
    draw_up_to(k0 + 2 * W + 2);
    __syncthreads();
    const int tested = max(0, min(W, Kt - j - first));                          // positions this round decided on
    const unsigned long long rejected = __ballot(lane < tested && verdict[par][lane & 7] != 0);
    bool window_ends = true;
    int adv = Kt;
    have_d0 = at_y = false;
    if (rejected != 0ull) {
      const int r = __builtin_ctzll(rejected);
      adv = j + first + r + 1;
      ++rejections;
      if (p.reused && n + adv < p.T) {             // the next window's frozen prediction
        have_d0 = true;
        if (p.carry_last) {
          get(means, par, r, d0);
        } else if (r + 1 < W) {                    // at the rejected draft: the next wavefront's state
          get(means, par, r + 1, d0);
        } else {                                   // nobody's: walk there once more
          if (w == 0) {
            float dr[E];
#pragma unroll
            for (int e = 0; e < E; ++e) dr[e] = y[e];
            for (int t = j; t < adv; ++t) draft(dr, n + t, dr);
            predict(dr, n + adv, m);
            put(means, par ^ 1, 0, m);
          }
          __syncthreads();
          get(means, par ^ 1, 0, d0);
          __syncthreads();                         // read before the next round writes there
        }
      }
      get(states, par, r, y);
    } else if (j + first + tested == Kt) {         // all accepted: the state behind the last draft
      if (tested < W && n + Kt < p.T) {            // and its prediction, if someone had it
        get(means, par, tested, d0);
        know_d0_at_y();
      }
      get(states, par, tested > 0 ? tested - 1 : 0, y);
    } else {                                       // the window goes on
      j += first + tested;
      get(states, par, tested - 1, y);
      have_d0 = true;
      window_ends = false;
    }
    par ^= 1;
    if (window_ends) {
      n += adv;
      j = 0;
      windows += 1;
      kt_sum += Kt;
    }
  }
  windows = max(windows, 1);                       // handed over at T: one window, of no positions, that keeps the state
  if (w > 0) return;
  float* o = p.out + id * d;
#pragma unroll
  for (int e = 0; e < E; ++e)
    if (E * lane + e < d) o[E * lane + e] = y[e];
  if (lane == 0) {
    if (p.counters) {
      if (n > n_start) atomicAdd(p.counters + 0, static_cast<unsigned long long>(n - n_start));
      atomicAdd(p.counters + 1, static_cast<unsigned long long>(windows));
      if (rejections) atomicAdd(p.counters + 2, static_cast<unsigned long long>(rejections));
      if (kt_sum) atomicAdd(p.counters + 4, static_cast<unsigned long long>(kt_sum));
    }
    atomicMax(p.longest, windows);
  }
}

__global__ void run_begin_kernel(int32_t* longest) { *longest = 0; }

// A batch stepped window by window makes as many windows as its longest chain.
__global__ void run_end_kernel(const int32_t* longest, unsigned long long* counters, int32_t* B_active) {
  if (counters) counters[3] += static_cast<unsigned long long>(*longest);
  *B_active = 0;
}

template <int E, int C>
void launch_rows(const GmmArgs& p, bool fine, dim3 grid, size_t shmem, hipStream_t st) {
  if (fine) hipLaunchKernelGGL((gmm_rows_kernel<E, C, true>), grid, dim3(64 * kRowsPerBlock), shmem, st, p);
  else hipLaunchKernelGGL((gmm_rows_kernel<E, C, false>), grid, dim3(64 * kRowsPerBlock), shmem, st, p);
}

struct GmmDenoiser final : sdden {
  sdgmm::Model g{};
  float* dev_f = nullptr;     // fp32 tables: row table, lane table and radii, or (more than 64 components) mu, sd, muT, sdT, ab
  double* dev_d = nullptr;    // cst [T,M], then (ab, sqrt(ab)) [T]
  bool lanes = false;         // at most 64 components: gmm_rows.h
  bool often_alone = false;   // gmm_run_kernel, ALONE
  const float *mu = nullptr, *sd = nullptr, *muT = nullptr, *sdT = nullptr, *ab = nullptr;
  ~GmmDenoiser() override {
    if (dev_f) (void)hipFree(dev_f);
    if (dev_d) (void)hipFree(dev_d);
  }
  int eval(int R, const float* X, const int32_t* krow, float* out, hipStream_t st) override {
    GmmArgs p;
    p.X = X; p.krow = krow; p.out = out; p.g = g;
    p.mu = mu; p.sd = sd; p.muT = muT; p.sdT = sdT; p.ab = ab;
    p.active = active; p.rows_per_chain = rows_per_chain; p.R = R;
    const dim3 grid(static_cast<unsigned>((R + kRowsPerBlock - 1) / kRowsPerBlock)), block(64 * kRowsPerBlock);
    prof.mark(1, st);
    if (g.M == 1) {
      hipLaunchKernelGGL(gmm_one_component_kernel, grid, block, 0, st, p);
    } else if (lanes) {
      const size_t shmem = sizeof(double) * kRowsPerBlock * (static_cast<size_t>(g.nslots) << (6 - g.lm));
      const bool fine = sdgmm::needs_fine(g.M, d, g.lm);
      if (d <= 64) launch_rows<1, 1>(p, fine, grid, shmem, st);
      else if (d <= 128) launch_rows<2, 1>(p, fine, grid, shmem, st);
      else if (d <= 256) launch_rows<4, 1>(p, fine, grid, shmem, st);
      else if (d <= 512) launch_rows<4, 2>(p, fine, grid, shmem, st);
      else if (d <= 1024) launch_rows<4, 4>(p, fine, grid, shmem, st);
      else hipLaunchKernelGGL((gmm_rows_kernel<4, 8, true>), grid, block, shmem, st, p);
    } else {
      const size_t shmem = sizeof(double) * kRowsPerBlock * static_cast<size_t>(g.M + d);
      hipLaunchKernelGGL(gmm_many_components_kernel, grid, block, shmem, st, p);
    }
    prof.mark(1, st);
    SD_HIP_TRY(err, hipGetLastError());
    return SD_OK;
  }
  int run(sdden* draft, sd_ctx* ctx, int B, const float* y, const int32_t* n, const int64_t* chain_id, const float* D_frozen,
          float* out, int32_t* B_active, int64_t* counters, hipStream_t st) override;
};

// ALONE and SHARES as the run needs them.
template <bool MAY_SHARE, class Launch>
void choose_run(bool alone, bool shares, Launch launch) {
  using std::true_type, std::false_type;
  if constexpr (MAY_SHARE) {
    if (shares) return alone ? launch(true_type{}, true_type{}) : launch(false_type{}, true_type{});
  }
  alone ? launch(true_type{}, false_type{}) : launch(false_type{}, false_type{});
}

template <int E, bool LDS, bool FINE = !LDS>
void launch_window_run(const RunArgs& p, bool alone, bool shares, unsigned block, size_t shmem, hipStream_t st) {
  choose_run<E == 1 && LDS>(alone, shares, [&](auto a, auto s) {
    hipLaunchKernelGGL((gmm_window_run_kernel<E, LDS, FINE, a(), s()>), dim3(static_cast<unsigned>(p.B)), dim3(block), shmem, st, p);
  });
}
template <int E, bool LDS, bool FINE>
hipError_t prepare_window_run() {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gmm_window_run_kernel<E, LDS, FINE, true, false>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 256);
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gmm_window_run_kernel<E, LDS, FINE, false, false>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 256);
  return e;
}

template <int E, int C, bool LDS, bool FINE = !LDS>
void launch_run(const RunArgs& p, bool indep, bool alone, bool shares, unsigned grid, unsigned block, size_t shmem, hipStream_t st) {
  choose_run<E * C == 1>(alone, shares, [&](auto a, auto s) {
    if (indep && grid == static_cast<unsigned>(p.B) && block == 128)        // a workgroup of two wavefronts per chain
      hipLaunchKernelGGL((gmm_run_kernel<E, C, LDS, true, FINE, a(), kPair, s()>), dim3(grid), dim3(block), shmem, st, p);
    else if (indep && p.B > 3 * 1024)      // a wavefront per chain, 1024 SIMDs
      hipLaunchKernelGGL((gmm_run_kernel<E, C, LDS, true, FINE, a(), E * C == 1 && a() ? kDense : kPlain, s()>), dim3(grid), dim3(block), shmem, st, p);
    else if (indep)
      hipLaunchKernelGGL((gmm_run_kernel<E, C, LDS, true, FINE, a(), kPlain, s()>), dim3(grid), dim3(block), shmem, st, p);
    else                                   // out of LDS one model has too many pairs per lane to share
      hipLaunchKernelGGL((gmm_run_kernel<E, C, LDS, false, FINE, a(), kPlain, LDS && s()>), dim3(grid), dim3(block), shmem, st, p);
  });
}

int GmmDenoiser::run(sdden* draft, sd_ctx* ctx, int B, const float* y, const int32_t* n, const int64_t* chain_id,
                     const float* D_frozen, float* out, int32_t* B_active, int64_t* counters, hipStream_t st) {
  const bool indep = ctx->mode == SD_DRAFT_EXPLICIT;
  GmmDenoiser* q = indep ? dynamic_cast<GmmDenoiser*>(draft) : nullptr;
  // what needs the separate calls: more than 64 components, kernels timed one by one, a batch size kept on the device
  if (!lanes || prof.which || active || ctx->active || (indep && (!q || !q->lanes || q->prof.which || q->active)))
    return sdi::fail(err, SD_ERR_UNSUPPORTED, "sdden_run: this denoiser's chains run window by window");
  RunArgs p{};
  p.t = g;
  if (q) p.q = q->g;
  p.y = y; p.n = n; p.id = chain_id; p.Dfz = D_frozen; p.out = out;
  p.a = ctx->dev_a; p.c = ctx->dev_c; p.sigma = ctx->dev_sigma;
  p.B = B; p.K = ctx->K; p.T = ctx->T; p.seed = ctx->seed; p.inv_tau = 1.0 / ctx->tau;
  p.reused = ctx->mode == SD_DRAFT_FROZEN_REUSED;
  p.carry_last = ctx->carry_rule == SD_CARRY_LAST_ACCEPTED;
  p.counters = reinterpret_cast<unsigned long long*>(counters);
  p.longest = ctx->dev_queue + 1;
  // Few chains: a workgroup each, spread over the CUs.  From 1024 on two, from 2048 on four share a workgroup and its table.
  // The two models of the independent drafter take a wavefront each while there are no more than two per SIMD; us of 60 steps
  // with / without at 1, 300 and 1000 chains: d = 75, M = 12 180 / 228, 218 / 246, 221 / 256; d = 180, M = 40 578 / 767,
  // 752 / 800, 756 / 809.
  const bool pair = indep && B <= 1024;
  const int waves = pair ? 2 : B >= 2048 ? 4 : (B >= 1024 ? 2 : 1);
  const unsigned grid = static_cast<unsigned>(pair ? B : (B + waves - 1) / waves), block = 64u * waves;
  size_t npad = static_cast<size_t>(g.nslots) << (6 - g.lm), slots = g.nslots;
  if (q) {
    npad = std::max(npad, static_cast<size_t>(q->g.nslots) << (6 - q->g.lm));
    slots += q->g.nslots;
  }
  npad = (npad + 1) / 2 * 2;
  // The tables go to LDS as fp64 (no conversion and no square per pair) while four workgroups still fit a CU.
  const size_t table = sizeof(double2) * sdgmm::kTabStride * slots, xs = (sizeof(double) * npad + (d <= 128 ? 1024 : 0)) * waves;
  const bool lds = d <= 256 && table <= 36 * 1024;
  const int per_lane = d <= 64 ? 1 : d <= 128 ? 2 : d <= 256 ? 4 : d <= 512 ? 8 : d <= 1024 ? 16 : 32;
  const size_t shmem = xs + (lds ? table : 0) + (pair ? 1024 * static_cast<size_t>(per_lane) : 0);
  hipLaunchKernelGGL(run_begin_kernel, dim3(1), dim3(1), 0, st, p.longest);
  // a table that fits LDS has at most 32 pairs per lane, and at d > 64 at most 32 components too
  const bool fine = g.M > 32 || (q && q->g.M > 32);
  // Few chains, frozen prediction: gmm_window_run_kernel with as many wavefronts a chain as a window has positions (and its
  // next start), up to two per SIMD; us of 100 steps in it / one wavefront a chain at 1, 256 and 1000 chains: d = 2, M = 8, K = 4
  // 107 / 156, 121 / 168, 199 / 210; d = 60, M = 20, K = 8 128 / 194, 172 / 237, 260 / 282 (with four per SIMD 286).
  const int useful = p.K + p.reused;
  int W = indep || d > 256 || p.K < 2 ? 1 : useful >= 6 ? 8 : useful >= 3 ? 4 : 2;
  while (W > 1 && static_cast<int64_t>(B) * W > 2048) W /= 2;
  const int row = d <= 64 ? 64 : d <= 128 ? 128 : 256;
  int sh = row == 256 ? 0 : 6;             // log2 of the steps whose noise one pass draws
  while (row < 256 && (256 >> sh) < d) --sh;
  const size_t wshmem = (lds ? table : 0) + sizeof(double) * npad * W + sizeof(float) * (4 * W * row + 256 * (((2 * W + 1) >> sh) + 2));
  // where a lane has one coordinate: one pair per lane, or enough components that more than two per pair can be live
  auto may_share = [](const sdgmm::Model& m) { return m.nslots == 1 || m.M > 2 * m.nslots; };
  const bool shares = may_share(g) || (q && may_share(q->g));
  if (B == 0) {}                           // no chains: the end kernel leaves the count
  else if (W > 1 && lds && fine) launch_window_run<1, true, true>(p, often_alone, shares, 64 * W, wshmem, st);
  else if (W > 1 && lds && d <= 64) launch_window_run<1, true>(p, often_alone, shares, 64 * W, wshmem, st);
  else if (W > 1 && lds && d <= 128) launch_window_run<2, true>(p, often_alone, shares, 64 * W, wshmem, st);
  else if (W > 1 && lds) launch_window_run<4, true>(p, often_alone, shares, 64 * W, wshmem, st);
  else if (W > 1 && d <= 64) launch_window_run<1, false>(p, often_alone, shares, 64 * W, wshmem, st);
  else if (W > 1 && d <= 128) launch_window_run<2, false>(p, often_alone, shares, 64 * W, wshmem, st);
  else if (W > 1) launch_window_run<4, false>(p, often_alone, shares, 64 * W, wshmem, st);
  else if (lds && fine) launch_run<1, 1, true, true>(p, indep, often_alone, shares, grid, block, shmem, st);
  else if (lds && d <= 64) launch_run<1, 1, true>(p, indep, often_alone, shares, grid, block, shmem, st);
  else if (lds && d <= 128) launch_run<2, 1, true>(p, indep, often_alone, shares, grid, block, shmem, st);
  else if (lds) launch_run<4, 1, true>(p, indep, often_alone, shares, grid, block, shmem, st);
  else if (d <= 64) launch_run<1, 1, false>(p, indep, often_alone, shares, grid, block, shmem, st);
  else if (d <= 128) launch_run<2, 1, false>(p, indep, often_alone, shares, grid, block, shmem, st);
  else if (d <= 256) launch_run<4, 1, false>(p, indep, often_alone, shares, grid, block, shmem, st);
  else if (d <= 512) launch_run<4, 2, false>(p, indep, often_alone, shares, grid, block, shmem, st);
  else if (d <= 1024) launch_run<4, 4, false>(p, indep, often_alone, shares, grid, block, shmem, st);
  else launch_run<4, 8, false>(p, indep, often_alone, shares, grid, block, shmem, st);
  hipLaunchKernelGGL(run_end_kernel, dim3(1), dim3(1), 0, st, p.longest, p.counters, B_active);
  SD_HIP_TRY(err, hipGetLastError());
  return SD_OK;
}

}  // namespace

extern "C" {

int sdden_gmm_create(int32_t M, int32_t d, const float* means, const float* stds, const float* logw,
                     int32_t T, const float* alpha_bar_state, sdden** out) {
  std::string& E = sdi::g_den_create_error;
  if (!means || !stds || !logw || !alpha_bar_state || !out || M <= 0 || d <= 0 || T <= 0)
    return sdi::fail(E, SD_ERR_ARG, "sdden_gmm_create: bad argument");
  if (static_cast<size_t>(M + d) * sizeof(double) * kRowsPerBlock > 60000)
    return sdi::fail(E, SD_ERR_UNSUPPORTED, "sdden_gmm_create: M+d=%d too large for the LDS staging", M + d);
  const size_t md = static_cast<size_t>(M) * d;
  for (size_t i = 0; i < md; ++i)
    if (!(stds[i] > 0.f)) return sdi::fail(E, SD_ERR_ARG, "sdden_gmm_create: stds must be > 0");
  const bool lanes = M <= sdgmm::kMaxLaneComponents;
  int lm = 0;                                                // lanes per component: 64 / (M rounded up to a power of two)
  while (lm < 6 && (1 << lm) < M) ++lm;
  const int parts = 64 >> lm;
  int nslots = (d + parts - 1) / parts;
  if (nslots > 2) nslots = (nslots + 3) / 4 * 4;             // whole groups of four pairs
  std::vector<float> h;
  std::vector<double> dbl(static_cast<size_t>(T) * M + 1 + 2 * static_cast<size_t>(T));
  const size_t step_off = (static_cast<size_t>(T) * M + 1) / 2 * 2;       // 16-byte aligned
  if (lanes) {
    h.resize(2 * md + 128 * static_cast<size_t>(nslots) + static_cast<size_t>(T) * M + 1);
    for (size_t i = 0; i < md; ++i) {
      h[2 * i] = means[i];
      h[2 * i + 1] = stds[i];
    }
    for (int j = 0; j < nslots; ++j)
      for (int lane = 0; lane < 64; ++lane) {
        const int m = lane >> (6 - lm), i = (lane & (parts - 1)) + parts * j;
        const bool has = m < M && i < d;
        float* slot = h.data() + 2 * md + 2 * (static_cast<size_t>(j) * 64 + lane);
        slot[0] = has ? means[m * static_cast<size_t>(d) + i] : 0.f;
        slot[1] = has ? stds[m * static_cast<size_t>(d) + i] : 1.f;
      }
  } else {
    h.resize(4 * md + T + 1);
    for (int m = 0; m < M; ++m)
      for (int i = 0; i < d; ++i) {
        const float mu = means[m * static_cast<size_t>(d) + i], s = stds[m * static_cast<size_t>(d) + i];
        h[m * static_cast<size_t>(d) + i] = mu;
        h[md + m * static_cast<size_t>(d) + i] = s;
        h[2 * md + i * static_cast<size_t>(M) + m] = mu;
        h[3 * md + i * static_cast<size_t>(M) + m] = s;
      }
    for (int k = 0; k <= T; ++k) h[4 * md + k] = alpha_bar_state[k];
  }
  for (int k = 0; k < T; ++k) {
    const double ab = alpha_bar_state[k];
    for (int m = 0; m < M; ++m) {
      double ld = 0.0;
      for (int i = 0; i < d; ++i) {
        const double sd = stds[m * static_cast<size_t>(d) + i];
        ld += std::log(ab * sd * sd + (1.0 - ab));
      }
      dbl[static_cast<size_t>(k) * M + m] = static_cast<double>(logw[m]) - 0.5 * ld;
    }
    dbl[step_off + 2 * k] = ab;
    dbl[step_off + 2 * k + 1] = std::sqrt(ab);
  }
  GmmDenoiser* g = new (std::nothrow) GmmDenoiser;
  if (!g) return sdi::fail(E, SD_ERR_ARG, "sdden_gmm_create: out of host memory");
  g->d = d; g->T = T; g->lanes = lanes;
  hipError_t e = hipMalloc(&g->dev_f, h.size() * sizeof(float));
  if (e == hipSuccess) e = hipMalloc(&g->dev_d, dbl.size() * sizeof(double));
  if (e == hipSuccess) e = hipMemcpy(g->dev_f, h.data(), h.size() * sizeof(float), hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(g->dev_d, dbl.data(), dbl.size() * sizeof(double), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    delete g;
    return sdi::fail(E, SD_ERR_HIP, "sdden_gmm_create: %s", hipGetErrorString(e));
  }
  g->g.M = M; g->g.d = d; g->g.T = T; g->g.lm = lm; g->g.nslots = nslots;
  g->g.cst = g->dev_d;
  g->g.steps = reinterpret_cast<const double2*>(g->dev_d + step_off);
  if (lanes) {
    g->g.row_tab = reinterpret_cast<const float2*>(g->dev_f);
    g->g.lane_tab = reinterpret_cast<const float2*>(g->dev_f + 2 * md);
    float* radius2 = g->dev_f + 2 * md + 128 * static_cast<size_t>(nslots);
    g->g.radius2 = radius2;
    const unsigned grid = static_cast<unsigned>((static_cast<int64_t>(T) * M + kRowsPerBlock - 1) / kRowsPerBlock);
    int32_t* count = reinterpret_cast<int32_t*>(radius2 + static_cast<size_t>(T) * M);      // 0 by the copy above
    int32_t holds = 0;
    hipLaunchKernelGGL(gmm_radius_kernel, dim3(grid), dim3(64 * kRowsPerBlock), 0, nullptr, g->g, radius2, count);
    e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpy(&holds, count, sizeof(holds), hipMemcpyDeviceToHost);
    if (e != hipSuccess) {
      delete g;
      return sdi::fail(E, SD_ERR_HIP, "sdden_gmm_create: %s", hipGetErrorString(e));
    }
    // LDS of more than 64 KiB: up to 72 at d = 128, up to 104 at d = 256; rows of up to 64 need 56 at most
    if (d > 128 && d <= 256) {
      e = prepare_window_run<4, true, false>();
      if (e == hipSuccess) e = prepare_window_run<4, false, true>();
    } else if (d > 64 && d <= 128) {
      e = prepare_window_run<2, true, false>();
      if (e == hipSuccess) e = prepare_window_run<2, false, true>();
    }
    if (e != hipSuccess) {
      delete g;
      return sdi::fail(E, SD_ERR_HIP, "sdden_gmm_create: %s", hipGetErrorString(e));
    }
    g->often_alone = static_cast<double>(holds) >= (nslots >= 24 ? 0.35 : 0.45) * static_cast<double>(T) * M;
  } else {
    g->mu = g->dev_f; g->sd = g->dev_f + md; g->muT = g->dev_f + 2 * md; g->sdT = g->dev_f + 3 * md; g->ab = g->dev_f + 4 * md;
  }
  *out = g;
  return SD_OK;
}

int sdden_eval(sdden* den, int32_t R, const float* X, const int32_t* krow, float* out, void* stream) {
  if (!den) return SD_ERR_ARG;
  if (R < 0 || (R > 0 && (!X || !krow || !out))) return sdi::fail(den->err, SD_ERR_ARG, "sdden_eval: bad argument");
  if (R == 0) return SD_OK;
  den->prof.cur_rows = R;
  return den->eval(R, X, krow, out, static_cast<hipStream_t>(stream));
}

int sdden_run(sdden* den, sdden* draft_den, sd_ctx* ctx, int32_t B, const float* y, const int32_t* n, const int64_t* chain_id,
              const float* D_frozen, float* out, int32_t* B_active, int64_t* counters, void* stream) {
  if (!den || !ctx) return SD_ERR_ARG;
  if (B < 0 || !B_active || (ctx->mode == SD_DRAFT_EXPLICIT && !draft_den) ||
      (B > 0 && (!y || !n || !chain_id || !out || (ctx->mode == SD_DRAFT_FROZEN_REUSED && !D_frozen))))
    return sdi::fail(den->err, SD_ERR_ARG, "sdden_run: bad argument");
  const bool indep = ctx->mode == SD_DRAFT_EXPLICIT;
  if (den->d != ctx->d || (indep && draft_den->d != ctx->d))
    return sdi::fail(den->err, SD_ERR_ARG, "sdden_run: denoiser and context describe chains of different sizes");
  // steps the denoiser does not have: sdden_eval masks their rows, the loop goes on with what the buffers hold
  if (den->T < ctx->T || (indep && draft_den->T < ctx->T))
    return sdi::fail(den->err, SD_ERR_UNSUPPORTED, "sdden_run: the denoiser has fewer steps than the chains");
  return den->run(draft_den, ctx, B, y, n, chain_id, D_frozen, out, B_active, counters, static_cast<hipStream_t>(stream));
}

int sdden_eval_mirror(sdden* den, int32_t R, const float* X, const uint16_t* Xbf16, const int32_t* krow, float* out,
                      void* stream) {
  if (!den) return SD_ERR_ARG;
  if (R < 0 || (R > 0 && (!X || !Xbf16 || !krow || !out)))
    return sdi::fail(den->err, SD_ERR_ARG, "sdden_eval_mirror: bad argument");
  if (R == 0) return SD_OK;
  den->prof.cur_rows = R;
  return den->eval_mirror(R, X, Xbf16, krow, out, static_cast<hipStream_t>(stream));
}

int sdden_reserve(sdden* den, int32_t Rmax) {
  if (!den) return SD_ERR_ARG;
  if (Rmax <= 0) return sdi::fail(den->err, SD_ERR_ARG, "sdden_reserve: Rmax must be > 0");
  return den->reserve(Rmax);
}

int sdden_profile(sdden* den, int32_t which) {
  if (!den || which < 0) return SD_ERR_ARG;
  den->prof.which = which;
  den->prof.used = 0;
  return SD_OK;
}

int sdden_profile_min_rows(sdden* den, int32_t min_rows) {
  if (!den || min_rows < 0) return SD_ERR_ARG;
  den->prof.min_rows = min_rows;
  return SD_OK;
}

int sdden_profile_collect(sdden* den, double* total_ms, int64_t* launches) {
  if (!den || !total_ms || !launches) return SD_ERR_ARG;
  sdden_profiler& pr = den->prof;
  double tot = 0.0;
  const size_t pairs = pr.used / 2;
  if (pairs) SD_HIP_TRY(den->err, hipEventSynchronize(pr.events[2 * pairs - 1]));
  for (size_t i = 0; i < pairs; ++i) {
    float ms = 0.f;
    SD_HIP_TRY(den->err, hipEventElapsedTime(&ms, pr.events[2 * i], pr.events[2 * i + 1]));
    tot += ms;
  }
  *total_ms = tot;
  *launches = static_cast<int64_t>(pairs);
  pr.used = 0;
  return SD_OK;
}

int sdden_set_active_count(sdden* den, const int32_t* count, int32_t rows_per_chain) {
  if (!den) return SD_ERR_ARG;
  if (count && rows_per_chain <= 0) return sdi::fail(den->err, SD_ERR_ARG, "sdden_set_active_count: rows_per_chain must be > 0");
  den->active = count;
  den->rows_per_chain = count ? rows_per_chain : 1;
  return SD_OK;
}

int sdden_destroy(sdden* den) {
  if (!den) return SD_ERR_ARG;
  delete den;
  return SD_OK;
}

const char* sdden_last_error(const sdden* den) {
  return den ? den->err.c_str() : sdi::g_den_create_error.c_str();
}

}  // extern "C"
