// E[x0 | x_t] for x0 ~ N(mu, U U^T + s2 I): the closed-form linear denoiser of the image-shaped
// linear-Gaussian workload, evaluated for all rows of a batched target call with two skinny
// fp32 GEMMs (paper: the target is queried on all drafted states of a window in one batch,
// Alg. "Speculative Sampling for DDM", (Par.) line).
//
// In the eigenbasis Q (d x r, orthonormal columns) of U U^T = Q diag(lam) Q^T the posterior-mean
// map G = sqrt(ab) S (ab S + (1-ab) I)^-1, S = U U^T + s2 I, is diagonal:
//   G = g_perp I + Q diag(g_i - g_perp) Q^T,  g_i = sqrt(ab)(lam_i+s2)/(ab(lam_i+s2)+1-ab),
//                                            g_perp = sqrt(ab) s2/(ab s2+1-ab),
//   D(x,k) = mu + G (x - sqrt(ab) mu)
//          = g_perp x + (1 - sqrt(ab) g_perp) mu + Q [ (g - g_perp) .* (Q^T x - sqrt(ab) Q^T mu) ].
// GEMM 1: P = X Q with the bracket applied per row in the epilogue (each row has its own step k);
// GEMM 2: out = P' Q^T + g_perp(k) x + (1 - sqrt(ab_k) g_perp(k)) mu.
//
// Both products go through lowrank_gemm.h: bf16 matrix instructions on operands split into three pieces, the first one
// split over K into slabs that a small kernel adds and scales.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <vector>

#include "lowrank_gemm.h"
#include "sdden_internal.h"
#include "sdden_rows.h"

namespace {

constexpr int kDimStep = 16;      // d: whole 16-column blocks

// Cyclic Jacobi eigen-decomposition of a symmetric n x n matrix (fp64, host).
// On return A's diagonal holds the eigenvalues and V's columns the eigenvectors.
void jacobi_eigen(std::vector<double>& A, std::vector<double>& V, int n) {
  V.assign(static_cast<size_t>(n) * n, 0.0);
  for (int i = 0; i < n; ++i) V[static_cast<size_t>(i) * n + i] = 1.0;
  for (int sweep = 0; sweep < 60; ++sweep) {
    double off = 0.0, diag = 0.0;
    for (int i = 0; i < n; ++i)
      for (int j = 0; j < n; ++j) (i == j ? diag : off) += A[static_cast<size_t>(i) * n + j] * A[static_cast<size_t>(i) * n + j];
    if (off <= 1e-30 * diag) break;
    for (int p = 0; p < n - 1; ++p)
      for (int q = p + 1; q < n; ++q) {
        const double apq = A[static_cast<size_t>(p) * n + q];
        if (apq == 0.0) continue;
        const double app = A[static_cast<size_t>(p) * n + p], aqq = A[static_cast<size_t>(q) * n + q];
        const double theta = (aqq - app) / (2.0 * apq);
        const double tt = (theta >= 0 ? 1.0 : -1.0) / (std::fabs(theta) + std::sqrt(theta * theta + 1.0));
        const double c = 1.0 / std::sqrt(tt * tt + 1.0), s = tt * c;
        for (int k = 0; k < n; ++k) {                       // columns p, q
          const double akp = A[static_cast<size_t>(k) * n + p], akq = A[static_cast<size_t>(k) * n + q];
          A[static_cast<size_t>(k) * n + p] = c * akp - s * akq;
          A[static_cast<size_t>(k) * n + q] = s * akp + c * akq;
        }
        for (int k = 0; k < n; ++k) {                       // rows p, q
          const double apk = A[static_cast<size_t>(p) * n + k], aqk = A[static_cast<size_t>(q) * n + k];
          A[static_cast<size_t>(p) * n + k] = c * apk - s * aqk;
          A[static_cast<size_t>(q) * n + k] = s * apk + c * aqk;
        }
        for (int k = 0; k < n; ++k) {
          const double vkp = V[static_cast<size_t>(k) * n + p], vkq = V[static_cast<size_t>(k) * n + q];
          V[static_cast<size_t>(k) * n + p] = c * vkp - s * vkq;
          V[static_cast<size_t>(k) * n + q] = s * vkp + c * vkq;
        }
      }
  }
}

// One instantiation of the product kernel and whether it also compacts the rows.
#define SD_LR_SHAPES(X)                                                                            \
  X(1, 2, 2, 4, 4, 2, false) X(1, 2, 2, 2, 2, 2, false) X(1, 2, 1, 1, 2, 4, false) X(1, 1, 1, 1, 1, 6, false) \
  X(1, 2, 2, 2, 2, 2, true) X(1, 2, 1, 1, 2, 4, true) X(1, 1, 1, 1, 1, 6, true)                    \
  X(2, 2, 2, 2, 4, 2, false) X(2, 2, 2, 2, 2, 3, false) X(2, 2, 1, 1, 2, 4, false) X(2, 1, 1, 1, 1, 6, false)

int64_t tiles(int R, int N, int bm, int bn) { return static_cast<int64_t>((R + bm - 1) / bm) * ((N + bn - 1) / bn); }

struct LowRankDenoiser final : sdden {
  int r = 0, rpad = 0;          // rank, rank padded to a multiple of a slice (extra columns are zero)
  int nk = 0;                   // slices of the first product's contraction: ceil(d / 32)
  float* dev = nullptr;         // all float tables in one allocation
  unsigned char* wdev = nullptr;   // Q and Q^T as split blocks
  unsigned char *wQ = nullptr, *wQT = nullptr;
  float *gain = nullptr, *sab = nullptr, *gperp = nullptr, *coef = nullptr, *qmu = nullptr, *mu = nullptr;
  // per-call scratch, sized by sdden_reserve
  int32_t* rowidx = nullptr;
  int32_t* count = nullptr;
  unsigned char* P = nullptr;   // the second product's A as split blocks, whole row tiles
  float* part = nullptr;        // K-split partial sums of the first product, one slab of R rows per K range
  lrgemm::RowInfo* rowinfo = nullptr;   // per compacted row: source row and the second product's per-row scalars
  int nsplit = 1;               // K split of the first product: fixed per denoiser, so that the order in which a
                                // prediction's terms are added never depends on how many rows a call carries
  int cap_rows = 0;

  void free_scratch() {
    if (rowidx) (void)hipFree(rowidx);
    if (P) (void)hipFree(P);
    if (part) (void)hipFree(part);
    if (rowinfo) (void)hipFree(rowinfo);
    rowidx = nullptr; P = nullptr; part = nullptr; rowinfo = nullptr; cap_rows = 0;
  }

  ~LowRankDenoiser() override {
    free_scratch();
    if (dev) (void)hipFree(dev);
    if (wdev) (void)hipFree(wdev);
    if (count) (void)hipFree(count);
  }

  int reserve(int R) override {
    if (R <= cap_rows) return SD_OK;
    free_scratch();
    const size_t rows = static_cast<size_t>(R), whole = (rows + lrgemm::kRowTile - 1) / lrgemm::kRowTile * lrgemm::kRowTile;
    SD_HIP_TRY(err, hipMalloc(&rowidx, sizeof(int32_t) * rows));
    SD_HIP_TRY(err, hipMalloc(&P, whole / 16 * (rpad / lrgemm::BK) * lrgemm::kBlockBytes));
    SD_HIP_TRY(err, hipMalloc(&part, sizeof(float) * nsplit * rows * rpad));
    SD_HIP_TRY(err, hipMalloc(&rowinfo, sizeof(lrgemm::RowInfo) * rows));
    if (!count) SD_HIP_TRY(err, hipMalloc(&count, sizeof(int32_t)));
    cap_rows = R;
    return SD_OK;
  }

  int eval(int R, const float* X, const int32_t* krow, float* out, hipStream_t st) override {
    if (!sdi::aligned16(X)) return sdi::fail(err, SD_ERR_ARG, "sdden_eval(lowrank): X must be 16-byte aligned");
    if (R > cap_rows)
      return sdi::fail(err, SD_ERR_WORKSPACE, "sdden_eval(lowrank): %d rows exceed the %d reserved (sdden_reserve)", R, cap_rows);
    // Tiles: the largest that still gives every CU work, two workgroups each for the 128 x 128 one (80 KiB of LDS, two
    // per CU).  Measured back to back on one set of rows, us, K split 4 (d = 3072, r = 256; inside a pass, where the rows
    // come from HBM, the first product takes 34 to 37 at 2048 rows):
    //   first product   20480 rows 128x128 166, 64x64 195    2048 rows 44 / 26    512 rows 64x64 19, 32x32 16, 16x16 23
    //                   133 rows 64x64 18, 32x32 13, 16x16 11
    //   (18000 rows, r = 160, where a second 128-column tile is mostly padding: 128x128 147, 64x64 136)
    //   second product  20480 rows 64x128 231, 64x64 250     2048 rows 27 / 25    512 rows 64x64 11, 32x32 13
    //                   133 rows 64x64 7.6, 32x32 6.6, 16x16 9.1; at d = 1104, r = 64: 4.7, 4.0, 3.9
    // Up to kRankRows rows every workgroup finds its rows itself (+1 us) in place of a compaction launch (5 us).
    const int s1 = 5 * rpad > 4 * 128 * ((rpad + 127) / 128) && tiles(R, rpad, 128, 128) * nsplit >= 512 ? 0
                   : tiles(R, rpad, 64, 64) * nsplit >= 256              ? 1
                   : tiles(R, rpad, 32, 32) * nsplit >= 256              ? 2
                                                                         : 3;
    const int s2 = tiles(R, d, 64, 128) >= 2048 ? 0 : tiles(R, d, 64, 64) >= 256 ? 1 : tiles(R, d, 32, 32) >= 256 ? 2 : 3;
    const bool rank = R <= lrgemm::kRankRows && s1 > 0;
    if (!rank)
      hipLaunchKernelGGL(sdrows::compact_rows_kernel, dim3(sdrows::compact_rows_grid(R)), dim3(sdrows::kScan), 0, st, krow, rowidx,
                         count, active, rows_per_chain, R, T);
    // part_s = X[rowidx] Q over K range s, then P' = gain .* (sum_s part_s - sab qmu)
    lrgemm::Args a{};
    a.A = X; a.d = d; a.Bt = wQT; a.N = rpad; a.nk = nk; a.count = count; a.rowidx = rowidx;
    a.krow = krow; a.active = active; a.rows_per_chain = rows_per_chain; a.R = R; a.T = T;
    a.part = part; a.slab_stride = static_cast<int64_t>(R) * rpad;
    prof.mark(1, st);
    hipError_t e = s1 == 0 ? lrgemm::launch<2, 2, 4, 4, 2, 1, false>(a, R, nsplit, st)
                   : rank  ? (s1 == 1   ? lrgemm::launch<2, 2, 2, 2, 2, 1, true>(a, R, nsplit, st)
                              : s1 == 2 ? lrgemm::launch<2, 1, 1, 2, 4, 1, true>(a, R, nsplit, st)
                                        : lrgemm::launch<1, 1, 1, 1, 6, 1, true>(a, R, nsplit, st))
                           : (s1 == 1   ? lrgemm::launch<2, 2, 2, 2, 2, 1, false>(a, R, nsplit, st)
                              : s1 == 2 ? lrgemm::launch<2, 1, 1, 2, 4, 1, false>(a, R, nsplit, st)
                                        : lrgemm::launch<1, 1, 1, 1, 6, 1, false>(a, R, nsplit, st));
    SD_HIP_TRY(err, e);
    prof.mark(1, st);
    lrgemm::Args b{};
    b.A = P; b.d = d; b.Bt = wQ; b.N = d; b.nk = rpad / lrgemm::BK; b.count = count;
    b.rowinfo = rowinfo; b.X = X; b.out = out; b.out_aligned = sdi::aligned16(out); b.mu = mu;
    // out = P' Q^T + gperp x + coef mu
    // The reduction inside the second product is done again by every column tile, a thread per row and eight columns at a time:
    // ahead of its launch at ranks of up to 64 while a row's slabs hold 512 floats and all tiles' 16 MB at most.  us a call, inside / by a launch: d = 1104,
    // r = 50 1 row 11.9 / 13.6, 133 rows 13.1 / 14.0; d = 512, r = 30 133 rows 10.3 / 13.3; but d = 3072, r = 50 (768 floats) 13 rows
    // 14.0 / 13.5, 250 rows (73 MB) 21.3 / 16.6; d = 2000, r = 100 40 rows 14.9 / 14.5; d = 3072, r = 200 1 row 23.3 / 17.6.
    const int fm = s2 == 2 ? 32 : 16;
    const bool fused = s2 >= 2 && rpad <= 64 && rpad * nsplit <= 512 && tiles(R, d, fm, fm) * fm * rpad * nsplit * 4 <= (16 << 20);
    if (fused) {
      b.rowidx = rowidx; b.krow = krow; b.part = part; b.slab_stride = a.slab_stride; b.nsplit = nsplit;
      b.gain = gain; b.sab = sab; b.qmu = qmu; b.gperp = gperp; b.coef = coef;
      prof.mark(2, st);
      e = s2 == 2 ? lrgemm::launch_fused<2, 1, 1, 2, 4>(b, R, st) : lrgemm::launch_fused<1, 1, 1, 1, 6>(b, R, st);
    } else {
      const int64_t octs = static_cast<int64_t>(R) * (rpad / 8);
      hipLaunchKernelGGL(lrgemm::reduce_gain_kernel, dim3(static_cast<unsigned>((octs + 255) / 256)), dim3(256), 0, st, part,
                         a.slab_stride, nsplit, count, rowidx, krow, gain, sab, qmu, P, rpad, gperp, coef, rowinfo);
      prof.mark(2, st);
      e = s2 == 0   ? lrgemm::launch<2, 2, 2, 4, 2, 2, false>(b, R, 1, st)
          : s2 == 1 ? lrgemm::launch<2, 2, 2, 2, 3, 2, false>(b, R, 1, st)
          : s2 == 2 ? lrgemm::launch<2, 1, 1, 2, 4, 2, false>(b, R, 1, st)
                    : lrgemm::launch<1, 1, 1, 1, 6, 2, false>(b, R, 1, st);
    }
    SD_HIP_TRY(err, e);
    prof.mark(2, st);
    SD_HIP_TRY(err, hipGetLastError());
    return SD_OK;
  }
};

// One weight as three bf16 (round to nearest even; |q| <= 1 here), whose sum is within 2^-25 of it.
void split_weight(float q, uint16_t (&piece)[3]) {
  for (int i = 0; i < 3; ++i) {
    uint32_t u;
    std::memcpy(&u, &q, 4);
    u = (u + 0x7fffu + ((u >> 16) & 1u)) & 0xffff0000u;
    piece[i] = static_cast<uint16_t>(u >> 16);
    float f;
    std::memcpy(&f, &u, 4);
    q -= f;
  }
}

void store_split(uint16_t* blocks, int row, int k, int nk, const uint16_t (&piece)[3]) {
  uint16_t* at = blocks + lrgemm::block_offset(row, k & ~7, nk) / 2 + (k & 7);
  at[0] = piece[0]; at[512] = piece[1]; at[1024] = piece[2];
}

}  // namespace

extern "C" int sdden_lowrank_create(int32_t d, int32_t r, const float* mu, const float* U, float s2, int32_t T,
                                    const float* alpha_bar_state, sdden** out) {
  std::string& E = sdi::g_den_create_error;
  if (!mu || !U || !alpha_bar_state || !out || d <= 0 || r <= 0 || T <= 0 || !(s2 > 0.f))
    return sdi::fail(E, SD_ERR_ARG, "sdden_lowrank_create: bad argument");
  if (d % kDimStep != 0)
    return sdi::fail(E, SD_ERR_UNSUPPORTED, "sdden_lowrank_create: d=%d must be a multiple of %d", d, kDimStep);
  const int rpad = ((r + lrgemm::BK - 1) / lrgemm::BK) * lrgemm::BK;     // whole slices
  // Gram matrix G = U^T U (r x r), its eigen-decomposition, and Q = U V diag(lam^-1/2)
  std::vector<double> G(static_cast<size_t>(r) * r, 0.0), V;
  for (int i = 0; i < d; ++i) {
    const float* row = U + static_cast<size_t>(i) * r;
    for (int a = 0; a < r; ++a) {
      const double ua = row[a];
      for (int b = a; b < r; ++b) G[static_cast<size_t>(a) * r + b] += ua * row[b];
    }
  }
  for (int a = 0; a < r; ++a)
    for (int b = 0; b < a; ++b) G[static_cast<size_t>(a) * r + b] = G[static_cast<size_t>(b) * r + a];
  double trace = 0.0;
  for (int a = 0; a < r; ++a) trace += G[static_cast<size_t>(a) * r + a];
  jacobi_eigen(G, V, r);
  std::vector<double> lam(r), scale(r);
  for (int a = 0; a < r; ++a) {
    lam[a] = G[static_cast<size_t>(a) * r + a];
    if (lam[a] > 1e-12 * trace) scale[a] = 1.0 / std::sqrt(lam[a]);
    else { lam[a] = 0.0; scale[a] = 0.0; }                 // rank-deficient direction: no gain there
  }
  const int nk = (d + lrgemm::BK - 1) / lrgemm::BK;
  const size_t bytes_QT = static_cast<size_t>(rpad / 16) * nk * lrgemm::kBlockBytes;                  // rows: rank, k: d
  const size_t bytes_Q = static_cast<size_t>(d / 16) * (rpad / lrgemm::BK) * lrgemm::kBlockBytes;     // rows: d, k: rank
  std::vector<uint16_t> hw((bytes_QT + bytes_Q) / 2, 0);
  std::vector<float> h(static_cast<size_t>(T) * rpad + 3 * static_cast<size_t>(T) + rpad + d, 0.f);
  float* hgain = h.data();
  float* hsab = hgain + static_cast<size_t>(T) * rpad; float* hgperp = hsab + T; float* hcoef = hgperp + T;
  float* hqmu = hcoef + T; float* hmu = hqmu + rpad;
  std::vector<double> qmu(r, 0.0), qrow(r);
  for (int i = 0; i < d; ++i) {
    const float* urow = U + static_cast<size_t>(i) * r;
    for (int a = 0; a < r; ++a) qrow[a] = 0.0;
    for (int b = 0; b < r; ++b) {
      const double ub = urow[b];
      const double* vrow = V.data() + static_cast<size_t>(b) * r;
      for (int a = 0; a < r; ++a) qrow[a] += ub * vrow[a];
    }
    for (int a = 0; a < r; ++a) {
      const double q = qrow[a] * scale[a];
      uint16_t piece[3];
      split_weight(static_cast<float>(q), piece);
      store_split(hw.data(), a, i, nk, piece);
      store_split(hw.data() + bytes_QT / 2, i, a, rpad / lrgemm::BK, piece);
      qmu[a] += q * mu[i];
    }
    hmu[i] = mu[i];
  }
  for (int a = 0; a < r; ++a) hqmu[a] = static_cast<float>(qmu[a]);
  for (int k = 0; k < T; ++k) {
    const double ab = alpha_bar_state[k], sab = std::sqrt(ab), om = 1.0 - ab;
    const double gp = sab * s2 / (ab * s2 + om);
    hsab[k] = static_cast<float>(sab);
    hgperp[k] = static_cast<float>(gp);
    hcoef[k] = static_cast<float>(1.0 - sab * gp);
    for (int a = 0; a < r; ++a) {
      const double ls = lam[a] + s2;
      hgain[static_cast<size_t>(k) * rpad + a] = scale[a] > 0.0 ? static_cast<float>(sab * ls / (ab * ls + om) - gp) : 0.f;
    }
  }
  LowRankDenoiser* L = new (std::nothrow) LowRankDenoiser;
  if (!L) return sdi::fail(E, SD_ERR_ARG, "sdden_lowrank_create: out of host memory");
  L->d = d; L->T = T; L->r = r; L->rpad = rpad; L->nk = nk;
  // K split of the first product: ranges of 8 slices or more (a call of few rows has nothing else to fill the chip
  // with), and slabs that move no more bytes than two thirds of the rows themselves (at 20480 rows, d = 3072, r = 256:
  // the first product takes 166 us with 4 slabs and 173 with 8, and the reduction twice as long)
  L->nsplit = std::max(1, std::min({nk / 8, d / (3 * rpad), 16}));
  hipError_t e = hipSuccess;                                // dynamic-LDS limits of the product kernels
#define SD_LR_PREPARE(ST, WM, WN, TM, TN, NS, RANK) \
  if (e == hipSuccess) e = lrgemm::prepare<WM, WN, TM, TN, NS, ST, RANK>();
  SD_LR_SHAPES(SD_LR_PREPARE)
#undef SD_LR_PREPARE
  if (e == hipSuccess) e = hipMalloc(&L->dev, h.size() * sizeof(float));
  if (e == hipSuccess) e = hipMemcpy(L->dev, h.data(), h.size() * sizeof(float), hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMalloc(&L->wdev, bytes_QT + bytes_Q);
  if (e == hipSuccess) e = hipMemcpy(L->wdev, hw.data(), bytes_QT + bytes_Q, hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    delete L;
    return sdi::fail(E, SD_ERR_HIP, "sdden_lowrank_create: %s", hipGetErrorString(e));
  }
  L->wQT = L->wdev; L->wQ = L->wdev + bytes_QT;
  L->gain = L->dev; L->sab = L->gain + static_cast<size_t>(T) * rpad;
  L->gperp = L->sab + T; L->coef = L->gperp + T; L->qmu = L->coef + T; L->mu = L->qmu + rpad;
  *out = L;
  return SD_OK;
}
