// The two skinny products of the low-rank Gaussian denoiser, fp32 in and out, on the bf16 matrix instructions:
// C[M,N] = A[M,K] * Bt[N,K]^T with every fp32 operand as the sum of three bf16 pieces.
//
// Why split.  The fp32 MFMA runs at a sixteenth of the bf16 rate and was what both products hung on (0.65 of its
// 157 TFLOP/s).  24 bits of mantissa are three pieces of 8, x = x0 + x1 + x2 exactly (truncation) or to 2^-25 (rounding);
// the six products of order 2^0, 2^-8 and 2^-16 keep everything above 2^-24 of a term, go through v_mfma_f32_16x16x32_bf16
// with fp32 accumulation, small ones first, and cost 6/16 of the fp32 instruction's time.  Error against fp64 sums
// (N(0.3, 1) times N(0, 1/K), relative 2-norm, the same K ranges): K = 256 2.3e-7 (fp32 MFMA 2.9e-7), K = 768 4.2e-7
// (5.0e-7), K = 3072 8.6e-7 (9.8e-7): fewer roundings per term, so slightly closer than the fp32 instruction.  Whole calls,
// dense bases: rank 1 1.0e-7 (1.3e-7), rank 8 1.2e-7 (1.6e-7), rank 50 2.6e-7 (6.0e-7).  A basis along the axes gives the
// same bits; one with two entries per column 6.9e-8 (6.4e-8): this instruction rounds its sums down, not to nearest.
// Truncation cannot overflow; an infinite or NaN input makes its own row NaN (as inf * q of both signs did).
//
// Layout.  16 rows x 32 k of a split operand are one block: three pieces of 1 KiB in which lane (l16, lq) of a wavefront
// finds its 16 bytes (row l16, k = 8 lq .. 8 lq + 7) at 16 * lane; the blocks of 16 rows follow each other along k.  A
// direct load into LDS is then eight whole cache lines and a fragment read is conflict free.  The weights are kept so
// from the denoiser's creation, the second product's A is written so by reduce_gain_kernel; the first product's A are
// gathered fp32 rows (8 rows of 128 B per load, chunk c of a row at c ^ ((row >> 1) & 7): conflict free on 64 banks),
// split in registers.
//
// Order of sums.  An output is one chain of MFMAs over its K range, the same whatever the tile, and the ranges of the
// first product (fixed per denoiser) go to slabs that reduce_gain_kernel adds in order: a prediction has the same bits
// however many rows a call has, and tiles can be chosen by size alone.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "lds_ring.h"
#include "sdden_internal.h"

namespace lrgemm {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int BK = 32;
constexpr int kBlockBytes = 3072;      // 16 rows x 32 k, three pieces
constexpr int kRowTile = 128;          // split operands are allocated for whole tiles of the largest height
constexpr int kRankRows = 512;         // calls of up to this many rows are compacted by the first product itself

struct __attribute__((aligned(16))) RowInfo {
  int32_t src;
  float gp, cf;
  int32_t pad;
};

struct Args {
  // STAGE 1: fp32 rows of `d` floats, tile row r reads row rowidx[r]; STAGE 2: split blocks
  const void* A;
  int d;
  const unsigned char* Bt;  // split blocks, ceil(N / 16) x nk
  int N, nk;                // output columns, slices of 32 of the whole contraction
  int32_t* count;           // device: M
  int32_t* rowidx;
  // STAGE 1 with RANK: the compaction (rows r < active rows with 0 <= krow[r] < T, in order) is done here and left in
  // rowidx / count
  const int32_t* krow;
  const int32_t* active;
  int rows_per_chain, R, T;
  // STAGE 1: partial sums, slab s = part + s * slab_stride, dense rows of N floats
  float* part;
  int64_t slab_stride;
  // STAGE 2 with RANK (calls of few rows): P' is made by every workgroup for its own rows, from the slabs above
  int nsplit;
  const float *gain, *sab, *qmu, *gperp, *coef;
  // STAGE 2 epilogue: out[src] = acc + gp X[src] + cf mu with (src, gp, cf) = rowinfo[row]
  const RowInfo* rowinfo;
  const float* X;
  float* out;
  int out_aligned;          // 16-byte stores into out
  const float* mu;
};

// byte offset of (row, k .. k + 7) of piece 0 in split blocks of nk slices; the pieces are 1024 apart
__host__ __device__ __forceinline__ size_t block_offset(int row, int k, int nk) {
  return (static_cast<size_t>(row >> 4) * nk + (k >> 5)) * kBlockBytes + (((k & 31) >> 3) * 16 + (row & 15)) * 16;
}

// Eight floats -> three vectors of eight bf16 whose sum is exact: each piece is the upper half of what is left.  No
// contraction: where x is a product, the first difference would be formed from the unrounded one, and the pieces would add
// up to the product cut off at 24 bits instead of rounded to them.
__device__ __forceinline__ void split8(const float (&x)[8], u32x4 (&piece)[3]) {
#pragma clang fp contract(off)
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    uint32_t u[2][3];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      float v = x[2 * h + e];
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        u[e][q] = __builtin_bit_cast(uint32_t, v);
        v -= __builtin_bit_cast(float, u[e][q] & 0xffff0000u);
      }
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) piece[q][h] = __builtin_amdgcn_perm(u[1][q], u[0][q], 0x07060302u);
  }
}

template <int WM, int WN, int TM, int TN, int NS, int STAGE>
struct Shape {
  static constexpr int NW = WM * WN, BM = 16 * TM * WM, BN = 16 * TN * WN;
  static constexpr int NA = STAGE == 1 ? BM / 8 : 3 * BM / 16, NB = 3 * BN / 16;   // 1 KiB loads per slice
  static constexpr int OPS = (NA + NB) / NW, kSlice = (NA + NB) * 1024;
  static constexpr size_t lds = static_cast<size_t>(NS) * kSlice;
  static_assert(NA % NW == 0 && NB % NW == 0, "loads must divide evenly over the wavefronts");
  static_assert(NS >= 2 && lds + 4 * BM <= 160 * 1024 && (NS - 1) * OPS < 64, "ring");
};
// STAGE 2 with RANK: the ring holds B alone, the tile's whole A lies behind it
template <int WM, int WN, int TM, int TN, int NS>
constexpr size_t fused_lds(int nk) {
  return static_cast<size_t>(NS) * Shape<WM, WN, TM, TN, NS, 2>::NB * 1024 + static_cast<size_t>(nk) * Shape<WM, WN, TM, TN, NS, 2>::NA * 1024;
}

// Eight columns of P': gain[k] .* (sum_s part_s - sab[k] qmu), slabs added in order, as split pieces.
__device__ __forceinline__ void gained8(const float* __restrict__ o, int64_t slab_stride, int nsplit, const float* __restrict__ gk,
                                        float sb, const float* __restrict__ qmu, u32x4 (&piece)[3]) {
  f32x4 s0 = *reinterpret_cast<const f32x4*>(o), s1 = *reinterpret_cast<const f32x4*>(o + 4);
#pragma unroll 4
  for (int i = 1; i < nsplit; ++i) {
    s0 += *reinterpret_cast<const f32x4*>(o + i * slab_stride);
    s1 += *reinterpret_cast<const f32x4*>(o + i * slab_stride + 4);
  }
  float x[8];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    x[e] = gk[e] * (s0[e] - sb * qmu[e]);
    x[4 + e] = gk[4 + e] * (s1[e] - sb * qmu[4 + e]);
  }
  split8(x, piece);
}

// STAGE 2 with RANK (calls of few rows): every workgroup adds up and scales its own rows of P' into LDS, which for 16 or 32 rows is
// a few loads per thread, in place of a launch of reduce_gain_kernel and a round trip through memory (LowRankDenoiser::eval has
// the figures).
// Workgroup of WM x WN wavefronts, wavefront tile 16 TM x 16 TN, NS slices of 32 k in an LDS ring.  Grid: (column tiles x
// row tiles, K ranges).  The weights are the first MFMA operand: a lane holds 4 consecutive output columns of one row.
template <int WM, int WN, int TM, int TN, int NS, int STAGE, bool RANK>
__global__ __launch_bounds__(64 * WM * WN) void kernel(Args p) {
  using S = Shape<WM, WN, TM, TN, NS, STAGE>;
  // FUSED: no loads of A; the ring's slices hold B and the whole tile of A, made here, follows the ring
  constexpr bool FUSED = STAGE == 2 && RANK;
  constexpr int NW = S::NW, BM = S::BM, BN = S::BN, ASZ = FUSED ? 0 : S::NA * 1024;
  constexpr int NA = FUSED ? 0 : S::NA, OPS = (NA + S::NB) / NW, kSlice = (NA + S::NB) * 1024;
  extern __shared__ __align__(1024) unsigned char ring[];
  __shared__ int src_row[STAGE == 1 && RANK ? BM : 1];

  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int tiles_n = (p.N + BN - 1) / BN;
  const int tile_m = blockIdx.x / tiles_n, tile_n = blockIdx.x % tiles_n;
  int M;
  if constexpr (STAGE == 1 && RANK) {
    // every wavefront ranks all rows by itself (one load per 64 rows) and notes those of this tile
    const int Ract = sdi::active_rows(p.active, p.rows_per_chain, p.R);
    int ks[kRankRows / 64];
#pragma unroll
    for (int c = 0; c < kRankRows / 64; ++c) ks[c] = c * 64 + lane < Ract ? p.krow[c * 64 + lane] : -1;
    M = 0;
#pragma unroll
    for (int c = 0; c < kRankRows / 64; ++c) {
      const bool keep = static_cast<unsigned>(ks[c]) < static_cast<unsigned>(p.T);
      const unsigned long long m = __ballot(keep);
      const int pos = M + __popcll(m & ((1ull << lane) - 1ull)) - tile_m * BM;
      if (keep && pos >= 0 && pos < BM) src_row[pos] = c * 64 + lane;
      M += __popcll(m);
    }
    __syncthreads();
    if (tile_n == 0 && blockIdx.y == 0) {
      for (int i = t; i < BM; i += 64 * NW)
        if (tile_m * BM + i < M) p.rowidx[tile_m * BM + i] = src_row[i];
      if (tile_m == 0 && t == 0) *p.count = M;
    }
  } else {
    M = *p.count;
  }
  if (tile_m * BM >= M) return;
  const int k_lo = static_cast<int>(static_cast<int64_t>(p.nk) * blockIdx.y / gridDim.y);
  const int nk = static_cast<int>(static_cast<int64_t>(p.nk) * (blockIdx.y + 1) / gridDim.y) - k_lo;
  const bool half_end = STAGE == 1 && (p.d & 16) && k_lo + nk == p.nk;     // the last slice has 16 columns only

  const int wm = wave / WN, wn = wave % WN, l16 = lane & 15, lq = lane >> 4;
  const unsigned char* src[OPS];      // this lane's source per load; rows and columns past the end are clamped
  int back = 0;                          // bit i: load i reads chunks 4..7, absent from a half slice
#pragma unroll
  for (int i = 0; i < NA / NW; ++i) {
    const int g = i * NW + wave;
    if constexpr (STAGE == 1) {
      const int row = 8 * g + (lane >> 3), chunk = (lane & 7) ^ ((row >> 1) & 7);
      int r = tile_m * BM + row;
      r = r < M ? r : M - 1;
      const int64_t from = RANK ? src_row[r - tile_m * BM] : p.rowidx[r];
      src[i] = static_cast<const unsigned char*>(p.A) + from * p.d * 4 + static_cast<int64_t>(k_lo) * 128 + 16 * chunk;
      back |= (chunk >> 2) << i;
    } else {
      const int64_t rb = tile_m * (BM / 16) + g / 3;
      src[i] = static_cast<const unsigned char*>(p.A) + rb * p.nk * kBlockBytes + (g % 3) * 1024 + 16 * lane;
    }
  }
#pragma unroll
  for (int i = 0; i < S::NB / NW; ++i) {
    const int g = i * NW + wave;
    int cb = tile_n * (BN / 16) + g / 3;
    cb = 16 * cb < p.N ? cb : p.N / 16 - 1;
    src[NA / NW + i] = p.Bt + (static_cast<int64_t>(cb) * p.nk + k_lo) * kBlockBytes + (g % 3) * 1024 + 16 * lane;
  }
  typedef __attribute__((address_space(3))) void* lds_ptr;
  typedef const __attribute__((address_space(1))) void* gbl_ptr;
  auto fetch = [&](int slot, int kt) {
    unsigned char* base = ring + slot * kSlice;
    const bool half = half_end && kt == nk - 1;
#pragma unroll
    for (int i = 0; i < NA / NW; ++i) {
      const unsigned char* a = src[i] + static_cast<int64_t>(kt) * (STAGE == 1 ? 128 : kBlockBytes);
      if (STAGE == 1 && half) a -= ((back >> i) & 1) * 64;       // any in-bounds chunk: its fragments become zero
      __builtin_amdgcn_global_load_lds((gbl_ptr)a, (lds_ptr)(base + (i * NW + wave) * 1024), 16, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < S::NB / NW; ++i)
      __builtin_amdgcn_global_load_lds((gbl_ptr)(src[NA / NW + i] + static_cast<int64_t>(kt) * kBlockBytes),
                                       (lds_ptr)(base + ASZ + (i * NW + wave) * 1024), 16, 0, 0);
  };

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < NS - 1; ++k)
    if (k < nk) fetch(k, k);

  // STAGE 2: what the epilogue needs from memory is requested while the first slices are on their way (the K loop, K =
  // rank, is as short as these round trips)
  const int row0 = tile_m * BM + wm * 16 * TM + l16, col0 = tile_n * BN + wn * 16 * TN + 4 * lq;
  f32x4 xv[STAGE == 2 ? TM : 1][TN], muv[TN];
  RowInfo info[TM];
  if constexpr (STAGE == 2) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int gm = row0 + 16 * i < M ? row0 + 16 * i : M - 1;
      if constexpr (FUSED) {
        const int from = p.rowidx[gm], k = p.krow[from];
        info[i] = RowInfo{from, p.gperp[k], p.coef[k], 0};
      } else {
        info[i] = p.rowinfo[gm];
      }
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int gn = col0 + 16 * j < p.N ? col0 + 16 * j : 0;
      muv[j] = *reinterpret_cast<const f32x4*>(p.mu + gn);
#pragma unroll
      for (int i = 0; i < TM; ++i) xv[i][j] = *reinterpret_cast<const f32x4*>(p.X + static_cast<int64_t>(info[i].src) * p.N + gn);
    }
  }

  if constexpr (FUSED) {
    // the tile's rows of P': a thread keeps its row, rows fastest, so that a wavefront's writes are whole blocks
    static_assert(64 * NW % BM == 0, "a row per thread");
    const int rank = 32 * nk, row = t % BM, gm = tile_m * BM + row < M ? tile_m * BM + row : M - 1;
    const int k = p.krow[p.rowidx[gm]];
    const float *from = p.part + static_cast<int64_t>(gm) * rank, *gk = p.gain + static_cast<int64_t>(k) * rank;
    const float sb = p.sab[k];
#pragma unroll 2
    for (int c = t / BM * 8; c < rank; c += 64 * NW / BM * 8) {
      u32x4 piece[3];
      gained8(from + c, p.slab_stride, p.nsplit, gk + c, sb, p.qmu + c, piece);
      unsigned char* dst = ring + NS * kSlice + (c >> 5) * S::NA * 1024 + (row >> 4) * kBlockBytes + (((c & 31) >> 3) * 16 + (row & 15)) * 16;
#pragma unroll
      for (int q = 0; q < 3; ++q) *reinterpret_cast<u32x4*>(dst + 1024 * q) = piece[q];
    }                                                        // the first slice's barrier makes it everyone's
  }

  int slot = 0, free_slot = NS - 1;
  for (int kt = 0; kt < nk; ++kt) {
    // slice kt has landed once only the younger ones are outstanding; past the barrier every wavefront has read slice
    // kt - 1, whose slot takes slice kt + NS - 1
    ldsring::wait_stages<OPS, NS - 2>(nk - 1 - kt);
    ldsring::barrier_keep_loads();
    if (kt + NS - 1 < nk) fetch(free_slot, kt + NS - 1);
    const unsigned char* base = ring + slot * kSlice;
    const unsigned char* abase = FUSED ? ring + NS * kSlice + kt * S::NA * 1024 : base;
    u32x4 a[TM][3];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      if constexpr (STAGE == 1) {
        const unsigned char* row = base + (wm * 16 * TM + 16 * i + l16) * 128;
        const f32x4 lo = *reinterpret_cast<const f32x4*>(row + (((2 * lq) ^ ((l16 >> 1) & 7)) << 4));
        const f32x4 hi = *reinterpret_cast<const f32x4*>(row + (((2 * lq + 1) ^ ((l16 >> 1) & 7)) << 4));
        const bool none = half_end && kt == nk - 1 && lq >= 2;
        float x[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) { x[e] = none ? 0.f : lo[e]; x[4 + e] = none ? 0.f : hi[e]; }
        split8(x, a[i]);
      } else {
#pragma unroll
        for (int q = 0; q < 3; ++q)
          a[i][q] = *reinterpret_cast<const u32x4*>(abase + ((wm * TM + i) * 3 + q) * 1024 + 16 * lane);
      }
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      u32x4 b[3];
#pragma unroll
      for (int q = 0; q < 3; ++q)
        b[q] = *reinterpret_cast<const u32x4*>(base + ASZ + ((wn * TN + j) * 3 + q) * 1024 + 16 * lane);
      constexpr int pa[6] = {2, 1, 0, 1, 0, 0}, pb[6] = {0, 1, 2, 0, 1, 0};
#pragma unroll
      for (int q = 0; q < 6; ++q)
#pragma unroll
        for (int i = 0; i < TM; ++i)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, b[pb[q]]),
                                                              __builtin_bit_cast(bf16x8, a[i][pa[q]]), acc[i][j], 0, 0, 0);
    }
    free_slot = slot;
    slot = slot + 1 == NS ? 0 : slot + 1;
  }

  // lane (l16, lq): columns col0 + 16 j .. + 3 of row row0 + 16 i
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int gm = row0 + 16 * i;
    if (gm >= M) continue;
    if constexpr (STAGE == 1) {
      float* dst = p.part + blockIdx.y * p.slab_stride + static_cast<int64_t>(gm) * p.N;
#pragma unroll
      for (int j = 0; j < TN; ++j)
        if (col0 + 16 * j < p.N) *reinterpret_cast<f32x4*>(dst + col0 + 16 * j) = acc[i][j];
    } else {
      float* dst = p.out + static_cast<int64_t>(info[i].src) * p.N;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int gn = col0 + 16 * j;
        if (gn >= p.N) continue;
        f32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = acc[i][j][e] + info[i].gp * xv[i][j][e] + info[i].cf * muv[j][e];
        if (p.out_aligned) *reinterpret_cast<f32x4*>(dst + gn) = o;
        else
#pragma unroll
          for (int e = 0; e < 4; ++e) dst[gn + e] = o[e];
      }
    }
  }
}

// P'[row][a] = gain[k][a] * (sum_s part_s[row][a] - sab[k] qmu[a]),  k = krow[rowidx[row]], slabs added in order, written
// as split blocks.  Also leaves the per-row record of the second product's epilogue.  One thread per 8 columns.
__global__ __launch_bounds__(256) void reduce_gain_kernel(const float* __restrict__ part, int64_t slab_stride, int nsplit,
                                                          const int32_t* __restrict__ count, const int32_t* __restrict__ rowidx,
                                                          const int32_t* __restrict__ krow, const float* __restrict__ gain,
                                                          const float* __restrict__ sab, const float* __restrict__ qmu,
                                                          unsigned char* __restrict__ P, int N, const float* __restrict__ gperp,
                                                          const float* __restrict__ coef, RowInfo* __restrict__ rowinfo) {
  const int M = *count;
  const int n8 = N / 8;
  const int64_t g = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (g >= static_cast<int64_t>(M) * n8) return;
  const int gm = static_cast<int>(g / n8), c = static_cast<int>(g % n8) * 8;
  const int src = rowidx[gm];
  const int k = krow[src];
  if (c == 0) rowinfo[gm] = RowInfo{src, gperp[k], coef[k], 0};
  u32x4 piece[3];
  gained8(part + static_cast<int64_t>(gm) * N + c, slab_stride, nsplit, gain + static_cast<int64_t>(k) * N + c, sab[k], qmu + c, piece);
  unsigned char* dst = P + block_offset(gm, c, N / 32);
#pragma unroll
  for (int q = 0; q < 3; ++q) *reinterpret_cast<u32x4*>(dst + 1024 * q) = piece[q];
}

// Raises the kernel's dynamic-LDS limit on the current device; done for every instantiation when a denoiser is
// created, never on the launch path (a HIP graph can capture the very first use).
template <int WM, int WN, int TM, int TN, int NS, int STAGE, bool RANK>
hipError_t prepare() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&kernel<WM, WN, TM, TN, NS, STAGE, RANK>),
                             hipFuncAttributeMaxDynamicSharedMemorySize,
                             static_cast<int>(Shape<WM, WN, TM, TN, NS, STAGE>::lds));
}

// The second product with the reduction in it (STAGE 2, RANK).
template <int WM, int WN, int TM, int TN, int NS>
hipError_t launch_fused(const Args& a, int R, hipStream_t st) {
  using S = Shape<WM, WN, TM, TN, NS, 2>;
  const int tiles = ((R + S::BM - 1) / S::BM) * ((a.N + S::BN - 1) / S::BN);
  hipLaunchKernelGGL((kernel<WM, WN, TM, TN, NS, 2, true>), dim3(tiles), dim3(64 * S::NW), (fused_lds<WM, WN, TM, TN, NS>(a.nk)), st, a);
  return hipGetLastError();
}

template <int WM, int WN, int TM, int TN, int NS, int STAGE, bool RANK>
hipError_t launch(const Args& a, int R, int nsplit, hipStream_t st) {
  using S = Shape<WM, WN, TM, TN, NS, STAGE>;
  const int tiles = ((R + S::BM - 1) / S::BM) * ((a.N + S::BN - 1) / S::BN);
  hipLaunchKernelGGL((kernel<WM, WN, TM, TN, NS, STAGE, RANK>), dim3(tiles, nsplit), dim3(64 * S::NW), S::lds, st, a);
  return hipGetLastError();
}

}  // namespace lrgemm
