// The MLP denoiser's three products for calls of few rows (one image-sized chain, a handful of requests, the window
// start of a batch):  C[M,N] = A[M,K] * Bt[N,K]^T with the epilogues of mlp_gemm.h.
//
// What bounds such a call is reading the weights once, and the tiles of mlp_gemm.h cannot: an output of 16 rows is
// 32 tiles of 64 x 128 at N = 4096, so 32 of 256 CUs pull the whole matrix, each through one chain of dependent
// slices.  Here a tile is 16 * MT rows x 16 * NT columns, so 16 columns already give every CU one at N = 4096, and a
// ring in LDS keeps RING - 1 stages of S steps of 32 k on their way per workgroup (56 KiB for one row tile).
//
// Every output is summed over k in one chain and in order, as in the tiles of mlp_gemm.h and mlp_gemm_pp.h (32 at a time
// here and in kernel_pp, 16 in the others), and predictions have come out with the same bits from every one of them,
// however many rows a call had (tested against each tile; the instruction set does not promise it).  Splitting k over the
// wavefronts of a workgroup measured 44 us against 51 for one row and 61 against 77 for 64 (the three products at
// d = 12288, H = 4096), but moves every prediction by 3e-4 (a hidden activation that rounds to the other bf16 moves all
// that follow), and with it the drafts that are made from it.
//
// Layout.  Both operands are stored in fragment order: 16 rows x 32 k are one block of 1 KiB in which lane (l16, lq)
// of the wavefront finds its 16 bytes (row l16, k = 8 lq .. 8 lq + 7) at 16 * lane, and the blocks of 16 rows follow
// each other along k.  A direct load into LDS is then eight whole cache lines and a fragment read is conflict free
// with no permutation; out of row-major operands a block is 16 half lines one row stride apart, which for these widths
// (multiples of 512 bytes) meet on few cache channels (16 rows, split k: 57.6 us row-major, 40.3 in fragment order).
// The weights' copy in this order is made when the denoiser is created; the call's rows the first product takes as they are
// (their bf16 image, or few short fp32 ones) or from pack_rows_kernel, and each product's epilogue writes the next one's operand.
//
// Measured, the three products with pack_rows_kernel against the LDS tiles without their compaction and conversion:
//   d = 12288, H = 4096    1 row 51 / 161 us   32 rows 54 / 169   64 rows 72 / 170   200 rows 136 / 158
//   d = 3072, H = 1024     1 row 17 / 39 us    32 rows 17 / 46    64 rows 20 / 46    200 rows 25 / 48
// 237 MB of weights in 47 us are 5 TB/s; from 64 rows on it is the operands' path out of L2 that counts.
#pragma once
#include "lds_ring.h"
#include "mlp_gemm.h"
#include "sdden_internal.h"

namespace mlpfew {

using mlpgemm::bf16x8;
using mlpgemm::u32x4;
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kPackThreads = 256;
constexpr int kMaxRows = 1024;    // rows of a call: pack_rows_kernel ranks them four per thread, the first product 16 per lane

// Element offset of (row, k .. k + 7), k a multiple of 8, in fragment order.
__host__ __device__ __forceinline__ size_t frag_offset(int row, int k, int K) {
  return (static_cast<size_t>(row >> 4) * (K >> 5) + (k >> 5)) * 512 + (((k & 31) >> 3) * 16 + (row & 15)) * 8;
}

// W[N,K] row-major -> fragment order; one 16-byte chunk per thread.
__global__ __launch_bounds__(256) void pack_weights_kernel(const uint16_t* __restrict__ W, uint16_t* __restrict__ F, int N, int K) {
  const int64_t g = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  const int chunks = K / 8;
  if (g >= static_cast<int64_t>(N) * chunks) return;
  const int n = static_cast<int>(g / chunks), k = static_cast<int>(g % chunks) * 8;
  *reinterpret_cast<u32x4*>(F + frag_offset(n, k, K)) = *reinterpret_cast<const u32x4*>(W + static_cast<size_t>(n) * K + k);
}

// The rows r < active rows with 0 <= krow[r] < T, in increasing order, as dense rows of F in fragment order, rounded to bf16:
// for calls without a bf16 image of more than 16 rows or, up to 16, of more than 1024 coordinates (the others' first product loads the
// rows itself).  Every workgroup ranks all (at most kMaxRows) rows itself -- one load per 256 rows -- and moves its 16 dense rows x `kchunk` columns; the first column of workgroups leaves
// rowidx and the count for the products.  One launch in place of a compaction and a conversion.
__global__ __launch_bounds__(kPackThreads) void pack_rows_kernel(const float* __restrict__ X, const int32_t* __restrict__ krow, const int32_t* active,
                                                                 int rows_per_chain, int R, int T, int K, int kchunk,
                                                                 uint16_t* __restrict__ F, int32_t* __restrict__ rowidx,
                                                                 int32_t* __restrict__ count) {
  constexpr int NW = kPackThreads / 64, NC = kMaxRows / kPackThreads;
  __shared__ int tot[NC][NW];
  __shared__ int src_row[16];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int Ract = sdi::active_rows(active, rows_per_chain, R);
  unsigned long long m[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int r = c * kPackThreads + t;
    const bool keep = r < Ract && static_cast<unsigned>(krow[r < R ? r : 0]) < static_cast<unsigned>(T);
    m[c] = __ballot(keep);
    if (lane == 0) tot[c][wave] = __popcll(m[c]);
  }
  if (t < 16) src_row[t] = -1;
  __syncthreads();
  const int first = blockIdx.y * 16;
  int base = 0;
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      if (w == wave && ((m[c] >> lane) & 1ull)) {
        const int pos = base + __popcll(m[c] & ((1ull << lane) - 1ull));
        if (pos >= first && pos < first + 16) src_row[pos - first] = c * kPackThreads + t;
      }
      base += tot[c][w];
    }
  __syncthreads();
  if (blockIdx.x == 0) {
    if (t < 16 && src_row[t] >= 0) rowidx[first + t] = src_row[t];
    if (blockIdx.y == 0 && t == 0) *count = base;
  }
  if (first >= base) return;
  const int k0 = blockIdx.x * kchunk, k1 = k0 + kchunk < K ? k0 + kchunk : K;
  // 16 lanes share a k chunk of 8 and take one row each: stores of 256 contiguous bytes
  const int row = t & 15, src = src_row[row];
  if (src < 0) return;
  for (int k = k0 + 8 * (t >> 4); k < k1; k += 8 * (kPackThreads / 16)) {
    const float* s = X + static_cast<size_t>(src) * K + k;
    const f32x4 lo = *reinterpret_cast<const f32x4*>(s), hi = *reinterpret_cast<const f32x4*>(s + 4);
    bf16x8 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      o[e] = static_cast<__bf16>(lo[e]);
      o[4 + e] = static_cast<__bf16>(hi[e]);
    }
    *reinterpret_cast<bf16x8*>(F + frag_offset(first + row, k, K)) = o;
  }
}

struct Args {
  const void* A;            // kPacked: [rows rounded up to a whole tile, K] bf16, fragment order; else row-major rows of K
  const uint16_t* W;        // [N, K] bf16, fragment order
  int N, K;
  int32_t* count;           // device: M                     (found and left here unless kPacked)
  int32_t* rowidx;          // dense row -> source row       (the same)
  const int32_t* krow;      // source row -> chain step
  const int32_t* active;    // not kPacked: which of the R rows count, as in pack_rows_kernel
  int rows_per_chain, R, T;
  const float* bias;        // EPI 1: per-step table [T, N]; EPI 2, 3: [N]
  uint16_t* outb;           // EPI 1, 2: bf16 [M, N], fragment order (N is the next product's K)
  float* outf;              // EPI 3: fp32 [*, N] at source rows
};

// Where a product's rows come from.  kPacked: dense rows in fragment order.  kRowsBf16, kRowsF32: the caller's own rows, which the
// workgroup finds in krow itself (at most 16 loads a lane, ahead of its first weights) and loads without a packing launch;
// fp32 rows are rounded as fragments are read.  A stage then holds S * 64 (or 128) contiguous bytes of each row, chunk c of
// row r at c ^ swizzle(r), which makes the fragment reads conflict free on 64 banks.  Without the packing launch (4.6 to 5.6
// us of kernel) a pass takes, us: 23 chains, d = 3072, H = 1024, K = 9 28.3 (30.0); one chain, d = 12288, H = 4096, K = 16
// 115 (119), its first product 21.5 as before.  fp32 rows only up to 16 and for short rows: every workgroup loads them all, and
// at d = 12288 the product takes 40 us with them.
enum Source { kPacked, kRowsBf16, kRowsF32 };

// EPI as in mlp_gemm.h.  Grid: (N / (16 NT), tiles of 16 MT rows), MT wavefronts; wavefront i owns rows 16 i .. 16 i + 15
// of the tile.  A stage of the ring is S steps of 32 k: the rows' part, then per step NT blocks of W (kPacked: per step MT
// blocks of A, then NT of W).  Rows >= M of the last tile are computed on whatever is there and never stored.
template <int EPI, int MT, int NT, int S, int RING, int SRC = kPacked>
__global__ __launch_bounds__(64 * MT) void kernel(Args p) {
  constexpr int AL = (SRC == kRowsF32 ? 2 : 1) * S;          // loads of 1 KiB per wavefront and stage: its rows' A
  constexpr int kStep = (MT + NT) * 1024, kRows = MT * AL * 1024;
  constexpr int kStage = SRC == kPacked ? S * kStep : kRows + S * NT * 1024;
  constexpr int WLOADS = S * NT / MT, OPS = AL + WLOADS;     // and a share of W
  static_assert(S * NT % MT == 0 && RING >= 2 && RING * kStage <= 160 * 1024 && (RING - 1) * OPS < 64, "ring");
  static_assert(SRC != kRowsF32 || MT == 1, "fp32 rows");
  __shared__ __align__(1024) unsigned char ring[RING * kStage];
  int* src_row = reinterpret_cast<int*>(ring + (RING - 1) * kStage);   // not kPacked; the last slot is free until the first stage is read
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int row0 = blockIdx.y * 16 * MT, col0 = blockIdx.x * 16 * NT;
  int M = 0, my_src = 0;
  if (SRC == kPacked) {
    M = *p.count;
    if (blockIdx.y > 0 && row0 >= M) return;         // the first tile need not wait for the count
  }

  const int steps = p.K / 32, nk = steps / S;        // steps: blocks of 1 KiB per 16 rows
  const unsigned char* asrc = static_cast<const unsigned char*>(p.A) + static_cast<size_t>(row0 / 16 + wave) * steps * 1024 + 16 * lane;
  const unsigned char* wsrc = reinterpret_cast<const unsigned char*>(p.W) + static_cast<size_t>(col0 / 16) * steps * 1024 + 16 * lane;
  typedef __attribute__((address_space(3))) void* lds_ptr;
  typedef const __attribute__((address_space(1))) void* gbl_ptr;
  // rows: load u of a stage brings chunks 64 u + lane of the wavefront's 16 rows, kRowChunks of 16 bytes each
  constexpr int kRowChunks = 4 * AL;
  auto swizzle = [](int row) { return kRowChunks == 8 ? (row >> 1) & 7 : row & 15; };
  const unsigned char* rsrc[AL];
  auto fetch_a = [&](int slot, int kt) {
    if constexpr (SRC == kPacked) {
#pragma unroll
      for (int u = 0; u < S; ++u)
        __builtin_amdgcn_global_load_lds((gbl_ptr)(asrc + static_cast<size_t>(kt * S + u) * 1024),
                                         (lds_ptr)(ring + slot * kStage + u * kStep + wave * 1024), 16, 0, 0);
    } else {
#pragma unroll
      for (int u = 0; u < AL; ++u)
        __builtin_amdgcn_global_load_lds((gbl_ptr)(rsrc[u] + static_cast<size_t>(kt) * kRowChunks * 16),
                                         (lds_ptr)(ring + slot * kStage + (wave * AL + u) * 1024), 16, 0, 0);
    }
  };
  auto fetch_w = [&](int slot, int kt) {
#pragma unroll
    for (int u = 0; u < WLOADS; ++u) {
      const int b = u * MT + wave, step = b / NT, j = b % NT;          // the stage's W blocks, dealt to the wavefronts
      __builtin_amdgcn_global_load_lds((gbl_ptr)(wsrc + (static_cast<size_t>(j) * steps + kt * S + step) * 1024),
                                       (lds_ptr)(ring + slot * kStage + (SRC == kPacked ? step * kStep + (MT + j) * 1024 : kRows + b * 1024)), 16, 0, 0);
    }
  };

  if constexpr (SRC == kPacked) {
#pragma unroll
    for (int k = 0; k < RING - 1; ++k)
      if (k < nk) {
        fetch_a(k, k);
        fetch_w(k, k);
      }
  } else {
    // the rows' numbers are on their way before the first weights and are ranked while those come
    const int Ract = sdi::active_rows(p.active, p.rows_per_chain, p.R);
    int ks[kMaxRows / 64];
#pragma unroll
    for (int c = 0; c < kMaxRows / 64; ++c) ks[c] = c * 64 + lane < Ract ? p.krow[c * 64 + lane] : -1;
    if (lane < 16) src_row[16 * wave + lane] = 0;    // rows past the last: any that exists
#pragma unroll
    for (int k = 0; k < RING - 1; ++k)
      if (k < nk) fetch_w(k, k);
    if (MT > 1) ldsring::barrier_keep_loads();
    else ldsring::wait_reads();
#pragma unroll
    for (int c = 0; c < kMaxRows / 64; ++c) {
      const bool keep = static_cast<unsigned>(ks[c]) < static_cast<unsigned>(p.T);
      const unsigned long long m = __ballot(keep);
      const int pos = M + __popcll(m & ((1ull << lane) - 1ull)) - row0;
      if (keep && pos >= 0 && pos < 16 * MT) src_row[pos] = c * 64 + lane;   // the same from every wavefront
      M += __popcll(m);
    }
    if (MT > 1) ldsring::barrier_keep_loads();
    else ldsring::wait_reads();
    if (blockIdx.x == 0) {
      for (int i = t; i < 16 * MT; i += 64 * MT)
        if (row0 + i < M) p.rowidx[row0 + i] = src_row[i];
      if (blockIdx.y == 0 && t == 0) *p.count = M;
    }
    if (blockIdx.y > 0 && row0 >= M) {
      ldsring::wait_loads<0>();                      // nothing of this workgroup may land in LDS that is another's by then
      return;
    }
#pragma unroll
    for (int u = 0; u < AL; ++u) {
      const int c = 64 * u + lane, row = c / kRowChunks, chunk = (c % kRowChunks) ^ swizzle(row);
      rsrc[u] = static_cast<const unsigned char*>(p.A) + static_cast<size_t>(src_row[16 * wave + row]) * p.K * (SRC == kRowsF32 ? 4 : 2) + 16 * chunk;
    }
    my_src = src_row[16 * wave + (lane & 15)];
#pragma unroll
    for (int k = 0; k < RING - 1; ++k)
      if (k < nk) fetch_a(k, k);
  }

  f32x4 acc[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  int slot = 0, free_slot = RING - 1;
  for (int kt = 0; kt < nk; ++kt) {
    // stage kt has landed once only the younger ones are outstanding; past the barrier every wavefront has read stage
    // kt - 1 (a lone one has waited for its reads), whose slot takes stage kt + RING - 1
    // (rows: the first stages' weights came first and their A stage by stage, so fewer loads are younger than a stage's last)
    if (SRC != kPacked && kt < RING - 1) ldsring::wait_stages<AL, RING - 2>(nk - 1 - kt);
    else ldsring::wait_stages<OPS, RING - 2>(nk - 1 - kt);
    if (MT > 1) ldsring::barrier_keep_loads();
    else ldsring::wait_reads();
    if (kt + RING - 1 < nk) {
      fetch_a(free_slot, kt + RING - 1);
      fetch_w(free_slot, kt + RING - 1);
    }
    const unsigned char* base = ring + slot * kStage + 16 * lane;
    const unsigned char* rows = ring + slot * kStage + wave * AL * 1024 + (lane & 15) * kRowChunks * 16;
    u32x4 a[S], w[S][NT];
#pragma unroll
    for (int u = 0; u < S; ++u) {
      const int c = 4 * u + (lane >> 4), x = swizzle(lane & 15);       // chunk of 8 k, the row's permutation
      if constexpr (SRC == kPacked) {
        a[u] = *reinterpret_cast<const u32x4*>(base + u * kStep + wave * 1024);
      } else if constexpr (SRC == kRowsBf16) {
        a[u] = *reinterpret_cast<const u32x4*>(rows + ((c ^ x) << 4));
      } else {
        const f32x4 lo = *reinterpret_cast<const f32x4*>(rows + (((2 * c) ^ x) << 4));
        const f32x4 hi = *reinterpret_cast<const f32x4*>(rows + (((2 * c + 1) ^ x) << 4));
        bf16x8 b;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          b[e] = static_cast<__bf16>(lo[e]);
          b[4 + e] = static_cast<__bf16>(hi[e]);
        }
        a[u] = __builtin_bit_cast(u32x4, b);
      }
#pragma unroll
      for (int j = 0; j < NT; ++j)
        w[u][j] = *reinterpret_cast<const u32x4*>(base + (SRC == kPacked ? u * kStep + (MT + j) * 1024 : kRows + (u * NT + j) * 1024));
    }
    __builtin_amdgcn_sched_barrier(0);               // every read is on its way before the first product waits for one
    // the weights are the first operand: a lane then holds 4 consecutive output columns of one row
#pragma unroll
    for (int u = 0; u < S; ++u)
#pragma unroll
      for (int j = 0; j < NT; ++j)
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[u][j]), __builtin_bit_cast(bf16x8, a[u]),
                                                         acc[j], 0, 0, 0);
    free_slot = slot;
    slot = slot + 1 == RING ? 0 : slot + 1;
  }

  // lane (l16, lq): columns col0 + 16 j + 4 lq .. + 3 of row row0 + 16 wave + l16
  const int gm = row0 + 16 * wave + (lane & 15);
  if (gm >= M) return;
  const int src = EPI == 2 ? 0 : SRC != kPacked ? my_src : p.rowidx[gm];
  const float* b = EPI == 1 ? p.bias + static_cast<size_t>(p.krow[src]) * p.N : p.bias;
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int gn = col0 + 16 * j + 4 * (lane >> 4);
    const f32x4 c = acc[j] + *reinterpret_cast<const f32x4*>(b + gn);
    if (EPI == 3) {
      *reinterpret_cast<f32x4*>(p.outf + static_cast<size_t>(src) * p.N + gn) = c;
    } else {
      uint2 o;
      o.x = mlpgemm::to_bf16_bits(mlpgemm::silu(c[0])) | (static_cast<uint32_t>(mlpgemm::to_bf16_bits(mlpgemm::silu(c[1]))) << 16);
      o.y = mlpgemm::to_bf16_bits(mlpgemm::silu(c[2])) | (static_cast<uint32_t>(mlpgemm::to_bf16_bits(mlpgemm::silu(c[3]))) << 16);
      *reinterpret_cast<uint2*>(p.outb + frag_offset(gm, gn & ~7, p.N) + (gn & 4)) = o;
    }
  }
}

template <int EPI, int MT, int NT, int S, int RING, int SRC = kPacked>
hipError_t launch(const Args& a, int R, hipStream_t st) {
  hipLaunchKernelGGL((kernel<EPI, MT, NT, S, RING, SRC>), dim3(a.N / (16 * NT), (R + 16 * MT - 1) / (16 * MT)), dim3(64 * MT), 0, st, a);
  return hipGetLastError();
}

}  // namespace mlpfew
