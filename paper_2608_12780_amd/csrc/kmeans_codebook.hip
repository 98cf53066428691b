// K-means codebooks: the kernels that write centroids.
//
// One wave (or block) per centroid row takes the row's fp32 values from
//   km_init_kernel    the starting row of X, or the centroid that is there
//                     (warm start), or
//   km_finish_kernel  the update's per-block sums: exact int64 totals, one
//                     fp64 division by count * 2^24 rounded to fp32; an empty
//                     cluster keeps its centroid,
// and, for the matrix-core assignment, prepares the row in the same launch:
// its two-term bf16 split, canonical squared norm and residual bound.  Per
// Lloyd iteration that leaves three launches (assign, accumulate, finish) of
// four, and one launch starts every subspace.  Measured per iteration, as
// separate finalize and preparation kernels -> here: 27.9 -> 11.7 us (40 heads
// x 256 rows x 128 channels, 5 slabs per head: bound by the slabs' 52 MB),
// 12.1 -> 4.7 us (3 heads x 32 rows, 9 slabs: about a launch's floor).
#include <math.h>

#include "common.h"
#include "kernels.h"

namespace scope {

namespace {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr int kRowThreads = 256;
constexpr int kRowWaves = kRowThreads / 64;
constexpr int kRowPitch = 132;  // floats per staged row: 128 channels, padded

__device__ __forceinline__ uint16_t to_bf16(float f) {
  bf16x2 r;
  r[0] = static_cast<__bf16>(f);
  r[1] = static_cast<__bf16>(0.0f);
  return static_cast<uint16_t>(__builtin_bit_cast(uint32_t, r) & 0xFFFFu);
}

// One wave prepares row r of subspace K for the matrix cores; lane l holds
// channels l and l + 64 of the row in xs (0 from dx on) and leaves them in the
// wave's row of `rows` for block_norms.  Rows of the two-term codebook are
// [2 * dxp] (hi then lo terms, zero padded); bnd >= |u - hi - lo|: the
// residuals are exact in fp32, their squares summed in fp32 lose at most 2^-16
// of the sum and 2^-143 to underflow, which the factor and the constant cover.
__device__ __forceinline__ void prepare_row(const Codebook &K, int h, int r, const float (&xs)[2],
                                            float *rows) {
  const int lane = threadIdx.x & 63;
  const int dxp = K.dxp;
  const size_t row = static_cast<size_t>(h) * K.cpad + r;
  uint16_t *dst = K.ubf + row * (2 * dxp);
  float e2 = 0.0f;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int c = lane + 64 * j;
    const float x = xs[j];
    rows[c] = x;
    const uint16_t bh = to_bf16(x);
    const float rest = x - bf16_to_f32(bh);  // exact
    const uint16_t bl = to_bf16(rest);
    const float df = rest - bf16_to_f32(bl);  // exact
    e2 = fmaf(df, df, e2);
    if (c < dxp) {
      dst[c] = bh;
      dst[dxp + c] = bl;
    }
  }
  e2 = wave_sum(e2);
  if (lane == 0) K.bnd[row] = sqrtf(e2) * 1.001f + 1e-21f;
}

// The canonical norms of the block's prepared rows r0 + i (live[i] set): one
// fma per channel in channel order, one thread per row (the rows' zero padding
// past dx adds nothing).  All threads of the block call it.
template <int NR>
__device__ __forceinline__ void block_norms(const Codebook &K, int h, int r0, const bool *live,
                                            const float (*rows)[kRowPitch]) {
  __syncthreads();
  const int i = threadIdx.x;
  if (i >= NR || !live[i]) return;
  float n = 0.0f;
  for (int c = 0; c < K.dx; c += 8) {
    const float4 a = *reinterpret_cast<const float4 *>(&rows[i][c]);
    const float4 b = *reinterpret_cast<const float4 *>(&rows[i][c + 4]);
    n = fmaf(a.x, a.x, n);
    n = fmaf(a.y, a.y, n);
    n = fmaf(a.z, a.z, n);
    n = fmaf(a.w, a.w, n);
    n = fmaf(b.x, b.x, n);
    n = fmaf(b.y, b.y, n);
    n = fmaf(b.z, b.z, n);
    n = fmaf(b.w, b.w, n);
  }
  K.nu[static_cast<size_t>(h) * K.cpad + r0 + i] = n;
}

// Starting centroids of every subspace (rows of all padded codebooks in one
// launch, one wave per row), prepared for the first assignment; also clears
// the grouping histogram and stores the launch arguments that later kernels
// of the call read from device memory (both optional).
template <typename T>
__global__ __launch_bounds__(kRowThreads) void km_init_kernel(
    const T *__restrict__ X, size_t x_hs, int ld, int n, bool warm, const int32_t *__restrict__ init,
    int init_hs, int init_ms, const Codebooks B, int32_t *status, int32_t *zero, size_t zero_count,
    const DeviceArgs args) {
  const int lane = threadIdx.x & 63, h = blockIdx.y;
  const size_t tid =
      ((static_cast<size_t>(blockIdx.z) * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x) * kRowThreads +
      threadIdx.x;
  const size_t threads = static_cast<size_t>(gridDim.x) * gridDim.y * gridDim.z * kRowThreads;
  for (size_t i = tid; i < zero_count; i += threads) zero[i] = 0;
  if (tid < static_cast<size_t>(args.words)) args.dst[tid] = args.w[tid];
  __shared__ __attribute__((aligned(16))) float rows[kRowWaves][kRowPitch];
  __shared__ bool live[kRowWaves];
  const int m = blockIdx.z, w = threadIdx.x >> 6;
  const Codebook &K = B.c[m];
  const int r = blockIdx.x * kRowWaves + w;
  if (lane == 0) live[w] = r < K.C;
  if (r < K.C) {
    float *u = B.u + h * B.u_hs + K.ucol + static_cast<size_t>(r) * K.dx;
    float xs[2];
    if (warm) {
#pragma unroll
      for (int j = 0; j < 2; ++j) xs[j] = lane + 64 * j < K.dx ? u[lane + 64 * j] : 0.0f;
    } else {
      const int def = static_cast<int>(((2LL * r + 1) * n) / (2LL * K.C));
      int src = def;
      if (init) {
        src = init[static_cast<size_t>(h) * init_hs + static_cast<size_t>(m) * init_ms + r];
        if (src < 0 || src >= n) {
          if (lane == 0 && status) atomicOr(status, kStatusBadInit);
          src = def;
        }
      }
      const T *x = X + h * x_hs + static_cast<size_t>(src) * ld + K.col0;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int c = lane + 64 * j;
        xs[j] = c < K.dx ? load_elem(x, c) : 0.0f;
        if (c < K.dx) u[c] = xs[j];
      }
    }
    if (K.ubf) prepare_row(K, h, r, xs, rows[w]);
  } else if (r < K.rows) {
    // padding of the matrix-core codebook: zero terms and a norm that never wins
    const size_t prow = static_cast<size_t>(h) * K.cpad + r;
    uint16_t *dst = K.ubf + prow * (2 * K.dxp);
    for (int c = lane; c < 2 * K.dxp; c += 64) dst[c] = 0;
    if (lane == 0) {
      K.nu[prow] = 0x1.fffffep127f;
      K.bnd[prow] = 0.0f;
    }
  }
  if (K.ubf) block_norms<kRowWaves>(K, h, blockIdx.x * kRowWaves, live, rows);
}

// The new centroids from the update's per-block sums (slab layout: like the
// centroids; counts one per cluster), prepared for the next assignment where
// the subspace has a matrix-core codebook.  SPLIT: the row's slabs are shared
// by the block's four waves (many slabs per head), else one row per wave.
// Bound: the latency of the slab loads, up to 16 in flight per lane.
template <bool SPLIT>
__global__ __launch_bounds__(kRowThreads) void km_finish_kernel(
    const Codebooks B, int S, int SC, int blocks, const long long *__restrict__ slab,
    const int32_t *__restrict__ cslab) {
  constexpr int NR = SPLIT ? 1 : kRowWaves;  // rows of a block
  __shared__ long long part[SPLIT ? kRowWaves : 1][2][64];
  __shared__ int pcnt[SPLIT ? kRowWaves : 1];
  __shared__ __attribute__((aligned(16))) float rows[NR][kRowPitch];
  __shared__ bool live[NR];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, h = blockIdx.y;
  const Codebook &K = B.c[blockIdx.z];
  const int r0 = blockIdx.x * NR, wr = SPLIT ? 0 : w;
  const int r = min(r0 + wr, K.C - 1);
  if (r0 >= K.C) return;  // the whole block
  const size_t pos = static_cast<size_t>(K.ucol) + static_cast<size_t>(r) * K.dx;
  const int c0 = min(lane, K.dx - 1), c1 = min(lane + 64, K.dx - 1);
  const long long *sl = slab + static_cast<size_t>(h) * blocks * S + pos;
  const int32_t *cs = cslab + static_cast<size_t>(h) * blocks * SC + K.ccol + r;
  long long t0 = 0, t1 = 0;
  int cnt = 0;
  const int b0 = SPLIT ? w : 0, bs = SPLIT ? kRowWaves : 1;
  for (int b = b0 + bs * lane; b < blocks; b += bs * 64) cnt += cs[static_cast<size_t>(b) * SC];
  if (K.dx > 64) {
#pragma unroll 8
    for (int b = b0; b < blocks; b += bs) {
      t0 += sl[static_cast<size_t>(b) * S + c0];
      t1 += sl[static_cast<size_t>(b) * S + c1];
    }
  } else {
#pragma unroll 8
    for (int b = b0; b < blocks; b += bs) t0 += sl[static_cast<size_t>(b) * S + c0];
  }
  cnt = wave_sum(cnt);
  if constexpr (SPLIT) {
    part[w][0][lane] = t0;
    part[w][1][lane] = t1;
    if (lane == 0) pcnt[w] = cnt;
    __syncthreads();
    t0 = t1 = 0;
    cnt = 0;
#pragma unroll
    for (int i = 0; i < kRowWaves; ++i) {
      t0 += part[i][0][lane];
      t1 += part[i][1][lane];
      cnt += pcnt[i];
    }
  }
  // an empty cluster keeps its centroid, and with it what was prepared
  const bool write = r0 + wr < K.C && cnt > 0;
  if (!SPLIT || w == 0) {
    if (lane == 0) live[wr] = write;
    if (write) {
      float *u = B.u + h * B.u_hs + pos;
      float xs[2];
      const double den = static_cast<double>(cnt) * 16777216.0;
      const long long tot[2] = {t0, t1};
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int c = lane + 64 * j;
        xs[j] = c < K.dx ? static_cast<float>(static_cast<double>(tot[j]) / den) : 0.0f;
        if (c < K.dx) u[c] = xs[j];
      }
      if (K.ubf) prepare_row(K, h, r, xs, rows[wr]);
    }
  }
  if (K.ubf) block_norms<NR>(K, h, r0, live, rows);
}

// The codebooks of the subspaces p[0..nsub); `prepare`: with their
// matrix-core codebooks.  *rows: the most rows of one subspace (padded ones
// included where they are prepared).
Codebooks codebooks(const KmProblem *p, int nsub, bool prepare, int *rows) {
  Codebooks B{};
  B.u = p[0].u;
  B.u_hs = p[0].u_head_stride;
  int ccol = 0;
  *rows = 0;
  for (int m = 0; m < nsub; ++m) {
    Codebook &K = B.c[m];
    const bool mf = p[m].mfma && prepare;
    K.C = p[m].C;
    K.cpad = p[m].cpad;
    K.rows = mf ? p[m].cpad : p[m].C;
    K.dx = p[m].dx;
    K.dxp = p[m].dxp;
    K.col0 = p[m].col0;
    K.ucol = static_cast<int>(p[m].u - p[0].u);
    K.ccol = ccol;
    K.ubf = mf ? p[m].ubf : nullptr;
    K.nu = mf ? p[m].nu : nullptr;
    K.bnd = mf ? p[m].bnd : nullptr;
    ccol += K.C;
    *rows = K.rows > *rows ? K.rows : *rows;
  }
  return B;
}

}  // namespace

hipError_t km_init(const KmProblem *p, int nsub, bool warm, const int32_t *init, int init_hs,
                   int init_ms, int32_t *status, int32_t *zero, size_t zero_count,
                   const DeviceArgs &args, hipStream_t s) {
  int rows = 0;
  const Codebooks B = codebooks(p, nsub, true, &rows);
  const dim3 grid((rows + kRowWaves - 1) / kRowWaves, p[0].heads, nsub);
  if (p[0].bf16)
    hipLaunchKernelGGL(km_init_kernel<uint16_t>, grid, dim3(kRowThreads), 0, s,
                       static_cast<const uint16_t *>(p[0].x), p[0].x_head_stride, p[0].ld, p[0].n,
                       warm, init, init_hs, init_ms, B, status, zero, zero_count, args);
  else
    hipLaunchKernelGGL(km_init_kernel<float>, grid, dim3(kRowThreads), 0, s,
                       static_cast<const float *>(p[0].x), p[0].x_head_stride, p[0].ld, p[0].n,
                       warm, init, init_hs, init_ms, B, status, zero, zero_count, args);
  return hipGetLastError();
}

// From 8 slabs per head on, four waves share a row's slabs, as long as the chip
// holds the waves of all rows at once (256 CUs of 32): beyond, a wave per row
// keeps it as full with a quarter of the blocks.  Whole key clusterings, 209
// centroids per subspace of 64 channels, a wave per row against four: 31 heads x
// 19721 745 and 834 us, 16 x 2600 200 and 248 us; on the other side queries, 32
// centroids, one head x 42000 175 and 135 us.
bool km_finish_shared(const AccPlan &plan, int heads) {
  return plan.blocks >= 8 && static_cast<long long>(plan.SC) * heads <= 2048;
}

hipError_t km_finish(const AccPlan &plan, const KmProblem *p, int nsub, bool prepare,
                     const long long *slab, const int32_t *cslab, hipStream_t s) {
  int rows = 0;
  const Codebooks B = codebooks(p, nsub, prepare, &rows);
  if (km_finish_shared(plan, p[0].heads))
    hipLaunchKernelGGL(km_finish_kernel<true>, dim3(rows, p[0].heads, nsub), dim3(kRowThreads), 0,
                       s, B, plan.S, plan.SC, plan.blocks, slab, cslab);
  else
    hipLaunchKernelGGL(km_finish_kernel<false>,
                       dim3((rows + kRowWaves - 1) / kRowWaves, p[0].heads, nsub),
                       dim3(kRowThreads), 0, s, B, plan.S, plan.SC, plan.blocks, slab, cslab);
  return hipGetLastError();
}

}  // namespace scope
