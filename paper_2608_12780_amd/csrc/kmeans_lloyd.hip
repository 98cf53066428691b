// Lloyd iterations of small problems: assignment and update in one launch.
//
// With few rows an iteration is not bound by its work but by its chain of
// launches (3 heads x 2185 rows x 32 centroids x 128 channels: assign 16 us,
// accumulate 8 us, finish 5 us, each little above an empty launch's 4.5 us).
// Here a wave that has assigned a 32-row slice (assign_slice, the same exact
// filter) adds the slice's rows to the block's int64 sums at once, while they
// are in cache.  Where the rows of a head are few enough for one block, the
// block also turns the sums into the next centroids and goes round again: all
// iterations of a (head, subspace) are one launch.
// Measured, separate launches -> here: a layer of 3 heads x 2185 rows (C = 32;
// 16, 16, 16) 754 -> 491 us; Tiny (2 x 256 fp32, 8; 8, 8, 8) 276 -> 160 us; 8
// heads x 6417 fp32 (64; 32, 32, 32) 1155 -> 1030 us.
//
// Block (b, h, m): a share of the slices of head h in subspace m.  LDS: the
// two-term codebook, norms, int64 sums laid out so that the lanes of a row hit
// consecutive slots (channel c of a row of L pairs at (c mod 2) L + c / 2).
#include <math.h>

#include "common.h"
#include "kernels.h"
#include "kmeans_slice.h"

namespace scope {

namespace {

constexpr int kLloydWaves = 8;
constexpr int kLloydThreads = 64 * kLloydWaves;
constexpr int kLloydLds = 150 * 1024;

struct LloydSub {
  int col0, dx, dxp, C, cpad;
  int ucol, ccol;         // float offset and first cluster within a head
  const uint16_t *ubf;    // prepared codebook (km_init, km_finish)
  const float *nu, *bnd;
  float *u;
  int32_t *assign;
};
struct LloydArgs {
  const void *X;
  size_t x_hs, u_hs, a_hs;
  int ld, n, nchunks;
  int iters, final_assign;  // one-block form
  int32_t *chunk_hist;      // grouping histogram of the last assignment, or null
  long long *slab;          // several blocks: their sums and counts
  int32_t *cslab;
  int S, SC;
  int32_t *status;
  float lim;
  LloydSub sub[kMaxSub];
};

// Pairs of channels of a row of sums.
__device__ __host__ __forceinline__ int pairs_of(int dx) { return (dx + 1) / 2; }

struct LloydLds {
  uint16_t *Us;
  unsigned long long *sums;
  float *nus, *nhs, *bnd;
  int *cnts;
};
// Bytes of LDS, and with l the arrays at base.
__device__ __host__ __forceinline__ size_t lloyd_lds(int C, int cpad, int dx, int dxp, char *base, LloydLds *l) {
  auto up = [](size_t bytes) { return (bytes + 15) / 16 * 16; };
  const size_t us = 0, su = us + up(static_cast<size_t>(cpad) * (2 * dxp + 8) * 2);
  const size_t nu = su + up(static_cast<size_t>(C) * 2 * pairs_of(dx) * 8);
  const size_t row = up(4 * static_cast<size_t>(cpad));
  if (l)
    *l = LloydLds{reinterpret_cast<uint16_t *>(base + us),
                  reinterpret_cast<unsigned long long *>(base + su),
                  reinterpret_cast<float *>(base + nu), reinterpret_cast<float *>(base + nu + row),
                  reinterpret_cast<float *>(base + nu + 2 * row),
                  reinterpret_cast<int *>(base + nu + 3 * row)};
  return nu + 3 * row + up(4 * static_cast<size_t>(C));
}

// The rows of one slice as the update takes them: each step kRowsPerStep rows,
// the lanes of a row holding a pair of channels each.
template <int DXP, typename T>
struct SliceRows {
  static constexpr int kRowsPerStep = 128 / DXP;
  static constexpr int kSteps = 32 / kRowsPerStep;
  static constexpr int kWords = sizeof(T) == 2 ? 1 : 2;  // registers of a pair
  uint32_t v[kSteps][kWords];
};

template <int DXP, typename T>
__device__ __forceinline__ void load_rows(const LloydArgs &A, const LloydSub &K, int h, int sl,
                                          SliceRows<DXP, T> &R) {
  using Rows = SliceRows<DXP, T>;
  const int lane = threadIdx.x & 63, P = pairs_of(K.dx);
  const int rows = min(32, A.n - 32 * sl);
  const int rr = lane / P, c2 = lane - rr * P;  // the lane's row of a step and its pair
  const bool two = 2 * c2 + 1 < K.dx;
  const T *x0 = static_cast<const T *>(A.X) + h * A.x_hs + static_cast<size_t>(32 * sl) * A.ld + K.col0 + 2 * c2;
#pragma unroll
  for (int k = 0; k < Rows::kSteps; ++k) {
    const T *x = x0 + static_cast<size_t>(min(k * Rows::kRowsPerStep + rr, rows - 1)) * A.ld;
    if constexpr (sizeof(T) == 2) {
      R.v[k][0] = *reinterpret_cast<const bf16_pair *>(x);
    } else {
      R.v[k][0] = __float_as_uint(x[0]);
      R.v[k][1] = two ? __float_as_uint(x[1]) : 0u;
    }
  }
}

// Adds the rows of slice sl (whose centroids the wave's lanes hold in arg) to
// the sums and counts.
template <int DXP, typename T, bool CHECK>
__device__ __forceinline__ void accumulate_slice(const LloydArgs &A, const LloydSub &K, const LloydLds &L,
                                                 int sl, int arg, const SliceRows<DXP, T> &R, uint32_t &most) {
  using Rows = SliceRows<DXP, T>;
  const int lane = threadIdx.x & 63, P = pairs_of(K.dx);
  const int rows = min(32, A.n - 32 * sl);
  if (lane < rows) atomicAdd(&L.cnts[arg], 1);
  const int rr = lane / P, c2 = lane - rr * P;
#pragma unroll
  for (int k = 0; k < Rows::kSteps; ++k) {
    const int row = k * Rows::kRowsPerStep + rr;
    const int g = __shfl(arg, min(row, 31));
    if (rr < Rows::kRowsPerStep && row < rows) {
      float a, b;
      if constexpr (sizeof(T) == 2) {
        a = __uint_as_float(R.v[k][0] << 16);
        b = __uint_as_float(R.v[k][0] & 0xFFFF0000u);
      } else {
        a = __uint_as_float(R.v[k][0]);
        b = __uint_as_float(R.v[k][1]);
      }
      if (CHECK) {
        check_value(a, most);
        check_value(b, most);
      }
      unsigned long long *s = L.sums + static_cast<size_t>(g) * 2 * P + c2;
      atomicAdd(s, fixed24(a));
      atomicAdd(s + P, fixed24(b));
    }
  }
}

// The next centroids of the block's sums, in global memory and as two-term
// codebook, norms and residual bounds in LDS; an empty cluster keeps its own.
// Leaves the sums and counts cleared.
template <int DXP>
__device__ __forceinline__ void finish_block(const LloydSub &K, const LloydLds &L, float *U) {
  constexpr int US = 2 * DXP + 8;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, P = pairs_of(K.dx);
  __syncthreads();
  for (int r = w; r < K.C; r += kLloydWaves) {
    const int cnt = L.cnts[r];
    if (cnt <= 0) continue;
    unsigned long long *s = L.sums + static_cast<size_t>(r) * 2 * P;
    const double den = static_cast<double>(cnt) * 16777216.0;
    float xs[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int c = lane + 64 * j;
      xs[j] = c < K.dx ? static_cast<float>(static_cast<double>(static_cast<long long>(
                                                s[(c & 1) * P + (c >> 1)])) / den)
                       : 0.0f;
    }
    float e2 = 0.0f;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int c = lane + 64 * j;
      const float hi = bf16_to_f32(to_bf16(xs[j])), rest = xs[j] - hi;  // exact
      const float df = rest - bf16_to_f32(to_bf16(rest));               // exact
      e2 = fmaf(df, df, e2);
      if (c < K.dx) {
        U[static_cast<size_t>(r) * K.dx + c] = xs[j];
        L.Us[r * US + c] = to_bf16(xs[j]);
        L.Us[r * US + DXP + c] = to_bf16(rest);
      }
    }
    e2 = wave_sum(e2);
    wave_sync();  // the wave has read the row's sums
    float *row = reinterpret_cast<float *>(s);
#pragma unroll
    for (int j = 0; j < 2; ++j)
      if (lane + 64 * j < K.dx) row[lane + 64 * j] = xs[j];
    if (lane == 0) L.bnd[r] = sqrtf(e2) * 1.001f + 1e-21f;
  }
  __syncthreads();
  // the canonical norms, one thread per row
  for (int r = t; r < K.C; r += kLloydThreads)
    if (L.cnts[r] > 0) {
      const float *row = reinterpret_cast<const float *>(L.sums + static_cast<size_t>(r) * 2 * P);
      float n = 0.0f;
#pragma unroll 8
      for (int c = 0; c < K.dx; ++c) n = fmaf(row[c], row[c], n);
      L.nus[r] = n;
      L.nhs[r] = -0.5f * n;
    }
  __syncthreads();
  for (int e = t; e < K.C * 2 * P; e += kLloydThreads) L.sums[e] = 0ull;
  for (int r = t; r < K.C; r += kLloydThreads) L.cnts[r] = 0;
  __syncthreads();
}

// fp32 rows are requested before their slice is scored, so that they have
// arrived when its centroids are known (8 heads x 6417 x 64 centroids, one slice
// per wave: 34.7 -> 24.6 us).  bf16 rows are not: their registers would leave
// room for one block per CU instead of two (keys of 5 heads x 32760: 52 us
// against 45).
template <typename T, bool ONE>
constexpr bool kPrefetch = sizeof(T) == 4 && !ONE;

template <int DXP, typename T, bool ONE>
__device__ __forceinline__ void lloyd_block(const LloydArgs &A, const LloydSub &K, char *lds,
                                            uint32_t *cand, unsigned long long *best, int *ncand,
                                            int *next, float (*red)[kLloydWaves]) {
  const int t = threadIdx.x, w = t >> 6, lane = t & 63, b = blockIdx.x, h = blockIdx.y;
  LloydLds L;
  lloyd_lds(K.C, K.cpad, K.dx, DXP, lds, &L);
  const int P = pairs_of(K.dx);
  for (int e = t; e < K.C * 2 * P; e += kLloydThreads) L.sums[e] = 0ull;
  for (int r = t; r < K.C; r += kLloydThreads) L.cnts[r] = 0;
  if (t == 0) *next = 0;
  FilterBound B = stage_codebook<DXP, kLloydWaves, sizeof(T) == 4>(L.Us, L.nus, L.nhs, red, K.ubf, K.nu,
                                                                  K.bnd, h, K.C, K.cpad);
  float *U = K.u + h * A.u_hs;
  SliceArgs<T> S{static_cast<const T *>(A.X), A.x_hs, A.ld, K.col0, K.dx, A.n, K.C, K.cpad, K.u,
                 A.u_hs, K.assign, A.a_hs, nullptr, A.nchunks};
  const int nslices = (A.n + 31) / 32;
  const int lo = static_cast<int>(static_cast<long long>(nslices) * b / gridDim.x);
  const int hi = static_cast<int>(static_cast<long long>(nslices) * (b + 1) / gridDim.x);
  const int rounds = ONE ? A.iters + A.final_assign : 1;
  uint32_t most = 0;  // largest |x| seen, as bits
  if constexpr (ONE) {
    for (int r = t; r < K.C; r += kLloydThreads) L.bnd[r] = K.bnd[static_cast<size_t>(h) * K.cpad + r];
  }
  for (int it = 0; it < rounds; ++it) {
    const bool update = !ONE || it < A.iters;
    if (it + 1 == rounds) S.chunk_hist = A.chunk_hist;
    // a wave that is done takes the block's next slice
    for (;;) {
      int u = 0;
      if (lane == 0) u = atomicAdd(next, 1);
      u = lo + __builtin_amdgcn_readfirstlane(u);
      if (u >= hi) break;
      SliceRows<DXP, T> R;
      if (kPrefetch<T, ONE> && update) load_rows<DXP, T>(A, K, h, u, R);
      const int arg = assign_slice<DXP, T>(S, L.Us, L.nus, L.nhs, B, h, u, cand, best, ncand);
      if (update) {
        if (!kPrefetch<T, ONE>) load_rows<DXP, T>(A, K, h, u, R);
        if (A.status && it == 0) accumulate_slice<DXP, T, true>(A, K, L, u, arg, R, most);
        else accumulate_slice<DXP, T, false>(A, K, L, u, arg, R, most);
      }
    }
    if constexpr (ONE) {
      if (!update) break;
      finish_block<DXP>(K, L, U);
      if (t == 0) *next = 0;
      // the bound constants of the new codebook (finish_block ended on a
      // barrier; every wave works them out for itself)
      float e_max = 0.0f, nu_max = 0.0f;
      for (int r = lane; r < K.C; r += 64) {
        e_max = fmaxf(e_max, L.bnd[r]);
        nu_max = fmaxf(nu_max, fabsf(L.nus[r]));
        if (sizeof(T) == 4 && !(fabsf(L.nus[r]) < kNuLimit)) nu_max = INFINITY;
      }
      B = filter_bound(wave_max(e_max), wave_max(nu_max));
      __syncthreads();
    }
  }
  if (A.status) {
    const int bad = status_of(most, A.lim);
    if (bad) atomicOr(A.status, bad);
  }
  if constexpr (!ONE) {
    __syncthreads();
    const size_t hb = static_cast<size_t>(h) * gridDim.x + b;
    long long *sl = A.slab + hb * A.S + K.ucol;
    for (int r = w; r < K.C; r += kLloydWaves)
      for (int c = lane; c < K.dx; c += 64)
        sl[static_cast<size_t>(r) * K.dx + c] =
            static_cast<long long>(L.sums[static_cast<size_t>(r) * 2 * P + (c & 1) * P + (c >> 1)]);
    for (int r = t; r < K.C; r += kLloydThreads) A.cslab[hb * A.SC + K.ccol + r] = L.cnts[r];
  }
}

// Blocks of eight waves whose registers fit a CU.
template <typename T, bool ONE>
constexpr int kPerCu = sizeof(T) == 2 && !ONE ? 2 : 1;

template <typename T, bool ONE>
__global__ __launch_bounds__(kLloydThreads)
__attribute__((amdgpu_waves_per_eu(kPerCu<T, ONE> * 2))) void km_lloyd_kernel(const LloydArgs A) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  __shared__ uint32_t cand[kLloydWaves][kWaveCand];
  __shared__ unsigned long long best[kLloydWaves][32];
  __shared__ int ncand[kLloydWaves];
  __shared__ int next;
  __shared__ float red[2][kLloydWaves];
  const int w = threadIdx.x >> 6;
  const LloydSub &K = A.sub[blockIdx.z];
  switch (K.dxp) {
    case 16: lloyd_block<16, T, ONE>(A, K, lds, cand[w], best[w], &ncand[w], &next, red); break;
    case 32: lloyd_block<32, T, ONE>(A, K, lds, cand[w], best[w], &ncand[w], &next, red); break;
    case 48: lloyd_block<48, T, ONE>(A, K, lds, cand[w], best[w], &ncand[w], &next, red); break;
    case 64: lloyd_block<64, T, ONE>(A, K, lds, cand[w], best[w], &ncand[w], &next, red); break;
    default: lloyd_block<128, T, ONE>(A, K, lds, cand[w], best[w], &ncand[w], &next, red); break;
  }
}

}  // namespace

// Up to 48 MiB of rows: their second and third reads come from the L2s and the
// memory-side cache.  Beyond, the separate launches win, which stream the rows
// with 16 waves per CU (a whole clustering, here against there: keys 5 heads x
// 32760 tokens x 64 centroids, 42 MB, 555 / 605 us; layer 24 x 8192, 50 MB, 2041
// / 2117 us; fp32 layer 8 x 16384, 67 MB, 2112 / 1920 us; keys 3 x 118800 x 128,
// 91 MB, 1080 / 1002 us; keys 40 x 32760, 335 MB, 3320 / 2528 us).
// All iterations in one block up to 10 slices (queries 3 heads x 300 rows x 16:
// 173 us against 181 with several blocks, 700 rows x 32: 269 against 205).
//
// With so many (head, subspace) pairs that each gets only one block, it runs
// - up to 32 slices all iterations, unless its rows are bf16 and wider than 64
//   channels, where two blocks of the iteration form share a CU (bf16 keys of 300
//   heads x 330 rows: all 379, iteration 445, separate 664 us; 300 x 640 520, 560,
//   694; queries, 128 channels, 300 x 330 511, 346, 474; 140 x 1000 562, 446, 428;
//   fp32 queries 150 x 600 363, 453, 416; fp32 keys 86 x 1000 420, 556, 478);
// - beyond, bf16 rows one iteration where every CU has a block (keys 100 x 1900
//   534, 516, 583 us; 8 subspaces 33 x 2000 376, 319, 361; queries, 64 channels,
//   130 x 2900 517, 586, 455);
// - beyond, fp32 rows all iterations where the rounds of blocks keep three fifths
//   of the CUs busy (8 subspaces 24 x 4096, 192 blocks, 392, 503, 480 us; keys 60 x
//   1600, 180 blocks, 431, 581, 485; 8 subspaces 33 x 2500, 264 blocks, 508, 647,
//   485; keys 50 x 1900, 150 blocks, 501, 649, 421; on the wrong side: 4 subspaces
//   33 x 2500, 132 blocks, 373, 456, 409).
constexpr size_t kLloydBytes = 48u << 20;
constexpr int kLloydOneBlock = 10, kLloydOneBlockMany = 32;
LloydForm km_lloyd_form(const KmProblem *p, int nsub, const AccPlan &plan) {
  const LloydForm separate{Lloyd::kSeparate, 0};
  const int slices = (p[0].n + 31) / 32;
  for (int m = 0; m < nsub; ++m)
    if (!p[m].mfma || lloyd_lds(p[m].C, p[m].cpad, p[m].dx, p[m].dxp, nullptr, nullptr) > kLloydLds) return separate;
  const size_t row_bytes = static_cast<size_t>(p[0].ld) * (p[0].bf16 ? 2 : 4);
  if (row_bytes * p[0].n * p[0].heads > kLloydBytes) return separate;
  if (slices <= kLloydOneBlock) return LloydForm{Lloyd::kAll, 1};
  // as many blocks as the CUs hold, each wave with a slice, and no more slabs
  // than the workspace has
  size_t lds = 0;
  for (int m = 0; m < nsub; ++m) {
    const size_t need = lloyd_lds(p[m].C, p[m].cpad, p[m].dx, p[m].dxp, nullptr, nullptr);
    lds = need > lds ? need : lds;
  }
  const int per_cu = p[0].bf16 && 2 * lds <= kLloydLds ? kPerCu<uint16_t, false> : 1;
  int blocks = per_cu * kAccTargetBlocks / (p[0].heads * nsub);
  const int most = (slices + kLloydWaves - 1) / kLloydWaves;
  if (blocks > most) blocks = most;
  if (blocks > plan.blocks) blocks = plan.blocks;
  if (blocks >= 2) return LloydForm{Lloyd::kIteration, blocks};
  bool wide = false;
  for (int m = 0; m < nsub; ++m) wide = wide || (p[m].bf16 && p[m].dxp > 64);
  if (slices <= kLloydOneBlockMany) return LloydForm{wide ? Lloyd::kIteration : Lloyd::kAll, 1};
  const int pairs = p[0].heads * nsub, rounds = (pairs + kAccTargetBlocks - 1) / kAccTargetBlocks;
  if (p[0].bf16) return pairs >= kAccTargetBlocks ? LloydForm{Lloyd::kIteration, 1} : separate;
  return 5 * pairs >= 3 * rounds * kAccTargetBlocks ? LloydForm{Lloyd::kAll, 1} : separate;
}

hipError_t km_lloyd(const KmProblem *p, int nsub, LloydForm form, int iters, bool final_assign,
                    int32_t *chunk_hist, const AccPlan &plan, long long *slab, int32_t *cslab,
                    int32_t *status, hipStream_t s) {
  LloydArgs A{};
  A.X = p[0].x;
  A.x_hs = p[0].x_head_stride;
  A.u_hs = p[0].u_head_stride;
  A.a_hs = p[0].a_head_stride;
  A.ld = p[0].ld;
  A.n = p[0].n;
  A.nchunks = km_nchunks(p[0].n);
  A.iters = iters;
  A.final_assign = final_assign ? 1 : 0;
  A.chunk_hist = chunk_hist;
  A.slab = slab;
  A.cslab = cslab;
  A.S = plan.S;
  A.SC = plan.SC;
  A.status = status;
  A.lim = km_range_limit(p[0].n);
  size_t lds = 0;
  for (int m = 0; m < nsub; ++m) {
    LloydSub &K = A.sub[m];
    K.col0 = p[m].col0;
    K.dx = p[m].dx;
    K.dxp = p[m].dxp;
    K.C = p[m].C;
    K.cpad = p[m].cpad;
    K.ucol = plan.ucol[m];
    K.ccol = plan.ccol[m];
    K.ubf = p[m].ubf;
    K.nu = p[m].nu;
    K.bnd = p[m].bnd;
    K.u = p[m].u;
    K.assign = p[m].assign;
    const size_t need = lloyd_lds(K.C, K.cpad, K.dx, K.dxp, nullptr, nullptr);
    lds = need > lds ? need : lds;
  }
  const dim3 grid(form.blocks, p[0].heads, nsub), block(kLloydThreads);
#define SCOPE_LLOYD(T)                                                                  \
  if (form.form == Lloyd::kAll) hipLaunchKernelGGL((km_lloyd_kernel<T, true>), grid, block, lds, s, A); \
  else hipLaunchKernelGGL((km_lloyd_kernel<T, false>), grid, block, lds, s, A)
  if (p[0].bf16) {
    SCOPE_LLOYD(uint16_t);
  } else {
    SCOPE_LLOYD(float);
  }
#undef SCOPE_LLOYD
  return hipGetLastError();
}

}  // namespace scope
