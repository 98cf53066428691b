// K-means assignment on the matrix cores (kmeans_slice.h): one pass over the
// rows of every head.
//
// Blocks are persistent per head: the two-term codebook is staged in LDS
// once, then each wave independently takes the block's next 32-point slice
// from a counter in LDS (so a wave slowed by a re-score does not hold up the
// others); chunk histograms for the grouping are accumulated with global
// atomics.
#include <math.h>
#include <string.h>

#include "common.h"
#include "kernels.h"
#include "kmeans_slice.h"

namespace scope {

namespace {

// The LDS of one block's assignment.
template <int NW>
struct AssignLds {
  __attribute__((aligned(16))) uint16_t Us[kUbfLds];
  __attribute__((aligned(16))) float nus[kMaxCpad];
  __attribute__((aligned(16))) float nhs[kMaxCpad];
  uint32_t cand[NW][kWaveCand];
  unsigned long long best[NW][32];
  int ncand[NW];
  float red[2][NW];
  int next_slice;
};

// Block b of nb: its contiguous range of (head, slice) pairs.
template <int DXP, typename T>
__device__ __forceinline__ void assign_range(const SliceArgs<T> &A, const uint16_t *__restrict__ ubf,
                                             const float *__restrict__ nu,
                                             const float *__restrict__ bnd, int heads, int b, int nb,
                                             AssignLds<kWaves<T>> &L) {
  constexpr int NW = kWaves<T>;
  const int w = threadIdx.x >> 6;
  const int nslices = (A.n + 31) / 32;
  const long long total = static_cast<long long>(heads) * nslices;
  const long long per = (total + nb - 1) / nb;
  long long beg = static_cast<long long>(b) * per;
  const long long end = beg + per < total ? beg + per : total;
  while (beg < end) {
    const int h = static_cast<int>(beg / nslices);
    const long long seg_end = end < static_cast<long long>(h + 1) * nslices
                                  ? end : static_cast<long long>(h + 1) * nslices;
    __syncthreads();
    if (threadIdx.x == 0) L.next_slice = 0;  // visible after the staging barrier
    const FilterBound B = stage_codebook<DXP, NW, sizeof(T) == 4>(L.Us, L.nus, L.nhs, L.red, ubf, nu, bnd,
                                                                 h, A.C, A.cpad);
    // a wave that is done takes the block's next slice
    const long long count = seg_end - beg;
    for (;;) {
      int u = 0;
      if ((threadIdx.x & 63) == 0) u = atomicAdd(&L.next_slice, 1);
      u = __builtin_amdgcn_readfirstlane(__shfl(u, 0));
      if (u >= count) break;
      const long long g = beg + u;
      assign_slice<DXP, T>(A, L.Us, L.nus, L.nhs, B, h, static_cast<int>(g - static_cast<long long>(h) * nslices),
                           L.cand[w], L.best[w], &L.ncand[w]);
    }
    beg = seg_end;
  }
}

template <int DXP, typename T>
__global__ __launch_bounds__(64 * kWaves<T>) void km_assign_mfma_kernel(
    const T *__restrict__ X, size_t x_hs, int ld, int col0, int dx,
    int n, int heads, const float *__restrict__ U, size_t u_hs,
    const uint16_t *__restrict__ ubf, const float *__restrict__ nu,
    const float *__restrict__ bnd, int C, int cpad, int32_t *assign,
    size_t a_hs, int32_t *chunk_hist, int nchunks) {
  __shared__ AssignLds<kWaves<T>> L;
  const SliceArgs<T> A{X, x_hs, ld, col0, dx, n, C, cpad, U, u_hs, assign, a_hs, chunk_hist, nchunks};
  assign_range<DXP, T>(A, ubf, nu, bnd, heads, blockIdx.x, gridDim.x, L);
}

// Several subspaces in one launch, each with blocks of its own (from first[m]
// on) in proportion to its work.  One launch per subspace leaves the last
// slices of each to a few waves: 5 heads x 32760 rows are 1.25 slices per wave
// of the chip, two rounds where one and a quarter would do.  A whole clustering
// of keys into 333 centroids per subspace, apart -> together: that one, 16 / 56 /
// 56 channels, 1320 -> 1048 us; 3 x 118800 2107 -> 1754 us; 40 x 32760 6149 ->
// 5819 us; 24 x 118800 12.82 -> 12.53 ms; fp32 3 x 118800 2479 -> 2134 us.
template <typename T>
struct ManyArgs {
  int nsub, heads;
  int first[kMaxSub + 1], dxp[kMaxSub];
  SliceArgs<T> a[kMaxSub];
  const uint16_t *ubf[kMaxSub];
  const float *nu[kMaxSub], *bnd[kMaxSub];
};
template <typename T>
__global__ __launch_bounds__(64 * kWaves<T>) void km_assign_mfma_many_kernel(const ManyArgs<T> M) {
  __shared__ AssignLds<kWaves<T>> L;
  int m = 0;
  while (m + 1 < M.nsub && static_cast<int>(blockIdx.x) >= M.first[m + 1]) ++m;
  const int b = blockIdx.x - M.first[m], nb = M.first[m + 1] - M.first[m];
  const SliceArgs<T> A = M.a[m];
  switch (M.dxp[m]) {
    case 16: assign_range<16, T>(A, M.ubf[m], M.nu[m], M.bnd[m], M.heads, b, nb, L); break;
    case 32: assign_range<32, T>(A, M.ubf[m], M.nu[m], M.bnd[m], M.heads, b, nb, L); break;
    case 48: assign_range<48, T>(A, M.ubf[m], M.nu[m], M.bnd[m], M.heads, b, nb, L); break;
    case 64: assign_range<64, T>(A, M.ubf[m], M.nu[m], M.bnd[m], M.heads, b, nb, L); break;
    default: assign_range<128, T>(A, M.ubf[m], M.nu[m], M.bnd[m], M.heads, b, nb, L); break;
  }
}

// The three key subspaces in one pass over the rows: their codebooks are
// staged in LDS side by side (subspace m at element offset uoff[m] and norm
// offset noff[m]), and the block's waves take work units (slice, subspace)
// from a counter in LDS, in slice order.  A wave that is done takes the next
// unit whatever its subspace, so the subspaces' different costs balance
// out, and the three units of a slice start at about the same time, so a
// row fetched from HBM for one is found in cache by the others.
template <typename T>
struct Sub3 {
  SliceArgs<T> a[3];
  const uint16_t *ubf[3];
  const float *nu[3];
  const float *bnd[3];
  int uoff[3], noff[3];
};

template <int D0, int D1, int D2, typename T>
__global__ __launch_bounds__(64 * kWaves<T>) void km_assign_mfma3_kernel(
    const Sub3<T> *__restrict__ Sp, int n, int heads) {
  constexpr int NW = kWaves<T>;
  constexpr bool CHK = sizeof(T) == 4;
  __shared__ __attribute__((aligned(16))) uint16_t Us[kUbfLds];
  __shared__ __attribute__((aligned(16))) float nus[kMaxCpad];
  __shared__ __attribute__((aligned(16))) float nhs[kMaxCpad];
  __shared__ uint32_t cand[NW][kWaveCand];
  __shared__ unsigned long long best[NW][32];
  __shared__ int ncand[NW];
  __shared__ float red[3][2][NW];
  __shared__ int next_unit;
  const int w = threadIdx.x >> 6;
  const int nslices = (n + 31) / 32;
  const long long total = static_cast<long long>(heads) * nslices;
  const long long per = (total + gridDim.x - 1) / gridDim.x;
  long long beg = static_cast<long long>(blockIdx.x) * per;
  const long long end = beg + per < total ? beg + per : total;
  while (beg < end) {
    const int h = static_cast<int>(beg / nslices);
    const long long seg_end = end < static_cast<long long>(h + 1) * nslices
                                  ? end : static_cast<long long>(h + 1) * nslices;
    __syncthreads();
    if (threadIdx.x == 0) next_unit = 0;  // visible after the staging barriers
    stage_codebook<D0, NW, CHK>(Us + Sp->uoff[0], nus + Sp->noff[0], nhs + Sp->noff[0], red[0], Sp->ubf[0], Sp->nu[0],
                       Sp->bnd[0], h, Sp->a[0].C, Sp->a[0].cpad);
    stage_codebook<D1, NW, CHK>(Us + Sp->uoff[1], nus + Sp->noff[1], nhs + Sp->noff[1], red[1], Sp->ubf[1], Sp->nu[1],
                       Sp->bnd[1], h, Sp->a[1].C, Sp->a[1].cpad);
    stage_codebook<D2, NW, CHK>(Us + Sp->uoff[2], nus + Sp->noff[2], nhs + Sp->noff[2], red[2], Sp->ubf[2], Sp->nu[2],
                       Sp->bnd[2], h, Sp->a[2].C, Sp->a[2].cpad);
    const long long first = static_cast<long long>(h) * nslices;
    const FilterBound B0 = reduce_bound<NW>(red[0]);
    const FilterBound B1 = reduce_bound<NW>(red[1]);
    const FilterBound B2 = reduce_bound<NW>(red[2]);
    const long long units = 3 * (seg_end - beg);
    for (;;) {
      int u = 0;
      if ((threadIdx.x & 63) == 0) u = atomicAdd(&next_unit, 1);
      u = __builtin_amdgcn_readfirstlane(__shfl(u, 0));
      if (u >= units) break;
      const long long g = beg + u / 3;
      const int m = u - 3 * (u / 3);
      if (m == 0)
        assign_slice<D0, T>(Sp->a[0], Us + Sp->uoff[0], nus + Sp->noff[0], nhs + Sp->noff[0], B0, h,
                         static_cast<int>(g - first), cand[w], best[w], &ncand[w]);
      else if (m == 1)
        assign_slice<D1, T>(Sp->a[1], Us + Sp->uoff[1], nus + Sp->noff[1], nhs + Sp->noff[1], B1, h,
                         static_cast<int>(g - first), cand[w], best[w], &ncand[w]);
      else
        assign_slice<D2, T>(Sp->a[2], Us + Sp->uoff[2], nus + Sp->noff[2], nhs + Sp->noff[2], B2, h,
                         static_cast<int>(g - first), cand[w], best[w], &ncand[w]);
    }
    beg = seg_end;
  }
}

// Codebooks larger than the LDS holds (e.g. 300 centroids at d = 128) are
// cut into chunks of at most CR rows, and every chunk gets its own
// persistent blocks, which keep the chunk in LDS for their whole range of
// slices (waves take slices independently, as above).  Per point, each chunk
// yields its three largest packed values (indices over the whole codebook),
// and chunk 0 also the point's norm bound.  The decision kernel below merges
// the lists, one point per thread.
template <int DXP, typename T>
__global__ __launch_bounds__(64 * kWaves<T>) void km_assign_mfma_part_kernel(
    const T *__restrict__ X, size_t x_hs, int ld, int col0, int dx,
    int n, int heads, const uint16_t *__restrict__ ubf, const float *__restrict__ nu,
    int cpad, int crows, float *part, float *pnx) {
  constexpr int US = 2 * DXP + 8;  // LDS row stride of the two-term codebook
  constexpr int KS = DXP / 16;     // MFMA k-steps per term
  constexpr int NW = kWaves<T>;
  __shared__ __attribute__((aligned(16))) uint16_t Us[kUbfLds];
  __shared__ __attribute__((aligned(16))) float nhs[kMaxCpad];
  __shared__ int next_slice;
  const int t = threadIdx.x;
  const int lane = t & 63, l32 = lane & 31, hf = lane >> 5;
  const int chunk = blockIdx.y, r0 = chunk * crows;
  const int rows = cpad - r0 < crows ? cpad - r0 : crows;  // a multiple of 32
  const int ib = 32 - __clz(cpad - 1);
  const uint32_t imask = (1u << ib) - 1u;
  const int nslices = (n + 31) / 32;
  const bool vec = rows_aligned(X + col0, x_hs, ld);

  const long long total = static_cast<long long>(heads) * nslices;
  const long long per = (total + gridDim.x - 1) / gridDim.x;
  long long beg = static_cast<long long>(blockIdx.x) * per;
  const long long end = beg + per < total ? beg + per : total;
  while (beg < end) {
    const int h = static_cast<int>(beg / nslices);
    const long long seg_end = end < static_cast<long long>(h + 1) * nslices
                                  ? end : static_cast<long long>(h + 1) * nslices;
    // stage this head's chunk (rows r0 .. r0+rows) and its start values
    __syncthreads();
    if (t == 0) next_slice = 0;
    const uint16_t *ub = ubf + (static_cast<size_t>(h) * cpad + r0) * (2 * DXP);
    for (int e = t; e < rows * (DXP / 4); e += 64 * NW) {
      const int r = e / (DXP / 4), q = e % (DXP / 4);
      *reinterpret_cast<uint4 *>(&Us[r * US + 8 * q]) =
          *reinterpret_cast<const uint4 *>(ub + static_cast<size_t>(r) * (2 * DXP) + 8 * q);
    }
    for (int r = t; r < rows; r += 64 * NW)
      nhs[r] = -0.5f * nu[static_cast<size_t>(h) * cpad + r0 + r];
    __syncthreads();
    const long long count = seg_end - beg;
    for (;;) {
      int u = 0;
      if (lane == 0) u = atomicAdd(&next_slice, 1);
      u = __builtin_amdgcn_readfirstlane(u);
      if (u >= count) break;
      const int sl = static_cast<int>(beg + u - static_cast<long long>(h) * nslices);
      const int i = sl * 32 + l32;
      const bool valid = i < n;
      const T *xrow = X + h * x_hs + static_cast<size_t>(valid ? i : 0) * ld + col0;
      PointFrag<KS, T> xf;
      float ss = load_point<KS, T>(xrow, hf, dx, valid, vec, xf);
      ss += __shfl_xor(ss, 32);
      const Top3 top = top_scores<DXP, T>(Us, nhs, xf, rows, imask, r0);
      if (valid && hf == 0) {
        *reinterpret_cast<float4 *>(part + ((static_cast<size_t>(chunk) * heads + h) * n + i) * 4) =
            make_float4(top.m1, top.m2, top.m3, 0.0f);
        if (chunk == 0) pnx[static_cast<size_t>(h) * n + i] = sqrtf(ss) * 1.0001f + 1e-30f;
      }
    }
    beg = seg_end;
  }
}

// The decision for chunked codebooks, one point per thread: the margin of the
// kernel above around the largest of all chunks' values.  A chunk whose third
// value lies outside it has at most two candidates, both listed; the listed
// candidates are re-scored canonically if there are several, and only a point
// with three candidates in one chunk (or more) scans every centroid.
constexpr int kOwnScans = 8;
template <int DXP, typename T>
__global__ __launch_bounds__(256) void km_assign_decide_kernel(
    const T *__restrict__ X, size_t x_hs, int ld, int col0, int dx, int n,
    int heads, const float *__restrict__ U, size_t u_hs, const float *__restrict__ nu,
    const float *__restrict__ bnd, int C, int cpad, int nparts,
    const float *__restrict__ part, const float *__restrict__ pnx,
    int32_t *assign, size_t a_hs, int32_t *chunk_hist, int nchunks) {
  __shared__ float red[2][4];
  const int h = blockIdx.y, t = threadIdx.x, lane = t & 63, w = t >> 6;
  // the head's bound constants, as in the assignment kernel
  float e_max = 0.0f, nu_max = 0.0f;
  for (int r = t; r < C; r += 256) {
    const size_t row = static_cast<size_t>(h) * cpad + r;
    e_max = fmaxf(e_max, bnd[row]);
    nu_max = fmaxf(nu_max, fabsf(nu[row]));
    if (sizeof(T) == 4 && !(fabsf(nu[row]) < kNuLimit)) nu_max = INFINITY;
  }
  e_max = wave_max(e_max);
  nu_max = wave_max(nu_max);
  if (lane == 0) {
    red[0][w] = e_max;
    red[1][w] = nu_max;
  }
  __syncthreads();
  const FilterBound B = reduce_bound<4>(red);
  // every lane of a wave stays for the joint scans; those past the end repeat
  // the last point
  const bool valid = static_cast<int>(blockIdx.x * 256 + t) < n;
  const int i = min(static_cast<int>(blockIdx.x * 256 + t), n - 1);
  const int ib = 32 - __clz(cpad - 1);
  const uint32_t imask = (1u << ib) - 1u;
  const float dpack = __uint_as_float(static_cast<uint32_t>(127 + ib - 23) << 23);
  auto listed = [&](int k) {
    return *reinterpret_cast<const float4 *>(part + ((static_cast<size_t>(k) * heads + h) * n + i) * 4);
  };
  float m1 = -0x1.1p127f;
  for (int k = 0; k < nparts; ++k) m1 = fmaxf(m1, listed(k).x);
  const float nx = pnx[static_cast<size_t>(h) * n + i];
  const float beta = margin<DXP, T>(nx, B);
  const float slack = (beta + 2.0f * dpack * fabsf(m1)) * 1.001f;
  const float lim = m1 - slack;
  const float thr = lim - fabsf(lim) * 2e-6f - 1e-30f;
  int arg = static_cast<int>(__float_as_uint(m1) & imask);
  int near = 0;         // listed candidates
  bool scan = false;
  for (int k = 0; k < nparts; ++k) {
    const float4 v = listed(k);
    near += (!(v.x < thr) ? 1 : 0) + (!(v.y < thr) ? 1 : 0);
    scan = scan || !(v.z < thr);
  }
  const T *xr = X + h * x_hs + static_cast<size_t>(i) * ld + col0;
  const float *Uh = U + h * u_hs;
  const float *nuh = nu + static_cast<size_t>(h) * cpad;
  auto score_key = [&](const T *x, int r) {
    const float dot = canon_dot(x, Uh + static_cast<size_t>(r) * dx, dx);
    const float sc = fmaf(-2.0f, dot, nuh[r]) + 0.0f;
    return (static_cast<unsigned long long>(asc_key(sc)) << 32) | static_cast<unsigned>(r);
  };
  const bool unsafe = sizeof(T) == 4 && !(nx < kNormLimit && B.numax < kNuLimit * 1.01f);
  // every centroid, canonically: points outside the filter's range, and where a wave
  // has several with three candidates in a chunk, each lane for its own
  bool own_scan = unsafe;
  if constexpr (sizeof(T) == 4) {
    const int scans = __popcll(__ballot(valid && scan));
    own_scan = unsafe || (scan && scans >= kOwnScans);
    if (own_scan) {
      const unsigned long long b = canon_scan(xr, Uh, nuh, C, dx, 0, 4);
      arg = b == ~0ull ? 0 : static_cast<int>(b & 0xFFFFFFFFu);
    }
  }
  if (!own_scan && !scan && near > 1) {
    unsigned long long b = ~0ull;
    for (int k = 0; k < nparts; ++k) {
      const float4 v = listed(k);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const float c = j ? v.y : v.x;
        if (!(c < thr)) {
          const unsigned long long key = score_key(xr, min(static_cast<int>(__float_as_uint(c) & imask), C - 1));
          b = key < b ? key : b;
        }
      }
    }
    arg = static_cast<int>(b & 0xFFFFFFFFu);
  }
  // a scan takes the whole wave, each lane every 64th centroid (one thread
  // going through 300 centroids held its block up for 350 us)
  for (uint64_t todo = __ballot(valid && scan && !own_scan); todo; todo &= todo - 1) {
    const int src = __ffsll(static_cast<long long>(todo)) - 1;
    const T *xs = X + h * x_hs + static_cast<size_t>(__shfl(i, src)) * ld + col0;
    unsigned long long b = ~0ull;
    for (int r = lane; r < C; r += 64) {
      const unsigned long long key = score_key(xs, r);
      b = key < b ? key : b;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const unsigned long long other = __shfl_xor(b, o);
      b = other < b ? other : b;
    }
    if (lane == src) arg = static_cast<int>(b & 0xFFFFFFFFu);
  }
  if (!valid) return;
  arg = min(max(arg, 0), C - 1);
  assign[h * a_hs + i] = arg;
  if (chunk_hist)
    atomicAdd(&chunk_hist[(static_cast<size_t>(h) * nchunks + (i / kAssignBlock)) * C + arg], 1);
}

int cu_count() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
    cus = 256;
  return cus;
}

template <int DXP, typename T>
hipError_t launch_mfma(const KmProblem &p, bool with_hist, hipStream_t s) {
  hipError_t e = hipSuccess;
  const int nch = km_nchunks(p.n);
  // persistent blocks, one per CU (the codebook fills most of the LDS),
  // each over a contiguous range of (head, 32-point slice) pairs
  const long long slices = static_cast<long long>(p.heads) * ((p.n + 31) / 32);
  const int cus = cu_count();
  const int blocks = static_cast<int>(slices < static_cast<long long>(cus) * kWaves<T>
                                          ? (slices + kWaves<T> - 1) / kWaves<T> : cus);
  const T *x = static_cast<const T *>(p.x);
  if (p.cpad * (2 * DXP + 8) <= kUbfLds) {
    hipLaunchKernelGGL((km_assign_mfma_kernel<DXP, T>), dim3(blocks), dim3(64 * kWaves<T>), 0, s,
                       x, p.x_head_stride, p.ld, p.col0, p.dx, p.n, p.heads, p.u,
                       p.u_head_stride, p.ubf, p.nu, p.bnd, p.C, p.cpad, p.assign,
                       p.a_head_stride, with_hist ? p.chunk_hist : nullptr, nch);
    return hipGetLastError();
  }
  // chunked codebook: balanced chunks, the CUs shared among them
  const int nparts = km_parts(p.C, p.dx);
  const int crows = (p.cpad / 32 + nparts - 1) / nparts * 32;
  const int per_part = cus / nparts > 1 ? cus / nparts : 1;
  const long long need = (slices + kWaves<T> - 1) / kWaves<T>;
  const int bpp = static_cast<int>(need < per_part ? need : per_part);
  hipLaunchKernelGGL((km_assign_mfma_part_kernel<DXP, T>), dim3(bpp, nparts),
                     dim3(64 * kWaves<T>), 0, s, x, p.x_head_stride, p.ld, p.col0, p.dx,
                     p.n, p.heads, p.ubf, p.nu, p.cpad, crows, p.part, p.pnx);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((km_assign_decide_kernel<DXP, T>), dim3((p.n + 255) / 256, p.heads), dim3(256), 0,
                     s, x, p.x_head_stride, p.ld, p.col0, p.dx, p.n, p.heads, p.u,
                     p.u_head_stride, p.nu, p.bnd, p.C, p.cpad, nparts, p.part, p.pnx,
                     p.assign, p.a_head_stride, with_hist ? p.chunk_hist : nullptr,
                     nch);
  return hipGetLastError();
}

// The launch arguments of the one-pass assignment (device memory).
template <int D0, int D1, int D2, typename T>
Sub3<T> sub3_args(const KmProblem (&p)[3]) {
  Sub3<T> S{};
  int uoff = 0, noff = 0;
  const int dxp[3] = {D0, D1, D2};
  for (int m = 0; m < 3; ++m) {
    const KmProblem &q = p[m];
    S.a[m] = SliceArgs<T>{static_cast<const T *>(q.x), q.x_head_stride, q.ld, q.col0, q.dx,
                       q.n, q.C, q.cpad, q.u, q.u_head_stride, q.assign, q.a_head_stride,
                       nullptr, 0};
    S.ubf[m] = q.ubf;
    S.nu[m] = q.nu;
    S.bnd[m] = q.bnd;
    S.uoff[m] = uoff;
    S.noff[m] = noff;
    uoff += q.cpad * (2 * dxp[m] + 8);
    noff += q.cpad;
  }
  return S;
}

template <int D0, int D1, int D2, typename T>
hipError_t launch_mfma3(const KmProblem (&p)[3], const void *dev_args, hipStream_t s) {
  const long long slices = static_cast<long long>(p[0].heads) * ((p[0].n + 31) / 32);
  const int cus = cu_count();
  const int blocks = static_cast<int>(slices < static_cast<long long>(cus) * kWaves<T>
                                          ? (slices + kWaves<T> - 1) / kWaves<T> : cus);
  hipLaunchKernelGGL((km_assign_mfma3_kernel<D0, D1, D2, T>), dim3(blocks), dim3(64 * kWaves<T>),
                     0, s, static_cast<const Sub3<T> *>(dev_args), p[0].n, p[0].heads);
  return hipGetLastError();
}

}  // namespace

bool km_assign3_ok(const KmProblem (&p)[3]) {
  int lds = 0, rows = 0;
  for (int m = 0; m < 3; ++m) {
    const KmProblem &q = p[m];
    if (!q.mfma || q.x != p[0].x || q.ld != p[0].ld || q.n != p[0].n ||
        q.heads != p[0].heads || q.x_head_stride != p[0].x_head_stride)
      return false;
    lds += q.cpad * (2 * q.dxp + 8);
    rows += q.cpad;
  }
  if (lds > kUbfLds || rows > kMaxCpad) return false;
  const int a = p[0].dxp, b = p[1].dxp, c = p[2].dxp;
  return (a == 16 && b == 64 && c == 64) || (a == 48 && b == 48 && c == 48) ||
         (a == 16 && b == 32 && c == 32);
}

// F<D0, D1, D2, T> for the widths and the element type of p (km_assign3_ok).
#define SCOPE_SUB3_T(F, T, ...)                                            \
  (p[0].dxp == 48   ? F<48, 48, 48, T>(__VA_ARGS__)                        \
   : p[1].dxp == 64 ? F<16, 64, 64, T>(__VA_ARGS__) : F<16, 32, 32, T>(__VA_ARGS__))

size_t km_assign3_scratch_bytes() { return sizeof(Sub3<float>); }

void km_assign3_args(const KmProblem (&p)[3], void *scratch, DeviceArgs *args) {
  using S16 = Sub3<uint16_t>;
  using S32 = Sub3<float>;
  static_assert(sizeof(S16) == sizeof(S32) && sizeof(S16) % 4 == 0 && sizeof(S16) <= 4 * kArgWords,
                "arguments fit DeviceArgs");
  args->dst = static_cast<uint32_t *>(scratch);
  args->words = static_cast<int>(sizeof(S16) / 4);
  if (p[0].bf16) {
    const S16 S = SCOPE_SUB3_T(sub3_args, uint16_t, p);
    memcpy(args->w, &S, sizeof(S));
  } else {
    const S32 S = SCOPE_SUB3_T(sub3_args, float, p);
    memcpy(args->w, &S, sizeof(S));
  }
}

hipError_t km_assign3(const KmProblem (&p)[3], void *scratch, hipStream_t s) {
  return p[0].bf16 ? SCOPE_SUB3_T(launch_mfma3, uint16_t, p, scratch, s)
                   : SCOPE_SUB3_T(launch_mfma3, float, p, scratch, s);
}
#undef SCOPE_SUB3_T

int km_cpad(int C) { return (C + 31) / 32 * 32; }
int km_dxp(int dx) { return dx <= 16 ? 16 : dx <= 32 ? 32 : dx <= 48 ? 48 : dx <= 64 ? 64 : 128; }

// Chunks of a codebook beyond the LDS (1 when it fits).
int km_parts(int C, int dx) {
  const int rows_max = kUbfLds / (2 * km_dxp(dx) + 8) / 32 * 32;
  return (km_cpad(C) + rows_max - 1) / rows_max;
}

size_t km_split_floats(int C, int dx, int heads, int n) {
  const int parts = km_parts(C, dx);
  if (parts <= 1) return 0;
  return static_cast<size_t>(heads) * n * (4 * static_cast<size_t>(parts) + 1);
}

// bf16 rows are read in channel pairs; fp32 rows have no condition.
// Codebooks beyond the LDS are split in chunks across blocks.
bool km_mfma_ok(bool bf16, int ld, int col0, int dx, int C) {
  if (dx > 128 || km_cpad(C) > kMaxCpad) return false;
  return !bf16 || !((ld | col0 | dx) & 1);
}

// Together never more than `cus` blocks (as long as that gives each one): the
// codebooks' LDS holds one block per CU, so a block too many would run alone
// after the others.
void km_block_shares(const double *cost, int nsub, int cus, long long most, int *blocks) {
  double sum = 0.0;
  for (int m = 0; m < nsub; ++m) sum += cost[m];
  int used = 0;
  for (int m = 0; m < nsub; ++m) {
    const int share = static_cast<int>(cus * cost[m] / sum);
    used += blocks[m] = share < 1 ? 1 : share;
  }
  // the blocks left over go where a block has the most to do; those that the
  // smallest subspaces got beyond their share come from where one is missed least
  for (; used < cus; ++used) {
    int at = 0;
    for (int m = 1; m < nsub; ++m)
      if (cost[m] * blocks[at] > cost[at] * blocks[m]) at = m;
    ++blocks[at];
  }
  for (; used > cus && used > nsub; --used) {
    int at = -1;
    for (int m = 0; m < nsub; ++m)
      if (blocks[m] > 1 && (at < 0 || cost[m] * (blocks[at] - 1) < cost[at] * (blocks[m] - 1))) at = m;
    --blocks[at];
  }
  for (int m = 0; m < nsub; ++m)
    if (blocks[m] > most) blocks[m] = static_cast<int>(most);
}

namespace {
template <typename T>
hipError_t assign_many(const KmProblem *p, int nsub, hipStream_t s) {
  ManyArgs<T> M{};
  M.heads = p[0].heads;
  // per 32 x 32 values: 4 dxp cycles of MFMA, 256 of the fold
  double cost[kMaxSub];
  for (int m = 0; m < nsub; ++m) cost[m] = static_cast<double>(p[m].cpad) * (4 * p[m].dxp + 256);
  const long long slices = static_cast<long long>(p[0].heads) * ((p[0].n + 31) / 32);
  int blocks[kMaxSub];
  km_block_shares(cost, nsub, cu_count(), (slices + kWaves<T> - 1) / kWaves<T>, blocks);
  for (int m = 0; m < nsub; ++m) {
    const KmProblem &q = p[m];
    M.first[m + 1] = M.first[m] + blocks[m];
    M.dxp[m] = q.dxp;
    M.a[m] = SliceArgs<T>{static_cast<const T *>(q.x), q.x_head_stride, q.ld, q.col0, q.dx,
                          q.n, q.C, q.cpad, q.u, q.u_head_stride, q.assign, q.a_head_stride,
                          nullptr, 0};
    M.ubf[m] = q.ubf;
    M.nu[m] = q.nu;
    M.bnd[m] = q.bnd;
  }
  M.nsub = nsub;
  hipLaunchKernelGGL(km_assign_mfma_many_kernel<T>, dim3(M.first[nsub]), dim3(64 * kWaves<T>), 0, s, M);
  return hipGetLastError();
}
template <typename T>
hipError_t assign_mfma(const KmProblem &p, bool with_hist, hipStream_t s) {
  switch (p.dxp) {
    case 16: return launch_mfma<16, T>(p, with_hist, s);
    case 32: return launch_mfma<32, T>(p, with_hist, s);
    case 48: return launch_mfma<48, T>(p, with_hist, s);
    case 64: return launch_mfma<64, T>(p, with_hist, s);
    default: return launch_mfma<128, T>(p, with_hist, s);
  }
}
}  // namespace

hipError_t km_assign_subspaces(const KmProblem *p, int nsub, hipStream_t s) {
  KmProblem fits[kMaxSub];
  int nfits = 0;
  for (int m = 0; m < nsub; ++m) {
    if (p[m].mfma && km_parts(p[m].C, p[m].dx) == 1) {
      fits[nfits++] = p[m];
    } else {
      const hipError_t e = km_assign(p[m], false, s);
      if (e != hipSuccess) return e;
    }
  }
  if (nfits == 0) return hipSuccess;
  if (nfits == 1) return km_assign(fits[0], false, s);
  return p[0].bf16 ? assign_many<uint16_t>(fits, nfits, s) : assign_many<float>(fits, nfits, s);
}

hipError_t km_assign_mfma(const KmProblem &p, bool with_hist, hipStream_t s) {
  return p.bf16 ? assign_mfma<uint16_t>(p, with_hist, s) : assign_mfma<float>(p, with_hist, s);
}

}  // namespace scope
