// K-means assignment on the matrix cores, exact with respect to the
// canonical assignment (argmin_r fl(||u_r||^2 - 2<x,u_r>) with fp32 fma-chain
// dot products in channel order, ties to the lowest r).
//
// bf16 points x are exact in bf16.  Each centroid is split into two bf16
// terms, u ~ hi + lo (hi = bf16(u), lo = bf16(u - hi)), so every product
// x_c hi_c and x_c lo_c is exact.  The MFMA accumulator starts at -nu_r / 2
// and two bf16 MFMAs per k-step add the products, which gives the halved,
// negated score
//   a_r = fl(-nu_r / 2 + <x, hi_r + lo_r>_mfma),   argmin_r c_r = argmax_r -c_r / 2.
// Summed in any order with one fp32 rounding per addition, the 2 DXP
// products and the start value err by at most 2 DXP 2^-24 (numax / 2 +
// |x| Nmax); the canonical score adds its dot product's DXP 2^-24 |x| Nmax and
// one rounding of the final fma.  So, in the canonical scale,
//   |-2 a_r - c_r| <= beta = 2|x| (E + 8 DXP 2^-24 Nmax)
//                            + 2^-23 ((2 DXP + 1) numax + 2.02 |x| Nmax)
// (E >= |u_r - hi_r - lo_r|, Nmax >= |hi_r| + |lo_r| and |u_r|, numax >=
// |nu_r|; twice the terms derived in numax, more in the others, for slack),
// inflated by 1%, and the canonical argmin r* satisfies a_{r*} >= max_r a_r - beta.
//
// One pass keeps, per point, the three largest a_r with the centroid index
// packed into the low mantissa bits (IB bits; this moves a value by less
// than delta = 2^(IB-23) |a|, added to the margin).  If the second-largest
// is more than beta + 2 delta below the largest, the largest's index is the
// only candidate and thus r*.  If only the third is, r* is one of the two
// largest, and the point's two half-wave lanes re-score one each with the
// canonical arithmetic.  For the very few points with three or more
// candidates, the wave recomputes the values, lists every candidate within
// the margin and re-scores them canonically.  In both cases the smallest
// canonical (score, r) wins, so equal scores keep the lowest index.
//
// fp32 points are split the same way, x = xh + xl + xr, and a third product
// joins the two: xh hi + xh lo + xl hi.  What is left out is xl lo (at most
// 2^-16 (1 + 2^-8)^2 |x| |u|) and xr u (2^-16 |x| |u|), so beta grows by
// 2 * 2^-15 * 1.02 |x| Nmax, and by 2^-110 (|x| + Nmax) where tiny terms are
// flushed; the constants above hold for 3 DXP products too (4/3 of the terms
// derived in numax, twice in |x| Nmax).  Points or
// codebooks so large that this arithmetic could overflow, or that are not
// finite, scan every centroid canonically.  With one thread per point and
// fma chains on the vector units a pass over 8 heads x 6417 points x 64
// centroids x 128 channels took 81 us; here it takes 20 us.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "common.h"
#include "kernels.h"

namespace scope {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// waves per block: fp32 points take twice the operand registers
template <typename T>
constexpr int kWaves = sizeof(T) == 2 ? 16 : 8;
constexpr int kUbfLds = 69632;            // two-term bf16 codebook elements in LDS
constexpr int kMaxCpad = 1024;
constexpr int kWaveCand = 64;             // candidate pairs per wave

__device__ __forceinline__ uint16_t to_bf16(float f) {
  bf16x2 r;
  r[0] = static_cast<__bf16>(f);
  r[1] = static_cast<__bf16>(0.0f);
  return static_cast<uint16_t>(__builtin_bit_cast(uint32_t, r) & 0xFFFFu);
}

// A pair of bf16 channels, at any element: the caller's pointer may be at an odd
// one (the hardware takes such loads whole; without the attribute the compiler
// could take them for aligned).
typedef uint32_t bf16_pair __attribute__((aligned(2)));

// Channels c0 .. c0+7 of one bf16 row as four packed pairs, zero from dx on
// and for invalid rows.  A whole group is one 16-byte load when the rows are
// 16-byte aligned (vec), else four loads of a pair (ld, col0 and dx are even, so
// no pair straddles dx).
__device__ __forceinline__ uint4 load_group8(const uint16_t *xrow, int c0, int dx, bool valid, bool vec) {
  uint4 v = make_uint4(0, 0, 0, 0);
  if (vec && c0 + 8 <= dx) {
    if (valid) v = *reinterpret_cast<const uint4 *>(xrow + c0);
  } else {
    uint32_t w[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int c = c0 + 2 * q;
      w[q] = valid && c < dx ? *reinterpret_cast<const bf16_pair *>(xrow + c) : 0u;
    }
    v = make_uint4(w[0], w[1], w[2], w[3]);
  }
  return v;
}

// The same 8 channels of an fp32 row.
__device__ __forceinline__ void load_group8(const float *xrow, int c0, int dx, bool valid, bool vec, float (&x)[8]) {
  if (vec && c0 + 8 <= dx) {
    float4 a = make_float4(0.0f, 0.0f, 0.0f, 0.0f), b = a;
    if (valid) {
      a = *reinterpret_cast<const float4 *>(xrow + c0);
      b = *reinterpret_cast<const float4 *>(xrow + c0 + 4);
    }
    x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
    x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
  } else {
#pragma unroll
    for (int q = 0; q < 8; ++q) x[q] = valid && c0 + q < dx ? xrow[c0 + q] : 0.0f;
  }
}

// Two floats -> packed bf16, rounded to nearest even.
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  bf16x2 r;
  r[0] = static_cast<__bf16>(a);
  r[1] = static_cast<__bf16>(b);
  return __builtin_bit_cast(uint32_t, r);
}

// Whether every row's first channel is 16-byte aligned.
template <typename T>
__device__ __forceinline__ bool rows_aligned(const T *x, size_t x_hs, int ld) {
  constexpr size_t per = 16 / sizeof(T);
  return (reinterpret_cast<uintptr_t>(x) & 15) == 0 && ((x_hs | static_cast<size_t>(ld)) & (per - 1)) == 0;
}

// A point's MFMA operands: one bf16 term per k-step, or for fp32 two.
template <int KS, typename T>
struct PointFrag {
  bf16x8 hi[KS];
  bf16x8 lo[sizeof(T) == 4 ? KS : 1];
};

// Loads the lane's half (channels 16 s + 8 hf ..) of a point's row; returns
// the partial sum of its squares (only sizes the margin).
template <int KS, typename T>
__device__ __forceinline__ float load_point(const T *xrow, int hf, int dx, bool valid, bool vec,
                                            PointFrag<KS, T> &f) {
  float ss = 0.0f;
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    if constexpr (sizeof(T) == 2) {
      const uint4 v4 = load_group8(xrow, 16 * s + 8 * hf, dx, valid, vec);
      const uint32_t wv[4] = {v4.x, v4.y, v4.z, v4.w};
      // two squares per dot2 (each rounding within 2^-23 relative, far inside
      // the 1e-4 slack of the norm)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bf16x2 p2 = __builtin_bit_cast(bf16x2, wv[q]);
        ss = __builtin_amdgcn_fdot2_f32_bf16(p2, p2, ss, false);
      }
      f.hi[s] = __builtin_bit_cast(bf16x8, v4);
    } else {
      float x[8];
      load_group8(xrow, 16 * s + 8 * hf, dx, valid, vec, x);
      uint32_t h[4], l[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float a = x[2 * q], b = x[2 * q + 1];
        ss = fmaf(a, a, ss);
        ss = fmaf(b, b, ss);
        h[q] = pack_bf16(a, b);
        l[q] = pack_bf16(a - __uint_as_float(h[q] << 16), b - __uint_as_float(h[q] & 0xFFFF0000u));
      }
      f.hi[s] = __builtin_bit_cast(bf16x8, make_uint4(h[0], h[1], h[2], h[3]));
      f.lo[s] = __builtin_bit_cast(bf16x8, make_uint4(l[0], l[1], l[2], l[3]));
    }
  }
  return ss;
}

// acc += <x, hi + lo> of the codebook rows at urow (this lane's row and half),
// for fp32 points without the product of the two low terms.
template <int DXP, typename T>
__device__ __forceinline__ void score_chain(const uint16_t *urow, const PointFrag<DXP / 16, T> &f,
                                            f32x16 &acc) {
#pragma unroll
  for (int s = 0; s < DXP / 16; ++s) {
    const bf16x8 a_hi = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(urow + 16 * s));
    const bf16x8 a_lo = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(urow + DXP + 16 * s));
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a_hi, f.hi[s], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a_lo, f.hi[s], acc, 0, 0, 0);
    if constexpr (sizeof(T) == 4)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a_hi, f.lo[s], acc, 0, 0, 0);
  }
}

// Canonical <x, u>: one fp32 fma per channel in ascending channel order, x
// in bf16 and u in fp32.  Both rows 16-byte aligned: eight channels per load
// step (the same chain), with the loads of four steps issued together; x
// 4-byte and u 8-byte aligned: two channels per step; then one at a time.
__device__ __forceinline__ float canon_dot(const uint16_t *xr, const float *u, int dx) {
  float dot = 0.0f;
  int c = 0;
  if (((reinterpret_cast<uintptr_t>(xr) | reinterpret_cast<uintptr_t>(u)) & 15) == 0) {
#pragma unroll 4
    for (; c + 8 <= dx; c += 8) {
      const uint4 xv = *reinterpret_cast<const uint4 *>(xr + c);
      const float4 u0 = *reinterpret_cast<const float4 *>(u + c);
      const float4 u1 = *reinterpret_cast<const float4 *>(u + c + 4);
      dot = fmaf(__uint_as_float(xv.x << 16), u0.x, dot);
      dot = fmaf(__uint_as_float(xv.x & 0xFFFF0000u), u0.y, dot);
      dot = fmaf(__uint_as_float(xv.y << 16), u0.z, dot);
      dot = fmaf(__uint_as_float(xv.y & 0xFFFF0000u), u0.w, dot);
      dot = fmaf(__uint_as_float(xv.z << 16), u1.x, dot);
      dot = fmaf(__uint_as_float(xv.z & 0xFFFF0000u), u1.y, dot);
      dot = fmaf(__uint_as_float(xv.w << 16), u1.z, dot);
      dot = fmaf(__uint_as_float(xv.w & 0xFFFF0000u), u1.w, dot);
    }
  }
  if (((reinterpret_cast<uintptr_t>(xr) & 3) | (reinterpret_cast<uintptr_t>(u) & 7)) == 0) {
#pragma unroll 4
    for (; c + 2 <= dx; c += 2) {
      const uint32_t xv = *reinterpret_cast<const uint32_t *>(xr + c);
      const float2 uv = *reinterpret_cast<const float2 *>(u + c);
      dot = fmaf(__uint_as_float(xv << 16), uv.x, dot);
      dot = fmaf(__uint_as_float(xv & 0xFFFF0000u), uv.y, dot);
    }
  }
  for (; c < dx; ++c) dot = fmaf(bf16_to_f32(xr[c]), u[c], dot);
  return dot;
}

// The same chain for fp32 points.
__device__ __forceinline__ float canon_dot(const float *xr, const float *u, int dx) {
  float dot = 0.0f;
  int c = 0;
  if (((reinterpret_cast<uintptr_t>(xr) | reinterpret_cast<uintptr_t>(u)) & 15) == 0) {
#pragma unroll 4
    for (; c + 8 <= dx; c += 8) {
      const float4 x0 = *reinterpret_cast<const float4 *>(xr + c);
      const float4 x1 = *reinterpret_cast<const float4 *>(xr + c + 4);
      const float4 u0 = *reinterpret_cast<const float4 *>(u + c);
      const float4 u1 = *reinterpret_cast<const float4 *>(u + c + 4);
      dot = fmaf(x0.x, u0.x, dot);
      dot = fmaf(x0.y, u0.y, dot);
      dot = fmaf(x0.z, u0.z, dot);
      dot = fmaf(x0.w, u0.w, dot);
      dot = fmaf(x1.x, u1.x, dot);
      dot = fmaf(x1.y, u1.y, dot);
      dot = fmaf(x1.z, u1.z, dot);
      dot = fmaf(x1.w, u1.w, dot);
    }
  }
#pragma unroll 4
  for (; c < dx; ++c) dot = fmaf(xr[c], u[c], dot);
  return dot;
}

// fp32 points and codebooks outside these limits (or not finite) take the
// full canonical scan.
constexpr float kNormLimit = 1e18f;      // |x|
constexpr float kNuLimit = 1e30f;        // |u|^2

// ascending-order key of a float score
__device__ __forceinline__ uint32_t asc_key(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// The canonical (score, index) key of the best of centroids first .. first + 3,
// first + stride .. first + stride + 3, ... for one fp32 point: the lowest score, of
// equal ones the lowest index.  NaN and +inf never win; ~0 if nothing does.  Four
// chains at a time share the point's loads; one at a time, half-zero or equal rows,
// whose centroids tie, made whole clusterings take several times as long (40 heads x
// 3000 rows of 64 channels, queries and keys, 4 iterations, all rows equal: 9.6 ms
// one at a time, 2.9 ms so).
__device__ __forceinline__ unsigned long long canon_scan(const float *xr, const float *u, const float *nu,
                                                         int C, int dx, int first, int stride) {
  const bool vec = ((reinterpret_cast<uintptr_t>(xr) | reinterpret_cast<uintptr_t>(u)) & 15) == 0 && (dx & 3) == 0;
  unsigned long long best = ~0ull;
  for (int r0 = first; r0 < C; r0 += stride) {
    const float *ur[4];
    float dot[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      ur[j] = u + static_cast<size_t>(min(r0 + j, C - 1)) * dx;
      dot[j] = 0.0f;
    }
    if (vec) {
#pragma unroll 2
      for (int c = 0; c < dx; c += 4) {
        const float4 x = *reinterpret_cast<const float4 *>(xr + c);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float4 w = *reinterpret_cast<const float4 *>(ur[j] + c);
          dot[j] = fmaf(x.x, w.x, dot[j]);
          dot[j] = fmaf(x.y, w.y, dot[j]);
          dot[j] = fmaf(x.z, w.z, dot[j]);
          dot[j] = fmaf(x.w, w.w, dot[j]);
        }
      }
    } else {
#pragma unroll 2
      for (int c = 0; c < dx; ++c) {
        const float x = xr[c];
#pragma unroll
        for (int j = 0; j < 4; ++j) dot[j] = fmaf(x, ur[j][c], dot[j]);
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int r = r0 + j;
      if (r >= C) break;
      const float sc = fmaf(-2.0f, dot[j], nu[r]) + 0.0f;
      if (!(sc < INFINITY)) continue;
      const unsigned long long key = (static_cast<unsigned long long>(asc_key(sc)) << 32) | static_cast<unsigned>(r);
      best = key < best ? key : best;
    }
  }
  return best;
}

// Keeps the compiler from moving this wave's LDS accesses across the call
// (the LDS completes one wave's operations in issue order).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The bound constants of one head's codebook.
struct FilterBound {
  float E, Nmax, numax;
};

// From the largest residual bound and the largest canonical norm.  Nmax bounds
// |u| (the norm's fma chain is within 2^-16 of |u|^2, or 2^-143 where it
// underflows) and |hi| + |lo| <= (1 + 2^-8)^2 |u|.
__device__ __forceinline__ FilterBound filter_bound(float e_max, float nu_max) {
  const float un = sqrtf(nu_max) * 1.001f + 1e-21f;
  return FilterBound{e_max + 1e-30f, un * 1.008f, nu_max * 1.001f};
}

// The head's bound constants from the per-wave maxima in red.
template <int NW>
__device__ __forceinline__ FilterBound reduce_bound(const float (*red)[NW]) {
  float E = 0.0f, numax = 0.0f;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    E = fmaxf(E, red[0][i]);
    numax = fmaxf(numax, red[1][i]);
  }
  return filter_bound(E, numax);
}

// Stages head h's two-term codebook (16-byte pieces of each row; LDS row
// stride 2 DXP + 8), its norms and the accumulator start values -nu / 2
// into LDS and returns the head's bound constants.  Ends with a block
// barrier; the caller makes sure no wave still reads the previous contents.
// CHECKED (fp32 points): a norm that is not below kNuLimit makes numax
// infinite.
template <int DXP, int NW, bool CHECKED>
__device__ __forceinline__ FilterBound stage_codebook(uint16_t *Us, float *nus, float *nhs,
                                                      float (*red)[NW],
                                                      const uint16_t *__restrict__ ubf,
                                                      const float *__restrict__ nu,
                                                      const float *__restrict__ bnd, int h,
                                                      int C, int cpad) {
  constexpr int US = 2 * DXP + 8;
  const int t = threadIdx.x;
  const int lane = t & 63, w = t >> 6;
  const uint16_t *ub = ubf + static_cast<size_t>(h) * cpad * (2 * DXP);
  for (int e = t; e < cpad * (DXP / 4); e += 64 * NW) {
    const int r = e / (DXP / 4), q = e % (DXP / 4);
    *reinterpret_cast<uint4 *>(&Us[r * US + 8 * q]) =
        *reinterpret_cast<const uint4 *>(ub + static_cast<size_t>(r) * (2 * DXP) + 8 * q);
  }
  // the head's bound constants: maxima over the rows
  float e_max = 0.0f, nu_max = 0.0f;
  for (int r = t; r < cpad; r += 64 * NW) {
    const size_t row = static_cast<size_t>(h) * cpad + r;
    const float v = nu[row];
    nus[r] = v;
    // exact for every norm at or above 2^-125 (smaller ones move by at most
    // 2^-150, far inside the margin); padding rows (nu = FLT_MAX) start at
    // -FLT_MAX / 2 and never win
    nhs[r] = -0.5f * v;
    if (r < C) {
      e_max = fmaxf(e_max, bnd[row]);
      nu_max = fmaxf(nu_max, fabsf(v));
      if (CHECKED && !(fabsf(v) < kNuLimit)) nu_max = INFINITY;
    }
  }
  e_max = wave_max(e_max);
  nu_max = wave_max(nu_max);
  if (lane == 0) {
    red[0][w] = e_max;
    red[1][w] = nu_max;
  }
  __syncthreads();
  return reduce_bound<NW>(red);
}

// The margin beta of a point of norm at most nx, in the canonical scale.
template <int DXP, typename T>
__device__ __forceinline__ float margin(float nx, FilterBound B) {
  const float kappa = 8.0f * DXP * 0x1p-24f;
  float beta = 2.0f * nx * (B.E + kappa * B.Nmax) +
               0x1p-23f * ((2.0f * DXP + 1.0f) * B.numax + 2.02f * nx * B.Nmax);
  if constexpr (sizeof(T) == 4) beta += 2.0f * 1.02f * 0x1p-15f * nx * B.Nmax + 0x1p-110f * (nx + B.Nmax);
  return beta * 1.01f + 1e-25f;
}

// a_r of the 32 centroids rb .. rb+31 of the staged codebook for the wave's 32
// points: the accumulator starts at -nu_r / 2 (lane holds rows rb + 8(e/4) +
// 4hf + e%4).
template <int DXP, typename T>
__device__ __forceinline__ f32x16 score_block(const uint16_t *Us, const float *nhs,
                                              const PointFrag<DXP / 16, T> &xf, int rb) {
  constexpr int US = 2 * DXP + 8;  // LDS row stride of the two-term codebook
  const int lane = threadIdx.x & 63, l32 = lane & 31, hf = lane >> 5;
  f32x16 acc;
  const float *nh = nhs + rb + 4 * hf;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float4 v = *reinterpret_cast<const float4 *>(nh + 8 * q);
    acc[4 * q + 0] = v.x;
    acc[4 * q + 1] = v.y;
    acc[4 * q + 2] = v.z;
    acc[4 * q + 3] = v.w;
  }
  score_chain<DXP, T>(&Us[(rb + l32) * US + 8 * hf], xf, acc);
  return acc;
}

// The three largest packed values of the codebook's first `rows` rows (a
// multiple of 32) per point, indices from r0 on (each med3 keeps the larger
// two of its inputs' lower pair; the start value lies below every value of
// valid inputs).  The index packed in the pass leaves out the lane's 4 hf,
// which is the same for all of the lane's values (so their order is that of
// the full index) and is added once after the pass.  The mask stays in a
// vector register so that the index, uniform across the wave, can come from a
// scalar register.
struct Top3 {
  float m1, m2, m3;
};
template <int DXP, typename T>
__device__ __forceinline__ Top3 top_scores(const uint16_t *Us, const float *nhs,
                                           const PointFrag<DXP / 16, T> &xf, int rows,
                                           uint32_t imask, int r0) {
  const int hf = (threadIdx.x & 63) >> 5;
  uint32_t vmask;
  asm volatile("v_mov_b32 %0, %1" : "=v"(vmask) : "s"(~imask));
  float m1 = -0x1.1p127f, m2 = -0x1.1p127f, m3 = -0x1.1p127f;
  auto chain = [&](int rb) { return score_block<DXP, T>(Us, nhs, xf, rb); };
  auto fold = [&](const f32x16 &acc, int rb) {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const uint32_t ru = static_cast<uint32_t>(
          __builtin_amdgcn_readfirstlane(r0 + rb + 8 * (e >> 2) + (e & 3)));
      const float sp = __uint_as_float((__float_as_uint(acc[e]) & vmask) | ru);
      m3 = __builtin_amdgcn_fmed3f(m2, m3, sp);
      m2 = __builtin_amdgcn_fmed3f(m1, m2, sp);
      m1 = __builtin_amdgcn_fmed3f(m1, sp, 0x1.1p127f);  // max without NaN quieting
    }
  };
  // software pipeline: the values of one block are folded while the MFMAs
  // of the next run; two accumulators alternate, so no copies
  f32x16 acc0 = chain(0), acc1;
  int rb = 32;
  for (; rb + 32 < rows; rb += 64) {
    acc1 = chain(rb);
    fold(acc0, rb - 32);
    acc0 = chain(rb + 32);
    fold(acc1, rb);
  }
  if (rb < rows) {
    acc1 = chain(rb);
    fold(acc0, rb - 32);
    fold(acc1, rb);
  } else {
    fold(acc0, rb - 32);
  }
  const uint32_t add = 4u * static_cast<uint32_t>(hf);
  m1 = __uint_as_float(__float_as_uint(m1) + add);
  m2 = __uint_as_float(__float_as_uint(m2) + add);
  m3 = __uint_as_float(__float_as_uint(m3) + add);
  // the other half-wave's three into this one's (same multiset, same
  // result in both halves)
  const float o[3] = {__shfl_xor(m1, 32), __shfl_xor(m2, 32), __shfl_xor(m3, 32)};
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    m3 = __builtin_amdgcn_fmed3f(m2, m3, o[q]);
    m2 = __builtin_amdgcn_fmed3f(m1, m2, o[q]);
    m1 = __builtin_amdgcn_fmed3f(m1, o[q], 0x1.1p127f);
  }
  return Top3{m1, m2, m3};
}

// One codebook's view of the rows: channels col0 .. col0+dx of X[h] (row
// stride ld), C centroids (padded to cpad) U[h] in fp32 for the canonical
// re-score, and where the assignment goes.
template <typename T>
struct SliceArgs {
  const T *X;
  size_t x_hs;
  int ld, col0, dx, n, C, cpad;
  const float *U;
  size_t u_hs;
  int32_t *assign;
  size_t a_hs;
  int32_t *chunk_hist;
  int nchunks;
};

// The assignment of the 32 points of slice sl of head h by one wave, against
// the codebook staged in Us/nus/nhs with bound constants B (candidate
// scratch of this wave: cand, best, ncand).
// Returns the lane's point's centroid (lane l and l + 32 hold the same point).
template <int DXP, typename T>
__device__ __forceinline__ int assign_slice(const SliceArgs<T> &A, const uint16_t *Us,
                                             const float *nus, const float *nhs, FilterBound B,
                                             int h, int sl,
                                             uint32_t *cand_w, unsigned long long *best_w,
                                             int *ncand_w) {
  constexpr int KS = DXP / 16;     // MFMA k-steps per term
  const int lane = threadIdx.x & 63, l32 = lane & 31, hf = lane >> 5;
  const T *X = A.X;
  const size_t x_hs = A.x_hs;
  const int ld = A.ld, col0 = A.col0, dx = A.dx, n = A.n, C = A.C, cpad = A.cpad;
  int32_t *assign = A.assign;
  const size_t a_hs = A.a_hs;
  int32_t *chunk_hist = A.chunk_hist;
  const int nchunks = A.nchunks;
  // index bits packed into the low mantissa of the scores
  const int ib = 32 - __clz(cpad - 1);
  const uint32_t imask = (1u << ib) - 1u;
  const float dpack = __uint_as_float(static_cast<uint32_t>(127 + ib - 23) << 23);  // 2^(ib-23)
  const bool vec = rows_aligned(X + col0, x_hs, ld);
  const float *Uh = A.U + h * A.u_hs;
  const int i = sl * 32 + l32;
  const bool valid = i < n;
  const T *xrow = X + h * x_hs + static_cast<size_t>(valid ? i : 0) * ld + col0;
  PointFrag<KS, T> xf;
  float ss = load_point<KS, T>(xrow, hf, dx, valid, vec, xf);
  ss += __shfl_xor(ss, 32);
  const float nx = sqrtf(ss) * 1.0001f + 1e-30f;
  const float beta = margin<DXP, T>(nx, B);

  auto chain = [&](int rb) { return score_block<DXP, T>(Us, nhs, xf, rb); };
  const Top3 top = top_scores<DXP, T>(Us, nhs, xf, cpad, imask, 0);
  const float m1 = top.m1, m2 = top.m2, m3 = top.m3;
  // candidates: a_r >= max a - beta (halved scale: 2 x beta / 2), less the
  // two packing perturbations
  const float slack = (beta + 2.0f * dpack * fabsf(m1)) * 1.001f;
  const float lim = m1 - slack;
  const float thr = lim - fabsf(lim) * 2e-6f - 1e-30f;
  // outside the filter's range (fp32 only): every centroid, canonically
  const bool unsafe = sizeof(T) == 4 && valid && !(nx < kNormLimit && B.numax < kNuLimit * 1.01f);
  const bool needy = valid && !unsafe && !(m2 < thr);
  // three or more candidates (very rare)
  const bool wide = needy && !(m3 < thr);
  int arg = static_cast<int>(__float_as_uint(m1) & imask);
  bool scan = unsafe;  // fp32: a canonical scan of every centroid

  if (__ballot(needy && !wide)) {
    // exactly two candidates, the two largest packed values: the point's
    // two half-wave lanes re-score one each canonically and exchange
    unsigned long long key = ~0ull;
    if (needy && !wide) {
      const int r = min(static_cast<int>(__float_as_uint(hf ? m2 : m1) & imask), C - 1);
      const T *xr = X + h * x_hs + static_cast<size_t>(i) * ld + col0;
      const float dot = canon_dot(xr, Uh + static_cast<size_t>(r) * dx, dx);
      const float sc = fmaf(-2.0f, dot, nus[r]) + 0.0f;
      key = (static_cast<unsigned long long>(asc_key(sc)) << 32) | static_cast<unsigned>(r);
    }
    const uint32_t ok_lo = __shfl_xor(static_cast<uint32_t>(key), 32);
    const uint32_t ok_hi = __shfl_xor(static_cast<uint32_t>(key >> 32), 32);
    const unsigned long long other = (static_cast<unsigned long long>(ok_hi) << 32) | ok_lo;
    if (needy && !wide) arg = static_cast<int>((key < other ? key : other) & 0xFFFFFFFFu);
  }
  const uint64_t wides = __ballot(wide);
  if (sizeof(T) == 4 && 3 * (__popcll(wides) / 2) > kWaveCand) {
    scan = scan || wide;  // their candidates cannot all be listed
  } else if (wides) {
    // every candidate of the wide points, re-scored canonically
    wave_sync();
    if (lane == 0) *ncand_w = 0;
    if (lane < 32) best_w[lane] = ~0ull;
    wave_sync();
    bool over = false;
    for (int rb = 0; rb < cpad; rb += 32) {
      const f32x16 acc = chain(rb);
      if (wide) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const uint32_t r = static_cast<uint32_t>(rb + 8 * (e >> 2) + 4 * hf + (e & 3));
          const float sp = __uint_as_float((__float_as_uint(acc[e]) & ~imask) | r);
          if (static_cast<int>(r) < C && sp >= thr) {
            const int slot = atomicAdd(ncand_w, 1);
            if (slot < kWaveCand)
              cand_w[slot] = (static_cast<uint32_t>(l32) << 16) | r;
            else
              over = true;
          }
        }
      }
    }
    // a point whose candidates did not fit scans every centroid
    const bool full = __shfl_xor(static_cast<int>(over), 32) || over;
    wave_sync();
    const int cnt = min(*ncand_w, kWaveCand);
    for (int k = lane; k < cnt; k += 64) {
      const uint32_t pr = cand_w[k];
      const int q = static_cast<int>(pr >> 16), r = static_cast<int>(pr & 0xFFFFu);
      const T *xr = X + h * x_hs + static_cast<size_t>(sl * 32 + q) * ld + col0;
      const float *u = Uh + static_cast<size_t>(r) * dx;
      const float dot = canon_dot(xr, u, dx);
      const float sc = fmaf(-2.0f, dot, nus[r]) + 0.0f;
      atomicMin(&best_w[q], (static_cast<unsigned long long>(asc_key(sc)) << 32) | static_cast<unsigned>(r));
    }
    wave_sync();
    if (wide && hf == 0) {
      unsigned long long b = best_w[l32];
      if (sizeof(T) == 2 && full) {
        const T *xr = X + h * x_hs + static_cast<size_t>(i) * ld + col0;
        b = ~0ull;
        for (int r = 0; r < C; ++r) {
          const float *u = Uh + static_cast<size_t>(r) * dx;
          const float dot = canon_dot(xr, u, dx);
          const float sc = fmaf(-2.0f, dot, nus[r]) + 0.0f;
          const unsigned long long key = (static_cast<unsigned long long>(asc_key(sc)) << 32) | static_cast<unsigned>(r);
          b = key < b ? key : b;
        }
      }
      arg = b == ~0ull ? 0 : static_cast<int>(b & 0xFFFFFFFFu);
    }
    arg = __shfl(arg, l32);  // the lower half-wave holds the result
    scan = scan || (wide && full);
  }
  if constexpr (sizeof(T) == 4) {
    if (__builtin_expect(__ballot(scan) != 0, 0)) {
      // the point's two lanes take every other four centroids
      unsigned long long key = ~0ull;
      if (scan) key = canon_scan(xrow, Uh, nus, C, dx, 4 * hf, 8);
      const unsigned long long other = __shfl_xor(key, 32);
      if (other < key) key = other;
      if (scan) arg = key == ~0ull ? 0 : static_cast<int>(key & 0xFFFFFFFFu);
    }
  }
  arg = min(max(arg, 0), C - 1);
  if (valid && hf == 0) {
    assign[h * a_hs + i] = arg;
    if (chunk_hist)
      atomicAdd(&chunk_hist[(static_cast<size_t>(h) * nchunks + (i / kAssignBlock)) * C + arg], 1);
  }
  return arg;
}

}  // namespace

}  // namespace scope
