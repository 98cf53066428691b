// Sparse attention over the selected keys (Eq. 11; Alg. 1 last step), and
// dense attention (Eq. 1) as the one-cluster special case.
//
// Work item = (head, query cluster c, chunk of up to 32*NW of its queries).
// The block gathers the cluster's selected keys 64 at a time, K and V rows
// both into LDS row-major.  Each wave owns 32 queries and runs
//   S^T (64 keys x 32 queries) = K_tile . Q^T       bf16 MFMA 32x32x16,
//                                 two 32-key chains interleaved
//   online softmax in fp32 (exp2 domain), one query per lane column, one
//                                 max / rescale decision per 64-key tile
//   O^T (d x 32 queries)      += V_tile^T . P^T      bf16 MFMA 32x32x16
// The S^T accumulator layout is reused directly as the B operand of the
// second product, so P never leaves registers; the matching V^T operand
// comes from the row-major V tile through transposing LDS reads
// (ds_read_b64_tr_b16).  K/V tiles are double buffered: the next tiles'
// gathers are in flight during the MFMAs.  bf16 gathers go through buffer
// resources, whose range checks turn every out-of-range index into a zero
// read instead of a fault, and the buffer unit writes the gathered rows
// straight into LDS (attn_kernel_dma).  fp32 inputs are rounded to bf16: K and
// V by one pass into the workspace, or without workspace row by row through
// registers (attn_kernel).
#include <math.h>

#include <mutex>

#include "common.h"
#include "kernels.h"

namespace scope {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4 lds_i16x4;

constexpr int kBN = 64;          // keys per tile
constexpr int kNW = 8;           // waves per block
constexpr int kQB = 1;           // 32-query column blocks per wave
constexpr int kBM = 32 * kQB * kNW;
constexpr float kRescale = 8.0f; // lazy rescale: running max may lag by 2^8

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 u) {
  return __builtin_bit_cast(bf16x8, u);
}

// Two floats -> packed bf16 (round to nearest even, v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  bf16x2 r;
  r[0] = static_cast<__bf16>(a);
  r[1] = static_cast<__bf16>(b);
  return __builtin_bit_cast(uint32_t, r);
}

// 8 consecutive input elements as packed bf16.
template <bool BF16IN>
__device__ __forceinline__ uint4 load8(const void *base, size_t elem) {
  if (BF16IN) {
    return *reinterpret_cast<const uint4 *>(static_cast<const uint16_t *>(base) + elem);
  } else {
    const float4 a = *reinterpret_cast<const float4 *>(static_cast<const float *>(base) + elem);
    const float4 b = *reinterpret_cast<const float4 *>(static_cast<const float *>(base) + elem + 4);
    return make_uint4(pack_bf16(a.x, a.y), pack_bf16(a.z, a.w), pack_bf16(b.x, b.y),
                      pack_bf16(b.z, b.w));
  }
}

// Work slots run in list order: heads one after the other and, within a
// head, by estimated cost, largest first, with a cluster's row chunks
// adjacent.  All XCDs work on the same head at a time, so one head's K/V
// (60 MB at 118800 x 128 bf16) is what the 256 MB memory-side cache has to
// hold.  (Where several heads' fit there, attn_plan_kernel gives the order.)
//
// Block b runs on XCD b mod 8.  Runs of kRun consecutive work slots (the
// chunks of one cluster, which gather the same K/V rows) go to one XCD so
// that they share its L2; windows of 8 * kRun slots still follow the list
// order.  A partial last window keeps the identity map.
constexpr int kXcds = 8, kRun = 4;
constexpr uint64_t kMemorySideCache = 256ull << 20;
__device__ __forceinline__ int xcd_item(int b, int total) {
  constexpr int W = kXcds * kRun;
  const int w0 = b / W * W;
  if (w0 + W > total) return b;
  const int r = b - w0;
  return w0 + (r % kXcds) * kRun + r / kXcds;
}

// fp32 inputs without workspace for bf16 copies of K and V: rows are rounded
// to bf16 on the way through registers.
template <int D>
__global__ __launch_bounds__(kNW * 64) void attn_kernel(
    int n, int c_q, int items_per_head, int total_items,
    const void *__restrict__ qv, const void *__restrict__ kv,
    const void *__restrict__ vv, void *ov, const int32_t *__restrict__ offsets,
    const int32_t *__restrict__ perm, const int32_t *__restrict__ sel_idx,
    const int4 *__restrict__ items, float scale_log2) {
  constexpr int NT = kNW * 64;
  // LDS row strides (bf16 elements): K rows are read 16 bytes per lane, 16
  // consecutive rows at a time, so 16 bytes of padding keep them on distinct
  // banks; the transposing V reads take 64 bytes from each of four rows per
  // 32 lanes, so V rows are padded by 64 bytes (stride = 64 mod 256 bytes)
  constexpr int KS = D + 8;
  constexpr int KSV = D + 32;
  constexpr int C8 = D / 8;       // 16-byte chunks per row
  // staging: the first half of the block stages V (4 consecutive keys of one
  // 8-channel column per thread), the second half K (RK consecutive rows of
  // one 16-byte column per thread)
  constexpr int HALF = NT / 2;
  constexpr int RK = kBN * C8 / HALF;       // rows per staging thread
  static_assert(kBN * C8 % HALF == 0 && RK >= 1 && RK <= 4, "tile/threads mismatch");
  constexpr int NR = 4;                     // rows fetched per thread per tile
  __shared__ __attribute__((aligned(16))) uint16_t Ks[2][kBN * KS];
  __shared__ __attribute__((aligned(16))) uint16_t Vs[2][kBN * KSV];

  const int item = xcd_item(static_cast<int>(blockIdx.x), total_items);
  if (item >= total_items) return;
  const int h = item / items_per_head;
  const int4 it = items[2 * item];  // work slots of this kernel hold one chunk
  const int c = it.x, row0 = it.y, rows = it.z, r = it.w;
  if (rows <= 0) return;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int l32 = lane & 31, hf = lane >> 5;
  const size_t hoff = static_cast<size_t>(h) * n * D;

  // queries: wave w owns rows w*32*kQB + 32*qb + l32 of the chunk
  int qi[kQB];
  bool qvalid[kQB];
  bf16x8 qf[kQB][D / 16];
#pragma unroll
  for (int qb = 0; qb < kQB; ++qb) {
    const int ql = w * 32 * kQB + 32 * qb + l32;
    qvalid[qb] = ql < rows;
    qi[qb] = 0;
    if (qvalid[qb]) {
      const int pb = offsets[static_cast<size_t>(h) * (c_q + 1) + c] + row0 + ql;
      qi[qb] = min(max(perm[static_cast<size_t>(h) * n + min(max(pb, 0), n - 1)], 0), n - 1);
    }
#pragma unroll
    for (int s = 0; s < D / 16; ++s)
      qf[qb][s] = as_bf16x8(qvalid[qb] ? load8<false>(qv, hoff + static_cast<size_t>(qi[qb]) * D + 16 * s + 8 * hf)
                                       : make_uint4(0, 0, 0, 0));
  }
  const bool wave_active = w * 32 * kQB < rows;

  f32x16 oacc[kQB][D / 32];
#pragma unroll
  for (int qb = 0; qb < kQB; ++qb)
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int e = 0; e < 16; ++e) oacc[qb][db][e] = 0.0f;
  float m_run[kQB], l_run[kQB];
#pragma unroll
  for (int qb = 0; qb < kQB; ++qb) {
    m_run[qb] = -INFINITY;
    l_run[qb] = 0.0f;
  }

  const int32_t *sel = sel_idx + (static_cast<size_t>(h) * c_q + c) * n;
  const int ntiles = (r + kBN - 1) / kBN;

  // this thread's staging role (wave-uniform, kept in scalar registers):
  // the first half of the block stages V rows, the second K rows, both
  // row-major, RK consecutive rows of one 16-byte column per thread
  const bool is_v = __builtin_amdgcn_readfirstlane(t) < HALF;
  const int u = is_v ? t : t - HALF;
  const int c8 = u % C8;
  const int key0 = RK * (u / C8) % kBN;
  const bool stores = true;
  // transposing reads of V (ds_read_b64_tr_b16): source lane s supplies
  // row 4*(s/32) + (s%16)/4 and channels 16*((s/16)%2) + 4*(s%4) .. +3 of a
  // 16-key step; lane L then holds 4 consecutive keys of channel L%32
  const int tr_off = (4 * (lane >> 5) + ((lane & 15) >> 2)) * KSV + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  const void *src = is_v ? vv : kv;
  // Software pipeline, two tiles deep: step T requests the row indices of
  // tile T+3 first and the rows of tile T+2 after its compute, so waiting for
  // indices never waits for rows in flight (vector loads complete in order)
  // and the rows have a whole step to arrive.  Every load is
  // unconditional with clamped indices, so the pipeline has no branches;
  // rows past the key set are fetched but masked (or never read).
  int selA[NR], selB[NR];
  uint4 dA[NR], dB[NR];
  auto load_sel = [&](int tile, int (&sx)[NR]) {
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      sx[i] = sel[min(tile * kBN + key0 + i % RK, n - 1)];
    }
  };
  auto load_rows = [&](const int (&sx)[NR], uint4 (&dx)[NR]) {
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int row = min(max(sx[i], 0), n - 1);
      dx[i] = load8<false>(src, hoff + static_cast<size_t>(row) * D + 8 * c8);
    }
  };
  auto store_rows = [&](int buf, const uint4 (&dx)[NR]) {
    if (!stores) return;
    uint16_t *dst = is_v ? Vs[buf] : Ks[buf];
#pragma unroll
    for (int i = 0; i < RK; ++i)
      *reinterpret_cast<uint4 *>(&dst[(key0 + i) * (is_v ? KSV : KS) + 8 * c8]) = dx[i];
  };

  auto compute = [&](int tile, int buf) {
    if (!wave_active) return;
    // S^T for both 32-key blocks of the tile: two independent MFMA chains,
    // interleaved so the matrix pipe never waits on one accumulator
    f32x16 sacc[2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int e = 0; e < 16; ++e) sacc[kb][e] = 0.0f;
#pragma unroll
    for (int s = 0; s < D / 16; ++s)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        const bf16x8 a = as_bf16x8(*reinterpret_cast<const uint4 *>(
            &Ks[buf][(kb * 32 + l32) * KS + 16 * s + 8 * hf]));
        sacc[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[0][s], sacc[kb], 0, 0, 0);
      }
    // lane holds keys 32kb + 8(e/4) + 4hf + (e%4) of query column l32
    const int kbase = tile * kBN;
    if (kbase + kBN > r) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int e = 0; e < 16; ++e)
          if (kbase + 32 * kb + 8 * (e >> 2) + 4 * hf + (e & 3) >= r) sacc[kb][e] = -INFINITY;
    }
    float mx0 = fmaxf(sacc[0][0], sacc[0][1]), mx1 = fmaxf(sacc[1][0], sacc[1][1]);
#pragma unroll
    for (int e = 2; e < 16; e += 2) {
      mx0 = fmaxf(fmaxf(mx0, sacc[0][e]), sacc[0][e + 1]);
      mx1 = fmaxf(fmaxf(mx1, sacc[1][e]), sacc[1][e + 1]);
    }
    float mx = fmaxf(mx0, mx1);
    {
      // the other half-wave holds the query's other keys
      const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
      mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
    }
    const float mt = mx * scale_log2;
    // rescale only when the running max falls too far behind; the branch is
    // wave-wide but each query decides for itself (alpha = 1 otherwise), so
    // a query's result never depends on its wave-mates
    const bool behind = mt > m_run[0] + kRescale;
    if (__ballot(behind)) {
      const float m_new = behind ? fmaxf(m_run[0], mt) : m_run[0];
      const float alpha = behind ? __builtin_amdgcn_exp2f(m_run[0] - m_new) : 1.0f;
      l_run[0] *= alpha;
#pragma unroll
      for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) oacc[0][db][e] *= alpha;
      m_run[0] = m_new;
    }
    const float neg_m = -m_run[0];
    uint4 pk[2][2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      float p[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) p[e] = __builtin_amdgcn_exp2f(fmaf(sacc[kb][e], scale_log2, neg_m));
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2)
        pk[kb][s2] = make_uint4(pack_bf16(p[8 * s2 + 0], p[8 * s2 + 1]),
                                pack_bf16(p[8 * s2 + 2], p[8 * s2 + 3]),
                                pack_bf16(p[8 * s2 + 4], p[8 * s2 + 5]),
                                pack_bf16(p[8 * s2 + 6], p[8 * s2 + 7]));
    }
    // the row sum of the bf16 weights the PV product uses, two per dot2
    {
      const bf16x2 one = __builtin_bit_cast(bf16x2, 0x3F803F80u);
      float ps[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
          const uint4 w4 = pk[kb][s2];
          ps[0] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w4.x), one, ps[0], false);
          ps[1] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w4.y), one, ps[1], false);
          ps[2] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w4.z), one, ps[2], false);
          ps[3] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w4.w), one, ps[3], false);
        }
      l_run[0] += (ps[0] + ps[1]) + (ps[2] + ps[3]);
    }
    // O^T += V_tile^T . P^T in 16-key steps, four independent accumulators
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
        for (int db = 0; db < D / 32; ++db) {
          const uint16_t *vt = &Vs[buf][(kb * 32 + 16 * s2) * KSV + db * 32 + tr_off];
          const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4 *)(vt));
          const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4 *)(vt + 8 * KSV));
          const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
          const bf16x8 a = as_bf16x8(make_uint4(l2.x, l2.y, h2.x, h2.y));
          oacc[0][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
              a, as_bf16x8(pk[kb][s2]), oacc[0][db], 0, 0, 0);
        }
  };

  // one pipeline step: compute tile T from LDS while tile T+1 (already in
  // registers `cur`) lands in the other LDS buffer; the rows of tile T+2
  // are requested after the compute (they have until the end of the next
  // step), so the MFMAs of this step never wait for them
  auto step = [&](int tile, int (&sel_next)[NR], uint4 (&cur)[NR],
                  int (&sel_far)[NR], uint4 (&far)[NR]) {
    load_sel(tile + 3, sel_next);
    compute(tile, tile & 1);
    load_rows(sel_far, far);
    store_rows((tile + 1) & 1, cur);
    __syncthreads();
  };

  if (ntiles > 0) {
    load_sel(0, selA);
    load_sel(1, selB);
    load_rows(selA, dA);   // tile 0
    load_sel(2, selA);
    load_rows(selB, dB);   // tile 1
    store_rows(0, dA);
  }
  __syncthreads();
  // registers: tile T+1 is in (T even ? dB : dA); the row indices of tile
  // T+2 in (T even ? selA : selB)
  for (int tile = 0; tile < ntiles; tile += 2) {
    step(tile, selB, dB, selA, dA);
    if (tile + 1 < ntiles) step(tile + 1, selA, dA, selB, dB);
  }

#pragma unroll
  for (int qb = 0; qb < kQB; ++qb) {
    // lanes l and l^32 hold the two halves of one query's row sum
    const float l_tot = l_run[qb] + __shfl_xor(l_run[qb], 32);
    if (!qvalid[qb]) continue;
    const float inv = l_tot > 0.0f ? 1.0f / l_tot : 0.0f;
    // lane holds O^T[32db + 8i + 4hf + j][query]
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int dim = db * 32 + 8 * i + 4 * hf;
        const size_t at = hoff + static_cast<size_t>(qi[qb]) * D + dim;
        const float o0 = oacc[qb][db][4 * i + 0] * inv, o1 = oacc[qb][db][4 * i + 1] * inv;
        const float o2 = oacc[qb][db][4 * i + 2] * inv, o3 = oacc[qb][db][4 * i + 3] * inv;
        *reinterpret_cast<float4 *>(static_cast<float *>(ov) + at) = make_float4(o0, o1, o2, o3);
      }
  }
}

__device__ __forceinline__ int key_tiles(const int4 &e) { return e.z > 0 ? (e.w + kBN - 1) / kBN : 0; }

// Half a slot: the queries of its waves 0 .. kNW/2 - 1 (half 1) or of the others
// (half 2).  A query's result depends neither on its wave nor on its block, so
// halves give the slot's results bit for bit.
__device__ __forceinline__ void take_half(int4 *a, int4 *b, int half) {
  const int first = half == 2 ? kNW / 2 : 0;
  // the rows of an entry, whose first wave is w0, that the half's waves hold
  auto cut = [&](int4 *e, int w0) {
    const int from = min(max(32 * (first - w0), 0), e->z);
    const int to = min(max(32 * (first + kNW / 2 - w0), 0), e->z);
    e->y += from;
    e->z = to - from;
  };
  const int wa = (a->z + 31) >> 5;
  cut(a, 0);
  cut(b, wa);
  if (a->z <= 0) {
    *a = *b;
    b->z = 0;
  }
}

// The same computation with bf16 K/V rows gathered straight into LDS by the
// buffer unit (one 1 KB load per 4 rows at d = 128, per 8 rows at d = 64; no
// staging registers).  fp32 inputs come here too, their K and V rounded to
// bf16 in the workspace by one pass before (Q is rounded on load, O written in
// fp32): the same values as rounding each gathered row.  Rows land unpadded,
// so 16-byte slots are XOR-swizzled.  d = 128 (a row is all 64 banks): slot =
// chunk ^ (row mod 16) in K tiles (16-row b128 reads) and chunk ^ 4 (row mod
// 4) in V tiles (4-row transposing reads).  d = 64 (two rows span the banks):
// chunk ^ (row / 2 mod 8) in K tiles, chunk ^ 4 (row / 2 mod 2) in V tiles.  A
// work slot may hold two chunks (A, B) of different clusters: A's waves come
// first, each chunk has its own tiles, and every wave gathers its share of
// both.  The four tile buffers (K and V, two steps) are distinct LDS objects,
// each holding the tiles of both chunks, so the compiler's waits for the loads
// into one never hold up the reads of another.
template <int D>
using DmaTile = uint16_t[2][kBN * D];

template <int D, bool BF16IO, bool PAIRED>
__device__ __forceinline__ void attn_dma_body(
    int n, int c_q, int h, const int4 &ia, const int4 &ib,
    const void *__restrict__ qv,
    const void *__restrict__ kv, const void *__restrict__ vv, void *ov,
    const int32_t *__restrict__ offsets, const int32_t *__restrict__ perm,
    const int32_t *__restrict__ sel_idx, float scale_log2, DmaTile<D> &K0, DmaTile<D> &K1,
    DmaTile<D> &V0, DmaTile<D> &V1) {
  constexpr int CH = D / 8;        // 16-byte chunks per row
  constexpr int RPL = 64 / CH;     // rows per gather load
  constexpr int NG = 8 / RPL;      // gather loads per wave, tile and matrix
  // the 16-byte slot of a row's chunk 0 (chunk c: slot ^ c)
  auto k_swz = [](int row) { return D == 128 ? row & 15 : (row >> 1) & 7; };
  auto v_swz = [](int row) { return D == 128 ? 4 * (row & 3) : 4 * ((row >> 1) & 1); };
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int l32 = lane & 31, hf = lane >> 5;
  const size_t hoff = static_cast<size_t>(h) * n * D;
  // this wave's chunk: A's ceil(rows / 32) waves first, then B's
  const int wa = (ia.z + 31) >> 5;
  const int g = PAIRED && w >= wa ? 1 : 0;
  const int4 it = g ? ib : ia;
  const int c = it.x, row0 = it.y, rows = it.z, r = it.w;
  const int wl = w - (g ? wa : 0);

  // queries: wave wl of the chunk owns its rows 32 wl + l32
  const int ql = wl * 32 + l32;
  const bool qvalid = ql < rows;
  int qi = 0;
  if (qvalid) {
    const int pb = offsets[static_cast<size_t>(h) * (c_q + 1) + c] + row0 + ql;
    qi = min(max(perm[static_cast<size_t>(h) * n + min(max(pb, 0), n - 1)], 0), n - 1);
  }
  bf16x8 qf[D / 16];
#pragma unroll
  for (int s = 0; s < D / 16; ++s)
    qf[s] = as_bf16x8(qvalid ? load8<BF16IO>(qv, hoff + static_cast<size_t>(qi) * D + 16 * s + 8 * hf)
                             : make_uint4(0, 0, 0, 0));
  const bool wave_active = wl * 32 < rows;

  f32x16 oacc[D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int e = 0; e < 16; ++e) oacc[db][e] = 0.0f;
  float m_run = -INFINITY, l_run = 0.0f;

  // key tiles of each chunk; the block steps through the longer list
  const int ntA = (ia.w + kBN - 1) / kBN, ntB = PAIRED ? (ib.w + kBN - 1) / kBN : 0;
  const int ntiles = ntA > ntB ? ntA : ntB;
  const int nt_own = (r + kBN - 1) / kBN;
  auto sel_rsrc = [&](const int4 &e) {
    return __builtin_amdgcn_make_buffer_rsrc(
        const_cast<int32_t *>(sel_idx + (static_cast<size_t>(h) * c_q + e.x) * n),
        static_cast<short>(0), e.w * 4, 0x00020000);
  };
  const __amdgpu_buffer_rsrc_t rselA = sel_rsrc(ia);
  const __amdgpu_buffer_rsrc_t rselB = PAIRED ? sel_rsrc(ib) : rselA;
  const int nbytes = static_cast<int>(static_cast<uint32_t>(n) * (D * 2));
  const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t *>(static_cast<const uint16_t *>(kv) + hoff), static_cast<short>(0), nbytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t *>(static_cast<const uint16_t *>(vv) + hoff), static_cast<short>(0), nbytes, 0x00020000);

  // gathers: wave w brings rows 8w .. 8w+7 of each chunk's tile, RPL rows
  // (1 KB) per load; lane L covers row 8w + RPL i + L/CH, slot L%CH, and
  // fetches the chunk that the swizzle puts there.  Past the end of a
  // chunk's key list its index loads read zeros, so its gathers fetch row 0
  // (the pairing matches key counts, so few such tiles).
  struct Idx {
    int a[NG], b[NG];
  };
  auto load_idx = [&](int tile, Idx &ix) {
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      const int at = (tile * kBN + 8 * w + RPL * i + lane / CH) * 4;
      ix.a[i] = __builtin_amdgcn_raw_buffer_load_b32(rselA, at, 0, 0);
      ix.b[i] = PAIRED ? __builtin_amdgcn_raw_buffer_load_b32(rselB, at, 0, 0) : 0;
    }
  };
  auto gather_k = [&](uint16_t (*kbuf)[kBN * D], const Idx &ix) {
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      const int row = 8 * w + RPL * i + lane / CH, s = lane % CH;
      const int col = 16 * (s ^ k_swz(row));
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rk, kbuf[0] + (8 * w + RPL * i) * D, 16, ix.a[i] * (D * 2) + col, 0, 0, 0);
      if constexpr (PAIRED)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rk, kbuf[1] + (8 * w + RPL * i) * D, 16, ix.b[i] * (D * 2) + col, 0, 0, 0);
    }
  };
  auto gather_v = [&](uint16_t (*vbuf)[kBN * D], const Idx &ix) {
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      const int row = 8 * w + RPL * i + lane / CH, s = lane % CH;
      const int col = 16 * (s ^ v_swz(row));
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rv, vbuf[0] + (8 * w + RPL * i) * D, 16, ix.a[i] * (D * 2) + col, 0, 0, 0);
      if constexpr (PAIRED)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rv, vbuf[1] + (8 * w + RPL * i) * D, 16, ix.b[i] * (D * 2) + col, 0, 0, 0);
    }
  };

  // transposing V reads: lane L supplies row rl = 4(L/32) + (L%16)/4 of a
  // 16-key step, chunk 4db + 2((L/16)%2) + (L%4)/2, half L%2
  const int rl = 4 * (lane >> 5) + ((lane & 15) >> 2);
  const int vch = 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
  const int vsw = v_swz(rl);
  const int vhalf = 4 * (lane & 1);   // elements

  // tile T of this wave's chunk from kt/vt0; the gathers of tile T+1 into
  // kn/vn are issued between the phases: K rows after the S MFMAs, V rows
  // before the PV MFMAs
  auto compute = [&](int tile, const uint16_t *kt, const uint16_t *vt0,
                     uint16_t (*kn)[kBN * D], uint16_t (*vn)[kBN * D], const Idx &ix) {
    if (!wave_active || tile >= nt_own) {
      gather_k(kn, ix);
      gather_v(vn, ix);
      return;
    }
    f32x16 sacc[2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int e = 0; e < 16; ++e) sacc[kb][e] = 0.0f;
    const int krow = l32;  // + 32 kb, which the swizzle does not see
#pragma unroll
    for (int s = 0; s < D / 16; ++s)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        const int slot = (2 * s + hf) ^ k_swz(krow);
        const bf16x8 a = as_bf16x8(*reinterpret_cast<const uint4 *>(
            &kt[(kb * 32 + krow) * D + 8 * slot]));
        sacc[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[s], sacc[kb], 0, 0, 0);
      }
    // each K operand is read from LDS two MFMAs ahead of its use
    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
#pragma unroll
    for (int i = 0; i < D / 8 - 2; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
    gather_k(kn, ix);
    const int kbase = tile * kBN;
    if (kbase + kBN > r) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int e = 0; e < 16; ++e)
          if (kbase + 32 * kb + 8 * (e >> 2) + 4 * hf + (e & 3) >= r) sacc[kb][e] = -INFINITY;
    }
    float mx0 = fmaxf(sacc[0][0], sacc[0][1]), mx1 = fmaxf(sacc[1][0], sacc[1][1]);
#pragma unroll
    for (int e = 2; e < 16; e += 2) {
      mx0 = fmaxf(fmaxf(mx0, sacc[0][e]), sacc[0][e + 1]);
      mx1 = fmaxf(fmaxf(mx1, sacc[1][e]), sacc[1][e + 1]);
    }
    float mx = fmaxf(mx0, mx1);
    {
      const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
      mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
    }
    const float mt = mx * scale_log2;
    const bool behind = mt > m_run + kRescale;
    if (__ballot(behind)) {
      const float m_new = behind ? fmaxf(m_run, mt) : m_run;
      const float alpha = behind ? __builtin_amdgcn_exp2f(m_run - m_new) : 1.0f;
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) oacc[db][e] *= alpha;
      m_run = m_new;
    }
    const float neg_m = -m_run;
    uint4 pk[2][2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      float p[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) p[e] = __builtin_amdgcn_exp2f(fmaf(sacc[kb][e], scale_log2, neg_m));
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2)
        pk[kb][s2] = make_uint4(pack_bf16(p[8 * s2 + 0], p[8 * s2 + 1]),
                                pack_bf16(p[8 * s2 + 2], p[8 * s2 + 3]),
                                pack_bf16(p[8 * s2 + 4], p[8 * s2 + 5]),
                                pack_bf16(p[8 * s2 + 6], p[8 * s2 + 7]));
    }
    {
      const bf16x2 one = __builtin_bit_cast(bf16x2, 0x3F803F80u);
      float ps[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
          const uint4 w4 = pk[kb][s2];
          ps[0] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w4.x), one, ps[0], false);
          ps[1] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w4.y), one, ps[1], false);
          ps[2] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w4.z), one, ps[2], false);
          ps[3] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w4.w), one, ps[3], false);
        }
      l_run += (ps[0] + ps[1]) + (ps[2] + ps[3]);
    }
    gather_v(vn, ix);
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
        for (int db = 0; db < D / 32; ++db) {
          const int vrow = kb * 32 + 16 * s2 + rl;  // hi: vrow + 8, same swizzle
          const int slot = (4 * db + vch) ^ vsw;
          const uint16_t *p0 = &vt0[vrow * D + 8 * slot + vhalf];
          const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4 *)(p0));
          const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4 *)(p0 + 8 * D));
          const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
          const bf16x8 a = as_bf16x8(make_uint4(l2.x, l2.y, h2.x, h2.y));
          oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, as_bf16x8(pk[kb][s2]), oacc[db], 0, 0, 0);
        }
  };

  // one step: indices of tile T+2 requested, tile T computed while tile T+1
  // is gathered into the free buffers; every wave's gathers land before the
  // barrier
  Idx cidx, nidx;
  auto step = [&](int tile, uint16_t (*kc)[kBN * D], uint16_t (*vc)[kBN * D],
                  uint16_t (*kn)[kBN * D], uint16_t (*vn)[kBN * D]) {
    load_idx(tile + 2, nidx);
    compute(tile, kc[g], vc[g], kn, vn, cidx);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wave's gathers are in LDS
    __syncthreads();
    cidx = nidx;
  };

  if (ntiles > 0) {
    Idx ix0;
    load_idx(0, ix0);
    load_idx(1, cidx);
    gather_k(K0, ix0);
    gather_v(V0, ix0);
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);
  __syncthreads();
  for (int tile = 0; tile < ntiles; tile += 2) {
    step(tile, K0, V0, K1, V1);
    if (tile + 1 < ntiles) step(tile + 1, K1, V1, K0, V0);
  }

  // lanes l and l^32 hold the two halves of one query's row sum
  const float l_tot = l_run + __shfl_xor(l_run, 32);
  if (!qvalid) return;
  const float inv = l_tot > 0.0f ? 1.0f / l_tot : 0.0f;
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int dim = db * 32 + 8 * i + 4 * hf;
      const size_t at = hoff + static_cast<size_t>(qi) * D + dim;
      const float o0 = oacc[db][4 * i + 0] * inv, o1 = oacc[db][4 * i + 1] * inv;
      const float o2 = oacc[db][4 * i + 2] * inv, o3 = oacc[db][4 * i + 3] * inv;
      if constexpr (BF16IO)
        *reinterpret_cast<uint2 *>(static_cast<uint16_t *>(ov) + at) =
            make_uint2(pack_bf16(o0, o1), pack_bf16(o2, o3));
      else
        *reinterpret_cast<float4 *>(static_cast<float *>(ov) + at) = make_float4(o0, o1, o2, o3);
    }
}

// d = 128: 192 registers, one block (two waves per SIMD) per CU.  d = 64 is
// bound by the softmax's vector instructions (per tile and wave about 950
// cycles against 512 of MFMA), so two blocks share a CU.
template <int D, bool BF16IO>
__global__ __launch_bounds__(kNW * 64)
__attribute__((amdgpu_waves_per_eu(D == 64 ? 4 : 2))) void attn_kernel_dma(
    int n, int c_q, int items_per_head, int total_items,
    const void *__restrict__ qv, const void *__restrict__ kv,
    const void *__restrict__ vv, void *ov, const int32_t *__restrict__ offsets,
    const int32_t *__restrict__ perm, const int32_t *__restrict__ sel_idx,
    const int4 *__restrict__ items, const int2 *__restrict__ order, float scale_log2) {
  __shared__ __attribute__((aligned(16))) DmaTile<D> K0;
  __shared__ __attribute__((aligned(16))) DmaTile<D> K1;
  __shared__ __attribute__((aligned(16))) DmaTile<D> V0;
  __shared__ __attribute__((aligned(16))) DmaTile<D> V1;
  int item, half = 0;
  if (order) {
    const int2 e = order[blockIdx.x];  // (slot, 0: all of it, 1 or 2: a half)
    item = e.x;
    half = e.y;
  } else {
    item = xcd_item(static_cast<int>(blockIdx.x), total_items);
  }
  if (item < 0 || item >= total_items) return;
  const int h = item / items_per_head;
  int4 ia = items[2 * item], ib = items[2 * item + 1];
  if (half) take_half(&ia, &ib, half);
  if (ia.z <= 0) return;
  // one block-uniform branch: a lone chunk gathers one set of tiles
  if (ib.z > 0)
    attn_dma_body<D, BF16IO, true>(n, c_q, h, ia, ib, qv, kv, vv, ov, offsets, perm,
                                   sel_idx, scale_log2, K0, K1, V0, V1);
  else
    attn_dma_body<D, BF16IO, false>(n, c_q, h, ia, ib, qv, kv, vv, ov, offsets, perm,
                                    sel_idx, scale_log2, K0, K1, V0, V1);
}

// K and V rounded to bf16, 8 elements per thread.
__global__ __launch_bounds__(256) void to_bf16_kernel(const float *__restrict__ k, const float *__restrict__ v,
                                                      uint16_t *kb, uint16_t *vb, size_t count) {
  const float *src = blockIdx.y ? v : k;
  uint16_t *dst = blockIdx.y ? vb : kb;
  for (size_t i = 8 * (static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x); i < count;
       i += 8 * 256 * static_cast<size_t>(gridDim.x))
    *reinterpret_cast<uint4 *>(dst + i) = load8<false>(src, i);
}

// A slot's estimated cost: its key tiles times the per-tile time of its wave
// count (about 1.45x for 5-8 waves against 1-4) and of a second chunk's gathers
// (about 1.15x).
__device__ __forceinline__ uint32_t slot_cost(const int4 &a, const int4 &b) {
  const int ta = key_tiles(a), tb = key_tiles(b);
  const int waves = (a.z + 31) / 32 + (b.z > 0 ? (b.z + 31) / 32 : 0);
  const uint32_t per = waves > 4 ? (b.z > 0 ? 196u : 171u) : (b.z > 0 ? 135u : 118u);
  return static_cast<uint32_t>(ta > tb ? ta : tb) * per;
}

// The block order of a call whose heads' K and V fit the memory-side cache
// together, or eight of them at a time (attention_ordered).  Block b runs on
// XCD b mod 8, whatever the XCDs' loads, so each XCD is given a queue of its
// own: the list of all heads' slots cut into eight runs of equal cost.  An XCD
// then works on one or two heads, whose rows its L2 serves to the 32 (d = 64:
// 64) blocks that sweep them at about the same pace, instead of on a share of
// every head in turn.
//
// Within a queue the slots run by cost, largest first, and where the queue is
// short its last round, partly empty, would be a large part of the launch: the
// first w rounds of slots run whole, and the rest as halves (take_half), which
// take kHalfCost of a slot's time (118 / 171 of slot_cost; from 0.60 on the
// times are the same, below every tail is halved: dense 4 x 8448 280 us for 203).
// w is that of the shortest estimated time;
// kRoundSlack: unequal slots fill a last round of whole ones badly.  Nothing is
// halved from kHalfRounds rounds on, where the last matters little.  (Slots cut
// along their keys would balance better, but a row's sums in parts round
// differently, so a result would depend on the other heads of the call and on
// the workspace.)
// Measured, list order -> here: 5 heads x 32760 tokens, d = 128: dense (2.5
// rounds of slots) 2641 -> 2454 us, 128 clusters 1627 -> 1397 us; 40 heads
// (nothing halved) 12.85 -> 11.99 ms; 3 heads x 118800, 300 clusters 10.69 ->
// 10.51 ms; 16 heads x 19721, d = 64, 96 clusters 1085 -> 971 us; 8 heads x 9504
// dense fp32 519 -> 457 us.
//
// One block per XCD, `slots` the most slots of a queue.  order[8 j + x], j <
// slots + max_halved: (slot, 0 or half), slot -1: nothing.
constexpr int kPlanThreads = 1024;
constexpr int kPlanSlots = 4096;      // slots of one queue (sorted in LDS)
constexpr int kHalfRounds = 8;
constexpr float kHalfCost = 0.69f, kRoundSlack = 0.15f;
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
__global__ __launch_bounds__(kPlanThreads) void attn_plan_kernel(
    int total_items, int slots, int resident, int max_halved, const int4 *__restrict__ items,
    int2 *order) {
  __shared__ unsigned long long key[kPlanSlots];
  __shared__ unsigned long long wsum[kPlanThreads / 64];
  __shared__ int used, wcnt[kPlanThreads / 64], in_queue[kXcds];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, x = blockIdx.x;
  if (t == 0) used = 0;
  if (t < kXcds) in_queue[t] = 0;
  auto cost_at = [&](int i) -> uint32_t {
    const int4 a = items[2 * static_cast<size_t>(i)], b = items[2 * static_cast<size_t>(i) + 1];
    return a.z > 0 ? max(slot_cost(a, b), 1u) : 0u;
  };
  // the cost before each slot of the list; this queue takes those whose cost
  // before lies in its eighth, or where that would overfill one of the queues
  // (very uneven slots) its eighth of their number
  const int per = (total_items + kPlanThreads - 1) / kPlanThreads;
  const int i0 = min(t * per, total_items), i1 = min(i0 + per, total_items);
  unsigned long long mine = 0;
#pragma unroll 4
  for (int i = i0; i < i1; ++i) mine += cost_at(i);
  const unsigned long long incl = wave_incl_scan(mine);
  if (lane == 63) wsum[w] = incl;
  __syncthreads();
  unsigned long long before = incl - mine, total = 0;
  for (int k = 0; k < kPlanThreads / 64; ++k) {
    if (k < w) before += wsum[k];
    total += wsum[k];
  }
  unsigned long long bound[kXcds];  // the ends of the eighths
#pragma unroll
  for (int k = 0; k < kXcds; ++k) bound[k] = total * (k + 1) / kXcds;
  int nth = 0;  // used slots of this thread
  unsigned long long at_cost = before;
  for (int i = i0; i < i1; ++i) {
    const uint32_t c = cost_at(i);
    if (c) {
      int k = 0;
#pragma unroll
      for (int j = 0; j < kXcds - 1; ++j) k += at_cost >= bound[j] ? 1 : 0;
      atomicAdd(&in_queue[k], 1);
      ++nth;
    }
    at_cost += c;
  }
  const int nincl = wave_incl_scan(nth);
  if (lane == 63) wcnt[w] = nincl;
  __syncthreads();
  int nbefore = nincl - nth, ntotal = 0;
  bool fits = true;
  for (int k = 0; k < kPlanThreads / 64; ++k) {
    if (k < w) nbefore += wcnt[k];
    ntotal += wcnt[k];
  }
  for (int k = 0; k < kXcds; ++k) fits = fits && in_queue[k] <= slots;
  const int eighth = (ntotal + kXcds - 1) / kXcds;
  const unsigned long long lo = x ? bound[x - 1] : 0, hi = bound[x];
  for (int i = i0; i < i1; ++i) {
    const uint32_t c = cost_at(i);
    if (!c) continue;
    if (fits ? before >= lo && before < hi : nbefore / eighth == x) {
      // descending cost, then ascending slot: unique keys, so the order does
      // not depend on where the slots were put
      const int at = atomicAdd(&used, 1);
      if (at < slots) key[at] = (static_cast<unsigned long long>(c) << 32) | static_cast<uint32_t>(~i);
    }
    before += c;
    ++nbefore;
  }
  __syncthreads();
  const int n = min(used, slots);
  int size = 64;
  while (size < n) size <<= 1;
  for (int i = n + t; i < size; i += kPlanThreads) key[i] = 0;
  __syncthreads();
  for (int k = 2; k <= size; k <<= 1)
    for (int j = k >> 1; j > 0; j >>= 1) {
      for (int p = t; p < size / 2; p += kPlanThreads) {
        const int i = 2 * (p & ~(j - 1)) + (p & (j - 1));
        const unsigned long long u = key[i], v = key[i + j];
        if (((i & k) == 0) == (u < v)) {
          key[i] = v;
          key[i + j] = u;
        }
      }
      // pairs at most 64 apart stay within the 128 keys of one wave (as does
      // the next step, of half the distance)
      if (j > 64 || (j == 1 && k >= 128)) __syncthreads();
      else wave_fence();
    }
  __syncthreads();
  // rounds of whole slots, or w of them and the rest as halves
  const int cap = resident / kXcds, full = n / cap;
  int whole = n;
  if (n < kHalfRounds * cap) {
    float least = static_cast<float>((n + cap - 1) / cap) + kRoundSlack;
    for (int wr = full; wr >= 0 && wr >= full - 2; --wr) {
      const int tail = n - wr * cap;
      const float e = wr + static_cast<float>((2 * tail + cap - 1) / cap) * kHalfCost;
      if (tail > 0 && tail <= max_halved && e < least) {
        least = e;
        whole = wr * cap;
      }
    }
  }
  for (int j = t; j < slots + max_halved; j += kPlanThreads) {
    int2 e = make_int2(-1, 0);
    const int p = j < whole ? j : whole + (j - whole) / 2;  // halves of a slot side by side
    if (p < n) e = make_int2(static_cast<int>(~static_cast<uint32_t>(key[p])), j < whole ? 0 : 1 + (j - whole) % 2);
    order[kXcds * static_cast<size_t>(j) + x] = e;
  }
}

// Work list of one head.  Every cluster's queries are cut into chunks of kBM
// rows; a block runs one work slot of two entries (A, B), each (cluster,
// first row, rows, selected keys), B empty (rows = 0) or a second chunk that
// shares the block: A's chunk takes waves 0 .. ceil(rows_A / 32) - 1 and
// B's the next ones.  Slots: the clusters' full chunks in cluster order,
// then their remainder chunks (fewer than kBM rows), then empty slots.  With
// `pair`, remainders are paired so that the two chunks need at most kNW
// waves together: bucketed by their wave count w and ordered by key count
// within a bucket, bucket w (largest first) takes partners from bucket
// min(8 - w, w) down to 1 in key-count order, so paired chunks run similar
// numbers of key tiles.  Remainders left without a partner (among them every
// remainder of 8 waves) run alone, and with d all of them where
// attention_runs_alone says so of as many heads like this one.  With `sort` (where attn_plan_kernel does
// not order them) and up to kSortMaxSlots slots per head, the head's slots are
// then reordered by estimated cost, largest first (ties
// keep their order, so a cluster's full chunks stay adjacent): the
// expensive blocks of each head start early and the cheap ones fill in
// behind them, which shortens the launch's tail.
constexpr int kPairMaxClusters = 2048;  // pairing up to this many clusters
constexpr int kRemKeyBits = 25;         // n <= 2^24
constexpr int kSortMaxSlots = 2048;     // cost-ordered work lists up to this many slots
__global__ __launch_bounds__(1024) void attn_items_kernel(
    int n, int c_q, int items_per_head, int pair, int d, int sort,
    const int32_t *__restrict__ offsets, const int32_t *__restrict__ sel_counts, int4 *items) {
  __shared__ int2 wtot[16];
  // a remainder's waves and key count, (waves << 25) + keys, 0: no remainder
  __shared__ uint32_t rem[kPairMaxClusters];
  __shared__ int ord[kPairMaxClusters];
  __shared__ int bucket_n[kNW + 1];
  __shared__ int4 seg[64];   // (A's first ordinal, B's first ordinal or -1, count, same bucket)
  __shared__ int seg_at[65], nseg;
  __shared__ int4 staged[2 * kSortMaxSlots];
  __shared__ unsigned long long cost[kSortMaxSlots];
  const int h = blockIdx.x, t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int32_t *off = offsets + static_cast<size_t>(h) * (c_q + 1);
  const int32_t *scnt = sel_counts + static_cast<size_t>(h) * c_q;
  int4 *out = items + static_cast<size_t>(h) * items_per_head * 2;
  const bool may_pair = pair && c_q <= kPairMaxClusters;
  const bool sorted = sort && items_per_head <= kSortMaxSlots;
  auto count_of = [&](int c) { return min(max(off[c + 1] - off[c], 0), n); };
  auto keys_of = [&](int c) { return min(max(scnt[c], 0), n); };
  auto put = [&](int slot, int4 a, int4 b) {
    if (slot < items_per_head) {
      if (sorted) {
        staged[2 * slot] = a;
        staged[2 * slot + 1] = b;
      } else {
        out[2 * slot] = a;
        out[2 * slot + 1] = b;
      }
    }
  };
  // the staged slots, largest estimated cost first.  The first `used` slots hold
  // chunks; the empty ones after them stay in place.
  auto emit_sorted = [&](int used) {
    if (!sorted) return;
    __syncthreads();
    for (int i = t; i < used; i += 1024) {
      const uint32_t k = slot_cost(staged[2 * i], staged[2 * i + 1]);
      // descending cost, then ascending slot: one unsigned comparison
      cost[i] = (static_cast<unsigned long long>(k) << 32) | static_cast<uint32_t>(~i);
    }
    __syncthreads();
    for (int i = t; i < items_per_head; i += 1024) {
      int rank = i;
      if (i < used) {
        const unsigned long long ci = cost[i];
        rank = 0;
#pragma unroll 8
        for (int j = 0; j < used; ++j) rank += cost[j] > ci ? 1 : 0;
      }
      out[2 * rank] = staged[2 * i];
      out[2 * rank + 1] = staged[2 * i + 1];
    }
  };
  const int4 none = make_int4(0, 0, 0, 0);
  if (t <= kNW) bucket_n[t] = 0;
  __syncthreads();
  // full chunks, in cluster order: of 1,024 clusters, the full chunks (x) and the
  // remainders (y) before each and of all
  auto prefix = [&](int k, bool has, int2 *tot) {
    const unsigned long long some = __ballot(has);
    const int incl = wave_incl_scan(k);
    if (lane == 63) wtot[w] = make_int2(incl, __popcll(some));
    __syncthreads();
    int2 base = make_int2(incl - k, __popcll(some & ((1ull << lane) - 1ull)));
    *tot = make_int2(0, 0);
    for (int i = 0; i < 16; ++i) {
      const int2 v = wtot[i];
      if (i < w) {
        base.x += v.x;
        base.y += v.y;
      }
      tot->x += v.x;
      tot->y += v.y;
    }
    __syncthreads();
    return base;
  };
  int run = 0;
  int own_at = 0, remainders = 0;  // of the last 1,024 clusters: this thread's remainder, and how many
  int4 own = none;
  for (int c0 = 0; c0 < c_q; c0 += 1024) {
    const int c = c0 + t;
    int cnt = 0, rsel = 0;
    if (c < c_q) {
      cnt = count_of(c);
      rsel = keys_of(c);
    }
    const int k = cnt / kBM, rows = cnt - k * kBM;
    int2 tot;
    const int2 before = prefix(k, rows > 0, &tot);
    const int first = run + before.x;
    for (int q = 0; q < k; ++q) put(first + q, make_int4(c, q * kBM, kBM, rsel), none);
    run += tot.x;
    own = make_int4(c, cnt - rows, rows, rsel);
    own_at = before.y;
    remainders = tot.y;
    // remainders, bucketed by wave count for pairing
    if (may_pair && c < c_q) {
      const int waves = (rows + 31) / 32;
      rem[c] = rows > 0 ? (static_cast<uint32_t>(waves) << kRemKeyBits) + rsel : 0u;
      if (rows > 0) atomicAdd(&bucket_n[waves], 1);
    }
  }
  __syncthreads();
  int rem_tot = 0, rem_waves = 0;
#pragma unroll
  for (int b = 1; b <= kNW; ++b) {
    const int some = bucket_n[b];
    rem_tot += some;
    rem_waves += b * some;
  }
  const bool alone = d && attention_runs_alone(d, static_cast<long long>(run + rem_tot) * gridDim.x,
                                               static_cast<long long>(kNW * run + rem_waves) * gridDim.x);
  if (!may_pair || alone) {
    // remainders alone, in cluster order, after the full chunks
    int at = 0;
    if (c_q <= 1024) {
      if (own.z > 0) put(run + own_at, own, none);
      at = remainders;
    }
    for (int c0 = c_q <= 1024 ? c_q : 0; c0 < c_q; c0 += 1024) {
      const int c = c0 + t;
      int cnt = 0, rsel = 0;
      if (c < c_q) {
        cnt = count_of(c);
        rsel = keys_of(c);
      }
      const int rows = cnt % kBM;
      int2 tot;
      const int2 before = prefix(0, rows > 0, &tot);
      if (rows > 0) put(run + at + before.y, make_int4(c, cnt - rows, rows, rsel), none);
      at += tot.y;
    }
    for (int slot = run + at + t; slot < items_per_head; slot += 1024) put(slot, none, none);
    emit_sorted(min(run + at, items_per_head));
    return;
  }
  // ordinal of each remainder within (bucket ascending, keys ascending,
  // cluster ascending)
  // (as many lanes share a cluster as the block has for each; with one thread per
  // cluster and its waves and keys read and compared apart, this was most of the
  // kernel: one head of 64 clusters 11.1 -> 4.6 us, 256 31.9 -> 10.2, 1000 138 -> 106)
  int share = 1;
  while (share < 64 && share < c_q && 2 * share * c_q <= 1024) share *= 2;
  for (int c0 = 0; c0 < c_q; c0 += 1024 / share) {
    const int c = c0 + t / share;
    const uint32_t mine = c < c_q ? rem[c] : 0u;
    int pos = 0;
    if (mine) {
#pragma unroll 4
      for (int o = t % share; o < c_q; o += share) {
        const uint32_t other = rem[o];
        pos += other != 0u && (other < mine || (other == mine && o < c)) ? 1 : 0;
      }
    }
    for (int k = share / 2; k > 0; k /= 2) pos += __shfl_xor(pos, k);
    if (mine && t % share == 0) ord[pos] = c;
  }
  // the pairing plan (at most kNW * kNW segments), one thread
  if (t == 0) {
    int nxt[kNW + 1], left[kNW + 1];
    nxt[0] = left[0] = 0;
    for (int b = 1; b <= kNW; ++b) {
      nxt[b] = nxt[b - 1] + left[b - 1];  // where the bucket starts
      left[b] = bucket_n[b];
    }
    int ns = 0;
    for (int wa = kNW; wa >= 1; --wa) {
      for (int wb = min(kNW - wa, wa); wb >= 1 && left[wa] > 0; --wb) {
        const int m = wb == wa ? left[wa] / 2 : min(left[wa], left[wb]);
        if (m <= 0) continue;
        seg[ns++] = make_int4(nxt[wa], nxt[wb], m, wb == wa ? 1 : 0);
        if (wb == wa) {
          nxt[wa] += 2 * m;
          left[wa] -= 2 * m;
        } else {
          nxt[wa] += m;
          left[wa] -= m;
          nxt[wb] += m;
          left[wb] -= m;
        }
      }
      if (left[wa] > 0) {  // no partner left: alone
        seg[ns++] = make_int4(nxt[wa], -1, left[wa], 0);
        nxt[wa] += left[wa];
        left[wa] = 0;
      }
    }
    int a = 0;
    for (int i = 0; i < ns; ++i) {
      seg_at[i] = a;
      a += seg[i].z;
    }
    seg_at[ns] = a;
    nseg = ns;
  }
  __syncthreads();
  const int total = seg_at[nseg];
  auto entry = [&](int c) {
    const int cnt = count_of(c), rows = cnt % kBM;
    return make_int4(c, cnt - rows, rows, static_cast<int>(rem[c] & ((1u << kRemKeyBits) - 1u)));
  };
  for (int i = t; i < total; i += 1024) {
    int s = 0;
    while (seg_at[s + 1] <= i) ++s;
    const int4 g = seg[s];
    const int j = i - seg_at[s];
    if (g.y < 0) {
      put(run + i, entry(ord[g.x + j]), none);
    } else if (g.w) {
      put(run + i, entry(ord[g.x + 2 * j]), entry(ord[g.x + 2 * j + 1]));
    } else {
      put(run + i, entry(ord[g.x + j]), entry(ord[g.y + j]));
    }
  }
  for (int slot = run + total + t; slot < items_per_head; slot += 1024) put(slot, none, none);
  emit_sorted(min(run + total, items_per_head));
}

// Blocks that the chip holds at once (256 CUs; two blocks per CU at d = 64).
int resident_blocks(int d) { return d == 64 ? 512 : 256; }

// Slots that one XCD's queue holds: half as many again as its share.
int queue_slots(int total_items) { return (total_items + total_items / 2 + kXcds - 1) / kXcds; }

// The most slots of a queue that run as halves: three rounds where even the
// fewest slots (all chunks full) fill fewer than kHalfRounds rounds; else none.
int halved_slots(int heads, int n, int d) {
  const int cap = resident_blocks(d);
  const long long least = static_cast<long long>(heads) * ((n + kBM - 1) / kBM);
  return least < static_cast<long long>(kHalfRounds) * cap ? 3 * cap / kXcds : 0;
}

template <int D, bool BF16IO>
hipError_t launch_dma(int heads, int n, const void *q, const void *k, const void *v, void *o,
                      int c_q, const int32_t *offsets, const int32_t *perm, const int32_t *sel_idx,
                      int iph, float scale_log2, const AttnScratch &w, hipStream_t s) {
  const int total = iph * heads;
  if (!w.order) {
    hipLaunchKernelGGL((attn_kernel_dma<D, BF16IO>), dim3(total), dim3(kNW * 64), 0, s, n, c_q,
                       iph, total, q, k, v, o, offsets, perm, sel_idx, w.items,
                       static_cast<const int2 *>(nullptr), scale_log2);
    return hipGetLastError();
  }
  const int slots = queue_slots(total), halved = halved_slots(heads, n, D);
  const int queue = slots + halved;
  hipLaunchKernelGGL(attn_plan_kernel, dim3(kXcds), dim3(kPlanThreads), 0, s, total, slots,
                     resident_blocks(D), halved, w.items, w.order);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((attn_kernel_dma<D, BF16IO>), dim3(kXcds * queue), dim3(kNW * 64), 0, s, n, c_q,
                     iph, total, q, k, v, o, offsets, perm, sel_idx, w.items, w.order, scale_log2);
  return hipGetLastError();
}

template <int D>
hipError_t launch_attn(int heads, int n, bool bf16, const void *q,
                       const void *k, const void *v, void *o, int c_q,
                       const int32_t *offsets, const int32_t *perm,
                       const int32_t *sel_idx, int iph, float scale_log2,
                       const AttnScratch &w, hipStream_t s) {
  if (bf16)
    return launch_dma<D, true>(heads, n, q, k, v, o, c_q, offsets, perm, sel_idx, iph, scale_log2,
                               w, s);
  if (w.kv16) {
    const size_t count = static_cast<size_t>(heads) * n * D;
    uint16_t *v16 = w.kv16 + count;
    const size_t blocks = (count / 8 + 255) / 256;
    hipLaunchKernelGGL(to_bf16_kernel, dim3(blocks < 2048 ? static_cast<unsigned>(blocks) : 2048u, 2),
                       dim3(256), 0, s, static_cast<const float *>(k), static_cast<const float *>(v),
                       w.kv16, v16, count);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_dma<D, false>(heads, n, q, w.kv16, v16, o, c_q, offsets, perm, sel_idx, iph,
                                scale_log2, w, s);
  }
  const int total = iph * heads;
  hipLaunchKernelGGL(attn_kernel<D>, dim3(total), dim3(kNW * 64), 0, s, n, c_q, iph,
                     total, q, k, v, o, offsets, perm, sel_idx, w.items, scale_log2);
  return hipGetLastError();
}

}  // namespace

// Work list of the no-allocation entry point: a fixed device array, one copy
// per GPU, held until the process ends.  Host code never passes `scratch`
// itself to a kernel (on the host it names a stand-in, not device memory);
// it looks up the array's device address once per device and uses that.
static __device__ __align__(256) int4 scratch[kAttnScratchItems];

namespace {
constexpr int kMaxDevices = 64;
std::mutex scratch_mu;
int4 *scratch_ptr[kMaxDevices];
}  // namespace

hipError_t attention_scratch(int4 **items) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(scratch_mu);
  if (!scratch_ptr[dev]) {
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    scratch_ptr[dev] = static_cast<int4 *>(p);
  }
  *items = scratch_ptr[dev];
  return hipSuccess;
}

// Work slots of one head: sum_c ceil(n_c / kBM) <= ceil(n / kBM) + c_q; each
// slot is two int4 entries.
int attn_items_per_head(int n, int c_q) { return (n + kBM - 1) / kBM + c_q; }

hipError_t attention_items(int heads, int n, int c_q, bool pair, const int32_t *offsets,
                           const int32_t *sel_counts, int4 *items, hipStream_t s) {
  hipLaunchKernelGGL(attn_items_kernel, dim3(heads), dim3(1024), 0, s, n, c_q,
                     attn_items_per_head(n, c_q), pair ? 1 : 0, 0, 1, offsets, sel_counts, items);
  return hipGetLastError();
}

// The copies cost a pass over all of K and V and a launch, and save by the gathered
// key.  Dense calls make them from 1,024 tokens on (one head of 1100, d = 128: 42 us
// with the copies, 49 us without; d = 64: 33 and 34 us).  Sparse ones keep from a
// tenth to half of the keys and gather once per chunk of queries, at most n / kBM +
// c_q of them; they make them
// - from where half of the keys pay at the latest (a tenth, a quarter, half of the
//   keys; d = 128, 2 x 3000: 29, 40, 58 us with, 26, 40, 62 without; d = 64, 8 x
//   6400: 45, 71, 115 with, 40, 68, 117 without; 2 x 4000: 25, 35, 52 with, 21, 32,
//   51 without);
// - with so many chunks that few keys pay too (d = 128, an eighth of the keys, 15 x
//   2688 tokens in 41 clusters 52 us with, 55 without, half of them, 6 x 2496 in 39
//   59 and 70 us; on the other side 10 x 3420 in 11, a seventh, 44 and 39 us; d = 64,
//   a fifth, 27 x 3861 in 89 82 and 105 us, half, 5 x 5022 in 225 95 and 140 us; on
//   the other side 9 x 5016 in 49, a seventh, 43 and 40 us).
bool attention_copies_kv(int n, int d, int c_q, bool bf16) {
  if (bf16 || (d != 64 && d != 128) || n < 1024 || static_cast<uint64_t>(n) * d * 2 >= (1ull << 32)) return false;
  return c_q == 1 || n >= (d == 128 ? 3072 : 6144) || n / kBM + c_q >= (d == 128 ? 48 : 96);
}

// Dense calls (one cluster) from 4,096 tokens on: one head of 4,224 tokens, d =
// 128, 103 us in list order, 80 us so.  Not those whose slots fill more than half
// the CUs but not a round, where every order is as good (4 heads x 8,448 tokens,
// 132 slots: 196 us in list order, 203 us with a plan; 8 x 5,280, d = 64, 168
// slots: 104 and 112 us).  Sparse calls have more slots of unequal cost; up to
// 16,384 tokens the order gains less than its launch costs (8 heads x 9,504
// tokens, 40 clusters: 277 us in list order, 280 us so; one head of 17,316: 254
// and 194 us).
bool attention_ordered(int heads, int n, int d, int c_q) {
  if ((d != 64 && d != 128) || n < (c_q > 1 ? 16384 : 4096)) return false;
  const int at_once = heads < kXcds ? heads : kXcds;
  if (static_cast<uint64_t>(at_once) * n * d * 4 > kMemorySideCache) return false;
  const long long total = static_cast<long long>(heads) * attn_items_per_head(n, c_q);
  if (total > (1 << 20) || queue_slots(static_cast<int>(total)) > kPlanSlots) return false;
  const long long full = static_cast<long long>(heads) * ((n + kBM - 1) / kBM);
  return c_q > 1 || 2 * full <= resident_blocks(128) || full > resident_blocks(d);
}

size_t attention_order_entries(int heads, int n, int d, int c_q) {
  return static_cast<size_t>(kXcds) *
         (queue_slots(heads * attn_items_per_head(n, c_q)) + halved_slots(heads, n, d));
}

hipError_t attention_run(int heads, int n, int d, bool bf16, const void *q,
                         const void *k, const void *v, void *o, int c_q,
                         const int32_t *offsets, const int32_t *perm,
                         const int32_t *sel_counts, const int32_t *sel_idx,
                         float scale, const AttnScratch &w, hipStream_t s) {
  const int iph = attn_items_per_head(n, c_q);
  // remainder chunks share blocks only in the LDS-DMA kernel (with a block order
  // always: fewer slots leave more of them room to run as halves)
  const int pair = c_q > 1 && (bf16 || w.kv16) ? 1 : 0;
  hipLaunchKernelGGL(attn_items_kernel, dim3(heads), dim3(1024), 0, s, n, c_q,
                     iph, pair, w.order ? 0 : d, w.order ? 0 : 1, offsets, sel_counts, w.items);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const float sl2 = scale * 1.4426950408889634f;
  if (d == 128)
    return launch_attn<128>(heads, n, bf16, q, k, v, o, c_q, offsets, perm,
                            sel_idx, iph, sl2, w, s);
  return launch_attn<64>(heads, n, bf16, q, k, v, o, c_q, offsets, perm,
                         sel_idx, iph, sl2, w, s);
}

}  // namespace scope
