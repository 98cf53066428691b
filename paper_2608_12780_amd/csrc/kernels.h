// Host-side launchers of the SCOPE kernels (internal to the library).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/scope.h"

namespace scope {

// One batch of k-means problems, one problem per head: the rows of
// X[h] (row stride ld elements, channels col0 .. col0+dx) clustered into C
// centroids U[h] ([C][dx] fp32).
struct KmProblem {
  const void *x;          // element type given by bf16 flag
  bool bf16;
  size_t x_head_stride;   // elements between heads
  int ld, col0, dx, n, C;
  float *u;               // centroids of head 0 (this subspace)
  size_t u_head_stride;   // floats between heads
  int32_t *assign;        // [heads][n] (a_head_stride apart)
  size_t a_head_stride;
  int32_t *counts;        // [heads][C]
  int32_t *offsets;       // [heads][C+1]
  int32_t *perm;          // [heads][n]
  int32_t *chunk_hist;    // [heads][nchunks][C]
  int32_t *chunk_rel;     // [heads][nchunks][C]
  int heads;
  // matrix-core assignment: two-term bf16 copy of the centroids,
  // their squared norms and the error-bound constants, refreshed per pass
  bool mfma;
  int cpad, dxp;          // centroids padded to 32, channels padded to 16
  uint16_t *ubf;          // [heads][cpad][2 * dxp]: bf16 hi then lo terms
  float *nu;              // [heads][cpad]
  float *bnd;             // [heads][cpad]: bound on the two terms' residual
  // codebooks beyond the LDS: per chunk and point the three largest packed
  // values ([parts][heads][n][4], the last unused) and the point's norm bound ([heads][n])
  float *part, *pnx;
};

// Whether the matrix-core assignment applies: fp32 rows, or bf16 rows at even
// offsets, and at most 1024 centroids (codebooks beyond the LDS are streamed in chunks).
bool km_mfma_ok(bool bf16, int ld, int col0, int dx, int C);
int km_parts(int C, int dx);
// floats of KmProblem::part and ::pnx together (0 when the codebook fits)
size_t km_split_floats(int C, int dx, int heads, int n);
int km_cpad(int C);
int km_dxp(int dx);

constexpr int kAssignBlock = 256;  // points per assign block == grouping chunk

inline int km_nchunks(int n) { return (n + kAssignBlock - 1) / kAssignBlock; }

// Launch arguments that later kernels of the call read from device memory,
// as 32-bit words stored to dst (words == 0: none).
constexpr int kArgWords = 160;
struct DeviceArgs {
  uint32_t *dst;
  int words;
  uint32_t w[kArgWords];
};

// The starting centroids of the call's subspaces p[0..nsub) (one set of rows,
// centroids back to back) in one launch: the rows init[h * init_hs + m *
// init_ms + r] of X (init null: the default rows), or with `warm` those in
// p[].u; matrix-core codebooks are prepared for the first assignment.  The
// same launch clears zero[0..zero_count) and stores args.
hipError_t km_init(const KmProblem *p, int nsub, bool warm, const int32_t *init, int init_hs,
                   int init_ms, int32_t *status, int32_t *zero, size_t zero_count,
                   const DeviceArgs &args, hipStream_t s);
hipError_t km_assign(const KmProblem &p, bool with_hist, hipStream_t s);
// The assignments of several subspaces of the same rows.
hipError_t km_assign_subspaces(const KmProblem *p, int nsub, hipStream_t s);
// Blocks for each of nsub subspaces of the given costs, out of `cus`: in
// proportion, at least one and at most `most` each.
void km_block_shares(const double *cost, int nsub, int cus, long long most, int *blocks);
hipError_t km_group(const KmProblem &p, hipStream_t s);
// The three key subspaces' assignments in one pass over the rows (matrix
// cores; codebooks side by side in LDS): applies when km_assign3_ok.
bool km_assign3_ok(const KmProblem (&p)[3]);
// scratch: km_assign3_scratch_bytes() of device memory that hold the launch's
// arguments; km_assign3_args fills in what km_init stores there
size_t km_assign3_scratch_bytes();
void km_assign3_args(const KmProblem (&p)[3], void *scratch, DeviceArgs *args);
hipError_t km_assign3(const KmProblem (&p)[3], void *scratch, hipStream_t s);

// Centroid update by one streaming pass over the rows.  Up to kMaxSub
// subspaces of the same rows (channels col0[m] .. col0[m]+dx[m], C[m]
// clusters, centroids [C[m]][dx[m]] at float offset ucol[m] of a head) are
// updated together; their channels are cut into windows whose int64 sums
// fit one block's LDS.
constexpr int kAccLds = 19200;           // int64 sums per block (150 KB of LDS)
constexpr int kAccCnt = 1024;            // int32 cluster counts per block
constexpr int kAccMaxPieces = 4;
constexpr int kAccMaxWindows = 16;
constexpr int kMaxSub = 8;               // subspaces of a key partition

// One subspace's codebook as the kernels that write centroids see it.
struct Codebook {
  int C, cpad, rows;    // centroids, padded, and the rows that are written
  int dx, dxp, col0;
  int ucol, ccol;       // float offset and first cluster within a head
  uint16_t *ubf;        // matrix-core codebook, norms and bounds, or null
  float *nu, *bnd;
};
struct Codebooks {
  float *u;             // centroids of head 0
  size_t u_hs;
  Codebook c[kMaxSub];
};

constexpr int kAccTargetBlocks = 256;    // blocks per launch, about one per CU
struct AccPiece {
  int m, sub0, width;   // channels sub0 .. sub0+width of subspace m
  int lds;              // first int64 LDS sum of the piece ([C][width])
  int cnt;              // first LDS count of subspace m, or -1 if not counted here
};
struct AccWindow {
  int npieces, lanes, elems, cnt_elems;
  AccPiece piece[kAccMaxPieces];
};
struct AccPlan {
  int nsub;
  int C[kMaxSub], dx[kMaxSub], col0[kMaxSub], ucol[kMaxSub], ccol[kMaxSub];
  int S, SC;            // centroid elements and clusters of one head
  int nwin, blocks;     // windows; blocks per (head, window)
  AccWindow win[kAccMaxWindows];
};
bool km_accum_plan(int nsub, const int *col0, const int *dx, const int *C,
                   int heads, int n, AccPlan *plan);
size_t km_accum_slab_bytes(const AccPlan &p, int heads);
size_t km_accum_cslab_bytes(const AccPlan &p, int heads);
// assign of subspace m, head h at assign[h * a_hs + m * a_ss]; with a
// status word, the visited inputs are also checked for |x| >= 2^22 and
// non-finite values.
hipError_t km_accum(const AccPlan &plan, const void *x, bool bf16, size_t x_hs,
                    int ld, int n, int heads, const int32_t *assign,
                    size_t a_hs, size_t a_ss, long long *slab, int32_t *cslab,
                    int32_t *status, hipStream_t s);
// The new centroids of p[0..nsub) from the blocks' sums; `prepare`: their
// matrix-core codebooks too (not needed after a call's last update).
hipError_t km_finish(const AccPlan &plan, const KmProblem *p, int nsub, bool prepare,
                     const long long *slab, const int32_t *cslab, hipStream_t s);
// Whether km_finish has four waves share a row's slabs instead of one take them all.
bool km_finish_shared(const AccPlan &plan, int heads);
// Largest |x| (exclusive) for which n rows' fixed-point sums are exact.
float km_range_limit(int n);
// Small problems: assignment and update of an iteration in one launch, or all
// iterations (and the keys' last assignment) in one block per head and subspace.
// km_lloyd_form: which of them, and the blocks per head and subspace, at most
// the plan's, whose block count is to be set to it.  km_finish follows each
// launch of a single iteration.
enum class Lloyd { kSeparate, kIteration, kAll };
struct LloydForm {
  Lloyd form;
  int blocks;
};
LloydForm km_lloyd_form(const KmProblem *p, int nsub, const AccPlan &plan);
hipError_t km_lloyd(const KmProblem *p, int nsub, LloydForm form, int iters, bool final_assign,
                    int32_t *chunk_hist, const AccPlan &plan, long long *slab, int32_t *cslab,
                    int32_t *status, hipStream_t s);
hipError_t km_pack_codes(const int32_t *a3, size_t a_head_stride,
                         size_t a_sub_stride, int n, int heads,
                         uint32_t *codes, hipStream_t s);
// Per-subspace codes of a general partition: z[h][m][j] = assign as uint16.
hipError_t km_codes16(const int32_t *assign, size_t count, uint16_t *codes,
                      hipStream_t s);
// dst[r][t] = src[r][chan[t]] for rows r < rows (each of d elements of
// elem_bytes = 2 or 4 bytes): the channels of a partition's sets, in order.
struct ChannelMap {
  int chan[128];
};
hipError_t gather_channels(const void *src, void *dst, size_t rows, int d,
                           int elem_bytes, const ChannelMap &map, hipStream_t s);

// Codebooks of the key subspaces: M sets, sizes c[0..M).  The logits read
// codes packed as zT | zH << 10 | zW << 20 (M = 3, codes32) or one uint16
// plane per subspace, [heads][M][n] (codes16).
struct Subspaces {
  int M;
  int c[kMaxSub];
};

// Tables over the M channel ranges (off[m], len[m]) of the query centroids
// (row stride d), one per subspace.
hipError_t score_tables(int heads, int d, const int *off, const int *len,
                        int c_q, const Subspaces &sub, const float *qc,
                        const float *kc, float *tables, hipStream_t s);
hipError_t score_logits(int heads, int n, int d, int c_q, const Subspaces &sub,
                        const float *tables, const uint32_t *codes32,
                        const uint16_t *codes16, float *scores, hipStream_t s);

constexpr int kSelMaxTable = 3072;    // LUT floats of one cluster row in LDS
hipError_t select_run(int heads, int n, int c_q, const Subspaces &sub, int d,
                      const float *scores, const float *tables,
                      const uint32_t *codes32, const uint16_t *codes16,
                      const int32_t *counts, float rho,
                      int k_fix, int32_t *base, int32_t *topp, int32_t *k_head,
                      int32_t *sel_counts, int32_t *sel_idx, float *row_max,
                      uint32_t *row_state, uint32_t *coarse_hist, uint32_t *dedup,
                      uint32_t *pack, int policy, hipStream_t s);
// whether select_run packs code planes given room for [heads][n] words in `pack`
bool planes_as_packed(int n, int M);
// 32-bit words of the distinct-code scratch of select_run
size_t select_dedup_words(int heads, int n);
constexpr int kSelCoarseBins = 2048;  // coarse histogram bins per cluster row
// Measured-peak microbenchmarks (diagnostics).
hipError_t peak_copy(const void *src, void *dst, size_t bytes, hipStream_t s);
hipError_t peak_mfma(float *out, int blocks, int iters, hipStream_t s);

hipError_t debug_fixexp(const float *y, uint64_t *out, int64_t count,
                        hipStream_t s);

int attn_items_per_head(int n, int c_q);
// 16-byte work-list entries of the no-allocation attention entry point
// (1 MiB; two per work slot).
constexpr size_t kAttnScratchItems = SCOPE_NOALLOC_MAX_WORK_ITEMS;
// Device address of that work list on the current device (looked up once
// per device).
hipError_t attention_scratch(int4 **items);
// The work list alone (as attention_run builds it), for diagnostics.
hipError_t attention_items(int heads, int n, int c_q, bool pair, const int32_t *offsets,
                           const int32_t *sel_counts, int4 *items, hipStream_t s);
// Scratch of one attention call: the work list, and where the workspace holds
// them bf16 copies of fp32 K and V (2 * heads * n * d elements; null: rows are
// rounded one by one) and the block order (attention_order_entries; null: list
// order, and for fp32 without the copies).  The result is the same with and
// without them.
struct AttnScratch {
  int4 *items;
  int2 *order;
  uint16_t *kv16;
};
hipError_t attention_run(int heads, int n, int d, bool bf16, const void *q,
                         const void *k, const void *v, void *o, int c_q,
                         const int32_t *offsets, const int32_t *perm,
                         const int32_t *sel_counts, const int32_t *sel_idx,
                         float scale, const AttnScratch &w, hipStream_t s);
// Whether the remainder chunks of a call without a block order run alone, given
// its work slots and their waves if they do.  Pairs spare gathers and blocks, but
// a pair's block takes longer than two that share a CU (d = 64) or have one each.
// Alone is better while the slots are hardly more than the chip holds and the
// waves few: two per SIMD at d = 64, one for every two SIMDs at d = 128.  Whole
// calls, alone and paired: d = 64, 8 heads x 800 tokens x 13 clusters 14.5 and 19.6
// us, 16 x 1372 x 22 24.3 and 32.7 us, 3 x 12512 x 211 (633 slots, 1460 waves) 176
// and 224 us, on the other side 9 x 11628 x 42 (599, 3470) 271 and 237 us; d = 128,
// fp32, 1 x 6417 x 106 (106, 420) 89 and 110 us, on the other side bf16 9 x 2835 x
// 22 (201, 900) 75 and 61 us.
inline __host__ __device__ bool attention_runs_alone(int d, long long slots, long long waves) {
  return d == 64 ? slots <= 768 && waves <= 2048 : slots <= 256 && waves <= 512;
}
// Whether the workspace holds bf16 copies of K and V.  One head's copy is
// addressed with 32-bit byte offsets.
bool attention_copies_kv(int n, int d, int c_q, bool bf16);
// Whether the call has a block order of its own, and that order's entries.
bool attention_ordered(int heads, int n, int d, int c_q);
size_t attention_order_entries(int heads, int n, int d, int c_q);

}  // namespace scope
