// Internal declarations shared by the translation units of libilargi (not installed).
#ifndef ILARGI_INTERNAL_H_
#define ILARGI_INTERNAL_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "ilargi.h"

namespace ilargi {

constexpr int kMaxPairLists = 4;     // pair lists of crossprod a plan holds (source pairs joined row by row)
constexpr int kMaxSources = 16;      // sources per plan (kernel argument arrays are this long)
constexpr int kWave = 64;            // gfx950 wavefront
constexpr int kBlock = 256;          // threads per workgroup in the streaming kernels
constexpr int kNarrowCT = 4;         // operand columns one narrow (VALU) pass handles
constexpr int kColredBlocks = 1024;  // most row chunks (= partial results) of the D^T Z reduction
constexpr int kColredTarget = 512;   // row chunks aimed at: two workgroups per compute unit, eight loads in flight per lane
constexpr int kSparseBlockRows = 1024;   // rows a row block of the sparse row-wise product holds at most
constexpr int kSparseChunk = 4096;   // entries of a column one workgroup sums
constexpr int kSegSlices = 8;        // slices of target rows of the sliced segment sum (one per XCD and its L2)
constexpr int kSlLong = 256;         // ... runs of a (slice, source row) longer than this are cut into chunks
constexpr int kSlChunk = 1024;       // ... of this many entries, each summed by a whole workgroup
constexpr int kLongSeg = 2048;       // inverse-index segments longer than this keep a plan off the join-order paths, and
                                     // the most entries of a segment that the segment sums leave uncut
constexpr int kSegCut = 256;         // least entries of a chunk of a longer segment (a plan picks its own length between the two)
constexpr int kSortChunk = 2048;     // keys per workgroup in one radix pass
constexpr int kMaxLdsFloats = 4096;  // 16 KiB of LDS for the staged operand rows (also the column limit of a source)
constexpr int64_t kGramPartialFloats = 16ll << 20;

// Row gathers of per-source products:  out[i,:] += P_s[row_s(i), :]  (assembly step of Sec. 2.2).
struct GatherArgs {
  int n;
  const int32_t* idx[kMaxSources];  // NULL: identity on the first rows[s] target rows
  const float* P[kMaxSources];
  int64_t rows[kMaxSources];
  int ldp;
};

struct LmmArgs {
  const float* D;         // fused identity-prefix source (may be NULL)
  int64_t d_rows;         // target rows [0, d_rows) take row i of D
  int ck;                 // columns of D
  const int32_t* colmap;  // device int32[ck]
  const float* X;         // c_T x ldx
  int ldx, col0, ncols;   // operand columns [col0, col0 + ncols)
  float* out;             // r_out x ldo
  int ldo;
  int64_t r_out;
  int logL;               // lanes per row = 1 << logL
  GatherArgs g;
  // gradient-descent modes
  const float* y;         // labels, r_out
  float* loss_partial;    // narrow kernel: [gridDim.x][kNarrowCT]; matrix-core kernel: [gridDim.x][ld_loss]
  int ld_loss;
  int nt_in;              // read the table past the caches (see stream_past_caches)
  int nt_out;             // store the output with non-temporal stores (large results nobody re-reads soon)
  int x_block;            // the table's columns are target columns [x_block - 1, x_block - 1 + ck); 0: no block, or not known
  int lds_products;       // the gathers are worth products in LDS (lmm_lane_lds_pays)
  float* scratch;         // optional device scratch of scratch_floats floats (the caller's, free for the launch)
  int64_t scratch_floats;
  float* grad_partial;    // optional partials of D^T e: narrow kernel [gridDim.x][ck][kNarrowCT],
                          // matrix-core kernel [gridDim.x][ck][ld_grad]
  int ld_grad;
};

// Tile shape of the matrix-core left multiply for a table with ck columns.
struct MfmaShape {
  int kp;            // ck rounded up to a multiple of 16
  int kc;            // table columns staged per step
  int lda;           // LDS row stride of the staged rows (floats)
  int rb;            // table rows per workgroup step
  size_t lds_bytes;
};

// A source table in compressed sparse rows with its column-sorted view (kernels_sparse.hip).
struct SparseArgs {
  const int32_t* rowptr;   // rows + 1
  const int32_t* col;      // nnz, strictly ascending within a row
  const float* val;        // nnz
  int64_t rows, nnz;
  int cols;
  const int32_t* colmap;   // device int32[cols]
  const int32_t* row_block;  // n_row_blocks + 1: runs of whole rows with at most sparse_row_block_cap(cols) entries
  int n_row_blocks;
  // column-sorted view, built with the plan
  const int32_t* csc_row;  // nnz: row of the p-th entry in column order
  const float* csc_val;    // nnz: its value
  const int32_t* chunk_beg, *chunk_end;   // n_chunks ranges of that order, each inside one column
  const int32_t* col_first_chunk;         // cols + 1
  int n_chunks;
  const int32_t* colptr;   // cols + 1: ranges of that order
  int logR, logC;          // lanes per row and per column of the lane-group products
};

// Lane-group products of several sparse sources in one launch (kernels_sparse.hip).
constexpr int kSparseMulti = 4;
struct SparsePart {
  SparseArgs a;
  const float* X; int ldx, col0, ncols;   // rows: the operand; columns: the rows of Z
  float* out; int ldo;                    // rows: P, rows x ldo; columns: [cols][kNarrowCT]
};
// What becomes of the transposed products: mode -1: the parts' outputs; 0: the result, row colmap[j] of column j; 1: the update
// of Alg. 1 and the loss (one more workgroup).  For modes 0 and 1 every row of the result is fed by one column of the parts.
struct SparseFin {
  int mode;
  float* out; int ldo, col0;          // c_T x ldo: the result, or the weights
  const float* lr;
  float inv_rT;
  const float* loss_partial;
  int n_loss_partial;
  float* loss;
  float loss_scale;
};
struct SparseMultiArgs {
  int n;
  int first[kSparseMulti + 1];
  SparsePart s[kSparseMulti];
  SparseFin f;
};

// Gradient-descent pass over a two-table star join for a wide batch of models (kernels_star.hip).
struct StarArgs {
  const float* S;            // r_T x cs, row i of S is target row i
  int cs;
  const int32_t* s_colmap;   // device int32[cs]
  const float* W;            // c_T x ldw
  int ldw, m;
  float* PZ;                 // r_R x ldp: in  P = R W_R,  out  Z = segment sums of the residual
  int ldp;
  int64_t r_R;
  const int32_t* rowptr;     // r_R + 1: inverse index of the dimension table (every target row joins one row)
  const int32_t* perm;       // r_T
  const int32_t* idx;        // r_T: row of R each target row joins
  const float* y;            // r_T
  const float* Sp;           // NULL, or S with its rows in join order (Sp[p, :] = S[perm[p], :]) ...
  const int32_t* keys;       // ... with the row of R each of those rows joins, r_T ...
  const float* yp;           // ... and, if not NULL, their labels, r_T
  float* loss_partial;       // [gridDim.x][ld_loss]
  int ld_loss;
  float* grad_partial;       // [gridDim.x][cs][ld_grad] partials of S^T E
  int ld_grad;
};

// The entity table's share of the Gram matrix of a two-table star join, one pass in join order
// (kernels_gram_star.hip).
struct GramStarArgs {
  const float* S; int cs;            // r_T x cs, row i of S is target row i
  int64_t r_R;                       // rows of the dimension table
  const int32_t* rowptr;             // r_R + 1: inverse index of R (every target row joins one row)
  const int32_t* perm;               // r_T
  const int32_t* idx;                // r_T: row of R each target row joins
  const float* Sp;                   // NULL, or S with its rows in join order (Sp[p, :] = S[perm[p], :]): then a plain stream
  float* ss_partial;                 // [gridDim.x][cs][cs] partials of S^T S (upper-triangle 16 x 16 tiles)
  float* zc;                         // r_R x cs: rows of S summed per row of R
};

// Join-order transposed multiply of one joined source (kernels_tmm_join.hip).
struct TmmJoinArgs {
  const float* D; int ck;            // r_k x ck source table
  int64_t r_k;
  const int32_t* rowptr;             // r_k + 1: inverse index
  const int32_t* perm;               // target rows in source-row order
  const float* Y; int ldy, col0, c;  // operand columns [col0, col0 + c), c <= 16
  float* partial;                    // [gridDim.x][ck][c]
};

struct SegArgs {
  const int32_t* rowptr;   // r_k + 1
  const int32_t* perm;     // nnz
  const int32_t* chunk_seg, *chunk_beg, *chunk_end;  // long-segment chunks
  const int32_t* long_seg, *long_first;              // long segments and their chunk ranges
  int n_chunks, n_long;
  int n_multi;             // chunks [0, n_multi) belong to segments of several; each of the others is a segment
  int long_thr;            // longest segment that is summed by a group of lanes
  int64_t r_k;
  const float* Y;          // rows addressed through perm (and gidx if given)
  int ldy, col0, ncols;
  const int32_t* gidx;     // optional second-level gather: Y row = gidx[perm[p]] (skip if < 0)
  int64_t g_rows;          // with gidx == NULL and g_rows >= 0: rows >= g_rows are skipped
  float* Z;                // r_k x ldz
  int ldz, zcol0;
  float* chunk_partial;    // n_chunks x ncols
  int logG;                // lanes per segment in the narrow kernel
  const int32_t* block_first;  // join-order column reduce: workgroup b owns source rows [block_first[b], block_first[b + 1])
  // sliced form (large target tables): a second copy of the index ordered by (slice of target rows, source row)
  const int32_t* sl_rowptr;    // [kSegSlices * r_k + 1] entries of (slice x, source row j) are sl_perm[sl_rowptr[x r_k + j] ..)
  const int32_t* sl_perm;      // NULL: no sliced index
  const int32_t* sl_chunk0;    // [kSegSlices][r_k] first chunk record of a run longer than kSlLong, else -1
  const int32_t* sl_ch_beg, *sl_ch_end;   // [kSegSlices][sl_cap] chunk records: ranges of sl_perm
  const int32_t* sl_nchunk;    // [kSegSlices] their number
  float* sl_ch_partial;        // [kSegSlices][sl_cap][CT] chunk sums
  int sl_cap, sl_logG;
  float* Zs;                   // [kSegSlices][r_k][CT] per-slice sums of the short runs
};

// Plain per-source products P_k = D_k (M_k^T X) of several sources in one launch (kernels_lmm.hip).
constexpr int kRowdotMulti = 4;
struct RowdotArgs {
  const float* D; int ck; int64_t rows;
  const int32_t* colmap;
  const float* X; int ldx, col0, ncols;
  float* out; int ldo;
  int logL, vw;                // lanes per row (log2), floats per vector load (4 or 2)
};
struct RowdotMulti {
  int n;
  int first[kRowdotMulti + 1];
  RowdotArgs a[kRowdotMulti];
};

// Segment sums of several sources in one launch, plain or sliced (kernels_tmm.hip).
constexpr int kSegMulti = 4;
struct SegMulti {
  int n;
  int first[kSegMulti + 1];    // workgroups [first[q], first[q + 1]) of the sum kernel serve source q (multiples of kSegSlices)
  int cfirst[kSegMulti + 1];   // ... of the kernel that adds the per-slice sums, or the chunks of long segments
  SegArgs s[kSegMulti];
};

// Segment sums in fixed point in LDS (kernels_segfix.hip).
constexpr int kFixThreads = 1024;
constexpr int kFixSlots = 20160;          // sums of 64 bits a workgroup holds
constexpr int kFixNear = 16;              // values outside the band of a walk that a wavefront lists in LDS ...
constexpr int kFixFar = 2048;             // ... and in memory
constexpr int kFixHead = 2;               // binades of the band above the largest of a run's first values
constexpr int kFixPerXcd = 32;            // workgroups an XCD holds
struct SegFix {
  const int32_t* idx;        // r_T
  const float* Y;            // r_T x ncols
  int64_t r_T, r_k;
  int64_t longest;           // target rows of the source row with the most of them; 0: not known
  float* Z;                  // r_k x ldz, columns [zcol0, zcol0 + ncols)
  int ldz, zcol0;
  int n_ranges, nsub, runs, bits, stride, room;   // set by the launcher
  float* partial;
  unsigned long long* far;   // room for each wavefront
};
struct SegFixMulti {
  int n;
  int first[kSegMulti + 1], cfirst[kSegMulti + 1], range_blocks[kSegMulti];
  SegFix s[kSegMulti];
};

// The assembly of gathered products alone with the segment sums of its residual (kernels_segfix.hip).
constexpr int kAsmFixSources = 4;
constexpr int kAsmFixSlots = 13420;       // sums of 64 bits and products of 32 a workgroup holds
struct AsmFix {
  int n;
  const int32_t* idx[kAsmFixSources];
  const float* P[kAsmFixSources];
  int keys[kAsmFixSources], off[kAsmFixSources];
  int ldp, col0, slots, bits, room;
  const float* y;
  int64_t r_T;
  float* loss_partial;       // [gridDim.x][kNarrowCT]
  float* partial;            // [gridDim.x][slots]
  unsigned long long* far;   // [gridDim.x][wavefronts][room]
};

struct ColredArgs {
  const float* D;
  int64_t rows;
  int ck;
  const float* Z;          // rows x ldz
  int ldz, col0, ncols;
  float* partial;          // [nblocks][ck][kNarrowCT]
  int64_t rows_per_block;
  int vec;
};

// Shares of a narrow transposed multiply that run in one launch (kernels_tmm.hip).
constexpr int kTmmParts = 4;
struct TmmParts {
  int n;
  int first[kTmmParts + 1];   // workgroups [first[q], first[q + 1]) serve part q
  int join[kTmmParts];        // 1: join-order form (segment sums in LDS), 0: operand rows read from c.Z
  ColredArgs c[kTmmParts];
  SegArgs s[kTmmParts];       // inverse index and operand of the join-order form
};

// Tables read through tiles of rows in LDS, several in one launch (kernels_tile.hip).
constexpr int kTileParts = 4;
struct TilePart {
  const float* D; int ck; int64_t rows;
  const int32_t* colmap;              // product
  const float* X; int ldx, col0, ncols;   // product: the operand; column reduce: the rows of Z
  float* out; int ldo;                // product: rows x ldo; column reduce: [workgroup][ck][kNarrowCT]
  int logR;                           // log2 of the rows per tile
};
struct TileMulti {
  int n;
  int first[kTileParts + 1];          // workgroups [first[q], first[q + 1]) serve part q
  TilePart a[kTileParts];
};

struct FinSource {
  const int32_t* tcol2src;  // c_T
  const float* partial;     // [nblocks][ck][kNarrowCT]
  int nblocks, ck;
};

struct FinArgs {
  int n;
  FinSource s[kMaxSources];
  float* out;  // c_T x ldo (or W for the update mode)
  int ldo, col0, ncols;
  // update mode
  const float* lr;
  float inv_rT;
  const float* loss_partial;
  int n_loss_partial;
  float* loss;
  float loss_scale;
};

struct MatArgs {
  int n;
  const float* D[kMaxSources];
  const int32_t* idx[kMaxSources];
  int64_t rows[kMaxSources];
  int ck[kMaxSources];
  float* T;
  int64_t r_T;
  int c_T;
  // optional tables for the flat form: per group of four target columns the feeding source slot (-1: nobody) and
  // its first source column; NULL unless every fed group is four 16-byte-aligned values of one source
  const int32_t* gslot;
  const int32_t* gj0;
};

// Join-gather through tiles of whole target rows in LDS (kernels_mat.hip): any column map, any alignment.
constexpr int kMatTileFloats = 5120;     // floats of a tile aimed at (20 KiB)
constexpr int kMatTileMaxCols = 3584;    // four rows of so many columns, and their row numbers, fit 64 KiB of LDS
struct MatTileSource {
  const float* D;
  const int32_t* idx;      // NULL: identity on the first `rows` target rows
  const int32_t* colmap;   // device int32[ck], read when c0 < 0
  const int32_t* tcol;     // device int32[c_T], column of D behind a target column (-1: none), read when c0 < 0
  int64_t rows;
  int ck, c0;              // c0 >= 0: column j feeds target column c0 + j
  int vec;                 // floats per load (1 when c0 < 0)
  unsigned nv, magic;      // ck / vec and ceil(2^32 / nv): e / nv = mulhi(e, magic) for e * nv < 2^32
};
struct MatTileArgs {
  int n;
  MatTileSource s[kMaxSources];
  float* T;
  int64_t r_T;
  int c_T, rt;             // rt: rows per tile (set by the launcher)
  int zero;                // some column has no feeder, or several: tiles start from zero
  int add;                 // some column has several feeders: sources are added one after the other
};

// Transposed reduction  C = sum_t w_t a_t^T b_t  on the matrix cores (see kernels_tred.hip).
struct TredArgs {
  const float* A; int lda, ca; const int32_t* ia; int64_t a_rows;   // row t of A = A[ia ? ia[t] : t]
  const float* B; int ldb, cb, bcol0; const int32_t* ib; int64_t b_rows;
  const int32_t* wptr;     // optional: w_t = wptr[t+1] - wptr[t]
  int64_t n_rows, rows_per_block;
  float* partial;          // [row chunk][ca][cb]
  int gx, gy;              // set by launch_tred: row chunks and output tiles of the launch (see tred_block_ids)
  int upper_only;          // A == B: only tiles touching the upper triangle are computed
};

struct ColAsmArgs {
  int n;
  const int32_t* tcol2src[kMaxSources];
  const float* G[kMaxSources];   // c_k x cx each; with nparts[k] > 1: that many such blocks, to be added in order
  int nparts[kMaxSources];       // (0 counts as 1)
  int ck[kMaxSources];
  int c_T, cx;
  float* out;                    // c_T x cx
  const float* lr;
  float inv_rT;
  const float* loss_partial;     // [n_loss_partial][cx]
  int n_loss_partial;
  float* loss;
  float loss_scale;
  // KMeans: sizes[n_sizes][cx], the shares of the cluster sizes; out receives the means of the clusters that have members
  const int32_t* sizes;
  int n_sizes;
  int32_t* counts;               // cx, or NULL
};

struct GramAsmPair { const float* block; int k, l, cb; };

// Records `msg` as the calling thread's last error (what ilargi_last_error returns) and returns `code`.
ilargi_status_t set_error(ilargi_status_t code, const char* msg);

// One gradient-descent iteration on a small two-table star join in a single workgroup (kernels_small.hip).
constexpr size_t kSmallGdMaxLds = 152 << 10;    // dynamic LDS the kernel may use (of the 160 KiB of a compute unit)
struct SmallStarArgs {
  const float* S; int cs;       // entity table r_T x cs: cs <= 16, a multiple of 4, 16-byte aligned
  const float* R; int cr, r_R;  // joined table (NULL: none), r_R <= 1024 rows, cr <= 16
  const int32_t* idx;           // r_T keys into R (-1: none)
  const int32_t* rowptr;        // inverse index of R
  const int32_t* perm;
  int nnz;
  const int32_t* tcol_s;        // device int32[c_T]: column of S feeding target column t, or -1
  const int32_t* tcol_r;
  int16_t colmap[2][16];        // target column of every column of S and of R, or -1
  int s_first;                  // S comes before R in the plan (order of the sums in shared target columns)
  float* W; int ldw, col;       // weight column `col` of the c_T x ldw matrix, updated in place
  const float* y; const float* lr; float* loss;
  int r_T, c_T;
  float inv_rT, loss_scale;
};
int small_star_max_rows(int nvs);
size_t small_star_lds_bytes(const SmallStarArgs& a);
hipError_t launch_small_star(const SmallStarArgs& a, int mode, hipStream_t st);

// Gradient-descent pass that joins the rows of its sources on the fly in target order (kernels_rowjoin.hip).
constexpr int kRowJoinSources = 3;
struct RowJoinArgs {
  int n;                                    // sources, 1 .. kRowJoinSources
  const float* D[kRowJoinSources];          // rows[s] x ck[s], 16-byte aligned, ck a multiple of 4, at most 64
  int ck[kRowJoinSources];
  int64_t rows[kRowJoinSources];
  const int32_t* idx[kRowJoinSources];      // r_T row indices (-1: none); NULL: identity on the first rows[s] target rows
  const int32_t* colmap[kRowJoinSources];   // device int32[ck]
  const float* W; int ldw, col;             // weight column `col` of the c_T x ldw matrix
  const float* y; int64_t r_T;
  float* loss_partial;                      // [gridDim.x][kNarrowCT]
  float* grad_partial[kRowJoinSources];     // [gridDim.x][ck][kNarrowCT] partials of D_s^T e
};
bool gd_rowjoin_supported(const RowJoinArgs& a);
hipError_t launch_gd_rowjoin(const RowJoinArgs& a, int mode, int max_grid, hipStream_t st, int* grid_out);

// Gradient-descent pass of one model over a two-table star join whose entity table is kept in join order
// (kernels_gd_cluster.hip): both tables are read once, no product, residual or segment sum is stored.
struct ClusterArgs {
  const float* Sp; int cs;                  // the entity table with its rows in join order, r_T x cs, 16-byte aligned
  const int32_t* keys;                      // int32[r_T], ascending: the row of the dimension table each of those rows joins
  const int32_t* perm;                      // int32[r_T]: its target row (where its label is)
  const float* R; int cr; int64_t r_R;      // dimension table, r_R x cr, 16-byte aligned, cr a multiple of 4, at most 256
  const int32_t* s_colmap;                  // device int32[cs], int32[cr]: target column of every table column (-1: none)
  const int32_t* r_colmap;
  const float* W; int ldw, col;             // weight column `col` of the c_T x ldw matrix
  const float* y; int64_t r_T;
  const float* yp;                          // the labels in join order, float[r_T], or NULL (then y is gathered through perm)
  float* loss_partial;                      // [gridDim.x][kNarrowCT]
  float* grad_partial_s;                    // [gridDim.x][cs][kNarrowCT] partials of S^T e
  float* grad_partial_r;                    // [gridDim.x][cr][kNarrowCT] partials of R^T (I_R^T e)
};
bool gd_cluster_supported(int cs, int cr);
// Sp[p, :] = S[perm[p], :], keys[p] = idx[perm[p]] and, with labels y, yp[p] = y[perm[p]] for p < r_T.
hipError_t launch_cluster_rows(const float* S, int cs, const int32_t* perm, const int32_t* idx, int64_t r_T, float* Sp,
                               int32_t* keys, const float* y, float* yp, hipStream_t st);
hipError_t launch_gd_cluster(const ClusterArgs& a, int mode, int max_grid, hipStream_t st, int* grid_out);

// ---- launchers (each enqueues on `st`; returns the HIP error of the launch) ----
// *lines += lines of 32 keys that 64 consecutive entries hold, summed over kLineSamples places spread over the r_T >= 64 entries.
constexpr int kLineSamples = 256;
hipError_t launch_count_lines(const int32_t* idx, int64_t r_T, int32_t* lines, hipStream_t st);
hipError_t launch_check_idx(const int32_t* idx, int64_t r_T, int64_t r_k, int32_t* flags, hipStream_t st);
hipError_t launch_sort_by_source_row(const int32_t* idx, int64_t r_T, int64_t r_k, int32_t* keys_a,
                                     int32_t* vals_a, int32_t* keys_b, int32_t* vals_b, int32_t* hist,
                                     int32_t* rowptr, int32_t* perm, hipStream_t st);
size_t sort_hist_ints(int64_t r_T);
// In-place exclusive prefix sum of n integers on the device; `totals` is scratch of ceil(n / 1024) integers.
void launch_exclusive_scan(int32_t* a, int64_t n, int32_t* totals, hipStream_t st);

hipError_t launch_lmm_rows(const LmmArgs& a, int vec, int mode, hipStream_t st, int* grid_out);
// Assembly with one lane per target row (kernels_lmm_lane.hip): one operand column, identity source with short rows.
bool lmm_lane_supported(const LmmArgs& a, int vec, int mode, bool fuseg);
hipError_t launch_lmm_lane(const LmmArgs& a, int vec, int mode, hipStream_t st, int* grid_out);
// The streaming product kernel: dense table, at most four operand columns, rows of aligned vectors of vec = 4 or 2
// floats; the products of up to kRowdotMulti sources (same operand columns) can share one launch.
bool rowdot_supported(const LmmArgs& a, int vec);
hipError_t launch_rowdot_multi(const LmmArgs* a, const int* vec, int n, hipStream_t st);
bool prod_tile_supported(const LmmArgs& a, int vec);
hipError_t launch_prod_tile(const LmmArgs* a, int n, hipStream_t st);
bool asm_tile_supported(const LmmArgs& a, int vec, bool fuseg);
hipError_t launch_asm_tile(const LmmArgs& a, int mode, hipStream_t st, int* grid_out);
bool colred_tile_supported(const ColredArgs& c);
bool colred_tile_pays(const ColredArgs& c);
hipError_t launch_colred_tile(const ColredArgs* c, int n, int* nblocks, hipStream_t st);
int lmm_grid(int64_t r_out, int logL, bool fuseg);
bool lmm_can_fuse_gradient(int ck, int vec, int logL);
MfmaShape lmm_mfma_shape(int ck, int nt, bool gathers, bool bf16);
bool lmm_mfma_can_fuse_gradient(int ck, int ncols, bool bf16);
hipError_t launch_lmm_mfma(const LmmArgs& a, int vec, int mode, bool bf16, hipStream_t st, int* grid_out);
bool lmm_flat_pair_supported(const LmmArgs& a, int vec, bool fuseg);
hipError_t launch_lmm_flat_pair(const LmmArgs& a, int mode, bool fuseg, hipStream_t st, int* grid_out);
bool lmm_prod_f32_wide_supported(const LmmArgs& a, int vec, int mode);
hipError_t launch_lmm_prod_f32_wide(const LmmArgs& a, hipStream_t st);
bool lmm_prod_bf16_supported(const LmmArgs& a, int vec, int mode);
hipError_t launch_lmm_prod_bf16(const LmmArgs& a, hipStream_t st);
bool lmm_prod_stream_supported(const LmmArgs& a, int vec, int mode);
hipError_t launch_lmm_prod_stream(const LmmArgs& a, hipStream_t st);
bool lmm_flat_wide_supported(const LmmArgs& a, int vec, int mode);
hipError_t launch_lmm_flat_wide(const LmmArgs& a, hipStream_t st, int* grid_out);
bool gd_star_wide_supported(int cs, int m);
bool gd_star_wide_pays(int cs, int m, int64_t r_R, int vec, int mode, bool bf16);
hipError_t launch_gd_star_wide(const StarArgs& a, int vec, int mode, bool bf16, int max_grid, hipStream_t st, int* grid_out);
bool gd_star_supported(int cs, int m);
hipError_t launch_gd_star(const StarArgs& a, int vec, int mode, bool bf16, int max_grid, hipStream_t st, int* grid_out);
hipError_t launch_csr_check(const SparseArgs& a, int32_t* flags, hipStream_t st);
hipError_t launch_csr_entry_rows(const SparseArgs& a, int32_t* entry_row, hipStream_t st);
hipError_t launch_csr_gather_rows(const int32_t* entry_row, const float* val, const int32_t* perm, int64_t nnz,
                                  int32_t* csc_row, float* csc_val, hipStream_t st);
int sparse_row_block_cap(int cols);
hipError_t launch_spmm_rows(const SparseArgs& a, const float* X, int ldx, int col0, int ncols, float* P, int ldp,
                            hipStream_t st);
hipError_t launch_spmm_t(const SparseArgs& a, const float* Z, int ldz, int col0, int ncols, float* partial, float* G,
                         hipStream_t st);
hipError_t launch_spmm_lanes_rows(const SparsePart* s, int n, hipStream_t st);
hipError_t launch_spmm_lanes_cols(const SparsePart* s, int n, const SparseFin& f, hipStream_t st);
hipError_t launch_mat_scatter(const SparseArgs* sparse, const float* D, int64_t rows, int ck, const int32_t* colmap,
                              const int32_t* idx, int64_t ident_rows, float* T, int64_t r_T, int c_T, hipStream_t st);
hipError_t launch_segsum(const SegArgs& a, hipStream_t st);
hipError_t launch_segsum_narrow(const SegArgs* a, int n, hipStream_t st);   // n <= kSegMulti sources, same operand columns
// Builds the sliced copy of an inverse index (see SegArgs): sl_rowptr, sl_perm, the chunk records of long runs.
// src_beg: scratch of kSegSlices * r_k integers; scan_scratch: of (kSegSlices * r_k + 1) / 1024 + 1 integers.
hipError_t launch_build_sliced_index(const int32_t* rowptr, const int32_t* perm, int64_t r_k, int64_t nnz, int64_t slice_rows,
                                     int32_t* sl_rowptr, int32_t* sl_perm, int32_t* sl_chunk0, int32_t* ch_beg, int32_t* ch_end,
                                     int32_t* sl_nchunk, int cap, int32_t* src_beg, int32_t* scan_scratch, hipStream_t st);
int64_t segsum_sliced_chunk_cap(int64_t nnz);
// n <= kSegMulti sources with the same number of operand columns; their sums and the sums over slices run as one
// launch each.
hipError_t launch_segsum_sliced(const SegArgs* a, int n, hipStream_t st);
// Segment sums in fixed point in LDS of n <= kSegMulti sources, and the assembly of gathered products with them.
bool segfix_pays(int64_t r_T, const int64_t* rows, const bool* in_order, int n, int ncols, bool cut, int64_t longest);
// lines: 128-byte lines of a column of the source that 64 target rows in a row read.
inline bool keys_in_order(float lines, int64_t rows) { return lines < 2.5f && rows > 64; }
hipError_t launch_segfix(const SegFix* a, int n, int ncols, float* scratch, int64_t scratch_floats, hipStream_t st);
bool asm_fix_supported(const LmmArgs& a, int mode);
bool asm_fix_pays(const LmmArgs& a, const float* lines);
hipError_t launch_asm_fix(const LmmArgs& a, int mode, float* const* Z, float* scratch, int64_t scratch_floats, hipStream_t st, int* grid_out);
hipError_t launch_colred(const ColredArgs& a, int nblocks, hipStream_t st);
// Whether the choice of the assembly over such a table asks for the lines that gathers go to, and the choice.  lines[s]: 128-byte
// lines of a column P_s that 64 target rows in a row read.
bool lmm_lane_wants_lines(int64_t rows, int64_t cols);
bool lmm_lane_lds_pays(const LmmArgs& a, const float* lines);
bool asm_row_supported(const LmmArgs& a, int mode, bool fuseg);
hipError_t launch_asm_row(const LmmArgs& a, int mode, hipStream_t st, int* grid_out);
bool lmm_flat_supported(const LmmArgs& a, int vec, bool fuseg);
hipError_t launch_lmm_flat(const LmmArgs& a, int mode, bool fuseg, hipStream_t st, int* grid_out);
hipError_t launch_finalize(const FinArgs& a, int c_T, int mode, hipStream_t st);
int colred_step_rows(int ck, int vec);
bool tmm_part_supported(const ColredArgs& c, const SegArgs* s);
hipError_t launch_tmm_parts(const TmmParts& t, hipStream_t st);
bool materialize_flat_supported(const MatArgs& a);
hipError_t launch_materialize_flat(const MatArgs& a, hipStream_t st);
bool materialize_tile_supported(const MatTileArgs& a);
hipError_t launch_materialize_tile(MatTileArgs a, hipStream_t st);
hipError_t launch_materialize_slab(const MatTileArgs& a, hipStream_t st);
hipError_t launch_gram_assemble(const GramAsmPair* pairs_dev, int npairs, const int32_t* const* tcol2src_dev,
                                int c_T, float* out, hipStream_t st);
bool tmm_join_supported(int ck, int c);
hipError_t launch_tmm_join(const TmmJoinArgs& a, int64_t partial_floats, hipStream_t st, int* grid_out);
bool gram_star_supported(int cs);
hipError_t launch_gram_star(const GramStarArgs& a, int vec, int max_grid, hipStream_t st, int* grid_out);
// Gram blocks of tables with at most 64 columns as streaming matrix-core kernels (kernels_gram_narrow.hip): the
// diagonal block of a table with 36..64 columns, and the block of two tables over a list of row pairs.
bool gram_narrow_supported(const TredArgs& a);
bool gram_pairs_supported(const TredArgs& a);
bool gram_pairs_pay(const TredArgs& a, int64_t r_T);
hipError_t launch_gram_narrow(TredArgs& a, float* partial, int64_t partial_floats, hipStream_t st, int* nch_out);
hipError_t launch_pair_list(const int32_t* idx_a, int64_t rows_a, const int32_t* idx_b, int64_t rows_b, int64_t r_T,
                            int32_t* scan, int32_t* totals, int32_t* list_a, int32_t* list_b, hipStream_t st);
bool gram_sym_supported(const TredArgs& a);
hipError_t launch_gram_sym(TredArgs& a, float* partial, int64_t partial_floats, float* block, hipStream_t st);
hipError_t launch_tred(const TredArgs& a, int nchunks, bool bf16, hipStream_t st);
// streaming column reduce over plain rows (kernels_wide_bf16.hip): a.partial receives a.gx blocks of ca x cb
bool tred_stream_supported(const TredArgs& a);
int tred_stream_grid(const TredArgs& a, int64_t partial_floats);
hipError_t launch_tred_stream(TredArgs& a, int grid, bool bf16, hipStream_t st);
void tred_occupancy(const TredArgs& a, bool bf16, int* slots, int* tiles);
// G = S^T Y for an identity source with rows of at most 16 float4 and 5..16 operand columns (kernels_colred_flat.hip).
struct ColredFlatArgs {
  const float* S; int64_t rows; int nvec;   // rows x (4 nvec), 16-byte aligned
  const float* Y; int ldy; int c;           // operand rows 0 .. rows - 1, columns 0 .. c - 1
  float* partial;                           // [workgroup][4 nvec][c]
};
bool colred_flat_supported(const float* S, int64_t cols, int c);
hipError_t launch_colred_flat(const ColredFlatArgs& a, int64_t partial_floats, hipStream_t st, int* grid_out);
// The flat column reduce of an identity source and the join-order pass of a joined source (nnz_j index entries) in one
// launch; *grid_f and *grid_j workgroups leave partial blocks in f.partial and j.partial.
bool tmm_pair_supported(const ColredFlatArgs& f, const TmmJoinArgs& j);
hipError_t launch_tmm_pair(const ColredFlatArgs& f, const TmmJoinArgs& j, int64_t nnz_j, int64_t room_f, int64_t room_j,
                           hipStream_t st, int* grid_f, int* grid_j);
// tcols > 0: the summed (elems / tcols) x tcols matrix is written transposed
hipError_t launch_tred_reduce(const float* partial, int nchunks, int64_t elems, float* block, hipStream_t st, int tcols = 0);
// The same for several matrices in one launch.
constexpr int kTredReduceMulti = 8;
struct TredReduce { const float* partial; int nchunks; int64_t elems; float* block; int tcols; };
struct TredReduceMulti { int n; int first[kTredReduceMulti + 1]; TredReduce r[kTredReduceMulti]; };
hipError_t launch_tred_reduce_multi(const TredReduce* r, int n, hipStream_t st);
// Blocks (nparts) of more than 64 operand columns: whole float4s, in partial buffers on 16 bytes.
inline bool colasm_wide_supported(int cx) { return cx > 64 && cx % 4 == 0; }
hipError_t launch_colasm(const ColAsmArgs& a, int mode, hipStream_t st);
hipError_t launch_probe(int kind, float* dst, const float* src, int64_t n_floats, int blocks, hipStream_t st);
hipError_t launch_fill_zero(float* p, int64_t n, hipStream_t st);
hipError_t launch_fill(float* p, int64_t n, float v, hipStream_t st);
hipError_t launch_transpose(const float* in, int64_t rows, int64_t cols, float* out, hipStream_t st);
hipError_t launch_eye_block(float* E, int64_t rows, int w, int64_t j0, hipStream_t st);   // columns j0.. of the identity
hipError_t launch_mirror_upper(float* G, int64_t n, hipStream_t st);                      // lower triangle := upper
constexpr int64_t kSparseGramMaxCols = 16384;   // crossprod over sparse sources: the c_T x c_T result stays below 1 GiB
constexpr int kSparseGramWidth = 16;            // identity columns multiplied through per round
hipError_t launch_fanout(const int32_t* rowptr, int64_t rows, float* cnt, hipStream_t st);
hipError_t launch_elementwise(int op, const float* in, float* out, int64_t n, float x, hipStream_t st);
// KMeans / Gaussian NMF row-local steps (kernels_models.hip)
constexpr int kKmeansMaxK = 256;
constexpr int kGnmfMaxRank = 64;
hipError_t launch_centroid_norm(const float* C, int64_t c_T, int k, float* cn, hipStream_t st);
hipError_t launch_kmeans_assign(float* P, const float* cn, int64_t r_T, int k, int32_t* assign, int32_t* counts_partial,
                                int64_t partial_ints, int32_t* counts, hipStream_t st);
constexpr int kKmeansTileK = 16;     // most centroids of the one-pass assignment (kernels_tile.hip)
bool kmeans_tile_supported(int ck, int k);
int kmeans_tile_grid(const LmmArgs& a, int* logR);
hipError_t launch_kmeans_tile(const LmmArgs& a, const float* cn, int64_t c_T, int32_t* assign, int32_t* counts_partial,
                              float* sum_partial, int grid, int logR, hipStream_t st);   // cn: centroid norms, NULL: formed there
// The same for entity tables of few columns over large target tables, a lane per row (kernels_kmeans.hip).
struct KmeansLaneArgs {
  const float* D; int ck; int64_t d_rows;   // the identity source: target rows [0, d_rows) take row i
  int t0;                                   // its columns are target columns [t0, t0 + ck); -1: they are no block
  const float* C; int c_T;                  // c_T x k
  const float* cn;                          // centroid norms, NULL: formed there
  int64_t r_T;
  int n;                                    // gathered sources
  const int32_t* idx[kTileParts];
  const float* P[kTileParts];               // rows x k
  int32_t* assign;                          // r_T
  int32_t* sizes;                           // [workgroup][k]
  float* sums;                              // [workgroup][ck][k]
};
bool kmeans_lane_supported(const KmeansLaneArgs& a, int k);
int kmeans_lane_grid(int64_t r_T);
hipError_t launch_kmeans_lane(const KmeansLaneArgs& a, int k, int grid, hipStream_t st);
hipError_t launch_kmeans_counts(const int32_t* partial, int nparts, int k, int32_t* counts, hipStream_t st);
hipError_t launch_kmeans_segcount(const int32_t* rowptr, const int32_t* perm, const int32_t* assign, int64_t r_k, int k,
                                  int logG, float* Z, hipStream_t st);
hipError_t launch_kmeans_update(float* C, const float* G, const int32_t* counts, int64_t c_T, int k,
                                int32_t* counts_out, hipStream_t st);
hipError_t launch_gnmf_update(float* X, const float* P, const float* Q, int64_t rows, int k, float tiny,
                              float* gram_partial, int64_t partial_floats, int* nparts_out, hipStream_t st);

// An entity table of more than half the last-level cache (256 MiB) is not there any more when the next iteration asks
// for it.  Read past the caches it leaves them to the gathered operands: the assembly over 5,000,000 x 10 with three
// joined tables takes 72 microseconds instead of 102, the iteration over 5,000,000 x 11 in tiles 221 instead of 246.
// A table that stays between calls loses by it (1,000,000 x 20, trained: 68.7 against 67.5 an iteration with three copies
// in turn, 67.9 against 65.2 with one), and so does a joined table, which an iteration reads twice.  Kernels take it as
// a template argument: of two branches with the same loads the compiler makes one.
inline int stream_past_caches(int64_t floats) { return floats >= (32ll << 20) ? 1 : 0; }

// A float4 read past the caches, or through them.
template <bool NT>
__device__ __forceinline__ float4 load4(const float* p) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  f4 t;
  if constexpr (NT) t = __builtin_nontemporal_load(reinterpret_cast<const f4*>(p));
  else t = *reinterpret_cast<const f4*>(p);
  return make_float4(t.x, t.y, t.z, t.w);
}
// sigmoid(z) - y, and log(1 + exp(z)) - y z added to the loss.  One exponential, e = exp(-|z|), serves both (its relative
// error grows with |z|, to 16 units of 2^-24 at 20).  The sigmoid is the quotient 1 / (1 + e) or e / (1 + e) with one
// correction, which also takes in the rounding of 1 + e.  The logarithm is 2 atanh t with t = e / (2 + e) <= 1/3, the
// remainder of that quotient carried along, and atanh t = t + t^3 p(t^2), p of degree four fitted to 2e-3 units.
// Errors against 64 bits on this device, rms in units of 2^-24, for z normal with deviation 0.5 / with deviation 2 / uniform
// in +-20: sigmoid 0.25 / 0.24 / 0.21, log(1 + exp(z)) 0.43 / 0.68 / 2.23 (the last is the rounding of values up to 20).
// Two exponentials, a division and log1pf: 0.33 / 0.38 / 0.40 and 0.43 / 0.68 / 2.23.  Five iterations of 256 logistic
// models over 1,000,000 x 20 with 100,000 x 200, float32 / bfloat16 inputs: those 7555 / 6805 microseconds, this form 4372 /
// 2944; a Newton step and the native logarithm 4292 / 2872, but the logarithm's rms is then 0.64 / 0.74 / 2.23.
__device__ __forceinline__ float logistic_residual(float z, float y, float& loss) {
  const float e = __expf(-fabsf(z));
  const float d = 1.0f + e, d_lo = e - (d - 1.0f), inv_d = __builtin_amdgcn_rcpf(d);
  const float n = z >= 0.0f ? 1.0f : e, q = n * inv_d;
  const float sigmoid = fmaf(fmaf(-d, q, n) - d_lo * q, inv_d, q);
  const float b = 2.0f + e, b_lo = e - (b - 2.0f), inv_b = __builtin_amdgcn_rcpf(b);
  const float t = e * inv_b, t_lo = (fmaf(-b, t, e) - b_lo * t) * inv_b;
  const float u = t * t, t2 = 2.0f * t;
  const float p = fmaf(fmaf(fmaf(fmaf(0.12144784f, u, 0.10715369f), u, 0.14308299f), u, 0.19999444f), u, 0.33333337f);
  loss += fmaxf(z, 0.0f) + (t2 + fmaf(t2 * u, p, 2.0f * fmaf(t_lo, u, t_lo))) - y * z;
  return sigmoid - y;
}

// Sum of float4 records rec[b * stride4] over b < count by a whole workgroup: threads stride the records
// (four independent loads in flight each), xor butterfly inside the wavefronts, wavefronts added in order.
__device__ __forceinline__ float4 block_sum4(const float4* __restrict__ rec, int64_t stride4, int count,
                                             float (*scratch)[4]) {
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  float4 s0 = make_float4(0.f, 0.f, 0.f, 0.f), s1 = s0, s2 = s0, s3 = s0;
  int b = tid;
  for (; b + 3 * kBlock < count; b += 4 * kBlock) {
    float4 v0 = rec[(int64_t)b * stride4], v1 = rec[(int64_t)(b + kBlock) * stride4];
    float4 v2 = rec[(int64_t)(b + 2 * kBlock) * stride4], v3 = rec[(int64_t)(b + 3 * kBlock) * stride4];
    s0.x += v0.x; s0.y += v0.y; s0.z += v0.z; s0.w += v0.w;
    s1.x += v1.x; s1.y += v1.y; s1.z += v1.z; s1.w += v1.w;
    s2.x += v2.x; s2.y += v2.y; s2.z += v2.z; s2.w += v2.w;
    s3.x += v3.x; s3.y += v3.y; s3.z += v3.z; s3.w += v3.w;
  }
  for (; b < count; b += kBlock) {
    float4 v0 = rec[(int64_t)b * stride4];
    s0.x += v0.x; s0.y += v0.y; s0.z += v0.z; s0.w += v0.w;
  }
  float r[4] = {(s0.x + s1.x) + (s2.x + s3.x), (s0.y + s1.y) + (s2.y + s3.y), (s0.z + s1.z) + (s2.z + s3.z),
                (s0.w + s1.w) + (s2.w + s3.w)};
#pragma unroll
  for (int n = 0; n < 4; ++n)
    for (int m = kWave / 2; m >= 1; m >>= 1) r[n] += __shfl_xor(r[n], m);
  __syncthreads();   // scratch may still be read from a previous call
  if (lane == 0) {
#pragma unroll
    for (int n = 0; n < 4; ++n) scratch[wave][n] = r[n];
  }
  __syncthreads();
  float4 out;
  out.x = ((scratch[0][0] + scratch[1][0]) + scratch[2][0]) + scratch[3][0];
  out.y = ((scratch[0][1] + scratch[1][1]) + scratch[2][1]) + scratch[3][1];
  out.z = ((scratch[0][2] + scratch[1][2]) + scratch[2][2]) + scratch[3][2];
  out.w = ((scratch[0][3] + scratch[1][3]) + scratch[2][3]) + scratch[3][3];
  return out;
}

inline int ilog2_ceil(int64_t v) { int l = 0; while ((1ll << l) < v) ++l; return l; }

}  // namespace ilargi
#endif
