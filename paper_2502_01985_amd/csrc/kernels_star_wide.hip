// The gradient-descent pass of kernels_star.hip (see there for the scheme) for more than 128 models and an entity table
// of at most 32 columns: four wavefronts walk the same tiles of R, each for its own 64 model columns, and share the
// staged rows of S.  Gathered in join order, a row of S costs 1.5 cache lines on average, which one wavefront per tile
// and slab of 64 models fetches again for every slab.
// The workgroup owns a run of consecutive tiles of R with its share of the target rows, and sees those as one stream of
// batches of ST rows: a batch ends at its tile's end, the next one starts there, and while batch k is computed the rows of
// S of batch k + 1 and the row list of batch k + 2 are on their way.  One barrier per batch.  Which row of the tile a
// target row joins follows from its place between the tile's row pointers, without a look at its key.
// In float32 the matrix cores bound it: 52 MFMAs of 32 cycles per 16 rows and 64 models are 180 microseconds of the
// chip; with bfloat16 inputs the arithmetic of the residuals between the products.
// 1,000,000 x 20 with 100,000 x 200, 256 linear models: 331 microseconds in float32 (367 with a wavefront per tile and
// slab), 161 with bfloat16 inputs (253).  A wavefront without models of its own only stages rows, but its place on the
// compute unit stays taken: gd_star_wide_pays says which counts of models and tiles come here.  With 128 models or fewer,
// or wider tables, too few wavefronts fit beside the shared buffers and the one-wavefront form is the faster one
// (64 models: 246 microseconds an iteration against 317 with this scheme, 128: 358 and 375).
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "ilargi_internal.h"

namespace ilargi {

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// LDS writes of some lanes of a wavefront become visible to the others (one wavefront executes its LDS
// instructions in order; the fences only keep the compiler from moving accesses across this point).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

constexpr int kN = 64;        // model columns of a wavefront (four 16-column tiles)
constexpr int kNT = 4;
constexpr int SL = 4;         // wavefronts of the workgroup
constexpr int ST = 64;        // target rows of a batch
constexpr int JG = 2;         // 16-column tiles of S
constexpr int KP = 16 * JG;
constexpr int kTileCost = 48;  // weight of a tile of R beside its target rows.  1,000,000 rows, 256 linear models, float32: half
                               // of them on the first 1 % of 600,000 keys 1031 microseconds an iteration with 32, 1050 with
                               // 48, 1474 with 128; of 300,000 keys 825, 819, 1023; keys spread evenly level

// MODE 1: linear, 2: logistic.  VEC4: rows of S are read as float4.  BF16: values of S, W and E are rounded
// to bfloat16 (nearest even) where they enter a product.  lda: row stride of the staged rows (a constant: with a
// runtime stride the addresses alone cost bfloat16 inputs 75 microseconds of 160).
template <int MODE, bool VEC4, bool BF16, int lda>
__global__ __launch_bounds__(kWave * SL) __attribute__((amdgpu_waves_per_eu(MODE == 1 ? 3 : 2)))
void gd_star_wide_kernel(StarArgs a, int xfloats, int rtiles, int fold) {
  constexpr int kThreads = kWave * SL;
  extern __shared__ float lds[];
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const int li = lane % 16, q = lane / 16;
  float* As = lds;                                            // [2][ST][lda] staged rows of S
  float* Ps = As + 2 * (size_t)ST * lda + (size_t)wave * 16 * kN;   // [16][64] tile of P, later of Z
  int* iS = reinterpret_cast<int*>(As + 2 * (size_t)ST * lda + (size_t)SL * 16 * kN);   // [2][ST] target rows
  int* jS = iS + 2 * ST;                                      // [2][ST] row of the R tile each joins (-1: none)
  float* yS = reinterpret_cast<float*>(jS + 2 * ST);          // [2][ST] label
  int* rS = reinterpret_cast<int*>(yS + 2 * ST);              // [2][20] first index entry of every row of a tile of R
  float* Xs = reinterpret_cast<float*>(rS + 40) + (size_t)wave * xfloats;   // [ceil(cs / 4)][64][4]  (bf16: [KP / 8][64][8])
  const int n0 = (blockIdx.y * SL + wave) * kN;
  const int nw = __builtin_amdgcn_readfirstlane(max(0, min(kN, a.m - n0)));
  // fold: the table has 1..4 columns beyond whole groups of 16.  A tile of R then has 12 rows, and rows 12..15
  // of the segment-sum MFMA (whose A operand is the 0/1 indicator) carry those columns of S instead, so the
  // same MFMA forms their share of S^T E; they are collected in the last gacc slot by the lanes q == 3.
  const int tr = fold ? 12 : 16;                              // rows of R per tile
  const int full = a.cs / 16;
  const int njt = fold ? full : (a.cs + 15) / 16;             // 16-column groups of S that take their own MFMAs

  // this wavefront's columns of W, one per lane, all requested together (they travel while the run is looked for)
  float x[KP];
#pragma unroll
  for (int k = 0; k < KP; ++k) {
    const int t = k < a.cs ? a.s_colmap[k] : -1;
    x[k] = (t >= 0 && lane < nw) ? a.W[(int64_t)t * a.ldw + n0 + lane] : 0.0f;
  }

  auto tile_first = [&](int t) { return a.rowptr[min((int64_t)t * tr, a.r_R)]; };
  // This workgroup's run of tiles: the tiles that start in its share of the work, where an index entry weighs one and a
  // tile kTileCost (by number of tiles alone, popular keys that lie side by side all fall to a few workgroups: half of
  // 1,000,000 rows on the first 1 % of 100,000 keys, 256 models, 7078 microseconds an iteration and 990 this way).  A half
  // wavefront looks for either end, 32 tiles at a time: first around an even share of the tiles, where it mostly is.
  auto work_before = [&](int t) { return (int64_t)tile_first(t) + (int64_t)kTileCost * t; };
  const int64_t share = (int64_t)blockIdx.x + lane / 32, want = work_before(rtiles) * share / gridDim.x;
  int lo = 0, hi = rtiles;                                    // the end looked for lies in [lo, hi]
  int first = max((int)(rtiles * share / gridDim.x) - 16, 0), step = 1;
  while (__any(lo < hi)) {
    const int t = min(first + (lane % 32 + 1) * step - 1, hi);
    const unsigned reached = (unsigned)(__ballot(t == hi || work_before(t) >= want) >> (lane & 32));
    const int f = reached != 0 ? __builtin_ctz(reached) : 32; // tile first + (f + 1) step - 1 is the first one past the end
    if (f < 32) hi = min(first + (f + 1) * step - 1, hi);
    if (f > 0) lo = min(first + f * step, hi);
    first = lo;
    step = (hi - lo) / 32 + 1;
  }
  int t_lo = __builtin_amdgcn_readlane(lo, 0), t_hi = __builtin_amdgcn_readlane(lo, 32);
  if (rtiles <= (int)gridDim.x) { t_lo = blockIdx.x; t_hi = t_lo + 1; }   // a workgroup per tile

#pragma unroll
  for (int k = 0; k < KP; ++k) {
    if constexpr (BF16) reinterpret_cast<__bf16*>(Xs)[((k >> 3) * kN + lane) * 8 + (k & 7)] = (__bf16)x[k];
    else if (k < (a.cs + 3) / 4 * 4) Xs[((k >> 2) * kN + lane) * 4 + (k & 3)] = x[k];
  }
  wave_sync();

  float loss_local[kNT];
  v4f gacc[JG][kNT], zacc[kNT];
#pragma unroll
  for (int nt = 0; nt < kNT; ++nt) { loss_local[nt] = 0.0f; zacc[nt] = (v4f){0.0f, 0.0f, 0.0f, 0.0f}; }
#pragma unroll
  for (int jt = 0; jt < JG; ++jt)
#pragma unroll
    for (int nt = 0; nt < kNT; ++nt) gacc[jt][nt] = (v4f){0.0f, 0.0f, 0.0f, 0.0f};

  // staging slots of this thread: (row of the batch, float4 or scalar column slot), the same for every batch
  typedef typename std::conditional<VEC4, float4, float>::type SVal;
  constexpr int NV = ST * JG * (VEC4 ? 4 : 16) / kThreads;
  constexpr int kSlots = VEC4 ? KP / 4 : KP;                  // slots per staged row
  const int glive = VEC4 ? a.cs / 4 : a.cs;                   // slots inside the table (cs % 4 == 0 with VEC4)

  const float* Sb = a.Sp != nullptr ? a.Sp : a.S;
  const bool p_vec = (a.ldp % 4 == 0) && (reinterpret_cast<uintptr_t>(a.PZ) % 16 == 0);
  const int pr = lane / 16, pq = lane % 16;                   // (row mod 4, float4 slot) of the P / Z tile this lane moves

  // the row the entry p of the inverse index stands for and its label: through the target row, or straight from the
  // join-ordered copy of the table (and of the labels) when the plan keeps one
  auto row_at = [&](int p) { return a.Sp != nullptr ? p : a.perm[p]; };
  auto label_at = [&](int r) { return a.Sp == nullptr ? a.y[r] : (a.yp != nullptr ? a.yp[r] : a.y[a.perm[r]]); };

  // Batches: tile t of R, index entries [p, min(p + ST, pe)) with pe the tile's end.  (An empty tile is a batch of none.)
  struct Batch { int t, p, pe; };
  Batch bc = {t_hi, 0, 0}, bs = {t_hi, 0, 0};                 // computed now; its rows of S are requested
  Batch bl = {t_lo, t_lo < t_hi ? tile_first(t_lo) : 0, t_lo < t_hi ? tile_first(t_lo + 1) : 0};   // its row list is requested
  int pe_next = t_lo + 1 < t_hi ? tile_first(t_lo + 2) : 0;   // end of the tile after bl's
  int pi = -1, rb = 0, jl = -1;
  float yv = 0.0f;
  SVal sv[NV];
#pragma unroll
  for (int u = 0; u < NV; ++u) {
    if constexpr (VEC4) sv[u] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    else sv[u] = 0.0f;
  }
  auto request_list = [&]() {
    pi = -1;
    if (bl.t < t_hi) {
      if (tid < ST && bl.p + tid < bl.pe) pi = row_at(bl.p + tid);
      if (tid <= tr) rb = a.rowptr[min((int64_t)bl.t * tr + tid, a.r_R)];
    }
  };
  request_list();

  int tile_now = -1;
  for (int c = 0; bc.t < t_hi || bs.t < t_hi || bl.t < t_hi; c ^= 1) {
    if (bc.t < t_hi && nw > 0) {                              // (a wavefront beyond the batch of models only stages rows)
      if (bc.t != tile_now) {
        // a new tile of R: its P into LDS (zero beyond the table and the slab)
        tile_now = bc.t;
        wave_sync();
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int r = pr + 4 * u;
          const int64_t j = (int64_t)bc.t * tr + r;
          float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
          if (r < tr && j < a.r_R && 4 * pq < nw) {
            const float* p = a.PZ + j * a.ldp + n0 + 4 * pq;
            if (p_vec && 4 * pq + 3 < nw) {
              v = *reinterpret_cast<const float4*>(p);
            } else {
              v.x = p[0];
              if (4 * pq + 1 < nw) v.y = p[1];
              if (4 * pq + 2 < nw) v.z = p[2];
              if (4 * pq + 3 < nw) v.w = p[3];
            }
          }
          *reinterpret_cast<float4*>(Ps + r * kN + 4 * pq) = v;
        }
        wave_sync();
#pragma unroll
        for (int nt = 0; nt < kNT; ++nt) zacc[nt] = (v4f){0.0f, 0.0f, 0.0f, 0.0f};
      }
      const int cnt = min(ST, bc.pe - bc.p);
      const float* Ab = As + (size_t)c * ST * lda;
      const int* jb_s = jS + c * ST;
      const float* yb_s = yS + c * ST;
      // residual tile t of the batch: ov[nt][r] = residual of row 4 q + r, model column li of tile nt (rounded to
      // bfloat16 with BF16), ind[r] = the indicator (or folded table) value of that row for row li of the tile of R
      auto residual_tile = [&](int t, float (&ov)[kNT][4], float (&ind)[4]) {
        // z tile = S rows x W_S
        v4f acc[kNT];
#pragma unroll
        for (int nt = 0; nt < kNT; ++nt) acc[nt] = (v4f){0.0f, 0.0f, 0.0f, 0.0f};
        if constexpr (BF16) {
          const float* arow = Ab + (t * 16 + li) * lda + 8 * q;
#pragma unroll
          for (int step = 0; step < KP / 32; ++step) {
            float4 a0 = *reinterpret_cast<const float4*>(arow + 32 * step);
            float4 a1 = *reinterpret_cast<const float4*>(arow + 32 * step + 4);
            bf16x8 av;
            av[0] = (__bf16)a0.x; av[1] = (__bf16)a0.y; av[2] = (__bf16)a0.z; av[3] = (__bf16)a0.w;
            av[4] = (__bf16)a1.x; av[5] = (__bf16)a1.y; av[6] = (__bf16)a1.z; av[7] = (__bf16)a1.w;
            const bf16x8* xb = reinterpret_cast<const bf16x8*>(Xs) + (4 * step + q) * kN + li;
#pragma unroll
            for (int nt = 0; nt < kNT; ++nt)
              acc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, xb[nt * 16], acc[nt], 0, 0, 0);
          }
        } else {
          // whole groups of 16 table columns: one 128-bit read feeds four MFMAs; the remaining columns in
          // groups of four (K slot q = column kb + q), so that 20 columns cost 20 MFMAs per tile, not 32
          const float* arow = Ab + (t * 16 + li) * lda + 4 * q;
          for (int kb = 16 * full; kb < a.cs; kb += 4) {
            const float av = Ab[(t * 16 + li) * lda + kb + q];
            const float* xb = Xs + ((kb >> 2) * kN + li) * 4 + q;
#pragma unroll
            for (int nt = 0; nt < kNT; ++nt)
              acc[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, xb[nt * 64], acc[nt], 0, 0, 0);
          }
          for (int step = 0; step < full; ++step) {
            float4 av = *reinterpret_cast<const float4*>(arow + 16 * step);
            const float* xb = Xs + ((4 * step + q) * kN + li) * 4;
#pragma unroll
            for (int nt = 0; nt < kNT; ++nt) {
              float4 bv = *reinterpret_cast<const float4*>(xb + nt * 64);
              acc[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.x, bv.x, acc[nt], 0, 0, 0);
              acc[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.y, bv.y, acc[nt], 0, 0, 0);
              acc[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.z, bv.z, acc[nt], 0, 0, 0);
              acc[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.w, bv.w, acc[nt], 0, 0, 0);
            }
          }
        }
        // residual of rows 4 q + r, model column li of each 16-column tile
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = t * 16 + 4 * q + r;
          const int j = jb_s[row];                            // -1 beyond the batch
          const float yi = yb_s[row];
          ind[r] = j == li ? 1.0f : 0.0f;
          if (fold && li >= 12) {
            ind[r] = Ab[row * lda + 16 * full + (li - 12)];
            if constexpr (BF16) ind[r] = (float)(__bf16)ind[r];
          }
          // branch-free: rows beyond the batch (j < 0) read row 0 of the tile and are zeroed by a select; model
          // columns beyond the slab carry finite values (their W and P are zero) that no store lets out
          const bool live = j >= 0;
          const float* prow = Ps + max(j, 0) * kN + li;
#pragma unroll
          for (int nt = 0; nt < kNT; ++nt) {
            const float z = acc[nt][r] + prow[nt * 16];
            if constexpr (MODE == 1) {
              const float o = live ? z - yi : 0.0f;
              ov[nt][r] = o;
              loss_local[nt] = fmaf(o, o, loss_local[nt]);
            } else {
              float l = 0.0f;
              const float o = logistic_residual(z, yi, l);
              ov[nt][r] = live ? o : 0.0f;
              loss_local[nt] += live ? l : 0.0f;
            }
          }
        }
        // With BF16 the residual is rounded once as it enters the two products below
        if constexpr (BF16) {
#pragma unroll
          for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int nt = 0; nt < kNT; ++nt) ov[nt][r] = (float)(__bf16)ov[nt][r];
        }
      };
      if constexpr (!BF16) {
        for (int t = 0; 16 * t < cnt; ++t) {
          float ov[kNT][4];
          float ind[4];
          residual_tile(t, ov, ind);
          // segment sums (the product with the 0/1 indicator matrix), then S^T E
#pragma unroll
          for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int nt = 0; nt < kNT; ++nt)
              zacc[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(ind[r], ov[nt][r], zacc[nt], 0, 0, 0);
          const float* acol = Ab + (t * 16 + 4 * q) * lda + li;
#pragma unroll
          for (int jt = 0; jt < JG; ++jt) {
            if (jt < njt) {
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const float av = acol[r * lda + jt * 16];
#pragma unroll
                for (int nt = 0; nt < kNT; ++nt)
                  gacc[jt][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, ov[nt][r], gacc[jt][nt], 0, 0, 0);
              }
            }
          }
        }
      } else {
        // Two tiles (32 rows) at a time: their residuals, as they sit in the lanes, are the B operand of one
        // 16x16x32 bfloat16 MFMA whose K octet q stands for the rows 4 q .. 4 q + 3 of the first tile followed by
        // those of the second; the indicator (segment sums) and the staged table values (S^T E) are packed in the
        // same order.  Every value is a bfloat16 value already, every product exact, the sums float32.
        for (int t = 0; 16 * t < cnt; t += 2) {
          bf16x8 ia, eb[kNT];
          {
            float ov[kNT][4];
            float ind[4];
            residual_tile(t, ov, ind);                        // packed at once: one tile of float residuals alive at a time
#pragma unroll
            for (int r = 0; r < 4; ++r) ia[r] = (__bf16)ind[r];
#pragma unroll
            for (int nt = 0; nt < kNT; ++nt)
#pragma unroll
              for (int r = 0; r < 4; ++r) eb[nt][r] = (__bf16)ov[nt][r];
          }
          if (16 * (t + 1) < cnt) {
            float ov[kNT][4];
            float ind[4];
            residual_tile(t + 1, ov, ind);
#pragma unroll
            for (int r = 0; r < 4; ++r) ia[4 + r] = (__bf16)ind[r];
#pragma unroll
            for (int nt = 0; nt < kNT; ++nt)
#pragma unroll
              for (int r = 0; r < 4; ++r) eb[nt][4 + r] = (__bf16)ov[nt][r];
          } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) ia[4 + r] = (__bf16)0.0f;
#pragma unroll
            for (int nt = 0; nt < kNT; ++nt)
#pragma unroll
              for (int r = 0; r < 4; ++r) eb[nt][4 + r] = (__bf16)0.0f;
          }
#pragma unroll
          for (int nt = 0; nt < kNT; ++nt)
            zacc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ia, eb[nt], zacc[nt], 0, 0, 0);
          const float* acol = Ab + (t * 16 + 4 * q) * lda + li;
#pragma unroll
          for (int jt = 0; jt < JG; ++jt) {
            if (jt < njt) {
              bf16x8 sa;
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                sa[r] = (__bf16)acol[r * lda + jt * 16];
                sa[4 + r] = (__bf16)acol[(16 + r) * lda + jt * 16];
              }
#pragma unroll
              for (int nt = 0; nt < kNT; ++nt)
                gacc[jt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(sa, eb[nt], gacc[jt][nt], 0, 0, 0);
            }
          }
        }
      }
      if (bc.p + ST >= bc.pe) {
        // the tile of R is finished: its Z through Ps, so that rows leave as float4
        if (fold && q == 3) {
#pragma unroll
          for (int nt = 0; nt < kNT; ++nt) gacc[JG - 1][nt] += zacc[nt];
        }
        wave_sync();
#pragma unroll
        for (int nt = 0; nt < kNT; ++nt)
#pragma unroll
          for (int r = 0; r < 4; ++r) Ps[(4 * q + r) * kN + nt * 16 + li] = zacc[nt][r];
        wave_sync();
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int r = pr + 4 * u;
          const int64_t j = (int64_t)bc.t * tr + r;
          if (r < tr && j < a.r_R && 4 * pq < nw) {
            const float4 v = *reinterpret_cast<const float4*>(Ps + r * kN + 4 * pq);
            float* p = a.PZ + j * a.ldp + n0 + 4 * pq;
            if (p_vec && 4 * pq + 3 < nw) {
              *reinterpret_cast<float4*>(p) = v;
            } else {
              p[0] = v.x;
              if (4 * pq + 1 < nw) p[1] = v.y;
              if (4 * pq + 2 < nw) p[2] = v.z;
              if (4 * pq + 3 < nw) p[3] = v.w;
            }
          }
        }
      }
    }
    // hand over: the rows of S of the next batch, and the row list of the one after it, into LDS
    if (bs.t < t_hi) {
      float* An = As + (size_t)(c ^ 1) * ST * lda;
#pragma unroll
      for (int u = 0; u < NV; ++u) {
        const int e = tid + u * kThreads, r = e / kSlots, g = e % kSlots;
        if ((VEC4 ? 4 * g : g) >= lda) continue;              // (beyond the columns this table needs staged)
        if constexpr (VEC4) *reinterpret_cast<float4*>(An + r * lda + 4 * g) = sv[u];
        else An[r * lda + g] = sv[u];
      }
      if (tid < ST) { jS[(c ^ 1) * ST + tid] = jl; yS[(c ^ 1) * ST + tid] = yv; }
    }
    if (tid < ST) iS[c * ST + tid] = pi;
    if (tid <= tr) rS[c * 20 + tid] = rb;
    __syncthreads();
    bc = bs;
    bs = bl;
    if (bs.t < t_hi) {
      const int cnt = min(ST, bs.pe - bs.p);
#pragma unroll
      for (int u = 0; u < NV; ++u) {
        if constexpr (VEC4) sv[u] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        else sv[u] = 0.0f;
        const int e = tid + u * kThreads, r = e / kSlots, g = e % kSlots;
        if (r < cnt && g < glive) {
          const int64_t row = iS[c * ST + r];
          if constexpr (VEC4) sv[u] = *reinterpret_cast<const float4*>(Sb + row * a.cs + 4 * g);
          else sv[u] = Sb[row * a.cs + g];
        }
      }
      yv = 0.0f;
      jl = -1;
      if (tid < cnt) {
        yv = label_at(pi);
        const int p = bs.p + tid;                             // its row of the tile: rows that start at or before p
        for (int r = 0; r < tr; ++r) jl += rS[c * 20 + r] <= p ? 1 : 0;
      }
    }
    if (bl.t < t_hi) {
      bl.p += ST;
      if (bl.p >= bl.pe) {
        bl.p = bl.pe;
        ++bl.t;
        bl.pe = pe_next;
        if (bl.t + 1 < t_hi) pe_next = tile_first(bl.t + 2);
      }
    }
    request_list();
  }

  // S^T E and the loss of this workgroup's rows: every wavefront holds its own columns
#pragma unroll
  for (int jt = 0; jt < JG; ++jt) {
    const bool tail_slot = fold && jt == JG - 1;              // rows 16 full + r, held by the lanes q == 3
    if ((jt >= njt && !tail_slot) || (tail_slot && q != 3)) continue;
#pragma unroll
    for (int nt = 0; nt < kNT; ++nt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = tail_slot ? 16 * full + r : jt * 16 + 4 * q + r;
        const int n = nt * 16 + li;
        if (row < a.cs && n < nw) a.grad_partial[((int64_t)blockIdx.x * a.cs + row) * a.ld_grad + n0 + n] = gacc[jt][nt][r];
      }
  }
#pragma unroll
  for (int nt = 0; nt < kNT; ++nt) {
    float s = loss_local[nt];
    s += __shfl_xor(s, 16);
    s += __shfl_xor(s, 32);
    const int n = nt * 16 + li;
    if (q == 0 && n < nw) a.loss_partial[(int64_t)blockIdx.x * a.ld_loss + n0 + n] = s;
  }
}

typedef void (*StarFn)(StarArgs, int, int, int);

template <int MODE, bool B>
StarFn pick_star(bool vec4, int lda) {
  if constexpr (!B) {
    if (lda == 20) return vec4 ? gd_star_wide_kernel<MODE, true, B, 20> : gd_star_wide_kernel<MODE, false, B, 20>;
  }
  return vec4 ? gd_star_wide_kernel<MODE, true, B, KP + 4> : gd_star_wide_kernel<MODE, false, B, KP + 4>;
}

// Workgroups resident at once, on the device and on one compute unit.
int star_slots(StarFn fn, size_t lds_bytes, int* on_cu) {
  static std::mutex cache_mutex;   // the cache below is shared by every plan of the process
  std::lock_guard<std::mutex> lock(cache_mutex);
  static int cus = 0;
  static StarFn seen_fn[32];
  static size_t seen_lds[32];
  static int seen_occ[32];
  static int n_seen = 0;
  if (cus == 0) {
    int dev = 0;
    hipDeviceProp_t prop;
    cus = 256;
    if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess && prop.multiProcessorCount > 0)
      cus = prop.multiProcessorCount;
  }
  for (int i = 0; i < n_seen; ++i)
    if (seen_fn[i] == fn && seen_lds[i] == lds_bytes) { *on_cu = seen_occ[i]; return seen_occ[i] * cus; }
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(fn), kWave * SL, lds_bytes) != hipSuccess || per_cu < 1)
    per_cu = 1;
  if (n_seen < 32) { seen_fn[n_seen] = fn; seen_lds[n_seen] = lds_bytes; seen_occ[n_seen] = per_cu; ++n_seen; }
  *on_cu = per_cu;
  return per_cu * cus;
}

}  // namespace

bool gd_star_wide_supported(int cs, int m) { return cs > 0 && cs <= KP && m > 2 * kN; }

namespace {

struct WideShape {
  StarFn fn;
  int fold, rtiles, xfloats, gy;
  size_t lds_bytes;
  int64_t slots;                // workgroups resident at once
  int per_cu;                   // ... on a compute unit
};

WideShape wide_shape(int cs, int m, int64_t r_R, int vec, int mode, bool bf16) {
  WideShape w;
  const int tail = cs % 16;
  w.fold = (tail >= 1 && tail <= 4) ? 1 : 0;           // see the kernel: 12-row tiles of R
  const int tr = w.fold ? 12 : 16;
  w.rtiles = (int)((r_R + tr - 1) / tr);
  const bool vec4 = vec == 4;
  // Row stride of the staged rows, 4 modulo 8 floats: the 128-bit reads of 16 rows then fall on different banks.  The
  // bfloat16 product reads 32 columns of a row; in float32 the columns that are read are whole groups of four, or of 16
  // where such a group takes its own MFMAs, and up to 20 columns leave room for a third workgroup on a compute unit.
  const int need = w.fold ? (cs + 3) / 4 * 4 : (cs + 15) / 16 * 16;
  const int lda = !bf16 && need <= 20 ? 20 : KP + 4;
  if (bf16) w.fn = mode == 1 ? pick_star<1, true>(vec4, lda) : pick_star<2, true>(vec4, lda);
  else w.fn = mode == 1 ? pick_star<1, false>(vec4, lda) : pick_star<2, false>(vec4, lda);
  w.xfloats = bf16 ? KP * kN / 2 : (cs + 3) / 4 * 4 * kN;
  w.lds_bytes = sizeof(float) * (2 * (size_t)ST * lda + (size_t)SL * (16 * kN + w.xfloats) + 6 * (size_t)ST + 40);
  if (w.lds_bytes > 64 * 1024)
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(w.fn), hipFuncAttributeMaxDynamicSharedMemorySize, (int)w.lds_bytes);
  w.gy = (m + SL * kN - 1) / (SL * kN);
  w.slots = star_slots(w.fn, w.lds_bytes, &w.per_cu);
  return w;
}

}  // namespace

// Whether the shared rows pay.  Iterations over 1,000,000 rows of 8, 20 and 32 columns, 1000 to 100,000 rows of R, 192,
// 256, 320 and 384 models, time in this form over the time with a wavefront per tile and slab:
//   linear models with bfloat16 inputs (bound by the staged rows): 0.49 to 0.87 everywhere
//   no more tiles than compute units: 0.57 to 0.92 everywhere
//   a last workgroup with two idle wavefronts of eight or one of four: 0.97 to 1.69; with none, or one of eight:
//     logistic models with bfloat16 inputs: 0.85 to 0.96
//     float32 logistic: 0.75 to 0.86, but 1.13 where the tiles fill 1.2 rounds of workgroups
//     float32 linear (bound by the matrix cores): 0.94 to 0.95 with three workgroups on a compute unit and the last round
//       nine tenths full, else 1.00 to 1.30
bool gd_star_wide_pays(int cs, int m, int64_t r_R, int vec, int mode, bool bf16) {
  if (!gd_star_wide_supported(cs, m)) return false;
  if (bf16 && mode == 1) return true;
  const WideShape w = wide_shape(cs, m, r_R, vec, mode, bf16);
  const int64_t work = (int64_t)w.rtiles * w.gy;              // a tile and its 256 models
  if (work <= w.slots / w.per_cu) return true;
  if (2 * ((m + kN - 1) / kN) < 7 * w.gy) return false;
  if (bf16) return true;
  const int64_t rounds = (work + w.slots - 1) / w.slots;
  return mode == 2 ? 10 * work >= 8 * rounds * w.slots : w.per_cu >= 3 && (rounds == 1 || 10 * work >= 9 * rounds * w.slots);
}

// max_grid: the caller's bound on workgroups per slab of 256 models (sizes of the partial buffers).
hipError_t launch_gd_star_wide(const StarArgs& a, int vec, int mode, bool bf16, int max_grid, hipStream_t st, int* grid_out) {
  if (grid_out) *grid_out = 0;
  if (!gd_star_wide_supported(a.cs, a.m) || (mode != 1 && mode != 2) || a.r_R <= 0 || max_grid < 1) return hipErrorInvalidValue;
  const WideShape w = wide_shape(a.cs, a.m, a.r_R, vec, mode, bf16);
  int64_t gx = w.rtiles;
  // every workgroup walks its run of tiles: one round of resident workgroups
  if (gx * w.gy > w.slots) gx = std::max<int64_t>(1, w.slots / w.gy);
  gx = std::min<int64_t>(gx, max_grid);
  if (grid_out) *grid_out = (int)gx;
  hipLaunchKernelGGL(w.fn, dim3((unsigned)gx, (unsigned)w.gy), dim3(kWave * SL), w.lds_bytes, st, a, w.xfloats, w.rtiles, w.fold);
  return hipGetLastError();
}

}  // namespace ilargi
