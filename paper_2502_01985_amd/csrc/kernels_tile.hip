// Narrow operands (at most four columns a pass) over tables whose rows have no useful alignment, in three kernels
// built on one step: a tile of whole table rows is read as a flat run of float4 (the run starts on a float4 whatever
// the row length, because a tile starts at a row number that is a multiple of four), parked in LDS, and used from there
// in the mapping that the arithmetic wants.
//   product        P_k = D_k X_k               lanes of a row sum its columns
//   assembly       out = D X + sum_s P_s[row]  with the residual, the loss and D^T e of Alg. 1
//   column reduce  G_k = D_k^T Z_k             a thread owns a column and every nsub-th row of the tile
// All three are bound by reading the tables once; a lane that reads such a row itself does it one float at a time.
// The next tile's loads (and row numbers) are requested before the current one is used, and a tile is at most 20 KiB,
// so that four or more workgroups share a compute unit.  Measured for three logistic models over 333,333 x 13 joined
// with 9,001 x 33 and 41,003 x 75, before (a lane group per row, one float per lane) and now, in microseconds: products
// 27 (two launches) and 7, assembly 41 and 18, column reduces 11 (two launches) and 6.
#include <algorithm>
#include <cstring>

#include "ilargi_internal.h"

namespace ilargi {

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kTileFloats = 5120;                        // most floats of a tile
constexpr int kTileV = kTileFloats / 4 / kBlock;         // float4 a thread carries
constexpr int kTileGather = 4;                           // gathered sources of the assembly

// The whole float4s among n floats from p on into registers.  AL: p is 16-byte aligned.  NT: past the caches.
template <bool AL, bool NT>
__device__ __forceinline__ void tile_load(const float* __restrict__ p, int n, v4f (&v)[kTileV]) {
#pragma unroll
  for (int i = 0; i < kTileV; ++i) {
    const unsigned e = 4 * (threadIdx.x + i * kBlock);
    if (e + 4 <= (unsigned)n) {
      if constexpr (AL && NT) v[i] = __builtin_nontemporal_load(reinterpret_cast<const v4f*>(p + e));
      else if constexpr (AL) v[i] = *reinterpret_cast<const v4f*>(p + e);
      else v[i] = (v4f){p[e], p[e + 1], p[e + 2], p[e + 3]};
    }
  }
}

// The tile into LDS; the floats after its last whole float4 (only a table's last tile has any) straight from p.
__device__ __forceinline__ void tile_put(float* lds, const float* __restrict__ p, int n, const v4f (&v)[kTileV]) {
#pragma unroll
  for (int i = 0; i < kTileV; ++i) {
    const unsigned e = 4 * (threadIdx.x + i * kBlock);
    if (e + 4 <= (unsigned)n) *reinterpret_cast<v4f*>(lds + e) = v[i];
  }
  const unsigned tail = (unsigned)n & ~3u;
  if (tail + threadIdx.x < (unsigned)n) lds[tail + threadIdx.x] = p[tail + threadIdx.x];
}

// Operand rows X_k = M_k^T X, [ck][CT].
template <int CT>
__device__ __forceinline__ void stage_operand(const float* X, int ldx, int col0, int ncols, const int32_t* colmap, int ck, float* Xs) {
  for (int e = threadIdx.x; e < ck * CT; e += kBlock) {
    const int j = e / CT, n = e - j * CT;
    const int t = colmap[j];
    Xs[e] = (t >= 0 && n < ncols) ? X[(int64_t)t * ldx + col0 + n] : 0.0f;
  }
}

// acc += row `row` of the tile times the operand: the L = 2^logL lanes of a row take every L-th column.  A row length
// that is an even multiple of L would put the rows of a wavefront on the same banks: each row then starts elsewhere.
template <int CT>
__device__ __forceinline__ void tile_dot(const float* tile, const float* Xs, int ck, int logL, int row, int l, bool rotate,
                                         float (&acc)[CT]) {
  const int steps = (ck + (1 << logL) - 1) >> logL;
  int k = rotate ? row % steps : 0;
  const float* d = tile + row * ck;
#pragma unroll 4
  for (int i = 0; i < steps; ++i) {
    const int j = l + (k << logL);
    if (j < ck) {
      const float x = d[j];
#pragma unroll
      for (int n = 0; n < CT; ++n) acc[n] = fmaf(x, Xs[j * CT + n], acc[n]);
    }
    k = k + 1 == steps ? 0 : k + 1;
  }
  for (int m = (1 << logL) >> 1; m >= 1; m >>= 1) {
#pragma unroll
    for (int n = 0; n < CT; ++n) acc[n] += __shfl_xor(acc[n], m);
  }
}

// g += column j of the tile times the rows es[row][CT], rows sub, sub + nsub, ...
template <int CT>
__device__ __forceinline__ void tile_grad(const float* tile, const float* es, int nrow, int ck, int j, int sub, int nsub,
                                          float (&g)[CT]) {
#pragma unroll 4
  for (int r = sub; r < nrow; r += nsub) {
    const float x = tile[r * ck + j];
#pragma unroll
    for (int n = 0; n < CT; ++n) g[n] = fmaf(x, es[r * CT + n], g[n]);
  }
}

// The threads' column sums added in order of `sub` and stored as the workgroup's partial block.
template <int CT>
__device__ __forceinline__ void tile_grad_store(float* lds, const float (&g)[CT], int ck, int nsub, float* partial) {
  __syncthreads();
#pragma unroll
  for (int n = 0; n < CT; ++n) lds[threadIdx.x * CT + n] = g[n];
  __syncthreads();
  for (int o = threadIdx.x; o < ck * CT; o += kBlock) {
    const int j = o / CT, n = o - j * CT;
    float s = 0.0f;
    for (int q = 0; q < nsub; ++q) s += lds[(q * ck + j) * CT + n];
    partial[(int64_t)j * kNarrowCT + n] = s;
  }
}

template <int CT, bool AL>
__global__ __launch_bounds__(kBlock, 4) void prod_tile_kernel(TileMulti m) {
  extern __shared__ v4f tile_lds4[];
  float* tile = reinterpret_cast<float*>(tile_lds4);
  float* Xs = tile + kTileFloats;
  int q = 0;
  while (q + 1 < m.n && (int)blockIdx.x >= m.first[q + 1]) ++q;
  const TilePart a = m.a[q];
  const int bid = (int)blockIdx.x - m.first[q], nb = m.first[q + 1] - m.first[q];
  stage_operand<CT>(a.X, a.ldx, a.col0, a.ncols, a.colmap, a.ck, Xs);
  const int Rt = 1 << a.logR, logL = 8 - a.logR;
  const int row = (int)threadIdx.x >> logL, l = (int)threadIdx.x & ((1 << logL) - 1);
  const bool rotate = ((a.ck >> logL) & 1) == 0;
  const int64_t stride = (int64_t)nb * Rt;
  v4f v[kTileV];
  int64_t i0 = (int64_t)bid * Rt;
  if (i0 < a.rows) tile_load<AL, false>(a.D + i0 * a.ck, (int)min((int64_t)Rt, a.rows - i0) * a.ck, v);
  for (; i0 < a.rows; i0 += stride) {
    const int nrow = (int)min((int64_t)Rt, a.rows - i0);
    tile_put(tile, a.D + i0 * a.ck, nrow * a.ck, v);
    __syncthreads();
    const int64_t in = i0 + stride;
    if (in < a.rows) tile_load<AL, false>(a.D + in * a.ck, (int)min((int64_t)Rt, a.rows - in) * a.ck, v);
    float acc[CT];
#pragma unroll
    for (int n = 0; n < CT; ++n) acc[n] = 0.0f;
    tile_dot<CT>(tile, Xs, a.ck, logL, row, l, rotate, acc);   // (rows beyond nrow: stale LDS values, not stored)
    if (l == 0 && row < nrow) {
      float* o = a.out + (i0 + row) * a.ldo + a.col0;
#pragma unroll
      for (int n = 0; n < CT; ++n)
        if (n < a.ncols) o[n] = acc[n];
    }
    __syncthreads();
  }
}

// Residual and loss of one row and column (MODE 1 linear, 2 logistic; 0: the product itself).
template <int MODE>
__device__ __forceinline__ float residual(float z, float y, float& loss) {
  if constexpr (MODE == 1) {
    const float r = z - y;
    loss = fmaf(r, r, loss);
    return r;
  } else if constexpr (MODE == 2) {
    return logistic_residual(z, y, loss);
  }
  return z;
}

// Loss of this workgroup: butterfly inside each wavefront, then the wavefronts in order.
template <int CT>
__device__ __forceinline__ void store_loss(const float (&loss)[CT], float (*lsum)[CT], float* partial) {
#pragma unroll
  for (int n = 0; n < CT; ++n) {
    float s = loss[n];
    for (int m = kWave / 2; m >= 1; m >>= 1) s += __shfl_xor(s, m);
    if (threadIdx.x % kWave == 0) lsum[threadIdx.x / kWave][n] = s;
  }
  __syncthreads();
  if (threadIdx.x < CT) {
    float s = 0.0f;
    for (int w = 0; w < kBlock / kWave; ++w) s += lsum[w][threadIdx.x];
    partial[(int64_t)blockIdx.x * kNarrowCT + threadIdx.x] = s;
  }
}

// Assembly without an identity source (every table is joined): a thread takes ROWS rows, 256 apart, with the row numbers and
// then the gathered values of all of them in flight.  1,000,000 rows over two tables with the logistic residual: 8
// microseconds (four rows a thread leave half of the wavefront slots empty: 0.7 more), of which 3 are its bytes; the rest is
// the chain row number -> value -> store of a kernel this short.
template <int CT, int MODE, int ROWS>
__global__ __launch_bounds__(kBlock) void asm_gather_kernel(LmmArgs a) {
  float loss_local[CT];
#pragma unroll
  for (int n = 0; n < CT; ++n) loss_local[n] = 0.0f;
  constexpr int64_t step = (int64_t)kBlock * ROWS;
  for (int64_t base = (int64_t)blockIdx.x * step + threadIdx.x; base < a.r_out + threadIdx.x; base += (int64_t)gridDim.x * step) {
    float z[ROWS][CT], y[ROWS];
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
      const int64_t i = base + u * kBlock;
#pragma unroll
      for (int n = 0; n < CT; ++n) z[u][n] = 0.0f;
      y[u] = 0.0f;
      if constexpr (MODE != 0) y[u] = i < a.r_out ? a.y[i] : 0.0f;
    }
    for (int s0 = 0; s0 < a.g.n; s0 += 2) {
      int j[2][ROWS];
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
          const int64_t i = base + u * kBlock;
          j[h][u] = -1;
          if (s0 + h < a.g.n && i < a.r_out)
            j[h][u] = a.g.idx[s0 + h] != nullptr ? (int)a.g.idx[s0 + h][i] : (i < a.g.rows[s0 + h] ? (int)i : -1);
        }
      float p[2][ROWS][CT];
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int u = 0; u < ROWS; ++u)
#pragma unroll
          for (int n = 0; n < CT; ++n)
            p[h][u][n] = (j[h][u] >= 0 && n < a.ncols) ? a.g.P[s0 + h][(int64_t)j[h][u] * a.g.ldp + a.col0 + n] : 0.0f;
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int u = 0; u < ROWS; ++u)
#pragma unroll
          for (int n = 0; n < CT; ++n) z[u][n] += p[h][u][n];
    }
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
      const int64_t i = base + u * kBlock;
      if (i >= a.r_out) break;
#pragma unroll
      for (int n = 0; n < CT; ++n) {
        if (n >= a.ncols) break;
        const float r = residual<MODE>(z[u][n], y[u], loss_local[n]);
        float* op = a.out + i * a.ldo + a.col0 + n;
        if (a.nt_out) __builtin_nontemporal_store(r, op);
        else *op = r;
      }
    }
  }
  if constexpr (MODE != 0) {
    __shared__ float lsum[kBlock / kWave][CT];
    store_loss<CT>(loss_local, lsum, a.loss_partial);
  }
}

// MODE 0: store the product.  1: linear residual z - y.  2: logistic residual sigmoid(z) - y.  FUSEG: this workgroup's
// share of D^T e as well (at most 256 columns).  The first lane of a row owns its target row.
template <int CT, int MODE, bool FUSEG, bool AL, bool NT>
__global__ __launch_bounds__(kBlock, 4) void asm_tile_kernel(LmmArgs a, int logR) {
  extern __shared__ v4f tile_lds4[];
  float* tile = reinterpret_cast<float*>(tile_lds4);
  float* es = tile + kTileFloats;                        // [Rt][CT] residuals of the tile
  float* Xs = es + kBlock * CT;
  const int ck = a.ck;
  stage_operand<CT>(a.X, a.ldx, a.col0, a.ncols, a.colmap, ck, Xs);
  const int Rt = 1 << logR, logL = 8 - logR;
  const int tid = threadIdx.x, row = tid >> logL, l = tid & ((1 << logL) - 1);
  const bool rotate = ((ck >> logL) & 1) == 0;
  const int nsub = FUSEG ? kBlock / ck : 1;
  const int gsub = FUSEG ? tid / ck : 0, gj = FUSEG ? tid - gsub * ck : 0;
  const int64_t stride = (int64_t)gridDim.x * Rt;
  float g[CT], loss_local[CT];
#pragma unroll
  for (int n = 0; n < CT; ++n) g[n] = loss_local[n] = 0.0f;
  auto table_rows = [&](int64_t i) { return (int)max((int64_t)0, min((int64_t)Rt, a.d_rows - i)); };   // rows of D in the tile
  auto row_of = [&](int s, int64_t i) {
    if (a.g.idx[s] != nullptr) return (int)a.g.idx[s][i];
    return i < a.g.rows[s] ? (int)i : -1;
  };
  // Requests run one tile ahead, row numbers two: when a tile starts, everything it uses was asked for a tile ago.
  v4f v[kTileV];
  int jn[kTileGather];
  float pn[kTileGather][CT], yn = 0.0f;
  auto load_index = [&](int64_t i) {
#pragma unroll
    for (int s = 0; s < kTileGather; ++s) jn[s] = (s < a.g.n && l == 0 && i < a.r_out) ? row_of(s, i) : -1;
  };
  auto gather = [&](int64_t i) {
#pragma unroll
    for (int s = 0; s < kTileGather; ++s) {
      const float* p = jn[s] >= 0 ? a.g.P[s] + (int64_t)jn[s] * a.g.ldp + a.col0 : nullptr;
#pragma unroll
      for (int n = 0; n < CT; ++n) pn[s][n] = (jn[s] >= 0 && n < a.ncols) ? p[n] : 0.0f;
    }
    if constexpr (MODE != 0) yn = (l == 0 && i < a.r_out) ? a.y[i] : 0.0f;
  };
  int64_t i0 = (int64_t)blockIdx.x * Rt;
  load_index(i0 + row);
  tile_load<AL, NT>(a.D + i0 * ck, i0 < a.r_out ? table_rows(i0) * ck : 0, v);
  gather(i0 + row);
  load_index(i0 + stride + row);
  for (; i0 < a.r_out; i0 += stride) {
    const int64_t i = i0 + row;
    const bool own = l == 0 && i < a.r_out;
    const int drow = table_rows(i0);
    float gsum[CT];
#pragma unroll
    for (int n = 0; n < CT; ++n) {
      gsum[n] = 0.0f;
#pragma unroll
      for (int s = 0; s < kTileGather; ++s) gsum[n] += pn[s][n];
    }
    const float yi = yn;
    if (own) {
      for (int s = kTileGather; s < a.g.n; ++s) {
        const int j = row_of(s, i);
        if (j >= 0) {
          const float* p = a.g.P[s] + (int64_t)j * a.g.ldp + a.col0;
#pragma unroll
          for (int n = 0; n < CT; ++n)
            if (n < a.ncols) gsum[n] += p[n];
        }
      }
    }
    tile_put(tile, a.D + i0 * ck, drow * ck, v);
    __syncthreads();
    const int64_t in = i0 + stride;
    gather(in + row);
    load_index(in + stride + row);
    if (in < a.r_out) tile_load<AL, NT>(a.D + in * ck, table_rows(in) * ck, v);
    float z[CT];
#pragma unroll
    for (int n = 0; n < CT; ++n) z[n] = 0.0f;
    tile_dot<CT>(tile, Xs, ck, logL, row, l, rotate, z);
    if (row >= drow) {
#pragma unroll
      for (int n = 0; n < CT; ++n) z[n] = 0.0f;
    }
    if (l == 0) {
#pragma unroll
      for (int n = 0; n < CT; ++n) {
        float r = 0.0f;
        if (own && n < a.ncols) {
          r = residual<MODE>(z[n] + gsum[n], yi, loss_local[n]);
          float* op = a.out + i * a.ldo + a.col0 + n;
          if (a.nt_out) __builtin_nontemporal_store(r, op);
          else *op = r;
        }
        if constexpr (FUSEG) es[row * CT + n] = r;
      }
    }
    __syncthreads();
    if constexpr (FUSEG) {
      if (gsub < nsub) tile_grad<CT>(tile, es, drow, ck, gj, gsub, nsub, g);
      __syncthreads();
    }
  }
  if constexpr (MODE != 0) {
    __shared__ float lsum[kBlock / kWave][CT];
    store_loss<CT>(loss_local, lsum, a.loss_partial);
  }
  if constexpr (FUSEG) tile_grad_store<CT>(tile, g, ck, nsub, a.grad_partial + (int64_t)blockIdx.x * ck * kNarrowCT);
}

// The squared norm of every centroid, by every workgroup of a kernel: while C is a few kilobytes, a launch for it takes as
// long as this.  Added in the order of centroid_norm_kernel, so that both ways give the same bits.  red: k x kBlock.
template <int KC>
__device__ __forceinline__ void centroid_norms(const float* __restrict__ C, int ldc, int c_T, int k, float* red, float* cns) {
  const int tid = threadIdx.x;
  float s[KC];
#pragma unroll
  for (int n = 0; n < KC; ++n) s[n] = 0.0f;
  for (int t = tid; t < c_T; t += kBlock) {
#pragma unroll
    for (int n = 0; n < KC; ++n) {
      const float v = n < k ? C[(int64_t)t * ldc + n] : 0.0f;
      s[n] = fmaf(v, v, s[n]);
    }
  }
#pragma unroll
  for (int n = 0; n < KC; ++n)
    if (n < k) red[n * kBlock + tid] = s[n];
  __syncthreads();
  static_assert(kBlock == 4 * kWave, "two steps of the tree before a wavefront's");
  const int lane = tid % kWave;
  for (int n = tid / kWave; n < KC; n += kBlock / kWave) {        // the tree of that kernel, a wavefront per centroid
    float v = 0.0f;
    if (n < k) {
      const float* r = red + n * kBlock + lane;
      v = (r[0] + r[2 * kWave]) + (r[kWave] + r[3 * kWave]);
      for (int w = kWave / 2; w > 0; w >>= 1) v += __shfl_down(v, w);
    }
    if (lane == 0) cns[n] = v;
  }
  __syncthreads();
}

// KMeans (at most 16 centroids): the assembly of T C, the nearest centroid of every row and the identity source's share
// of the per-cluster sums in one pass over its tiles.  Neither T C nor the 0/1 assignment matrix is written: the rows'
// products stay in registers (KC of them, KC = k rounded up to a multiple of four), and a thread owns a column of the
// tile and every nsub-th of its rows and adds each value to its sum for the row's cluster, kept in LDS.
// 1,000,000 x 20 joined with 100,000 rows, 10 centroids: 60 microseconds, 2 of them the norms; T C (65), the assignment (21)
// and S^T A (38) by themselves took 124.  Of the 60, 8 are the gathers, 8 the cluster sums and most of the rest the operand's
// way through LDS to every lane (smaller tiles, which spread a row over lanes, measure 3 to 26 % slower).
// (Tables of at most 20 columns over many rows take kernels_kmeans.hip: 46.)
// cn: the norms of the centroids, or NULL.
template <int KC, bool AL>
__global__ __launch_bounds__(kBlock, 4) void kmeans_tile_kernel(LmmArgs a, const float* __restrict__ cn, int c_T, int32_t* __restrict__ assign,
                                                             int32_t* __restrict__ counts_partial, float* __restrict__ sum_partial,
                                                             int logR) {
  extern __shared__ v4f tile_lds4[];
  const int ck = a.ck, k = a.ncols;
  float* tile = reinterpret_cast<float*>(tile_lds4);
  float* Xs = tile + kTileFloats;                        // [ck][KC]
  float* acc = Xs + ck * KC;                             // [k][kBlock]
  float* cns = acc + k * kBlock;                         // [KC]
  int* as = reinterpret_cast<int*>(cns + KC);            // [kBlock] cluster of every row of the tile
  int* hist = as + kBlock;                               // [k]
  const int tid = threadIdx.x;
  for (int e = tid; e < ck * KC; e += kBlock) {
    const int j = e / KC, n = e - j * KC;
    const int t = a.colmap[j];
    Xs[e] = (t >= 0 && n < k) ? a.X[(int64_t)t * a.ldx + n] : 0.0f;
  }
  if (tid < k) hist[tid] = 0;
  if (cn == nullptr) centroid_norms<KC>(a.X, a.ldx, c_T, k, acc, cns);      // (acc is scratch until here)
  else if (tid < KC) cns[tid] = tid < k ? cn[tid] : 0.0f;
  for (int e = tid; e < k * kBlock; e += kBlock) acc[e] = 0.0f;
  const int Rt = 1 << logR, logL = 8 - logR;
  const int row = tid >> logL, l = tid & ((1 << logL) - 1);
  const bool rotate = ((ck >> logL) & 1) == 0;
  const int steps = (ck + (1 << logL) - 1) >> logL;
  const int nsub = kBlock / ck, gsub = tid / ck, gj = tid - gsub * ck;
  const int64_t stride = (int64_t)gridDim.x * Rt;
  auto table_rows = [&](int64_t i) { return (int)max((int64_t)0, min((int64_t)Rt, a.d_rows - i)); };
  auto row_of = [&](int s, int64_t i) {
    if (a.g.idx[s] != nullptr) return (int)a.g.idx[s][i];
    return i < a.g.rows[s] ? (int)i : -1;
  };
  v4f v[kTileV];
  int jn[kTileGather];
  auto load_index = [&](int64_t i) {
#pragma unroll
    for (int s = 0; s < kTileGather; ++s) jn[s] = (s < a.g.n && l == 0 && i < a.r_out) ? row_of(s, i) : -1;
  };
  int64_t i0 = (int64_t)blockIdx.x * Rt;
  load_index(i0 + row);
  tile_load<AL, false>(a.D + i0 * ck, i0 < a.r_out ? table_rows(i0) * ck : 0, v);
  for (; i0 < a.r_out; i0 += stride) {
    const int64_t i = i0 + row;
    const bool own = l == 0 && i < a.r_out;
    const int drow = table_rows(i0);
    // gathered products: the first source's travel while the tile is multiplied
    float g[KC], g0[KC];
    auto product_row = [&](int s, int j, float (&t)[KC]) {
      const float* p = a.g.P[s] + (int64_t)max(j, 0) * a.g.ldp;   // a row of k floats: whole float4s, float2s or neither
      if (k % 4 == 0) {
#pragma unroll
        for (int n = 0; n < KC; n += 4) {
          const v4f w = j >= 0 ? *reinterpret_cast<const v4f*>(p + n) : (v4f){0.0f, 0.0f, 0.0f, 0.0f};
          t[n] = w[0]; t[n + 1] = w[1]; t[n + 2] = w[2]; t[n + 3] = w[3];
        }
      } else if (k % 2 == 0) {
#pragma unroll
        for (int n = 0; n < KC; n += 2) {
          const float2 w = j >= 0 && n < k ? *reinterpret_cast<const float2*>(p + n) : make_float2(0.0f, 0.0f);
          t[n] = w.x; t[n + 1] = w.y;
        }
      } else {
#pragma unroll
        for (int n = 0; n < KC; ++n) t[n] = j >= 0 && n < k ? p[n] : 0.0f;
      }
    };
#pragma unroll
    for (int n = 0; n < KC; ++n) g[n] = 0.0f;
#pragma unroll
    for (int s = 1; s < kTileGather; ++s) {
      if (s < a.g.n) {
        product_row(s, jn[s], g0);
#pragma unroll
        for (int n = 0; n < KC; ++n) g[n] += g0[n];
      }
    }
    for (int s = kTileGather; s < a.g.n; ++s) {
      product_row(s, own ? row_of(s, i) : -1, g0);
#pragma unroll
      for (int n = 0; n < KC; ++n) g[n] += g0[n];
    }
    product_row(0, a.g.n > 0 ? jn[0] : -1, g0);
    tile_put(tile, a.D + i0 * ck, drow * ck, v);
    __syncthreads();
    const int64_t in = i0 + stride;
    load_index(in + row);
    if (in < a.r_out) tile_load<AL, false>(a.D + in * ck, table_rows(in) * ck, v);
    float z[KC];
#pragma unroll
    for (int n = 0; n < KC; ++n) z[n] = 0.0f;
    {
      int kk = rotate ? row % steps : 0;
      const float* d = tile + row * ck;
#pragma unroll 4
      for (int it = 0; it < steps; ++it) {
        const int j = l + (kk << logL);
        if (j < ck) {
          const float x = d[j];
#pragma unroll
          for (int n = 0; n < KC; n += 4) {
            const v4f w = *reinterpret_cast<const v4f*>(Xs + j * KC + n);
            z[n] = fmaf(x, w[0], z[n]); z[n + 1] = fmaf(x, w[1], z[n + 1]);
            z[n + 2] = fmaf(x, w[2], z[n + 2]); z[n + 3] = fmaf(x, w[3], z[n + 3]);
          }
        }
        kk = kk + 1 == steps ? 0 : kk + 1;
      }
      for (int m = (1 << logL) >> 1; m >= 1; m >>= 1) {
#pragma unroll
        for (int n = 0; n < KC; ++n) z[n] += __shfl_xor(z[n], m);
      }
    }
    int best = -1;
    if (own) {
      const bool has = row < drow;
      best = 0;
      float bv = cns[0] - 2.0f * ((has ? z[0] : 0.0f) + (g0[0] + g[0]));
#pragma unroll
      for (int n = 1; n < KC; ++n) {
        const float u = cns[n] - 2.0f * ((has ? z[n] : 0.0f) + (g0[n] + g[n]));
        if (n < k && u < bv) { bv = u; best = n; }       // strict: the first of equal minima stays
      }
      assign[i] = best;
    }
    if (l == 0) as[row] = best;
    // cluster sizes: one count per wavefront and centroid instead of one atomic per row
    for (int n = 0; n < k; ++n) {
      const unsigned long long m = __ballot(best == n);
      if (tid % kWave == 0 && m != 0) atomicAdd(&hist[n], __popcll(m));
    }
    __syncthreads();
    if (gsub < nsub) {
      // four rows at a time: their sums are read together, and a row of the same cluster as an earlier one of the four
      // takes over that one's result (one at a time, the chain read - add - write through LDS is most of the pass)
      for (int r = gsub; r < drow; r += 4 * nsub) {
        int c[4];
        float x[4], u[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int q = r + e * nsub;
          c[e] = q < drow ? as[q] : -1;
          x[e] = q < drow ? tile[q * ck + gj] : 0.0f;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) u[e] = acc[max(c[e], 0) * kBlock + tid];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
#pragma unroll
          for (int f = 0; f < e; ++f) u[e] = c[f] == c[e] ? u[f] : u[e];
          u[e] += x[e];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (c[e] >= 0) acc[c[e] * kBlock + tid] = u[e];
      }
    }
    __syncthreads();
  }
  __syncthreads();
  for (int o = tid; o < ck * k; o += kBlock) {
    const int j = o / k, c = o - j * k;
    float s = 0.0f;
    for (int q = 0; q < nsub; ++q) s += acc[c * kBlock + q * ck + j];
    sum_partial[((int64_t)blockIdx.x * ck + j) * k + c] = s;
  }
  for (int c = tid; c < k; c += kBlock) counts_partial[(size_t)blockIdx.x * k + c] = hist[c];
}

template <int CT, bool AL>
__global__ __launch_bounds__(kBlock, 4) void colred_tile_kernel(TileMulti m) {
  extern __shared__ v4f tile_lds4[];
  float* tile = reinterpret_cast<float*>(tile_lds4);
  float* es = tile + kTileFloats;
  int q = 0;
  while (q + 1 < m.n && (int)blockIdx.x >= m.first[q + 1]) ++q;
  const TilePart a = m.a[q];
  const int bid = (int)blockIdx.x - m.first[q], nb = m.first[q + 1] - m.first[q];
  const int Rt = 1 << a.logR;
  const int nsub = kBlock / a.ck, gsub = (int)threadIdx.x / a.ck, gj = (int)threadIdx.x - gsub * a.ck;
  const int64_t stride = (int64_t)nb * Rt;
  float g[CT];
#pragma unroll
  for (int n = 0; n < CT; ++n) g[n] = 0.0f;
  v4f v[kTileV];
  float zr[CT];                                          // operand row of this thread (Rt <= kBlock)
  auto load = [&](int64_t i) {
    tile_load<AL, false>(a.D + i * a.ck, (int)min((int64_t)Rt, a.rows - i) * a.ck, v);
#pragma unroll
    for (int n = 0; n < CT; ++n)
      zr[n] = ((int)threadIdx.x < Rt && i + threadIdx.x < a.rows && n < a.ncols) ? a.X[(i + threadIdx.x) * a.ldx + a.col0 + n] : 0.0f;
  };
  int64_t i0 = (int64_t)bid * Rt;
  if (i0 < a.rows) load(i0);
  for (; i0 < a.rows; i0 += stride) {
    const int nrow = (int)min((int64_t)Rt, a.rows - i0);
    tile_put(tile, a.D + i0 * a.ck, nrow * a.ck, v);
    if ((int)threadIdx.x < Rt) {
#pragma unroll
      for (int n = 0; n < CT; ++n) es[threadIdx.x * CT + n] = zr[n];
    }
    __syncthreads();
    if (i0 + stride < a.rows) load(i0 + stride);
    if (gsub < nsub) tile_grad<CT>(tile, es, nrow, a.ck, gj, gsub, nsub, g);
    __syncthreads();
  }
  tile_grad_store<CT>(tile, g, a.ck, nsub, a.out + (int64_t)bid * a.ck * kNarrowCT);
}

// Rows per tile (a power of two of 4 to 256): as many as fit, fewer (not below 64) where the table would not give 512
// tiles.
int tile_logR(int64_t rows, int ck) {
  int logR = 8;
  while (logR > 2 && (int64_t)ck << logR > kTileFloats) --logR;
  while (logR > 6 && rows >> logR < 512) --logR;
  return logR;
}

// A launch reads all its tables as float4 or, when one of them does not start on one, all of them float by float.
bool all_aligned(const TileMulti& m) {
  for (int q = 0; q < m.n; ++q)
    if (reinterpret_cast<uintptr_t>(m.a[q].D) % 16 != 0) return false;
  return true;
}

#define ILARGI_TILE(kernel, ct, al, grid, lds, st, ...)                                            \
  do {                                                                                             \
    if (ct == 1 && al) kernel<1, true><<<grid, kBlock, lds, st>>>(__VA_ARGS__);                    \
    else if (ct == 1) kernel<1, false><<<grid, kBlock, lds, st>>>(__VA_ARGS__);                    \
    else if (ct == 2 && al) kernel<2, true><<<grid, kBlock, lds, st>>>(__VA_ARGS__);               \
    else if (ct == 2) kernel<2, false><<<grid, kBlock, lds, st>>>(__VA_ARGS__);                    \
    else if (al) kernel<4, true><<<grid, kBlock, lds, st>>>(__VA_ARGS__);                          \
    else kernel<4, false><<<grid, kBlock, lds, st>>>(__VA_ARGS__);                                 \
  } while (0)

constexpr int kTileMaxCols = kTileFloats / 4;            // four rows of so many columns fill a tile

}  // namespace

// Rows of whole float4s are left to the kernels that read them in place: above 256 columns (the streaming product kernel
// has the shorter ones) the tile costs more than it gives, 100,000 x 800: 59 microseconds in place, 81 through tiles.
bool prod_tile_supported(const LmmArgs& a, int vec) {
  if (vec == 4 && a.ck > 256) return false;
  return a.D != nullptr && a.g.n == 0 && a.ncols >= 1 && a.ncols <= kNarrowCT && a.r_out > 0 && a.ck >= 1 && a.ck <= kTileMaxCols;
}

// The products of n <= kTileParts sources with the same operand columns in one launch.
hipError_t launch_prod_tile(const LmmArgs* a, int n, hipStream_t st) {
  if (n < 1 || n > kTileParts) return hipErrorInvalidValue;
  TileMulti m;
  memset(&m, 0, sizeof(m));
  m.n = n;
  int64_t tiles[kTileParts], total = 0;
  int ckmax = 1;
  for (int q = 0; q < n; ++q) {
    if (!prod_tile_supported(a[q], 1) || a[q].ncols != a[0].ncols) return hipErrorInvalidValue;
    TilePart& t = m.a[q];
    t.D = a[q].D; t.ck = a[q].ck; t.rows = std::min(a[q].r_out, a[q].d_rows); t.colmap = a[q].colmap;
    t.X = a[q].X; t.ldx = a[q].ldx; t.col0 = a[q].col0; t.ncols = a[q].ncols; t.out = a[q].out; t.ldo = a[q].ldo;
    t.logR = tile_logR(t.rows, t.ck);
    tiles[q] = (t.rows + (1 << t.logR) - 1) >> t.logR;
    total += tiles[q];
    ckmax = std::max(ckmax, t.ck);
  }
  const int64_t cap = 2048;
  for (int q = 0; q < n; ++q)
    m.first[q + 1] = m.first[q] + (int)std::max<int64_t>(1, total > cap ? tiles[q] * cap / total : tiles[q]);
  const int ct = a[0].ncols <= 1 ? 1 : (a[0].ncols <= 2 ? 2 : 4);
  const size_t lds = sizeof(float) * (kTileFloats + (size_t)ckmax * ct);
  ILARGI_TILE(prod_tile_kernel, ct, all_aligned(m), m.first[n], lds, st, m);
  return hipGetLastError();
}

// One operand column over rows of float4 or float2 is where the kernel that reads such rows in place, 2^k lanes to a row,
// keeps up: the tiles win as far as its lanes idle and the table is long enough to fill the chip with them.  Time through
// tiles over time in place at 300,000 / 2,000,000 rows joined with 8 columns:
//   an iteration, rows of float4     36 and 40 columns (9 or 10 of 16 lanes at work) 1.06 / 0.93, 44 to 60 1.13 / 1.10,
//                                    68 to 80 (17 to 20 of 32) 1.08 / 0.95, 84 to 92 (tiles of 32 rows) 1.28 / 1.25
//                 rows of float2     18 (9 of 16) 0.97 / 0.79, 22 to 30 1.03 / 0.91 (700,000: 1.04 to 1.08), 34 to 42
//                                    (17 to 21 of 32) 0.97 / 0.76, 46 1.02 / 0.88;  18 columns of 30,000 rows 1.10
//   a product, rows of float4        68 to 80 0.91 / 0.81, 84 to 92 1.08 / 0.98;  rows of float2  34 to 46 0.82 / 0.61
// With several operand columns the tiles win everywhere (300,000 rows, two models: 36 columns 0.80, 46 0.82, 52 0.86).
// (Iterations over at most 24 columns take kernels_asm_row.hip where that is the faster one.)
bool asm_tile_supported(const LmmArgs& a, int vec, bool fuseg) {
  if (a.ncols < 1 || a.ncols > kNarrowCT || a.r_out <= 0) return false;
  if (a.D == nullptr) return !fuseg;
  if (a.ck < 1 || a.ck > (fuseg ? kBlock : kTileMaxCols)) return false;
  const int nvec = a.ck / vec;
  if (vec >= 2 && a.ncols == 1 && nvec >= 9) {
    const int lanes = 1 << ilog2_ceil(nvec);
    const bool million = a.r_out >= (1 << 20);
    if (nvec > kWave || (nvec >= 16 && 4 * nvec >= 3 * lanes)) return false;
    if (fuseg && vec == 4) return million && 8 * nvec <= 5 * lanes && a.ck <= 80;
    if (fuseg && nvec < 16) return million || (8 * nvec <= 5 * lanes && a.r_out >= 256 * 1024);
    if (fuseg) return a.r_out >= (16 * nvec <= 11 * lanes ? 256 * 1024 : 512 * 1024);
    if (vec == 4 && a.ck > 80 && !million) return false;
  }
  return vec != 4 || a.ck <= 256;
}

namespace {

// Rows of a thread of asm_gather_kernel: two fill more wavefront slots, four have more in flight.  Iterations of one logistic
// model, two rows / four, by target rows: one table 100,000 to 1,000,000 0.96 to 0.99, 1,500,000 and 2,000,000 1.02, 3,000,000
// 0.99, 5,000,000 and 10,000,000 1.00; several tables to 1,000,000 0.96 to 0.99, 1,500,000 1.02, 3,000,000 0.99, 5,000,000 1.01,
// 10,000,000 1.01 to 1.04.  Three models: one table 0.93 to 0.99 (10,000,000 1.01), several to 300,000 0.92 to 0.96, 500,000 1.01,
// 10,000,000 1.03 to 1.05; their products alone 1.05 from 500,000 on.
int gather_rows(const LmmArgs& a) {
  if (a.ncols > 1) return a.g.n > 1 && a.r_out >= 400000 ? 4 : 2;
  return a.r_out >= 1250000 && (a.g.n > 1 || a.r_out < 2500000) ? 4 : 2;
}

template <int CT, int MODE>
void launch_asm_gather(const LmmArgs& a, int rows, int grid, hipStream_t st) {
  if (rows == 2) asm_gather_kernel<CT, MODE, 2><<<grid, kBlock, 0, st>>>(a);
  else asm_gather_kernel<CT, MODE, 4><<<grid, kBlock, 0, st>>>(a);
}

}  // namespace

hipError_t launch_asm_tile(const LmmArgs& a, int mode, hipStream_t st, int* grid_out) {
  const bool fuseg = a.grad_partial != nullptr && mode != 0;
  if (!asm_tile_supported(a, 1, fuseg)) return hipErrorInvalidValue;
  if (a.D == nullptr) {
    const int rows = gather_rows(a);
    int64_t grid = (a.r_out + kBlock * rows - 1) / (kBlock * rows);
    if (grid > 4096) grid = 4096;
    if (grid_out) *grid_out = (int)grid;
#define ILARGI_GATHER(C)                                                                  \
  do {                                                                                    \
    if (mode == 0) launch_asm_gather<C, 0>(a, rows, (int)grid, st);                       \
    else if (mode == 1) launch_asm_gather<C, 1>(a, rows, (int)grid, st);                  \
    else launch_asm_gather<C, 2>(a, rows, (int)grid, st);                                 \
  } while (0)
    if (a.ncols <= 1) ILARGI_GATHER(1);
    else if (a.ncols <= 2) ILARGI_GATHER(2);
    else ILARGI_GATHER(4);
#undef ILARGI_GATHER
    return hipGetLastError();
  }
  const int logR = tile_logR(a.r_out, a.ck);
  int64_t grid = (a.r_out + (1 << logR) - 1) >> logR;
  const int64_t cap = fuseg ? kColredBlocks : 4096;
  if (grid > cap) {
    const int64_t per = (grid + cap - 1) / cap;
    grid = (grid + per - 1) / per;
  }
  if (grid_out) *grid_out = (int)grid;
  const int ct = a.ncols <= 1 ? 1 : (a.ncols <= 2 ? 2 : 4);
  const size_t lds = sizeof(float) * (kTileFloats + (size_t)(kBlock + a.ck) * ct);
#define ILARGI_ASM(C, AL, NT)                                                                                   \
  do {                                                                                                          \
    if (mode == 0) asm_tile_kernel<C, 0, false, AL, NT><<<(int)grid, kBlock, lds, st>>>(a, logR);               \
    else if (mode == 1 && fuseg) asm_tile_kernel<C, 1, true, AL, NT><<<(int)grid, kBlock, lds, st>>>(a, logR);  \
    else if (mode == 1) asm_tile_kernel<C, 1, false, AL, NT><<<(int)grid, kBlock, lds, st>>>(a, logR);          \
    else if (fuseg) asm_tile_kernel<C, 2, true, AL, NT><<<(int)grid, kBlock, lds, st>>>(a, logR);               \
    else asm_tile_kernel<C, 2, false, AL, NT><<<(int)grid, kBlock, lds, st>>>(a, logR);                         \
  } while (0)
#define ILARGI_ASM_CT(C)                       \
  do {                                         \
    if (!al) ILARGI_ASM(C, false, false);      \
    else if (a.nt_in) ILARGI_ASM(C, true, true); \
    else ILARGI_ASM(C, true, false);           \
  } while (0)
  const bool al = reinterpret_cast<uintptr_t>(a.D) % 16 == 0;
  if (ct == 1) ILARGI_ASM_CT(1);
  else if (ct == 2) ILARGI_ASM_CT(2);
  else ILARGI_ASM_CT(4);
#undef ILARGI_ASM_CT
#undef ILARGI_ASM
  return hipGetLastError();
}

bool colred_tile_supported(const ColredArgs& c) {
  return c.ck >= 1 && c.ck <= kBlock && c.ncols >= 1 && c.ncols <= kNarrowCT && c.rows > 0;
}

// Whether a table that shares its launch with no other goes through tiles (several always do: a launch costs more than any
// of the differences below).  Time of the tiles over that of the kernel that reads rows in place:
//   fewer than 65,536 rows                      20,000: 0.93 to 1.40
//   rows of float2, 300,000 / 3,000,000         one column: 10 columns of the table 1.12 / 1.06, 30 1.10 / 1.05, 98 0.92 / 0.92
//                                               two: 10 1.13 / 0.97, 46 1.01 / 0.81;  three: 10 1.07 / 0.89, 30 1.02 / 0.84
//                                               four: 10 0.91 / 0.55, 98 0.71 / 0.69
//   rows on any float, 300,000 / 3,000,000      one column: 3 1.12 / 1.32, 7 1.04 / 0.96, 13 1.01 / 0.67, 33 0.71 / 0.43
//                                               four: 3 1.01 / 0.87, 13 0.76 / 0.37, 199 0.64
bool colred_tile_pays(const ColredArgs& c) {
  if (c.rows < 65536) return false;
  const bool many = c.rows >= (1 << 20);
  if (c.ncols == 4) return true;
  if (c.vec == 1) return c.ck >= 12 || (many && c.ck >= 6);
  return c.ck * c.ncols >= 64 || (many && c.ncols >= 2 && c.ck >= 6);
}

// The column reduces of n <= kTileParts sources in one launch; nblocks[q] receives the number of partial blocks that
// source q leaves (at most kColredBlocks).
hipError_t launch_colred_tile(const ColredArgs* c, int n, int* nblocks, hipStream_t st) {
  if (n < 1 || n > kTileParts) return hipErrorInvalidValue;
  TileMulti m;
  memset(&m, 0, sizeof(m));
  m.n = n;
  int64_t tiles[kTileParts], total = 0;
  for (int q = 0; q < n; ++q) {
    if (!colred_tile_supported(c[q]) || c[q].ncols != c[0].ncols) return hipErrorInvalidValue;
    TilePart& t = m.a[q];
    t.D = c[q].D; t.ck = c[q].ck; t.rows = c[q].rows;
    t.X = c[q].Z; t.ldx = c[q].ldz; t.col0 = c[q].col0; t.ncols = c[q].ncols; t.out = c[q].partial;
    t.logR = tile_logR(t.rows, t.ck);
    tiles[q] = (t.rows + (1 << t.logR) - 1) >> t.logR;
    total += tiles[q];
  }
  for (int q = 0; q < n; ++q) {
    nblocks[q] = (int)std::max<int64_t>(1, total > kColredBlocks ? tiles[q] * kColredBlocks / total : tiles[q]);
    m.first[q + 1] = m.first[q] + nblocks[q];
  }
  // (one operand column takes the kernel for two, as a kernel of its own measures slower: 3,000,000 x 50 149 microseconds
  // and 112)
  const int ct = c[0].ncols <= 2 ? 2 : 4;
  const size_t lds = sizeof(float) * (kTileFloats + (size_t)kBlock * ct);
  const bool al = all_aligned(m);
  if (ct == 2 && al) colred_tile_kernel<2, true><<<m.first[n], kBlock, lds, st>>>(m);
  else if (ct == 2) colred_tile_kernel<2, false><<<m.first[n], kBlock, lds, st>>>(m);
  else if (al) colred_tile_kernel<4, true><<<m.first[n], kBlock, lds, st>>>(m);
  else colred_tile_kernel<4, false><<<m.first[n], kBlock, lds, st>>>(m);
  return hipGetLastError();
}

// k <= 16 centroids, an identity source of at most kBlock columns.
bool kmeans_tile_supported(int ck, int k) { return ck >= 1 && ck <= kBlock && k >= 1 && k <= kKmeansTileK; }

int kmeans_tile_grid(const LmmArgs& a, int* logR) {
  *logR = tile_logR(a.r_out, a.ck);
  int64_t grid = (a.r_out + (1 << *logR) - 1) >> *logR;
  if (grid > kColredBlocks) {
    const int64_t per = (grid + kColredBlocks - 1) / kColredBlocks;
    grid = (grid + per - 1) / per;
  }
  return (int)grid;
}

// counts_partial: grid x k integers, sum_partial: grid x ck x k floats.
hipError_t launch_kmeans_tile(const LmmArgs& a, const float* cn, int64_t c_T, int32_t* assign, int32_t* counts_partial, float* sum_partial,
                              int grid, int logR, hipStream_t st) {
  if (!kmeans_tile_supported(a.ck, a.ncols) || a.D == nullptr || a.r_out <= 0) return hipErrorInvalidValue;
  const int kc = (a.ncols + 3) / 4 * 4;
  const size_t lds = sizeof(float) * (kTileFloats + (size_t)a.ck * kc + (size_t)a.ncols * kBlock + kc + kBlock + a.ncols);
  const bool al = reinterpret_cast<uintptr_t>(a.D) % 16 == 0;
#define ILARGI_KMEANS(C)                                                                                               \
  do {                                                                                                                 \
    if (al) kmeans_tile_kernel<C, true><<<grid, kBlock, lds, st>>>(a, cn, (int)c_T, assign, counts_partial, sum_partial, logR);  \
    else kmeans_tile_kernel<C, false><<<grid, kBlock, lds, st>>>(a, cn, (int)c_T, assign, counts_partial, sum_partial, logR);    \
  } while (0)
  if (kc == 4) ILARGI_KMEANS(4);
  else if (kc == 8) ILARGI_KMEANS(8);
  else if (kc == 12) ILARGI_KMEANS(12);
  else ILARGI_KMEANS(16);
#undef ILARGI_KMEANS
  return hipGetLastError();
}

}  // namespace ilargi
