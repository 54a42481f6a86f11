// Join-gather baseline: the materialized target table  T = sum_k I_k D_k M_k^T  (Sec. 2.2 with X = I).
// Every cell is the float32 sum, in source order and starting from +0.0, of the source cells mapped to it,
// which makes the table reproducible bit for bit.
#include "ilargi_internal.h"

namespace ilargi {

namespace {

// General form: a workgroup builds a tile of whole target rows in LDS, one source after the other, and writes it out
// as one contiguous run of float4.  Bound by the write of T.  The rows are built in LDS because a schema whose column
// blocks start anywhere (10 + 50 + 100 + 40 columns) leaves no aligned float4 a lane could move from a source to T by
// itself: every source is read in the widest vectors its own rows allow, and the stores fill whole 128-byte lines
// whatever the alignment of the column blocks.  The tile is small enough for eight workgroups on a compute unit, which
// overlap one another's gathers and stores (20 KiB; 10 KiB measures 18 % slower, 40 KiB 3 %; non-temporal stores 9 %
// faster than plain ones).  5,000,000 x 200 from tables of 10, 50, 100 and 40 columns: 1280 microseconds (a lane per
// target column, as before: 2726); 3,400,000 x 96 from two overlapping tables: 400 (1333).  What is left in the first
// is the gathered rows, 2.6 GB of lines beside the 4 GB written.
constexpr int kTileU = 4;      // vectors in flight per lane

template <int V> struct TileVec;
template <> struct TileVec<1> { typedef float T; };
template <> struct TileVec<2> { typedef float T __attribute__((ext_vector_type(2))); };
template <> struct TileVec<4> { typedef float T __attribute__((ext_vector_type(4))); };

// Source s into the tile.  MAP: the target column of every source column is looked up (V = 1), else the columns form
// the block [c0, c0 + ck).  Without `add` the source is the only feeder of its columns and writes their cells.
template <int V, bool MAP>
__device__ void tile_source(const MatTileSource& s, float* tile, const int* jrow, int nrow, int c_T, bool add) {
  typedef typename TileVec<V>::T VT;
  const unsigned total = (unsigned)nrow * s.nv;
  const bool whole = (c_T % V == 0) && (s.c0 % V == 0);    // the tile's vectors are aligned as well
  for (unsigned e0 = threadIdx.x; e0 < total; e0 += kBlock * kTileU) {
    VT v[kTileU];
    int dst[kTileU];
    bool fed[kTileU];
#pragma unroll
    for (int u = 0; u < kTileU; ++u) {
      const unsigned e = min(e0 + u * kBlock, total - 1);
      const unsigned row = s.nv == 1 ? e : __umulhi(e, s.magic);     // e / nv
      const unsigned j = (e - row * s.nv) * V;
      const int r = jrow[row];
      fed[u] = r >= 0;
      v[u] = *reinterpret_cast<const VT*>(s.D + (int64_t)max(r, 0) * s.ck + j);   // (a source here has rows)
      int t = s.c0 + (int)j;
      if (MAP) t = s.colmap[j];
      dst[u] = t < 0 ? -1 : (int)row * c_T + t;
    }
#pragma unroll
    for (int u = 0; u < kTileU; ++u) {
      if (e0 + u * kBlock >= total || dst[u] < 0 || (add && !fed[u])) continue;
      float x[V];
#pragma unroll
      for (int i = 0; i < V; ++i) {
        if constexpr (V == 1) x[i] = fed[u] ? v[u] : 0.0f;
        else x[i] = fed[u] ? v[u][i] : 0.0f;
      }
      float* out = tile + dst[u];
      if (add) {
#pragma unroll
        for (int i = 0; i < V; ++i) out[i] += x[i];
      } else if (V > 1 && whole) {
        VT o;
        if constexpr (V > 1) {
#pragma unroll
          for (int i = 0; i < V; ++i) o[i] = 0.0f + x[i];
        }
        *reinterpret_cast<VT*>(out) = o;
      } else {
        // 0.0f + x: a source cell holding -0.0 becomes +0.0, as in the sum that defines the cell
#pragma unroll
        for (int i = 0; i < V; ++i) out[i] = 0.0f + x[i];
      }
    }
  }
}

__global__ __launch_bounds__(kBlock) void materialize_tile_kernel(MatTileArgs a) {
  extern __shared__ float tile_lds[];
  float* tile = tile_lds;                                            // rt x c_T, flat
  int* srow = reinterpret_cast<int*>(tile_lds + a.rt * a.c_T);       // [source][rt]: the row each target row takes
  const int64_t i0 = (int64_t)blockIdx.x * a.rt;
  const int nrow = (int)min((int64_t)a.rt, a.r_T - i0);
  for (int e = threadIdx.x; e < a.n * a.rt; e += kBlock) {
    const int k = e / a.rt, u = e - k * a.rt;
    const int64_t i = i0 + u;
    int r = -1;
    if (u < nrow) r = a.s[k].idx != nullptr ? a.s[k].idx[i] : (i < a.s[k].rows ? (int)i : -1);
    srow[e] = r;
  }
  if (a.zero)
    for (int e = threadIdx.x; e < nrow * a.c_T; e += kBlock) tile[e] = 0.0f;
  __syncthreads();
  for (int k = 0; k < a.n; ++k) {
    const MatTileSource& s = a.s[k];
    const int* jrow = srow + k * a.rt;
    if (s.c0 < 0) tile_source<1, true>(s, tile, jrow, nrow, a.c_T, a.add != 0);
    else if (s.vec == 4) tile_source<4, false>(s, tile, jrow, nrow, a.c_T, a.add != 0);
    else if (s.vec == 2) tile_source<2, false>(s, tile, jrow, nrow, a.c_T, a.add != 0);
    else tile_source<1, false>(s, tile, jrow, nrow, a.c_T, a.add != 0);
    if (a.add) __syncthreads();          // cells with several feeders receive them in source order
  }
  if (!a.add) __syncthreads();
  const int64_t base = i0 * a.c_T;
  const int count = nrow * a.c_T;
  if (reinterpret_cast<uintptr_t>(a.T + base) % 16 == 0) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    const f4* src = reinterpret_cast<const f4*>(tile);
    f4* out = reinterpret_cast<f4*>(a.T + base);
    // the table is written once and not read back here: keep it out of the caches' way
    for (int e = threadIdx.x; e < count / 4; e += kBlock) __builtin_nontemporal_store(src[e], out + e);
    for (int e = count / 4 * 4 + threadIdx.x; e < count; e += kBlock) a.T[base + e] = tile[e];
  } else {
    for (int e = threadIdx.x; e < count; e += kBlock) __builtin_nontemporal_store(tile[e], a.T + base + e);
  }
}

// Target tables too wide for a tile of whole rows: a wavefront builds kSlabCols columns of one row in LDS, one source after
// the other, and writes them out.  The slab starts in LDS as far from a float4 as it does in T.  Bound by the write of T.
// 100,000 rows of 4001 columns from four tables: 442 microseconds, 3.6 TB/s written (a lane per target column: 1100; a walk
// over all sources for every column: 2281); scattered columns 1484 (3198, 4239).
constexpr int kSlabCols = 1280;
constexpr int kSlabU = 4;      // values in flight per lane
constexpr int kSlabWaves = kBlock / kWave;

__global__ __launch_bounds__(kBlock) void materialize_slab_kernel(MatTileArgs a) {
  __shared__ __align__(16) float rows_lds[kSlabWaves][kSlabCols + 4];
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int64_t i = (int64_t)blockIdx.x * kSlabWaves + wave;
  if (i >= a.r_T) return;                                            // (no barrier below: wavefronts share nothing)
  auto wave_sync = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  const int c_lo = (int)blockIdx.y * kSlabCols, cw = min(kSlabCols, a.c_T - c_lo);
  float* out = a.T + i * a.c_T + c_lo;
  const int lead = (int)((reinterpret_cast<uintptr_t>(out) / sizeof(float)) & 3);
  float* row = rows_lds[wave] + lead;
  if (a.zero)
    for (int e = lane; e < cw; e += kWave) row[e] = 0.0f;
  wave_sync();
  for (int k = 0; k < a.n; ++k) {
    const MatTileSource& s = a.s[k];
    const int r = s.idx != nullptr ? s.idx[i] : (i < s.rows ? (int)i : -1);
    if (r < 0 && a.add != 0) continue;
    const float* d = s.D + (int64_t)max(r, 0) * s.ck;                // (a source here has rows)
    // a block of columns: those of its own that fall in the slab; else every column of the slab by its place in the table
    const bool block = s.c0 >= 0;
    const int e_lo = block ? max(s.c0 - c_lo, 0) : 0, e_hi = block ? min(s.c0 + s.ck - c_lo, cw) : cw;
    for (int e0 = e_lo + lane; e0 < e_hi; e0 += kWave * kSlabU) {
      float v[kSlabU];
      int j[kSlabU];
#pragma unroll
      for (int u = 0; u < kSlabU; ++u) {
        const int e = min(e0 + u * kWave, e_hi - 1);
        j[u] = block ? c_lo + e - s.c0 : s.tcol[c_lo + e];
      }
#pragma unroll
      for (int u = 0; u < kSlabU; ++u) v[u] = r >= 0 && j[u] >= 0 ? d[j[u]] : 0.0f;
#pragma unroll
      for (int u = 0; u < kSlabU; ++u) {
        const int e = e0 + u * kWave;
        if (e < e_hi && j[u] >= 0) row[e] = (a.add != 0 ? row[e] : 0.0f) + v[u];   // 0.0f + x: no -0.0
      }
    }
    wave_sync();                                                     // cells with several feeders receive them in source order
  }
  typedef float f4 __attribute__((ext_vector_type(4)));
  const int head = min((4 - lead) & 3, cw), quads = (cw - head) / 4, tail = head + 4 * quads;
  if (lane < head) __builtin_nontemporal_store(row[lane], out + lane);
  for (int e = lane; e < quads; e += kWave)
    __builtin_nontemporal_store(*reinterpret_cast<const f4*>(row + head + 4 * e), reinterpret_cast<f4*>(out + head + 4 * e));
  if (tail + lane < cw) __builtin_nontemporal_store(row[tail + lane], out + tail + lane);
}

// Fast form for schemas whose every aligned group of four target columns is an aligned float4 of one source, or fed by
// nobody (gslot / gj0 tables, built with the plan): the table is written as one flat stream of float4, element e is
// column group e % (c_T / 4) of row e / (c_T / 4).  A wavefront stores kFlatU runs of 64 consecutive float4, so every store instruction fills whole
// 128-byte lines whatever the row length (880-byte rows otherwise leave partial lines at both ends of each row).
// The loop body has no branches: all
// row indices of a step are requested, then all source values, then all stores go out; elements nobody feeds
// read a dummy location and are replaced by zero.
constexpr int kFlatU = 4;
constexpr int kFlatMaxCols = 1024;
typedef const int32_t __attribute__((address_space(1)))* GIntPtr;
typedef float mf4 __attribute__((ext_vector_type(4)));
typedef const mf4 __attribute__((address_space(1)))* GVecPtr;

__global__ __launch_bounds__(kBlock) void materialize_flat_kernel(MatArgs a, int64_t total) {
  __shared__ const float* sD[kMaxSources];
  __shared__ const int32_t* sIdx[kMaxSources];
  __shared__ int64_t sRows[kMaxSources];
  __shared__ int sCk[kMaxSources];
  __shared__ short gS[kFlatMaxCols / 4];
  __shared__ short gJ[kFlatMaxCols / 4];
  const int ngroups = a.c_T / 4;
  if (threadIdx.x < kMaxSources) {
    int k = threadIdx.x;
    sD[k] = k < a.n ? a.D[k] : nullptr;
    sIdx[k] = k < a.n ? a.idx[k] : nullptr;
    sRows[k] = k < a.n ? a.rows[k] : 0;
    sCk[k] = k < a.n ? a.ck[k] : 0;
  }
  for (int g = threadIdx.x; g < ngroups; g += kBlock) { gS[g] = (short)a.gslot[g]; gJ[g] = (short)a.gj0[g]; }
  __syncthreads();
  const int lane = threadIdx.x % kWave;
  const int32_t* dummy = a.gslot;                   // 16-byte aligned, at least four values long
  constexpr int64_t kRun = (int64_t)kWave * kFlatU;
  const int64_t wave0 = ((int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave) * kRun;
  const int64_t stride = (int64_t)gridDim.x * (kBlock / kWave) * kRun;
  for (int64_t c0 = wave0; c0 < total; c0 += stride) {
    const int64_t row0 = c0 / ngroups;
    const unsigned g0 = (unsigned)(c0 - row0 * ngroups);
    int64_t irow[kFlatU];
    int slot[kFlatU], joff[kFlatU], ridx[kFlatU];
    bool gathered[kFlatU];
#pragma unroll
    for (int u = 0; u < kFlatU; ++u) {
      const unsigned off = g0 + lane + u * kWave;
      const unsigned dr = off / (unsigned)ngroups;
      const int g = (int)(off - dr * (unsigned)ngroups);
      irow[u] = row0 + dr;
      const bool live = c0 + lane + u * kWave < total;
      slot[u] = live ? (int)gS[g] : -1;
      joff[u] = gJ[g];
      const int32_t* ip = slot[u] >= 0 ? sIdx[slot[u]] : nullptr;
      gathered[u] = ip != nullptr;
      ridx[u] = *(GIntPtr)(gathered[u] ? ip + irow[u] : dummy);
    }
    mf4 v[kFlatU];
    bool fed[kFlatU];
#pragma unroll
    for (int u = 0; u < kFlatU; ++u) {
      const int sl = max(slot[u], 0);
      const int64_t r = gathered[u] ? (int64_t)ridx[u] : (irow[u] < sRows[sl] ? irow[u] : -1);
      fed[u] = slot[u] >= 0 && r >= 0;
      const float* src = fed[u] ? sD[sl] + r * sCk[sl] + joff[u] : reinterpret_cast<const float*>(dummy);
      v[u] = *(GVecPtr)src;
    }
#pragma unroll
    for (int u = 0; u < kFlatU; ++u) {
      const int64_t e = c0 + lane + u * kWave;
      if (e < total) {
        // 0.0f + x: a source cell holding -0.0 becomes +0.0, as in the sum that defines the cell
        mf4 o = {0.0f + v[u].x, 0.0f + v[u].y, 0.0f + v[u].z, 0.0f + v[u].w};
        if (!fed[u]) o = (mf4){0.0f, 0.0f, 0.0f, 0.0f};
        // the table is written once and not read back here: keep it out of the caches' way
        __builtin_nontemporal_store(o, reinterpret_cast<mf4*>(a.T) + e);
      }
    }
  }
}

}  // namespace

// Above 2048 columns a tile of four rows leaves room for few workgroups, and blocks of columns go through slabs: 100,000
// rows, tiles / slabs, microseconds: 1501 columns 153 / 168, 2001 210 / 210, 3001 344 / 319, 3501 610 / 377.  Scattered
// columns, which a slab reads one by one, keep the tiles as long as four rows fit (2001: 270 / 507, 3501: 837 / 1366).
bool materialize_tile_supported(const MatTileArgs& a) {
  bool blocks = true;
  for (int k = 0; k < a.n; ++k) blocks = blocks && a.s[k].c0 >= 0;
  return a.c_T <= (blocks ? 2048 : kMatTileMaxCols);
}

hipError_t launch_materialize_tile(MatTileArgs a, hipStream_t st) {
  if (a.r_T <= 0 || a.c_T <= 0) return hipSuccess;
  // Rows per tile: about 20 KiB of LDS, and tiles of whole 128-byte lines where the row length allows it in that space.
  int line = 32;                                     // rows whose cells fill whole lines: 32 / gcd(32, c_T)
  while (line > 1 && (line / 2) * a.c_T % 32 == 0) line /= 2;
  line = line < 4 ? 4 : line;                        // (tiles start on float4s)
  int rt = kMatTileFloats / a.c_T;
  if (rt >= line) rt = rt / line * line;
  else rt = rt / 4 * 4;
  rt = rt < 4 ? 4 : (rt > 256 ? 256 : rt);
  if (a.r_T < (int64_t)rt * 1024) {
    // fewer tiles than four per compute unit: smaller ones, so that every unit has some
    int64_t want = (a.r_T + 1023) / 1024;
    want = (want + line - 1) / line * line;
    rt = (int)(want < rt ? want : rt);
  }
  a.rt = rt;
  const size_t lds = sizeof(float) * (size_t)rt * a.c_T + sizeof(int) * (size_t)rt * a.n;
  const int64_t grid = (a.r_T + rt - 1) / rt;
  materialize_tile_kernel<<<(unsigned)grid, kBlock, lds, st>>>(a);
  return hipGetLastError();
}

hipError_t launch_materialize_slab(const MatTileArgs& a, hipStream_t st) {
  if (a.r_T <= 0 || a.c_T <= 0) return hipSuccess;
  const dim3 grid((unsigned)((a.r_T + kSlabWaves - 1) / kSlabWaves), (unsigned)((a.c_T + kSlabCols - 1) / kSlabCols));
  materialize_slab_kernel<<<grid, kBlock, 0, st>>>(a);
  return hipGetLastError();
}

bool materialize_flat_supported(const MatArgs& a) {
  return a.gslot != nullptr && a.c_T % 4 == 0 && a.c_T <= kFlatMaxCols && reinterpret_cast<uintptr_t>(a.T) % 16 == 0 &&
         reinterpret_cast<uintptr_t>(a.gslot) % 16 == 0;
}

hipError_t launch_materialize_flat(const MatArgs& a, hipStream_t st) {
  if (a.r_T <= 0 || a.c_T <= 0) return hipSuccess;
  const int64_t total = a.r_T * (a.c_T / 4);
  int64_t waves = (total + kWave * kFlatU - 1) / (kWave * kFlatU);
  int64_t grid = (waves + (kBlock / kWave) - 1) / (kBlock / kWave);
  if (grid > 65536) grid = 65536;
  materialize_flat_kernel<<<(int)grid, kBlock, 0, st>>>(a, total);
  return hipGetLastError();
}

}  // namespace ilargi
