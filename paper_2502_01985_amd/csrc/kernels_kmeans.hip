// KMeans over a short-rowed entity table (at most 20 columns, 3 to 16 centroids, at least 131,072 target rows): the assembly of
// T C, the nearest centroid of every row and the entity table's share of the per-cluster sums in one pass, a lane per row.
//
// A wavefront reads 64 rows as a flat stream of float4, passes them through an LDS tile of its own and reads them back row by
// lane.  The centroids come as scalars (the entity table's columns are a block of the target's, so their coordinates lie side by
// side); a row's products are added from column (row mod 256) mod columns on, in the order of kernels_tile.hip, so that two
// centroids that are equally near are told apart alike whatever the size of the table: all rows take the columns twice, and a
// column counts as zero for those whose turn it is not.  The cluster sums are the product of the rows' indicator and the rows on
// the matrix cores, sixteen products of four rows a step, with a column of ones for the cluster sizes.
// No barrier in the loop: wavefronts run apart, the next rows and keys are requested a step ahead.
// 1,000,000 x 20 joined with 100,000 rows, 10 centroids: 46 microseconds (through tiles that workgroups share, with the operand
// read from LDS by every lane for every column, 59); bound by instructions, 820 a step of 64 rows, 440 of them the products and
// 32 on the matrix cores.  Scalars that the compiler keeps over the step spill into vector registers (53): they are requested
// anew for every four columns.  Four workgroups a compute unit instead of three: the same.  Over 131,072 to 3,000,000 rows, 1 to
// 20 columns and 3 to 16 centroids an iteration takes 0.62 to 0.95 of the other form's time.
#include <algorithm>
#include <cstdint>

#include "ilargi_internal.h"

namespace ilargi {

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
constexpr int kLaneThreads = 256, kLaneWaves = kLaneThreads / kWave;
constexpr int kLaneColumns = 20;
constexpr int kLaneTile = kWave * kLaneColumns + 64;      // floats of a wavefront's tile: rows, and 16 floats after every 16 rows

// Values that are the same in every lane and that no kernel in flight changes, read as scalars.
typedef const float __attribute__((address_space(4))) scalar_float;
__device__ __forceinline__ const scalar_float* to_scalar(const float* p) { return (const scalar_float*)(uintptr_t)p; }

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ float uniform(float x) { return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(x))); }

// A row of K products: whole float4s, float2s or floats, as its length allows.
template <int K>
__device__ __forceinline__ void product_row(const float* p, bool there, float (&t)[K]) {
  if constexpr (K % 4 == 0) {
#pragma unroll
    for (int n = 0; n < K; n += 4) {
      const v4f w = *reinterpret_cast<const v4f*>(p + n);
#pragma unroll
      for (int c = 0; c < 4; ++c) t[n + c] = w[c];
    }
  } else if constexpr (K % 2 == 0) {
#pragma unroll
    for (int n = 0; n < K; n += 2) {
      const float2 w = *reinterpret_cast<const float2*>(p + n);
      t[n] = w.x; t[n + 1] = w.y;
    }
  } else {
#pragma unroll
    for (int n = 0; n < K; ++n) t[n] = p[n];
  }
#pragma unroll
  for (int n = 0; n < K; ++n) t[n] = there ? t[n] : 0.0f;
}

// CK: columns, rounded up to whole float4s (the others count as zero).
template <int K, int CK>
__global__ __launch_bounds__(kLaneThreads, 3) void kmeans_lane_kernel(KmeansLaneArgs a) {
  constexpr bool TWO = CK > 12;                           // the columns and the ones take two tiles of 16
  __shared__ __align__(16) float lds[kLaneWaves * kLaneTile];
  __shared__ float cns[16];
  const int tid = (int)threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const int ck = a.ck, pad = ck % 2 == 0 ? 16 : 0;
  // norms of the centroids, in the order of centroid_norm_kernel
  if (a.cn == nullptr) {
    float s[K];
#pragma unroll
    for (int n = 0; n < K; ++n) s[n] = 0.0f;
    if (tid < kBlock)
      for (int t = tid; t < a.c_T; t += kBlock)
#pragma unroll
        for (int n = 0; n < K; ++n) {
          const float v = a.C[(int64_t)t * K + n];
          s[n] = fmaf(v, v, s[n]);
        }
    static_assert(16 * kBlock <= kLaneWaves * kLaneTile && kBlock == 4 * kWave, "scratch of the norms; two steps before a wavefront's");
    if (tid < kBlock)
#pragma unroll
      for (int n = 0; n < K; ++n) lds[n * kBlock + tid] = s[n];
    __syncthreads();
    for (int n = wave; n < K; n += kLaneWaves) {
      const float* r = lds + n * kBlock + lane;
      float v = (r[0] + r[2 * kWave]) + (r[kWave] + r[3 * kWave]);
      for (int w = kWave / 2; w > 0; w >>= 1) v += __shfl_down(v, w);
      if (lane == 0) cns[n] = v;
    }
  } else if (tid < K) {
    cns[tid] = a.cn[tid];
  }
  bool plain = true;                                      // every centroid's coordinates of these columns are finite
  for (int e = lane; e < CK * K; e += kWave) plain = plain && fabsf(a.C[(int64_t)a.t0 * K + e]) <= __FLT_MAX__;
  plain = __all(plain);
  __syncthreads();
  float norm[K];
#pragma unroll
  for (int n = 0; n < K; ++n) norm[n] = uniform(cns[n]);
  float* tile = lds + wave * kLaneTile;
  const scalar_float* w = to_scalar(a.C + (int64_t)a.t0 * K);
  const int64_t chunks = (a.r_T + kWave - 1) / kWave, step = (int64_t)gridDim.x * kLaneWaves;
  const int64_t first = (int64_t)blockIdx.x * kLaneWaves + wave;
  const int64_t last4 = a.d_rows * ck / 4 - 1;            // whole float4s of the table
  v4f acc[2] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};

  int place[CK / 4];
#pragma unroll
  for (int u = 0; u < CK / 4; ++u) {
    const int e = 4 * (lane + u * kWave);
    place[u] = e + (pad != 0 ? e / (16 * ck) * 16 : 0);
  }
  v4f v[CK / 4];
  int j0 = -1;
  auto request = [&](int64_t ch) {
    const int64_t base = ch * (kWave * ck / 4) + lane;    // (64 rows are whole float4s)
#pragma unroll
    for (int u = 0; u < CK / 4; ++u) v[u] = reinterpret_cast<const v4f*>(a.D)[min(base + u * kWave, last4)];
    const int64_t i = min(ch * kWave + lane, a.r_T - 1);
    if (a.n > 0) j0 = a.idx[0][i];
  };
  if (first < chunks) request(first);
  for (int64_t ch = first; ch < chunks; ch += step) {
    const int64_t i = ch * kWave + lane;
    // the rows into the tile
    wave_sync();
    const int64_t rows = min((int64_t)kWave, max(a.d_rows - ch * kWave, (int64_t)0));
    const int floats = (int)rows * ck;
#pragma unroll
    for (int u = 0; u < CK / 4; ++u) {
      const int e = 4 * (lane + u * kWave);
      if (e >= kWave * ck) continue;
      v4f t = v[u];
      if (floats < kWave * ck) {                          // the table's last rows
#pragma unroll
        for (int c = 0; c < 4; ++c) t[c] = e + c < floats ? a.D[ch * kWave * ck + e + c] : 0.0f;   // (zeros beyond)
      }
      // (rows of an odd number of columns have no room between the groups of 16, so a float4 is never torn)
      *reinterpret_cast<v4f*>(tile + place[u]) = t;
    }
    float g[K];
    product_row<K>(a.n > 0 ? a.P[0] + (int64_t)max(j0, 0) * K : a.C, a.n > 0 && j0 >= 0, g);
    if (a.n > 1) {
      float more[K];
#pragma unroll
      for (int n = 0; n < K; ++n) more[n] = 0.0f;
      for (int s = 1; s < a.n; ++s) {
        const int j = a.idx[s][min(i, a.r_T - 1)];
        float t[K];
        product_row<K>(a.P[s] + (int64_t)max(j, 0) * K, j >= 0, t);
#pragma unroll
        for (int n = 0; n < K; ++n) more[n] += t[n];
      }
#pragma unroll
      for (int n = 0; n < K; ++n) g[n] += more[n];
    }
    wave_sync();
    request(min(ch + step, chunks - 1));
    float z[K];
#pragma unroll
    for (int n = 0; n < K; ++n) z[n] = 0.0f;
    const float* d = tile + lane * ck + lane / 16 * pad;
    const int from = ck % 2 == 0 ? (int)(i % kBlock) % ck : 0;
    if (plain) {
      float x[CK];
      if (ck % 4 == 0) {
#pragma unroll
        for (int j = 0; j < CK; j += 4) {
          const v4f t = *reinterpret_cast<const v4f*>(d + j);
#pragma unroll
          for (int c = 0; c < 4; ++c) x[j + c] = t[c];
        }
      } else {
#pragma unroll
        for (int j = 0; j < CK; ++j) {
          x[j] = d[j];
          if (j > CK - 4) x[j] = j < ck ? x[j] : 0.0f;
        }
      }
      const scalar_float* wj = w;
#pragma unroll
      for (int j = 0; j < CK; ++j) {
        if (j % 4 == 0) asm volatile("" : "+s"(wj));     // (scalars are requested again: there is no room for all of them)
        const float xj = j >= from ? x[j] : 0.0f;
#pragma unroll
        for (int n = 0; n < K; ++n) z[n] = fmaf(xj, wj[j * K + n], z[n]);
      }
      if (ck % 2 == 0) {
#pragma unroll
        for (int j = 0; j < CK; ++j) {
          if (j % 4 == 0) asm volatile("" : "+s"(wj));
          const float xj = j < from ? x[j] : 0.0f;
#pragma unroll
          for (int n = 0; n < K; ++n) z[n] = fmaf(xj, wj[j * K + n], z[n]);
        }
      }
    } else {
      int j = from;
      for (int it = 0; it < ck; ++it) {
#pragma unroll
        for (int n = 0; n < K; ++n) z[n] = fmaf(d[j], a.C[(int64_t)(a.t0 + j) * K + n], z[n]);
        j = j + 1 == ck ? 0 : j + 1;
      }
#pragma unroll
      for (int n = 0; n < K; ++n) z[n] = i < a.d_rows ? z[n] : 0.0f;   // (zeros beyond the table are no product)
    }
    int best = 0;
    float bv = norm[0] - 2.0f * (z[0] + g[0]);
#pragma unroll
    for (int n = 1; n < K; ++n) {
      const float u = norm[n] - 2.0f * (z[n] + g[n]);
      if (u < bv) { bv = u; best = n; }                   // strict: the first of equal minima stays
    }
    if (i < a.r_T) a.assign[i] = best;
    else best = -1;
    // step q: rows 16 k + q (k: the lane's group of 16), sixteen clusters, sixteen columns and, with TWO, four more and the ones
    const int n16 = lane % 16, k4 = lane / 16;
    const float* b0 = tile + k4 * (16 * ck + pad);
    const float ones0 = n16 == ck ? 1.0f : 0.0f, ones1 = 16 + n16 == ck ? 1.0f : 0.0f;
#define ILARGI_STEP(q)                                                                                              \
  {                                                                                                                 \
    const int of = __builtin_amdgcn_update_dpp(0, best, 0x150 + q, 0xf, 0xf, true);     /* of lane q of the group */ \
    const float ind = of == n16 ? 1.0f : 0.0f;                                                                      \
    float c0 = b0[q * ck + (CK > 16 || n16 < ck ? n16 : 0)];                                                        \
    if constexpr (CK <= 16) c0 = n16 < ck ? c0 : ones0;                                                             \
    acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(ind, c0, acc[0], 0, 0, 0);                                        \
    if constexpr (TWO) {                                                                                            \
      const float c1 = b0[q * ck + (16 + n16 < ck ? 16 + n16 : 0)];                                                 \
      acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(ind, 16 + n16 < ck ? c1 : ones1, acc[1], 0, 0, 0);              \
    }                                                                                                               \
  }
    ILARGI_STEP(0) ILARGI_STEP(1) ILARGI_STEP(2) ILARGI_STEP(3)
    __builtin_amdgcn_sched_barrier(0);
    ILARGI_STEP(4) ILARGI_STEP(5) ILARGI_STEP(6) ILARGI_STEP(7)
    __builtin_amdgcn_sched_barrier(0);
    ILARGI_STEP(8) ILARGI_STEP(9) ILARGI_STEP(10) ILARGI_STEP(11)
    __builtin_amdgcn_sched_barrier(0);
    ILARGI_STEP(12) ILARGI_STEP(13) ILARGI_STEP(14) ILARGI_STEP(15)
#undef ILARGI_STEP
  }
  // a wavefront's sums, [16 clusters][ck + 1]; where one is not finite (a value of the table, which the other clusters' zeros
  // turn into NaN) they are added again, each row to its own
  wave_sync();
  const int ld = ck + 1;
  bool finite = true;
#pragma unroll
  for (int q = 0; q < 4; ++q) finite = finite && fabsf(acc[0][q]) <= __FLT_MAX__ && fabsf(acc[1][q]) <= __FLT_MAX__;
#pragma unroll
  for (int h = 0; h < (TWO ? 2 : 1); ++h)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int c = 4 * (lane / 16) + q, j = 16 * h + lane % 16;
      if (j <= ck) tile[c * ld + j] = acc[h][q];
    }
  wave_sync();
  if (!__all(finite)) {
    __threadfence();                                      // (the assignments this wavefront wrote)
    for (int e = lane; e < K * ck; e += kWave) {
      const int c = e / ck, j = e - c * ck;
      float s = 0.0f;
      for (int64_t ch = first; ch < chunks; ch += step)
        for (int64_t i = ch * kWave; i < min((ch + 1) * kWave, a.d_rows); ++i)
          if (__hip_atomic_load(a.assign + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == c) s += a.D[i * ck + j];
      tile[c * ld + j] = s;
    }
  }
  __syncthreads();
  for (int o = tid; o < ck * K; o += kLaneThreads) {
    const int j = o / K, c = o - j * K;
    float s = 0.0f;
#pragma unroll
    for (int q = 0; q < kLaneWaves; ++q) s += lds[q * kLaneTile + c * ld + j];
    a.sums[((int64_t)blockIdx.x * ck + j) * K + c] = s;
  }
  if (tid < K) {
    int s = 0;
#pragma unroll
    for (int q = 0; q < kLaneWaves; ++q) s += (int)lds[q * kLaneTile + tid * ld + ck];
    a.sizes[(size_t)blockIdx.x * K + tid] = s;
  }
}

}  // namespace

bool kmeans_lane_supported(const KmeansLaneArgs& a, int k) {
  if (k < 3 || k > 16 || a.ck < 1 || a.ck > kLaneColumns || a.t0 < 0 || a.t0 + (a.ck + 3) / 4 * 4 > a.c_T || a.r_T < 131072 || a.d_rows < 4 || a.n > kTileParts) return false;
  if (reinterpret_cast<uintptr_t>(a.D) % 16 != 0) return false;
  for (int s = 0; s < a.n; ++s)
    if (a.idx[s] == nullptr) return false;
  return true;
}

// Three workgroups a compute unit (256 of them), as many as fit; each leaves a block of sums that a later launch adds up.
int kmeans_lane_grid(int64_t r_T) { return (int)std::min<int64_t>(768, (r_T + kLaneThreads - 1) / kLaneThreads); }

hipError_t launch_kmeans_lane(const KmeansLaneArgs& a, int k, int grid, hipStream_t st) {
  if (!kmeans_lane_supported(a, k)) return hipErrorInvalidValue;
#define ILARGI_KMEANS(C)                                                           \
  case C:                                                                          \
    if (a.ck <= 4) kmeans_lane_kernel<C, 4><<<grid, kLaneThreads, 0, st>>>(a);       \
    else if (a.ck <= 8) kmeans_lane_kernel<C, 8><<<grid, kLaneThreads, 0, st>>>(a);   \
    else if (a.ck <= 12) kmeans_lane_kernel<C, 12><<<grid, kLaneThreads, 0, st>>>(a); \
    else if (a.ck <= 16) kmeans_lane_kernel<C, 16><<<grid, kLaneThreads, 0, st>>>(a); \
    else kmeans_lane_kernel<C, 20><<<grid, kLaneThreads, 0, st>>>(a);                 \
    break;
  switch (k) {
    ILARGI_KMEANS(3) ILARGI_KMEANS(4) ILARGI_KMEANS(5) ILARGI_KMEANS(6) ILARGI_KMEANS(7) ILARGI_KMEANS(8) ILARGI_KMEANS(9)
    ILARGI_KMEANS(10) ILARGI_KMEANS(11) ILARGI_KMEANS(12) ILARGI_KMEANS(13) ILARGI_KMEANS(14) ILARGI_KMEANS(15) ILARGI_KMEANS(16)
    default: return hipErrorInvalidValue;
  }
#undef ILARGI_KMEANS
  return hipGetLastError();
}

}  // namespace ilargi
