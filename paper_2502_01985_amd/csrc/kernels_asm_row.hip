// Assembly pass of the left multiply with residual, loss and the entity table's block of the gradient, for one to four operand
// columns over short rows that start anywhere (at most 24 columns), a lane per row.
//
// A wavefront reads 64 rows as a flat stream of float4, passes them through an LDS tile of its own and reads them back row by
// lane: dot products against operand values that come as scalars (the table's columns are a block of the target's), gathered
// products and residual are plain per-lane arithmetic.  The gradient is a product of the staged rows and their residuals on the
// matrix cores.  No barrier in the loop; requests run a step ahead, row numbers two.
// 333,333 x 13 with two joined tables, three logistic models: 13.3 microseconds (17.7 through tiles that workgroups share; 14.2
// with the gradient as per-lane sums, whose meeting across the lanes is a third of the instructions).  Bound by latency: a
// wavefront has two steps of 64 rows, 860 instructions in all.
#include <algorithm>
#include <cstdint>
#include <cstring>

#include "ilargi_internal.h"

namespace ilargi {

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
constexpr int kRowWaves = kBlock / kWave;
constexpr int kRowGather = 4;

typedef const float __attribute__((address_space(4))) scalar_float;

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int CTRL, int ROWS>
__device__ __forceinline__ float add_moved(float v) {
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xf, true));
}
// Sum of a wavefront's values, in its last lane.
__device__ __forceinline__ float sum_of_wave(float v) {
  v = add_moved<0x111, 0xf>(v);
  v = add_moved<0x112, 0xf>(v);
  v = add_moved<0x114, 0xf>(v);
  v = add_moved<0x118, 0xf>(v);
  v = add_moved<0x142, 0xa>(v);
  return add_moved<0x143, 0xc>(v);
}

// CK: columns, rounded up to whole float4s (the others count as zero).
template <int CT, int MODE, int CK>
__global__ __launch_bounds__(kBlock, 4) void asm_row_kernel(LmmArgs a) {
  constexpr int JT = (CK + 15) / 16;                            // tiles of 16 columns of the gradient
  // (the last row's tile of 16 columns may be read past its end)
  __shared__ __align__(16) float lds[kRowWaves * kWave * (CK + CT) + 32];
  const int tid = (int)threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const int ck = a.ck;
  float* tile = lds + wave * kWave * CK;
  float* res = lds + kRowWaves * kWave * CK + wave * kWave * CT;   // the rows' residuals
  const int n16 = lane % 16, k4 = lane / 16;
  const scalar_float* w0 = (const scalar_float*)(uintptr_t)(a.X + (int64_t)(a.x_block - 1) * a.ldx + a.col0);
  const int64_t chunks = (a.r_out + kWave - 1) / kWave, step = (int64_t)gridDim.x * kRowWaves;
  int64_t ch = (int64_t)blockIdx.x * kRowWaves + wave;
  const int64_t last4 = a.d_rows * ck / 4 - 1;                  // whole float4s of the table
  v4f v[CK / 4];
  int jn[kRowGather];
  float pn[kRowGather][CT], yn = 0.0f;
  auto row_of = [&](int64_t c) { return min(c * kWave + lane, a.r_out - 1); };
  auto load_rows = [&](int64_t c) {
    const int64_t base = c * (kWave * ck / 4) + lane;           // (64 rows are whole float4s)
#pragma unroll
    for (int u = 0; u < CK / 4; ++u) v[u] = reinterpret_cast<const v4f*>(a.D)[min(base + u * kWave, last4)];
  };
  auto load_index = [&](int64_t c) {
    const int64_t i = row_of(c);
#pragma unroll
    for (int s = 0; s < kRowGather; ++s) jn[s] = s < a.g.n ? a.g.idx[s][i] : -1;
  };
  auto gather = [&](int64_t c) {
#pragma unroll
    for (int s = 0; s < kRowGather; ++s) {
      if (s >= a.g.n) break;
      const float* p = a.g.P[s] + (int64_t)max(jn[s], 0) * a.g.ldp + a.col0;
#pragma unroll
      for (int n = 0; n < CT; ++n) pn[s][n] = p[n];
#pragma unroll
      for (int n = 0; n < CT; ++n) pn[s][n] = jn[s] >= 0 ? pn[s][n] : 0.0f;
    }
    yn = a.y[row_of(c)];
  };
  float loss[CT];
  v4f g[JT];                                                    // column 16 h + 4 (lane / 16) + register, operand column lane % 16
#pragma unroll
  for (int h = 0; h < JT; ++h) g[h] = (v4f){0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int n = 0; n < CT; ++n) loss[n] = 0.0f;
  if (ch < chunks) {
    load_index(ch);
    load_rows(ch);
    gather(ch);
    load_index(ch + step);
  }
  for (; ch < chunks; ch += step) {
    const int64_t i = ch * kWave + lane;
    wave_sync();                                                // the previous step's tile is consumed
    const int64_t rows = min((int64_t)kWave, max(a.d_rows - ch * kWave, (int64_t)0));
    const int floats = (int)rows * ck;
#pragma unroll
    for (int u = 0; u < CK / 4; ++u) {
      const int e = 4 * (lane + u * kWave);
      if (e >= kWave * ck) continue;
      v4f t = v[u];
      if (floats < kWave * ck) {                                // the table's last rows
#pragma unroll
        for (int c = 0; c < 4; ++c) t[c] = e + c < floats ? a.D[ch * kWave * ck + e + c] : 0.0f;
      }
      *reinterpret_cast<v4f*>(tile + e) = t;
    }
    float z[CT], more[CT];
    const float yi = yn;
#pragma unroll
    for (int n = 0; n < CT; ++n) {
      z[n] = more[n] = 0.0f;
#pragma unroll
      for (int s = 0; s < kRowGather; ++s)
        if (s < a.g.n) more[n] += pn[s][n];
    }
    wave_sync();
    if (ch + step < chunks) {
      load_rows(ch + step);
      gather(ch + step);
      load_index(ch + 2 * step);
    }
    const float* d = tile + lane * ck;
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
        x[j] = j < CK - 3 || j < ck ? d[j] : 0.0f;
      }
    }
    const scalar_float* w = w0;
#pragma unroll
    for (int j = 0; j < CK; ++j) {
      if (j % 8 == 0) asm volatile("" : "+s"(w));               // (scalars are requested again: kept, they would spill)
      if (j < CK - 3 || j < ck) {
#pragma unroll
        for (int n = 0; n < CT; ++n) z[n] = fmaf(x[j], w[(int64_t)j * a.ldx + n], z[n]);
      }
    }
    float r[CT];
    const bool live = i < a.r_out, has = i < a.d_rows;            // (a row beyond the table has no product, whatever the weights)
#pragma unroll
    for (int n = 0; n < CT; ++n) {
      float l = 0.0f;
      z[n] = has ? z[n] : 0.0f;
      if constexpr (MODE == 1) {
        r[n] = z[n] + more[n] - yi;
        l = r[n] * r[n];
      } else {
        r[n] = logistic_residual(z[n] + more[n], yi, l);
      }
      r[n] = live ? r[n] : 0.0f;
      loss[n] += live ? l : 0.0f;
    }
    if (live) {
      float* o = a.out + i * a.ldo + a.col0;
#pragma unroll
      for (int n = 0; n < CT; ++n) o[n] = r[n];
    }
    // the gradient: four rows a product, 16 k + q for the lanes' groups k; what lies beyond the columns or the operand columns
    // goes to sums that nobody reads, and a row that the table does not feed has no part in it
#pragma unroll
    for (int n = 0; n < CT; ++n) res[lane * CT + n] = has ? r[n] : 0.0f;
    wave_sync();
    const float* ra = tile + k4 * 16 * ck + n16;
    const float* rb = res + k4 * 16 * CT + n16 % CT;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const float e = rb[q * CT];
#pragma unroll
      for (int h = 0; h < JT; ++h) g[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(ra[q * ck + 16 * h], e, g[h], 0, 0, 0);
      if (q % 8 == 7) __builtin_amdgcn_sched_barrier(0);
    }
  }
  // the wavefronts in order
  __syncthreads();
  constexpr int kSums = 16 * JT * CT + CT;
#pragma unroll
  for (int h = 0; h < JT; ++h)
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (n16 < CT) lds[wave * kSums + (16 * h + 4 * k4 + u) * CT + n16] = g[h][u];
#pragma unroll
  for (int n = 0; n < CT; ++n) {
    const float s = sum_of_wave(loss[n]);
    if (lane == kWave - 1) lds[wave * kSums + 16 * JT * CT + n] = s;
  }
  __syncthreads();
  for (int e = tid; e < kSums; e += kBlock) {
    float s = 0.0f;
#pragma unroll
    for (int q = 0; q < kRowWaves; ++q) s += lds[q * kSums + e];
    const int j = e / CT, n = e % CT;
    if (j == 16 * JT) a.loss_partial[(int64_t)blockIdx.x * kNarrowCT + n] = s;
    else if (j < ck) a.grad_partial[((int64_t)blockIdx.x * ck + j) * kNarrowCT + n] = s;
  }
}

template <int CT, int MODE>
void start(const LmmArgs& a, int grid, hipStream_t st) {
  const int ck = (a.ck + 3) / 4 * 4;
  if (ck == 4) asm_row_kernel<CT, MODE, 4><<<grid, kBlock, 0, st>>>(a);
  else if (ck == 8) asm_row_kernel<CT, MODE, 8><<<grid, kBlock, 0, st>>>(a);
  else if (ck == 12) asm_row_kernel<CT, MODE, 12><<<grid, kBlock, 0, st>>>(a);
  else if (ck == 16) asm_row_kernel<CT, MODE, 16><<<grid, kBlock, 0, st>>>(a);
  else if (ck == 20) asm_row_kernel<CT, MODE, 20><<<grid, kBlock, 0, st>>>(a);
  else asm_row_kernel<CT, MODE, 24><<<grid, kBlock, 0, st>>>(a);
}

}  // namespace

bool asm_row_supported(const LmmArgs& a, int mode, bool fuseg) {
  if (!fuseg || (mode != 1 && mode != 2) || a.D == nullptr || a.x_block < 1 || a.nt_in != 0 || a.nt_out != 0) return false;
  if (a.ncols < 1 || a.ncols > kNarrowCT || a.ck < 1 || a.ck > 24) return false;
  if (a.r_out < kWave || a.d_rows < 4 || a.g.n > kRowGather || reinterpret_cast<uintptr_t>(a.D) % 16 != 0) return false;
  if (a.y == nullptr || a.loss_partial == nullptr) return false;
  for (int s = 0; s < a.g.n; ++s)
    if (a.g.idx[s] == nullptr) return false;
  return true;
}

hipError_t launch_asm_row(const LmmArgs& a, int mode, hipStream_t st, int* grid_out) {
  if (!asm_row_supported(a, mode, a.grad_partial != nullptr)) return hipErrorInvalidValue;
  int64_t grid = ((a.r_out + kWave - 1) / kWave + kRowWaves - 1) / kRowWaves;
  if (grid > kColredBlocks) {                                   // the same number of steps for every wavefront
    const int64_t per = (grid + kColredBlocks - 1) / kColredBlocks;
    grid = (grid + per - 1) / per;
  }
  if (grid_out) *grid_out = (int)grid;
#define ILARGI_ROW(C) \
  if (mode == 1) start<C, 1>(a, (int)grid, st); else start<C, 2>(a, (int)grid, st);
  switch (a.ncols) {
    case 1: ILARGI_ROW(1) break;
    case 2: ILARGI_ROW(2) break;
    case 3: ILARGI_ROW(3) break;
    default: ILARGI_ROW(4) break;
  }
#undef ILARGI_ROW
  return hipGetLastError();
}

}  // namespace ilargi
