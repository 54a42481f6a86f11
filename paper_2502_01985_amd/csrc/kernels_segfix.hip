// Segment sums  Z_k = I_k^T Y  of one to four operand columns over large target tables, summed in LDS in fixed point, in
// target-row order; and the assembly of gathered products alone with the segment sums of its residual.
//
// The gathering forms of kernels_tmm.hip pay one L2 request per index entry and operand: 265 G entries a second on this device,
// whatever the kernel looks like.  Here a workgroup of 16 wavefronts holds the sums of a range of source rows (at most 20,416
// of 64 bits) in LDS, walks its share of the target rows in order and adds every row whose key lies in its range: row indices
// and operand are plain streams, and no inverse index is read or kept.  Sums are 64-bit integers: ds_add_u64 takes 13 cycles a
// wavefront instruction with 64 different places (ds_add_f64 22, ds_add_f32 194 on this device), returns nothing that anyone
// waits for, and whole numbers add up to the same in any order, so the result is the same on every run.
//
// The unit of a run's sums is a power of two: a run of 2^n rows leaves 62 - n bits (at most 50) for a value, 2^6 times the
// largest of the run's first rows is the limit.  Float sums of the same length lose more than this keeps.  Where a value is
// beyond the limit the run is walked again, with its own largest finite value as the limit; infinities and NaN are then added to
// the run's sums as they are.
//
// 5,000,000 rows over 100,000 uniform, 50,000 Zipf and 10,000 uniform keys: 33 microseconds and 6 for the runs' sums (with an
// index by windows, float sums that belong to one wavefront each, 51 and 8; gathering, by slice of the target rows, 78 and 10).
// Bound by instructions: nine ranges look at 5,000,000 rows each, about ten vector instructions a row, two of them in 64 bits.
// Two more rows a thread in flight, or the conversion ahead of the test for the range (42), gain nothing.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>

#include "ilargi_internal.h"

namespace ilargi {

namespace {

typedef unsigned long long u64;
typedef float f4 __attribute__((ext_vector_type(4)));
typedef int i4 __attribute__((ext_vector_type(4)));

constexpr double kFixMagic = 6755399441055744.0;      // 1.5 * 2^52: the last 52 bits of a double around it count in ones
constexpr uint32_t kFixMagicHigh = 0x43380000u;

// v * scale as a 64-bit integer, rounded to nearest; |v * scale| < 2^51.
__device__ __forceinline__ u64 to_fixed(float v, double scale) {
  const u64 d = (u64)__double_as_longlong(fma((double)v, scale, kFixMagic));
  return d - ((u64)kFixMagicHigh << 32);
}

__device__ __forceinline__ uint32_t magnitude(float v) { return __float_as_uint(v) & 0x7fffffffu; }
constexpr uint32_t kFixInf = 0x7f800000u;

struct FixScale { float limit; double up, down; };

// The unit of a run's sums: values below 2^(e + head) in magnitude, where the largest is below 2^e, get `bits` bits.
__device__ __forceinline__ FixScale fix_scale(uint32_t largest, int head, int bits) {
  const int e = max((int)(largest >> 23), 1) - 126 + head;
  return FixScale{ldexpf(1.0f, e), ldexp(1.0, bits - e), ldexp(1.0, e - bits)};
}

// v moved across the lanes of a wavefront without LDS; lanes without a source get 0.
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ uint32_t dpp(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, true);
}
constexpr int kRowShr = 0x110, kRowBcast15 = 0x142, kRowBcast31 = 0x143;

// Largest of a wavefront's values.
__device__ __forceinline__ uint32_t largest_of_wave(uint32_t v) {
  v = max(v, dpp<kRowShr + 1>(v));
  v = max(v, dpp<kRowShr + 2>(v));
  v = max(v, dpp<kRowShr + 4>(v));
  v = max(v, dpp<kRowShr + 8>(v));
  v = max(v, dpp<kRowBcast15, 0xa>(v));
  v = max(v, dpp<kRowBcast31, 0xc>(v));
  return (uint32_t)__builtin_amdgcn_readlane((int)v, kWave - 1);
}

// Sum of a wavefront's values, in its last lane.
__device__ __forceinline__ float sum_of_wave(float v) {
  v += __uint_as_float(dpp<kRowShr + 1>(__float_as_uint(v)));
  v += __uint_as_float(dpp<kRowShr + 2>(__float_as_uint(v)));
  v += __uint_as_float(dpp<kRowShr + 4>(__float_as_uint(v)));
  v += __uint_as_float(dpp<kRowShr + 8>(__float_as_uint(v)));
  v += __uint_as_float(dpp<kRowBcast15, 0xa>(__float_as_uint(v)));
  v += __uint_as_float(dpp<kRowBcast31, 0xc>(__float_as_uint(v)));
  return v;
}

// Largest of the threads' values, in every thread (one barrier).
__device__ __forceinline__ uint32_t largest_of(uint32_t v, uint32_t* most) {
  v = largest_of_wave(v);
  if (threadIdx.x % kWave == 0) most[threadIdx.x / kWave] = v;
  __syncthreads();
  return largest_of_wave(most[threadIdx.x % (kFixThreads / kWave)]);
}

// A sum as a float.
__device__ __forceinline__ float from_fixed(u64 v, double down) {
  return (float)fma((double)(int)(v >> 32), down * 4294967296.0, (double)(uint32_t)v * down);
}

__device__ __forceinline__ void add_fixed(u64* sum, u64 v) { __hip_atomic_fetch_add(sum, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }

// Adds four rows a thread holds to their sums at[r] (value(r, c): column c of row r; rows with in(r) only).  Keys in order often
// bring a thread four rows of one sum: added up first they cost LDS one addition, and 64 lanes at one sum take ten times what
// 64 sums do.
template <int CT, class In, class Value>
__device__ __forceinline__ void add_four(u64* acc, const uint32_t (&at)[4], In in, Value value) {
  bool apart = true;
  if (__ballot(at[0] == at[3]) != 0 && at[0] == at[3] && at[0] == at[1] && at[0] == at[2]) {
    apart = false;
    if (in(0)) {
#pragma unroll
      for (int c = 0; c < CT; ++c) add_fixed(&acc[at[0] * CT + c], (value(0, c) + value(1, c)) + (value(2, c) + value(3, c)));
    }
  }
  if (apart) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (in(r)) {
#pragma unroll
        for (int c = 0; c < CT; ++c) add_fixed(&acc[at[r] * CT + c], value(r, c));
      }
  }
}

// A run's rows are blocks of 4096, every runs-th: rows in order of their keys then keep all workgroups of a range busy alike.
// The runs of XCD x are those with run % 8 == x, whose workgroups for all ranges read the same rows at about the same time.
template <int CT, bool ALIGNED>
__global__ __launch_bounds__(kFixThreads, 4) void segfix_kernel(SegFixMulti m) {
  extern __shared__ __align__(16) u64 acc[];
  __shared__ uint32_t most[kFixThreads / kWave];
  __shared__ uint32_t found;
  constexpr int U = CT == 1 ? 4 : CT == 2 ? 2 : 1;       // blocks a thread requests at once
  const int x = (int)blockIdx.x % kSegSlices, i = (int)blockIdx.x / kSegSlices;
  int q = 0;
  while (q + 1 < m.n && i >= m.first[q + 1]) ++q;
  const SegFix& a = m.s[q];
  const int range = (i - m.first[q]) / a.nsub, run = (i - m.first[q]) % a.nsub * kSegSlices + x;
  const int key0 = (int)(a.r_k * range / a.n_ranges);
  const uint32_t keys = (uint32_t)(a.r_k * (range + 1) / a.n_ranges) - (uint32_t)key0;
  const int tid = (int)threadIdx.x;
  const int slots = (int)keys * CT;
  const int64_t units = a.r_T / 4;                       // groups of four rows
  const int64_t stride = (int64_t)a.runs * kFixThreads, u0 = (int64_t)run * kFixThreads + tid;
  const int64_t blocks = (units + kFixThreads - 1) / kFixThreads;
  const int steps = run < blocks ? (int)((blocks - run + (int64_t)a.runs * U - 1) / ((int64_t)a.runs * U)) : 0;
  const int tail = run == 0 ? (int)(a.r_T % 4) : 0;      // rows beyond the last group

  // (clamped addresses instead of a branch around the loads, which would wait for them)
  struct Group { i4 k[U]; f4 y[U][CT]; };
  auto request = [&](int64_t u, Group& g) {
#pragma unroll
    for (int n = 0; n < U; ++n) {
      const int64_t at = min(u + n * stride, units - 1);
      if constexpr (ALIGNED) {
        g.k[n] = reinterpret_cast<const i4*>(a.idx)[at];
#pragma unroll
        for (int c = 0; c < CT; ++c) g.y[n][c] = reinterpret_cast<const f4*>(a.Y)[at * CT + c];
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) g.k[n][r] = a.idx[at * 4 + r];
#pragma unroll
        for (int r = 0; r < 4 * CT; ++r) g.y[n][r / 4][r % 4] = a.Y[at * 4 * CT + r];
      }
    }
  };
  auto clear = [&]() {                                   // (the stride of the runs' sums is a multiple of four)
    for (int s = 2 * tid; s < a.stride; s += 2 * kFixThreads) *reinterpret_cast<ulonglong2*>(acc + s) = ulonglong2{0, 0};
  };
  Group g0, g1;
  request(u0, g0);
  clear();
  if (tid == 0) found = 0;
  float* out = a.partial + ((int64_t)range * a.runs + run) * a.stride;
  uint32_t beyond = 0, largest = 0;
#pragma unroll
  for (int n = 0; n < U; ++n)
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r) { const uint32_t b = magnitude(g0.y[n][c][r]); largest = b < kFixInf ? max(largest, b) : largest; }
  FixScale sc = fix_scale(largest_of(largest, most), kFixHead, a.bits);
  // The rows are walked once, in kSum.  Where a value is beyond the limit that the first rows gave, again: for the largest
  // finite one, for the sums with that limit, and for what is not finite, which makes the same of a sum in any order.
  enum { kSum, kLargest, kSumAgain, kOdd };
  auto again = [&](int phase, uint32_t at, int c, float v) {
    const uint32_t b = magnitude(v);
    if (phase == kLargest) {
      if (b < kFixInf) largest = max(largest, b); else beyond |= 2u;
    } else if (at < keys) {
      if (phase == kSumAgain && b < kFixInf) add_fixed(&acc[at * CT + c], to_fixed(v, sc.up));
      if (phase == kOdd && b >= kFixInf) atomicAdd(&out[at * CT + c], v);
    }
  };
  for (int phase = kSum;;) {
    uint64_t over = 0;                                   // lanes that found a value beyond the limit
    auto spend = [&](int64_t u, const Group& g) {
#pragma unroll
      for (int n = 0; n < U; ++n) {
        if (u + n * stride >= units) continue;
        auto value = [&](int r, int c) { return g.y[n][(r * CT + c) / 4][(r * CT + c) % 4]; };
        uint32_t at[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) at[r] = (uint32_t)(g.k[n][r] - key0);
        if (phase == kSum) {
#pragma unroll
          for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < CT; ++c) over |= __ballot(!(fabsf(value(r, c)) < sc.limit));
          add_four<CT>(acc, at, [&](int r) { return at[r] < keys; }, [&](int r, int c) { return to_fixed(value(r, c), sc.up); });
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < CT; ++c) again(phase, at[r], c, value(r, c));
        }
      }
    };
    int64_t u = u0;
    for (int it = 0; it < steps; it += 2) {
      request(u + U * stride, g1);
      spend(u, g0);
      request(u + 2 * U * stride, g0);
      spend(u + U * stride, g1);
      u += 2 * U * stride;
    }
    if (tid < tail) {
      const int64_t t = units * 4 + tid;
      const uint32_t at = (uint32_t)(a.idx[t] - key0);
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        const float v = a.Y[t * CT + c];
        if (phase != kSum) {
          again(phase, at, c, v);
        } else {
          if (!(fabsf(v) < sc.limit)) beyond |= 1u;
          else if (at < keys) add_fixed(&acc[at * CT + c], to_fixed(v, sc.up));
        }
      }
    }
    if (over != 0) beyond |= 1u;
    if (phase == kOdd) break;
    if (beyond) atomicOr(&found, beyond);
    __syncthreads();
    if (phase == kSum && found != 0) {
      beyond = 0;
      phase = kLargest;
    } else if (phase == kLargest) {
      clear();
      sc = fix_scale(largest_of(largest, most), 0, a.bits);             // (its barrier stands between clearing and adding)
      phase = kSumAgain;
    } else {
      for (int s = tid; s < slots; s += kFixThreads) out[s] = from_fixed(acc[s], sc.down);
      if ((found & 2u) == 0) break;
      __threadfence();
      __syncthreads();
      phase = kOdd;
    }
    request(u0, g0);
  }
}

// The assembly of gathered products alone, with residual and loss, and the segment sums of the residual: products and sums of
// all tables in LDS, the residual never written.  MODE 1 linear, 2 logistic.  NS: tables.
// 1,000,000 rows over 6040 and 3710 keys, one logistic model: 12.5 microseconds and 4 for the workgroups' sums, where assembly,
// segment sums and their runs' sums took 8, 10 and 4.5 (an iteration with 250,000 sparse cells 30 -> 24).  About 9 of the 12.5
// are there with any number of rows: the launch, the round trips for indices and products, the sums' way out.  Hence few
// workgroups: 64 to 256 take 13.8, 12.0 (128), 13.1, and the sums of 256 take a microsecond longer to add up.
// A row without a key takes the place after its table's last: a product of zero, and a sum that nobody reads.
template <int NS, int CT, int MODE>
__global__ __launch_bounds__(kFixThreads, 4) void asm_fix_kernel(AsmFix a) {
  extern __shared__ __align__(16) u64 acc[];
  __shared__ uint32_t most[kFixThreads / kWave];
  __shared__ uint32_t found;
  __shared__ float lsum[kFixThreads / kWave][CT];
  float* prod = reinterpret_cast<float*>(acc + (size_t)a.slots);
  const int tid = (int)threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const int units = (int)(a.r_T / 4);                    // groups of four rows
  const int u0 = (int)((int64_t)units * blockIdx.x / gridDim.x), u1 = (int)((int64_t)units * (blockIdx.x + 1) / gridDim.x);
  const int steps = (u1 - u0 + kFixThreads - 1) / kFixThreads;
  const int tail = blockIdx.x + 1 == gridDim.x ? (int)(a.r_T % 4) : 0;         // rows beyond the last group

  struct Group { i4 j[NS]; f4 y; };
  auto request = [&](int u, Group& g) {                  // (see segfix_kernel)
    const int64_t at = min(u, u1 - 1);
#pragma unroll
    for (int s = 0; s < NS; ++s) g.j[s] = reinterpret_cast<const i4*>(a.idx[s])[at];
    g.y = reinterpret_cast<const f4*>(a.y)[at];
  };
  auto clear = [&]() {
    for (int s = 2 * tid; s < a.slots; s += 2 * kFixThreads) *reinterpret_cast<ulonglong2*>(acc + s) = ulonglong2{0, 0};
  };

  Group g;
  request(u0 + tid, g);
  // (the products of all tables are requested together: one after the other they cost a round trip each)
  constexpr int kAhead = CT == 1 ? 4 : 2;
  int most_keys = a.keys[0];
#pragma unroll
  for (int s = 1; s < NS; ++s) most_keys = max(most_keys, a.keys[s]);
  for (int k0 = tid; k0 < most_keys; k0 += kAhead * kFixThreads) {
    float p[NS][kAhead][CT];
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        const float* from = a.P[s] + (uint32_t)(min(k0 + u * kFixThreads, a.keys[s] - 1) * a.ldp) + a.col0;
#pragma unroll
        for (int c = 0; c < CT; ++c) p[s][u][c] = from[c];
      }
    if (k0 == tid) clear();
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int u = 0; u < kAhead; ++u)
        if (k0 + u * kFixThreads < a.keys[s]) {
#pragma unroll
          for (int c = 0; c < CT; ++c) prod[(a.off[s] + k0 + u * kFixThreads) * CT + c] = p[s][u][c];
        }
  }
  if (tid >= most_keys) clear();                         // (a thread without a product)
  if (tid < NS)
#pragma unroll
    for (int c = 0; c < CT; ++c) prod[(a.off[tid] + a.keys[tid]) * CT + c] = 0.0f;
  if (tid == 0) found = 0;
  __syncthreads();

  float loss[CT], lost[CT];
#pragma unroll
  for (int c = 0; c < CT; ++c) loss[c] = lost[c] = 0.0f;
  float* out = a.partial + (int64_t)blockIdx.x * a.slots;
  FixScale sc = {0.0f, 0.0, 0.0};
  uint32_t beyond = 0, largest = 0;
  // The rows are walked once, in kSum.  Where a value is beyond the limit that the first rows gave, again: for the largest
  // finite one, for the sums with that limit, and for what is not finite, which makes the same of a sum in any order.
  enum { kSum, kLargest, kSumAgain, kOdd };
  for (int phase = kSum;;) {
    int u = u0 + tid;
    for (int it = 0; it < steps + (tail > 0 ? 1 : 0); ++it, u += kFixThreads) {
      Group now = g;
      if (it + 1 < steps) request(u + kFixThreads, g);
      bool live = u < u1;
      if (it == steps) {
        live = tid == 0;
        for (int r = 0; r < tail; ++r) {
          const int64_t t = a.r_T - tail + r;
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (q == r) {
#pragma unroll
              for (int s = 0; s < NS; ++s) now.j[s][q] = a.idx[s][t];
              now.y[q] = a.y[t];
            }
        }
        __builtin_amdgcn_s_waitcnt(0x0f70);              // vmcnt(0) here, not where the ways meet
      }
      float e[4][CT];
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < CT; ++c) e[r][c] = 0.0f;
      if (live) {
        float add[4][CT];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
#pragma unroll
          for (int s = 0; s < NS; ++s) now.j[s][r] = (int)min((uint32_t)now.j[s][r], (uint32_t)a.keys[s]) + a.off[s];
#pragma unroll
          for (int c = 0; c < CT; ++c) {
            float z = 0.0f;
#pragma unroll
            for (int s = 0; s < NS; ++s) z += prod[now.j[s][r] * CT + c];
            add[r][c] = 0.0f;
            if constexpr (MODE == 1) {
              e[r][c] = z - now.y[r];
              add[r][c] = e[r][c] * e[r][c];
            } else {
              e[r][c] = logistic_residual(z, now.y[r], add[r][c]);
            }
          }
        }
        if (it == steps) {
#pragma unroll
          for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < CT; ++c)
              if (r >= tail) e[r][c] = add[r][c] = 0.0f;
        }
        if (phase == kSum) {
#pragma unroll
          for (int c = 0; c < CT; ++c) {                 // compensated; what is infinite stays so
            const float t = ((add[0][c] + add[1][c]) + (add[2][c] + add[3][c])) - lost[c], sum = loss[c] + t;
            lost[c] = fabsf(sum) <= __FLT_MAX__ ? (sum - loss[c]) - t : 0.0f;
            loss[c] = sum;
          }
        }
      }
      if (phase == kSum && it == 0) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int c = 0; c < CT; ++c) { const uint32_t b = magnitude(e[r][c]); largest = b < kFixInf ? max(largest, b) : largest; }
        sc = fix_scale(largest_of(largest, most), kFixHead, a.bits);
      }
      if (!live) continue;
      if (phase == kSum || phase == kSumAgain) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int c = 0; c < CT; ++c) {
            const bool in = fabsf(e[r][c]) < sc.limit;   // (below the largest finite limit: finite)
            beyond |= in ? 0u : 1u;
            e[r][c] = in ? e[r][c] : 0.0f;
          }
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          const uint32_t at[4] = {(uint32_t)now.j[s][0], (uint32_t)now.j[s][1], (uint32_t)now.j[s][2], (uint32_t)now.j[s][3]};
          add_four<CT>(acc, at, [](int) { return true; }, [&](int r, int c) { return to_fixed(e[r][c], sc.up); });
        }
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int c = 0; c < CT; ++c) {
            const uint32_t b = magnitude(e[r][c]);
            if (phase == kLargest) {
              largest = b < kFixInf ? max(largest, b) : largest;
            } else if (b >= kFixInf) {
#pragma unroll
              for (int s = 0; s < NS; ++s) atomicAdd(&out[now.j[s][r] * CT + c], e[r][c]);
            }
          }
      }
    }
    if (phase == kSum) {
      if (beyond) atomicOr(&found, 1u);
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        const float t = sum_of_wave(loss[c]);
        if (lane == kWave - 1) lsum[wave][c] = t;
      }
    }
    __syncthreads();
    if (phase == kOdd) break;
    if (phase == kSum && tid < CT) {
      float part[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int w = 0; w < kFixThreads / kWave; ++w) part[w / 4] += lsum[w][tid];
      a.loss_partial[(int64_t)blockIdx.x * kNarrowCT + tid] = (part[0] + part[1]) + (part[2] + part[3]);
    }
    const bool again = phase == kSum && found != 0;
    if (!again && phase != kLargest) {
      for (int s = tid; s < a.slots; s += kFixThreads) out[s] = from_fixed(acc[s], sc.down);
      if (phase == kSum || !__syncthreads_or((int)beyond)) break;       // (beyond the largest finite one: not finite)
      __threadfence();
      __syncthreads();
      phase = kOdd;
    } else if (again) {
      phase = kLargest;
    } else {
      clear();
      sc = fix_scale(largest_of(largest, most), 0, a.bits);             // (its barrier stands between clearing and adding)
      beyond = 0;
      phase = kSumAgain;
    }
    request(u0 + tid, g);
  }
}

// Z[j] = the runs' sums of key j: the threads of a workgroup are PARTS parts, each adds every PARTS-th run of
// 4 * kBlock / PARTS sums of a range (pairwise: the sums are rounded less often on their way).
template <int CT, int PARTS>
__global__ __launch_bounds__(kBlock) void segfix_combine_kernel(SegFixMulti m) {
  __shared__ f4 part[kBlock];
  int q = 0;
  while (q + 1 < m.n && (int)blockIdx.x >= m.cfirst[q + 1]) ++q;
  const SegFix& a = m.s[q];
  const int b = (int)blockIdx.x - m.cfirst[q], range = b / m.range_blocks[q];
  const int key0 = (int)(a.r_k * range / a.n_ranges);
  const int slots = ((int)(a.r_k * (range + 1) / a.n_ranges) - key0) * CT;
  constexpr int kGroup = kBlock / PARTS;
  const int l = threadIdx.x % kGroup, g = (int)threadIdx.x / kGroup;
  const int s = (b - range * m.range_blocks[q]) * (4 * kGroup) + 4 * l;
  f4 z = {0.0f, 0.0f, 0.0f, 0.0f};
  if (s < slots) {                                       // (the stride is a multiple of four)
    const float* p = a.partial + (int64_t)range * a.runs * a.stride + s;
    for (int c = g; c < a.runs; c += 8 * PARTS) {
      f4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int r = c + u * PARTS;
        v[u] = r < a.runs ? *reinterpret_cast<const f4*>(p + (int64_t)r * a.stride) : f4{0.0f, 0.0f, 0.0f, 0.0f};
      }
      z += ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
    }
  }
  part[threadIdx.x] = z;
  __syncthreads();
  if (g == 0) {
    f4 p[PARTS];
#pragma unroll
    for (int c = 0; c < PARTS; ++c) p[c] = part[c * kGroup + l];
#pragma unroll
    for (int d = PARTS / 2; d >= 1; d /= 2)
#pragma unroll
      for (int c = 0; c < d; ++c) p[c] += p[c + d];
    z = p[0];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (s + u < slots) a.Z[(int64_t)(key0 + (s + u) / CT) * a.ldz + a.zcol0 + (s + u) % CT] = z[u];
  }
}

// Sums up the runs of m's sources.
hipError_t launch_combine(SegFixMulti& m, int ncols, hipStream_t st) {
  int runs = 0;
  for (int q = 0; q < m.n; ++q) runs = std::max(runs, m.s[q].runs);
  const int parts = runs >= 64 ? 16 : 4;
  for (int q = 0; q < m.n; ++q) {
    const SegFix& s = m.s[q];
    const int64_t slots = (s.r_k + s.n_ranges - 1) / s.n_ranges * ncols, per = 4 * kBlock / parts;
    m.range_blocks[q] = (int)((slots + per - 1) / per);
    m.cfirst[q + 1] = m.cfirst[q] + s.n_ranges * m.range_blocks[q];
  }
  const unsigned grid = (unsigned)m.cfirst[m.n];
#define ILARGI_COMBINE(C)                                                   \
  if (parts == 16) segfix_combine_kernel<C, 16><<<grid, kBlock, 0, st>>>(m); \
  else segfix_combine_kernel<C, 4><<<grid, kBlock, 0, st>>>(m);
  switch (ncols) {
    case 1: ILARGI_COMBINE(1) break;
    case 2: ILARGI_COMBINE(2) break;
    case 3: ILARGI_COMBINE(3) break;
    default: ILARGI_COMBINE(4) break;
  }
#undef ILARGI_COMBINE
  return hipGetLastError();
}

}  // namespace

namespace {

// How the sources of a launch share the workgroups of an XCD: ranges of source rows, and runs of target rows per XCD.
struct FixShare { int ranges[kSegMulti], nsub[kSegMulti], stride[kSegMulti]; double us; };

// A round (4096 rows of a run) takes longer the more of its rows a range holds, and a megabyte of the runs' sums costs a
// microsecond for every three: a workgroup more for the source with the longest runs, until none is left, and of these
// shares the best.
FixShare segfix_share(int64_t r_T, const int64_t* rows, int n, int ncols) {
  FixShare now, best;
  memset(&now, 0, sizeof(now));
  const int keys = kFixSlots / ncols;
  const int64_t blocks = (r_T / 4 + kFixThreads - 1) / kFixThreads;
  int items = 0;
  for (int q = 0; q < n; ++q) {
    now.ranges[q] = (int)((rows[q] + keys - 1) / keys);
    now.nsub[q] = 1;
    now.stride[q] = (int)((rows[q] + now.ranges[q] - 1) / now.ranges[q] * ncols + 3) / 4 * 4;
    items += now.ranges[q];
  }
  best = now;
  best.us = 1e30;
  for (;;) {
    double longest = 0.0, mb = 0.0;
    int at = -1;
    for (int q = 0; q < n; ++q) {
      const int64_t runs = (int64_t)kSegSlices * now.nsub[q];
      const double us = (double)((blocks + runs - 1) / runs) * 0.043 * (10.0 + 6.0 * (ncols - 1) + 13.0 * ncols / now.ranges[q]);
      if (us > longest) { longest = us; at = q; }
      mb += 4e-6 * (double)(now.ranges[q] * runs * now.stride[q]);
    }
    now.us = longest + 0.33 * mb;
    if (now.us < best.us) best = now;
    if (at < 0 || items + now.ranges[at] > kFixPerXcd) return best;
    items += now.ranges[at];
    ++now.nsub[at];
  }
}

}  // namespace

// Whether the segment sums of n sources with so many rows run in LDS or gather (cut: some segment would be summed in chunks by a
// launch of their own).  Both sides are estimates in microseconds, fitted to iterations over one to three joined tables.
// Keys in order gain by gathering and not here, so sums in LDS are taken where evenly spread keys gain more than those lose.
// Iterations, gathering / in LDS:
//   one model      1,000,000 rows  20,000 uniform keys              38 / 40     gathers
//                                  50,000 and 20,000                49 / 48     in LDS
//                                  twice 3000                       44 / 39     in LDS
//                  5,000,000 rows  20,000 uniform; in order         93 / 81; 77 / 79   in LDS
//                                  180,000 uniform                  110 / 110
//                                  100,000, 50,000 Zipf and 10,000  182 / 132   in LDS
//   two models     1,000,000 rows  twice 3000                       62 / 47     in LDS
//   three models   5,000,000 rows  three times 3000                 344 / 187   in LDS
//                                  100,000, 50,000 and 10,000       377 / 417   gathers: too many ranges
bool segfix_pays(int64_t r_T, const int64_t* rows, int n, int ncols, bool cut) {
  if (n < 1 || r_T < 100000 || n > kSegMulti) return false;
  int64_t ranges = 0;
  for (int q = 0; q < n; ++q) ranges += (rows[q] + kFixSlots / ncols - 1) / (kFixSlots / ncols);
  if (ranges > 20) return false;
  const double near = 1e-6 * n * (double)std::min<int64_t>(r_T, 1500000), far = 1e-6 * n * (double)std::max<int64_t>(r_T - 1500000, 0);
  const double gather = 7.2 * near + 4.9 * far + (ncols - 1) * (2.6 * near + 3.6 * far) + (cut ? 5.0 : 0.0) +
                        (r_T >= 1500000 ? std::max(0.0, 6.0 * n - 9.0) : 0.0);
  return 5.0 + segfix_share(r_T, rows, n, ncols).us < gather;
}

hipError_t launch_segfix(const SegFix* a, int n, int ncols, float* scratch, int64_t scratch_floats, hipStream_t st) {
  if (n < 1 || n > kSegMulti || ncols < 1 || ncols > kNarrowCT) return hipErrorInvalidValue;
  SegFixMulti m;
  memset(&m, 0, sizeof(m));
  m.n = n;
  int64_t at = 0;
  int slots = 0;
  int64_t rows[kSegMulti];
  bool aligned = true;
  for (int q = 0; q < n; ++q) {
    SegFix& s = m.s[q];
    s = a[q];
    if (s.idx == nullptr || s.Y == nullptr || s.r_k <= 0 || s.r_T < 4) return hipErrorInvalidValue;
    rows[q] = s.r_k;
    aligned = aligned && reinterpret_cast<uintptr_t>(s.Y) % 16 == 0 && reinterpret_cast<uintptr_t>(s.idx) % 16 == 0;
  }
  const FixShare share = segfix_share(a[0].r_T, rows, n, ncols);
  for (int q = 0; q < n; ++q) {
    SegFix& s = m.s[q];
    s.n_ranges = share.ranges[q]; s.nsub = share.nsub[q]; s.stride = share.stride[q];
    slots = std::max(slots, s.stride);
    int count = 1;
    s.runs = kSegSlices * s.nsub;
    const int64_t run = ((s.r_T + 4 * kFixThreads - 1) / (4 * kFixThreads) + s.runs - 1) / s.runs * (4 * kFixThreads);   // rows
    while (((int64_t)1 << count) <= run) ++count;
    s.bits = std::min(50, 62 - count);
    s.partial = scratch + at;
    at += (int64_t)s.n_ranges * kSegSlices * s.nsub * s.stride;
    m.first[q + 1] = m.first[q] + s.n_ranges * s.nsub;
  }
  if (at > scratch_floats) return hipErrorInvalidValue;
  const size_t lds = sizeof(u64) * (size_t)slots;
  const unsigned grid = (unsigned)m.first[n] * kSegSlices;
#define ILARGI_SEGFIX(C)                                                              \
  {                                                                                   \
    if (aligned) segfix_kernel<C, true><<<grid, kFixThreads, lds, st>>>(m);           \
    else segfix_kernel<C, false><<<grid, kFixThreads, lds, st>>>(m);                  \
  }
  switch (ncols) {
    case 1: ILARGI_SEGFIX(1) break;
    case 2: ILARGI_SEGFIX(2) break;
    case 3: ILARGI_SEGFIX(3) break;
    default: ILARGI_SEGFIX(4) break;
  }
#undef ILARGI_SEGFIX
  return launch_combine(m, ncols, st);
}

// Where the tables lie in the products and sums of a workgroup; the number of sums, or 0 if they do not fit.
static int asm_fix_places(const GatherArgs& g, int ncols, int (&off)[kAsmFixSources]) {
  if (g.n < 1 || g.n > kAsmFixSources) return 0;
  int64_t at = 0;
  for (int s = 0; s < g.n; ++s) {
    if (g.idx[s] == nullptr || g.rows[s] < 1 || g.rows[s] > kAsmFixSlots || g.rows[s] * g.ldp > (1 << 28)) return 0;
    off[s] = (int)at;
    at += (g.rows[s] + 4) / 4 * 4;                       // (a place for rows without a key)
  }
  return at * ncols <= kAsmFixSlots ? (int)at * ncols : 0;
}

bool asm_fix_supported(const LmmArgs& a, int mode) {
  int off[kAsmFixSources];
  for (int s = 0; s < a.g.n; ++s)
    if (reinterpret_cast<uintptr_t>(a.g.idx[s]) % 16 != 0) return false;
  return a.D == nullptr && reinterpret_cast<uintptr_t>(a.y) % 16 == 0 && (mode == 1 || mode == 2) && a.ncols >= 1 && a.ncols <= kNarrowCT && a.y != nullptr && a.loss_partial != nullptr &&
         a.r_out >= 4096 && a.r_out < 2147483647ll && asm_fix_places(a.g, a.ncols, off) > 0;
}

// Whether it pays: the more sums there are, the more rows it takes to make up for clearing and adding up the workgroups' copies.
// lines[s]: lines of a product that 64 target rows in a row read; keys in order (one or two lines) gather well, so they ask for
// more rows.  Iterations of one to four logistic models, separate launches / one: 1,000,000 rows over 300 keys 42 / 20, over 3000
// 31 / 23 (four models 55 / 40), over 12,000 32 / 27, over twice 6000 38 / 28, over 3000 in order 22 / 24; 300,000 over 3000
// 21 / 22, over twice 300 and more 24 / 19; 100,000 over 3000 19 / 20 (four models 24 / 29); 3,000,000 over three times 2000
// 74 / 33, over 3000 in order 38 / 27.
bool asm_fix_pays(const LmmArgs& a, const float* lines) {
  int64_t keys = 0;
  int in_order = 0;
  for (int s = 0; s < a.g.n; ++s) {
    keys += a.g.rows[s];
    in_order += lines[s] < 2.5f && a.g.rows[s] > 64 ? 1 : 0;
  }
  const int64_t rows = in_order == 0 ? 40 : in_order < a.g.n ? 100 : 700;
  return a.r_out >= 100000 && a.r_out >= rows * keys * a.ncols;
}

hipError_t launch_asm_fix(const LmmArgs& a, int mode, float* const* Z, float* scratch, int64_t scratch_floats, hipStream_t st, int* grid_out) {
  if (!asm_fix_supported(a, mode)) return hipErrorInvalidValue;
  AsmFix f;
  memset(&f, 0, sizeof(f));
  f.slots = asm_fix_places(a.g, a.ncols, f.off);
  f.n = a.g.n;
  f.ldp = a.g.ldp; f.col0 = a.col0;
  f.y = a.y; f.r_T = a.r_out; f.loss_partial = a.loss_partial; f.partial = scratch;
  SegFixMulti m;
  memset(&m, 0, sizeof(m));
  m.n = f.n;
  const int64_t units = a.r_out / 4;
  // (balances 0.9 microseconds a round of 4096 rows and workgroup, against 0.5 a megabyte of their sums)
  const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(std::min(256.0, sqrt(440.0 * (double)units / f.slots)),
                                                               (units + kFixThreads / 2 - 1) / (kFixThreads / 2)));
  if ((int64_t)grid * f.slots > scratch_floats) return hipErrorInvalidValue;
  for (int s = 0; s < f.n; ++s) {
    f.idx[s] = a.g.idx[s]; f.P[s] = a.g.P[s]; f.keys[s] = (int)a.g.rows[s];
    SegFix& z = m.s[s];
    z.r_k = a.g.rows[s]; z.n_ranges = 1; z.runs = grid; z.stride = f.slots;
    z.partial = scratch + (int64_t)f.off[s] * a.ncols;
    z.Z = Z[s]; z.ldz = a.g.ldp; z.zcol0 = a.col0;
  }
  int count = 1;
  while (((int64_t)1 << count) <= a.r_out / grid + 8) ++count;
  f.bits = std::min(50, 62 - count);
  if (grid_out) *grid_out = grid;
  const size_t lds = (size_t)f.slots * (sizeof(u64) + sizeof(float));
#define ILARGI_ASM_FIX(N, C)                                                \
  if (mode == 1) asm_fix_kernel<N, C, 1><<<grid, kFixThreads, lds, st>>>(f); \
  else asm_fix_kernel<N, C, 2><<<grid, kFixThreads, lds, st>>>(f);
#define ILARGI_ASM_FIX_CT(N)                \
  switch (a.ncols) {                        \
    case 1: ILARGI_ASM_FIX(N, 1) break;     \
    case 2: ILARGI_ASM_FIX(N, 2) break;     \
    case 3: ILARGI_ASM_FIX(N, 3) break;     \
    default: ILARGI_ASM_FIX(N, 4) break;    \
  }
  switch (f.n) {
    case 1: ILARGI_ASM_FIX_CT(1) break;
    case 2: ILARGI_ASM_FIX_CT(2) break;
    case 3: ILARGI_ASM_FIX_CT(3) break;
    default: ILARGI_ASM_FIX_CT(4) break;
  }
#undef ILARGI_ASM_FIX_CT
#undef ILARGI_ASM_FIX
  return launch_combine(m, a.ncols, st);
}

}  // namespace ilargi
