// Assembly pass of the left multiply for ONE operand column over an identity source with short, 8-byte aligned rows
// (a number of columns that is 2 modulo 4, such as the 10-column entity table of the three-dimension benchmark), one
// lane per pair of target rows (the kernel is written for RPL rows per lane; RPL = 2 is what is built):
//   out[i] = D[i, :] x_D + sum_s P_s[row_idx_s[i]]                (paper, Sec. 2.2)
// with the residual and loss of Alg. 1 as epilogue (MODE 1 linear, MODE 2 logistic) and this workgroup's share of
// D^T e, the identity source's block of the gradient.
//
// A wavefront step covers 64 units (a unit = RPL consecutive rows = NV aligned float4): one contiguous run of
// memory that the wavefront reads as a flat stream of float4 (lane l takes float4 64 u + l: whole cache lines per
// instruction), writes to a private LDS tile and reads back transposed, lane l the NV float4 of unit l (a stride of
// NV float4 between lanes, conflict-free for the odd NV of 8-byte aligned rows).  From there on a row lives in one
// lane: the dot product with the operand (uniform values), the gathered product values, the epilogue and the
// gradient terms are plain per-lane arithmetic without partial sums through LDS or cross-lane exchange.
// The loop is branch-free for whole steps: every address is clamped to the table instead of guarded, lanes beyond the
// end contribute zeros, and only the store is predicated.  Requests run one step ahead (row indices two): at the top
// of a step everything it consumes was requested a whole step earlier (requesting the table rows two steps ahead
// measured the same).  Wavefronts are autonomous; the per-lane
// gradient and loss sums meet once, at the end, in a fixed order.
#include <algorithm>
#include <cstdint>
#include <cstring>
#include <mutex>

#include "ilargi_internal.h"

namespace ilargi {

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kLaneGather = 3;                 // gathered sources
constexpr int kLaneBlockWaves = kBlock / kWave;

__device__ __forceinline__ void lane_wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ float lane_uniform(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x)));
}

// The first n[s] products of source s in LDS, from float off[s] on.
struct LaneLds { int n[kLaneGather], off[kLaneGather]; };
constexpr int kLaneLdsWaves = 16, kLaneLdsBytes = 156 << 10;

// RPL rows per lane (1: rows of whole float4, 2: rows of an odd number of float2), NV float4 per unit.
// WAVES: wavefronts of a workgroup.  With kLaneLdsWaves of them a workgroup has a compute unit for itself, and what its LDS
// holds beside the tiles takes products of the smaller tables: a gather from there costs an eighteenth of one that goes to
// the L2, whose request rate bounds this kernel.  The lanes that find theirs in LDS request the first product of the table
// instead, one line for all of them.  5,000,000 x 10 with three joined tables of 100,000, 50,000 and 10,000 rows, all of the
// last and 9,456 products of the second in LDS (19,456 are room beside tiles of 10 columns, 27,648 beside 6): 81 microseconds,
// 89 without.
template <int RPL, int NV, int MODE, bool NT, int WAVES>
__global__ __launch_bounds__(WAVES * kWave) void lmm_lane_kernel(LmmArgs a, LaneLds pl) {
  constexpr int CK = 4 * NV / RPL;                              // columns of the table
  constexpr int kLaneWaves = WAVES;
  constexpr bool LDSP = WAVES == kLaneLdsWaves;
  extern __shared__ v4f lds4[];
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  v4f* tile = lds4 + (size_t)wave * kWave * NV;

  float w[CK];                                                  // operand values, the same in every lane
#pragma unroll
  for (int j = 0; j < CK; ++j) {
    const int t = a.colmap[j];
    w[j] = lane_uniform(t >= 0 ? a.X[(int64_t)t * a.ldx + a.col0] : 0.0f);
  }
  const int ng = a.g.n;
  const int32_t* gidx[kLaneGather];
  const float* gP[kLaneGather];
#pragma unroll
  for (int s = 0; s < kLaneGather; ++s) {
    gidx[s] = s < ng ? a.g.idx[s] : nullptr;
    gP[s] = s < ng ? a.g.P[s] + a.col0 : nullptr;
  }
  const int64_t ldp = a.g.ldp;
  const int64_t nunits = a.r_out / RPL;                         // r_out is a multiple of RPL
  const int64_t nchunks = (nunits + kWave - 1) / kWave;
  const int64_t last_f4 = nunits * NV - 1;
  const v4f* D4 = reinterpret_cast<const v4f*>(a.D);
  const int64_t cstride = (int64_t)gridDim.x * kLaneWaves;
  int64_t chunk = (int64_t)blockIdx.x * kLaneWaves + wave;

  auto load_rows = [&](int64_t ch, v4f (&dst)[NV]) {
    const int64_t base = ch * (kWave * NV) + lane;
#pragma unroll
    for (int u = 0; u < NV; ++u) {
      const v4f* p = D4 + min(base + u * kWave, last_f4);
      if constexpr (NT) dst[u] = __builtin_nontemporal_load(p);
      else dst[u] = *p;
    }
  };
  auto load_idx = [&](int64_t ch, int (&j)[kLaneGather][RPL]) {
    const int64_t unit = min(ch * kWave + lane, nunits - 1);
#pragma unroll
    for (int s = 0; s < kLaneGather; ++s) {
#pragma unroll
      for (int h = 0; h < RPL; ++h) j[s][h] = -1;
      if (s < ng) {
        if constexpr (RPL == 2) {
          const int2 t = *reinterpret_cast<const int2*>(gidx[s] + 2 * unit);
          j[s][0] = t.x; j[s][1] = t.y;
        } else {
          j[s][0] = gidx[s][unit];
        }
      }
    }
  };
  auto load_y = [&](int64_t ch, float (&y)[RPL]) {
    if constexpr (MODE != 0) {
      const int64_t unit = min(ch * kWave + lane, nunits - 1);
      if constexpr (RPL == 2) {
        const float2 t = *reinterpret_cast<const float2*>(a.y + 2 * unit);
        y[0] = t.x; y[1] = t.y;
      } else {
        y[0] = a.y[unit];
      }
    } else {
#pragma unroll
      for (int h = 0; h < RPL; ++h) y[h] = 0.0f;
    }
  };
  const float* prod = reinterpret_cast<const float*>(lds4 + (size_t)WAVES * kWave * NV);
  // a missing key reads row 0; its value is dropped when it is used, like that of a product that is in LDS
  auto gather = [&](const int (&j)[kLaneGather][RPL], float (&p)[kLaneGather][RPL]) {
#pragma unroll
    for (int s = 0; s < kLaneGather; ++s) {
#pragma unroll
      for (int h = 0; h < RPL; ++h) p[s][h] = 0.0f;
      if (s < ng) {
#pragma unroll
        for (int h = 0; h < RPL; ++h) {
          const int row = LDSP && j[s][h] < pl.n[s] ? 0 : max(j[s][h], 0);
          p[s][h] = gP[s][(int64_t)row * ldp];
        }
      }
    }
  };

  float gacc[CK];
#pragma unroll
  for (int j = 0; j < CK; ++j) gacc[j] = 0.0f;
  float loss_local = 0.0f, loss_lost = 0.0f;

  v4f vn[NV];
  int jc[kLaneGather][RPL], jn[kLaneGather][RPL];
  float pn[kLaneGather][RPL], yn[RPL];
  load_idx(chunk, jc);
  load_rows(chunk, vn);
  load_y(chunk, yn);
  load_idx(chunk + cstride, jn);
  gather(jc, pn);
  if constexpr (LDSP) {
    float* to = reinterpret_cast<float*>(lds4 + (size_t)WAVES * kWave * NV);
#pragma unroll
    for (int s = 0; s < kLaneGather; ++s)
      if (s < ng)
        for (int k = tid; k < pl.n[s]; k += WAVES * kWave) to[pl.off[s] + k] = gP[s][(int64_t)k * ldp];
    __syncthreads();
  }
  for (; chunk < nchunks; chunk += cstride) {
    // this step's values (all requested a step ago) leave the request registers
    float pc[kLaneGather][RPL], yc[RPL];
#pragma unroll
    for (int s = 0; s < kLaneGather; ++s)
#pragma unroll
      for (int h = 0; h < RPL; ++h) {
        float v = pn[s][h];
        if constexpr (LDSP) {
          const bool in = (uint32_t)jc[s][h] < (uint32_t)pl.n[s];       // (not a missing key, whose place may be past the end)
          const float w = prod[in ? pl.off[s] + jc[s][h] : 0];
          v = in ? w : v;
        }
        pc[s][h] = jc[s][h] >= 0 ? v : 0.0f;
      }
#pragma unroll
    for (int h = 0; h < RPL; ++h) yc[h] = yn[h];
    lane_wave_sync();                                           // the previous step's tile is consumed
#pragma unroll
    for (int u = 0; u < NV; ++u) tile[u * kWave + lane] = vn[u];
    lane_wave_sync();
    // the next step's requests
#pragma unroll
    for (int s = 0; s < kLaneGather; ++s)
#pragma unroll
      for (int h = 0; h < RPL; ++h) jc[s][h] = jn[s][h];
    gather(jc, pn);
    load_y(chunk + cstride, yn);
    load_idx(chunk + 2 * cstride, jn);
    load_rows(chunk + cstride, vn);
    // lane = unit
    float f[4 * NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const v4f t = tile[lane * NV + k];
      f[4 * k] = t[0]; f[4 * k + 1] = t[1]; f[4 * k + 2] = t[2]; f[4 * k + 3] = t[3];
    }
    const int64_t unit = chunk * kWave + lane;
    const bool live = unit < nunits;
    float r[RPL];
#pragma unroll
    for (int h = 0; h < RPL; ++h) {
      float z0 = 0.0f, z1 = 0.0f;                               // two chains
#pragma unroll
      for (int j = 0; j < CK; j += 2) {
        z0 = fmaf(f[h * CK + j], w[j], z0);
        if (j + 1 < CK) z1 = fmaf(f[h * CK + j + 1], w[j + 1], z1);
      }
      float zz = z0 + z1;
#pragma unroll
      for (int s = 0; s < kLaneGather; ++s) zz += pc[s][h];
      if constexpr (MODE == 0) {
        r[h] = zz;
      } else if constexpr (MODE == 1) {
        r[h] = live ? zz - yc[h] : 0.0f;
        loss_local = fmaf(r[h], r[h], loss_local);
      } else {
        float loss = 0.0f;
        r[h] = logistic_residual(zz, yc[h], loss);
        if (!live) r[h] = loss = 0.0f;
        const float add = loss - loss_lost, sum = loss_local + add;   // compensated: with zero weights every row adds log 2,
        // and the roundings of a lane's sum all go one way; what is infinite stays so
        loss_lost = fabsf(sum) <= __FLT_MAX__ ? (sum - loss_local) - add : 0.0f;
        loss_local = sum;
      }
    }
    if (live) {
      float* op = a.out + unit * RPL * a.ldo + a.col0;
      if (a.ldo == 1 && RPL == 2) {
        typedef float v2f __attribute__((ext_vector_type(2)));
        const v2f t = {r[0], r[RPL - 1]};
        if (a.nt_out) __builtin_nontemporal_store(t, reinterpret_cast<v2f*>(op));
        else *reinterpret_cast<v2f*>(op) = t;
      } else {
#pragma unroll
        for (int h = 0; h < RPL; ++h) {
          if (a.nt_out) __builtin_nontemporal_store(r[h], op + (int64_t)h * a.ldo);
          else op[(int64_t)h * a.ldo] = r[h];
        }
      }
    }
    if constexpr (MODE != 0) {
#pragma unroll
      for (int h = 0; h < RPL; ++h)
#pragma unroll
        for (int j = 0; j < CK; ++j) gacc[j] = fmaf(f[h * CK + j], r[h], gacc[j]);
    }
  }

  if constexpr (MODE != 0) {
    // lanes by a fixed butterfly, then the wavefronts in order
    __syncthreads();
    float* red = reinterpret_cast<float*>(lds4);               // [waves][CK + 1]
#pragma unroll
    for (int j = 0; j <= CK; ++j) {
      float s = j < CK ? gacc[j < CK ? j : 0] : loss_local;
      for (int m = kWave / 2; m >= 1; m >>= 1) s += __shfl_xor(s, m);
      if (lane == 0) red[wave * (CK + 1) + j] = s;
    }
    __syncthreads();
    if (tid <= CK) {
      float part[4] = {0.0f, 0.0f, 0.0f, 0.0f};                  // (four at a time: sixteen in a row would round more often)
#pragma unroll
      for (int wv = 0; wv < kLaneWaves; ++wv) part[wv / 4] += red[wv * (CK + 1) + tid];
      const float s = (part[0] + part[1]) + (part[2] + part[3]);
      if (tid < CK) a.grad_partial[((int64_t)blockIdx.x * CK + tid) * kNarrowCT] = s;
      else a.loss_partial[(int64_t)blockIdx.x * kNarrowCT] = s;
    }
  }
}

typedef void (*LaneFn)(LmmArgs, LaneLds);

template <int RPL, int NV, bool NT>
LaneFn pick_lane(int mode, bool in_lds) {
  if constexpr (NT && NV <= 5)
    if (in_lds) return mode == 1 ? lmm_lane_kernel<RPL, NV, 1, NT, kLaneLdsWaves> : lmm_lane_kernel<RPL, NV, 2, NT, kLaneLdsWaves>;
  return mode == 0 ? lmm_lane_kernel<RPL, NV, 0, NT, kLaneBlockWaves>
                   : (mode == 1 ? lmm_lane_kernel<RPL, NV, 1, NT, kLaneBlockWaves> : lmm_lane_kernel<RPL, NV, 2, NT, kLaneBlockWaves>);
}

// Built for rows of 6, 10 and 14 columns (pairs of 8-byte aligned rows).  For rows of whole float4 the same kernel
// (RPL = 1) measured 2 us faster than the flat-stream assembly on tables that sit in the last-level cache and 2 us
// slower on tables that come from memory, so those keep the flat-stream kernel.
LaneFn lane_fn(int rpl, int nv, int mode, bool nt, bool in_lds = false) {
  if (rpl != 2) return nullptr;
  switch (nv) {
    case 3: return nt ? pick_lane<2, 3, true>(mode, in_lds) : pick_lane<2, 3, false>(mode, in_lds);
    case 5: return nt ? pick_lane<2, 5, true>(mode, in_lds) : pick_lane<2, 5, false>(mode, in_lds);
    case 7: return nt ? pick_lane<2, 7, true>(mode, in_lds) : pick_lane<2, 7, false>(mode, in_lds);
    default: return nullptr;
  }
}

int lane_slots(LaneFn fn, size_t lds_bytes, int threads) {
  static std::mutex cache_mutex;
  std::lock_guard<std::mutex> lock(cache_mutex);
  static LaneFn seen_fn[64];
  static int seen_slots[64];
  static int n_seen = 0;
  for (int i = 0; i < n_seen; ++i)
    if (seen_fn[i] == fn) return seen_slots[i];
  int dev = 0, cus = 256, per_cu = 0;
  hipDeviceProp_t prop;
  if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess && prop.multiProcessorCount > 0)
    cus = prop.multiProcessorCount;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(fn), threads, lds_bytes) != hipSuccess ||
      per_cu < 1)
    per_cu = 1;
  if (n_seen < 64) { seen_fn[n_seen] = fn; seen_slots[n_seen] = per_cu * cus; ++n_seen; }
  return per_cu * cus;
}

void lane_shape(const LmmArgs& a, int vec, int* rpl, int* nv) {
  *rpl = (vec == 2 && a.ck % 4 == 2) ? 2 : 1;
  *nv = *rpl * a.ck / 4;
}

// The products a workgroup of kLaneLdsWaves wavefronts keeps in LDS beside its tiles, the smallest tables first.
LaneLds lane_lds(const LmmArgs& a, int nv) {
  LaneLds pl;
  memset(&pl, 0, sizeof(pl));
  int order[kLaneGather];
  for (int s = 0; s < a.g.n; ++s) order[s] = s;
  std::sort(order, order + a.g.n, [&](int x, int y) { return a.g.rows[x] < a.g.rows[y]; });
  int at = 0;
  for (int i = 0; i < a.g.n; ++i) {
    const int s = order[i], room = kLaneLdsBytes / 4 - kLaneLdsWaves * kWave * nv * 4 - at;
    pl.n[s] = (int)std::min<int64_t>(a.g.rows[s], room);
    pl.off[s] = at;
    at += pl.n[s];
  }
  return pl;
}

}  // namespace

bool lmm_lane_wants_lines(int64_t rows, int64_t cols) { return (cols == 6 || cols == 10) && stream_past_caches(rows * cols) != 0; }

// Whether products in LDS pay: with a residual (without one the chip holds more wavefronts), rows of 6 or 10 columns (wider ones
// would spill registers), an entity table that is read past the caches, and gathers that go to many lines: what 64 target rows
// in a row read beyond 30 lines, weighted with the part of the table in LDS, has to be a quarter of the most there could be.
// Iterations in microseconds, without / with, 5,000,000 x 10 and one table of 20,000 rows: uniform keys (61 lines) 94 / 86, by a
// power law whose first key has a fifth of the rows (48) 98 / 94, in blocks of 1000 (28) 99 / 102, sorted (1) 84 / 90; 38,000
// uniform keys, half of them in LDS, 97 / 96; 300 keys (10) 78 / 79.  By rows, uniform keys: 3,400,000 75.5 / 71.4; read through
// the caches 3,000,000 64.7 / 67.2, 1,000,000 38.3 / 41.7; three tables 5,000,000 174.9 / 166.2, 3,400,000 135.5 / 132.3; through
// the caches 3,000,000 129.8 / 127.3, 1,000,000 77.3 / 79.9.
bool lmm_lane_lds_pays(const LmmArgs& a, const float* lines) {
  if (a.D == nullptr || a.nt_in == 0 || !lmm_lane_wants_lines(a.d_rows, a.ck) || a.g.n < 1 || a.g.n > kLaneGather) return false;
  const LaneLds pl = lane_lds(a, a.ck / 2);
  double gain = 0.0;
  for (int s = 0; s < a.g.n; ++s)
    if (a.g.rows[s] > 0) gain += std::max(lines[s] - 30.0, 0.0) / (kWave - 30) * pl.n[s] / (double)a.g.rows[s];
  return gain >= 0.25;
}

// One operand column; the identity source covers every target row (d_rows == r_out, an even number); rows of 6, 10
// or 14 columns (vec 2) on a 16-byte aligned base; one to three
// sources gathered through row indices (8-byte aligned when a lane takes two rows); with a gradient-descent mode the
// fused gradient is part of the kernel.
bool lmm_lane_supported(const LmmArgs& a, int vec, int mode, bool fuseg) {
  if (a.D == nullptr || a.ncols != 1 || a.g.n < 1 || a.g.n > kLaneGather || a.r_out <= 0 || a.d_rows != a.r_out) return false;
  if ((mode != 0) != fuseg) return false;
  if (mode != 0 && (a.y == nullptr || a.loss_partial == nullptr || a.grad_partial == nullptr)) return false;
  if (reinterpret_cast<uintptr_t>(a.D) % 16 != 0) return false;
  if (!((vec == 4 && a.ck % 4 == 0) || (vec == 2 && a.ck % 4 == 2))) return false;
  int rpl, nv;
  lane_shape(a, vec, &rpl, &nv);
  if (lane_fn(rpl, nv, mode, a.nt_in != 0) == nullptr || a.r_out % rpl != 0) return false;
  for (int s = 0; s < a.g.n; ++s) {
    if (a.g.idx[s] == nullptr) return false;
    if (rpl == 2 && reinterpret_cast<uintptr_t>(a.g.idx[s]) % 8 != 0) return false;
  }
  if (rpl == 2 && mode != 0 && reinterpret_cast<uintptr_t>(a.y) % 8 != 0) return false;
  if (rpl == 2 && a.ldo == 1 && reinterpret_cast<uintptr_t>(a.out + a.col0) % 8 != 0) return false;
  return true;
}

hipError_t launch_lmm_lane(const LmmArgs& a, int vec, int mode, hipStream_t st, int* grid_out) {
  if (grid_out) *grid_out = 0;
  if (!lmm_lane_supported(a, vec, mode, mode != 0)) return hipErrorInvalidValue;
  int rpl, nv;
  lane_shape(a, vec, &rpl, &nv);
  const bool in_lds = mode != 0 && a.lds_products != 0 && rpl == 2 && nv <= 5;
  LaneLds pl;
  memset(&pl, 0, sizeof(pl));
  if (in_lds) pl = lane_lds(a, nv);
  const int waves = in_lds ? kLaneLdsWaves : kLaneBlockWaves;
  LaneFn fn = lane_fn(rpl, nv, mode, a.nt_in != 0, in_lds);
  size_t lds_bytes = (size_t)waves * kWave * nv * sizeof(v4f);
  lds_bytes = std::max(lds_bytes, (size_t)waves * (a.ck + 1) * sizeof(float));
  if (in_lds) lds_bytes = kLaneLdsBytes;
  const int64_t nchunks = (a.r_out / rpl + kWave - 1) / kWave;
  int64_t grid = (nchunks + waves - 1) / waves;
  int64_t cap = lane_slots(fn, lds_bytes, waves * kWave);
  if (mode != 0) cap = std::min<int64_t>(cap, kColredBlocks);
  if (grid > cap) grid = cap;
  if (grid_out) *grid_out = (int)grid;
  hipLaunchKernelGGL(fn, dim3((unsigned)grid), dim3((unsigned)(waves * kWave)), lds_bytes, st, a, pl);
  return hipGetLastError();
}

}  // namespace ilargi
