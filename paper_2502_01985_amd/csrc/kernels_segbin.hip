// Segment sums  Z_k = I_k^T Y  for one operand column over large target tables, summed in LDS in target-row order.
//
// The gathering forms of kernels_tmm.hip pay one L2 request per index entry, and a residual of megabytes does not stay
// in the 32 KB next to a compute unit: 265 G entries a second on this device, whatever the kernel looks like.  Here the
// residual is read in order, once per range of source rows, into LDS, and the entries are summed into LDS as well.
//
// The source rows (keys) of a table are split into ranges of at most 20480, the target rows into windows of 4096 to 16384
// rows.  A workgroup of 16 wavefronts serves one range over a run of windows: it stages a window of the residual, and every
// wavefront adds its entries of that window to its keys' sums.  An index entry is 32 bits: the row within the window, and
// the slot of the sum.  Every slot belongs to one wavefront, so a sum has a fixed order and needs no atomics (which would
// cost more than the gathers: ds_add_f32 takes 194 cycles a wavefront instruction on this device, a read and a write 14).
// Keys with more than 1/128 of their range's entries have one slot per wavefront, and bits of the target row say which
// takes an entry; the other keys are dealt to the wavefronts in runs of about the same number of entries.
// The runs of windows of XCD x lie in the x-th eighth of the target rows, so an XCD's L2 serves the residual to all ranges.
//
// 5,000,000 rows over 100,000 uniform, 50,000 Zipf and 10,000 uniform keys: 50 microseconds and 8 for the runs' sums
// (gathering, by slice of the target rows: 78 and 10); one such source alone 15 to 25 and 6 to 8.  Bound by instructions and
// LDS round trips: FETCH_SIZE is the index and the residual once (84 MB with three sources of 100,000 keys), 40
// instructions a group of 64 entries and 60 a window and wavefront.  Hence one workgroup per compute unit with all of its
// LDS: two with windows and ranges half as long took 54 where this takes 42 (three sources of 100,000 keys), eight
// wavefronts instead of 16 took 71 instead of 54.
#include <algorithm>
#include <cstring>
#include <vector>

#include "ilargi_internal.h"

namespace ilargi {

namespace {

constexpr int kBinThreads = kBinWaves * kWave;

// v moved across the lanes by a data-parallel primitive (no LDS); lanes without a source get 0.
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xf, true));
}
constexpr int kRowShr = 0x110, kWaveShr1 = 0x138, kRowBcast15 = 0x142, kRowBcast31 = 0x143;

__device__ __forceinline__ void add_where(float& v, uint64_t lanes, float t) { v += __builtin_amdgcn_inverse_ballot_w64(lanes) ? t : 0.0f; }

// Adds 64 entries to the sums of a wavefront: lane l holds entry e and its row v, lanes from `live` on none.  The entries
// of a group lie in order of their slot, so those of one slot are neighbours: they are summed across the lanes first and
// the last lane of a run adds the sum to its slot, no two lanes to the same.  Runs of up to four take two steps at most;
// longer ones (keys with many entries) the steps of a scan: within rows of 16 lanes, then from row to row.  The masks of
// lanes that take part in a step are scalars.
__device__ __forceinline__ void bin_add(uint32_t e, float v, int live, float* acc) {
  const uint32_t slot = e >> kBinRowBits;
  const uint32_t before = (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)slot, kWaveShr1, 0xf, 0xf, false);
  const uint64_t lanes = live >= kWave ? ~0ull : (1ull << live) - 1;
  const uint64_t n1 = __ballot(slot == before) & lanes;           // lanes whose slot is that of the lane below
  if (n1 != 0) {
    const uint64_t n2 = n1 & n1 << 1;                             // nd, md: ... and of the d lanes below (md: within the row)
    if ((n2 & n2 << 2) == 0) {
      add_where(v, n1, dpp<kWaveShr1>(v));
      if (n2 != 0) add_where(v, n2, dpp<kWaveShr1>(dpp<kWaveShr1>(v)));
    } else {
      constexpr uint64_t first = 0x0001000100010001ull;
      const uint64_t m1 = n1 & ~first, m2 = m1 & m1 << 1, m4 = m2 & m2 << 2, m8 = m4 & m4 << 4;
      add_where(v, m1, dpp<kRowShr + 1>(v));
      add_where(v, m2, dpp<kRowShr + 2>(v));
      add_where(v, m4, dpp<kRowShr + 4>(v));
      add_where(v, m8, dpp<kRowShr + 8>(v));
      uint64_t c = n1;                                            // lanes whose run reaches into the row before
      c &= c << 1 | first;
      c &= c << 2 | first * 3;
      c &= c << 4 | first * 15;
      c &= c << 8 | first * 255;
      add_where(v, c & 0xffff0000ffff0000ull, dpp<kRowBcast15, 0xa>(v));
      const uint64_t c32 = c & ((c >> 47 & 1) ? 0xffffffff00000000ull : 0x0000ffff00000000ull);
      add_where(v, c32, dpp<kRowBcast31, 0xc>(v));
    }
  }
  if (__builtin_amdgcn_inverse_ballot_w64(lanes & ~(n1 >> 1))) acc[slot] += v;
}

typedef float f4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

// `bytes` from p on as a buffer: loads past its end return zero without touching memory.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t bin_buffer(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}

// The sums of one workgroup over the windows [w0, w1).  Two windows are under way while one is summed, each in registers
// of its own; rows are requested as soon as the last ones are in LDS, entries as soon as the last ones are spent, so no
// register is copied while a load is under way, and no load of the loop is on one way of a branch only: either would make
// the compiler wait for all of them.
// U: groups of 64 entries a wavefront requests ahead (the array is padded for reading past its end); what a window has
// beyond them is loaded when it is its turn.
// ALIGNED: the operand starts on 16 bytes.
template <int RV, int U, bool ALIGNED>
__device__ __forceinline__ void segbin_windows_sum(const SegBin& a, const float* Y, const int32_t* off, int w0, int w1, float* win, float* acc) {
  constexpr int WIN = RV * kBinThreads;
  const int tid = (int)threadIdx.x, lane = tid % kWave;
  const uint32_t lane4 = (uint32_t)lane * 4, rT = (uint32_t)a.r_T;
  const char* entries = reinterpret_cast<const char*>(a.entries);
  const int n_win = a.n_win;
  float r0[RV], r1[RV];
  uint32_t e0[U], e1[U];
  int wb = w0;                                              // lane l holds off[wb + l]
  int offs = off[min(wb + lane, n_win)];
  __builtin_amdgcn_s_waitcnt(0x0f70);                       // vmcnt(0) here, not where the loop's ways meet
  auto entries_from = [&](int p, uint32_t (&e)[U]) {
    const char* base = entries + (int64_t)(uint32_t)p * 4;
#pragma unroll
    for (int u = 0; u < U; ++u) e[u] = *reinterpret_cast<const uint32_t*>(base + lane4 + u * kWave * 4);
  };
  auto rows_of = [&](int w, float (&r)[RV]) {
    const uint32_t t0 = (uint32_t)w * WIN;                  // (32 bits throughout, which scalar instructions compare)
    const uint32_t left = w < w1 ? min(rT - t0, (uint32_t)WIN) : 0u;
    const __amdgpu_buffer_rsrc_t rows = bin_buffer(Y + t0, left * 4u);
    // (all of an offset goes into the lane's: the scalar one has no part in the check against the buffer's length)
    if constexpr (ALIGNED) {
#pragma unroll
      for (int u = 0; u < RV / 4; ++u) {
        const u4 v = __builtin_amdgcn_raw_buffer_load_b128(rows, tid * 16 + u * kBinThreads * 16, 0, 0);
#pragma unroll
        for (int c = 0; c < 4; ++c) r[4 * u + c] = __uint_as_float(v[c]);
      }
    } else {
#pragma unroll
      for (int u = 0; u < RV; ++u)
        r[u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rows, (u / 4 * kBinThreads * 4 + u % 4 + tid * 4) * 4, 0, 0));
    }
  };
  int p0 = __builtin_amdgcn_readlane(offs, 0), p1 = __builtin_amdgcn_readlane(offs, 1), p2 = __builtin_amdgcn_readlane(offs, min(2, w1 - w0));
  auto step = [&](int w, float (&r)[RV], uint32_t (&e)[U]) {
#pragma unroll
    for (int u = 0; u < RV / 4; ++u) reinterpret_cast<f4*>(win)[u * kBinThreads + tid] = f4{r[4 * u], r[4 * u + 1], r[4 * u + 2], r[4 * u + 3]};
    if (w + 3 - wb >= kWave) {
      wb = w;
      offs = off[min(wb + lane, n_win)];
      __builtin_amdgcn_s_waitcnt(0x0f70);
    }
    const int p3 = __builtin_amdgcn_readlane(offs, min(w + 3, w1) - wb);
    __syncthreads();
    rows_of(w + 2, r);
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = win[e[u] & (WIN - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (p0 + u * kWave < p1) bin_add(e[u], v[u], p1 - (p0 + u * kWave), acc);
    for (int p = p0 + U * kWave; p < p1; p += kWave) {
      const uint32_t more = *reinterpret_cast<const uint32_t*>(entries + (int64_t)(uint32_t)p * 4 + lane4);
      __builtin_amdgcn_s_waitcnt(0x0f70);
      bin_add(more, win[more & (WIN - 1)], p1 - p, acc);
    }
    entries_from(p2, e);
    p0 = p1; p1 = p2; p2 = p3;
    __syncthreads();
  };
  rows_of(w0, r0);
  entries_from(p0, e0);
  rows_of(w0 + 1, r1);
  entries_from(p1, e1);
  int w = w0;
  for (; w + 1 < w1; w += 2) {                              // (both steps always: see above)
    step(w, r0, e0);
    step(w + 1, r1, e1);
  }
  if (w < w1) step(w, r0, e0);
}

// Run `sub` of the nsub runs of windows of XCD x.
struct BinRun { int w0, w1; };
__host__ __device__ __forceinline__ BinRun segbin_run(int n_win, int x, int sub, int nsub) {
  const int wx0 = (int)((int64_t)n_win * x / kSegSlices), wx1 = (int)((int64_t)n_win * (x + 1) / kSegSlices);
  return BinRun{wx0 + (int)((int64_t)(wx1 - wx0) * sub / nsub), wx0 + (int)((int64_t)(wx1 - wx0) * (sub + 1) / nsub)};
}

template <bool ALIGNED>
__global__ __launch_bounds__(kBinThreads, 4) void segbin_kernel(SegBinMulti m) {
  extern __shared__ float lds[];
  float* win = lds;                               // the residual of a window
  float* acc = lds + kBinWinFloats;               // the sums
  const int x = (int)blockIdx.x % kSegSlices, i = (int)blockIdx.x / kSegSlices;
  int q = 0;
  while (q + 1 < m.n && i >= m.first[q + 1]) ++q;
  const SegBin& a = m.s[q];
  BinItem it = a.items[i - m.first[q]];
  it.range = __builtin_amdgcn_readfirstlane(it.range); it.sub = __builtin_amdgcn_readfirstlane(it.sub);
  BinRange rg = a.ranges[it.range];
  rg.slots = __builtin_amdgcn_readfirstlane(rg.slots); rg.nsub = __builtin_amdgcn_readfirstlane(rg.nsub);
  const BinRun run = segbin_run(a.n_win, x, it.sub, rg.nsub);
  const int w0 = run.w0, w1 = run.w1;
  const int tid = (int)threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  for (int s = tid; s < rg.slots; s += kBinThreads) acc[s] = 0.0f;
  __syncthreads();
  if (w0 < w1) {
    const int32_t* off = a.off + (int64_t)(it.range * kBinWaves + wave) * (a.n_win + 1);
    if (a.win_log == 12) segbin_windows_sum<4, 5, ALIGNED>(a, a.Y, off, w0, w1, win, acc);
    else if (a.win_log == 13) segbin_windows_sum<8, 5, ALIGNED>(a, a.Y, off, w0, w1, win, acc);
    else segbin_windows_sum<16, 5, ALIGNED>(a, a.Y, off, w0, w1, win, acc);
  }
  float* out = a.partial + rg.partial0 + (int64_t)(x * rg.nsub + it.sub) * rg.slots;
  for (int s = tid; s < rg.slots; s += kBinThreads) out[s] = acc[s];
}

// Z[j] = the runs' sums of key j: a workgroup takes 32 keys of a range, eight threads a key add every eighth run each and
// their sums are added in order.  The last workgroups of a source serve the keys with a slot per wavefront, a wavefront each.
constexpr int kBinCombineKeys = 32, kBinCombineParts = kBlock / kBinCombineKeys;
__global__ __launch_bounds__(kBlock) void segbin_combine_kernel(SegBinMulti m) {
  __shared__ float part[kBlock];
  int q = 0;
  while (q + 1 < m.n && (int)blockIdx.x >= m.cfirst[q + 1]) ++q;
  const SegBin& a = m.s[q];
  const int b = (int)blockIdx.x - m.cfirst[q];
  const int key_blocks = a.n_ranges * m.range_blocks[q];
  float* Z = a.Z;
  if (b < key_blocks) {
    const int range = b / m.range_blocks[q];
    const BinRange rg = a.ranges[range];
    const int keys = (range + 1 < a.n_ranges ? a.ranges[range + 1].key0 : (int)a.r_k) - rg.key0;
    const int l = threadIdx.x % kBinCombineKeys, g = (int)threadIdx.x / kBinCombineKeys;
    const int s = (b - range * m.range_blocks[q]) * kBinCombineKeys + l;
    float z = 0.0f;
    if (s < keys) {
      const float* p = a.partial + rg.partial0 + s;
      const int nb = rg.nsub * kSegSlices;
      for (int c = g; c < nb; c += 8 * kBinCombineParts) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = c + u * kBinCombineParts < nb ? p[(c + u * kBinCombineParts) * rg.slots] : 0.0f;
#pragma unroll
        for (int u = 0; u < 8; ++u) z += v[u];
      }
    }
    part[threadIdx.x] = z;
    __syncthreads();
    if (g == 0 && s < keys && !(a.keyinfo[rg.key0 + s] & kBinHeavy)) {
      for (int c = 1; c < kBinCombineParts; ++c) z += part[c * kBinCombineKeys + l];
      Z[rg.key0 + s] = z;
    }
    return;
  }
  const int h = (b - key_blocks) * (kBlock / kWave) + (int)threadIdx.x / kWave, lane = threadIdx.x % kWave;
  if (h >= a.n_heavy) return;
  const int j = a.heavy[h];
  const uint32_t info = a.keyinfo[j];
  const BinRange rg = a.ranges[(info >> kBinSlotBits & 255) / kBinWaves];
  const float* p = a.partial + rg.partial0 + (info & ((1u << kBinSlotBits) - 1));
  const int n = rg.nsub * kSegSlices * kBinWaves;
  float z = 0.0f;
  for (int c = lane; c < n; c += 8 * kWave) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int k = c + u * kWave;
      v[u] = k < n ? p[k / kBinWaves * rg.slots + k % kBinWaves] : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) z += v[u];
  }
  for (int k = kWave / 2; k >= 1; k >>= 1) z += __shfl_xor(z, k);
  if (lane == 0) Z[j] = z;
}

// ---- the index, built with the plan ----
// Key of the sort: the wavefront (range x 16 + wavefront) an entry belongs to, above it the slot; rows without an entry last.
__global__ __launch_bounds__(kBlock) void bin_keys_kernel(const int32_t* __restrict__ idx, const uint32_t* __restrict__ keyinfo, int64_t r_T,
                                                          int32_t* __restrict__ keys, int32_t* __restrict__ rows) {
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < r_T; t += (int64_t)gridDim.x * blockDim.x) {
    const int32_t j = idx[t];
    uint32_t digit = 255, slot = 0;
    if (j >= 0) {
      const uint32_t info = keyinfo[j];
      digit = info >> kBinSlotBits & 255;
      slot = info & ((1u << kBinSlotBits) - 1);
      const uint32_t w = (uint32_t)t / kWave % kBinWaves;         // (not the low bits: those are the LDS bank of the row)
      if (info & kBinHeavy) { digit += w; slot += w; }
    }
    keys[t] = (int32_t)(digit | slot << 8);
    rows[t] = (int32_t)t;
  }
}

// off[d][w]: first entry of wavefront d with a target row in window w or later (digit_start[d nchunks]: its first entry).
__global__ __launch_bounds__(kBlock) void bin_offsets_kernel(const int32_t* __restrict__ rows, const int32_t* __restrict__ digit_start,
                                                             int nchunks, int n_digits, int n_win, int win_log,
                                                             int32_t* __restrict__ off) {
  const int64_t total = (int64_t)n_digits * (n_win + 1);
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int d = (int)(e / (n_win + 1)), w = (int)(e - (int64_t)d * (n_win + 1));
    const int64_t bound = (int64_t)w << win_log;
    int lo = digit_start[(int64_t)d * nchunks], hi = digit_start[(int64_t)(d + 1) * nchunks];   // (there are at most 240 of 256 digits)
    while (lo < hi) {
      const int mid = lo + (hi - lo) / 2;
      if ((int64_t)rows[mid] < bound) lo = mid + 1; else hi = mid;
    }
    off[e] = lo;
  }
}

// groups[range][w]: groups of 64 entries in window w of the wavefront of the range that has the most.
__global__ __launch_bounds__(kBlock) void bin_groups_kernel(const int32_t* __restrict__ off, int n_ranges, int n_win, int32_t* __restrict__ groups) {
  const int64_t total = (int64_t)n_ranges * n_win;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t range = e / n_win, w = e - range * n_win;
    int most = 0;
    for (int v = 0; v < kBinWaves; ++v) {
      const int32_t* o = off + (range * kBinWaves + v) * (n_win + 1) + w;
      most = max(most, (o[1] - o[0] + kWave - 1) / kWave);
    }
    groups[e] = most;
  }
}

// Packs the entries of every wavefront's windows, 64 at a time in order of their slot (a bitonic sort across the lanes).
__global__ __launch_bounds__(kBlock) void bin_pack_kernel(const int32_t* __restrict__ keys, const int32_t* __restrict__ rows,
                                                          const int32_t* __restrict__ off, int n_digits, int n_win, int win_log,
                                                          uint32_t* __restrict__ entries) {
  const int lane = threadIdx.x % kWave;
  const int64_t total = (int64_t)n_digits * n_win, waves = (int64_t)gridDim.x * (kBlock / kWave);
  for (int64_t l = (int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave; l < total; l += waves) {
    const int64_t o = l + l / n_win;                                       // off has n_win + 1 entries a wavefront
    const int p1 = off[o + 1];
    for (int p = off[o]; p < p1; p += kWave) {
      uint32_t e = 0xffffffffu;
      if (p + lane < p1) e = ((uint32_t)rows[p + lane] & ((1u << win_log) - 1)) | (uint32_t)keys[p + lane] >> 8 << kBinRowBits;
      for (int size = 2; size <= kWave; size <<= 1)
        for (int d = size >> 1; d >= 1; d >>= 1) {
          const uint32_t o2 = (uint32_t)__shfl_xor((int)e, d);
          const bool up = (lane & size) == 0, low = (lane & d) == 0;
          e = up == low ? min(e, o2) : max(e, o2);
        }
      if (p + lane < p1) entries[p + lane] = e;
    }
  }
}

}  // namespace

// Rows of a window: about 256 entries a wavefront, which it requests ahead, for tables of few ranges, and at least 24 windows
// an XCD, so that its workgroups share them evenly.
int segbin_win_log(int64_t r_T, int64_t rows) {
  const int n = segbin_ranges(rows);
  int log = n >= 4 ? 14 : n >= 2 ? 13 : 12;
  while (log > 12 && r_T < (int64_t)24 * kSegSlices << log) --log;
  return log;
}

int segbin_ranges(int64_t rows) { return (int)((rows + kBinKeys - 1) / kBinKeys); }

void segbin_layout(const std::vector<int32_t>& rowptr, SegBinPlan& plan) {
  std::vector<uint32_t>& keyinfo = plan.keyinfo;
  std::vector<int32_t>& heavy = plan.heavy;
  const int64_t rows = (int64_t)rowptr.size() - 1;
  const int n_ranges = segbin_ranges(rows);
  keyinfo.assign((size_t)rows, 0);
  for (int g = 0; g < n_ranges; ++g) {
    const int64_t k0 = rows * g / n_ranges, k1 = rows * (g + 1) / n_ranges;
    const int64_t entries = rowptr[(size_t)k1] - rowptr[(size_t)k0];
    int slots = (int)(k1 - k0);
    int64_t light = 0;
    for (int64_t k = k0; k < k1; ++k) {
      const int64_t len = rowptr[(size_t)k + 1] - rowptr[(size_t)k];
      if (len > entries / kBinHeavyShare && len > kWave) {
        keyinfo[(size_t)k] = (uint32_t)slots | (uint32_t)(g * kBinWaves) << kBinSlotBits | kBinHeavy;
        heavy.push_back((int32_t)k);
        slots += kBinWaves;
      } else {
        light += len;
      }
    }
    int64_t seen = 0, next = light / kBinWaves;                   // (a wavefront's keys start below its share of the entries)
    int wave = 0;
    for (int64_t k = k0; k < k1; ++k) {
      if (keyinfo[(size_t)k] & kBinHeavy) continue;
      while (wave + 1 < kBinWaves && seen >= next && light > 0) { ++wave; next = light * (wave + 1) / kBinWaves; }
      keyinfo[(size_t)k] = (uint32_t)(k - k0) | (uint32_t)(g * kBinWaves + wave) << kBinSlotBits;
      seen += rowptr[(size_t)k + 1] - rowptr[(size_t)k];
    }
    plan.ranges.push_back(BinRange{(int)k0, slots, 1, 0, (int)entries});
  }
}

namespace {

struct BinPart { BinRange* r; const int32_t* groups; double window; int windows, n_win, log; };

// Instructions of a wavefront in a window: its rows, and its groups of 64 entries.
double window_cost(int log, double groups) { return 60.0 + (1 << log) / 400.0 + 40.0 * groups; }

// Shares the workgroups of an XCD out to the ranges of the sources of a launch: one more run of windows for the range whose
// runs are the longest, until the XCD is full.
void segbin_share(std::vector<BinPart>& parts) {
  auto cost = [](const BinPart& p) { return p.window * ((p.windows + p.r->nsub - 1) / p.r->nsub); };
  const int room = ((int)parts.size() + kBinPerXcd - 1) / kBinPerXcd * kBinPerXcd;
  for (BinPart& p : parts) p.r->nsub = 1;
  for (int used = (int)parts.size(); used < room; ++used) {
    BinPart* most = nullptr;
    for (BinPart& p : parts)
      if (p.r->nsub < p.windows && (most == nullptr || cost(p) > cost(*most))) most = &p;
    if (most == nullptr) break;
    ++most->r->nsub;
  }
}

// Microseconds that the sources ks[0 .. n) gain by a launch in LDS over gathering.
// In LDS: the longest run of windows, had every wavefront of a workgroup the same number of entries in every window; what it
// is longer because they have not (then one wavefront works and its requests are not hidden: 13 microseconds per 1000
// instructions instead of 6), as where the rows of a key lie together; and the runs' sums, a microsecond per million.
// Gathering: the entries; keys of thousands of rows, which are summed in chunks; and the launch, unless another source takes
// one in any case.  All sources of a launch or none: where one gathers it costs the others little to join it (3,000,000 rows
// over 100,000 sorted and twice 20,000 keys: 122 with the two in LDS, 110 without).  Iterations of one model, gathering / in LDS:
//   5,000,000 rows   100,000, 50,000 and 10,000 uniform keys     205 / 175   in LDS
//                    180,000 uniform keys                        111 / 109   in LDS
//                    50,000 keys, the rows of each together       97 / 99    gathers
//                    30,000 sorted and 5000 uniform keys         105 / 645   gathers
//   2,000,000 rows   20,000, 50,000 or 180,000 uniform keys       51 / 53, 53 / 55, 58 / 63   gathers
//   1,500,000 rows   50,000 uniform keys; by a power law          47 / 52; 93 / 51            gathers; in LDS
//   1,000,000 rows   twice 20,000 or twice 3000 uniform keys      49 / 50; 43 / 41            gathers; in LDS
//                    30,000 slowly moving and 5000 uniform keys   48 / 100  gathers
//     500,000 rows   three times 60,000 or 3000 uniform keys      47 / 54; 39 / 38            gathers; in LDS
double segbin_gain(int64_t r_T, std::vector<SegBinPlan>& plans, const int* ks, int n) {
  std::vector<BinPart> parts;
  double gather = 0.0, launch = 0.0, chunks = 0.0;
  for (int q = 0; q < n; ++q) {
    SegBinPlan& s = plans[(size_t)ks[q]];
    const int64_t rows = (int64_t)s.keyinfo.size();
    const int log = segbin_win_log(r_T, rows), n_win = (int)segbin_windows(r_T, rows);
    for (size_t g = 0; g < s.ranges.size(); ++g) {
      BinRange& r = s.ranges[g];
      const double groups = std::max(1.0, r.entries / (double)n_win / kBinWaves / kWave + 0.5);
      parts.push_back(BinPart{&r, s.groups == nullptr ? nullptr : s.groups + g * (size_t)n_win, window_cost(log, groups),
                              std::max(1, n_win / kSegSlices), n_win, log});
    }
    gather += 6.2e-6 * (double)s.entries;
    if (!s.joins_launch) launch = 8.0;
    if (s.very_long) chunks = 10.0;
  }
  segbin_share(parts);
  double even = 0.0, longest = 0.0, sums = 0.0;
  for (const BinPart& p : parts) {
    sums += (double)p.r->nsub * kSegSlices * p.r->slots;
    for (int x = 0; x < kSegSlices; ++x)
      for (int sub = 0; sub < p.r->nsub; ++sub) {
        const BinRun run = segbin_run(p.n_win, x, sub, p.r->nsub);
        double c = p.window * (run.w1 - run.w0);
        even = std::max(even, c);
        if (p.groups != nullptr) {
          c = 0.0;
          for (int w = run.w0; w < run.w1; ++w) c += window_cost(p.log, p.groups[w]);
        }
        longest = std::max(longest, c);
      }
  }
  return gather + launch + chunks - (12.2 + 6e-3 * even + 13e-3 * std::max(longest - even, 0.0) + 1e-6 * sums);
}

}  // namespace

// Below these sizes the two launches cost more than the gathers: 250,000 rows and three tables 50 / 51 microseconds an
// iteration (gathering / in LDS), 500,000 and one 33 / 36, 1,000,000 and one 37..45 / 39..45.
bool segbin_enough(int64_t r_T, int n) { return n > 0 && (r_T >= 1500000 || (n >= 2 && r_T >= 500000 && n * r_T >= 1500000)); }

void segbin_choose(int64_t r_T, std::vector<SegBinPlan>& plans, std::vector<int>& in_bins) {
  for (bool again = true; again;) {
    again = false;
    if (!segbin_enough(r_T, (int)in_bins.size())) in_bins.clear();
    for (size_t i = 0; i < in_bins.size() && !again; i += kSegMulti) {       // (the sources of a launch, as they are called)
      const int n = (int)std::min<size_t>(kSegMulti, in_bins.size() - i);
      if (segbin_gain(r_T, plans, in_bins.data() + i, n) > 0.0) continue;
      in_bins.erase(in_bins.begin() + i, in_bins.begin() + i + n);
      for (int k : in_bins) plans[(size_t)k].joins_launch = true;
      again = true;
    }
  }
}

void segbin_items(std::vector<BinRange>& ranges, std::vector<BinItem>& items, int64_t* partial_floats) {
  int64_t partial = 0;
  for (size_t g = 0; g < ranges.size(); ++g) {
    ranges[g].partial0 = (int)partial;
    partial += (int64_t)ranges[g].nsub * kSegSlices * ranges[g].slots;
    for (int s = 0; s < ranges[g].nsub; ++s) items.push_back(BinItem{(int)g, s});
  }
  *partial_floats = partial;
}

hipError_t launch_build_segbin(const int32_t* idx, int64_t r_T, int64_t nnz, int n_ranges, int n_win, int win_log, const uint32_t* keyinfo,
                               int32_t* sortbuf, int64_t sort_n, int32_t* hist, int32_t* off, uint32_t* entries, int32_t* groups, hipStream_t st) {
  if (r_T <= 0) return hipSuccess;
  const int nchunks = (int)((r_T + kSortChunk - 1) / kSortChunk);
  int32_t* keys_a = sortbuf, *vals_a = sortbuf + sort_n, *keys_b = sortbuf + 2 * sort_n, *vals_b = sortbuf + 3 * sort_n;
  const int grid = (int)std::min<int64_t>((r_T + kBlock - 1) / kBlock, 8192);
  bin_keys_kernel<<<grid, kBlock, 0, st>>>(idx, keyinfo, r_T, keys_a, vals_a);
  hipError_t e = launch_radix_digit(keys_a, vals_a, r_T, keys_b, vals_b, hist, st);
  if (e != hipSuccess) return e;
  const int64_t n_off = (int64_t)n_ranges * kBinWaves * (n_win + 1);
  bin_offsets_kernel<<<(int)std::min<int64_t>((n_off + kBlock - 1) / kBlock, 8192), kBlock, 0, st>>>(vals_b, hist, nchunks, n_ranges * kBinWaves,
                                                                                                   n_win, win_log, off);
  const int64_t n_groups = (int64_t)n_ranges * n_win;
  bin_groups_kernel<<<(int)std::min<int64_t>((n_groups + kBlock - 1) / kBlock, 8192), kBlock, 0, st>>>(off, n_ranges, n_win, groups);
  if (nnz > 0) {
    const int64_t lists = (int64_t)n_ranges * kBinWaves * n_win;
    bin_pack_kernel<<<(int)std::min<int64_t>((lists + 3) / 4, 16384), kBlock, 0, st>>>(keys_b, vals_b, off, n_ranges * kBinWaves, n_win, win_log, entries);
  }
  return hipGetLastError();
}

hipError_t launch_segbin(const SegBin* a, int n, float* scratch, int64_t scratch_floats, hipStream_t st) {
  if (n < 1 || n > kSegMulti) return hipErrorInvalidValue;
  SegBinMulti m;
  memset(&m, 0, sizeof(m));
  m.n = n;
  int64_t at = 0;
  size_t slots = 0;
  bool aligned = true;
  for (int q = 0; q < n; ++q) {
    SegBin& s = m.s[q];
    s = a[q];
    if (s.entries == nullptr || s.r_k <= 0 || s.n_items <= 0) return hipErrorInvalidValue;
    s.partial = scratch + at;
    at += s.partial_floats;
    slots = std::max(slots, (size_t)s.max_slots);
    m.first[q + 1] = m.first[q] + s.n_items;
    m.range_blocks[q] = (int)((s.r_k + s.n_ranges - 1) / s.n_ranges + kBinCombineKeys - 1) / kBinCombineKeys;
    m.cfirst[q + 1] = m.cfirst[q] + s.n_ranges * m.range_blocks[q] + (s.n_heavy + kBlock / kWave - 1) / (kBlock / kWave);
    aligned = aligned && reinterpret_cast<uintptr_t>(s.Y) % 16 == 0;
  }
  if (at > scratch_floats) return hipErrorInvalidValue;
  const size_t lds = sizeof(float) * (kBinWinFloats + slots);
  const unsigned grid = (unsigned)m.first[n] * kSegSlices;
  if (aligned) segbin_kernel<true><<<grid, kBinThreads, lds, st>>>(m);
  else segbin_kernel<false><<<grid, kBinThreads, lds, st>>>(m);
  segbin_combine_kernel<<<(unsigned)m.cfirst[n], kBlock, 0, st>>>(m);
  return hipGetLastError();
}

}  // namespace ilargi
