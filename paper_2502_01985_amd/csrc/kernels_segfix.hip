// Segment sums  Z_k = I_k^T Y  of one to four operand columns over large target tables, summed in LDS in fixed point, in
// target-row order; and the assembly of gathered products alone with the segment sums of its residual.
//
// The gathering forms of kernels_tmm.hip pay one L2 request per index entry and operand: 265 G entries a second on this device,
// whatever the kernel looks like.  Here a workgroup of 16 wavefronts holds the sums of a range of source rows (at most 20,160
// of 64 bits) in LDS, walks its share of the target rows in order and adds every row whose key lies in its range: row indices
// and operand are plain streams, and no inverse index is read or kept.  Sums are 64-bit integers: ds_add_u64 takes 13 cycles a
// wavefront instruction with 64 different places (ds_add_f64 22, ds_add_f32 194 on this device), returns nothing that anyone
// waits for, and whole numbers add up to the same in any order, so the result is the same on every run.
//
// A value is either added exactly or kept aside, so every sum is as accurate as it is by itself, whatever other keys and columns
// hold.  A run has a unit for every column, a power of two: sums of up to 2^n rows leave 62 - n bits (at most 50) for a value, and
// a float in the upper 62 - n - 24 binades of these is a whole number of units.  What is typical of the largest of the run's first
// rows lies two binades below their top.  Each wavefront lists what is outside, in LDS and then in memory.  Short lists (one value
// in 100,000 is outside where all are of one kind) are added in doubles to their sums on the way out; longer ones are walked like
// rows, with a unit for the largest that is left; where they have no room, the rows are walked again.  A sum is rounded to float
// once for every walk that found values of its own.  Infinities and NaN are listed as they are, or added in a walk of their own.
//
// 5,000,000 rows over 100,000 uniform, 50,000 Zipf and 10,000 uniform keys: 32 microseconds and 6 for the runs' sums (with an
// index by windows, float sums that belong to one wavefront each, 51 and 8; gathering, by slice of the target rows, 78 and 10).
// Bound by instructions: nine ranges look at 5,000,000 rows each, about ten vector instructions a row, two of them in 64 bits.
// Four blocks a thread requested at once instead of two, or the conversion ahead of the test for the range (42), gain nothing.
// T^T Y with these tables takes 47 microseconds for normal or constant values, nine tenths zeros or single outliers (57 through
// the index by windows, whatever the values), 56 for Cauchy values, 92 where one value in 70 is far below the others (logistic
// functions of N(0, 64)), 100 for lognormal values (sigma 3) and 616 where values spread evenly over 200 binades (12 walks).
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

constexpr int kFixWaves = kFixThreads / kWave;

__device__ __forceinline__ uint32_t magnitude(float v) { return __float_as_uint(v) & 0x7fffffffu; }
constexpr uint32_t kFixInf = 0x7f800000u;

// What earlier walks have summed, by column: magnitudes of the first walk's band, and finite ones from `done` up.  (In LDS.)
// down: the walk's unit.
struct Summed { double down; uint32_t low, high, done; };
struct Left { uint32_t largest, others; };

// What the kernels of up to four operand columns hold in LDS beside their sums (loss: the assembly's), and that there is room for it.
constexpr size_t lds_beside(bool loss) {
  const size_t column = sizeof(uint32_t) * kFixWaves + sizeof(Summed) + sizeof(Left) + (loss ? sizeof(float) * kFixWaves : 0);
  return (sizeof(u64) * kFixWaves * kFixNear + sizeof(uint32_t) * (kFixWaves + 1) + kNarrowCT * column + 15) / 16 * 16;
}
static_assert(lds_beside(false) + sizeof(u64) * kFixSlots <= 160 * 1024, "sums in LDS");
static_assert(lds_beside(true) + (sizeof(u64) + sizeof(float)) * kAsmFixSlots <= 160 * 1024, "sums and products in LDS");

// The magnitudes that a walk sums, by column: [low, low + span), multiples of the unit, 1 / up.
template <int CT>
struct Bands {
  uint32_t low[CT], span[CT];
  double up[CT];

  // [2^(top - bits + 23), 2^top): the unit is 2^(top - bits); down to the smallest float where that is a multiple.
  __device__ __forceinline__ void set(int c, int top, int bits) {
    up[c] = __longlong_as_double((long long)(bits - top + 1023) << 52);
    const int field = top - bits + 23 + 127;
    low[c] = field <= 0 ? 1u : (uint32_t)field << 23;
    span[c] = ((uint32_t)min(top + 127, 255) << 23) - low[c];
  }
  static __device__ __forceinline__ int above(uint32_t largest) { return max((int)(largest >> 23), 1) - 126; }   // largest < 2^above
  // (a column that begins with nothing but zeros is taken for one of values about one)
  __device__ __forceinline__ void first(int c, uint32_t largest, int bits, Summed* summed) {
    set(c, (largest == 0 ? 1 : above(largest)) + kFixHead, bits);
    summed[c].down = down(c);
  }
  // The walk after this one: for the largest that is left (0: none).
  __device__ __forceinline__ void next(int c, uint32_t largest, int bits, Summed* summed) {
    Summed was = summed[c];
    if (was.done == kFixInf) { was.low = low[c]; was.high = low[c] + span[c]; }
    if (largest == 0) {
      low[c] = was.done = 1u;
      span[c] = 0;
    } else {
      set(c, above(largest), bits);
      const uint32_t high = low[c] + span[c];
      if (largest >= was.high) low[c] = max(low[c], was.high);
      span[c] = (largest >= was.high ? high : min(high, was.low)) - low[c];
      was.done = low[c];
    }
    was.down = down(c);
    __syncthreads();                                     // (all threads have read)
    summed[c] = was;
  }
  // (twice the distance from the low end; twice the span and more is outside)
  __device__ __forceinline__ uint32_t offset(float v, int c) const { return (__float_as_uint(v) << 1) - (low[c] << 1); }
  __device__ __forceinline__ bool outside(float v, int c) const { return offset(v, c) >= span[c] << 1; }
  // Whether some of N values a thread and column are outside and not zero, in any lane.
  template <int N, class Value>
  __device__ __forceinline__ bool some_outside(Value value) const {
    uint32_t off[CT];
    bool any = false;
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      off[c] = 0;
#pragma unroll
      for (int i = 0; i < N; ++i) off[c] = max(off[c], offset(value(i, c), c));
      any = any || off[c] >= span[c] << 1;
    }
    if (__builtin_expect(__ballot(any) == 0, 1)) return false;
    // (zeros come behind what is above the band, and before what is below)
    any = false;
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      uint32_t most = 0;
#pragma unroll
      for (int i = 0; i < N; ++i) most = max(most, __float_as_uint(value(i, c)) << 1);
      any = any || off[c] > 0u - (low[c] << 1) || most >= (low[c] + span[c]) << 1;
    }
    return __ballot(any) != 0;
  }
  __device__ __forceinline__ double down(int c) const { return __longlong_as_double((2046ll << 52) - __double_as_longlong(up[c])); }
};

// The state in LDS before the first walk.
template <int CT>
__device__ __forceinline__ void none_summed(Summed* summed, Left* left, uint32_t* counts) {
  if (threadIdx.x <= kFixWaves) counts[threadIdx.x] = 0;
  if (threadIdx.x < CT) {
    summed[threadIdx.x].low = summed[threadIdx.x].high = 1;
    summed[threadIdx.x].done = kFixInf;
    left[threadIdx.x] = Left{0, 0};
  }
}

// Of a value outside the band: whether it is still to be summed.
__device__ __forceinline__ bool still_left(float v, const Summed& s) {
  const uint32_t b = __float_as_uint(v) & 0x7fffffffu;
  return b != 0 && b - s.low >= s.high - s.low && (b < s.done || b >= kFixInf);
}

// The values that a wavefront has kept aside, sum << 32 | value: kFixNear of them in LDS, up to `room` more in memory.
struct Strays {
  u64* near;
  u64* far;
  uint32_t room, n;                                      // (lanes that are out of rows keep an older n; lane 0 is the last of them)

  // Lanes with `is`; whether their value found no room.
  __device__ __forceinline__ bool add(bool is, uint32_t slot, float v) {
    const uint64_t m = __ballot(is);
    if (m == 0) return false;
    const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, n));
    const u64 entry = (u64)slot << 32 | __float_as_uint(v);
    if (is && at < kFixNear) near[at] = entry;
    else if (is && at - kFixNear < room) far[at - kFixNear] = entry;
    n += (uint32_t)__popcll(m);
    return is && at >= kFixNear + room;
  }
};

// v moved across the lanes of a wavefront without LDS; lanes without a source get 0.
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ uint32_t dpp(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, true);
}
constexpr int kRowShr = 0x110, kRowRor = 0x120, kRowBcast15 = 0x142, kRowBcast31 = 0x143;

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

// Largest of sixteen lanes' values, in all of them.
__device__ __forceinline__ uint32_t largest_of_row(uint32_t v) {
  v = max(v, dpp<kRowRor + 1>(v));
  v = max(v, dpp<kRowRor + 2>(v));
  v = max(v, dpp<kRowRor + 4>(v));
  return max(v, dpp<kRowRor + 8>(v));
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

// By column the second of the wavefronts' largest values (the largest where the others have nothing but zeros), in every thread (one
// barrier): a value that stands out does not take the bits of all others.
template <int CT>
__device__ __forceinline__ void typical_largest(uint32_t (&v)[CT], uint32_t (*most)[kFixThreads / kWave]) {
  constexpr int W = kFixThreads / kWave;
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    const uint32_t w = largest_of_wave(v[c]);
    if (threadIdx.x % kWave == 0) most[c][threadIdx.x / kWave] = w;
  }
  __syncthreads();
  // (sixteen lanes a column; the lowest bits tell the wavefronts apart)
  static_assert(W == 16 && CT * W <= kWave, "a row of lanes for each column");
  const int l = (int)threadIdx.x % kWave;
  const uint32_t x = l < CT * W ? (most[l / W % CT][l % W] & ~15u) | (uint32_t)(l % W) : 0;
  const uint32_t first = largest_of_row(x), second = largest_of_row(x == first ? 0 : x), typical = second < 16 ? first : second;
#pragma unroll
  for (int c = 0; c < CT; ++c) v[c] = (uint32_t)__builtin_amdgcn_readlane((int)typical, c * W) & ~15u;
}

// A sum in doubles.
__device__ __forceinline__ double from_fixed(u64 v, double down) {
  return fma((double)(int)(v >> 32), down * 4294967296.0, (double)(uint32_t)v * down);
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

// A sum that has gone out with its strays (a sum of a walk is less than 2^62).
constexpr u64 kFixTaken = 1ull << 63;

// Adds the lists of all wavefronts, which lie in LDS as a whole, to the walk's sums, in doubles.  The entries are put in order first.
template <int CT>
__device__ __forceinline__ void add_listed(u64* acc, u64* near, const uint32_t* listed, const Summed* summed) {
  const int tid = (int)threadIdx.x;
  const bool has = tid < kFixWaves * kFixNear && tid % kFixNear < (int)listed[tid / kFixNear];
  u64 mine = 0;
  int rank = 0, n = 0;
  for (int w = 0; w < kFixWaves; ++w) n += (int)listed[w];
  if (has) {
    mine = near[tid];
    for (int w = 0; w < kFixWaves; ++w)
      for (int j = w * kFixNear; j < w * kFixNear + (int)listed[w]; ++j) rank += near[j] < mine || (near[j] == mine && j < tid) ? 1 : 0;
  }
  __syncthreads();
  if (has) near[rank] = mine;
  __syncthreads();
  double t = 0.0;
  int s = -1;
  if (tid < n) {
    s = (int)(near[tid] >> 32);
    if (tid > 0 && (int)(near[tid - 1] >> 32) == s) s = -1;                // (its first entry adds them all)
    for (int j = tid; s >= 0 && j < n && (int)(near[j] >> 32) == s; ++j) t += (double)__uint_as_float((uint32_t)near[j]);
  }
  __syncthreads();
  if (s >= 0) {
    t += from_fixed(acc[s], summed[s % CT].down);
    near[tid] = (u64)__double_as_longlong(t);
    acc[s] = kFixTaken | (u64)tid;
  }
  __syncthreads();
}

// Notes a value of column c that the walk leaves: the next one goes by the largest finite one, and by whether there are others.
__device__ __forceinline__ void note_left(float v, int c, Left* left) {
  const uint32_t b = magnitude(v);
  if (b >= kFixInf) left[c].others = 1;
  else if (b > *(volatile uint32_t*)&left[c].largest) atomicMax(&left[c].largest, b);
}

// A walk over what the wavefront has listed, or (sums: false) a look at what is left of it.
template <int CT>
__device__ __forceinline__ void walk_list(u64* acc, bool sums, const Bands<CT>& band, const Summed* summed, const Strays& strays, bool odd, float* out,
                                          Left* left) {
  const uint32_t n = min((uint32_t)__builtin_amdgcn_readfirstlane((int)strays.n), kFixNear + strays.room);
  for (uint32_t i = threadIdx.x % kWave; i < n; i += kWave) {
    const u64 entry = i < kFixNear ? strays.near[i] : strays.far[i - kFixNear];
    const uint32_t s = (uint32_t)(entry >> 32);
    const float v = __uint_as_float((uint32_t)entry);
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      if (s % CT != c) continue;
      if (sums && !band.outside(v, c)) add_fixed(&acc[s], to_fixed(v, band.up[c]));
      else if (!still_left(v, summed[c])) continue;
      else if (odd) atomicAdd(out + s, v);
      else note_left(v, c, left);
    }
  }
}

// What follows a walk over the rows or, once they are all there, over the lists: its sums go to out (rest: are added to what
// earlier walks left there; by the same threads).  False: no more walks.  Else the next one's bands, and where it looks.
template <int CT>
__device__ __forceinline__ bool walk_done(u64* acc, int slots, int cleared, Bands<CT>& band, int bits, Summed* summed, Strays& strays, u64* near, uint32_t* counts,
                                          Left* left, bool& lists, bool& rest, bool& odd, float* out) {
  const int tid = (int)threadIdx.x;
  if (!lists && tid % kWave == 0 && strays.n > 0) {
    counts[tid / kWave] = strays.n;
    atomicMax(&counts[kFixWaves], strays.n);
  }
  __syncthreads();
  const uint32_t longest = counts[kFixWaves];            // list of a walk over the rows
  const bool last = !lists && longest <= (uint32_t)kFixNear;
  if (last && longest == 0 && !rest) {
    const double d = summed[tid % CT].down;              // (of all sums of the thread, but for three columns)
#pragma unroll 4
    for (int s = tid; s < slots; s += kFixThreads) out[s] = (float)from_fixed(acc[s], CT == 3 ? summed[s % CT].down : d);
    return false;
  }
  if (last && longest > 0) add_listed<CT>(acc, near, counts, summed);
  for (int s = tid; s < slots; s += kFixThreads) {
    const u64 v = acc[s];
    if (rest && v == 0) continue;
    double t = from_fixed(v, summed[s % CT].down);
    if (last && longest > 0 && v >> 32 == kFixTaken >> 32) t = __longlong_as_double((long long)near[(uint32_t)v]);
    out[s] = rest ? out[s] + (float)t : (float)t;
  }
  if (last) return false;
  if (!lists) {
    walk_list<CT>(acc, false, band, summed, strays, false, out, left);
    lists = longest <= kFixNear + strays.room;
    __syncthreads();
  }
  __builtin_amdgcn_s_waitcnt(0x0f70);                    // (vmcnt(0): other threads add infinities and NaN to out; a fence for the
                                                         // device would write back the L2)
  odd = true;
  bool others = false;
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    odd = odd && left[c].largest == 0;
    others = others || left[c].others != 0;
    band.next(c, left[c].largest, bits, summed);
  }
  if (odd && !others) return false;
  if (tid < CT) left[tid] = Left{0, 0};                  // (behind a barrier of the above)
  for (int s = 2 * tid; s < cleared; s += 2 * kFixThreads) *reinterpret_cast<ulonglong2*>(acc + s) = ulonglong2{0, 0};
  rest = true;
  if (!lists) {
    strays.n = 0;
    if (tid <= kFixWaves) counts[tid] = 0;
  }
  __syncthreads();
  return true;
}

// N rows' values of which some are outside the band: those still to be summed are listed, and all are made zero for the walk's
// sums.  here(i): whether the thread has row i; value(i, c), clear(i, c); sum(i, s): the row's place among the sums of table s of NS,
// or -1.  odd: a walk for infinities and NaN, which make the same of a sum in any order.
template <int CT, int N, int NS, class Here, class Value, class Clear, class Sum>
__device__ __forceinline__ void keep_aside(const Bands<CT>& band, const Summed* summed, Strays& strays, bool rest, bool odd, float* out, Left* left,
                                           Here here, Value value, Clear clear, Sum sum) {
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    uint32_t mask = 0;
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (here(i) && band.outside(value(i, c), c) && value(i, c) != 0.0f && (!rest || still_left(value(i, c), summed[c]))) mask |= 1u << i;
    while (__ballot(mask != 0) != 0) {                   // (one value of every thread at a time)
      const int k = mask != 0 ? __builtin_ctz(mask) : -1;
      float v = 0.0f;
#pragma unroll
      for (int i = 0; i < N; ++i) v = k == i ? value(i, c) : v;
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        int place = -1;
#pragma unroll
        for (int i = 0; i < N; ++i) place = k == i ? sum(i, s) : place;
        const uint32_t at = (uint32_t)(place * CT + c);
        if (!odd) {
          if (strays.add(place >= 0, at, v)) note_left(v, c, left);
        } else if (place >= 0) {
          atomicAdd(out + at, v);
        }
      }
      mask &= mask - 1;
    }
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (band.outside(value(i, c), c)) clear(i, c);
  }
}

// A run's rows are blocks of 4096, every runs-th: rows in order of their keys then keep all workgroups of a range busy alike.
// The runs of XCD x are those with run % 8 == x, whose workgroups for all ranges read the same rows at about the same time.
template <int CT, bool ALIGNED>
__global__ __launch_bounds__(kFixThreads, 4) void segfix_kernel(SegFixMulti m) {
  extern __shared__ __align__(16) u64 acc[];
  __shared__ u64 near[kFixWaves * kFixNear];
  __shared__ uint32_t most[CT][kFixWaves], counts[kFixWaves + 1];
  __shared__ Summed summed[CT];
  __shared__ Left left[CT];
  constexpr int U = CT == 1 ? 2 : 1;       // blocks a thread requests at once
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
  none_summed<CT>(summed, left, counts);
  float* out = a.partial + ((int64_t)range * a.runs + run) * a.stride;
  uint32_t largest[CT];                                  // of the first rows
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    largest[c] = 0;
#pragma unroll
    for (int n = 0; n < U; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const uint32_t b = magnitude(g0.y[n][(r * CT + c) / 4][(r * CT + c) % 4]);
        largest[c] = b < kFixInf ? max(largest[c], b) : largest[c];
      }
  }
  typical_largest<CT>(largest, most);
  Bands<CT> band;
#pragma unroll
  for (int c = 0; c < CT; ++c) band.first(c, largest[c], a.bits, summed);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  Strays strays = {near + wave * kFixNear, a.far + ((int64_t)blockIdx.x * kFixWaves + wave) * a.room, (uint32_t)a.room, 0};
  // a walk over the lists; one after the first; the one for infinities and NaN
  bool lists = false, rest = false, odd = false;
  for (;;) {
    auto spend = [&](int64_t u, Group& g) {
      auto value = [&](int i, int c) -> float { return g.y[i / 4][(i % 4 * CT + c) / 4][(i % 4 * CT + c) % 4]; };
      if (__builtin_expect(band.template some_outside<4 * U>(value), 0)) {
#pragma unroll
        for (int n = 0; n < U; ++n)
          keep_aside<CT, 4, 1>(
              band, summed, strays, rest, odd, out, left,
              [&](int r) { return u + n * stride < units && (uint32_t)(g.k[n][r] - key0) < keys; }, [&](int r, int c) { return value(4 * n + r, c); },
              [&](int r, int c) { g.y[n][(r * CT + c) / 4][(r * CT + c) % 4] = 0.0f; }, [&](int r, int) { return g.k[n][r] - key0; });
      }
#pragma unroll
      for (int n = 0; n < U; ++n) {
        if (u + n * stride >= units) continue;
        uint32_t at[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) at[r] = (uint32_t)(g.k[n][r] - key0);
        add_four<CT>(acc, at, [&](int r) { return at[r] < keys; }, [&](int r, int c) { return to_fixed(value(4 * n + r, c), band.up[c]); });
      }
    };
    if (lists) {
      walk_list<CT>(acc, true, band, summed, strays, odd, out, left);
    } else {
      int64_t u = u0;
      for (int it = 0; it < steps; it += 2) {
        request(u + U * stride, g1);
        spend(u, g0);
        request(u + 2 * U * stride, g0);
        spend(u + U * stride, g1);
        u += 2 * U * stride;
      }
      if (tail > 0) {
        const bool has = tid < tail;
        const int64_t t = units * 4 + (has ? tid : 0);
        const uint32_t at = has ? (uint32_t)(a.idx[t] - key0) : keys;
        float v[CT];
#pragma unroll
        for (int c = 0; c < CT; ++c) v[c] = a.Y[t * CT + c];
        keep_aside<CT, 1, 1>(band, summed, strays, rest, odd, out, left, [&](int) { return at < keys; },
                             [&](int, int c) { return v[c]; }, [&](int, int c) { v[c] = 0.0f; }, [&](int, int) { return (int)at; });
        if (at < keys)
#pragma unroll
          for (int c = 0; c < CT; ++c) add_fixed(&acc[at * CT + c], to_fixed(v[c], band.up[c]));
      }
    }
    if (odd || !walk_done<CT>(acc, slots, a.stride, band, a.bits, summed, strays, near, counts, left, lists, rest, odd, out)) break;
    request(u0, g0);                                     // (also where it is not needed: else the rows live on in registers)
  }
}

// The assembly of gathered products alone, with residual and loss, and the segment sums of the residual: products and sums of
// all tables in LDS, the residual never written.  MODE 1 linear, 2 logistic.  NS: tables.
// 1,000,000 rows over 6040 and 3710 keys, one logistic model: 12.9 microseconds and 4 for the workgroups' sums, where assembly,
// segment sums and their runs' sums took 8, 10 and 4.5 (an iteration with 250,000 sparse cells 30 -> 24).  About 9 of the 12.9
// are there with any number of rows: the launch, the round trips for indices and products, the sums' way out.  Hence few
// workgroups: 64 to 256 take 13.8, 12.0 (128), 13.1, and the sums of 256 take a microsecond longer to add up.
// A row without a key takes the place after its table's last: a product of zero, and a sum that nobody reads.
template <int NS, int CT, int MODE>
__global__ __launch_bounds__(kFixThreads, 4) void asm_fix_kernel(AsmFix a) {
  extern __shared__ __align__(16) u64 acc[];
  __shared__ u64 near[kFixWaves * kFixNear];
  __shared__ uint32_t most[CT][kFixWaves], counts[kFixWaves + 1];
  __shared__ Summed summed[CT];
  __shared__ Left left[CT];
  __shared__ float lsum[kFixThreads / kWave][CT];
  float* prod = reinterpret_cast<float*>(acc + (size_t)a.slots);
  const int tid = (int)threadIdx.x, lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
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
  none_summed<CT>(summed, left, counts);
  __syncthreads();

  float loss[CT], lost[CT];
#pragma unroll
  for (int c = 0; c < CT; ++c) loss[c] = lost[c] = 0.0f;
  float* out = a.partial + (int64_t)blockIdx.x * a.slots;
  Bands<CT> band;
  Strays strays = {near + wave * kFixNear, a.far + ((int64_t)blockIdx.x * kFixWaves + wave) * a.room, (uint32_t)a.room, 0};
  bool lists = false, rest = false, odd = false;         // (see segfix_kernel)
  for (;;) {
    if (lists) walk_list<CT>(acc, true, band, summed, strays, odd, out, left);
    int u = u0 + tid;
    for (int it = lists ? steps + 1 : 0; it < steps + (tail > 0 ? 1 : 0); ++it, u += kFixThreads) {
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
        if (!rest) {
#pragma unroll
          for (int c = 0; c < CT; ++c) {                 // compensated; what is infinite stays so
            const float t = ((add[0][c] + add[1][c]) + (add[2][c] + add[3][c])) - lost[c], sum = loss[c] + t;
            lost[c] = fabsf(sum) <= __FLT_MAX__ ? (sum - loss[c]) - t : 0.0f;
            loss[c] = sum;
          }
        }
      }
      if (!rest && it == 0) {
        uint32_t largest[CT];
#pragma unroll
        for (int c = 0; c < CT; ++c) largest[c] = 0;
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
          for (int r = 0; r < 4; ++r) { const uint32_t b = magnitude(e[r][c]); largest[c] = b < kFixInf ? max(largest[c], b) : largest[c]; }
        typical_largest<CT>(largest, most);
#pragma unroll
        for (int c = 0; c < CT; ++c) band.first(c, largest[c], a.bits, summed);
      }
      if (!live) continue;
      if (__builtin_expect(band.template some_outside<4>([&](int r, int c) { return e[r][c]; }), 0))
        keep_aside<CT, 4, NS>(
            band, summed, strays, rest, odd, out, left, [](int) { return true; }, [&](int r, int c) { return e[r][c]; },
            [&](int r, int c) { e[r][c] = 0.0f; },
            [&](int r, int s) { return now.j[s][r] < a.off[s] + a.keys[s] ? now.j[s][r] : -1; });
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const uint32_t at[4] = {(uint32_t)now.j[s][0], (uint32_t)now.j[s][1], (uint32_t)now.j[s][2], (uint32_t)now.j[s][3]};
        add_four<CT>(acc, at, [](int) { return true; }, [&](int r, int c) { return to_fixed(e[r][c], band.up[c]); });
      }
    }
    if (!rest) {
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        const float t = sum_of_wave(loss[c]);
        if (lane == kWave - 1) lsum[wave][c] = t;
      }
    }
    const bool first = !rest;
    const bool more = !odd && walk_done<CT>(acc, a.slots, a.slots, band, a.bits, summed, strays, near, counts, left, lists, rest, odd, out);
    if (first && tid < CT) {                             // (behind a barrier of the above)
      float part[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int w = 0; w < kFixWaves; ++w) part[w / 4] += lsum[w][tid];
      a.loss_partial[(int64_t)blockIdx.x * kNarrowCT + tid] = (part[0] + part[1]) + (part[2] + part[3]);
    }
    if (!more) break;
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
// launch of their own; longest: entries of the longest segment).  Both sides are estimates in microseconds, fitted to iterations
// over one to three joined tables.  Keys in order gather well: by themselves for next to nothing below 1,500,000 rows, beside
// others for less.  Rows of one key are added to one place of LDS one after the other, which costs several columns more.
// Iterations, gathering / in LDS:
//   one model      1,000,000 rows  20,000 uniform keys              38 / 44     gathers
//                                  50,000 and 20,000                49 / 49     in LDS
//                                  three times 3000                 51 / 42     in LDS
//                                  twice 20,000 in order            36 / 46     gathers
//                                  50,000 in order and 20,000       42 / 46     gathers
//                  5,000,000 rows  20,000 uniform; in order         93 / 84; 84 / 80   in LDS
//                                  100,000, 50,000 Zipf and 10,000  178 / 132   in LDS
//   two models     1,000,000 rows  three times 3000                 70 / 49     in LDS
//   three models   1,000,000 rows  20,000, half of them one key     57 / 65     gathers
//                  5,000,000 rows  three times 3000                 345 / 190   in LDS
//                                  20,000 in order                  126 / 130   gathers
//                                  100,000, 50,000 and 10,000       379         gathers: too many ranges
bool segfix_pays(int64_t r_T, const int64_t* rows, const bool* in_order, int n, int ncols, bool cut, int64_t longest) {
  if (n < 1 || r_T < 100000 || n > kSegMulti) return false;
  int64_t ranges = 0;
  int ordered = 0;
  for (int q = 0; q < n; ++q) {
    ranges += (rows[q] + kFixSlots / ncols - 1) / (kFixSlots / ncols);
    ordered += in_order[q] ? 1 : 0;
  }
  if (ranges > 20) return false;
  const bool far_apart = r_T >= 1500000;                 // (the residual does not stay in an XCD's L2: segments are cut by slice)
  const double all = 1e-6 * (double)r_T, near = std::min(all, 1.5), more = ncols - 1;
  const double one = 7.2 * near + 4.9 * (all - near) + more * (2.6 * near + 3.6 * (all - near));
  double gather = n * one + (cut ? 5.0 : 0.0) + (far_apart ? std::max(0.0, 6.0 * n - 9.0) : 0.0);
  for (int q = 0; q < n; ++q) {
    if (!in_order[q]) continue;
    const double less = far_apart ? 5.0 + 1.7 * all + more * (0.8 + 0.4 * all) + 1e-3 * (double)rows[q] * (0.1 + 0.12 * ncols) : 0.0;
    gather -= std::max(one - less, 0.0) * (ordered == n ? 1.0 : 0.4);
  }
  return 5.0 + segfix_share(r_T, rows, n, ncols).us + 2.2e-6 * (double)longest * ncols * more < gather;
}

// Room of a wavefront's list in what is left of the scratch space.
static int list_room(float* rest, int64_t floats, int64_t grid, unsigned long long** far) {
  *far = reinterpret_cast<unsigned long long*>(rest);                        // (the runs' sums are whole float4s)
  return (int)std::min<int64_t>(kFixFar, floats / 2 / (grid * kFixWaves));
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
    while (((int64_t)1 << count) <= (s.longest > 0 ? std::min(run, s.longest) : run)) ++count;
    s.bits = std::min(50, 62 - count);
    s.partial = scratch + at;
    at += (int64_t)s.n_ranges * kSegSlices * s.nsub * s.stride;
    m.first[q + 1] = m.first[q] + s.n_ranges * s.nsub;
  }
  if (at > scratch_floats) return hipErrorInvalidValue;
  const size_t lds = sizeof(u64) * (size_t)slots;
  const unsigned grid = (unsigned)m.first[n] * kSegSlices;
  for (int q = 0; q < n; ++q) m.s[q].room = list_room(scratch + at, scratch_floats - at, grid, &m.s[q].far);
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
// more rows.  Iterations of one to four logistic models, separate launches / one: 1,000,000 rows over 300 keys 42 / 19, over 3000
// 31 / 23 (four models 56 / 42), over 12,000 32 / 27, over twice 6000 38 / 27, over 3000 in order 23 / 23; 300,000 over 3000
// 22 / 20, over 300 25 / 18; 100,000 over 3000 19 / 20 (four models 24 / 29); 3,000,000 over three times 2000
// 74 / 33, over 3000 in order 38 / 27.
bool asm_fix_pays(const LmmArgs& a, const float* lines) {
  int64_t keys = 0;
  int in_order = 0;
  for (int s = 0; s < a.g.n; ++s) {
    keys += a.g.rows[s];
    in_order += keys_in_order(lines[s], a.g.rows[s]) ? 1 : 0;
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
  const int64_t floats = (int64_t)grid * f.slots;
  if (floats > scratch_floats) return hipErrorInvalidValue;
  f.room = list_room(scratch + floats, scratch_floats - floats, grid, &f.far);
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
