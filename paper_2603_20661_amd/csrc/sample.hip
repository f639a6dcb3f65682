// Temperature / nucleus (top-p) sampling from next-token logits (App. C of the paper lists temperature and top-p among
// the generation parameters; its own runs use temperature 0, i.e. the greedy argmax of the decode path).
//
// Per row: z_i = logit_i / T, e_i = exp(z_i - max z).  The nucleus is {i : e_i >= tau}, tau being the largest of the e
// values for which the members' sum reaches top_p * sum of all e (elements equal to tau are all in).  The token is drawn
// by the inverse CDF over the nucleus taken in index order: the first member whose running sum exceeds u * (nucleus sum),
// u in [0, 1) supplied by the caller.
//
// No sort, and no pass over the row per bit of tau.  The scores t = log2(e) * z are dropped into 256 bins of an eighth of
// an octave below the largest one, with the mass of each bin; the bins alone tell which one holds tau, and only that
// bin's elements (one to three per cent of a row, up to seven of a flat one) are looked at individually.  All masses are integers - units of 2^-44 of
// a power of two at the largest score, so every fp32 probability above 2^-20 enters with all its bits - and integer sums
// do not depend on their order: a call is reproducible although the bins are filled with LDS atomics.  Rows of more than
// 2^19 tokens take a unit twice as large per doubling (mass_unit), so that the masses of a row add up to 2^63 at most.
// Probabilities are formed from the difference to the largest logit of the row or chunk, never from the score itself, which
// is as large as the temperature is small.  The bins take the score as it is, rounded and clamped: all they have to be is a
// monotone function of the logit alone, the same in every chunk.  Scores beyond 2^21 share bins, at worst all of a row,
// whose members are then told apart by their logits like those of any other bin.
//
// A row is 501 KB at 128 256 tokens and one compute unit fetches some 120 GB/s, so one workgroup per row is bound by its
// compute unit's loads and exponentials whatever it does (the 33 passes of the bisection that stood here: 849 us for 64
// rows, 25 us a pass, against 6.4 us to read the logits once at the rate of a copy).  Long rows are therefore cut into
// at most 64 chunks, of up to 16 384 tokens where that will do, one workgroup each (512 workgroups for 64 rows), in two launches: bins of every chunk; then
// probabilities and members of the decisive bin of every chunk, with tau and the token by the workgroup of a row that finishes
// last.  What the launches and workgroups hand on lies in the first RESERVED floats of every chunk's part of the scratch buffer,
// which receive their probabilities last.  Rows of up to 8192 tokens fit one workgroup's registers and take one launch.
//
// What bounds it: with few rows the chain of dependent steps, each one to two microseconds of memory round trips, barriers and above all
// fetches of instructions that run once per launch on one compute unit.  So the code is kept short (rolled loops over registers, one
// instance of every step), sums and scans go through DPP moves, and the last step of a row reads 256 logits, not a chunk.  With many rows
// it is the instructions per element (about 25 for a mass and its bin).  Measured (us, against three launches and unrolled code): 128 256
// tokens, 1, 8, 16 and 64 rows 29.4 -> 15.9, 32.9 -> 18.9, 33.5 -> 19.5 and 44.3 -> 30.8; 32 000 tokens, 1, 16 and 64 rows 25.8 -> 14.1,
// 26.2 -> 14.5 and 27.6 -> 16.0; 1024 tokens, 1 and 48 rows 7.0 -> 6.1 and 7.5 -> 6.5.  The logits of 64 rows of 128 256 tokens read once and
// their probabilities written once at the rate of a copy: 13.6 us.  One launch for rows of up to 32 768 tokens took 24.5 us (32 000 tokens:
// one compute unit's loads 5.4, bins 8, members of the decisive bin 5, masses 4).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cfloat>
#include <mutex>

#include "../../include/www.h"

#define WWW_EXPORT extern "C" __attribute__((visibility("default")))

void set_error(const char* fmt, ...);

namespace {

constexpr int BINS = 256, BINS_PER_OCTAVE_LOG2 = 3;
constexpr int TPB = 1024;
constexpr int WAVES = TPB / 64;
constexpr int ROW_PER = 2;           // groups of four elements a thread holds where one workgroup takes a row,
constexpr int BLOCK_PER = 4;         // and where it reads elements again
// Chunks of a row, one a lane; longer rows take longer chunks (2 000 000 normal logits of standard deviation 3, 1 and 16 rows 171 -> 74 and 427 -> 193 us
// against three launches with up to 1024 chunks; 9 000 001 near-equal ones 17 870 -> 10 030, one workgroup reading the row).
constexpr int MAX_CHUNKS = 64;
constexpr int MAX_RUNS = TPB;        // runs of a row, see RowRuns
// start of a chunk's scratch: largest logit, candidates found, their least and largest key, workgroups of the row
// that have finished (first chunk); bin masses (low words, high words); masses of its runs (low, high); candidates (logit, place)
enum { H_MAX = 0, H_COUNT = 1, H_KLO = 2, H_KHI = 3, H_DONE = 4, H_BINS = 8 };
constexpr int H_RUNS = H_BINS + 2 * BINS;
constexpr int RESERVED = 4096;
__device__ __host__ constexpr int head_of(int runs) { return H_RUNS + 2 * runs; }
__device__ __host__ constexpr int cand_max(int runs) { return (RESERVED - head_of(runs)) / 2; }
// Candidates of a row that are looked at in LDS, two workgroups to a compute unit.  With more the chunks' lists are read, once per round (128 256
// normal logits of standard deviation 0.4 to 1, top_p 0.8 and 0.9: 4000 to 9000; 1, 16 and 64 rows 30 to 35, 31 to 39 and 54 to 66 us, where a list
// of 8192 in LDS took 70 to 90 and the row itself 123 to 175).  A list of 9216 is slower where it is needed: 2 000 000 tokens of standard deviation 3,
// 5000 candidates, 1 and 4 rows 73.7 and 86.9, the chunks' lists 58.5 and 65.8.
constexpr int ROW_CAND = 4096;

typedef unsigned long long u64;
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));  // (rows start anywhere)

// bin of a score, clamped far outside the range of ordinary scores (NaN falls to the bottom: the median of a NaN is the least of
// the others)
__device__ __forceinline__ int bin_of(float logit, float c) {
  return (int)floorf(__builtin_amdgcn_fmed3f(logit * (c * (float)(1 << BINS_PER_OCTAVE_LOG2)), -536870912.f, 536870912.f));
}
// number of a bin, counted down from bin `top`; the last one takes everything below
__device__ __forceinline__ int bin_number(int top, int bin) { return min(BINS - 1, max(0, top - bin)); }
// Reference of the masses of a row or chunk with largest logit m (made finite, so that differences to it are numbers):
// 2^oct lies at most one octave above the largest probability, and r (-1 .. 0) is the way down from there.  Octaves are whole
// numbers, in double because a score may exceed any integer, so that masses of different chunks differ by shifts.
__device__ __forceinline__ float finite(float m) { return fminf(fmaxf(m, -FLT_MAX), FLT_MAX); }
__device__ __forceinline__ double octave_of(float m, float c) { return floor((double)m * (double)c) + 1.; }
__device__ __forceinline__ float way_down(float m, float c) { return (float)((double)m * (double)c - octave_of(m, c)); }
__device__ __forceinline__ int octaves_between(double row, double chunk) { return (int)fmin(row - chunk, 64.); }
// 2^(r + score - largest score), in [0, 1] (+inf: as FLT_MAX; NaN: 0)
__device__ __forceinline__ float prob(float logit, float c, float m, float r) {
  return __builtin_amdgcn_fmed3f(__builtin_amdgcn_exp2f(__builtin_fmaf(logit - m, c, r)), 0.f, 1.f);
}
// e in [0, 1] in units of 2^-24 / unit
__device__ __forceinline__ u64 mass_of(float e, float unit) {
  const float s = e * unit;
  const uint32_t hi = (uint32_t)s;
  const uint32_t lo = (uint32_t)((s - (float)hi) * 16777216.f);
  return ((u64)hi << 24) + lo;
}
__device__ __forceinline__ u64 shifted(u64 v, int k) { return k < 64 ? v >> k : 0ull; }
// order-preserving integer of a float, the same for both zeros
__device__ __forceinline__ uint32_t key_of(float x) {
  const uint32_t b = __float_as_uint(x);
  return (b & 0x80000000u) ? 0u - b : b | 0x80000000u;
}

// Sums, scans and extremes over a wavefront by moves between neighbouring lanes, rows of 16 and halves (all lanes active): a step is two
// instructions where one through LDS waits for its result, and half of these kernels' time is such chains
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t moved(uint32_t v, uint32_t otherwise) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)otherwise, (int)v, CTRL, ROWS, 15, false);
}
template <typename F>
__device__ __forceinline__ void wave_steps(F&& f) {  // lanes 1, 2, 4, 8 down the row, the row before, the half before
  f([](uint32_t v, uint32_t o) { return moved<0x111, 15>(v, o); });
  f([](uint32_t v, uint32_t o) { return moved<0x112, 15>(v, o); });
  f([](uint32_t v, uint32_t o) { return moved<0x114, 15>(v, o); });
  f([](uint32_t v, uint32_t o) { return moved<0x118, 15>(v, o); });
  f([](uint32_t v, uint32_t o) { return moved<0x142, 10>(v, o); });
  f([](uint32_t v, uint32_t o) { return moved<0x143, 12>(v, o); });
}
__device__ __forceinline__ uint32_t lane_of(uint32_t v, int lane) { return (uint32_t)__builtin_amdgcn_readlane((int)v, lane); }
__device__ __forceinline__ u64 lane_of(u64 v, int lane) { return (u64)lane_of((uint32_t)(v >> 32), lane) << 32 | lane_of((uint32_t)v, lane); }
__device__ __forceinline__ u64 wave_scan(u64 v) {  // inclusive
  wave_steps([&](auto&& move) __attribute__((always_inline)) { v += (u64)move((uint32_t)(v >> 32), 0u) << 32 | move((uint32_t)v, 0u); });
  return v;
}
__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
  wave_steps([&](auto&& move) __attribute__((always_inline)) { v += move(v, 0u); });
  return v;
}
__device__ __forceinline__ u64 wave_sum(u64 v) { return lane_of(wave_scan(v), 63); }
// least lo and largest hi of the wavefront
__device__ __forceinline__ void wave_range(uint32_t& lo, uint32_t& hi) {
  wave_steps([&](auto&& move) __attribute__((always_inline)) { lo = min(lo, move(lo, lo)); hi = max(hi, move(hi, hi)); });
  lo = lane_of(lo, 63);
  hi = lane_of(hi, 63);
}
__device__ __forceinline__ float wave_max(float v) {
  wave_steps([&](auto&& move) __attribute__((always_inline)) { v = fmaxf(v, __uint_as_float(move(__float_as_uint(v), __float_as_uint(v)))); });
  return __uint_as_float(lane_of(__float_as_uint(v), 63));
}

template <int NT>
__device__ __forceinline__ float block_max(float v, float* red) {
  v = wave_max(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return wave_max(red[threadIdx.x & (NT / 64 - 1)]);
}

// The first of BINS bins, largest elements first, at which the mass so far reaches `share` of the total (want < 0) or
// `want`; `need` is what its own members have to contribute.  Called by one whole wavefront.
__device__ __forceinline__ void find_boundary(const u64* hist, float share, double want, int* bin, double* need) {
  const int lane = threadIdx.x & 63;
  u64 h[4], s = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) { h[i] = hist[lane * 4 + i]; s += h[i]; }
  const u64 incl = wave_scan(s);
  const double total = (double)lane_of(incl, 63);
  want = want < 0. ? (double)share * total : fmin(want, total);
  const u64 reached = __ballot((double)incl >= want);
  if (lane == (reached ? __ffsll((long long)reached) - 1 : 63)) {
    u64 before = incl - s, own = h[0];
    int i = 0;
#pragma unroll
    for (int k = 0; k < 3; ++k)
      if (i == k && (double)(before + h[k]) < want) { before += h[k]; own = h[k + 1]; ++i; }
    *bin = lane * 4 + i;
    *need = fmin(want - (double)before, (double)own);  // (sums beyond 2^53 are rounded: never more than the bin holds)
  }
}

// tau among n candidates: the largest key whose members' mass reaches `need` (the smallest key if rounding keeps even
// that from it).  A search with sixteen thresholds a round, one per wavefront.
__device__ __forceinline__ uint32_t find_tau(const uint32_t* keys, const u64* mass, int n, double need, uint32_t lo, uint32_t hi, int* reached) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int turn = 0;  // two sets of answers, so that a round needs one barrier
  while (hi - lo > 1u) {  // members of lo suffice, members of hi do not
    const uint32_t step = (hi - lo - 1u) / (WAVES + 1) + 1u;
    const u64 at = (u64)lo + (u64)step * (wave + 1);
    bool ok = false;
    if (at < hi) {
      u64 s = 0;
      for (int i = lane; i < n; i += 64) s += keys[i] >= (uint32_t)at ? mass[i] : 0ull;
      ok = (double)wave_sum(s) >= need;
    }
    if (lane == 0) reached[turn + wave] = ok;
    __syncthreads();
    const int c = __popcll(__ballot(lane < WAVES && reached[turn + (lane & (WAVES - 1))]));  // (monotone: the first c thresholds reach it)
    turn = WAVES - turn;
    const uint32_t l = lo + step * c;
    if (c < WAVES && hi - l > step) hi = l + step;
    lo = l;
  }
  return lo;
}

// tau among the keys lo .. last: 256 linear bins a round until one key is left (four rounds at most).  members(use) calls
// use(key, mass) for every element in question; share and want as for find_boundary.  `copies` holds COPIES sets of bins, by
// lane, so that the lanes of a wavefront seldom meet in one.
constexpr int COPIES = 16;
template <int CP>
__device__ __forceinline__ void sum_copies(const u64* copies, u64* hist) {
  const int tid = threadIdx.x;
  if (tid < BINS) {
    u64 s = 0;
#pragma unroll
    for (int k = 0; k < CP; ++k) s += copies[tid * CP + ((k + tid) & (CP - 1))];
    hist[tid] = s;
  }
}
template <typename M>
__device__ __forceinline__ uint32_t search_keys(M&& members, uint32_t lo, uint32_t last, float share, double want, u64* copies, u64* hist, int* bin, double* need) {
  const int tid = threadIdx.x;
  while (last > lo) {
    const int shift = max(0, 24 - __clz(last - lo));  // (last - lo) >> shift < 256
    for (int i = tid; i < BINS * COPIES; i += TPB) copies[i] = 0;
    __syncthreads();
    members([&](uint32_t key, auto&& mass) {
      if (key < lo || key > last) return;
      const u64 w = mass();
      if (w) atomicAdd(&copies[(BINS - 1 - ((key - lo) >> shift)) * COPIES + (tid & (COPIES - 1))], w);
    });
    __syncthreads();
    sum_copies<COPIES>(copies, hist);
    __syncthreads();
    if (tid < 64) find_boundary(hist, share, want, bin, need);
    __syncthreads();
    want = *need;
    const uint32_t first = lo + ((uint32_t)(BINS - 1 - *bin) << shift);
    last = min(last, first + ((1u << shift) - 1u));
    lo = first;
  }
  return lo;
}

// Elements i .. i + 3 of the n at p (-inf behind the end)
__device__ __forceinline__ f32x4 load4(const float* p, int i, int n) {
  f32x4 v = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
  if (i + 4 <= n) v = *reinterpret_cast<const f32x4u*>(p + i);
  else
#pragma unroll
    for (int e = 0; e < 3; ++e)
      if (i + e < n) v[e] = p[i + e];
  return v;
}
// the groups of a block: at most one of them is not whole
template <int N>
__device__ __forceinline__ void load_groups(f32x4 (&x)[N], const float* p, int n) {
  const int whole = n / (4 * TPB), i = threadIdx.x * 4;
#pragma unroll
  for (int k = 0; k < N; ++k)
    if (k < whole) x[k] = *reinterpret_cast<const f32x4u*>(p + k * (4 * TPB) + i);
  const f32x4 rest = load4(p, whole * (4 * TPB) + i, n);
#pragma unroll
  for (int k = 0; k < N; ++k)
    if (k >= whole) x[k] = k == whole ? rest : f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
}
__device__ __forceinline__ void store4(float* p, int i, int first, int n, f32x4 v) {  // those that lie in [first, n)
  if (i >= first && i + 4 <= n) {
    *reinterpret_cast<f32x4u*>(p + i) = v;
    return;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (i + e >= first && i + e < n) p[i + e] = v[e];
}
// The logit that a key belongs to: x >= it for the keys from this one on (a NaN has no mass and is left out)
__device__ __forceinline__ float logit_of(uint32_t key) {
  if (key <= 0x00800000u) return -INFINITY;  // (keys of -inf and below)
  return __uint_as_float(key & 0x80000000u ? key & 0x7FFFFFFFu : 0u - key);
}
// The least float that is no smaller than n, |n| < 2^30: a score t, a float, has floor(t) >= n exactly where t >= at_least(n).  (Beyond 2^24
// a whole number need not be a float, and between 2^22 and 2^23 floats are halves: the next float after a bin's own is not its end there.)
__device__ __forceinline__ float at_least(int n) {
  const float f = (float)n;
  return (int)f < n ? __uint_as_float(f > 0.f ? __float_as_uint(f) + 1u : __float_as_uint(f) - 1u) : f;
}
// bin_of(x, c) == bin, compared as scores; bottom and top: everything below or above belongs to it too (a NaN does not: it has no mass)
struct InBin {
  float scale, lo, hi;
  bool open;
  __device__ __forceinline__ InBin(int bin, bool bottom, bool top, float c) {
    scale = c * (float)(1 << BINS_PER_OCTAVE_LOG2);
    lo = bottom || bin <= -536870912 ? -INFINITY : (float)bin;  // (any but the lowest is the bin of a score, which is a float)
    hi = at_least(bin + 1);
    open = top || bin >= 536870912;
  }
  __device__ __forceinline__ float above() const { return open ? NAN : hi; }  // scores from here on lie above (none, if it is open)
  __device__ __forceinline__ bool operator()(float x) const {
    const float t = x * scale;
    return t >= lo && (t < hi || open);
  }
};

// The token is the first member (logit >= tau), in index order, whose running mass exceeds a target.  A block of 4 N * TPB elements has
// elements 4 (k * TPB + tid) .. + 3 in x[k]; `part` receives the members' masses of every run of 256 elements (k, wavefront), which is
// index order.  All threads of the workgroup call it; behind a barrier choose() may follow.
// f(group, k) for every group of four in turn, as a rolled loop over registers that change places: these kernels run once through
// their code, on few workgroups, and wait for instructions more than for anything else when it is unrolled
template <int N, typename F>
__device__ __forceinline__ void each_group(f32x4 (&x)[N], F&& f) {
#pragma unroll 1
  for (int k = 0; k < N; ++k) {
    f(x[0], k);
    const f32x4 first = x[0];
#pragma unroll
    for (int i = 0; i + 1 < N; ++i) x[i] = x[i + 1];
    x[N - 1] = first;
  }
}
struct Masses {
  float c, m, r, unit, tau;
  __device__ __forceinline__ u64 operator()(float v) const { return v >= tau ? mass_of(prob(v, c, m, r), unit) : 0ull; }
  __device__ __forceinline__ int member(f32x4 v, u64 left) const {  // the first of four whose running mass exceeds `left`
    u64 at = 0;
    int e = 0;
#pragma unroll
    for (int i = 0; i < 3; ++i)
      if (e == i && (at += (*this)(v[i])) <= left) ++e;
    return e;
  }
  __device__ __forceinline__ u64 operator()(f32x4 v) const { return ((*this)(v[0]) + (*this)(v[1])) + ((*this)(v[2]) + (*this)(v[3])); }
};
template <int N>
__device__ __forceinline__ void member_masses(f32x4 (&x)[N], const Masses& mass, u64* part) {
  const int tid = threadIdx.x;
  each_group(x, [&](f32x4 v, int k) __attribute__((always_inline)) {
    u64 w = 0;
    if (__any(fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])) >= mass.tau)) w = wave_sum(mass(v));  // (most runs of an ordinary row have no member)
    if ((tid & 63) == 0) part[k * WAVES + (tid >> 6)] = w;
  });
}
template <int N>
__device__ __forceinline__ u64 total_mass(const u64* part) {
  const int lane = threadIdx.x & 63;
  u64 s = 0;
#pragma unroll
  for (int i = 0; i < N * WAVES; i += 64) s += i + lane < N * WAVES ? part[i + lane] : 0ull;
  return wave_sum(s);
}
template <int N>
__device__ __forceinline__ void choose(const f32x4 (&x)[N], const Masses& mass, const u64* part, u64 target, int base, int32_t* token) {
  constexpr int E = (N * WAVES + 63) / 64;  // runs per lane
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  u64 h[E], s = 0;
#pragma unroll
  for (int i = 0; i < E; ++i) { h[i] = lane * E + i < N * WAVES ? part[lane * E + i] : 0ull; s += h[i]; }
  const u64 incl = wave_scan(s), past = __ballot(incl > target);
  if (!past) return;
  const int owner = __ffsll((long long)past) - 1;
  u64 before = incl - s;
  int run = lane * E;
#pragma unroll
  for (int i = 0; i < E - 1; ++i)
    if (run == lane * E + i && before + h[i] <= target) { before += h[i]; ++run; }
  before = lane_of(before, owner);
  run = (int)lane_of((uint32_t)run, owner);
  if (run % WAVES != wave) return;
  f32x4 v = x[0];
#pragma unroll
  for (int k = 1; k < N; ++k)
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = run / WAVES == k ? x[k][e] : v[e];  // (whole groups: chosen by address, from scratch memory)
  const u64 w = mass(v), upto = before + wave_scan(w);
  const u64 hit = __ballot(upto > target);
  if (hit && lane == __ffsll((long long)hit) - 1) *token = base + (run / WAVES * TPB + tid) * 4 + mass.member(v, target - (upto - w));
}
// the token among elements [0, n) of p in memory, block by block; `base` is added to the index
__device__ __forceinline__ void choose_among(const float* p, int n, const Masses& mass, u64 target, int base, u64* part, int32_t* token) {
#pragma unroll 1
  for (int b0 = 0; b0 < n; b0 += 4 * BLOCK_PER * TPB) {
    f32x4 v[BLOCK_PER];
    load_groups(v, p + b0, n - b0);
    if (b0) __syncthreads();  // the masses of the block before have been read
    member_masses(v, mass, part);
    __syncthreads();
    const u64 here = total_mass<BLOCK_PER>(part);
    if (target < here) {
      choose(v, mass, part, target, base + b0, token);
      return;
    }
    target -= here;
  }
}

// target of the draw inside a nucleus of mass `nucleus`
__device__ __forceinline__ u64 draw_target(float u, u64 nucleus) {
  const u64 t = (u64)((double)fmaxf(u, 0.f) * (double)nucleus);
  return t < nucleus ? t : (nucleus ? nucleus - 1 : 0ull);
}

// put(place, logit, index) for every element of a block (of the n that are valid) that lies in a bin; places are counted in LDS, in no particular order, and
// the range of the keys is kept: step by step, or with the larger blocks, which come where all compute units have several workgroups, once at the
// end (128 256 tokens, 256 rows of standard deviation 2, top_p 0.8 125.7 -> 122.7 us, of 0.02 310 -> 292; but one row of 32 000, in smaller
// blocks, 53.0 -> 55.7)
template <int N, typename P>
__device__ __forceinline__ void list_members(f32x4 (&x)[N], const InBin& in_bin, int n, int* count, uint32_t* klo, uint32_t* khi, P&& put) {
  constexpr bool AT_END = N > ROW_PER;
  uint32_t least = 0xFFFFFFFFu, largest = 0u;
  each_group(x, [&](f32x4 v, int k) __attribute__((always_inline)) {
    const int i = (k * TPB + (int)threadIdx.x) * 4;
    uint32_t mine = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) mine |= in_bin(v[e]) && i + e < n ? 1u << e : 0u;
#pragma unroll 1
    while (__any(mine)) {  // (seldom: one element of every lane that has one)
      const u64 who = __ballot(mine);
      const int lane = threadIdx.x & 63, leader = __ffsll((long long)who) - 1, e = __ffs((int)mine) - 1;
      const float y = e == 0 ? v[0] : e == 1 ? v[1] : e == 2 ? v[2] : v[3];
      uint32_t lo = mine ? key_of(y) : 0xFFFFFFFFu, hi = mine ? key_of(y) : 0u;
      if constexpr (AT_END) {
        least = min(least, lo);
        largest = max(largest, hi);
      } else {
        wave_range(lo, hi);
      }
      int at = 0;
      if (lane == leader) {
        at = atomicAdd(count, __popcll(who));
        if constexpr (!AT_END) {
          atomicMin(klo, lo);
          atomicMax(khi, hi);
        }
      }
      at = __shfl(at, leader) + __popcll(who & ((1ull << lane) - 1));
      if (mine) put(at, y, i + e);
      mine &= mine - 1;
    }
  });
  if (AT_END && __any(largest)) {
    wave_range(least, largest);
    if ((threadIdx.x & 63) == 0) {
      atomicMin(klo, least);
      atomicMax(khi, largest);
    }
  }
}

// ---- rows of up to 16 N * TPB bytes: one workgroup per row, everything in registers and LDS
constexpr int LIST = 4 * ROW_PER * TPB;  // candidates looked at in LDS, where all of a row may be some (one workgroup to a compute unit)
template <int CP>
struct SmallLds {
  uint32_t keys[LIST];
  u64 mass[LIST];
  u64 copies[BINS * CP];
  u64 hist[BINS];
  u64 part[ROW_PER * WAVES];
  double need;
  float red[WAVES];
  int reached[2 * WAVES];
  uint32_t klo, khi;
  int bin, count;
};

// CP: sets of bins, so that the lanes of a wavefront seldom meet in one (clearing and adding them up costs short rows more than it gives)
template <int N, int CP>
__global__ __launch_bounds__(TPB) void sample_row_kernel(const float* logits, int V, float c, float unit, float top_p, const float* __restrict__ u01,
                                                         float* scratch, int32_t* __restrict__ tokens) {
  extern __shared__ __align__(16) char smem[];
  static_assert(4 * N * TPB <= LIST);
  SmallLds<CP>& S = *reinterpret_cast<SmallLds<CP>*>(smem);
  const int tid = threadIdx.x, row = blockIdx.x;
  const bool in_place = scratch == logits;  // the probabilities then wait until the logits have been read for the last time
  const float* lg = logits + (int64_t)row * V;
  float* out = scratch + (int64_t)row * V;
  f32x4 x[N];
  float m = -INFINITY;
  load_groups(x, lg, V);
  const float u = u01[row];
  for (int i = tid; i < BINS * CP; i += TPB) S.copies[i] = 0;
  if (tid == 0) { S.count = 0; S.klo = 0xFFFFFFFFu; S.khi = 0u; }
#pragma unroll
  for (int k = 0; k < N; ++k) m = fmaxf(m, fmaxf(fmaxf(x[k][0], x[k][1]), fmaxf(x[k][2], x[k][3])));
  m = finite(block_max<TPB>(m, S.red));
  const int top = bin_of(m, c);
  each_group(x, [&](f32x4 v, int k) __attribute__((always_inline)) {
    f32x4 e4;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      e4[e] = prob(v[e], c, m, 0.f);
      const u64 w = mass_of(e4[e], unit);  // (0 for the -inf behind the end)
      if (w) atomicAdd(&S.copies[bin_number(top, bin_of(v[e], c)) * CP + (tid & (CP - 1))], w);
    }
    if (!in_place) store4(out, (k * TPB + tid) * 4, 0, V, e4);
  });
  __syncthreads();
  sum_copies<CP>(S.copies, S.hist);
  __syncthreads();
  if (tid < 64) find_boundary(S.hist, top_p, -1., &S.bin, &S.need);
  __syncthreads();
  const InBin in_bin(top - S.bin, S.bin == BINS - 1, S.bin == 0, c);
  list_members(x, in_bin, V, &S.count, &S.klo, &S.khi, [&](int at, float v, int) __attribute__((always_inline)) {
    S.keys[at] = key_of(v);
    S.mass[at] = mass_of(prob(v, c, m, 0.f), unit);
  });
  __syncthreads();
  const uint32_t klo = S.klo, khi = S.khi;
  uint32_t tau = 0u;
  if (S.count) tau = find_tau(S.keys, S.mass, S.count, S.need, klo, khi == 0xFFFFFFFFu ? khi : khi + 1u, S.reached);
  const Masses mass{c, m, 0.f, unit, logit_of(tau)};
  member_masses(x, mass, S.part);
  __syncthreads();
  const u64 nucleus = total_mass<N>(S.part);
  if (nucleus) choose(x, mass, S.part, draw_target(u, nucleus), 0, tokens + row);
  else if (tid == 0) tokens[row] = 0;  // (a row without any finite logit)
  if (!in_place) return;
  each_group(x, [&](f32x4 v, int k) __attribute__((always_inline)) {  // (every thread has read its own)
    f32x4 e4;
#pragma unroll
    for (int e = 0; e < 4; ++e) e4[e] = prob(v[e], c, m, 0.f);
    store4(out, (k * TPB + tid) * 4, 0, V, e4);
  });
}

// ---- longer rows whose probabilities are to replace the logits themselves: the launches below have no room for what they
// hand on before the logits have been read for the last time, so one workgroup takes a row, in about nine passes over it
// (64 rows of 128 256 normal logits: 261 us, one row 180; 8193 tokens 22.8 and 21.5).
__global__ __launch_bounds__(TPB) void sample_in_place_kernel(float* rows, int V, float c, float unit, float top_p, const float* __restrict__ u01,
                                                              int32_t* __restrict__ tokens) {
  __shared__ u64 copies[BINS * COPIES], hist[BINS], wave_tot[WAVES];
  __shared__ double need;
  __shared__ float red[WAVES];
  __shared__ int bin;
  const int tid = threadIdx.x;
  float* x = rows + (int64_t)blockIdx.x * V;
  float m = -INFINITY;
#pragma unroll 8
  for (int i = tid; i < V; i += TPB) m = fmaxf(m, x[i]);
  m = finite(block_max<TPB>(m, red));
  auto members = [&](auto&& use) __attribute__((always_inline)) {
#pragma unroll 8
    for (int i = tid; i < V; i += TPB) {
      const float v = x[i];
      use(key_of(v), [&] { return mass_of(prob(v, c, m, 0.f), unit); });
    }
  };
  const uint32_t tau = search_keys(members, 0u, 0xFFFFFFFFu, top_p, -1., copies, hist, &bin, &need);
  u64 mine = 0;
  members([&](uint32_t key, auto&& mass) { mine += key >= tau ? mass() : 0ull; });
  mine = wave_sum(mine);
  if ((tid & 63) == 0) wave_tot[tid >> 6] = mine;
  __syncthreads();
  u64 nucleus = 0;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) nucleus += wave_tot[w];
  __syncthreads();
  if (nucleus) choose_among(x, V, Masses{c, m, 0.f, unit, logit_of(tau)}, draw_target(u01[blockIdx.x], nucleus), 0, copies, tokens + blockIdx.x);
  else if (tid == 0) tokens[blockIdx.x] = 0;
  __syncthreads();  // the logits have been read for the last time
#pragma unroll 8
  for (int i = tid; i < V; i += TPB) x[i] = prob(x[i], c, m, 0.f);
}

// ---- longer rows, first launch: largest logit and bin masses of every chunk
template <int PER>
__global__ __launch_bounds__(TPB) void sample_bins_kernel(const float* __restrict__ logits, int V, int chunk, float c, float unit, float* __restrict__ scratch) {
  __shared__ u64 copies[BINS * COPIES], hist[BINS];
  __shared__ float red[WAVES];
  const int tid = threadIdx.x, first = blockIdx.y * chunk, n = min(chunk, V - first);
  constexpr int SUB = 4 * PER * TPB;
  const float* lg = logits + (int64_t)blockIdx.x * V + first;
  f32x4 x[PER];
  auto load = [&](int base) __attribute__((always_inline)) { load_groups(x, lg + base, n - base); };
  float m = -INFINITY;
  for (int base = 0; base < n; base += SUB) {
    load(base);
#pragma unroll
    for (int k = 0; k < PER; ++k) m = fmaxf(m, fmaxf(fmaxf(x[k][0], x[k][1]), fmaxf(x[k][2], x[k][3])));
  }
  for (int i = tid; i < BINS * COPIES; i += TPB) copies[i] = 0;
  m = finite(block_max<TPB>(m, red));
  const int top = bin_of(m, c);
  const float r = way_down(m, c);
  for (int base = 0; base < n; base += SUB) {
    if (n > SUB) load(base);
    each_group(x, [&](f32x4 v, int) __attribute__((always_inline)) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const u64 w = mass_of(prob(v[e], c, m, r), unit);  // (0 for the -inf behind the end)
        if (w) atomicAdd(&copies[bin_number(top, bin_of(v[e], c)) * COPIES + (tid & (COPIES - 1))], w);
      }
    });
  }
  __syncthreads();
  sum_copies<COPIES>(copies, hist);
  float* region = scratch + (int64_t)blockIdx.x * V + first;
  if (tid < BINS) {
    region[H_BINS + tid] = __uint_as_float((uint32_t)hist[tid]);
    region[H_BINS + BINS + tid] = __uint_as_float((uint32_t)(hist[tid] >> 32));
  }
  if (tid == 0) {
    region[H_MAX] = m;
    region[H_DONE] = __int_as_float(0);
  }
}

__device__ __forceinline__ u64 chunk_bin(const float* region, int bin) {
  return ((u64)__float_as_uint(region[H_BINS + BINS + bin]) << 32) | __float_as_uint(region[H_BINS + bin]);
}

// What a workgroup of the second launch hands to the last one of its row, which may run behind another L2, is written and read with
// device-scope accesses; the writers wait for theirs to complete, then one thread counts the workgroup in.
__device__ __forceinline__ void hand_on(float* p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ float handed_on(const float* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void wait_for_stores() {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
}

// ---- second launch: probabilities of every chunk (but its reserved head) and its members of the bin that holds tau; the workgroup of
// a row that finishes last looks for tau and the token, and writes the probabilities of the reserved heads
struct DrawLds {
  u64 hist[BINS];
  u64 runs[MAX_RUNS];
  int chunk_at[MAX_CHUNKS + 1];  // first candidate of a chunk in the lists
  u64 wave_tot[WAVES];
  double need;
  int reached[2 * WAVES];
  uint32_t klo, khi;
  int bin, count, where, last;
  // candidates: masses (or copies of bins), keys, and the runs they lie in, counted through the row
  u64 mass[ROW_CAND];
  uint32_t keys[ROW_CAND];
  uint16_t run[ROW_CAND];
};
static_assert(2 * sizeof(DrawLds) <= 160 * 1024, "two workgroups to a compute unit");
static_assert(ROW_CAND >= BINS * COPIES, "what shares the masses' space");

// The elements of a chunk in runs of `length` (a multiple of 256), `per_chunk` of them, of which a row has at most MAX_RUNS: masses by run lead to the token
// without another look at a chunk
struct RowRuns {
  int length, per_chunk;
  __device__ __host__ RowRuns(int chunk, int n_chunks) {
    const int most = MAX_RUNS / n_chunks, parts = (chunk + 255) / 256;
    length = (parts + most - 1) / most * 256;
    per_chunk = (chunk + length - 1) / length;
  }
};
// Largest logit of a chunk, its way down, and how far bins and masses lie below the row's; lane k holds those of chunk k
struct Ref { float m, r; int down, back; };
struct Refs {
  Ref lane;
  __device__ __forceinline__ Refs(float head, float c, int top, double oct) : lane{head, way_down(head, c), top - bin_of(head, c), octaves_between(oct, octave_of(head, c))} {}
  __device__ __forceinline__ Ref operator[](int k) const {  // k: the same in all lanes
    k = __builtin_amdgcn_readfirstlane(k);
    return Ref{__uint_as_float(lane_of(__float_as_uint(lane.m), k)), __uint_as_float(lane_of(__float_as_uint(lane.r), k)), (int)lane_of((uint32_t)lane.down, k),
               (int)lane_of((uint32_t)lane.back, k)};
  }
};

// Where the row's list in LDS does not do.  LISTS: the chunks' lists hold all members of bin b, too many of them together (128 256 normal logits
// of a standard deviation up to 1: 4000 to 8000).  ROW: one of them does not (a row that is flat to within a tenth of an octave), and the row
// itself is read: by one wavefront per chunk, or several where there are fewer chunks (512 rows of 32 000 near-equal tokens: 163 us)
enum { IN_LDS = 0, LISTS = 1, ROW = 2 };
struct RowReader {
  const float *lg_row, *row;
  int V, chunk, n_chunks;
  float c, unit;
  int top, b;
  Refs refs;
  __device__ __forceinline__ int team() const {  // wavefronts per chunk
    int t = 1;
    while (2 * t * n_chunks <= WAVES) t *= 2;
    return t;
  }
  // use(key, mass, place) of every entry of the chunks' lists, four a lane on their way
  template <bool PLACES, typename U>
  __device__ __forceinline__ void listed(const DrawLds& S, int list0, U&& use) const {
    constexpr int F = 4;
    const int t = team(), lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int k = wave / t; k < n_chunks; k += WAVES / t) {
      const float* list = row + (int64_t)k * chunk + list0;
      const int cnt = S.chunk_at[k + 1] - S.chunk_at[k];
      const Ref R = refs[k];
#pragma unroll 1
      for (int i0 = wave % t * (64 * F) + lane; i0 - lane < cnt; i0 += 64 * F * t) {
        float v[F], at[F];
#pragma unroll
        for (int u = 0; u < F; ++u) {
          const int i = min(i0 + 64 * u, cnt - 1);
          v[u] = handed_on(list + 2 * i);
          if constexpr (PLACES) at[u] = handed_on(list + 2 * i + 1);
        }
#pragma unroll
        for (int u = 0; u < F; ++u)
          if (i0 + 64 * u < cnt) use(key_of(v[u]), [&] { return shifted(mass_of(prob(v[u], c, R.m, R.r), unit), R.back); }, k, PLACES ? __float_as_int(at[u]) : 0);
      }
    }
  }
  // use(key, mass) of every member of bin b in chunk k, and done(i) behind every 256 elements from i on (one wavefront's)
  template <typename U, typename D>
  __device__ __forceinline__ void members(int k, int t, U&& use, D&& done) const {
    const int64_t f = (int64_t)k * chunk;
    const int n = min(chunk, (int)(V - f)), lane = threadIdx.x & 63;
    const Ref R = refs[k];
    auto at = [&](int i) __attribute__((always_inline)) { return load4(lg_row + f, i + lane * 4, n); };
    int i = __builtin_amdgcn_readfirstlane((threadIdx.x >> 6) % t * 256);
    f32x4 next = at(i);
#pragma unroll 1
    for (; i < n; i += 256 * t) {
      const f32x4 v = next;
      next = at(i + 256 * t);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (i + lane * 4 + e < n && bin_number(top, bin_of(v[e], c)) == b) use(key_of(v[e]), [&] { return shifted(mass_of(prob(v[e], c, R.m, R.r), unit), R.back); });
      done(i);
    }
  }
  // the keys of the bin are binned again, 256 linear bins at a time, until one is left; three or four passes
  __device__ __forceinline__ uint32_t tau(DrawLds& S, int where, int list0, double need, uint32_t klo, uint32_t khi) const {
    const int t = team();
    auto all = [&](auto&& use) __attribute__((always_inline)) {
      if (where == LISTS)
        listed<false>(S, list0, [&](uint32_t key, auto&& mass, int, int) __attribute__((always_inline)) { use(key, mass); });
      else
        for (int k = (threadIdx.x >> 6) / t; k < n_chunks; k += WAVES / t) members(k, t, use, [](int) {});
    };
    return search_keys(all, klo, khi, 0.f, need, S.mass, S.hist, &S.bin, &S.need);  // (copies of the bins in the space of the masses)
  }
  __device__ __forceinline__ void add_masses(DrawLds& S, int where, int list0, uint32_t tau, RowRuns runs) const {  // of the bin's members that are in, to their runs
    if (where == LISTS) {
      listed<true>(S, list0, [&](uint32_t key, auto&& mass, int k, int place) __attribute__((always_inline)) {
        if (key >= tau) atomicAdd(&S.runs[k * runs.per_chunk + place / runs.length], mass());
      });
      return;
    }
    const int t = team();
    for (int k = (threadIdx.x >> 6) / t; k < n_chunks; k += WAVES / t) {
      u64 q = 0;
      members(k, t, [&](uint32_t key, auto&& mass) { q += key >= tau ? mass() : 0ull; }, [&](int i) {
        q = wave_sum(q);
        if ((threadIdx.x & 63) == 0 && q) atomicAdd(&S.runs[k * runs.per_chunk + i / runs.length], q);
        q = 0;
      });
    }
  }
};

// The workgroup of a row that finishes last: tau, the token, and the probabilities that the chunks' headers and lists stood in the way of.
struct RowEnd { const float* u01; float* row; int32_t* tokens; float m; RowRuns runs; };
__device__ __forceinline__ void end_of_row(const RowReader& reader, const RowEnd& end, DrawLds& S) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), n_chunks = reader.n_chunks, chunk = reader.chunk, V = reader.V;
  const int per_chunk = end.runs.per_chunk, n_runs = n_chunks * per_chunk, list0 = head_of(per_chunk), most = cand_max(per_chunk);
  const float *lg_row = reader.lg_row, c = reader.c, unit = reader.unit, m = end.m;
  float* const row = end.row;
  // a thread looks after a run of the row
  const int run_chunk = min(tid / per_chunk, n_chunks - 1);
  u64 run_mass = 0;
  if (tid < n_runs) {
    const float* reg = row + (int64_t)run_chunk * chunk + H_RUNS + 2 * (tid - run_chunk * per_chunk);
    const uint32_t lo = __float_as_uint(handed_on(reg)), hi = __float_as_uint(handed_on(reg + 1));
    run_mass = (u64)hi << 32 | lo;
  }
  if (wave == 0) {  // places of the chunks' candidates in one list
    uint32_t mine = 0, klo = 0xFFFFFFFFu, khi = 0u;
    if (lane < n_chunks) {
      const float* reg = row + (int64_t)lane * chunk;
      mine = __float_as_uint(handed_on(reg + H_COUNT));
      klo = __float_as_uint(handed_on(reg + H_KLO));
      khi = __float_as_uint(handed_on(reg + H_KHI));
    }
    const uint32_t upto = wave_scan(mine);
    const int where = __any(mine > (uint32_t)most) ? ROW : lane_of(upto, 63) > ROW_CAND ? LISTS : IN_LDS;
    S.chunk_at[lane + 1] = (int)upto;
    wave_range(klo, khi);
    if (lane == 0) { S.chunk_at[0] = 0; S.where = where; S.klo = klo; S.khi = khi; }
  }
  const float u = *end.u01;
  S.runs[tid] = shifted(run_mass, __shfl(reader.refs.lane.back, run_chunk));
  __syncthreads();
  const uint32_t klo = S.klo, khi = S.khi;
  const int where = S.where;
  if (__builtin_expect(where == IN_LDS, 1)) {  // a wavefront looks after chunk number `wave` and every sixteenth from there
#pragma unroll 1
    for (int k = wave; k < n_chunks; k += WAVES) {
      const int at = S.chunk_at[k], cnt = S.chunk_at[k + 1] - at;
      const float* reg = row + (int64_t)k * chunk + list0;
      const Ref R = reader.refs[k];
#pragma unroll 1
      for (int i = lane; i < cnt; i += 64) {
        const float v = handed_on(reg + 2 * i);
        S.run[at + i] = (uint16_t)(k * per_chunk + __float_as_int(handed_on(reg + 2 * i + 1)) / end.runs.length);
        S.keys[at + i] = key_of(v);
        S.mass[at + i] = shifted(mass_of(prob(v, c, R.m, R.r), unit), R.back);
      }
    }
  }
  __syncthreads();
  uint32_t tau;
  if (__builtin_expect(where == IN_LDS, 1)) {
    const int n = S.chunk_at[n_chunks];
    tau = n ? find_tau(S.keys, S.mass, n, S.need, klo, khi == 0xFFFFFFFFu ? khi : khi + 1u, S.reached) : 0u;
#pragma unroll 1
    for (int i = tid; i < n; i += TPB)
      if (S.keys[i] >= tau) atomicAdd(&S.runs[S.run[i]], S.mass[i]);
  } else {
    tau = reader.tau(S, where, list0, S.need, klo, khi);
    reader.add_masses(S, where, list0, tau, end.runs);
  }
  __syncthreads();
  // the run, in units of the row's reference; it is the owner of this thread's or of no thread (a row without any finite logit)
  const u64 mine = S.runs[tid], incl = wave_scan(mine);
  if (lane == 63) S.wave_tot[wave] = incl;
  __syncthreads();
  const u64 upto_wave = wave_scan(lane < WAVES ? S.wave_tot[lane] : 0ull), nucleus = lane_of(upto_wave, WAVES - 1);
  const u64 before = incl - mine + (wave ? lane_of(upto_wave, wave - 1) : 0ull);
  const u64 target = draw_target(u, nucleus);
  const u64 found = __ballot(before <= target && target < before + mine);
  if (found) {  // this wavefront takes it
    const int owner = __ffsll((long long)found) - 1;
    const int k = (int)lane_of((uint32_t)run_chunk, owner), first = ((wave * 64 + owner) - k * per_chunk) * end.runs.length;
    const int64_t f = (int64_t)k * chunk;
    const int n = min(min(chunk, (int)(V - f)), first + end.runs.length);
    const Ref R = reader.refs[k];
    // the running mass is counted in the chunk's own units, in which it is at least what was counted above
    u64 left = (target - lane_of(before, owner)) << R.back;
    const Masses mass{c, R.m, R.r, unit, logit_of(tau)};
#pragma unroll 1
    for (int i0 = first; i0 < n; i0 += 256) {
      const f32x4 v = load4(lg_row + f, i0 + lane * 4, n);
      const u64 w = mass(v), upto = wave_scan(w), hit = __ballot(upto > left);
      if (hit) {
        if (lane == __ffsll((long long)hit) - 1) *end.tokens = (int)f + i0 + lane * 4 + mass.member(v, left - (upto - w));
        break;
      }
      left -= lane_of(upto, 63);
    }
  } else if (!nucleus && tid == 0) {
    *end.tokens = 0;
  }
  // the headers are no longer needed
#pragma unroll 1
  for (int k = wave; k < n_chunks; k += WAVES) {
    const int64_t f = (int64_t)k * chunk;
    const int used = list0 + 2 * min(S.chunk_at[k + 1] - S.chunk_at[k], most);
#pragma unroll 1
    for (int i = lane * 4; i < used; i += 256) {
      f32x4 v = load4(lg_row + f, i, RESERVED);  // (every chunk is longer than its reserved head)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = prob(v[e], c, m, 0.f);
      store4(row + f, i, 0, used, v);
    }
  }
}

template <int PER>
__global__ __launch_bounds__(TPB, 8) void sample_draw_kernel(const float* __restrict__ logits, int V, int chunk, int n_chunks, float c, float unit, float top_p,
                                                          const float* __restrict__ u01, float* scratch, int32_t* __restrict__ tokens) {
  extern __shared__ __align__(16) char smem[];
  DrawLds& S = *reinterpret_cast<DrawLds*>(smem);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), own = blockIdx.y;
  const int first = own * chunk, n = min(chunk, V - first);
  const float* lg_row = logits + (int64_t)blockIdx.x * V;
  const float* lg = lg_row + first;
  float* row = scratch + (int64_t)blockIdx.x * V;
  float* region = row + first;
  constexpr int SUB = 4 * PER * TPB;
  f32x4 x[PER];
  auto load = [&](int base) __attribute__((always_inline)) { load_groups(x, lg + base, n - base); };
  // bins of the row's chunks: four chunks side by side, one bin a thread, NB times in flight; they, the headers and the logits arrive together
  constexpr int SIDE = TPB / BINS, NB = PER > 2 ? 2 : 4;
  u64 w[NB];
  const int bin_mine = tid & (BINS - 1), k_mine = tid / BINS;
  auto load_bins = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < NB; ++q) w[q] = chunk_bin(row + (int64_t)min(k0 + q * SIDE + k_mine, n_chunks - 1) * chunk, bin_mine);
  };
  const float head = lane < n_chunks ? row[(int64_t)lane * chunk + H_MAX] : -FLT_MAX;  // largest logit of chunk `lane`
  load_bins(0);
  load(0);
  const float m = wave_max(head);
  if (tid < BINS) S.hist[tid] = 0;
  S.runs[tid] = 0;
  if (tid == 0) { S.count = 0; S.klo = 0xFFFFFFFFu; S.khi = 0u; }
  const RowRuns runs(chunk, n_chunks);
  const int list0 = head_of(runs.per_chunk), most = cand_max(runs.per_chunk);
  const int top = bin_of(m, c);
  __syncthreads();
  const Refs refs(head, c, top, octave_of(m, c));
#pragma unroll 1
  for (int k0 = 0; k0 < n_chunks; k0 += NB * SIDE) {
    if (k0) load_bins(k0);
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      const int k = k0 + q * SIDE + k_mine;
      if (k >= n_chunks) break;
      const Ref R = refs[k];
      const u64 v = shifted(w[q], R.back);
      if (v) atomicAdd(&S.hist[min(BINS - 1, bin_mine + R.down)], v);
    }
  }
  __syncthreads();
  if (tid < 64) find_boundary(S.hist, top_p, -1., &S.bin, &S.need);
  __syncthreads();
  const int b = S.bin;
  const InBin in_bin(top - b, b == BINS - 1, b == 0, c);
  const Ref R = refs[own];
  const float above = in_bin.above();
  for (int base = 0; base < n; base += SUB) {
    if (base) load(base);
    list_members(x, in_bin, n - base, &S.count, &S.klo, &S.khi, [&](int at, float v, int i) __attribute__((always_inline)) {
      if (at < most) {
        hand_on(region + list0 + 2 * at, v);
        hand_on(region + list0 + 2 * at + 1, __int_as_float(base + i));
      }
    });
    each_group(x, [&](f32x4 v, int k) __attribute__((always_inline)) {  // masses of what lies above, by run
      const f32x4 t = v * in_bin.scale;
      if (!__any(fmaxf(fmaxf(t[0], t[1]), fmaxf(t[2], t[3])) >= above)) return;
      u64 w = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) w += t[e] >= above ? mass_of(prob(v[e], c, R.m, R.r), unit) : 0ull;
      w = wave_sum(w);
      if (lane == 0 && w) atomicAdd(&S.runs[(base + (k * TPB + wave * 64) * 4) / runs.length], w);
    });
    if (base + SUB >= n) wait_for_stores();  // in front of the probabilities, whose completion nobody waits for
    each_group(x, [&](f32x4 v, int k) __attribute__((always_inline)) {
      f32x4 e4;
#pragma unroll
      for (int e = 0; e < 4; ++e) e4[e] = prob(v[e], c, m, 0.f);
      store4(region, base + (k * TPB + tid) * 4, RESERVED, n, e4);
    });
  }
  __syncthreads();
  if (tid < runs.per_chunk) {
    hand_on(region + H_RUNS + 2 * tid, __uint_as_float((uint32_t)S.runs[tid]));
    hand_on(region + H_RUNS + 2 * tid + 1, __uint_as_float((uint32_t)(S.runs[tid] >> 32)));
    if (tid == 0) {
      hand_on(region + H_COUNT, __int_as_float(S.count));
      hand_on(region + H_KLO, __uint_as_float(S.klo));
      hand_on(region + H_KHI, __uint_as_float(S.khi));
    }
    wait_for_stores();  // (one wavefront: a chunk has at most 64 runs)
  }
  if (tid == 0) {
    S.last = __hip_atomic_fetch_add(reinterpret_cast<int*>(row + H_DONE), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n_chunks - 1;
  }
  {  // the part of the reserved head that no candidate took
    static_assert(RESERVED == 4 * TPB, "a thread's first group");
    f32x4 v = n > SUB ? load4(lg, tid * 4, n) : x[0];
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = prob(v[e], c, m, 0.f);
    store4(region, tid * 4, list0 + 2 * min(S.count, most), RESERVED, v);
  }
  __syncthreads();
  if (!S.last) return;
  const RowReader reader{lg_row, row, V, chunk, n_chunks, c, unit, top, b, refs};
  const RowEnd end{u01 + blockIdx.x, row, tokens + blockIdx.x, m, runs};
  end_of_row(reader, end, S);
}

// factor that turns a probability into the high part of its mass: 2^20, and half of that per doubling of the row beyond 2^19
float mass_unit(int vocab) {
  float unit = 1048576.f;
  for (int64_t n = 1 << 19; n < vocab; n *= 2) unit *= 0.5f;
  return unit;
}

constexpr int MAX_DEVICES = 64;
std::mutex g_device_mutex;         // guards the two tables below
bool g_lds_allowed[MAX_DEVICES];   // the kernels with more than 64 KiB of LDS have been announced to the device
float* g_scratch_ptr[MAX_DEVICES]; // device address of the static scratch array on each device, once looked up

int current_device(int* dev) {
  *dev = -1;
  const hipError_t e = hipGetDevice(dev);
  if (e != hipSuccess) { set_error("hipGetDevice failed: %s", hipGetErrorString(e)); return WWW_E_HIP; }
  if (*dev < 0 || *dev >= MAX_DEVICES) { set_error("device index %d out of range", *dev); return WWW_E_HIP; }
  return WWW_OK;
}

int allow_lds() {
  int dev;
  if (int rc = current_device(&dev)) return rc;
  std::lock_guard<std::mutex> lock(g_device_mutex);
  if (g_lds_allowed[dev]) return WWW_OK;
  auto allow = [](const void* kernel, size_t bytes) { return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes); };
  hipError_t e = allow(reinterpret_cast<const void*>(&sample_row_kernel<2, 2>), sizeof(SmallLds<2>));
  if (e == hipSuccess) e = allow(reinterpret_cast<const void*>(&sample_draw_kernel<2>), sizeof(DrawLds));
  if (e == hipSuccess) e = allow(reinterpret_cast<const void*>(&sample_draw_kernel<4>), sizeof(DrawLds));
  if (e != hipSuccess) { set_error("hipFuncSetAttribute failed: %s", hipGetErrorString(e)); return WWW_E_HIP; }
  g_lds_allowed[dev] = true;
  return WWW_OK;
}

}  // namespace

WWW_EXPORT int www_sample_top_p(const float* logits_dev, int32_t batch, int32_t vocab, float temperature, float top_p,
                                const float* u01_dev, float* scratch_dev, int32_t* tokens_dev, void* hip_stream) {
  if (batch < 0 || vocab <= 0) { set_error("negative batch or non-positive vocab"); return WWW_E_INVALID_ARG; }
  if (!(temperature > 0.f) || !(top_p > 0.f && top_p <= 1.f)) {
    set_error("temperature must be positive (temperature 0 is the greedy token of www_decode_step) and top_p in (0, 1]");
    return WWW_E_INVALID_ARG;
  }
  if (batch == 0) return WWW_OK;
  if (!logits_dev || !u01_dev || !scratch_dev || !tokens_dev) { set_error("NULL pointer argument"); return WWW_E_INVALID_ARG; }
  const uint64_t from = (uint64_t)logits_dev, to = (uint64_t)scratch_dev, bytes = (uint64_t)batch * (uint64_t)vocab * sizeof(float);
  if (from != to && from < to + bytes && to < from + bytes) {
    set_error("scratch_dev overlaps logits_dev (it may be the same buffer, or one that does not overlap)");
    return WWW_E_INVALID_ARG;
  }
  const hipStream_t st = (hipStream_t)hip_stream;
  const float c = std::min(1.4426950408889634f / temperature, FLT_MAX / 8.f);  // (finite, times the bins of an octave too: no 0 * inf)
  if (c == 0.f) top_p = 1.f;  // infinite temperature: equal probabilities, which enter the nucleus together
  const float unit = mass_unit(vocab);
  if (int rc = allow_lds()) return rc;
  if (vocab <= 8 * TPB) {
    hipLaunchKernelGGL((sample_row_kernel<2, 2>), dim3(batch), dim3(TPB), sizeof(SmallLds<2>), st, logits_dev, vocab, c, unit, top_p, u01_dev, scratch_dev, tokens_dev);
  } else if (scratch_dev == logits_dev) {
    hipLaunchKernelGGL(sample_in_place_kernel, dim3(batch), dim3(TPB), 0, st, scratch_dev, vocab, c, unit, top_p, u01_dev, tokens_dev);
  } else {
    // chunks of equal length, of up to 8192 tokens, or 16 384 where there would be more of these than compute units (us with the shorter and the
    // longer: 128 256 tokens, 1, 16, 20, 48 and 64 rows 16.2 / 18.4, 19.7 / 22.4, 24.8 / 23.6, 33.5 / 31.8 and 36.7 / 30.7; 32 000 tokens, 64 rows
    // 16.0 / 19.3); longer only where MAX_CHUNKS do not hold the row.  The last one falls short of the others by less than the number of
    // chunks, so every chunk has room for its reserved head.
    const int shorter = (vocab + 8191) / 8192, n_chunks = std::min((int64_t)batch * shorter <= 256 ? shorter : (vocab + 16383) / 16384, MAX_CHUNKS);
    const int chunk = (int)(((int64_t)vocab + n_chunks - 1) / n_chunks);
    const dim3 grid(batch, n_chunks);
    auto bins = chunk > 8192 ? sample_bins_kernel<4> : sample_bins_kernel<2>;
    auto draw = chunk > 8192 ? sample_draw_kernel<4> : sample_draw_kernel<2>;
    hipLaunchKernelGGL(bins, grid, dim3(TPB), 0, st, logits_dev, vocab, chunk, c, unit, scratch_dev);
    hipLaunchKernelGGL(draw, grid, dim3(TPB), sizeof(DrawLds), st, logits_dev, vocab, chunk, n_chunks, c, unit, top_p, u01_dev, scratch_dev, tokens_dev);
  }
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess) { set_error("sampling kernel launch failed: %s", hipGetErrorString(err)); return WWW_E_HIP; }
  return WWW_OK;
}

// ------------------------------------------------------------------------------------------------
// The same sampling for callers that cannot allocate device memory (code under HIP graph capture, serving loops and
// harnesses that forbid hipMalloc): the [batch][vocab] buffer of unnormalised probabilities lives in a file-scope
// device array instead of a caller-provided one.  Every GPU holds its own copy of the array at its own address until
// the process ends; the address is looked up once per device and kept.  All calls on one GPU share the array: calls
// that overlap on one GPU (different streams, different host threads) race.  Nothing in it has to start at zero - the
// kernel writes every element it later reads.
static __device__ __align__(256) float scratch[WWW_SAMPLE_STATIC_MAX_FLOATS];

namespace {
// device address of this device's copy of `scratch` (the array's name itself is only a host-side stand-in)
int static_scratch(float** out) {
  int dev;
  if (int rc = current_device(&dev)) return rc;
  std::lock_guard<std::mutex> lock(g_device_mutex);
  if (!g_scratch_ptr[dev]) {
    float* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr) { set_error("hipGetSymbolAddress failed: %s", hipGetErrorString(e)); return WWW_E_HIP; }
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return WWW_OK;
}
}  // namespace

WWW_EXPORT int www_sample_top_p_static(const float* logits_dev, int32_t batch, int32_t vocab, float temperature, float top_p,
                                       const float* u01_dev, int32_t* tokens_dev, void* hip_stream) {
  if (batch < 0 || vocab <= 0) { set_error("negative batch or non-positive vocab"); return WWW_E_INVALID_ARG; }
  if ((uint64_t)batch * (uint64_t)vocab > (uint64_t)WWW_SAMPLE_STATIC_MAX_FLOATS) {
    set_error("batch * vocab = %llu exceeds the %llu floats of the built-in scratch array; use www_sample_top_p with a buffer of your own",
              (unsigned long long)((uint64_t)batch * (uint64_t)vocab), (unsigned long long)WWW_SAMPLE_STATIC_MAX_FLOATS);
    return WWW_E_CAPACITY;
  }
  if (batch == 0) {  // still validate, as www_sample_top_p does
    if (!(temperature > 0.f) || !(top_p > 0.f && top_p <= 1.f)) { set_error("temperature must be positive and top_p in (0, 1]"); return WWW_E_INVALID_ARG; }
    return WWW_OK;
  }
  float* ptr = nullptr;
  if (int rc = static_scratch(&ptr)) return rc;
  return www_sample_top_p(logits_dev, batch, vocab, temperature, top_p, u01_dev, ptr, tokens_dev, hip_stream);
}
