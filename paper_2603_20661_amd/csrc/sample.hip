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
// bin's elements (one to three per cent of a row) are looked at individually.  All masses are integers - units of 2^-44 of
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
// chunks of at most 8192 tokens, one workgroup each (1024 workgroups for 64 rows), in three launches: bins of every chunk;
// probabilities and members of the decisive bin of every chunk; tau and the token of every row.  What the launches hand
// on lies in the first RESERVED floats of every chunk's part of the scratch buffer, which receive their probabilities
// last.
// Measured at 64 rows of 128 256 tokens: 849 -> 45 us (12 + 18 + 15; the 99 MB the first two launches cannot avoid moving
// take 19 us), 32 us for one row.  Rows of up to 8192 tokens fit one workgroup's registers and take one launch: 18 us at
// 8192 tokens, where the three launches take 27 (64 rows; 36 against 45 us for 512 rows).
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
constexpr int SUB = 8192;            // elements a workgroup of 256 threads holds in registers at a time
constexpr int MAX_CHUNKS = 1024;     // chunks of a row (longer rows take longer chunks)
constexpr int HEAD = 4 + 2 * BINS;   // start of a chunk's scratch: largest logit, candidates found, their least and largest key if they
                                     // are too many, bin masses (low words, high words)
constexpr int CAND_MAX = 508;        // room for a chunk's candidates behind that
constexpr int RESERVED = HEAD + CAND_MAX;
constexpr int ROW_CAND = 8192;       // candidates of a row that are looked at in LDS
constexpr int TPB = 1024;
constexpr int WAVES = TPB / 64;

typedef unsigned long long u64;

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

__device__ __forceinline__ u64 wave_sum(u64 v) {
#pragma unroll
  for (int s = 32; s >= 1; s >>= 1) v += __shfl_xor(v, s);
  return v;
}
__device__ __forceinline__ u64 wave_scan(u64 v) {  // inclusive
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int s = 1; s < 64; s <<= 1) {
    const u64 up = __shfl_up(v, s);
    if (lane >= s) v += up;
  }
  return v;
}

// least lo and largest hi of the wavefront
__device__ __forceinline__ void wave_range(uint32_t& lo, uint32_t& hi) {
#pragma unroll
  for (int s = 32; s >= 1; s >>= 1) {
    lo = min(lo, (uint32_t)__shfl_xor((int)lo, s));
    hi = max(hi, (uint32_t)__shfl_xor((int)hi, s));
  }
}
// place in a list, counted in LDS, for every lane that has something: one addition per wavefront (the order does not matter)
__device__ __forceinline__ int list_place(bool has, int* count) {
  const u64 who = __ballot(has);
  if (!who) return 0;
  const int lane = threadIdx.x & 63, leader = __ffsll((long long)who) - 1;
  int at = 0;
  if (lane == leader) at = atomicAdd(count, __popcll(who));
  return __shfl(at, leader) + __popcll(who & ((1ull << lane) - 1));
}

template <int NT>
__device__ float block_max(float v, float* red) {
#pragma unroll
  for (int s = 32; s >= 1; s >>= 1) v = fmaxf(v, __shfl_xor(v, s));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  float t = red[0];
#pragma unroll
  for (int w = 1; w < NT / 64; ++w) t = fmaxf(t, red[w]);
  return t;
}

// The first of BINS bins, largest elements first, at which the mass so far reaches `share` of the total (want < 0) or
// `want`; `need` is what its own members have to contribute.  Called by one whole wavefront.
__device__ void find_boundary(const u64* hist, float share, double want, int* bin, double* need) {
  const int lane = threadIdx.x & 63;
  u64 h[4], s = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) { h[i] = hist[lane * 4 + i]; s += h[i]; }
  const u64 incl = wave_scan(s);
  const double total = (double)__shfl(incl, 63);
  want = want < 0. ? (double)share * total : fmin(want, total);
  const u64 reached = __ballot((double)incl >= want);
  if (lane == (reached ? __ffsll((long long)reached) - 1 : 63)) {
    u64 before = incl - s;
    int i = 0;
    while (i < 3 && (double)(before + h[i]) < want) before += h[i++];
    *bin = lane * 4 + i;
    *need = fmin(want - (double)before, (double)h[i]);  // (sums beyond 2^53 are rounded: never more than the bin holds)
  }
}

// tau among n candidates: the largest key whose members' mass reaches `need` (the smallest key if rounding keeps even
// that from it).  A search with sixteen thresholds a round, one per wavefront.
__device__ uint32_t find_tau(const uint32_t* keys, const u64* mass, int n, double need, uint32_t lo, uint32_t hi, int* reached) {
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
    int c = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) c += reached[turn + w];  // (monotone: the first c thresholds reach it)
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
template <typename M>
__device__ uint32_t search_keys(M&& members, uint32_t lo, uint32_t last, float share, double want, u64* copies, u64* hist, int* bin, double* need) {
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
    if (tid < BINS) {
      u64 s = 0;
#pragma unroll
      for (int k = 0; k < COPIES; ++k) s += copies[tid * COPIES + ((k + tid) & (COPIES - 1))];
      hist[tid] = s;
    }
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

// The token: the first member (key >= tau) among elements [0, n) of x whose running mass exceeds `target`.  Each thread
// takes a contiguous run, so that the running masses of the threads follow index order.  All threads of the workgroup
// call it; `base` is added to the index.
__device__ void pick(const float* x, int n, float c, float m, float r, float unit, uint32_t tau, u64 target, int base, u64* wave_tot, int32_t* token) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int per = (n + TPB - 1) / TPB;
  const int i0 = min(tid * per, n), i1 = min(i0 + per, n);
  u64 mine = 0;
#pragma unroll 8
  for (int i = i0; i < i1; ++i) {
    const float v = x[i];
    mine += key_of(v) >= tau ? mass_of(prob(v, c, m, r), unit) : 0ull;
  }
  const u64 incl = wave_scan(mine);
  if (lane == 63) wave_tot[wave] = incl;
  __syncthreads();
  u64 before = incl - mine;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) before += w < wave ? wave_tot[w] : 0ull;
  if (before <= target && target < before + mine) {
    u64 run = before;
    int at = i0;
    for (int i = i0; i < i1; ++i) {
      const float v = x[i];
      if (key_of(v) >= tau) run += mass_of(prob(v, c, m, r), unit);
      if (target < run) { at = i; break; }
    }
    *token = base + at;
  }
}

// target of the draw inside a nucleus of mass `nucleus`
__device__ __forceinline__ u64 draw_target(float u, u64 nucleus) {
  const u64 t = (u64)((double)fmaxf(u, 0.f) * (double)nucleus);
  return t < nucleus ? t : (nucleus ? nucleus - 1 : 0ull);
}

// ---- rows of up to SUB tokens: one workgroup per row, everything in LDS
struct SmallLds {
  uint32_t keys[ROW_CAND];
  u64 mass[ROW_CAND];
  u64 hist[BINS];
  u64 wave_tot[WAVES];
  double need;
  float red[WAVES];
  int reached[2 * WAVES];
  uint32_t klo, khi;
  int bin, count;
};

__global__ __launch_bounds__(TPB) void sample_row_kernel(const float* logits, int V, float c, float unit, float top_p, const float* __restrict__ u01,
                                                         float* scratch, int32_t* __restrict__ tokens) {
  extern __shared__ __align__(16) char smem[];
  SmallLds& S = *reinterpret_cast<SmallLds*>(smem);
  const int tid = threadIdx.x, row = blockIdx.x;
  const bool in_place = scratch == logits;  // the probabilities then wait until the logits have been read for the last time
  const float* lg = logits + (int64_t)row * V;
  constexpr int PER = SUB / TPB;
  float x[PER];
  float m = -INFINITY;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = k * TPB + tid;
    x[k] = i < V ? lg[i] : -INFINITY;
    m = fmaxf(m, x[k]);
  }
  if (tid < BINS) S.hist[tid] = 0;
  if (tid == 0) { S.count = 0; S.klo = 0xFFFFFFFFu; S.khi = 0u; }
  m = finite(block_max<TPB>(m, S.red));
  const int top = bin_of(m, c);
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = k * TPB + tid;
    if (i < V) {
      const float e = prob(x[k], c, m, 0.f);
      if (!in_place) scratch[(int64_t)row * V + i] = e;
      const u64 w = mass_of(e, unit);
      if (w) atomicAdd(&S.hist[bin_number(top, bin_of(x[k], c))], w);
    }
  }
  __syncthreads();
  if (tid < 64) find_boundary(S.hist, top_p, -1., &S.bin, &S.need);
  __syncthreads();
  uint32_t klo = 0xFFFFFFFFu, khi = 0u;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const bool cand = k * TPB + tid < V && bin_number(top, bin_of(x[k], c)) == S.bin;
    const int at = list_place(cand, &S.count);
    if (cand) {
      const uint32_t key = key_of(x[k]);
      S.keys[at] = key;
      S.mass[at] = mass_of(prob(x[k], c, m, 0.f), unit);
      klo = min(klo, key);
      khi = max(khi, key);
    }
  }
  if (__any(khi)) {
    wave_range(klo, khi);
    if ((tid & 63) == 0) { atomicMin(&S.klo, klo); atomicMax(&S.khi, khi); }
  }
  __syncthreads();
  klo = S.klo; khi = S.khi;
  const uint32_t tau = S.count ? find_tau(S.keys, S.mass, S.count, S.need, klo, khi == 0xFFFFFFFFu ? khi : khi + 1u, S.reached) : 0u;
  // mass of the nucleus
  u64 mine = 0;
#pragma unroll
  for (int k = 0; k < PER; ++k)
    if (k * TPB + tid < V && key_of(x[k]) >= tau) mine += mass_of(prob(x[k], c, m, 0.f), unit);
  mine = wave_sum(mine);
  if ((tid & 63) == 0) S.wave_tot[tid >> 6] = mine;
  __syncthreads();
  u64 nucleus = 0;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) nucleus += S.wave_tot[w];
  __syncthreads();
  if (nucleus) pick(lg, V, c, m, 0.f, unit, tau, draw_target(u01[row], nucleus), 0, S.wave_tot, tokens + row);
  else if (tid == 0) tokens[row] = 0;  // (a row without any finite logit)
  if (!in_place) return;
  __syncthreads();  // the logits have been read for the last time
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = k * TPB + tid;
    if (i < V) scratch[(int64_t)row * V + i] = prob(x[k], c, m, 0.f);
  }
}

// ---- longer rows whose probabilities are to replace the logits themselves: the launches below have no room for what they
// hand on before the logits have been read for the last time, so one workgroup takes a row, in about nine passes over it
// (64 rows of 128 256 tokens: 323 us, one row 212).
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
  if (nucleus) pick(x, V, c, m, 0.f, unit, tau, draw_target(u01[blockIdx.x], nucleus), 0, wave_tot, tokens + blockIdx.x);
  else if (tid == 0) tokens[blockIdx.x] = 0;
  __syncthreads();  // the logits have been read for the last time
#pragma unroll 8
  for (int i = tid; i < V; i += TPB) x[i] = prob(x[i], c, m, 0.f);
}

// ---- longer rows, first launch: largest logit and bin masses of every chunk
__global__ __launch_bounds__(256) void sample_bins_kernel(const float* __restrict__ logits, int V, int chunk, float c, float unit, float* __restrict__ scratch) {
  __shared__ u64 hist[BINS * COPIES];
  __shared__ float red[4];
  const int tid = threadIdx.x, first = blockIdx.y * chunk, n = min(chunk, V - first);
  const float* lg = logits + (int64_t)blockIdx.x * V + first;
  float x[SUB / 256];
  auto load = [&](int base) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < SUB / 256; ++k) {
      const int i = base + k * 256 + tid;
      x[k] = i < n ? lg[i] : -INFINITY;
    }
  };
  float m = -INFINITY;
  for (int base = 0; base < n; base += SUB) {
    load(base);
#pragma unroll
    for (int k = 0; k < SUB / 256; ++k) m = fmaxf(m, x[k]);
  }
#pragma unroll
  for (int k = 0; k < COPIES; ++k) hist[k * 256 + tid] = 0;
  m = finite(block_max<256>(m, red));
  const int top = bin_of(m, c);
  const float r = way_down(m, c);
  for (int base = 0; base < n; base += SUB) {
    if (n > SUB) load(base);
#pragma unroll
    for (int k = 0; k < SUB / 256; ++k) {
      const u64 w = mass_of(prob(x[k], c, m, r), unit);  // (0 for the -inf behind the end)
      if (w) atomicAdd(&hist[bin_number(top, bin_of(x[k], c)) * COPIES + (tid & (COPIES - 1))], w);
    }
  }
  __syncthreads();
  u64 s = 0;
#pragma unroll
  for (int k = 0; k < COPIES; ++k) s += hist[tid * COPIES + ((k + tid) & (COPIES - 1))];
  float* region = scratch + (int64_t)blockIdx.x * V + first;
  region[4 + tid] = __uint_as_float((uint32_t)s);
  region[4 + BINS + tid] = __uint_as_float((uint32_t)(s >> 32));
  if (tid == 0) region[0] = m;
}

// Largest logit of a row, from its chunks' headers (called by every thread, the same value everywhere); lane k keeps the one
// of chunk k in `head`.
__device__ __forceinline__ float row_max(const float* row, int chunk, int n_chunks, float& head) {
  const int lane = threadIdx.x & 63;
  head = lane < n_chunks ? row[(int64_t)lane * chunk] : -FLT_MAX;
  float m = head;
  for (int k = lane + 64; k < n_chunks; k += 64) m = fmaxf(m, row[(int64_t)k * chunk]);
#pragma unroll
  for (int s = 32; s >= 1; s >>= 1) m = fmaxf(m, __shfl_xor(m, s));
  return m;
}
__device__ __forceinline__ u64 chunk_bin(const float* region, int bin) {
  return ((u64)__float_as_uint(region[4 + BINS + bin]) << 32) | __float_as_uint(region[4 + bin]);
}
// ---- second launch: probabilities of every chunk (but its reserved head) and its members of the bin that holds tau
__global__ __launch_bounds__(256) void sample_split_kernel(const float* __restrict__ logits, int V, int chunk, float c, float top_p, float* scratch) {
  __shared__ u64 hist[BINS];
  __shared__ double need;
  __shared__ uint32_t klo[4], khi[4];
  __shared__ int bin, count;
  const int tid = threadIdx.x, first = blockIdx.y * chunk, n = min(chunk, V - first);
  const float* lg = logits + (int64_t)blockIdx.x * V + first;
  float* row = scratch + (int64_t)blockIdx.x * V;
  float* region = row + first;
  float x[SUB / 256];
  auto load = [&](int base) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < SUB / 256; ++k) {
      const int i = base + k * 256 + tid;
      x[k] = i < n ? lg[i] : -INFINITY;
    }
  };
  load(0);
  hist[tid] = 0;
  if (tid == 0) count = 0;
  // bins of the row's chunks, one bin a thread, sixteen chunks in flight: they and the headers arrive together
  constexpr int NB = 16;
  u64 w[NB];
  const int n_chunks = gridDim.y;
  auto load_bins = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < NB; ++k) w[k] = chunk_bin(row + (int64_t)min(k0 + k, n_chunks - 1) * chunk, tid);
  };
  load_bins(0);
  float head;
  const float m = row_max(row, chunk, n_chunks, head);
  const int top = bin_of(m, c);
  const double oct = octave_of(m, c);
  __syncthreads();
  for (int k0 = 0; k0 < n_chunks; k0 += NB) {
    if (k0) load_bins(k0);
    const int k_lane = k0 + (tid & (NB - 1));  // lane k: chunk k0 + k
    const float mc = k0 < 64 ? __shfl(head, k_lane) : row[(int64_t)min(k_lane, n_chunks - 1) * chunk];
    const int down = top - bin_of(mc, c), back = octaves_between(oct, octave_of(mc, c));
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      const u64 v = k0 + k < n_chunks ? shifted(w[k], __builtin_amdgcn_readlane(back, k)) : 0ull;
      if (v) atomicAdd(&hist[min(BINS - 1, tid + __builtin_amdgcn_readlane(down, k))], v);
    }
  }
  __syncthreads();
  if (tid < 64) find_boundary(hist, top_p, -1., &bin, &need);
  __syncthreads();
  const int b = bin;
  for (int base = 0; base < n; base += SUB) {
    if (base) load(base);
#pragma unroll
    for (int k = 0; k < SUB / 256; ++k) {
      const int i = base + k * 256 + tid;
      if (i >= RESERVED && i < n) region[i] = prob(x[k], c, m, 0.f);
      const bool cand = i < n && bin_number(top, bin_of(x[k], c)) == b;
      const int at = list_place(cand, &count);
      if (cand && at < CAND_MAX) region[HEAD + at] = x[k];
    }
  }
  __syncthreads();
  if (tid == 0) region[1] = __int_as_float(count);
  if (count <= CAND_MAX) return;
  // more than the list holds: the range of their keys, for the search that replaces it
  uint32_t lo = 0xFFFFFFFFu, hi = 0u;
  for (int base = 0; base < n; base += SUB) {
    if (n > SUB) load(base);
#pragma unroll
    for (int k = 0; k < SUB / 256; ++k)
      if (base + k * 256 + tid < n && bin_number(top, bin_of(x[k], c)) == b) { lo = min(lo, key_of(x[k])); hi = max(hi, key_of(x[k])); }
  }
  wave_range(lo, hi);
  if ((tid & 63) == 0) { klo[tid >> 6] = lo; khi[tid >> 6] = hi; }
  __syncthreads();
  if (tid == 0) {
    region[2] = __uint_as_float(min(min(klo[0], klo[1]), min(klo[2], klo[3])));
    region[3] = __uint_as_float(max(max(khi[0], khi[1]), max(khi[2], khi[3])));
  }
}

// ---- third launch: tau and the token of every row, and the probabilities of the reserved heads
struct PickLds {
  uint32_t keys[ROW_CAND];
  u64 mass[ROW_CAND];
  u64 hist[BINS];
  u64 chunk_mass[MAX_CHUNKS];
  int chunk_at[MAX_CHUNKS];  // first candidate of a chunk in the lists above
  u64 wave_tot[WAVES];
  u64 target;
  double need;
  int reached[2 * WAVES];
  uint32_t klo[WAVES], khi[WAVES];
  int bin, n_cand, overflow, chunk;
};

__global__ __launch_bounds__(TPB) void sample_pick_kernel(const float* __restrict__ logits, int V, int chunk, int n_chunks, float c, float unit, float top_p,
                                                          const float* __restrict__ u01, float* scratch, int32_t* __restrict__ tokens) {
  extern __shared__ __align__(16) char smem[];
  PickLds& S = *reinterpret_cast<PickLds*>(smem);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float* lg = logits + (int64_t)blockIdx.x * V;
  float* row = scratch + (int64_t)blockIdx.x * V;
  // A wavefront looks after chunk number `wave` (and every sixteenth from there): its bins, and the logits of its reserved
  // head, are requested before anything else and kept, so that the chain of dependent reads below starts with one round trip.
  constexpr int HREG = RESERVED / 64;
  float hx[HREG];
  u64 hb[BINS / 64];
  {
    const int64_t f = (int64_t)min(wave, n_chunks - 1) * chunk;
#pragma unroll
    for (int i = 0; i < BINS / 64; ++i) hb[i] = chunk_bin(row + f, i * 64 + lane);
#pragma unroll
    for (int i = 0; i < HREG; ++i) hx[i] = lg[f + i * 64 + lane];
  }
  const float u = u01[blockIdx.x];
  if (tid < BINS) S.hist[tid] = 0;
  if (wave == 0) {  // places of the chunks' candidates in one list
    int at = 0, over = 0;
    for (int k0 = 0; k0 < n_chunks; k0 += 64) {
      const int k = k0 + lane;
      const int mine = k < n_chunks ? __float_as_int(row[(int64_t)k * chunk + 1]) : 0;
      over |= mine > CAND_MAX;
      int incl = mine;
#pragma unroll
      for (int s = 1; s < 64; s <<= 1) {
        const int up = __shfl_up(incl, s);
        if (lane >= s) incl += up;
      }
      if (k < n_chunks) S.chunk_at[k] = at + incl - mine;
      at += __shfl(incl, 63);
    }
    over = __any(over) || at > ROW_CAND;
    if (lane == 0) { S.n_cand = at; S.overflow = over; }
  }
  float head;
  const float m = row_max(row, chunk, n_chunks, head);
  const int top = bin_of(m, c);
  const double oct = octave_of(m, c);
  struct Ref { float m, r; int down, back; };  // largest logit of a chunk, its way down, and how far bins and masses lie below the row's
  auto ref_of = [&](float mc) __attribute__((always_inline)) { return Ref{mc, way_down(mc, c), top - bin_of(mc, c), octaves_between(oct, octave_of(mc, c))}; };
  const Ref own = ref_of(__shfl(head, wave));
  __syncthreads();
  const bool listed = !S.overflow;
  uint32_t klo = 0xFFFFFFFFu, khi = 0u;
  for (int k = wave; k < n_chunks; k += WAVES) {
    const float* region = row + (int64_t)k * chunk;
    const Ref R = k == wave ? own : ref_of(region[0]);
#pragma unroll
    for (int i = 0; i < BINS / 64; ++i) {
      const u64 v = shifted(k == wave ? hb[i] : chunk_bin(region, i * 64 + lane), R.back);
      if (v) atomicAdd(&S.hist[min(BINS - 1, i * 64 + lane + R.down)], v);
    }
    const int cnt = __float_as_int(region[1]);
    if (cnt <= CAND_MAX) {
      const int at = S.chunk_at[k];
      for (int i = lane; i < cnt; i += 64) {
        const float v = region[HEAD + i];
        const uint32_t key = key_of(v);
        if (listed) {
          S.keys[at + i] = key;
          S.mass[at + i] = shifted(mass_of(prob(v, c, R.m, R.r), unit), R.back);
        }
        klo = min(klo, key);
        khi = max(khi, key);
      }
    } else if (lane == 0) {
      klo = min(klo, __float_as_uint(region[2]));
      khi = max(khi, __float_as_uint(region[3]));
    }
  }
  wave_range(klo, khi);
  if (lane == 0) { S.klo[wave] = klo; S.khi[wave] = khi; }
  __syncthreads();
  if (wave == 0) find_boundary(S.hist, top_p, -1., &S.bin, &S.need);
#pragma unroll
  for (int w = 0; w < WAVES; ++w) { klo = min(klo, S.klo[w]); khi = max(khi, S.khi[w]); }
  __syncthreads();
  const int b = S.bin;
  // Where the lists do not do, the row itself is read: by one wavefront per chunk, or several where there are fewer chunks (512
  // rows of 32 000 near-equal tokens, 4 chunks: 530 -> 226 us)
  int team = 1;
  while (2 * team * n_chunks <= WAVES) team *= 2;
  auto members_of = [&](int k, const Ref& R, auto&& use) __attribute__((always_inline)) {  // use(key, mass) of every member of bin b
    const int64_t f = (int64_t)k * chunk;
    const int n = min(chunk, (int)(V - f));
#pragma unroll 8
    for (int i = wave % team * 64 + lane; i < n; i += 64 * team) {
      const float v = lg[f + i];
      if (bin_number(top, bin_of(v, c)) == b) use(key_of(v), [&] { return shifted(mass_of(prob(v, c, R.m, R.r), unit), R.back); });
    }
  };
  uint32_t tau;
  if (listed) {
    tau = S.n_cand ? find_tau(S.keys, S.mass, S.n_cand, S.need, klo, khi == 0xFFFFFFFFu ? khi : khi + 1u, S.reached) : 0u;
  } else {
    // The bin holds more elements than the lists (a row that is flat to within a tenth of an octave): its keys are binned
    // again, 256 linear bins at a time, until one key is left; three or four passes over the row.
    auto members = [&](auto&& use) __attribute__((always_inline)) {
      for (int k = wave / team; k < n_chunks; k += WAVES / team) members_of(k, ref_of(row[(int64_t)k * chunk]), use);
    };
    tau = search_keys(members, klo, khi, 0.f, S.need, S.mass, S.hist, &S.bin, &S.need);  // (copies of the bins in the space of the lists)
  }
  // mass of the nucleus in every chunk, in units of the row's reference
  for (int k = wave; k < n_chunks; k += WAVES) {
    const float* region = row + (int64_t)k * chunk;
    const Ref R = k == wave ? own : ref_of(region[0]);
    u64 s = 0;
#pragma unroll
    for (int i = 0; i < BINS / 64; ++i)
      if (min(BINS - 1, i * 64 + lane + R.down) < b) s += k == wave ? hb[i] : chunk_bin(region, i * 64 + lane);
    s = shifted(wave_sum(s), R.back);
    u64 q = 0;
    if (listed) {
      const int at = S.chunk_at[k], cnt = __float_as_int(region[1]);
      for (int i = lane; i < cnt; i += 64) q += S.keys[at + i] >= tau ? S.mass[at + i] : 0ull;
      q = wave_sum(q);
    }
    if (lane == 0) S.chunk_mass[k] = s + q;
  }
  if (!listed) {
    __syncthreads();
    for (int k = wave / team; k < n_chunks; k += WAVES / team) {
      u64 q = 0;
      members_of(k, ref_of(row[(int64_t)k * chunk]), [&](uint32_t key, auto&& mass) { q += key >= tau ? mass() : 0ull; });
      q = wave_sum(q);
      if (lane == 0) atomicAdd(&S.chunk_mass[k], q);
    }
  }
  __syncthreads();
  if (wave == 0) {
    u64 nucleus = 0;
    for (int k = lane; k < n_chunks; k += 64) nucleus += S.chunk_mass[k];
    nucleus = wave_sum(nucleus);
    const u64 target = draw_target(u, nucleus);
    u64 run = 0;
    int owner = -1;
    for (int k0 = 0; k0 < n_chunks && owner < 0; k0 += 64) {
      const u64 mine = k0 + lane < n_chunks ? S.chunk_mass[k0 + lane] : 0ull;
      const u64 incl = wave_scan(mine) + run;
      const u64 past = __ballot(incl > target);
      if (past) {
        owner = k0 + __ffsll((long long)past) - 1;
        if (k0 + lane == owner) S.target = target - (incl - mine);
      }
      run = __shfl(incl, 63);
    }
    if (lane == 0) { S.chunk = owner; if (owner < 0) tokens[blockIdx.x] = 0; }  // (no finite logit in the row)
  }
  __syncthreads();
  if (S.chunk >= 0) {
    const int64_t f = (int64_t)S.chunk * chunk;
    const Ref R = ref_of(row[f]);
    // the running mass inside the chunk is counted in the chunk's own units, in which it is at least what was counted above
    pick(lg + f, min(chunk, (int)(V - f)), c, R.m, R.r, unit, tau, S.target << R.back, (int)f, S.wave_tot, tokens + blockIdx.x);
  }
  __syncthreads();  // the headers are no longer needed
  for (int k = wave; k < n_chunks; k += WAVES) {
    const int64_t f = (int64_t)k * chunk;
#pragma unroll
    for (int i = 0; i < HREG; ++i) row[f + i * 64 + lane] = prob(k == wave ? hx[i] : lg[f + i * 64 + lane], c, m, 0.f);
  }
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
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&sample_row_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(SmallLds));
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&sample_pick_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(PickLds));
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
  if (vocab <= SUB) {
    hipLaunchKernelGGL(sample_row_kernel, dim3(batch), dim3(TPB), sizeof(SmallLds), st, logits_dev, vocab, c, unit, top_p, u01_dev, scratch_dev,
                       tokens_dev);
  } else if (scratch_dev == logits_dev) {
    hipLaunchKernelGGL(sample_in_place_kernel, dim3(batch), dim3(TPB), 0, st, scratch_dev, vocab, c, unit, top_p, u01_dev, tokens_dev);
  } else {
    // chunks of equal length, 4097 .. 8192 tokens (longer only above 8 Mi tokens); the last one falls short of the others
    // by less than the number of chunks, so every chunk has room for its reserved head
    const int n_chunks = std::min((vocab + SUB - 1) / SUB, MAX_CHUNKS), chunk = (int)(((int64_t)vocab + n_chunks - 1) / n_chunks);
    const dim3 grid(batch, n_chunks);
    hipLaunchKernelGGL(sample_bins_kernel, grid, dim3(256), 0, st, logits_dev, vocab, chunk, c, unit, scratch_dev);
    hipLaunchKernelGGL(sample_split_kernel, grid, dim3(256), 0, st, logits_dev, vocab, chunk, c, top_p, scratch_dev);
    hipLaunchKernelGGL(sample_pick_kernel, dim3(batch), dim3(TPB), sizeof(PickLds), st, logits_dev, vocab, chunk, n_chunks, c, unit, top_p, u01_dev,
                       scratch_dev, tokens_dev);
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
