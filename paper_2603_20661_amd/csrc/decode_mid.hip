// Residual GEMMs (O and down projection) of a decode step of 33 to 64 tokens: Y^T[n][t] = sum_k W[n][k] X[t][k], added to the
// residual stream, with the packed operand and the sums of squares of the next norm.
#include "decode_gemm.h"

// A workgroup of eight wavefronts owns 16 R rows, 64 tokens and a range of k.  Wavefront kw takes every eighth chunk of k and loads
// weights and activations straight into registers: no LDS and no barrier in the loop.  Against skinny_gemm_kernel (128 rows, activations
// through LDS, two or four times as many splits of k) a compute unit takes in twice the activations, from L2, but a tile is handed over by
// half as many workgroups, its epilogue has eight wavefronts instead of four, and 32 or 64 rows instead of 128 to finish.
// Bound by the memory's latency, the intake of a compute unit (24 KB per us from memory, 115 from L2) and the hand-over.
// 64 tokens, us, skinny_gemm_kernel -> this: 4096 x 4096 16.9 -> 14.7, 2048 x 2048 11.8 -> 9.0 (FP8 11.6 -> 8.4), 2048 x 8192 19.8 -> 16.8
// (FP8 17.7 -> 13.8), 1536 x 6144 17.6 -> 12.1.  FP8 weights with 64 rows spill 36 registers, int4 is slower but in 4096 x 4096: not built.
constexpr int MG_NW = 8, MG_TB = 4;
constexpr int mg_kc(int wmode) { return wmode == WMODE_FP8 ? 2 : 1; }  // k blocks of a chunk: of one 16-byte unit of weights
constexpr int mg_depth(int wmode) { return wmode == WMODE_FP8 ? 2 : 3; }  // chunks of weights, and k blocks of activations, on their way

template <int WMODE, int R>
__global__ __launch_bounds__(64 * MG_NW, 2) void mid_gemm_kernel(const GemmP p) {
  constexpr bool W8 = WMODE == WMODE_FP8;
  constexpr int KC = mg_kc(WMODE), D = mg_depth(WMODE), TB = MG_TB;
  static_assert((D * KC) % D == 0 && MG_NW % R == 0);
  __shared__ f32x4 red[MG_NW][R][TB][64];
  __shared__ float s_sq[R][16 * TB];
  __shared__ int s_last;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // Workgroup id -> work item: the k splits of a row tile, which hand partial results over, get ids that are equal modulo 8, so they
  // run behind one L2.
  const int slot = blockIdx.x >> 3, split = slot % p.ksplit, tile = (blockIdx.x & 7) + 8 * (slot / p.ksplit);
  if (tile >= p.row_tiles) return;  // grid padding when the row tiles are not a multiple of 8
  const int rg0 = tile * R;
  const int kb_begin = split * p.kb_per_split, nkb = min(p.KB, kb_begin + p.kb_per_split) - kb_begin, last = kb_begin + nkb - 1;
  const int n_w = ((nkb + KC - 1) / KC - wave + MG_NW - 1) / MG_NW;  // chunks of this wavefront (none: it only helps with the rest)

  // what this wavefront finishes: row group fr of the tile, token groups tbase, tbase + TSTEP ..
  constexpr int TSTEP = MG_NW / R, NT = TB / TSTEP;
  const int tsub = lane & 15, rsub = (lane >> 4) * 4, fr = wave % R, tbase = wave / R;
  const int frg = rg0 + fr, n0 = frg * 16 + rsub;  // (p.NRG is a multiple of R)

  struct WSet { u32x4 w[R]; } ws[D];
  struct XSet { u32x4 x[TB][2]; } xs[D];
  // columns without a token read the last one's lines again, groups of 16 without a token the last group's
  int xo[TB];
#pragma unroll
  for (int tb = 0; tb < TB; ++tb) {
    const int g = min(tb, (p.M - 1) / 16);
    xo[tb] = g * 128 + (lane & 48) + min(tsub, p.M - 1 - g * 16);
  }
  // (loads past the end of the k range are redirected to its last valid block, their products are skipped)
  auto load_w = [&](WSet& s, int i) __attribute__((always_inline)) {
    const int c = min(kb_begin / KC + wave + MG_NW * i, last / KC);  // (kb_begin is a multiple of 4)
#pragma unroll
    for (int r = 0; r < R; ++r) s.w[r] = p.W[((int64_t)c * p.NRG + rg0 + r) * 64 + lane];
  };
  auto load_x = [&](XSet& s, int i, int j) __attribute__((always_inline)) {  // k block j of the wavefront's chunk i
    const u32x4* x = p.X + (int64_t)min(kb_begin + (wave + MG_NW * i) * KC + j, last) * (TB * 128);
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
      s.x[tb][0] = x[xo[tb]];
      s.x[tb][1] = x[xo[tb] + 64];
    }
  };
  f32x4 acc[R][TB];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) acc[r][tb] = f32x4{0.f, 0.f, 0.f, 0.f};
  // chunk i, in weight set s of the ring; nv: k blocks of it that lie in the range
  auto chunk = [&](int s, int i, int nv) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < KC; ++j) {
      if (j >= nv) break;
      XSet& x = xs[(s * KC + j) % D];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        f16x8 a;
        if constexpr (W8) {
          const u32x4 raw = ws[s].w[r];
          a = j ? fp8x8_to_f16x8(raw.z, raw.w) : fp8x8_to_f16x8(raw.x, raw.y);
        } else {
          a = as_f16x8(ws[s].w[r]);
        }
#pragma unroll
        for (int hl = 0; hl < 2; ++hl)
#pragma unroll
          for (int tb = 0; tb < TB; ++tb) acc[r][tb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, as_f16x8(x.x[tb][hl]), acc[r][tb], 0, 0, 0);
      }
      load_x(x, i + (j + D) / KC, (j + D) % KC);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto valid = [&](int i) __attribute__((always_inline)) { return min(KC, nkb - (wave + MG_NW * i) * KC); };

#pragma unroll
  for (int s = 0; s < D; ++s) {
    load_w(ws[s], s);
    load_x(xs[s], s / KC, s % KC);
  }
  __builtin_amdgcn_sched_barrier(0);
  int i = 0;
  for (; i + 2 * D <= n_w; i += D) {
#pragma unroll
    for (int s = 0; s < D; ++s) {
      chunk(s, i + s, KC);
      load_w(ws[s], i + s + D);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int s = 0; s < D; ++s) {
    if (i + s < n_w) chunk(s, i + s, valid(i + s));
    if (i + s + D < n_w) load_w(ws[s], i + s + D);
  }
#pragma unroll
  for (int s = 0; s < D - 1; ++s)
    if (i + s + D < n_w) chunk(s, i + s + D, valid(i + s + D));

#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) red[wave][r][tb][lane] = acc[r][tb];
  __syncthreads();
  f32x4 v[NT];
#pragma unroll
  for (int q = 0; q < NT; ++q) {  // in wavefront order
    v[q] = red[0][fr][tbase + q * TSTEP][lane];
#pragma unroll
    for (int w = 1; w < MG_NW; ++w) v[q] += red[w][fr][tbase + q * TSTEP][lane];
  }
  // parked as [split][row group][tb][lane]; the workgroup of the tile that comes last adds the splits in order
  const __amdgpu_buffer_rsrc_t prs = shared_rsrc(p.partial);
  auto unit = [&](int sp, int tb) __attribute__((always_inline)) { return (uint32_t)(((sp * p.NRG + frg) * TB + tb) * 64 + lane) * 16u; };
#pragma unroll
  for (int q = 0; q < NT; ++q) store_shared_f32x4(prs, unit(split, tbase + q * TSTEP), v[q]);
  wait_own_memory_ops();
  __syncthreads();
  if (tid == 0) s_last = arrive_last(&p.counters[tile], p.ksplit, p.fence_handover, p.fault_flag);
  __syncthreads();
  if (!s_last) return;
  // the fenced hand-over's other half (acquire side of the producers' release fences)
  if (p.fence_handover) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  if (tid == 0) __hip_atomic_store(&p.counters[tile], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const f32x4 gv = *reinterpret_cast<const f32x4*>(p.gain_next + n0);
  f32x4 hv[NT];
#pragma unroll
  for (int q = 0; q < NT; ++q) {
    hv[q] = *reinterpret_cast<const f32x4*>(p.h + (int64_t)min((tbase + q * TSTEP) * 16 + tsub, p.M - 1) * p.d + n0);
    v[q] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  f32x4 pv[4][NT];
  add_in_order<4>(p.ksplit,
      [&](int u, int sp) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < NT; ++q) pv[u][q] = load_shared_f32x4(prs, unit(sp, tbase + q * TSTEP));
      },
      [&](int u) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < NT; ++q) v[q] += pv[u][q];
      });
#pragma unroll
  for (int q = 0; q < NT; ++q) {
    const int t = (tbase + q * TSTEP) * 16 + tsub;
    float s = 0.f;
    union { uint16_t s[4]; u32x2 v; } hi, lo;
    f32x4 hn;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      hn[e] = hv[q][e] + v[q][e] * p.wfactor;
      s += hn[e] * hn[e];
      split_f16(hn[e] * gv[e], hi.s[e], lo.s[e]);
    }
    s += __shfl_xor(s, 16);
    s += __shfl_xor(s, 32);
    if (t < p.M) {
      *reinterpret_cast<f32x4*>(p.h + (int64_t)t * p.d + n0) = hn;
      *reinterpret_cast<u32x2*>(p.xnext + packed_x_offset(n0, t, TB, 0)) = hi.v;
      *reinterpret_cast<u32x2*>(p.xnext + packed_x_offset(n0, t, TB, 1)) = lo.v;
    }
    if (lane < 16) s_sq[fr][(tbase + q * TSTEP) * 16 + lane] = s;
  }
  __syncthreads();
  if (tid < p.M) {  // one entry per token and tile, its row groups added in order
    float s = s_sq[0][tid];
#pragma unroll
    for (int w = 1; w < R; ++w) s += s_sq[w][tid];
    p.ssq_out[(int64_t)tid * SSQ_TILES + tile] = s;
  }
}

// ------------------------------------------------------------------------------------------------
// Host side
// the kernels there are
static constexpr bool mg_built(int wmode, int R) { return (R == 2 && (wmode == WMODE_F16 || wmode == WMODE_FP8)) || (R == 4 && wmode == WMODE_F16); }
static int mg_wmode(const www_model* m) { return m->wsplit ? WMODE_SPLIT : m->int4_group ? WMODE_INT4 : m->fp8 ? WMODE_FP8 : WMODE_F16; }
bool mid_gemm_built(const www_model* m, const MidShape& s) { return mg_built(mg_wmode(m), s.R); }

static int mid_rows(int NRG) { return NRG > 128 ? 4 : 2; }  // a tile's sums of squares: SSQ_TILES entries up to 4096 columns
static int mid_splits(int tiles) { return tiles ? min(8, decode_wg_target() / tiles) : 0; }

uint64_t mid_gemm_partial_bytes(int NRG) {
  const int R = mid_rows(NRG), tiles = (NRG + R - 1) / R;
  return tiles <= SSQ_TILES ? (uint64_t)NRG * mid_splits(tiles) * MG_TB * 1024 : 0;
}

// A range of k of up to 96 blocks: the activations, twice what skinny_gemm_kernel reads, cost more than the hand-over beyond (4096 rows,
// 64 tokens, us: 64 blocks 24.0 -> 22.8, 88 28.2 -> 27.7, 112 33 -> 35), and eight wavefronts with a chunk each at least.
MidShape mid_gemm_route(const www_model* m, int epi, int NRG, int KB, int M) {
  MidShape s = {0, 0, 0};
  const int R = mid_rows(NRG), tiles = NRG / R, chunk = MG_NW * mg_kc(mg_wmode(m));
  if (epi != EPI_RESID || M <= 32 || M > 64 || NRG % R || !mg_built(mg_wmode(m), R)) return s;
  const int ks = min(mid_splits(tiles), KB / chunk), per = ks > 1 ? ((KB + ks - 1) / ks + 3) / 4 * 4 : 0;
  if (tiles > SSQ_TILES || ks < 2 || per > 96) return s;
  s = {R, (KB + per - 1) / per, per};
  return s;
}

template <int WMODE, int R>
static bool launch_mid_as(const GemmP& p, hipStream_t st) {
  if constexpr (mg_built(WMODE, R))
    hipLaunchKernelGGL((mid_gemm_kernel<WMODE, R>), dim3(8 * ((p.row_tiles + 7) / 8) * p.ksplit), dim3(64 * MG_NW), 0, st, p);
  return mg_built(WMODE, R);
}
bool launch_mid_gemm(www_model* m, GemmP& p, const MidShape& s, hipStream_t st) {
  if (!mid_gemm_built(m, s) || p.NRG % s.R) return false;
  p.ksplit = s.ks;
  p.kb_per_split = s.per;
  p.partial = m->partial;
  p.counters = m->counters;
  p.fault_flag = m->fault_dev;
  p.fence_handover = m->handover_fence;
  if (p.wfactor == 0.f) p.wfactor = 1.f;  // not set: an unscaled matrix
  p.row_tiles = p.NRG / s.R;
  if (m->fp8) return s.R == 2 ? launch_mid_as<WMODE_FP8, 2>(p, st) : launch_mid_as<WMODE_FP8, 4>(p, st);
  return s.R == 2 ? launch_mid_as<WMODE_F16, 2>(p, st) : launch_mid_as<WMODE_F16, 4>(p, st);
}
